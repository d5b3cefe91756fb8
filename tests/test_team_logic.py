"""Host logic of the teams of workgroups (no GPU): the counts by which a launch
whose team did not form orders its bands."""
import os
import shutil
import subprocess

import pytest

from host_lib import host  # noqa: F401

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1606_00310_amd", "csrc")


def test_counts_are_relative_to_the_launch(tmp_path):
    """A band's progress word holds whatever an earlier launch left, or zero:
    neither may count as progress, however many half-steps the context has run
    (a sign test on 32-bit half-step numbers failed past 2^31 of them)."""
    if shutil.which("g++") is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("g++ or the HIP headers not available")
    exe = tmp_path / "team_count"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC,
                           os.path.join(HERE, "helpers", "team_count.cpp"), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout


def test_a_launch_is_bounded(host):
    """A team holds every compute unit for a launch: a long step comes in launches
    of some milliseconds, between which other streams' kernels get in."""
    host("""
c = lattice(16384, 16384)
log()
assert lib.sca_step(c, 5000, 0.5, 0.0) == 0
runs = [dict(w.split("=") for w in l.split() if "=" in w) for l in launches("team_kernel")]
assert [int(r["t"]) for r in runs] == [sum(int(s["n"]) for s in runs[:i]) for i in range(len(runs))]
assert sum(int(r["n"]) for r in runs) == 5000 and max(int(r["n"]) for r in runs) <= 512
assert [int(r["epoch"]) for r in runs] == list(range(1, len(runs) + 1))
""")


def test_teams_are_tried_again(host):
    """After a launch whose team did not form, 256 steps or epochs go without, and
    then one tries again."""
    host("""
c = lattice(16384, 16384)
fake.fake_apart(1)
log()
teams = []
for i in range(600):
    planned = team_planned(c, 64)
    assert lib.sca_step(c, 64, 0.5, 0.0) == 0
    ran = len(launches("team_kernel")) > 0
    assert ran == planned
    if ran:
        teams.append(i)
assert teams == [0, 257, 514]
fake.fake_apart(0)
for i in range(600):
    assert lib.sca_step(c, 64, 0.5, 0.0) == 0
assert 300 < len(launches("team_kernel")) < 600

e = Ensemble([(2048, 2048), (64, 64)], n_mcs=10**6)
fake.fake_apart(1)
log()
teams = []
for i in range(600):
    assert e.run(3) == 0
    if launches("onchip_kernel")[0].endswith("teams"):
        teams.append(i)
assert teams == [0, 257, 514]
fake.fake_apart(0)
for i in range(300):
    assert e.run(3) == 0
assert e.t(0) == 2700 and [l for l in launches("onchip_kernel") if l.endswith("teams")]
""")
