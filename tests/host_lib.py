"""Runs code against libsca.so on a HIP runtime without a GPU (helpers/fake_hip.cpp),
in a process of its own: no kernel runs, and a log tells what was enqueued."""
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(os.path.dirname(HERE), "paper_1606_00310_amd")

PRELUDE = r"""
import ctypes, importlib.util, sys, types
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)  # ahead of the library: its references bind here
fake.fake_log.restype = ctypes.c_char_p
fake.fake_fail_malloc.argtypes = [ctypes.c_size_t]
sys.modules["torch"] = types.ModuleType("torch")          # the binding loads it for the real runtime only
spec = importlib.util.spec_from_file_location("binding", sys.argv[2] + "/_lib.py")
L = importlib.util.module_from_spec(spec)
spec.loader.exec_module(L)
lib = L.lib()

def log():
    out = fake.fake_log().decode().splitlines()
    fake.fake_reset_log()
    return out

def launches(name, lines=None):
    return [l for l in (log() if lines is None else lines) if l.startswith("launch") and name in l]

def lattice(X, Y):
    c = ctypes.c_void_p()
    assert lib.sca_init(ctypes.byref(c), X, Y, 1, 1 << 40, 1 << 41, None) == 0
    assert lib.sca_set_pass_buffer(c, 1 << 42, 1 << 36) == 0
    return c

def team_planned(c, n, p=0.5, q=0.0):
    out = L.StepPlan()
    assert lib.sca_plan_step(c, n, p, q, 0, ctypes.byref(out)) == 0
    return out.kernel.startswith(b"team_kernel")

class Ensemble:
    def __init__(self, sizes, n_mcs=1000, p=0.5, **config):
        self.b = ctypes.c_void_p()
        assert lib.sca_batch_create(ctypes.byref(self.b), len(sizes), 1 << 40, 1 << 40, None) == 0
        if config:
            c = L.BatchConfig()
            assert lib.sca_batch_get_config(self.b, ctypes.byref(c)) == 0
            for k, v in config.items():
                setattr(c, k, v)
            assert lib.sca_batch_set_config(self.b, ctypes.byref(c)) == 0
        self.slots = (ctypes.c_int32 * len(sizes))()
        reqs = (L.Req * len(sizes))(*[L.Req(X, Y, p, 0.0, n_mcs, i, 0, 0) for i, (X, Y) in enumerate(sizes)])
        assert lib.sca_batch_admit(self.b, reqs, len(sizes), self.slots) == 0
    def run(self, n):
        self.active = ctypes.c_int32(-1)
        return lib.sca_batch_run(self.b, n, ctypes.byref(self.active))
    def t(self, i):
        s = L.SlotInfo()
        assert lib.sca_batch_slot(self.b, self.slots[i], ctypes.byref(s)) == 0
        return s.t
"""


@pytest.fixture(scope="session")
def host(tmp_path_factory):
    """host(code): runs it behind PRELUDE; fails with its output."""
    if shutil.which("g++") is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("g++ or the HIP headers not available")
    lib = os.path.join(PKG, "libsca.so")
    if not os.path.exists(lib):
        from paper_1606_00310_amd import build

        build.build()
    so = tmp_path_factory.mktemp("hip") / "fake_hip.so"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-w", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__",
                           "-I/opt/rocm/include", "-I", os.path.join(PKG, "csrc"),
                           os.path.join(HERE, "helpers", "fake_hip.cpp"), "-o", str(so)])

    def run(code):
        r = subprocess.run([sys.executable, "-c", PRELUDE + code, str(so), PKG], capture_output=True, text=True,
                           timeout=120)
        assert r.returncode == 0, r.stdout + r.stderr

    return run
