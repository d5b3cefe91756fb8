"""Timing cases of the lattice, measurement, ensemble and serving entry points.

Each case is a dict of plain values of one of three kinds:

  steps    one lattice advanced by n_mcs MCS in one call, as in the middle of
           a growth run, with the exact moments, the two-time sums against an
           earlier snapshot, or nothing measured afterwards
  measure  the exact moments, the two-time sums and all heights of a given
           rough surface (no step)
  reals    an ensemble of independent lattices of uneven size: admitted, run
           to the end of every MCS budget and collected, either directly in
           one epoch per call or through the continuous-batching server

`prepare` builds what a program holds before the call, `run` is one pass.
"""
from __future__ import annotations

import math
import random

import torch

import paper_1606_00310_amd as sca
from paper_1606_00310_amd import batch, serve

# The launch shape that tuning picks for large ensembles; the server case
# keeps the library's default one.
TUNED = dict(block_threads=1024, blocks_per_cu=1, lds_bytes=65536, order=0, words_per_lane=1, depth=2, max_parts=4)


def _steps(name, X, Y, p, q, n_mcs, after="none", warm=16):
    return {"name": name, "kind": "steps", "X": X, "Y": Y, "p": p, "q": q, "n_mcs": n_mcs, "after": after,
            "warm": warm}


def listed():
    return [
        # the validation run: moments after every single MCS
        _steps("mcs-128", 128, 128, 0.5, 0.0, 1, after="moments"),
        # the same lattice for its whole 1000 MCS
        _steps("run-128", 128, 128, 0.5, 0.0, 1000),
        # a mid-sized, non-square lattice between two measurements, odd number of MCS
        _steps("run-1024x512", 1024, 512, 0.5, 0.0, 37, after="moments"),
        # deposition and removal at 2^12 squared, between two of its log-spaced measurement times
        _steps("medium-4096", 4096, 4096, 0.75, 0.25, 100, after="moments"),
        # the p = 1/2 throughput workload at a quarter of its lateral size
        _steps("half-16384", 16384, 16384, 0.5, 0.0, 64),
        # the four-digit mask at the full lateral size, a number of MCS that leaves remainder passes
        _steps("random-65536", 65536, 65536, 0.9375, 0.0, 21),
        # the headline sweep, no random words
        _steps("headline-65536", 65536, 65536, 1.0, 0.0, 104),
        # arbitrary probabilities: a small surface at p = 0.95 ...
        _steps("persite-1024", 1024, 1024, 0.95, 0.0, 20, after="moments", warm=64),
        # ... and the aging run with its two-time function
        _steps("persite-16384", 16384, 16384, 0.93, 0.07, 10, after="autocorr", warm=64),
        # every measurement of one large surface
        {"name": "measure-8192", "kind": "measure", "X": 8192, "Y": 8192},
        # an uneven ensemble in one epoch
        {"name": "ensemble-512", "kind": "reals", "n": 512, "l_min": 6, "l_max": 11, "mcs_min": 20, "mcs_max": 500,
         "q": 0.0, "serve": False},
        # small requests through the server, each collected with its moments and state
        {"name": "serve-96", "kind": "reals", "n": 96, "l_min": 6, "l_max": 9, "mcs_min": 20, "mcs_max": 200,
         "q": 0.0, "serve": True},
    ]


def draw(rng: random.Random):
    kind = rng.choices(["steps", "persite", "measure", "reals"], [5, 2, 2, 2])[0]
    if kind in ("steps", "persite"):
        while True:
            lx, ly = rng.randint(5, 16), rng.randint(5, 16)
            # from square to strips, none longer than 2^8 times its width
            if abs(lx - ly) <= 8 and (kind == "steps" or lx + ly <= 28):
                break
        sites = 2.0 ** (lx + ly)
        # at most about a hundred MCS of the largest lattice, 1000 of a small one
        most = min(1000.0, max(1.0, (6e10 if kind == "steps" else 2.6e9) / sites))
        n_mcs = max(1, int(round(math.exp(rng.uniform(0.0, math.log(most + 1e-9))))))
        if kind == "steps":
            p, q = rng.choice([(0.5, 0.0), (0.5, 0.0), (1.0, 0.0), (0.75, 0.25), (0.9375, 0.0), (0.5, 0.5),
                               (0.625, 0.125), (1.0, 1.0)])
        else:
            p, q = rng.choice([(0.95, 0.0), (0.93, 0.07), (round(rng.uniform(0.05, 0.99), 3), 0.0), (0.3, 0.3)])
        c = _steps(None, 1 << lx, 1 << ly, p, q, n_mcs, after=rng.choice(["none", "none", "moments", "autocorr"]),
                   warm=64 if kind == "persite" else 16)
        del c["name"]
        return c
    if kind == "measure":
        lx, ly = rng.randint(6, 14), rng.randint(6, 13)
        return {"kind": "measure", "X": 1 << lx, "Y": 1 << ly}
    server = rng.random() < 0.5
    l_min = rng.randint(5, 8)
    l_max = rng.randint(l_min, 9 if server else 11)
    n = int(round(math.exp(rng.uniform(math.log(8), math.log(96 if server else 512)))))
    mcs_min = rng.randint(5, 40)
    return {"kind": "reals", "n": n, "l_min": l_min, "l_max": l_max, "mcs_min": mcs_min,
            "mcs_max": mcs_min + rng.randint(1, 160 if server else 400), "q": rng.choice([0.0, 0.0, 0.25]),
            "serve": server}


# ------------------------------------------------------------------ inputs
def _surface(X, Y, seed, rounds=8):
    """A rough periodic surface on the GPU: explicit heights h[y, x] (int32),
    |h(site) - h(neighbour)| = 1, h = x + y mod 2.  Random bridges along x and
    y, then some random lifts of minima and drops of maxima, one sublattice at
    a time."""
    g = torch.Generator(device="cuda").manual_seed(seed)

    def bridge(n):
        e = torch.ones(n, dtype=torch.int32, device="cuda")
        e[torch.randperm(n, generator=g, device="cuda")[: n // 2]] = -1
        return torch.cumsum(e, 0, dtype=torch.int32) - e[0]  # starts at 0, period n

    h = bridge(Y)[:, None] + bridge(X)[None, :]
    yy = torch.arange(Y, device="cuda")[:, None]
    xx = torch.arange(X, device="cuda")[None, :]
    odd = ((xx + yy) & 1).bool()
    for _ in range(rounds):
        for on in (~odd, odd):
            s = torch.zeros_like(h)
            for shift, dim in ((1, 0), (-1, 0), (1, 1), (-1, 1)):
                s += torch.roll(h, shift, dim) - h
            hit = on & (torch.rand((Y, X), generator=g, device="cuda") < 0.75)
            h += 2 * (hit & (s == 4)).int() - 2 * (hit & (s == -4)).int()
            del s, hit
    return h


def _pack(h):
    """The packed state (slopes, then h(0,0)) of explicit heights."""
    Y, X = h.shape
    W, nb = max(1, X // 128), min(64, X // 2)
    bit = torch.tensor([(1 << k) - (1 << 64) if k == 63 else 1 << k for k in range(nb)], device="cuda")
    out = torch.empty(4 * Y * W + 1, dtype=torch.int64, device="cuda")
    S = out[:-1].view(2, 2, Y, W)
    for d, dim in ((0, 1), (1, 0)):
        up = ((h - torch.roll(h, 1, dim)) == 1).view(Y, X // 2, 2)
        for parity in (0, 1):
            for r in (0, 1):  # rows y = r mod 2 hold their sites of this parity at x = 2k + (parity ^ r)
                b = up[r::2, :, parity ^ r].reshape(-1, W, nb)
                for y0 in range(0, b.shape[0], 1024):
                    S[d, parity, r::2][y0:y0 + 1024] = (b[y0:y0 + 1024] * bit).sum(-1)
    out[-1] = h[0, 0]
    return out


def _realizations(case, seed):
    """Sizes, probabilities and budgets spread over the case's ranges (the
    same for every seed), in an order and with generator seeds of their own."""
    n, sizes, ps = case["n"], case["l_max"] - case["l_min"] + 1, (0.5, 0.75, 0.9375)
    lo, hi = math.log(case["mcs_min"]), math.log(case["mcs_max"])
    rng = random.Random(seed)
    out = []
    for i in range(n):
        L = 1 << (case["l_min"] + i % sizes)
        u = ((i * 0.6180339887498949) % 1.0)
        out.append((L, ps[(i // sizes) % 3], int(round(math.exp(lo + u * (hi - lo))))))
    rng.shuffle(out)
    return [batch.Realization(L, L, p, case["q"], m, rng.getrandbits(40)) for L, p, m in out]


def prepare(case, seed):
    if case["kind"] == "steps":
        lat = sca.Lattice(case["X"], case["Y"], seed=seed)
        # the surface the pass starts from: grown by the same rule, or at
        # p = 1/2 where the rule itself draws no random words
        draws = case["p"] not in (0.0, 1.0) or case["q"] not in (0.0, 1.0)
        lat.step(case["warm"], case["p"] if draws else 0.5, case["q"] if draws else 0.0)
        snap = lat.snapshot() if case["after"] == "autocorr" else None
        return {"case": case, "lat": lat, "snap": snap}
    if case["kind"] == "measure":
        lat = sca.Lattice(case["X"], case["Y"], seed=seed)
        earlier = _pack(_surface(case["X"], case["Y"], 2 * seed))
        lat.restore(_pack(_surface(case["X"], case["Y"], 2 * seed + 1)), 100)
        torch.cuda.synchronize()
        return {"case": case, "lat": lat, "snap": earlier}
    reals = _realizations(case, seed)
    b = batch.Batch(max_slots=len(reals), arena_bytes=sum(batch.state_bytes(r.X, r.Y) for r in reals),
                    config=None if case["serve"] else TUNED)
    return {"case": case, "reals": reals, "batch": b}


def run(state):
    case = state["case"]
    if case["kind"] == "steps":
        lat = state["lat"]
        lat.step(case["n_mcs"], case["p"], case["q"])
        out = {"slopes": lat.slopes, "h0": lat.aux[:1]}
        if case["after"] == "moments":
            out["moments"] = lat.roughness()
        elif case["after"] == "autocorr":
            out["autocorr"] = lat.autocorr(state["snap"])
        return out
    if case["kind"] == "measure":
        lat = state["lat"]
        return {"moments": lat.roughness(), "autocorr": lat.autocorr(state["snap"]), "heights": lat.heights()}
    b, reals = state["batch"], state["reals"]
    if not case["serve"]:
        slots = b.admit(reals)
        while b.run(case["mcs_max"]):
            pass
        parts = []
        for s in slots:
            S, h0 = b.state(s)
            parts += [S.reshape(-1), h0]
        out = torch.cat(parts)
        for s in slots:
            b.release(s)
        return {"states": out}
    srv = serve.Server(serve.BatchBackend(b), work_quota=100 * 2048 * 2048)
    for i in range(0, len(reals), 2):
        srv.submit(serve.Request(i // 2, reals[i:i + 2]))
    while srv.queue or srv.running:
        srv.step()
    done = sorted(srv.completed, key=lambda r: r.rid)
    results = [x for r in done for x in r.results]
    return {"slopes": torch.cat([x["slopes"].reshape(-1) for x in results]),
            "h0": torch.tensor([x["h0"] for x in results]),
            "sums": torch.tensor([x["moments"][:3] for x in results]),
            "w2": torch.tensor([x["moments"][3] for x in results], dtype=torch.float64)}


def _step_ops(sites, n_mcs, p, q):
    """32-bit integer operations that n_mcs MCS cannot do without: ten of the
    rule and the fold of the draws per 64-site word and half-step, and some 36
    per Philox call (four 32-bit words)."""
    words = sites / 64.0  # word updates per MCS, both half-steps together
    digits = 0
    while digits <= 32 and (p * 2 ** digits != int(p * 2 ** digits) or q * 2 ** digits != int(q * 2 ** digits)):
        digits += 1
    if digits > 32:
        # one 32-bit uniform for each site that can move, one in eight
        return n_mcs * words * (10 + 2 * 36 + 2 * 64)
    return n_mcs * words * (10 + digits * (2 + 36 / 2))


def work(case):
    if case["kind"] == "steps":
        sites = float(case["X"]) * case["Y"]
        extra = {"none": 0.0, "moments": sites / 8, "autocorr": sites / 4}[case["after"]]
        return {"bytes": sites / 2 + extra, "flops": _step_ops(sites, case["n_mcs"], case["p"], case["q"])}
    if case["kind"] == "measure":
        sites = float(case["X"]) * case["Y"]
        # x-slopes of the surface and of the snapshot, and four bytes per height
        return {"bytes": sites / 4 + 4 * sites, "flops": 3 * sites}
    nbytes = ops = 0.0
    for r in _realizations(case, 0):
        nbytes += r.sites / 4.0 * (3 if case["serve"] else 2)
        ops += _step_ops(r.sites, r.n_mcs, r.p, r.q)
    return {"bytes": nbytes, "flops": ops}


def exact(case, seed):
    """The measurements from explicit heights; the other cases return packed
    bits and whole numbers, which have one right value."""
    if case["kind"] != "measure":
        return None
    X, Y = case["X"], case["Y"]
    hs = _surface(X, Y, 2 * seed).long()
    ht = _surface(X, Y, 2 * seed + 1).long()
    n = X * Y
    s1, s2, ss, ts = int(ht.sum()), int((ht * ht).sum()), int(hs.sum()), int((ht * hs).sum())
    return {"moments": (n, s1, s2, (n * s2 - s1 * s1) / (n * n)),
            "autocorr": (n, ts, s1, ss, (n * ts - s1 * ss) / (n * n)),
            "heights": ht.int()}
