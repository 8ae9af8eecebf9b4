"""Workloads of the library as a user's program runs them, with their inputs, one pass and its results.

``listed()`` names the standing ones, ``draw(rng)`` gives more of the same ranges, ``prepare(case, seed)`` makes
what a program holds before the call (the lattices in their seeded hot start), ``run(state)`` is one call through
the public binding, ``work(case)`` what one pass cannot do without, ``exact(case, seed)`` a double-precision
evaluation of the continuous-spin records.

A case is a dict of plain values: kind (lattice, coarse, batch, msc, heis), model (0 Ising, 1 +-J glass), d, L,
sweeps per call, every (a record of E and M after every so many sweeps; 0: none), beta, and for some kinds host
(records into host arrays), tile and hits (coarse), realisations (batch).
"""
import math

import numpy as np
import torch

from paper_1006_3865_amd import spin, workloads

BATCH_SIZES = (16, 24, 32, 48, 64)  # the lattice sizes of the batched glass workload
BATCH_BETAS = 16


def _lat(name, model, d, L, sweeps, every, beta, **more):
    return dict(name=name, kind="lattice", model=model, d=d, L=L, sweeps=sweeps, every=every, beta=beta, **more)


def listed():
    bc, b3, bg = workloads.BETA_2D_CRIT, workloads.BETA_3D, workloads.ea_betas()[7]
    return [
        # the smallest configured job: 2D Ising at criticality, E and M of every sweep wanted on the host
        _lat("ising2d_L64", 0, 2, 64, 200, 1, bc, host=True),
        # the largest 2D size of the paper's own runs, a record every 10 sweeps
        _lat("ising2d_L1024", 0, 2, 1024, 100, 10, bc),
        # a decimal edge (not a multiple of 16), as sizes are often chosen; equilibration without records
        _lat("ising2d_L1000", 0, 2, 1000, 100, 0, bc),
        # the large 2D lattice of the benchmark: its step of 10 sweeps and one record
        _lat("ising2d_L8192", 0, 2, 8192, 10, 10, bc),
        # a small 3D lattice of the served stream's range, recorded every 10 sweeps
        _lat("ising3d_L64", 0, 3, 64, 100, 10, b3),
        # a decimal 3D edge that is no multiple of 8
        _lat("ising3d_L100", 0, 3, 100, 50, 10, b3),
        # the large 3D lattice of the benchmark: 10 sweeps and one record
        _lat("ising3d_L512", 0, 3, 512, 10, 10, b3),
        # one +-J glass of the served stream's middle range
        _lat("ea3d_L128", 1, 3, 128, 50, 10, bg),
        # the batched glass workload (many realisations x 16 temperatures) at a quarter of its width
        dict(name="batch_ea3d", kind="batch", realisations=128, sweeps=50, every=25),
        # 32 multi-spin-coded realisations of the 3D glass
        dict(name="msc3d_L256", kind="msc", d=3, L=256, sweeps=20, every=10, beta=bg),
        # the paper's own schedule with multi-hit at its size and best tile
        dict(name="coarse2d_L1024", kind="coarse", model=0, d=2, L=1024, sweeps=20, every=10, beta=bc, tile=16, hits=4),
        # continuous spins, mid-size
        dict(name="heis2d_L1024", kind="heis", d=2, L=1024, sweeps=20, every=10, beta=0.7),
    ]


def _edge(rng, lo, hi, ragged=0.25):
    """An edge, log-uniform: mostly a multiple of 8, with chance `ragged` just even."""
    x = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    step = 2 if rng.random() < ragged else 8
    return max(lo, min(hi, int(round(x / step)) * step))


def _sweeps(rng, sites, most):
    """Sweeps of a call, log-uniform in 1..200, and at most `most` attempts in all."""
    return max(1, min(int(most // sites), int(round(math.exp(rng.uniform(0.0, math.log(200.0)))))))


def draw(rng):
    kind = rng.choice(["ising2d", "ising2d", "ising3d", "ising3d", "ea2d", "ea3d", "batch", "msc", "coarse", "heis"])
    if kind in ("ising2d", "ising3d", "ea2d", "ea3d"):
        d = 2 if kind.endswith("2d") else 3
        model = 1 if kind.startswith("ea") else 0
        L = _edge(rng, 16, {"ising2d": 8192, "ising3d": 512, "ea2d": 4096, "ea3d": 256}[kind])
        n = _sweeps(rng, L ** d, 4e8 if L % 8 == 0 else 1e8)
        every = rng.choice([0, 0, 1, 5, 10])
        return dict(kind="lattice", model=model, d=d, L=L, sweeps=n, every=every if every <= n else 0,
                    beta=round(rng.uniform(0.1, 1.0), 3))
    if kind == "batch":
        return dict(kind="batch", realisations=rng.randrange(8, 65), sweeps=rng.randrange(10, 51), every=rng.choice([5, 10]))
    if kind == "msc":
        d = rng.choice([2, 3])
        L = _edge(rng, 32, 2048 if d == 2 else 256, ragged=0.0)
        n = _sweeps(rng, 32 * L ** d, 5e9)
        return dict(kind="msc", d=d, L=L, sweeps=n, every=n, beta=round(rng.uniform(0.5, 3.0), 3))
    if kind == "coarse":
        tile = rng.choice([8, 16, 32, 64])
        half = max(1, int(round(math.exp(rng.uniform(math.log(128.0), math.log(4096.0))) / (2 * tile))))
        hits = rng.choice([1, 2, 4, 8])
        n = _sweeps(rng, hits * (2 * tile * half) ** 2, 4e8)
        return dict(kind="coarse", model=rng.choice([0, 0, 1]), d=2, L=2 * tile * half, sweeps=n, every=n,
                    beta=round(rng.uniform(0.2, 0.6), 3), tile=tile, hits=hits)
    d = rng.choice([2, 3])
    L = _edge(rng, 32, 2048 if d == 2 else 160)
    n = min(20, _sweeps(rng, L ** d, 6e7))
    return dict(kind="heis", d=d, L=L, sweeps=n, every=n, beta=round(rng.uniform(0.3, 2.0), 3))


class _Span:
    """Device memory of the library as an array (spin_device_spins)."""

    def __init__(self, ptr, n):
        self.__cuda_array_interface__ = {"shape": (n,), "typestr": "|i1", "data": (ptr, False), "version": 2}


def _records(case):
    return case["sweeps"] // case["every"] if case.get("every") else 0


def prepare(case, seed):
    kind = case["kind"]
    s = workloads.seed(seed)
    st = dict(case, handle=None, views={}, E=None, M=None)
    if kind in ("lattice", "coarse"):
        glass = case["model"] == spin.SPIN_EA_PMJ
        h = spin.Lattice(case["model"], case["L"], case["d"], s, coupling_seed=s + 1 if glass else None)
        if kind == "coarse":
            h.set_schedule(spin.SPIN_SCHEDULE_COARSE, case["tile"], case["hits"])
        nrec = _records(case)
        if nrec and not case.get("host"):
            st["E"] = torch.zeros(nrec, dtype=torch.int64, device="cuda")
            st["M"] = torch.zeros(nrec, dtype=torch.int64, device="cuda")
    elif kind == "batch":
        descs = workloads.ea_batch(case["realisations"], BATCH_SIZES, rng_seed=0x12)
        for x in descs:
            x.update(seed=s, coupling_seed=s + 1)
        h = spin.Batch(descs)
        st["betas"] = np.array([x["beta"] for x in descs])
        nrec = _records(case) * len(descs)
        st["E"] = torch.zeros(nrec, dtype=torch.int64, device="cuda")
        st["M"] = torch.zeros(nrec, dtype=torch.int64, device="cuda")
    elif kind == "msc":
        h = spin.Msc(case["L"], case["d"], s + 1, 0, s)
    else:
        h = spin.Heis(case["L"], case["d"], s)
    h.synchronize()
    st["handle"] = h
    return st


def run(st):
    h, n, every = st["handle"], st["sweeps"], st.get("every", 0)
    kind = st["kind"]
    if kind == "batch":
        h.sweep_device(n, st["betas"], every, st["E"], st["M"])
        return {"E": st["E"], "M": st["M"]}
    if kind in ("msc", "heis"):
        E, M = h.sweep_record(n, st["beta"], every)
        return {"E": E, "M": M}
    out = {}
    if not every:
        h.sweep(n, st["beta"])
    elif st.get("host"):
        out["E"], out["M"] = h.sweep_record(n, st["beta"], every)
    else:
        h.sweep_record_device(n, st["beta"], every, st["E"], st["M"])
        out["E"], out["M"] = st["E"], st["M"]
    # the lattice as it lies in device memory (the library keeps two buffers at most); the tensor holds the
    # lattice, whose memory it shows
    ptr = spin.spin_device_spins(h.h)
    if ptr not in st["views"]:
        view = torch.as_tensor(_Span(ptr, h.N), device="cuda")
        view.lattice = h
        st["views"][ptr] = view
    out["spins"] = st["views"][ptr]
    return out


def _batch_sites(case):
    return sum(x["L"] ** 3 for x in workloads.ea_batch(case["realisations"], BATCH_SIZES, rng_seed=0x12))


def work(case):
    """Bytes: the spins read and written once, the couplings read once, the records written.  Operations: Philox
    words (10 per four-word block of the byte-coded models' attempts), the neighbour sums and the decisions, per
    attempted update."""
    kind = case["kind"]
    rec = 16 * _records(case)
    if kind == "batch":
        N = _batch_sites(case)
        return {"bytes": (2 + 3 / 8) * N + rec * BATCH_BETAS * case["realisations"], "flops": 17.75 * N * case["sweeps"]}
    N = case["L"] ** case["d"]
    if kind == "msc":
        return {"bytes": (8 + 4 * case["d"]) * N + 32 * rec, "flops": 1.7 * 32 * N * case["sweeps"]}
    if kind == "heis":
        return {"bytes": 32 * N + rec, "flops": 120.0 * N * case["sweeps"]}
    hits = case.get("hits", 1)
    couplings = case["d"] * N / 8 if case["model"] else 0
    ops = 16.5 if case["d"] == 2 else 17.75
    return {"bytes": 2 * N + couplings + rec, "flops": ops * N * hits * case["sweeps"]}


# ------------------------------------------------------------- the Heisenberg records in double precision

_MASK = 0xFFFFFFFF


def _mulhilo(m, x):
    """(high, low) 32 bits of m * x for 32-bit values held in int64 (m < 2^32): the product of 16-bit halves."""
    lo = m * (x & 0xFFFF)
    hi = m * (x >> 16) + (lo >> 16)
    return hi >> 16, ((hi & 0xFFFF) << 16) | (lo & 0xFFFF)


def _philox(c0, c1, c2, c3, seed):
    """Words 0..2 of Philox4x32-10 (Salmon et al., SC'11) for counters c0 (int64 tensor) and scalars c1..c3."""
    c = [c0, torch.full_like(c0, c1), torch.full_like(c0, c2), torch.full_like(c0, c3)]
    k0, k1 = seed & _MASK, (seed >> 32) & _MASK
    for _ in range(10):
        h0, l0 = _mulhilo(0xD2511F53, c[0])
        h1, l1 = _mulhilo(0xCD9E8D57, c[2])
        c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & _MASK, (k1 + 0xBB67AE85) & _MASK
    return c[0], c[1], c[2]


def _uniform(w):
    return (w >> 8).to(torch.float64) * 2.0 ** -24


def _direction(w0, w1):
    z = 2.0 * _uniform(w0) - 1.0
    phi = 2.0 * math.pi * _uniform(w1)
    rho = torch.sqrt(torch.clamp(1.0 - z * z, min=0.0))
    return torch.stack([rho * torch.cos(phi), rho * torch.sin(phi), z])


def exact(case, seed):
    """The Heisenberg records from a double-precision run of the stated chain (single trial decisions can differ
    from float arithmetic's where the draw falls on the edge); None for the integer-valued kinds."""
    if case["kind"] != "heis":
        return None
    d, L, key = case["d"], case["L"], workloads.seed(seed)
    N = L ** d
    if N * case["sweeps"] > 7e7:
        return None
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    site = torch.arange(N, dtype=torch.int64, device=dev)
    parity = sum((site // L ** k) % L for k in range(d)) % 2
    w0, w1, _ = _philox(site, 0, 0, 9, key)
    S = _direction(w0, w1).reshape([3] + [L] * d)
    axes = list(range(d, 0, -1))  # x is the last axis
    beta = float(np.float32(case["beta"]))
    E, M = [], []
    for t in range(case["sweeps"]):
        for c in range(2):
            h = sum(torch.roll(S, 1, ax) + torch.roll(S, -1, ax) for ax in axes)
            w0, w1, w2 = _philox(site, t, 0, 10 + c, key)
            trial = _direction(w0, w1).reshape(S.shape)
            dE = ((S - trial) * h).sum(0).reshape(-1)
            take = (parity == c) & ((dE <= 0) | (_uniform(w2) < torch.exp(-beta * torch.clamp(dE, min=0.0))))
            S = torch.where(take.reshape([1] + [L] * d), trial, S)
        if (t + 1) % case["every"] == 0:
            E.append(-sum(float((S * torch.roll(S, -1, ax)).sum()) for ax in axes))
            M.append(float(S.reshape(3, -1).sum(1).norm()))
    return {"E": np.array(E), "M": np.array(M)}
