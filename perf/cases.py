"""Performance cases of the RSOS deposition sweep.

Each case is one kind of work that a program using this package has it do,
through the public entry points (Surface, Batch, MultiSurface and the serving
Engine): whole calls on surfaces that start flat, as every run of the paper
does (Sec. II), and go on growing from call to call.

  listed()        the cases, smallest to largest
  draw(rng)       another case of the same ranges
  prepare(case, seed), run(state)   what the program keeps, and one pass
  exact(case, seed)   the first pass in plain numpy, with 64-bit integers
  work(case)      bytes and operations that a pass cannot do without
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1605_02620_amd import serve
from paper_1605_02620_amd.surface import Batch, MultiSurface, Surface

# Integer operations of one attempted deposition: the site's place in its
# tile (2), the least of the four neighbours (3), the limit and the new height
# (3), and a twentieth of a Philox block (10 rounds of 2 products and 4
# exclusive-ors, 20 site numbers at D = 8).
OPS_PER_ATTEMPT = 11
LOG_CAP = 4096
EXACT_ATTEMPTS = 6e7  # sweeps of more attempts than this are not recomputed in numpy


def listed():
    return [
        # the smallest surface that is studied for its width at all times
        # (L = 64, W^2 read over the first thousand sweeps), a stretch of it
        {"name": "small_L64", "kind": "surface", "L": 64, "N": 1, "D": 8, "sweeps": 64,
         "packed": False, "schedule": "checkerboard"},
        # a sample of the height distribution of a grown surface (the
        # skewness and kurtosis of Sec. III.B)
        {"name": "moments_L4096", "kind": "moments", "L": 4096, "N": 1, "D": 8, "packed": False},
        # one surface of ordinary size, read every few sweeps
        {"name": "single_L1024", "kind": "surface", "L": 1024, "N": 1, "D": 8, "sweeps": 32,
         "packed": False, "schedule": "checkerboard"},
        # a lattice side that is no power of two: 170 x 170 tiles
        {"name": "ragged_L1360_N2", "kind": "surface", "L": 1360, "N": 2, "D": 8, "sweeps": 16,
         "packed": False, "schedule": "checkerboard"},
        # steady-state finite-size scaling: many realizations of small sizes
        {"name": "steady_batch", "kind": "batch", "sizes": "32,64,128,256", "each": 64, "N": 1, "D": 8,
         "sweeps": 32},
        # the independent realizations of the growth regime
        {"name": "ensemble_batch", "kind": "batch", "sizes": "256,512,1024,2048", "each": 16, "N": 1, "D": 8,
         "sweeps": 16},
        # groups of 128 realizations in lock-step (multisurface coding)
        {"name": "lockstep_L256", "kind": "lockstep", "L": 256, "N": 1, "groups": 8, "sweeps": 16},
        # jobs of mixed sizes and restrictions through the serving engine
        {"name": "served_jobs", "kind": "served", "jobs": 24, "L_lo": 128, "L_hi": 2048, "t_lo": 16, "t_hi": 64},
        # a steeper restriction on a large surface
        {"name": "steps_L8192_N4", "kind": "surface", "L": 8192, "N": 4, "D": 8, "sweeps": 8,
         "packed": False, "schedule": "checkerboard"},
        # the paper's own double-tiling schedule
        {"name": "double_L8192", "kind": "surface", "L": 8192, "N": 1, "D": 8, "sweeps": 8,
         "packed": False, "schedule": "double"},
        # the largest single surface, with 16-bit storage and with int32 heights
        {"name": "packed_L16384", "kind": "surface", "L": 16384, "N": 1, "D": 8, "sweeps": 16,
         "packed": True, "schedule": "checkerboard"},
        {"name": "single_L16384", "kind": "surface", "L": 16384, "N": 1, "D": 8, "sweeps": 16,
         "packed": False, "schedule": "checkerboard"},
    ]


def _side(rng, lo, hi, step):
    """A lattice side, a multiple of step, its logarithm uniform; one in two
    is rounded to a power of two, the others fall where they fall."""
    L = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    if rng.random() < 0.5:
        L = 2 ** round(math.log2(L))
    return max(2 * step, int(round(L / step)) * step)


def draw(rng):
    kind = rng.choice(["surface", "surface", "surface", "surface", "moments", "batch", "batch", "lockstep", "served"])
    if kind == "surface":
        packed = rng.random() < 0.25
        double = not packed and rng.random() < 0.2
        D = rng.choice([8, 16]) if double else rng.choice([4, 8, 8, 8, 8, 16])
        L = _side(rng, 256 if packed else 32, 8192, 128 if packed else 2 * D)
        N = rng.choice([1, 1, 2, 3]) if packed else rng.choice([1, 1, 2, 3, 4, 5, 7])
        sweeps = 2 * max(2, min(32, int(2.0e9 / L ** 2 / 2) or 2))
        return {"kind": kind, "L": L, "N": N, "D": D, "sweeps": min(sweeps, rng.choice([4, 8, 16, 32, 64])),
                "packed": packed, "schedule": "double" if double else "checkerboard"}
    if kind == "moments":
        return {"kind": kind, "L": _side(rng, 256, 4096, 128), "N": rng.choice([1, 2, 4]), "D": 8,
                "packed": rng.random() < 0.3}
    if kind == "batch":
        lo = rng.choice([32, 128, 256])
        sizes = sorted({_side(rng, lo, 8 * lo, 16) for _ in range(rng.randint(1, 4))})
        sites = sum(L * L for L in sizes)
        each = max(2, min(rng.choice([8, 16, 32, 64]), int(6e7 / sites)))
        return {"kind": kind, "sizes": ",".join(str(L) for L in sizes), "each": each, "N": rng.choice([1, 1, 2, 4]),
                "D": 8, "sweeps": rng.choice([8, 16, 32])}
    if kind == "lockstep":
        L = _side(rng, 32, 512, 16)
        return {"kind": kind, "L": L, "N": rng.choice([1, 1, 2, 4, 7, 12]),
                "groups": max(1, min(rng.choice([1, 2, 4, 8]), int(6e5 / L ** 2))), "sweeps": rng.choice([8, 16, 32])}
    return {"kind": "served", "jobs": rng.randint(4, 32), "L_lo": 2 ** rng.choice([6, 7]),
            "L_hi": 2 ** rng.choice([9, 10, 11]), "t_lo": rng.choice([16, 32]), "t_hi": rng.choice([48, 80])}


# --------------------------------------------------------------------------
# what the program has in hand
# --------------------------------------------------------------------------
def _batch_specs(case, seed):
    sizes = [int(L) for L in case["sizes"].split(",")]
    return [(L, case["N"], 1000003 * seed + k) for L in sizes for k in range(case["each"])]


def _jobs(case, seed):
    """Sizes, restrictions, lengths and seeds of the served jobs: powers of
    two, N of 1, 2, 4 and log-uniform lengths, as in a request stream.  The
    mix is the case's own; the seeds come from `seed`."""
    rng = np.random.default_rng(16)
    lo, hi = int(math.log2(case["L_lo"])), int(math.log2(case["L_hi"]))
    out = []
    for k in range(case["jobs"]):
        L = 1 << int(rng.integers(lo, hi + 1))
        N = int(rng.choice([1, 2, 4]))
        t = int(round(math.exp(rng.uniform(math.log(case["t_lo"]), math.log(case["t_hi"])))))
        out.append((L, N, t, 1000003 * seed + k))
    return out


def _grid(t_max):
    return sorted({1 << k for k in range(20) if (1 << k) <= t_max} | {t_max})


def _hills(L, N, seed):
    """A surface with the spread of a grown one: random plane waves cut to
    the restriction by scaling their steps."""
    rng = np.random.default_rng(seed)
    x = np.arange(L) * (2 * np.pi / L)
    h = np.zeros((L, L))
    for _ in range(6):
        k, l = (int(v) for v in rng.integers(1, 5, size=2))
        a, b = rng.uniform(0, 2 * np.pi, size=2)
        h += rng.uniform(0.5, 2.0) * np.sin(k * x + a)[None, :] * np.sin(l * x + b)[:, None]
    step = max(np.abs(np.diff(h, axis=0, append=h[:1])).max(), np.abs(np.diff(h, axis=1, append=h[:, :1])).max())
    h *= min(1.0, 0.5 * N / step)
    h = np.floor(h + rng.uniform(0.0, 0.5) + 100)
    return np.ascontiguousarray(h.reshape(-1).astype(np.int32))


def prepare(case, seed):
    kind = case["kind"]
    stream = torch.cuda.Stream()
    if kind == "surface":
        s = Surface(case["L"], N=case["N"], seed=seed, D=case["D"], log_cap=LOG_CAP, stream=stream,
                    packed=case["packed"], schedule=case["schedule"])
    elif kind == "moments":
        s = Surface(case["L"], N=case["N"], seed=seed, D=case["D"], h0=_hills(case["L"], case["N"], seed),
                    log_cap=LOG_CAP, stream=stream, packed=case["packed"])
    elif kind == "batch":
        s = Batch(_batch_specs(case, seed), D=case["D"], log_cap=LOG_CAP, stream=stream)
    elif kind == "lockstep":
        s = MultiSurface(case["L"], N=case["N"], seed=1000003 * seed, groups=case["groups"], log_cap=256, stream=stream)
    else:
        s = (serve.Engine(pool_bytes=1 << 30, max_running=64, D=8), _jobs(case, seed))
    return {"case": case, "obj": s, "t": 0}


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------
def _fields(w):
    return {"t": w["t"], "s1": w["s1"], "s2": w["s2"], "accepted": w["accepted"], "w2": w["w2"]}


def run(state):
    case, s = state["case"], state["obj"]
    kind = case["kind"]
    if kind == "moments":
        # the power sums fit 64 bits on these surfaces
        return dict(s.moments())
    if kind == "served":
        engine, jobs = s
        ids = [engine.submit(L, N, sd, t, _grid(t)) for (L, N, t, sd) in jobs]
        while engine.stats()["finished"] < state["t"] + len(jobs):
            engine.step(64)
        state["t"] += len(jobs)
        rec = np.concatenate([engine.result(i)[0] for i in ids])
        for i in ids:
            engine.release(i)
        return _fields(rec)
    n = case["sweeps"]
    s.sweep(n)
    state["t"] += n
    if kind == "surface":
        out = _fields(s.log(state["t"] - n + 1, n))
        out["heights"] = s.heights_tensor()
        return out
    out = _fields(s.width())
    # the heights of an even time are in the first pool
    out["heights"] = s.lat if kind == "lockstep" else (s.pool if state["t"] % 2 == 0 else s.work)
    return out


# --------------------------------------------------------------------------
# bytes and operations
# --------------------------------------------------------------------------
def _surfaces(case):
    """(L, sweeps) of every surface that a pass advances."""
    kind = case["kind"]
    if kind == "surface":
        return [(case["L"], case["sweeps"])]
    if kind == "batch":
        return [(int(L), case["sweeps"]) for L in case["sizes"].split(",") for _ in range(case["each"])]
    if kind == "lockstep":
        return [(case["L"], case["sweeps"])] * (128 * case["groups"])
    if kind == "served":
        return [(L, t) for (L, N, t, sd) in _jobs(case, 0)]
    return [(case["L"], 0)]


def work(case):
    """The heights are read and written once a pass (they are only read for
    the moments, only born for served jobs), the record of every sweep is
    written; every attempt is made."""
    cell = 2 if case.get("packed") or case["kind"] == "lockstep" else 4
    sf = _surfaces(case)
    sites = sum(L * L for L, n in sf)
    if case["kind"] == "moments":
        return {"bytes": cell * sites, "flops": 7 * sites}
    moves = 1 if case["kind"] == "served" else 2
    return {"bytes": moves * cell * sites + 24 * sum(n for L, n in sf),
            "flops": OPS_PER_ATTEMPT * sum(L * L * n for L, n in sf)}


# --------------------------------------------------------------------------
# the same in plain numpy
# --------------------------------------------------------------------------
def _philox(c0, c1, c2, c3, key):
    """Philox4x32-10 (Salmon et al., SC'11) on arrays of counters."""
    m32 = np.uint64(0xFFFFFFFF)
    c = [np.asarray(v, dtype=np.uint64) for v in np.broadcast_arrays(c0, c1, c2, c3)]
    k0, k1 = key & 0xFFFFFFFF, (key >> 32) & 0xFFFFFFFF
    for _ in range(10):
        a, b = c[0] * np.uint64(0xD2511F53), c[2] * np.uint64(0xCD9E8D57)
        c = [(b >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), b & m32,
             (a >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), a & m32]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c


def _sites(D, count, tile, s, p, key):
    """The first `count` in-tile sites of every tile, one row per draw."""
    b = 2 * int(math.log2(D))
    per, out, j = 32 // b, [], 0
    while len(out) < count:
        for w in _philox(j, tile, s, p, key):
            out += [((w >> np.uint64(b * k)) & np.uint64(D * D - 1)).astype(np.int64) for k in range(per)]
        j += 1
    return out[:count]


def _grow(L, N, D, seed, sweeps, schedule="checkerboard", reals=0):
    """Heights and (s1, s2, accepted) of every sweep from a flat start; with
    `reals`, of that many realizations in lock-step."""
    seed &= 2 ** 64 - 1
    T = L // D
    h = np.zeros((max(reals, 1), L * L), dtype=np.int64)
    row = np.arange(h.shape[0])[:, None]
    logs = []
    ty, tx = (v.reshape(-1) for v in np.mgrid[0:T, 0:T])
    kind = (tx % 2) + 2 * (ty % 2) if schedule == "double" else (tx + ty) % 2
    codes = [(k, 4 + k) for k in range(4)] if schedule == "double" else [(0, 0), (1, 1)]
    for s in range(sweeps):
        ox, oy = (int(w) % (2 * D) for w in _philox(0, 0, s, 2, seed)[:2])
        acc = np.zeros(h.shape[0], dtype=np.int64)
        for k, p in codes:
            mx, my = tx[kind == k], ty[kind == k]
            tile = my * T + mx
            draws = _sites(D, 2 * D * D if reals else D * D, tile, s, p, seed)
            if reals:
                coins = _philox(0, tile[None, :], s, 8 + 2 * row + p, seed)
            for a, f in enumerate(draws):
                x, y = (ox + mx * D + f % D) % L, (oy + my * D + f // D) % L
                i = y * L + x
                c = h[:, i]
                low = np.minimum(np.minimum(h[:, y * L + (x + 1) % L], h[:, y * L + (x - 1) % L]),
                                 np.minimum(h[:, (y + 1) % L * L + x], h[:, (y - 1) % L * L + x]))
                ok = c + 1 - low <= N
                if reals:
                    ok &= ((coins[a // 32] >> np.uint64(a % 32)) & np.uint64(1)).astype(bool)
                h[:, i] = c + ok
                acc += ok.sum(axis=1)
        logs.append((h.sum(axis=1), (h * h).sum(axis=1), acc))
    return h, logs


def _w2(L, s1, s2):
    return np.array([(L * L * int(b) - int(a) ** 2) / L ** 4 for a, b in zip(s1, s2)])


def _out(t, s1, s2, acc, w2, heights):
    return {"t": np.asarray(t, dtype=np.int64), "s1": s1, "s2": s2, "accepted": acc, "w2": w2, "heights": heights}


def exact(case, seed):
    """The first pass on prepare(case, seed), laid out as run() returns it."""
    kind = case["kind"]
    if kind == "moments":
        L = case["L"]
        h = _hills(L, case["N"], seed).astype(np.int64)
        n = L * L
        ref = int(h.sum()) // n
        d = h - ref
        c = [int((d ** k).sum()) for k in range(1, 5)]
        m = [np.longdouble(v) / n for v in c]
        q = m[0]
        return {"t": 0, "ref": ref, "c1": c[0], "c2": c[1], "c3": c[2], "c4": c[3],
                "phi2": float(m[1] - q * q), "phi3": float(m[2] - 3 * q * m[1] + 2 * q ** 3),
                "phi4": float(m[3] - 4 * q * m[2] + 6 * q * q * m[1] - 3 * q ** 4)}
    if sum(L * L * n for L, n in _surfaces(case)) * (2 if kind == "lockstep" else 1) > EXACT_ATTEMPTS:
        return None
    if kind == "served":
        jobs = _jobs(case, seed)
        got = []
        for (L, N, t, sd) in jobs:
            logs = _grow(L, N, 8, sd, t)[1]
            g = _grid(t)
            rec = [np.array([logs[k - 1][i][0] for k in g]) for i in range(3)]
            got.append((np.array(g), *rec, _w2(L, rec[0], rec[1])))
        t, s1, s2, acc, w2 = (np.concatenate(v) for v in zip(*got))
        return {"t": t, "s1": s1, "s2": s2, "accepted": acc, "w2": w2}
    n = case["sweeps"]
    if kind == "surface":
        L = case["L"]
        h, logs = _grow(L, case["N"], case["D"], seed, n, case["schedule"])
        s1, s2, acc = (np.array([r[i][0] for r in logs]) for i in range(3))
        return _out(np.arange(1, n + 1), s1, s2, acc, _w2(L, s1, s2), h[0])
    if kind == "lockstep":
        L, got = case["L"], []
        for g in range(case["groups"]):
            h, logs = _grow(L, case["N"], 8, 1000003 * seed + g, n, reals=128)
            lat = np.ascontiguousarray(h.T).astype(np.uint16).view(np.int32).reshape(-1)
            got.append((*logs[-1], _w2(L, logs[-1][0], logs[-1][1]), lat))
        s1, s2, acc, w2, lat = (np.concatenate(v) for v in zip(*got))
        return _out(np.full(len(s1), n), s1, s2, acc, w2, lat)
    got = []
    for (L, N, sd) in _batch_specs(case, seed):
        h, logs = _grow(L, N, case["D"], sd, n)
        got.append((*logs[-1], _w2(L, logs[-1][0], logs[-1][1]), h[0]))
    s1, s2, acc, w2, h = (np.concatenate(v) for v in zip(*got))
    return _out(np.full(len(s1), n), s1, s2, acc, w2, h)
