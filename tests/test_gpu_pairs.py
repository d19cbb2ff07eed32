"""Launches of two sweeps: every site and every record of the sums agrees with
the oracle bit for bit, for each block shape, over lattices that it does not
divide, from any start time and where surfaces make unequal numbers of sweeps."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rsos():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    import paper_1605_02620_amd as pkg
    return pkg


def _check(oracle, s_log, s_h, h0, L, N, seed, t0, n, what):
    oracle.set_threads(16)
    try:
        h = h0.copy()
        ref = oracle.run(h, L, N, 8, seed=seed, t0=t0, n=n)
    finally:
        oracle.set_threads(0)
    for k, name in ((1, "s1"), (2, "s2"), (3, "accepted")):
        assert np.array_equal(s_log[name], ref[:, k]), f"{what}: {name} differs"
    assert np.array_equal(s_h, h), f"{what}: heights differ"


@pytest.mark.parametrize("L,N,start,t0,calls", [
    (256, 1, "flat", 0, (5, 4, 1)),    # 8 x 8 tiles in steps
    (272, 3, "rough", 1, (70,)),       # blocks that overlap, T = 34
    (1024, 40, "cone", 0, (7,)),
    (1360, 2, "rough", 0, (4, 7)),     # 32 x 8 tiles, one block per CU
    (1296, 1, "flat", 3, (11,)),       # an odd start time
    (1296, 6, "rough", 0, (9,)),       # the largest N of the byte staging
    (1296, 7, "rough", 0, (9,)),       # one more: single sweeps
    (1328, 5, "cone", 2, (8,)),        # int16 sub-blocks
    (2576, 1, "flat", 0, (6,)),        # 32 x 16
    (3088, 1, "rough", 1, (5,)),       # 32 x 8, three per CU
])
def test_pairs(rsos, oracle, L, N, start, t0, calls):
    print(f"[pairs] L={L} N={N} {start} t0={t0}", flush=True)
    h0 = (workloads.flat(L) if start == "flat" else workloads.cone(L, N, N * L // 4, seed=L) if start == "cone"
          else workloads.rough(L, min(N, 4), seed=L))
    s = rsos.Surface(L, N=N, seed=L + N, h0=h0, t0=t0)
    for n in calls:
        s.sweep(n)
    n = sum(calls)
    _check(oracle, s.log(t0 + 1, n), s.heights(), h0, L, N, L + N, t0, n, f"L={L} N={N}")
    s.close()


@pytest.mark.parametrize("L,copies", [(256, 16), (256, 64), (256, 66), (320, 40), (512, 16)])
def test_pairs_batch(rsos, oracle, L, copies):
    """Equal and unequal numbers of sweeps, replayed graphs included."""
    import torch
    print(f"[pairs] {copies} x L={L}", flush=True)
    stream = torch.cuda.Stream()
    specs = [(L, 1 + k % 2, 100 + k) for k in range(copies)]
    b = rsos.Batch(specs, stream=stream)
    total = np.zeros(copies, dtype=np.int64)
    uneven = np.array([3 + 5 * (k % 3) for k in range(copies)])
    for n in (70, uneven, 6, np.where(np.arange(copies) == 1, 0, 130)):
        b.sweep(n)
        total += n
    w = b.width()
    for k in (0, 1, 2, copies - 1):
        n = int(total[k])
        _check(oracle, b.log(k, 1, n), b.heights(k), workloads.flat(L), L, specs[k][1], specs[k][2], 0, n, f"surface {k}")
    assert [int(x["t"]) for x in w] == [int(x) for x in total]
    b.close()


def test_uneven_call_captures_nothing(rsos):
    """The first call with unequal counts makes as many runtime calls as a
    later one: its graph was captured when the batch was created."""
    import torch
    from paper_1605_02620_amd._lib import RsosError, lib
    stream = torch.cuda.Stream()

    def calls(before):
        """Runtime calls of an uneven call after `before` others."""
        for n in range(1, 64):
            b = rsos.Batch([(256, 1, 1), (256, 1, 2)], stream=stream)
            for _ in range(before):
                b.sweep([0, 70])
                b.width()
            lib().rsos_debug_fail(n)
            try:
                b.sweep([0, 70])
            except RsosError:
                continue
            finally:
                lib().rsos_debug_fail(0)
                b.close()
            return n - 1
        raise AssertionError("no call went through")

    print("[pairs] runtime calls of uneven calls", flush=True)
    assert calls(0) <= calls(1) + 3  # a rewrite of the descriptors is three


@pytest.mark.parametrize("L,N,start", [(144, 1, "flat"), (160, 2, "rough"), (144, 140, "cone"), (144, 141, "cone")])
def test_pairs_on_the_smallest_lattices(rsos, oracle, L, N, start):
    """The smallest sides of the tile-block path, whose regions are nearly as
    wide as the lattice, up to the largest N of the 16-bit staging and one
    more (single sweeps)."""
    print(f"[pairs] L={L} N={N} {start}", flush=True)
    h0 = (workloads.flat(L) if start == "flat" else workloads.cone(L, N, N * L // 4, seed=L) if start == "cone"
          else workloads.rough(L, min(N, 4), seed=L))
    s = rsos.Surface(L, N=N, seed=L + N, h0=h0)
    assert s.kernel_name().startswith("block_sweep2<8,8,8,512,true>") == (N <= 140)
    s.sweep(9)
    _check(oracle, s.log(1, 9), s.heights(), h0, L, N, L + N, 0, 9, f"L={L} N={N}")
    s.close()
