"""Lattices that no large tile block divides: the last blocks of a row and of
a column overlap the ones before, and every site and sum still agrees with
the oracle bit for bit."""
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


def _oracle(oracle, h0, L, N, D, seed, n, schedule):
    oracle.set_threads(16)
    try:
        h = h0.copy()
        lg = (oracle.run_dt if schedule == "double" else oracle.run)(h, L, N, D, seed=seed, t0=0, n=n)
    finally:
        oracle.set_threads(0)
    return h, lg


def _same(g_log, r_log, g_h, r_h, what):
    for k, name in ((1, "s1"), (2, "s2"), (3, "accepted")):
        assert np.array_equal(g_log[name], r_log[:, k]), f"{what}: {name} differs"
    assert np.array_equal(g_h, r_h), f"{what}: heights differ"


@pytest.mark.parametrize("L,N,D,start,schedule", [
    (272, 1, 8, "flat", "checkerboard"),     # T = 34
    (288, 2, 8, "rough", "checkerboard"),    # T = 36, one block more than half overlapped
    (528, 4, 8, "cone", "checkerboard"),     # T = 66: overlapping blocks on the wide path
    (1360, 2, 8, "rough", "checkerboard"),   # T = 170
    (1040, 7, 8, "rough", "checkerboard"),   # T = 130
    (1040, 40, 8, "rough", "checkerboard"),  # int16 staging
    (264, 1, 4, "flat", "checkerboard"),     # T = 66
    (416, 3, 16, "rough", "checkerboard"),   # T = 26
    (132, 1, 2, "flat", "checkerboard"),     # T = 66
    (304, 1, 8, "flat", "double"),           # T = 38
    (1360, 1, 8, "rough", "double"),
    (352, 1, 16, "flat", "double"),          # T = 22
])
def test_overlapping_blocks(rsos, oracle, L, N, D, start, schedule):
    print(f"[ragged] L={L} N={N} D={D} {start} {schedule}", flush=True)
    h0 = (workloads.flat(L) if start == "flat" else workloads.cone(L, N, N * L // 4, seed=L) if start == "cone"
          else workloads.rough(L, min(N, 4), seed=L))
    n = 5
    s = rsos.Surface(L, N=N, seed=L + N, D=D, h0=None if start == "flat" else h0, schedule=schedule)
    s.sweep(n)
    r_h, r_log = _oracle(oracle, h0, L, N, D, L + N, n, schedule)
    _same(s.log(1, n), r_log, s.heights(), r_h, s.kernel_name())
    s.close()


def test_mixed_batch(rsos, oracle):
    """Sizes that the batch's shape tiles and sizes that it does not."""
    specs = [(256, 1, 5), (400, 2, 6), (512, 1, 7), (1040, 1, 8)]
    print(f"[ragged] batch {specs}", flush=True)
    b = rsos.Batch(specs, D=8)
    b.sweep([4, 5, 3, 5])
    for i, ((L, N, seed), n) in enumerate(zip(specs, (4, 5, 3, 5))):
        r_h, r_log = _oracle(oracle, workloads.flat(L), L, N, 8, seed, n, "checkerboard")
        _same(b.log(i, 1, n), r_log, b.heights(i), r_h, f"surface {i}")
    b.close()
