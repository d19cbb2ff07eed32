"""Surfaces that live in LDS against the oracle, bit for bit: every domain
size, the smallest and largest sides, both schedules, the edge of the 16-bit
staging (N L = 8192), and a run long enough to move the staging's base."""
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


def _oracle(oracle, h0, L, N, D, seed, n, schedule="checkerboard"):
    h = h0.copy()
    lg = (oracle.run_dt if schedule == "double" else oracle.run)(h, L, N, D, seed=seed, t0=0, n=n)
    return h, lg


def _same(g_log, r_log, g_h, r_h, what):
    for k, name in ((1, "s1"), (2, "s2"), (3, "accepted")):
        assert np.array_equal(g_log[name], r_log[:, k]), f"{what}: {name} differs"
    assert np.array_equal(g_h, r_h), f"{what}: heights differ"


@pytest.mark.parametrize("L,N,D,n,schedule", [
    (4, 1, 2, 20, "checkerboard"), (124, 2, 2, 6, "checkerboard"),
    (8, 1, 4, 20, "checkerboard"), (120, 3, 4, 6, "checkerboard"),
    (16, 1, 8, 40, "checkerboard"), (48, 2, 8, 20, "checkerboard"), (64, 1, 8, 70, "checkerboard"),
    (80, 4, 8, 10, "checkerboard"), (128, 7, 8, 12, "checkerboard"),
    (128, 64, 8, 8, "checkerboard"), (128, 65, 8, 8, "checkerboard"), (128, 2 ** 31 - 1, 8, 4, "checkerboard"),
    (32, 1, 16, 12, "checkerboard"), (128, 2, 16, 6, "checkerboard"),
    (64, 1, 32, 6, "checkerboard"), (128, 3, 32, 4, "checkerboard"),
    (16, 1, 8, 30, "double"), (112, 2, 8, 8, "double"), (128, 1, 8, 8, "double"),
    (32, 3, 16, 10, "double"), (128, 1, 16, 6, "double"),
])
@pytest.mark.parametrize("start", ["flat", "rough"])
def test_small_surfaces(rsos, oracle, L, N, D, n, schedule, start):
    print(f"[lds] L={L} N={N} D={D} {schedule} {start}", flush=True)
    h0 = workloads.flat(L) if start == "flat" else workloads.rough(L, min(N, 64), seed=L + N, base=1000)
    s = rsos.Surface(L, N=N, seed=7 * L + N, D=D, h0=h0, schedule=schedule)
    s.sweep(n - 1)
    s.sweep(1)  # a second launch goes on from the record of the first
    r_h, r_log = _oracle(oracle, h0, L, N, D, 7 * L + N, n, schedule)
    _same(s.log(1, n), r_log, s.heights(), r_h, s.kernel_name())
    s.close()


def test_base_follows_the_surface(rsos, oracle):
    L, N, n = 16, 1, 4200
    print(f"[lds] L={L} {n} sweeps", flush=True)
    s = rsos.Surface(L, N=N, seed=3, D=8)
    s.sweep(n)
    r_h, r_log = _oracle(oracle, workloads.flat(L), L, N, 8, 3, n)
    _same(s.log(1, n), r_log, s.heights(), r_h, "rebase")
    s.close()


def test_mixed_launch(rsos, oracle):
    """Sides with different LDS needs in one launch, with and without one
    that the 16-bit staging does not take."""
    for specs in ([(16, 1, 1), (80, 2, 2), (64, 1, 3), (128, 4, 4)], [(128, 100, 5), (32, 1, 6)]):
        print(f"[lds] batch {specs}", flush=True)
        b = rsos.Batch(specs, D=8)
        b.sweep([3 + i for i in range(len(specs))])
        for i, (L, N, seed) in enumerate(specs):
            r_h, r_log = _oracle(oracle, workloads.flat(L), L, N, 8, seed, 3 + i)
            _same(b.log(i, 1, 3 + i), r_log, b.heights(i), r_h, f"surface {i}")
        b.close()


@pytest.mark.parametrize("L,N,D,schedule", [(64, 1, 8, "checkerboard"), (128, 3, 16, "double"),
                                            (128, 100, 8, "checkerboard")])
def test_sums_are_the_lattice_s_own(rsos, oracle, L, N, D, schedule):
    """rsos_sweep_static: the records of an LDS-resident surface are sums of
    its heights, whatever sums of the start the caller passes."""
    import ctypes

    import torch
    from paper_1605_02620_amd import _lib
    from paper_1605_02620_amd.surface import _params
    print(f"[lds] sums L={L} N={N} D={D} {schedule}", flush=True)
    n, h0 = 5, workloads.rough(L, min(N, 64), seed=L + N, base=1000)
    r_h, r_log = _oracle(oracle, h0, L, N, D, 9, n, schedule)
    s1, s2 = int(h0.astype(np.int64).sum()), int((h0.astype(np.int64) ** 2).sum())
    for sums in ((s1, s2), (0, 0), (s1 + 7, 2 * s2)):
        bufs = [torch.from_numpy(h0.astype(np.int32)).cuda(), torch.zeros(L * L, dtype=torch.int32, device="cuda")]
        log = torch.zeros(3 * n, dtype=torch.int64, device="cuda")
        p = _params(L, N, D, 9, schedule=schedule)
        _lib.check(_lib.lib().rsos_sweep_static(
            ctypes.byref(p), ctypes.c_void_p(bufs[0].data_ptr()), ctypes.c_void_p(bufs[1].data_ptr()), 0, *sums, n,
            ctypes.c_void_p(log.data_ptr()), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))
        torch.cuda.synchronize()
        assert np.array_equal(log.cpu().numpy().reshape(n, 3), r_log[:, 1:4]), f"sums given as {sums}"
        assert np.array_equal(bufs[n & 1].cpu().numpy(), r_h)


@pytest.mark.parametrize("sizes,each,D,schedule", [
    ((64,), 257, 8, "checkerboard"),      # one phase's steps at a time
    ((64,), 2048, 8, "checkerboard"),
    ((112,), 768, 8, "checkerboard"),
    ((32, 64), 1024, 8, "checkerboard"),
    ((64,), 300, 8, "double"),
    ((64,), 300, 16, "checkerboard"),
    ((32,), 700, 4, "checkerboard"),
])
def test_many_surfaces(rsos, oracle, sizes, each, D, schedule):
    """More surfaces than are resident at once: the kernel and the step lists
    go by their number, and the results do not."""
    print(f"[lds] {each} of each of {sizes} D={D} {schedule}", flush=True)
    specs = [(L, 1 + k % 2, 11 * L + k) for L in sizes for k in range(each)]
    b = rsos.Batch(specs, D=D, schedule=schedule, log_cap=8)
    b.sweep(3)
    b.sweep(2)
    for i in (0, 1, len(specs) // 2, len(specs) - 1):
        L, N, seed = specs[i]
        r_h, r_log = _oracle(oracle, workloads.flat(L), L, N, D, seed, 5, schedule)
        _same(b.log(i, 1, 5), r_log, b.heights(i), r_h, f"surface {i} of {len(specs)}")
    b.close()
