"""A choice that is entered for a key is what runs, one sweep per launch or
two, and every candidate gives the oracle's bits over whole fours of sweeps
and the rest of a call."""
import os

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu
PAIR = 64  # RSOS_TUNE_PAIR


@pytest.fixture()
def surface():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    from paper_1605_02620_amd import surface
    surface.tune_clear()
    yield surface
    surface.tune_clear()


def _check(oracle, log, h, L, N, seed, n, what):
    ref_h = workloads.flat(L)
    ref = oracle.run(ref_h, L, N, 8, seed=seed, t0=0, n=n)
    for k, name in ((1, "s1"), (2, "s2"), (3, "accepted")):
        assert np.array_equal(log[name], ref[:, k]), f"{what}: {name} differs"
    assert np.array_equal(h, ref_h), f"{what}: heights differ"


def test_the_entered_choice_runs(surface, oracle):
    L, N, n = 512, 1, 9
    cands = surface.tune_candidates(L, N, 8)
    assert {c["elem"] & PAIR for c in cands} == {0, PAIR}
    for c in cands:
        print(f"[tune] L={L} {c['TX']}x{c['TY']}x{c['NT']} elem={c['elem']} xmode={c['xmode']}", flush=True)
        surface.tune_set(L, N, 8, dict(c, graph_sweeps=4))
        s = surface.Surface(L, N=N, seed=3, D=8, tune=True)
        base = "block_sweep2" if c["elem"] & PAIR else "block_sweep"
        assert s.kernel_name().startswith(f"{base}<8,{c['TX']},{c['TY']},{c['NT']},")
        s.sweep(n)
        _check(oracle, s.log(1, n), s.heights(), L, N, 3, n, str(c))
        s.close()


def test_batch_of_both_kinds(surface, oracle):
    forced = {(256, 1): dict(TX=8, TY=8, NT=512, elem=2 | PAIR), (512, 2): dict(TX=16, TY=16, NT=256, elem=1),
              (1024, 1): dict(TX=32, TY=8, NT=256, elem=1 | PAIR)}
    for (L, N), c in forced.items():
        surface.tune_set(L, N, 8, dict(c, xmode=1, graph_sweeps=4), batch=True)
    specs = [(256, 1, 31), (512, 2, 32), (1024, 1, 33), (256, 1, 34)]
    os.environ["RSOS_BATCH_PLAN"] = "grouped"
    try:
        b = surface.Batch(specs, D=8, tune=True)
    finally:
        del os.environ["RSOS_BATCH_PLAN"]
    total = np.zeros(len(specs), dtype=np.int64)
    for counts in ([14] * 4, [3, 9, 0, 5]):
        print(f"[tune] batch {counts}", flush=True)
        b.sweep(counts)
        total += counts
    for i, (L, N, seed) in enumerate(specs):
        _check(oracle, b.log(i, 1, int(total[i])), b.heights(i), L, N, seed, int(total[i]), f"surface {i}")
    b.close()


def test_engine_and_file(surface, oracle, tmp_path):
    from paper_1605_02620_amd import serve
    choice = dict(TX=32, TY=8, NT=256, elem=1 | PAIR, xmode=0, graph_sweeps=8)
    surface.tune_set(512, 1, 8, choice, batch=True)
    path = tmp_path / "tune.txt"
    surface.tune_save(path)
    surface.tune_clear()
    surface.tune_load(path)
    t = surface.tune(512, 1, 8, batch=True)
    assert {k: t[k] for k in choice} == choice and t["measured"] == 0
    eng = serve.Engine(pool_bytes=64 << 20, max_running=8, D=8, tune=True)
    jobs = [(512, 1, 51, 22), (512, 1, 52, 9), (256, 4, 53, 17)]
    print(f"[tune] engine {jobs}", flush=True)
    ids = [eng.submit(L, N, seed, t_max, sample_t=range(1, t_max + 1), keep_heights=True) for (L, N, seed, t_max) in jobs]
    while eng.stats()["running"] or eng.stats()["queued"]:
        eng.step(16)
    for jid, (L, N, seed, t_max) in zip(ids, jobs):
        samples, heights, _ = eng.result(jid, heights=True)
        _check(oracle, samples, heights, L, N, seed, t_max, f"job L={L}")
    eng.close()


def test_tuned_is_not_slower_than_the_default(surface):
    t = surface.tune(1024, 1, 8)
    print(f"[tune] {t}", flush=True)
    # (ties within 1% go to the column strips)
    assert t["measured"] == 1 and t["ms_first_fit"] > 0 and t["ms_per_sweep"] <= 1.0101 * t["ms_first_fit"]


@pytest.mark.parametrize("L,batch,pairs", [(512, False, True), (4096, False, True), (8192, False, False), (512, True, False)])
def test_pairs_are_timed_where_launches_are_small(surface, L, batch, pairs):
    """Two sweeps per launch are a candidate alone, and where the blocks are
    few enough for the untuned rule to take them."""
    print(f"[tune] candidates L={L} batch={batch}", flush=True)
    assert any(c["elem"] & PAIR for c in surface.tune_candidates(L, 1, 8, batch=batch)) == pairs
