"""Reading widths needs no memory that the handle does not have: the first
read makes as many runtime calls as the second."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["batch", "lockstep"])
def test_first_width_makes_no_more_calls(kind):
    import paper_1605_02620_amd as rsos
    from paper_1605_02620_amd._lib import RsosError, lib

    def calls(before):
        for n in range(1, 32):
            b = rsos.Batch([(64, 1, 1), (256, 1, 2)]) if kind == "batch" else rsos.MultiSurface(16, N=1, seed=1, groups=1)
            b.sweep(1)
            for _ in range(before):
                b.width()
            lib().rsos_debug_fail(n)
            try:
                b.width()
            except RsosError:
                continue
            finally:
                lib().rsos_debug_fail(0)
                b.close()
            return n - 1
        raise AssertionError("no call went through")

    print(f"[reads] {kind}", flush=True)
    # the batch's first read waits for the upload of its descriptors
    assert calls(0) <= calls(1) + (1 if kind == "batch" else 0)
