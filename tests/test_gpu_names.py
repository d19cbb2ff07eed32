"""The kernel instance that rsos_kernel_name reports is one that is built and
that sweeps the surface: two sweeps per launch, attempts in steps, and the
single sweeps of the timing mode."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,D,kw,name,timed", [
    (64, 8, {}, "lds_run<8,512,0,true>", None),
    (128, 2, {}, "lds_run32<2,256,0>", None),
    (256, 8, {}, "block_sweep2<8,8,8,512,true>", "block_sweep<8,8,8,256,int16,void,2>"),
    (1360, 8, {}, "block_sweep2<8,32,8,256,false>", "block_sweep<8,16,8,512,int16,void,2>"),
    (4096, 8, {}, "block_sweep2<8,32,16,512,false>", "block_sweep<8,32,8,256,int8,int16,0>"),
    (1024, 16, {}, "block_sweep<16,4,4,384,int16,void,2>", None),
    (1024, 8, {"packed": True}, "block_sweep16<8,32,8,256,0>", None),
    (1024, 8, {"schedule": "double"}, "block_sweep<8,32,8,256,int8,int16,1>", None),
])
def test_kernel_name(L, D, kw, name, timed):
    import paper_1605_02620_amd as rsos
    print(f"[names] L={L} D={D} {kw}", flush=True)
    s = rsos.Surface(L, N=1, seed=1, D=D, **kw)
    assert s.kernel_name() == name
    s.timing(True)
    assert s.kernel_name() == (timed or name)
    s.timing(False)
    assert s.kernel_name() == name
    s.close()
