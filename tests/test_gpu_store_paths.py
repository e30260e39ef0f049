"""GPU: the marching tile's two kinds of stores, at sizes on either side of both
limits between them (both states of 32 MB and of 256 MB): the same arithmetic,
so the states must be the same bits.  The other side is the grid as a member of
a batch whose total size takes it to non-temporal stores, and the overlapped
step.
"""
import pytest

pytestmark = pytest.mark.gpu

CASES = [((74, 73, 74), 0), ((74, 74, 74), 0), ((160, 160, 124), 0), ((160, 160, 125), 0), ((161, 97, 130), 0),
         ((100, 100, 80), 1), ((100, 100, 81), 1), ((200, 200, 159), 1), ((200, 200, 160), 1), ((131, 67, 201), 1)]


@pytest.fixture(scope="module")
def C():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2006_02602_amd as C
    C.lib()
    return C


@pytest.mark.parametrize("n,dtype", CASES)
def test_stores_do_not_change_the_state(C, n, dtype):
    import torch
    print("stores", n, dtype, flush=True)
    g, prm = C.Grid(*n, dtype=dtype), C.Params(Ra=3e4)
    big = C.Grid.cube(192, dtype)                 # takes the batch past 256 MB
    wide = {0: 64, 1: 32}[dtype]
    b = C.Batch([(g, prm, 0, wide), (big, prm, 0, wide)]).init([7, 8], 0.3)
    a = C.Cavity(g, prm).init(7, 0.3)
    inner = (slice(None), slice(2, -2), slice(2, -2), slice(2, -2))
    b.step(3)
    a.step(3)
    torch.cuda.synchronize()
    assert torch.equal(a.fields()[inner], b.fields(0)[inner])
    if n[0] % 2 == 0:
        o = C.Cavity(g, prm, C.Halo((2, 1, 1), (1, 2, 2, 2, 2))).init(7, 0.3)
        o.step_overlap(3)
        torch.cuda.synchronize()
        assert torch.equal(o.fields()[inner], a.fields()[inner])
