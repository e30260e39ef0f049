"""GPU: splits along i, where the marching tile's loads take the
exchanged cells from the buffer and whose stores pack the next exchange.

The exchange is a round trip, so the states must be the bits of the run
without a split (as must the norms where both run the tile: same sums), and the buffer
after m steps must be halo_pack of the state before step m.  The grids put
cuts at a tile's edge, inside a tile and in a ragged last tile; k chunks are
whole and ragged, of odd and even length.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CASES = [((64, 64, 64), (8, 1, 1), 0), ((64, 64, 64), (2, 1, 1), 0), ((192, 64, 40), (3, 1, 1), 0),
         ((120, 66, 75), (5, 1, 1), 0), ((80, 80, 80), (20, 1, 1), 0), ((160, 80, 80), (40, 1, 1), 0),
         ((192, 160, 144), (8, 1, 1), 0), ((192, 160, 144), (4, 1, 1), 1), ((196, 157, 139), (7, 1, 1), 1),
         ((16, 16, 16), (2, 1, 1), 1), ((33, 5, 3), (3, 1, 1), 1), ((8, 2, 2), (2, 1, 1), 1), ((16, 16, 16), (2, 1, 1), 0),
         ((32, 32, 32), (8, 1, 1), 0)]
ONE_LAUNCH = {((16, 16, 16), 0)}     # faster with one cell per thread: its exchange stays a launch


@pytest.fixture(scope="module")
def C():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2006_02602_amd as C
    C.lib()
    return C


@pytest.mark.parametrize("wall", [False, True])
@pytest.mark.parametrize("width", [(1, 2, 2, 2, 2), (2, 1, 1, 1, 1), (0, 2, 0, 1, 2)])
@pytest.mark.parametrize("n,split,dtype", CASES)
def test_exchange_in_the_sweep(C, n, split, dtype, width, wall):
    import torch
    print("sweep exchange", n, split, dtype, width, wall, flush=True)
    g, h = C.Grid(*n, dtype=dtype), C.Halo(split, width)
    theta = None
    if wall:
        theta = torch.from_numpy(1.0 + 0.05 * np.random.default_rng(3).uniform(-1, 1, n[1] * n[2])).cuda()
    prm = C.Params(Ra=3e4, t_hot_field=theta)
    plain = C.Cavity(g, prm).init(7, 0.3)
    q0 = plain.q.clone()
    inner = (slice(None), slice(2, -2), slice(2, -2), slice(2, -2))
    for steps in (1, 2, 3):
        a = C.Cavity(g, prm, h)
        a.q.copy_(q0)
        a.buf.fill_(float("nan"))
        C.cavity_timing_read()
        C.cavity_timing_enable(True)
        a.step(steps)
        C.cavity_timing_enable(False)
        names = set(C.cavity_timing_read())
        assert "halo_unpack" not in names
        if (n, dtype) in ONE_LAUNCH:
            assert "halo_exchange" in names and "sweep_xchg" not in names
        else:
            assert "halo_exchange" not in names and (steps == 1 or "sweep_xchg" in names)
        ref = torch.full_like(a.buf, float("nan"))
        C.halo_pack(g, h, plain.q, ref)          # plain: steps - 1 steps so far
        plain.step(1)
        torch.cuda.synchronize()
        assert torch.equal(a.buf, ref)
        assert torch.equal(a.fields()[inner], plain.fields()[inner])
        na, nb = np.array(a.norms()), np.array(plain.norms())
        if n[0] * n[1] * n[2] <= 150000:         # the run without a split sums the norms in other groups
            assert (np.abs(na - nb) <= 64 * np.finfo(np.float64).eps * nb).all()
        else:
            assert a.norms() == plain.norms()
