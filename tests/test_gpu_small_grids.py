"""GPU: the step of small grids (one cell per thread) against the marching
tile, which runs the same per-cell update inside a batch: the states must be
the same bits, and the norms agree to the rounding of their differently
grouped sums (at most 2^23 terms, all >= 0: 64 eps is ample).  The grids sit
at the edges of its blocks (64, 192, 256, 448, 512 cells), of its lane moves
(rows shorter and longer than a wavefront, ending mid-wavefront) and of the
wall rules (extents 2, 3, 4).
"""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

GRIDS = [(2, 2, 2), (3, 2, 4), (4, 4, 4), (5, 3, 13), (2, 2, 48), (48, 2, 2), (64, 7, 2), (63, 3, 5), (65, 4, 3),
         (130, 5, 3), (16, 16, 16), (31, 29, 30), (61, 47, 20)]


@pytest.fixture(scope="module")
def C():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2006_02602_amd as C
    C.lib()
    return C


@pytest.mark.parametrize("wall", [False, True])
@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("n", GRIDS)
def test_small_grid_step_is_the_marching_step(C, n, dtype, wall):
    import torch
    print("small grid", n, dtype, wall, flush=True)
    g = C.Grid(*n, dtype=dtype)
    theta = None
    if wall:
        theta = torch.from_numpy(1.0 + 0.05 * np.random.default_rng(3).uniform(-1, 1, n[1] * n[2])).cuda()
    prm = C.Params(Ra=3e4, t_hot_field=theta)
    cav = C.Cavity(g, prm).init(7, 0.3)
    b = C.Batch([(g, prm, 3)])
    b.q[0].copy_(cav.q)
    cav.step(4)
    b.step(4)
    torch.cuda.synchronize()
    inner = (slice(None), slice(2, -2), slice(2, -2), slice(2, -2))
    a, r = cav.fields()[inner].cpu().numpy(), b.fields(0)[inner].cpu().numpy()
    assert np.isfinite(r).all() and np.array_equal(a, r)
    na, nr = np.array(cav.norms()), np.array(b.norms(0))
    assert (np.abs(na - nr) <= 64 * np.finfo(np.float64).eps * nr).all()


@pytest.mark.parametrize("n", [(2, 2, 2), (5, 3, 13), (65, 4, 3), (31, 29, 30)])
def test_small_grid_step_matches_oracle(C, n):
    import torch
    P = O.Problem(*n, Ra=3e4)
    q0 = O.init(P, 7, 0.05)
    ref = q0.copy()
    O.step(P, ref, 5)
    cav = C.Cavity(C.Grid(*n), C.Params(Ra=3e4))
    cav.fields().copy_(torch.from_numpy(q0))
    cav.step(5)
    torch.cuda.synchronize()
    a, r = P.interior(cav.fields().cpu().numpy()), P.interior(ref)
    for f in range(5):
        assert np.abs(a[f] - r[f]).max() <= 1e-12 * max(np.abs(r[f]).max(), 1e-300), O.FIELDS[f]
