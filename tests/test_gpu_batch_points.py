"""GPU: the batch step with one cell per thread against single cavities: the
same per-cell code, so the states are the same bits and the norms agree to
the rounding of their grouping (64 eps for sums of positive terms).  Members
of fewer cells than a wavefront, of exactly one block (448 cells), one less
and one more; more members than a wavefront has lanes (the member search
takes two rounds); and which batches take this launch.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

EDGES = [(2, 2, 2), (7, 8, 8), (149, 3, 1 + 1), (447, 1 + 1, 2), (3, 3, 50), (7, 16, 4), (64, 7, 2), (31, 29, 30)]


@pytest.fixture(scope="module")
def C():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2006_02602_amd as C
    C.lib()
    return C


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("grids", [EDGES, [EDGES[m % 7] for m in range(64)], [EDGES[m % 7] for m in range(130)],
                                   [(21, 20, 23)]])
def test_batch_points_equal_single_cavities(C, grids, dtype):
    import torch
    print("batch points", len(grids), dtype, flush=True)
    rng = np.random.default_rng(5)
    prm = [C.Params(Ra=2e4, t_hot_field=torch.from_numpy(1.0 + 0.05 * rng.uniform(-1, 1, n[1] * n[2])).cuda()
                    if m % 3 == 0 else None) for m, n in enumerate(grids)]
    b = C.Batch([(C.Grid(*n, dtype=dtype), p) for n, p in zip(grids, prm)]).init(range(len(grids)), 0.3)
    assert b.handle.points == sum(-(-n[0] * n[1] * n[2] // 448) for n in grids)
    b.step(3)
    b.step(2)
    torch.cuda.synchronize()
    inner = (slice(None), slice(2, -2), slice(2, -2), slice(2, -2))
    for m, n in enumerate(grids):
        a = C.Cavity(C.Grid(*n, dtype=dtype), prm[m]).init(m, 0.3)
        a.step(5)
        torch.cuda.synchronize()
        assert torch.equal(a.fields()[inner], b.fields(m)[inner]), (m, n)
        na, nb = np.array(a.norms()), np.array(b.norms(m))
        assert (np.abs(na - nb) <= 64 * np.finfo(np.float64).eps * na).all()


@pytest.mark.parametrize("dtype", [0, 1])
def test_which_batches_take_it(C, dtype):
    wide = {0: 64, 1: 32}[dtype]
    g = C.Grid(30, 28, 33, dtype=dtype)
    assert C.Batch([(g, C.Params())] * 4).handle.points > 0
    assert C.Batch([(g, C.Params())] * 3 + [(g, C.Params(), 8)]).handle.points == 0         # a chosen chunk
    assert C.Batch([(g, C.Params())] * 3 + [(g, C.Params(), 0, wide)]).handle.points == 0   # a chosen tile
    assert C.Batch([(C.Grid(96, 96, 96, dtype=dtype), C.Params())] * 40).handle.points == 0  # full tiles, many
