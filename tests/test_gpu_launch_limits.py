"""GPU: every launch stays below 2^32 threads, whatever sizes the host accepts.
The launches of the largest calls are captured, not run (their buffers stand
for memory that is never touched); a deep thin grid just past the limit of
one 1024-thread block per plane and field is stepped in full.
"""
import ctypes

import pytest

from launch_capture import launches

pytestmark = pytest.mark.gpu

FAKE = 0x7f0000000000


@pytest.fixture(scope="module")
def C():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2006_02602_amd as C
    C.lib()
    torch.zeros(1, device="cuda")
    return C


# the deepest planes of 2 x 2 cells that are accepted, the first depth past
# the limit, and the largest cubes
@pytest.mark.parametrize("n,dtype", [((2, 2, 11184806), 0), ((2, 2, 5592401), 1), ((2, 2, 838861), 0),
                                     ((1278, 1278, 1278), 0), ((1274, 1274, 1274), 1)])
@pytest.mark.parametrize("shift", [0, 1])
def test_launches_of_an_odd_step(C, n, dtype, shift):
    L, g = C.lib(), C.Grid(*n, dtype=dtype)
    assert C.cavity_state_elems(g) > 0
    size = C.cavity_state_elems(g) * (4 if dtype else 8)
    q = FAKE + shift * (4 if dtype else 8)
    t, ws, wb = q + size, FAKE - (1 << 40), C.cavity_workspace_bytes(g)
    print("odd step", n, dtype, shift, flush=True)
    rc, nodes = launches(L, lambda s: L.cavity_step(ctypes.byref(g.c()), ctypes.byref(C.Params().c()), None, q, t, ws, wb,
                                                    None, 0, 1, s))
    assert rc == C.CAV_OK and len(nodes) == 2             # the sweep, the copy back with the norms
    for grid, threads in nodes:
        assert 0 < grid * threads < 1 << 32, nodes


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("items", [1, 1023, 1024, 1 << 20, (1 << 20) + 1, 1 << 23, (1 << 31) - 1])
def test_launches_of_a_batch_with_open_blocks(C, items, dtype):
    from paper_2006_02602_amd import _lib
    L = C.lib()
    b = _lib.CavBatch(table=FAKE, members=1, items=items, dtype=dtype, parity=0, cells=items, shapes=1, points=0)
    print("batch", items, dtype, flush=True)
    rc, nodes = launches(L, lambda s: L.cavity_batch_step(ctypes.byref(b), 1, 0, s))
    assert rc == C.CAV_OK and len(nodes) == 2
    for grid, threads in nodes:
        assert 0 < grid * threads < 1 << 32, nodes
    assert nodes[0][0] <= max(items, 256)


@pytest.mark.parametrize("dtype", [0, 1])
def test_odd_step_of_a_deep_thin_grid(C, dtype):
    import torch
    g, prm = C.Grid(2, 2, 838900, dtype=dtype), C.Params(Ra=3e4)
    print("deep thin grid", dtype, flush=True)
    cav = C.Cavity(g, prm).init(3, 0.3)
    ref = torch.zeros_like(cav.q)
    C.cavity_step_from(g, prm, cav.q, ref, cav.ws)
    norms = C.cavity_residual_norm(g, cav.ws)
    cav.step(1)
    torch.cuda.synchronize()
    inner = (slice(None), slice(2, -2), slice(2, -2), slice(2, -2))
    assert torch.equal(cav.fields()[inner], C.state_view(g, ref)[inner])
    assert cav.norms() == norms
    assert bool(torch.isfinite(cav.fields()[inner]).all())
