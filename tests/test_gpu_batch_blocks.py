"""GPU: which launches a batch step takes for the blocks its caller asks for.
Fewer blocks than fill the device (one per compute unit in FP64, three in
FP32) are kept on every step, whatever the batch; the launch with one cell per
thread is for callers that leave the blocks open or fill the device anyway.
The launches are captured, not run; the states of all choices are compared.
"""
import ctypes

import pytest

from launch_capture import launches

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def C():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2006_02602_amd as C
    C.lib()
    return C


def grids(L, handle, nsteps, nblocks):
    h = type(handle).from_buffer_copy(handle)
    rc, nodes = launches(L, lambda s: L.cavity_batch_step(ctypes.byref(h), nsteps, nblocks, s))
    assert rc == 0
    return [g for g, _ in nodes]


@pytest.mark.parametrize("dtype", [0, 1])
def test_blocks_of_every_step(C, dtype):
    import torch
    print("batch blocks", dtype, flush=True)
    L, fill = C.lib(), (3 if dtype else 1) * torch.cuda.get_device_properties(0).multi_processor_count
    b = C.Batch([(C.Grid(30, 28, 33, dtype=dtype), C.Params())] * 4)
    h, pts = b.handle, b.handle.points
    assert pts > 0
    for nb in (1, 64, fill - 1):
        assert grids(L, h, 3, nb) == [nb, nb, nb, 4]          # the steps, the norms of 4 members
    for nb in (fill, fill + 1, 2 * fill):
        assert grids(L, h, 3, nb) == [pts, pts, nb, 4]
    assert grids(L, h, 3, 0)[:2] == [pts, pts]
    assert grids(L, h, 1, 0)[0] != pts


@pytest.mark.parametrize("dtype", [0, 1])
def test_states_do_not_depend_on_the_blocks(C, dtype):
    import torch
    mix = [(31, 29, 30), (2, 2, 2), (65, 9, 7), (20, 33, 12)]
    want = None
    for nb in (0, 1, 100, 767, 768):
        b = C.Batch([(C.Grid(*n, dtype=dtype), C.Params(Ra=2e4)) for n in mix]).init(range(4), 0.3)
        b.step(4, nblocks=nb)
        torch.cuda.synchronize()
        inner = (slice(None), slice(2, -2), slice(2, -2), slice(2, -2))
        got = [b.fields(m)[inner].clone() for m in range(4)]
        want = want or got
        for a, c in zip(want, got):
            assert torch.equal(a, c)
