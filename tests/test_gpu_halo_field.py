"""GPU: the exchange with one field a thread (up to 700 000 elements) and with
all fields a thread, on either side of the line between them and at ragged
faces: pack, unpack and the exchange of a step move the oracle's elements,
bit for bit.  Widths of 0, 1 and 2; boxes and states whose address allows
pairs of layers and ones whose address does not.
"""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

CASES = [((4, 4, 4), (2, 2, 2)), ((30, 12, 21), (5, 3, 7)), ((16, 512, 2), (2, 1, 1)), ((513, 8, 6), (1, 2, 3)),
         ((110, 110, 114), (2, 2, 2)), ((112, 112, 114), (2, 2, 2))]
WIDTHS = [(1, 2, 2, 2, 2), (2, 1, 1, 1, 1), (0, 2, 1, 0, 2)]


@pytest.fixture(scope="module")
def C():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2006_02602_amd as C
    C.lib()
    return C


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("width", WIDTHS)
@pytest.mark.parametrize("n,split", CASES)
def test_pack_and_unpack(C, n, split, width, dtype, shift):
    import torch
    print("halo field", n, split, width, dtype, shift, flush=True)
    P = O.Problem(*n)
    g, h = C.Grid(*n, dtype=dtype), C.Halo(split, width)
    real = (np.float64, np.float32)[dtype]
    q = np.random.default_rng(3).standard_normal(P.shape).astype(real)
    ref = O.halo_pack(P, (split, width), q.astype(np.float64)).astype(real)
    N = C.cavity_state_elems(g)
    state = torch.zeros(N + 2, dtype=g.torch_dtype, device="cuda")[shift:shift + N]
    buf = torch.full((ref.size + 2,), float("nan"), dtype=g.torch_dtype, device="cuda")
    box = buf[shift:shift + ref.size]
    view = C.state_view(g, state)
    view.copy_(torch.from_numpy(q))
    C.halo_pack(g, h, state, box)
    torch.cuda.synchronize()
    assert np.array_equal(box.cpu().numpy(), ref)
    assert torch.isnan(buf[:shift]).all() and torch.isnan(buf[shift + ref.size:]).all()
    mark = np.zeros(P.shape)
    O.halo_unpack(P, (split, width), np.ones(ref.size), mark)
    poisoned = q.copy()
    poisoned[mark == 1] = np.nan
    view.copy_(torch.from_numpy(poisoned))
    C.halo_unpack(g, h, box, state)
    torch.cuda.synchronize()
    assert np.array_equal(view.cpu().numpy(), q)


@pytest.mark.parametrize("n,split", [((4, 4, 4), (2, 2, 2)), ((110, 110, 114), (2, 2, 2)), ((112, 112, 114), (2, 2, 2))])
@pytest.mark.parametrize("dtype", [0, 1])
def test_exchange_of_a_step(C, n, split, dtype):
    import torch
    print("halo field step", n, split, dtype, flush=True)
    g, h, prm = C.Grid(*n, dtype=dtype), C.Halo(split, (1, 2, 2, 2, 2)), C.Params(Ra=1e4)
    a = C.Cavity(g, prm, h).init(7, 0.3)
    b = C.Cavity(g, prm).init(7, 0.3)
    a.step(2)
    b.step(1)
    ref = torch.full_like(a.buf, float("nan"))
    C.halo_pack(g, h, b.q, ref)
    b.step(1)
    torch.cuda.synchronize()
    inner = (slice(None), slice(2, -2), slice(2, -2), slice(2, -2))
    assert torch.equal(a.buf, ref) and torch.equal(a.fields()[inner], b.fields()[inner])
