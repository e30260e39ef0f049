"""GPU: an odd number of steps, whose state is copied back into q, against the
same steps one by one (cavity_step_from, no copy): the same bits, norms too
(same partials, same order).  Rows that end at, before and after a 128-byte
line, planes of less and more than a block of the copy, states aligned to 16
bytes and to one element, and sizes of both kinds of stores.
"""
import pytest

pytestmark = pytest.mark.gpu

GRIDS = [((2, 2, 2), 0), ((15, 4, 3), 0), ((16, 5, 2), 0), ((17, 3, 4), 0), ((130, 129, 5), 0), ((161, 97, 30), 0),
         ((160, 160, 126), 0), ((31, 4, 3), 1), ((32, 5, 2), 1), ((33, 3, 4), 1), ((260, 259, 5), 1), ((200, 200, 161), 1)]


@pytest.fixture(scope="module")
def C():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2006_02602_amd as C
    C.lib()
    return C


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("n,dtype", GRIDS)
def test_odd_steps_end_in_q(C, n, dtype, shift):
    import torch
    print("copy back", n, dtype, shift, flush=True)
    g, prm = C.Grid(*n, dtype=dtype), C.Params(Ra=3e4)
    ref = C.Cavity(g, prm).init(7, 0.3)
    N = ref.q.numel()
    big = [torch.full((N + 4,), float("nan"), dtype=ref.q.dtype, device="cuda") for _ in range(2)]
    q, tmp = (b[shift:shift + N] for b in big)
    q.copy_(ref.q)
    a, b = ref.q, ref.q_tmp
    for _ in range(3):
        C.cavity_step_from(g, prm, a, b, ref.ws)
        a, b = b, a
    ws = torch.zeros_like(ref.ws)
    C.cavity_step(g, prm, None, q, tmp, ws, None, 3)
    torch.cuda.synchronize()
    inner = (slice(None), slice(2, -2), slice(2, -2), slice(2, -2))
    assert torch.equal(C.state_view(g, q)[inner], C.state_view(g, a)[inner])
    assert C.cavity_residual_norm(g, ws) == C.cavity_residual_norm(g, ref.ws)
    for t in big:                                 # nothing written beyond the state
        assert torch.isnan(t[:shift]).all() and torch.isnan(t[shift + N:]).all()
