"""GPU: cavity_adjoint_step adds to dj_dthot by plain loads and stores, so the
sums come out the same whether it lies in device memory or in mapped host
memory, where floating-point atomics are dropped.  The same additions in the
same order: the same bits.
"""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def C():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2006_02602_amd as C
    C.lib()
    return C


@pytest.mark.parametrize("n", [(2, 2, 2), (5, 4, 3), (65, 9, 7), (70, 18, 33)])
def test_wall_cotangent_in_host_memory(C, n):
    import torch
    print("adjoint into host memory", n, flush=True)
    L, g = C.lib(), C.Grid(*n)
    rng = np.random.default_rng(11)
    rows = n[1] * n[2]
    prm = C.Params(Ra=2e4, t_hot_field=torch.from_numpy(1.0 + 0.05 * rng.uniform(-1, 1, rows)).cuda())
    q = torch.zeros(C.cavity_state_elems(g), dtype=torch.float64, device="cuda")
    C.cavity_init(g, prm, 3, 0.3, q)
    lam, out = torch.zeros_like(q), torch.zeros_like(q)
    C.state_view(g, lam)[:, 2:-2, 2:-2, 2:-2] = torch.from_numpy(rng.standard_normal((5, n[2], n[1], n[0]))).cuda()
    ws = torch.zeros(C.cavity_adjoint_workspace_bytes(g) // 8, dtype=torch.float64, device="cuda")
    start = torch.from_numpy(rng.standard_normal(rows))
    got = []
    for dth in (start.cuda(), start.clone().pin_memory()):
        assert dth.is_cuda or dth.is_pinned()
        for _ in range(2):                        # added to what two calls leave
            rc = L.cavity_adjoint_step(ctypes.byref(g.c()), ctypes.byref(prm.c()), q.data_ptr(), lam.data_ptr(),
                                       out.data_ptr(), ws.data_ptr(), ws.numel() * 8, dth.data_ptr(), None, None)
            assert rc == C.CAV_OK
        torch.cuda.synchronize()
        got.append(dth.cpu().numpy())
    assert np.array_equal(got[0], got[1])
    assert (got[0] != start.numpy()).all()
