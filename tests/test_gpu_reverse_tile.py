"""GPU: the reverse step's tile at the sizes where it can go wrong: tiny grids
(every cell within two of several walls, the centre's star reaching them),
and grids just past a tile's edge in i and j with k chunks of a few planes.

Tiny grids: every entry of the cotangent against the full transposed Jacobian
of one step, column by column from the complex-step tangent oracle.  An entry
sums at most ~100 products of O(1) rounding errors, each relative to the
largest: 1e-12 of the largest entry is ample.  Larger grids: the inner
products <lam_out, v> = <lam, J v>, within 1e-11 of their absolute sum.
"""
import numpy as np
import pytest

import oracle as O
from oracle import tangent as TG

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def C():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2006_02602_amd as C
    C.lib()
    return C


class Step:
    """One step at a random state: its reverse on the GPU, its tangent in the oracle."""

    def __init__(self, C, n, Ra, seed):
        import torch
        self.n, self.Ra = n, Ra
        ni, nj, nk = n
        rng = np.random.default_rng(seed)
        self.P = O.Problem(*n)
        self.theta = 1.0 + 0.05 * rng.uniform(-1, 1, nj * nk)
        self.q = O.init(self.P, seed, 0.3)
        self.P.interior(self.q)[0] = rng.uniform(-1, 1, (nk, nj, ni))
        self.lam = rng.standard_normal((5, nk, nj, ni))
        g = C.Grid(*n)
        prm = C.Params(Ra=Ra, t_hot_field=torch.from_numpy(self.theta).cuda())
        flat = [torch.zeros(C.cavity_state_elems(g), dtype=torch.float64, device="cuda") for _ in range(3)]
        inner = [C.state_view(g, t)[:, 2:-2, 2:-2, 2:-2] for t in flat]
        inner[0].copy_(torch.from_numpy(np.ascontiguousarray(self.P.interior(self.q))))
        inner[1].copy_(torch.from_numpy(self.lam))
        flat[2].fill_(float("nan"))
        ws = torch.full((C.cavity_adjoint_workspace_bytes(g) // 8,), float("nan"), dtype=torch.float64, device="cuda")
        dth = torch.zeros(nj * nk, dtype=torch.float64, device="cuda")
        dra = torch.zeros(1, dtype=torch.float64, device="cuda")
        C.cavity_adjoint_step(g, prm, flat[0], flat[1], flat[2], ws, dth, dra)
        torch.cuda.synchronize()
        self.out, self.dth, self.dra = inner[2].cpu().numpy(), dth.cpu().numpy(), float(dra.cpu()[0])

    def tangent(self, dq=None, dtheta=None, dRa=0.0):
        """<lam, J v> and its absolute sum."""
        ni, nj, nk = self.n
        h = TG.H_STEP
        zq = self.q.astype(np.complex128)
        if dq is not None:
            self.P.interior(zq)[:] += 1j * h * dq
        zt = self.theta + (0j if dtheta is None else 1j * h * dtheta)
        Jv = TG.step(TG.Case(ni, nj, nk, complex(self.Ra, h * dRa), zt), zq).imag / h
        w = self.lam * Jv[:, 2:2 + nk, 2:2 + nj, 2:2 + ni]
        return float(w.sum()), float(np.abs(w).sum())


@pytest.mark.parametrize("Ra", [1e2, 1e6])
@pytest.mark.parametrize("n", [(2, 2, 2), (3, 2, 4), (4, 3, 2), (5, 4, 3)])
def test_every_entry_on_tiny_grids(C, n, Ra):
    s = Step(C, n, Ra, 3)
    want = np.zeros_like(s.lam)
    for m in np.ndindex(want.shape):
        e = np.zeros_like(want)
        e[m] = 1.0
        want[m] = s.tangent(dq=e)[0]
    print(n, Ra, np.abs(s.out - want).max() / np.abs(want).max(), flush=True)
    assert np.abs(s.out - want).max() <= 1e-12 * np.abs(want).max()
    wt = np.array([s.tangent(dtheta=np.eye(n[1] * n[2])[m])[0] for m in range(n[1] * n[2])])
    assert np.abs(s.dth - wt).max() <= 1e-12 * np.abs(wt).max()
    got, scale = s.tangent(dRa=Ra)
    assert abs(s.dra * Ra - got) <= 1e-11 * scale


@pytest.mark.parametrize("n", [(64, 8, 5), (65, 9, 7), (66, 16, 4), (63, 7, 9), (130, 18, 33)])
def test_tile_edges(C, n):
    s = Step(C, n, 1e5, 5)
    assert np.isfinite(s.out).all()
    rng = np.random.default_rng(6)
    dq = rng.uniform(-1, 1, s.lam.shape)
    dt = rng.uniform(-1, 1, n[1] * n[2])
    for got, kw in ((float((s.out * dq).sum()), dict(dq=dq)), (float(s.dth @ dt), dict(dtheta=dt)),
                    (s.dra * s.Ra, dict(dRa=s.Ra))):
        want, scale = s.tangent(**kw)
        assert abs(got - want) <= 1e-11 * scale, (kw.keys(), got, want, scale)
