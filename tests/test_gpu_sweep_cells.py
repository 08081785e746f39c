"""The 2-D tile sweep with strides of whole cells (n_e <= 64 not dividing 64) and
the general sweep above: apply and the fused direction update against the
oracle, at widths of a part of a tile, whole tiles and a remainder, and at both
tile heights.  Tolerances as in the parity tests (1e-13 of ||A|| ||x||; true CG
residual below 1.1 rtol)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.skip("no GPU")
    return _t


@pytest.mark.parametrize("ne,L,delta,ell", [
    (3, 1, 1, 1), (3, 90, 1, 1), (5, 49, 1, 2), (7, 36, 2, 9 / 7), (30, 8, 3, 1), (30, 17, 2, 0.3),
    (33, 4, 3, 5 / 33), (33, 9, 3, 12 / 33), (48, 13, 4, 0.25), (63, 5, 4, 10 / 63),
    (65, 5, 4, 6 / 65), (12, 1100, 1, 3.5)])
def test_cell_strides(torch, ne, L, delta, ell):
    import paper_2311_08757_amd as dd
    from oracle.problem import Problem
    V = W.sep_fourier(60 + ne)
    P = Problem(W.small_config(1, 1, L, ne, delta, V, ell=ell))
    prob = dd.assemble(1, 1, L, ne, V, delta, ell=ell)
    x = W.random_vector(P.grid.n, 5)
    xd = torch.as_tensor(x, device="cuda")
    y = torch.empty_like(xd)
    for name, A in (("M", P.M), ("A", P.A)):
        dd.apply_op(prob, name, xd, y)
        torch.cuda.synchronize()
        tol = 1e-13 * abs(A).sum(axis=1).max() * np.abs(x).max()
        assert np.abs(y.cpu().numpy() - A @ x).max() <= tol, name
    if P.grid.n > 100000:
        return
    dd.set_shift(prob, P.sigma, P.cell["psi"])
    u = torch.zeros_like(xd)
    dd.pcg_solve(prob, xd, u, rtol=1e-10, maxit=500)
    assert np.linalg.norm(x - P.A_sigma @ u.cpu().numpy()) <= 1.1e-10 * np.linalg.norm(x)
