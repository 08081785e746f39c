"""Chain factorisation and solves of boxes at the edges of their kernels: slice
sizes around every register and thread tile (one workgroup per class up to 128
unknowns a slice, pivot blocks of 32 above), the row solves' part sizes, chains
too long for their LDS copy, and 3-D slices.  Thin strips (three lines) keep
the oracle cheap.

Tolerances as in the parity tests: FP64 applications 1e-11 in relative 2-norm
(sums in another order), cell shift 1e-12 and 1e-9; FP32 factors 1e-5 (2^-24
per entry, sums of a few hundred FP64 terms, two sweeps); hi/lo bf16 dense
inverses 1e-3 (operands to 2^-17, FP32 accumulation, and the clipped classes'
correction).
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

# ne, delta: interior slices of b = ne + 2 delta - 1 unknowns
SLICES = [(3, 1), (9, 4), (16, 1), (31, 1), (32, 1), (40, 1), (47, 1), (48, 1), (55, 1), (63, 1),
          (64, 1), (71, 1), (72, 1), (79, 1), (80, 1), (95, 1), (96, 1), (127, 1), (128, 1), (159, 1)]


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.skip("no GPU")
    return _t


def _check(torch, p, q, L, ne, delta, ell, V, precs):
    import paper_2311_08757_amd as dd
    from oracle.problem import Problem
    P = Problem(W.small_config(p, q, L, ne, delta, V, ell=ell))
    r = W.random_vector(P.grid.n, 3)
    rd = torch.as_tensor(r, device="cuda")
    z = torch.empty_like(rd)
    ref = P.preconditioner(False).apply(r)
    for prec, tol in precs:
        prob = dd.assemble(p, q, L, ne, V, delta, ell=ell, local_prec=prec)
        sigma, psi = dd.cell_shift(prob)
        assert abs(sigma - P.sigma) <= 1e-12 * max(abs(P.sigma), 1.0)
        d = psi - P.cell["psi"]
        assert np.sqrt(d @ (P.cell["M"] @ d)) <= 1e-9
        dd.set_shift(prob, P.sigma, P.cell["psi"])
        dd.apply_schwarz(prob, "as1", rd, z)
        torch.cuda.synchronize()
        assert np.linalg.norm(z.cpu().numpy() - ref) <= tol * np.linalg.norm(ref), prec


@pytest.mark.parametrize("ne,delta", SLICES)
def test_slice_sizes(torch, ne, delta):
    _check(torch, 1, 1, 5, ne, delta, 4 / ne, W.sep_fourier(40 + ne),
           [("fp64", 1e-11), ("fp32", 1e-5), ("bf16x3", 1e-3)])


@pytest.mark.parametrize("p,q,L,ne,delta,ell", [
    (1, 1, 2, 62, 1, 260 / 62),   # 63 x 259: longer than the LDS copy of the row solves
    (2, 1, 3, 11, 1, 4 / 11),     # slices of 12 x 12 and 11 x 11 in four clipped classes
    (1, 2, 3, 12, 1, 1),          # 13 x 11
    (1, 1, 1, 5, 1, 2 / 5),       # one line, one subdomain
])
def test_boxes(torch, p, q, L, ne, delta, ell):
    V = W.sep_fourier(7) if p == 1 else W.fourier2(8)
    _check(torch, p, q, L, ne, delta, ell, V, [("fp64", 1e-11), ("fp32", 1e-5)]
           + ([("bf16x3", 1e-3)] if p == 2 else []))
