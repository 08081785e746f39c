"""Local solves of 2-D boxes whose chains are longer than the row solves' LDS copy
(about 16,250 unknowns): slices of 4, 35 and 71 unknowns, 72 and 73 (the last that
is staged and the first that is not), in FP64 and FP32, against the oracle's direct
solves at a shift below the spectrum.  Tolerances as in the chain tests: FP64 1e-11
in relative 2-norm (sums in another order), FP32 factors 1e-5."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,ne,delta,nch", [
    (1, 5, 1, 4099), (3, 32, 2, 511), (2, 64, 8, 255), (2, 71, 2, 229), (2, 72, 2, 229)])
def test_long_chains(L, ne, delta, nch):
    import torch
    import paper_2311_08757_amd as dd
    from oracle.problem import Problem
    V, ell, sigma = W.sep_fourier(50 + ne), (nch + 1) / ne, -50.0
    P = Problem(W.small_config(1, 1, L, ne, delta, V, ell=ell), sigma=sigma, with_cell=False)
    r = W.random_vector(P.grid.n, 3)
    rd = torch.as_tensor(r, device="cuda")
    z = torch.empty_like(rd)
    ref = P.preconditioner(False).apply(r)
    for prec, tol in (("fp64", 1e-11), ("fp32", 1e-5)):
        prob = dd.assemble(1, 1, L, ne, V, delta, ell=ell, local_prec=prec, coarse=False)
        dd.set_shift(prob, sigma)
        dd.apply_schwarz(prob, "as1", rd, z)
        torch.cuda.synchronize()
        assert np.linalg.norm(z.cpu().numpy() - ref) <= tol * np.linalg.norm(ref), prec
