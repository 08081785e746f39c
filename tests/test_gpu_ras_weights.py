"""Distance-based weights with two expanding axes, which are not a product over the
axes: overlaps of two and three layers (with one they equal the equal weights),
nodes of one, two and four subdomains, and a single subdomain.  Tolerances as in
the parity tests of the restricted preconditioners: FP64 local solves 1e-11 in
relative 2-norm (sums in another order), hi/lo bf16 dense inverses 1e-3."""
import numpy as np
import pytest

import workloads as W
from test_gpu_ras import _dev, _oracle, _oracle_prec, _prob, torch  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu

CASES = [(2, 1, 4, 5, 2), (2, 1, 2, 6, 3), (2, 1, 1, 5, 2)]


@pytest.mark.parametrize("kind", ["as2", "ras1", "ras2"])
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-11), ("bf16x3", 1e-3)])
@pytest.mark.parametrize("case", CASES)
def test_distance_weights_on_two_axes(torch, case, prec, tol, kind):  # noqa: F811
    import paper_2311_08757_amd as dd
    case = case + (W.fourier2(4000),)
    P = _oracle(case, "distance")
    prob = _prob(case, P, pu="distance", local_prec=prec)
    r = W.random_vector(P.grid.n, 11)
    z = torch.empty(P.grid.n, dtype=torch.float64, device="cuda")
    dd.apply_schwarz(prob, kind, _dev(torch, r), z)
    torch.cuda.synchronize()
    zr = _oracle_prec(P, kind)(r)
    assert np.linalg.norm(z.cpu().numpy() - zr) <= tol * np.linalg.norm(zr)
