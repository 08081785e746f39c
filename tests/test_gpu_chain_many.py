"""FP32 chain solves of more subdomains than a launch has workgroups along its
second axis (65,535; a slot per subdomain and chain end): a long strip of small
3-D boxes, 33,000 cells with n_e = 3.  One application of the one-level
preconditioner against the FP64 local solves of the same problem: FP32 factors
(2^-24 per entry, sums of a few tens of terms, two sweeps) 1e-5 in relative
2-norm, on the whole vector and on the last subdomains alone."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def test_more_slots_than_grid_rows():
    import torch
    import paper_2311_08757_amd as dd
    L, ne = 33000, 3
    z = {}
    for prec in ("fp64", "fp32"):
        prob = dd.assemble(1, 2, L, ne, W.sep_fourier(5), 1, local_prec=prec, coarse=False)
        dd.cell_shift(prob)
        r = torch.as_tensor(W.random_vector(prob.n_dof, 9), device="cuda")
        z[prec] = torch.empty_like(r)
        dd.apply_schwarz(prob, "as1", r, z[prec])
    torch.cuda.synchronize()
    d, ref = (z[p].reshape(2, 2, -1) for p in ("fp32", "fp64"))  # the strip runs along the last axis
    d = d - ref
    assert d.norm() <= 1e-5 * ref.norm()
    assert d[..., -100 * ne:].norm() <= 1e-5 * ref[..., -100 * ne:].norm()
