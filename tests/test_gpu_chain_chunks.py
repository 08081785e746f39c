"""The products of the FP32 chain solves in every form that their size rule picks:
K chunks of 72, 144 and 272 rows, 16- and 32-wide matrix tiles, and the bounds on
the partials that a right-hand side adds (4 or 9; 8 or 16; 8, 16 or 18).  One
application of the one-level preconditioner against the FP64 local solves of the
same problem.  Tolerance 1e-6 in relative 2-norm: operands rounded to 2^-24, FP32
sums of at most 72 products, whose roundings add up like sqrt(72) 2^-25 = 2.5e-7,
and FP64 sums of those; a step's error is not amplified by the next."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,ne,delta", [
    (1, 20, 1),   # 361 unknowns a slice: chunks of 72, 6 of them
    (1, 30, 1),   # 841: 12 chunks of 72
    (1, 35, 1),   # 1156: 17 chunks of 72
    (2, 32, 2),   # 1023: chunks of 144, 8 of them, 16-wide
    (20, 25, 4),  # 768, 18 members of a class: chunks of 144, 32-wide
    (1, 37, 1),   # 1296: 9 chunks of 144
    (4, 32, 2),   # 1085: 4 chunks of 272, 16-wide
    (20, 32, 2),  # the same, 32-wide
])
def test_product_forms(L, ne, delta):
    import torch
    import paper_2311_08757_amd as dd
    z = {}
    for prec in ("fp64", "fp32"):
        prob = dd.assemble(1, 2, L, ne, W.sep_fourier(7), delta, local_prec=prec, coarse=False)
        dd.cell_shift(prob)
        r = torch.as_tensor(W.random_vector(prob.n_dof, 13), device="cuda")
        z[prec] = torch.empty_like(r)
        dd.apply_schwarz(prob, "as1", r, z[prec])
    torch.cuda.synchronize()
    assert (z["fp32"] - z["fp64"]).norm() <= 1e-6 * z["fp64"].norm()
