"""The dense GEMM's 64-row tiles, taken while they fit one to a CU, against its
128-row tiles: each output sums the same K stages in the same order, so PCG with
the single problem's GEMM (64 rows here) equals PCG in a reproducible batch of
one (128 rows) bit for bit, at subdomain counts around the tile edges.  Above
256 nodes per line the two paths cut the partials of their dot products
differently: iterates to 1e-8 relative there, as in the other batch tests."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["bf16", "bf16x3"])
@pytest.mark.parametrize("L,ne,delta", [(5, 4, 2), (63, 4, 2), (64, 4, 1), (65, 4, 2), (129, 4, 1)])
def test_tile_rows(prec, L, ne, delta):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2311_08757_amd as dd
    prob = dd.assemble(1, 1, L, ne, W.sep_fourier(70 + L), delta, local_prec=prec)
    dd.cell_shift(prob)
    b = torch.as_tensor(W.random_vector(prob.n_dof, L), dtype=torch.float64, device="cuda")
    x1 = torch.zeros_like(b)
    out = dd.pcg_solve(prob, b, x1, rtol=1e-10, maxit=500)
    batch = dd.batch_create([prob], reproducible=True)
    assert dd.batch_query(batch)["tile_rows"] == 128
    x2 = torch.zeros_like(b)
    st, info = dd.batch_pcg_solve(batch, [b], [x2], rtol=1e-10, maxit=500)
    assert st == "OK"
    if L * ne - 1 <= 256:
        assert info[0]["iters"] == out["iters"] and torch.equal(x1, x2)
    else:
        assert abs(info[0]["iters"] - out["iters"]) <= 2
        assert float((x1 - x2).abs().max()) <= 1e-8 * float(x1.abs().max())
