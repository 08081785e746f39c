"""The grouped GEMM with the K splits folded into one tile: a batch whose
128-column tiles fill the chip without the split (256 tiles) sums the split
partials in registers, in the order the extension would add them, so every
instance's PCG iterate equals bit for bit the one of a batch that holds this
instance alone, whose few tiles stay split."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _probs(prec, n, L_last):
    import paper_2311_08757_amd as dd
    probs = []
    for j in range(n):
        L = L_last if j == n - 1 else 5 + j % 5
        prob = dd.assemble(1, 1, L, 32, W.sep_fourier(900 + j), 2, local_prec=prec)
        dd.cell_shift(prob)
        probs.append(prob)
    return probs


def _solve(torch, probs, bs, tile64):
    import paper_2311_08757_amd as dd
    batch = dd.batch_create(probs, reproducible=True, tile64=tile64)
    q = dd.batch_query(batch)
    assert q["ksplit"] == 3
    xs = [torch.zeros_like(b) for b in bs]
    st, info = dd.batch_pcg_solve(batch, bs, xs, rtol=1e-10, maxit=500)
    assert st == "OK"
    return q["ntiles"], xs, [i["iters"] for i in info]


# the unclipped box has 35 x 31 = 1085 unknowns: nine column tiles each, so 28
# instances of at most 128 subdomains are 252 tiles (split), 29 are 261 (folded);
# the last instance's 130 subdomains take a second row tile
@pytest.mark.parametrize("prec", ["bf16", "bf16x3"])
@pytest.mark.parametrize("n,L_last,tiles", [(28, 7, 252 * 3), (29, 7, 261), (28, 130, 261)])
def test_folded_splits_bitwise(prec, n, L_last, tiles):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    probs = _probs(prec, n, L_last)
    bs = [torch.as_tensor(W.random_vector(p.n_dof, 60 + j), dtype=torch.float64, device="cuda")
          for j, p in enumerate(probs)]
    for tile64 in (False, True):
        nt, xs, its = _solve(torch, probs, bs, tile64)
        if not tile64:
            assert nt == tiles
        for j in list(range(5)) + [n - 1]:
            nt1, (x1,), (it1,) = _solve(torch, [probs[j]], [bs[j]], tile64)
            assert nt1 % 27 == 0       # nine column tiles, three splits
            assert its[j] == it1 and torch.equal(xs[j], x1), (tile64, j)
