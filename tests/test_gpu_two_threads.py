"""Two problems on two threads whose local solves run in one kernel with different
amounts of LDS (slices of 63 unknowns, chains of 255 lines and of three): every
application gives the bits it gives alone."""
import threading

import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def test_applications_on_two_threads():
    import torch
    import paper_2311_08757_amd as dd
    ne = 60
    jobs = []
    for nch in (255, 3):
        prob = dd.assemble(1, 1, 3, ne, W.sep_fourier(nch), 2, ell=(nch + 1) / ne,
                           stream=torch.cuda.Stream())
        dd.cell_shift(prob)
        r = torch.as_tensor(W.random_vector(prob.n_dof, nch), device="cuda")
        ref, z = torch.empty_like(r), torch.empty_like(r)
        torch.cuda.synchronize()
        dd.apply_schwarz(prob, "as2", r, ref)
        jobs.append((prob, r, ref, z))
    torch.cuda.synchronize()
    errors = []

    def work(prob, r, ref, z):
        try:
            for _ in range(200):
                dd.apply_schwarz(prob, "as2", r, z)
            torch.cuda.synchronize()
            if not torch.equal(z, ref):
                errors.append("another result")
        except Exception as e:  # reported by the test's thread
            errors.append(repr(e))

    threads = [threading.Thread(target=work, args=j) for j in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
