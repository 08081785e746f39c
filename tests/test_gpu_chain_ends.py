"""Row solves that eliminate a 2-D box's chain from both ends: chains of one to
seven lines (one line and two have no half on one side or either; an even count
leaves the mirrored half a step without a slice), at slices that use one wave of
rows and five, and the dense inverse formed from their identity columns.
Tolerances as in the chain tests of the other slice sizes."""
import pytest

import workloads as W
from test_gpu_chain import _check, torch  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nch", [1, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("ne,delta", [(8, 2), (70, 5)])
def test_chain_lengths(torch, nch, ne, delta):  # noqa: F811
    _check(torch, 1, 1, 3, ne, delta, (nch + 1) / ne, W.sep_fourier(20 + nch),
           [("fp64", 1e-11), ("fp32", 1e-5), ("bf16x3", 1e-3)])
