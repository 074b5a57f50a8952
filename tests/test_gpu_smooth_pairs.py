"""FP64 smoothing of the last two axes in one pass: axis lengths around the blocks
of 16 and 4, odd and even numbers of axes, and the limits beyond which they go
one at a time.  Each result is a sum of at most
32 x 32 products of positive weights that add up to one; the bound is the other
smoothing tests' (1e-13)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import oracle as O  # noqa: E402
import paper_2005_10494_amd as bmd  # noqa: E402
from paper_2005_10494_amd import workloads as W  # noqa: E402


@pytest.mark.parametrize("m", [
    [4097, 3, 2], [260, 17, 16, 15], [19, 14, 16, 16, 17], [66, 64, 5, 31], [64, 65, 32, 32], [64, 65, 32, 33],
    [7, 5, 6, 4, 20, 1 + 20], [16, 25, 24, 13, 33], [13, 20, 30, 17, 16], [2, 40, 17, 9, 5, 13], [24, 25, 4, 4, 8, 8],
    [31, 20, 30, 16, 17],
])
def test_two_axes_at_a_time(m):
    spec = W.base_problem(len(m), m, 0.3, 0.05)
    f = W.noisy_surface(tuple(m), seed=sum(m)).reshape(-1)
    ref = np.asarray(O.smooth_separable(spec, f)).reshape(-1)
    with bmd.Problem(spec) as p:
        got = p.smooth(torch.tensor(f, dtype=torch.float64, device="cuda"), "fp64").cpu().numpy()
    assert np.max(np.abs(got - ref)) <= 1e-13
