"""Points on both sides of the line from which a point's setup takes 16 lanes in
place of 64 (one workgroup of four points per compute unit): the same values to
the order of the setup's sums (a few ulp; 1e-12 relative, 1e-14 absolute)."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2005_10494_amd as bmd  # noqa: E402
from paper_2005_10494_amd import workloads as W  # noqa: E402


@pytest.mark.parametrize("d", [1, 4])
def test_lanes_per_point(d):
    edge = 4 * torch.cuda.get_device_properties(0).multi_processor_count
    spec = W.base_problem(d, None, 0.0 if d == 1 else 0.3, 0.03, width=0.01, seed=2)
    q = W.design_points(edge + 1, d, seed=3)
    with bmd.Problem(spec) as p:
        few = p.grad_design(q[:edge].copy(), 70, "fp64")
        many = p.grad_design(q, 70, "fp64")
    for x, y in zip(few, many):
        assert torch.allclose(x, y[:edge], rtol=1e-12, atol=1e-14)
