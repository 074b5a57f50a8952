"""The gradient kernel at the shapes where its mapping changes: point counts
around the pairs a wavefront takes and the wavefronts of a workgroup (1, 2, 3,
4, 5, 9), draw counts around a wavefront and a slice, one to six biomarkers,
rules that switch a test off, and node counts up to the largest; against the
oracle (tolerances of the gradient parity tests: FP64 1e-7, FP32 2e-4 of
max(|g|, 1e-2); objective 1e-9 and 1e-5)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import oracle as O  # noqa: E402
import paper_2005_10494_amd as bmd  # noqa: E402
from paper_2005_10494_amd import workloads as W  # noqa: E402


def _check(spec, q, M):
    ref = O.grad_points(spec, q, M)
    with bmd.Problem(spec) as p:
        for prec, to, tg in (("fp64", 1e-9, 1e-7), ("fp32", 1e-5, 2e-4)):
            obj, gq, gmu = (t.cpu().numpy() for t in p.grad_design(q, M, prec))
            assert np.all(np.abs(obj - ref[0]) <= to * np.maximum(np.abs(ref[0]), 1e-3)), prec
            assert np.all(np.abs(gq - ref[1]) <= tg * np.maximum(np.abs(ref[1]), 1e-2)), prec
            assert np.all(np.abs(gmu - ref[2]) <= tg * np.maximum(np.abs(ref[2]), 1e-2)), prec


@pytest.mark.parametrize("B,M", [(1, 1), (2, 63), (3, 65), (4, 128), (5, 257), (9, 300)])
@pytest.mark.parametrize("d,width", [(1, 0.01), (2, 0.0), (3, 0.02), (6, 0.01)])
def test_point_and_draw_counts(B, M, d, width):
    spec = W.base_problem(d, None, 0.0 if d == 1 else 0.3, 0.03, width=width, seed=B)
    _check(spec, W.design_points(B, d, seed=M), M)


@pytest.mark.parametrize("kw", [dict(alpha_rule="bonferroni"), dict(alpha_rule="fixed", alpha_fixed=(0.02, 0.0)),
                                dict(alpha_rule="fixed", alpha_fixed=(0.0, 0.02)), dict(gh_nodes=128),
                                dict(gh_nodes=4, rho_b=0.0)])   # any rule is exact for independent biomarkers
def test_rules_and_node_counts(kw):
    kw = dict(kw)
    spec = W.base_problem(4, None, kw.pop("rho_b", 0.2), 0.03, width=0.01, seed=5, **kw)
    _check(spec, W.design_points(6, 4, seed=3), 200)


def test_repeat_and_order_of_points():
    """The same points in another order and number give the same values."""
    spec = W.base_problem(5, None, 0.3, 0.03, width=0.01, seed=1)
    q = W.design_points(11, 5, seed=2)
    with bmd.Problem(spec) as p:
        a = p.grad_design(q, 1000, "fp64")
        b = p.grad_design(q[::-1].copy(), 1000, "fp64")
        c = p.grad_design(q[4:6].copy(), 1000, "fp64")
    for x, y, z in zip(a, b, c):
        assert torch.equal(x, torch.flip(y, [0]))
        assert torch.allclose(x[4:6], z, rtol=1e-12, atol=1e-15)   # other slices


def test_many_points_share_a_wavefront():
    """Beyond 2,048 points a point's setup takes 16 lanes in place of 64."""
    spec = W.base_problem(3, None, 0.3, 0.03, width=0.01, seed=4)
    q = W.design_points(2051, 3, seed=6)
    with bmd.Problem(spec) as p:
        many = p.grad_design(q, 70, "fp64")
        few = p.grad_design(q[-7:].copy(), 70, "fp64")
    for x, y in zip(many, few):
        assert torch.allclose(x[-7:], y, rtol=1e-12, atol=1e-14)
    _check(spec, q[::293].copy(), 70)
