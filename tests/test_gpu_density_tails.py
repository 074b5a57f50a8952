"""Derivatives where the power saturates: their terms are a density times a
normal probability deep in the lower tail (at -6 and at -9 here), so the digits
of that probability are digits of the result.  Point-mass priors; relative error
against the oracle.  Bound: the arguments h and k (20 at most) carry a few units
in the last place (4e-14), which a factor of their size magnifies to 1e-12 of a
density or a tail; 1e-10 allows for a hundred times that.  The second level of
rule "split" is a root found to 1e-12 on either side: 1e-9."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import oracle as O  # noqa: E402
import paper_2005_10494_amd as bmd  # noqa: E402
from paper_2005_10494_amd import workloads as W  # noqa: E402

STRONG = [(0.9, 1.4), (1.3, 2.0)]


def _spec(d, m, effect, **kw):
    return W.base_problem(d, m, 0.0, 0.05, mu_b0=effect[0], sd_b0=0.0, mu_b1=effect[1], sd_b1=0.0, tau_lo=0.5, tau_hi=0.5,
                          **kw)


@pytest.mark.parametrize("effect", STRONG)
@pytest.mark.parametrize("d", [1, 2])
def test_gradient_of_a_saturated_power(d, effect):
    spec = _spec(d, None, effect, alpha_rule="bonferroni", width=0.01)
    q = np.full((3, d), 0.5) + 0.02 * np.arange(3)[:, None]
    ref = O.grad_points(spec, q, 3)[2]
    with bmd.Problem(spec) as p:
        gmu = p.grad_design(q, 3, "fp64")[2].cpu().numpy()
    assert np.all(ref > 0.0) and np.all(ref < 1e-20)
    assert np.all(np.abs(gmu - ref) <= 1e-10 * ref), (gmu, ref)


@pytest.mark.parametrize("effect", STRONG)
@pytest.mark.parametrize("d,m", [(1, [19]), (2, [5, 7])])
@pytest.mark.parametrize("rule,levels,tol", [("fixed", (0.0125, 0.0125), 1e-10), ("split", (0.0125, 0.0), 1e-9)])
def test_level_derivative_of_a_saturated_power(d, m, effect, rule, levels, tol):
    spec = _spec(d, m, effect, alpha_rule=rule, alpha_fixed=levels)
    ref = O.eval_grid_dalpha(spec, np.arange(O.grid_size(spec)), 3)[1]
    with bmd.Problem(spec) as p:
        got = p.eval_grid_dalpha(3, "fp64")[1].cpu().numpy()
    # "split": the two levels' terms have opposite signs; designs where they cancel are left out
    used = np.abs(ref) > (1e-300 if rule == "fixed" else 0.1 * np.median(np.abs(ref)))
    assert used.sum() >= 5
    assert np.all(np.abs(got - ref)[used] <= tol * np.abs(ref)[used]), (got, ref)
