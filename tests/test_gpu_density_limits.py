"""Derivatives at arguments far outside any table or range: effects so large that
every density is zero give zero derivatives (the oracle's, exactly), and a logistic
indicator of vanishing width is the exact indicator."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import oracle as O  # noqa: E402
import paper_2005_10494_amd as bmd  # noqa: E402
from paper_2005_10494_amd import workloads as W  # noqa: E402

RULES = [dict(alpha_rule="fwer"), dict(alpha_rule="fixed", alpha_fixed=(0.02, 0.0)), dict(alpha_rule="split", alpha_fixed=(0.01, 0.0))]


@pytest.mark.parametrize("effect", [1e22, -1e40, 1e100])
@pytest.mark.parametrize("rule", RULES, ids=lambda r: r["alpha_rule"])
@pytest.mark.parametrize("d", [1, 3])
def test_huge_effects(d, rule, effect):
    spec = W.base_problem(d, [4] * d, 0.0 if d == 1 else 0.3, 0.05, mu_b0=effect, sd_b0=0.0, mu_b1=-3.0 * effect, sd_b1=0.0, **rule)
    with bmd.Problem(spec) as p:
        obj, gq, gmu = (t.cpu().numpy() for t in p.grad_design(W.design_points(3, d, seed=1), 65, "fp64"))
        assert np.all(gq == 0.0) and np.all(gmu == 0.0) and np.all((obj >= 0.0) & (obj <= 1.0))
        if rule["alpha_rule"] != "fwer":
            assert np.all(p.eval_grid_dalpha(65, "fp64")[1].cpu().numpy() == 0.0)
            assert np.all(O.eval_grid_dalpha(spec, np.arange(4 ** d), 65)[1] == 0.0)


@pytest.mark.parametrize("width", [1e-12, 1e-60, 1e-300])
def test_vanishing_width(width):
    q = W.design_points(5, 2, seed=1)
    out = []
    for w in (0.0, width):
        with bmd.Problem(W.base_problem(2, None, 0.3, 0.05, width=w)) as p:
            out.append([t.cpu().numpy() for t in p.grad_design(q, 500, "fp64")])
    for sharp, got in zip(*out):
        assert np.allclose(got, sharp, rtol=1e-12, atol=1e-14)
