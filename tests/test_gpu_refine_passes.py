"""Refinements whose evaluations differ in their passes over the draws: the
first evaluation (one point) and the later ones (eight) round a pass to slices of
different lengths, so at some draw counts only one of them makes all draws at
once.  The result does not depend on the passes or on what the workspace held."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2005_10494_amd as bmd  # noqa: E402
from paper_2005_10494_amd import workloads as W  # noqa: E402


@pytest.mark.parametrize("M", [700, 769, 832, 896, 960, 1100])
def test_refinement_twice_with_a_small_budget(M, monkeypatch):
    spec = W.base_problem(5, None, 0.3, 0.03, width=0.01, gh_nodes=24)
    q0 = [0.45, 0.5, 0.55, 0.5, 0.45]
    with bmd.Problem(spec) as p:
        want = p.refine_design(q0, M, "fp64", max_iter=3)
        monkeypatch.setenv("BMD_GRAD_BUDGET", str(1 << 20))
        for _ in range(2):   # the second finds the workspace of the first
            got = p.refine_design(q0, M, "fp64", max_iter=3)
            assert np.array_equal(got[0], want[0]) and got[1] == want[1] and got[2] == want[2]
