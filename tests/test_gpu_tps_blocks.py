"""Thin-plate fits whose reduced system ends at, before and after the edges of
the Cholesky factor's blocks of 64 (and, inside the first, of 16), against the
oracle's direct solution: the bound of the other surface tests, 1e-9 of
max |f|."""
import numpy as np
import pytest

import oracle as O
from paper_2005_10494_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2005_10494_amd as bmd  # noqa: E402


@pytest.mark.parametrize("rows", [1, 2, 15, 16, 17, 62, 63, 64, 65, 79, 80, 81, 127, 128, 129, 191, 192, 193, 256, 257])
def test_reduced_system_sizes(rows):
    """One dimension: the reduced system has two rows fewer than designs."""
    m = rows + 2
    spec = W.base_problem(1, [m], 0.0, 0.05)
    f = W.noisy_surface((m,), seed=rows)
    with bmd.Problem(spec) as p:
        s, n = p.smooth_tps(torch.tensor(f, dtype=torch.float64, device="cuda"), 1e-3)
        s = s.cpu().numpy()
    assert n == m
    assert np.max(np.abs(s - O.smooth_tps(spec, f, 1e-3))) <= 1e-9 * np.max(np.abs(f))


@pytest.mark.parametrize("seed", [0, 2, 10, 11, 21, 23, 36, 38])
def test_refinement_ends_at_the_maximum(seed):
    """The step Newton would still take at the returned design: the gradient's
    rounding (1e-10) over the curvature (1e5), with a margin; steps of 1e-10
    were left where the value's own rounding decided on the last one."""
    spec = W.base_problem(2, [45, 45], 0.3, 0.05)
    f = W.noisy_surface((45, 45), seed=seed)
    with bmd.Problem(spec) as p:
        fit, _ = p.smooth_tps(torch.tensor(f, dtype=torch.float64, device="cuda"), 1e-4)
        _, best, cell = p.argmax(fit)
        lo, hi = p.spec["q_lo"], p.spec["q_hi"]
        q0 = [lo + (hi - lo) * i / 44 for i in cell]
        q, v, _ = p.refine_tps(q0)
        _, g, H = p.tps_at(q)
    assert v >= best - 1e-12
    g, H, q = np.asarray(g), np.asarray(H), np.asarray(q)
    if np.all((q > lo) & (q < hi)):
        assert np.max(np.abs(np.linalg.solve(H, g))) <= 1e-12
