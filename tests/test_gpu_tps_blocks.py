"""Thin-plate fits whose reduced system ends at, before and after the edges of
the Cholesky factor's blocks of 32 and the update's tiles of 64 (whose launches
carry the forward solve), against the oracle's direct solution: the bound of the
other surface tests, 1e-9 of max |f|."""
import numpy as np
import pytest

import oracle as O
from paper_2005_10494_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2005_10494_amd as bmd  # noqa: E402


@pytest.mark.parametrize("rows", [1, 2, 15, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 160, 161, 257])
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
