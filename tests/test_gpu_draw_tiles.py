"""Prior draws by tiles of at most 32: draw counts around a tile and node
tables that shrink it (K = 128 nodes, six biomarkers: 4 draws a tile), through
the sweeps and the batch, against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import oracle as O  # noqa: E402
import paper_2005_10494_amd as bmd  # noqa: E402
from paper_2005_10494_amd import workloads as W  # noqa: E402


@pytest.mark.parametrize("d,m,K", [(1, [5], 0), (2, [4, 3], 0), (3, [3, 2, 3], 64), (6, [2] * 6, 128)])
@pytest.mark.parametrize("M", [1, 31, 33, 70])
def test_sweep_draw_counts_around_a_tile(d, m, K, M):
    spec = W.base_problem(d, m, 0.0 if d == 1 else 0.3, 0.05, gh_nodes=K, seed=9 + M)
    ref, _ = O.eval_grid(spec, np.arange(O.grid_size(spec)), M)
    with bmd.Problem(spec) as p:
        f64, f32 = (p.eval_grid(M, prec).cpu().numpy() for prec in ("fp64", "fp32"))
        bat = bmd.eval_batch([p, p], [M, M + 5], "fp64")[0][0].cpu().numpy()
    assert np.all(np.abs(f64 - ref) <= 1e-9 * np.maximum(np.abs(ref), 1e-3))
    assert np.all(np.abs(f32 - ref) <= 1e-5 * np.maximum(np.abs(ref), 1e-3))
    assert np.allclose(bat, f64, rtol=1e-13, atol=0)
