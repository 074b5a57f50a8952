"""Small calls: slices of 16 draws and the shared reduction of their sums, the
best design of surfaces on both sides of the one-workgroup limit, and smoothing
passes around the blocks of 32 rows that few columns load ahead."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import oracle as O  # noqa: E402
import paper_2005_10494_amd as bmd  # noqa: E402
from paper_2005_10494_amd import workloads as W  # noqa: E402


@pytest.mark.parametrize("m", [[1 + 16], [4, 4, 3]])
@pytest.mark.parametrize("M", [1, 16, 240, 241, 700])
def test_few_draws(m, M):
    """1, 15, 16 and 44 slices; a workgroup of the reduction holds 16 designs."""
    spec = W.base_problem(len(m), m, 0.0 if len(m) == 1 else 0.3, 0.05, seed=M)
    ref, var = O.eval_grid(spec, np.arange(O.grid_size(spec)), M)
    with bmd.Problem(spec) as p:
        mean, second = (x.cpu().numpy() for x in p.eval_grid(M, "fp64", want_var=True))
        again = p.eval_grid(M, "fp64").cpu().numpy()
    assert np.all(np.abs(mean - ref) <= 1e-9 * np.maximum(np.abs(ref), 1e-3))
    if M > 1:
        assert np.all(np.abs(second - var) <= 1e-9 * np.maximum(np.abs(var), 1e-3))
    assert np.array_equal(again, mean)


@pytest.mark.parametrize("n", [3, 1023, 1025, 16383, 16384, 16385, 40000])
def test_best_design(n):
    rng = np.random.default_rng(n)
    x = np.round(rng.standard_normal(n), 2)   # ties: the first wins
    x[rng.random(n) < 0.3] = np.nan
    x[n // 2] = x[np.nanargmax(x)] if not np.all(np.isnan(x)) else 1.0
    spec = W.base_problem(1, [n], 0.0, 0.05)
    with bmd.Problem(spec) as p:
        index, value, cell = p.argmax(torch.tensor(x, device="cuda"))
        assert index == np.nanargmax(x) and value == np.nanmax(x) and list(cell) == [index]
        index, value, _ = p.argmax(torch.full((n,), float("nan"), dtype=torch.float64, device="cuda"))
        assert index == 0 and np.isnan(value)


@pytest.mark.parametrize("m", [[31], [32], [33], [65], [100], [33, 64], [5, 40, 3]])
def test_smoothing_of_few_columns(m):
    """Bounds: sums of at most 100 products of positive weights that add up to
    one, in FP64 and with FP32 weights, values and sums."""
    spec = W.base_problem(len(m), m, 0.0 if len(m) == 1 else 0.3, 0.05)
    f = W.noisy_surface(tuple(m), seed=sum(m)).reshape(-1)
    ref = np.asarray(O.smooth_separable(spec, f)).reshape(-1)
    with bmd.Problem(spec) as p:
        x = torch.tensor(f, dtype=torch.float64, device="cuda")
        f64, f32 = (p.smooth(x, prec).cpu().numpy() for prec in ("fp64", "fp32"))
    scale = np.max(np.abs(f))
    assert np.max(np.abs(f64 - ref)) <= 1e-12 * scale
    assert np.max(np.abs(f32 - ref)) <= 2e-5 * scale
