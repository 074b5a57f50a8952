"""bmd_eval_grid_noalloc just below its scratch: FP64 sweeps whose workspace fits
with the slices of one workgroup a compute unit (eight rounds of them), and not
with those of two, as for the kernels that hold two."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2005_10494_amd as bmd  # noqa: E402
from paper_2005_10494_amd import workloads as W  # noqa: E402

SCRATCH = 128 << 20


def _need(p, M, workgroups):
    """Workspace of M draws with slices of `workgroups` workgroups a compute unit."""
    al = lambda b: -(-b // 256) * 256  # noqa: E731
    K, tiles = bmd.gh_nodes(p, "fp64"), -(-p.G // 256)
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    n = min(-(-8 * cu * workgroups // tiles), -(-M // 64))
    n = -(-M // -(-M // n))
    return (9 * al(8 * M) + al(4 * p.d * M) + al(32 * M) + al(8 * p.d * M) + al(8 * M * p.d * K)) + 16 * p.G * n


@pytest.mark.parametrize("spec", [W.nested4_design(5), W.alpha4_design(6),
                                  W.base_problem(6, [3] * 6, 0.3, 0.03, width=0.01, gh_nodes=4)],
                         ids=["nested4", "alpha4", "logistic6"])
def test_sweeps_that_fitted_still_fit(spec):
    with bmd.Problem(spec) as p:
        hi = SCRATCH // 100
        M = max(m for m in range(1000, hi, 50) if _need(p, m, 1) <= SCRATCH)
        assert _need(p, M, 2) > SCRATCH   # the case is met
        got = p.eval_grid(M, "fp64", noalloc=True)
        assert torch.equal(torch.nan_to_num(got, nan=-1.0), torch.nan_to_num(p.eval_grid(M, "fp64"), nan=-1.0))
