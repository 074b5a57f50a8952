"""The two-layer counts from ranks and bit sets at the sizes where they can go
wrong: outer groups that end inside a wavefront's 64 draws, a last partial
block of draws, a chunk of 512 inner draws over two inner groups, designs
that share fractions in runs (levels fixed, rows of an (r_2, alpha_1) grid) or
not at all, and outer counts on both sides of the rule that picks the
kernel.  Counts are whole numbers: FP64 equals the oracle's bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import oracle as O  # noqa: E402
import paper_2005_10494_amd as bmd  # noqa: E402
from paper_2005_10494_amd import workloads as W  # noqa: E402


def _spec(name):
    return {
        "alpha": lambda: W.alpha_design(21),
        "alpha_rows": lambda: W.alpha_design(19, m_r=3),
        "alpha3": lambda: W.alpha3_design(6),
        "alpha4": lambda: W.alpha4_design(4),
        "cutoff": lambda: W.base_problem(1, [5], 0.0, 0.05, info=211.0, effect="paper", paper_a=0.3, paper_b=0.1),
        "one_test": lambda: W.base_problem(1, [5], 0.0, 0.05, info=211.0, effect="paper", paper_a=0.3, paper_b=0.1,
                                           alpha_rule="fixed", alpha_fixed=(0.01, 0.0)),
    }[name]()


@pytest.mark.parametrize("name", ["alpha", "alpha_rows", "alpha3", "alpha4", "cutoff", "one_test"])
@pytest.mark.parametrize("sizes", [(4104, 1024, 8, 4), (4128, 3072, 16, 4), (4096, 2048, 2, 8), (4088, 1024, 8, 2),
                                   (2, 1024, 2, 4)])
def test_counts_equal_the_oracle(name, sizes):
    N1, N2, A, B = sizes
    spec = _spec(name)
    G = O.grid_size(spec)
    ref_m, ref_v, _ = O.eval_grid_two_layer(spec, np.arange(G), N1, N2, A, B)
    with bmd.Problem(spec) as p:
        m, v = (t.cpu().numpy() for t in p.eval_grid_two_layer(N1, N2, "fp64", (A, B)))
        m32 = p.eval_grid_two_layer(N1, N2, "fp32", (A, B))[0].cpu().numpy()
    nan = np.isnan(ref_m)
    assert np.array_equal(np.isnan(m), nan) and np.array_equal(np.isnan(m32), nan)
    assert np.array_equal(m[~nan], ref_m[~nan])
    assert np.allclose(v[~nan], ref_v[~nan], rtol=1e-12, atol=1e-18)
    assert np.all(np.abs(m32 - ref_m)[~nan] <= 1e-5 * np.maximum(ref_m[~nan], 1e-3))


@pytest.mark.parametrize("spec", [W.alpha3_design(12), W.alpha_design(20, m_r=8), W.alpha4_design(5)],
                         ids=["alpha3", "alpha_rows", "alpha4"])
def test_groups_of_designs_equal_the_oracle(spec):
    """Several designs to a workgroup (4 of 144, 5 of rows of 20, 4 of 125)."""
    N1, N2, A, B = 1032, 16384, 8, 16
    if spec["design"] == "alpha4":
        N2 = 32768
    G = O.grid_size(spec)
    with bmd.Problem(spec) as p:
        m, v = (t.cpu().numpy() for t in p.eval_grid_two_layer(N1, N2, "fp64", (A, B)))
        again = p.eval_grid_two_layer(N1, N2, "fp64", (A, B))[0].cpu().numpy()
    gs = np.unique(np.linspace(0, G - 1, 13).astype(int))
    ref_m, ref_v, _ = O.eval_grid_two_layer(spec, gs, N1, N2, A, B)
    ok = ~np.isnan(ref_m)
    assert np.array_equal(np.isnan(m[gs]), ~ok) and np.array_equal(m, again, equal_nan=True)
    assert np.array_equal(m[gs][ok], ref_m[ok])
    assert np.allclose(v[gs][ok], ref_v[ok], rtol=1e-12, atol=1e-18)
