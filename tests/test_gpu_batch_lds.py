"""Batches whose tuned settings come from problems of fewer nodes: the draws per
LDS chunk chosen there may not leave room for the FP64 kernel's own table beside a
chunk of more nodes; the plan takes a smaller one, the means stay."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2005_10494_amd as bmd  # noqa: E402
from paper_2005_10494_amd import workloads as W  # noqa: E402


def test_tuned_chunk_beside_the_table():
    d, table = 6, 545 * 16
    specs = [W.base_problem(d, [2, 3, 2, 3, 2, 3], 0.3, 0.03, gh_nodes=k, scenario=k) for k in range(4, 132, 4)]
    try:
        bmd.batch_autotune(2)
        bmd.batch_autotune(1)
        with bmd.Problem(specs[0]) as p:
            bmd.eval_batch([p], [4000], "fp64")
            chunk = bmd.batch_settings("fp64", d, 1)["chunk"]
        lds = [8 * chunk * (256 + d * s["gh_nodes"] + 8) + 4 * chunk * d for s in specs]
        met = [s for s, b in zip(specs, lds) if (64 << 10) - table < b <= (64 << 10)]
        assert met or chunk in (0, 4)   # a chunk of four draws always fits
        for s in met[:2]:
            with bmd.Problem(s) as p:
                got = bmd.eval_batch([p], [777], "fp64")[0][0]
                assert (got - p.eval_grid(777, "fp64")).abs().max().item() <= 1e-12
    finally:
        bmd.batch_autotune(2)
        bmd.batch_autotune(1)
