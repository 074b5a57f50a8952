"""The FP64 integrands' own 2^x and normal CDF, replayed on the CPU in double
precision (their fused multiply-adds rounded once) against 40-digit values, and
the sweeps that use them at draw counts around the two draws they take at a
time, against the oracle.

Tolerances.  2^f = 1 + f Q(f): the polynomial is within 2e-17 and Horner's last
fused multiply-add rounds once, half an ulp of a value in [0.7, 1.42): at most
1.6e-16 relative.  Phi from the table: a cell's F is within one ulp of a value
below 1/2 (5.6e-17 with erf's own ulp), the series' last multiply-add rounds
once more (2.8e-17 to 5.6e-17), the final addition of 1/2 once (5.6e-17 below
1/2, 1.1e-16 above): below 2.5e-16 absolute."""
import importlib.util
import os
import re

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2005_10494_amd", "csrc")
mp = pytest.importorskip("mpmath")


def _generator():
    spec = importlib.util.spec_from_file_location("gen_exp2", os.path.join(CSRC, "gen_exp2_fit.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def test_exp2_header_and_error():
    gen = _generator()
    text = open(os.path.join(CSRC, "exp2_fit.hpp")).read()
    vals = [float.fromhex(v) for v in re.findall(r"^    (-?0x[0-9a-f.]+p[-+]\d+),", text, re.M)]
    assert vals == gen.fit()   # the header is the generator's output
    poly, evald = gen.errors(vals, 801)
    assert poly <= 2e-17 and evald <= 1.6e-16


def _fma(a, b, c):
    return float(mp.mpf(a) * mp.mpf(b) + mp.mpf(c))


def _cdf_table(x):
    """norm_cdf_table(x) of device_math.hpp, operation by operation."""
    y = min(abs(x), 8.5)
    k = 6755399441055744.0 / 64
    s = y + k
    xj = s - k
    F = float(mp.erf(mp.mpf(xj) / mp.sqrt(2)) / 2)
    p = float(mp.npdf(xj)) if xj < 8.5 else 0.0
    d = y - xj
    u, v = xj * d, d * d
    c0 = _fma(v, _fma(v, 1 / 40, -1 / 6), 1.0)
    c1 = _fma(v, _fma(v, -1 / 48, 1 / 8), -0.5)
    c2 = _fma(v, -1 / 20, 1 / 6)
    c3 = _fma(v, 1 / 72, -1 / 24)
    q = _fma(u, -1 / 720, 1 / 120)
    for c in (c3, c2, c1, c0):
        q = _fma(u, q, c)
    return 0.5 + float(np.copysign(_fma(p * d, q, F), x))


def test_table_cdf_error():
    mp.mp.dps = 40
    rng = np.random.default_rng(0)
    xs = list(rng.uniform(-9, 9, 1500)) + [(j + 0.5) / 64 + e for j in range(0, 545, 8) for e in (-1e-9, 0.0, 1e-9)]
    xs += [0.0, -0.0, 8.5, -8.5, 8.4999999, 1e6, -1e6, 1e300, float("inf"), float("-inf")]
    err = max(abs(mp.mpf(_cdf_table(x)) - (mp.ncdf(x) if np.isfinite(x) else mp.mpf(x > 0))) for x in xs)
    assert err <= 2.5e-16, float(err)


@pytest.mark.gpu
@pytest.mark.parametrize("design", ["cutoffs1", "cutoffs2", "width2", "alpha", "alpha3", "nested4"])
def test_gpu_draw_counts_around_a_pair(design):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle as O
    import paper_2005_10494_amd as bmd
    from paper_2005_10494_amd import workloads as W

    spec = {"cutoffs1": lambda: W.base_problem(1, [7], 0.0, 0.05),
            "cutoffs2": lambda: W.base_problem(2, [5, 17], 0.3, 0.05),
            "width2": lambda: W.base_problem(2, [4, 3], 0.3, 0.05, width=0.02),
            "alpha": lambda: W.alpha_design(5, m_r=4, bandwidth=(0.02, 0.0015)),
            "alpha3": lambda: W.alpha3_design(4),
            "nested4": lambda: W.nested4_design(4)}[design]()
    with bmd.Problem(spec) as p:
        for M in ((1, 2, 3, 37) if design != "nested4" else (1, 3)):
            ref, rvar = O.eval_grid(spec, np.arange(p.G), M)
            ok = ~np.isnan(ref)
            for prec, tol in (("fp64", 1e-9), ("fp32", 1e-5)):
                mean, var = (t.cpu().numpy() for t in p.eval_grid(M, prec, want_var=True))
                assert np.array_equal(np.isnan(mean), ~ok), (design, M, prec)
                assert np.all(np.abs(mean - ref)[ok] <= tol * np.maximum(np.abs(ref[ok]), 1e-3)), (design, M, prec)
                plain = p.eval_grid(M, prec).cpu().numpy()
                assert np.allclose(plain[ok], mean[ok], rtol=1e-6 if prec == "fp32" else 1e-13, atol=0)
            if M > 1:
                var = p.eval_grid(M, "fp64", want_var=True)[1].cpu().numpy()
                assert np.all(np.abs(var - rvar)[ok] <= 1e-9)
