"""Mills' ratio of the FP64 derivatives, replayed on the CPU (fused multiply-adds
rounded once) against 40-digit values.  Bound: the polynomial within 1e-16; s = 1 -
8 r carries two ulp of the reciprocal's rounding where F' / F is largest (y = 0,
F' / F = -2.4): 2.6e-16 at most; Horner's last step and the final product one
rounding each: 5e-16."""
import importlib.util
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2005_10494_amd", "csrc")
pytest.importorskip("mpmath")


def test_header_and_error():
    spec = importlib.util.spec_from_file_location("gen_mills", os.path.join(CSRC, "gen_mills_fit.py"))
    gen = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(gen)
    text = open(os.path.join(CSRC, "mills_fit.hpp")).read()
    vals = [float.fromhex(v) for v in re.findall(r"^    (-?0x[0-9a-f.]+p[-+]\d+),", text, re.M)]
    assert vals == gen.fit()   # the header is the generator's output
    assert "kMillsK = %d;" % gen.K in text and "kMillsDeg = %d;" % gen.DEG in text
    poly, evald = gen.errors(vals, 801)
    assert poly <= 1e-16 and evald <= 5e-16
    for y in (60.0, 1e3, 1e9):
        assert abs(gen.replay(vals, y) / float(gen.mills(gen.mp.mpf(y))) - 1) <= 5e-16
