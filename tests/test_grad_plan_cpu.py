"""Slices and passes of a gradient call (csrc/grad_plan.hpp, host arithmetic,
compiled here by itself): a refinement's evaluations never read draws that the
workspace does not hold."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2005_10494_amd", "csrc")


def _run(tmp_path, body):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text('#include <cstdio>\n#include <initializer_list>\n#include "grad_plan.hpp"\nusing namespace bmd;\n'
                   "int main() {\n%s\n}\n" % body)
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-I", CSRC, str(src), "-o", str(exe)])
    return [int(x) for x in subprocess.check_output([str(exe)], text=True).split()]


@pytest.mark.parametrize("budget", [1 << 20, 1 << 24])
def test_refinement_reuses_only_draws_that_are_there(tmp_path, budget):
    """One point (workgroups of 256 draws), then eight (64 draws): the workspace
    holds the last pass made; draws 0..M-1 must be what a call that makes none
    finds.  Counted besides: the draw counts at which the first call takes several
    passes and the later ones a single one, so that the case is met."""
    bad, met, reused = _run(tmp_path, """
    long bad = 0, met = 0, reused = 0;
    for (double per : {100.0, 632.0, 1144.0, 1200.0, 4200.0})
        for (int64_t cu : {64, 256})
            for (int64_t nb : {1, 2, 3})
                for (int64_t M = 1; M < 3 * static_cast<int64_t>(%d / per); M += M < 4096 ? 1 : 37) {
                    const GradPlan one = grad_plan_of(1, 256, cu * nb, 8, M, per, %d);
                    const GradPlan few = grad_plan_of(1, 64, cu * nb, 8, M, per, %d);
                    met += one.pass < M && few.pass >= M;
                    int64_t first = 0, count = 0;   // what the workspace holds
                    bool left = false;
                    for (const GradPlan* g : {&one, &few, &few}) {
                        const bool ready = grad_draws_ready(left, *g, M);
                        reused += ready;
                        if (ready) bad += first != 0 || count != M;
                        else
                            for (int64_t k0 = 0; k0 < M; k0 += g->pass) {
                                first = k0;
                                count = std::min(g->pass, M - k0);
                            }
                        left = grad_leaves_draws(*g, M);
                    }
                }
    std::printf("%%ld %%ld %%ld\\n", bad, met, reused);""" % (budget, budget, budget))
    assert bad == 0 and met > 0 and reused > 0
