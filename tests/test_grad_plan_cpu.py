"""Slices and passes of a gradient call (csrc/grad_plan.hpp, host arithmetic,
compiled here by itself): a refinement's evaluations never read draws that the
workspace does not hold, and no pass outgrows its memory or the kernel's 32-bit
byte offsets."""
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


def test_passes_stay_within_their_bounds(tmp_path):
    """Over point groups, draw counts, draw sizes and budgets: the slices cover the
    draws; a pass holds whole slices, at most 2^28 draws (byte offsets below 2^32 at
    8 bytes a draw and row need 2^29) and at most the default budget where that is the
    budget; the slices do not depend on the budget; and a call whose slices fit
    anyway (counted) keeps those it had without the bound."""
    bad, kept, cut = _run(tmp_path, """
    long bad = 0, kept = 0, cut = 0;
    for (int64_t groups : {1L, 2L, 257L, 512L, 1125L, 6200L, 8192L, 131072L, 1L << 22})
        for (int64_t step : {64L, 128L, 256L})
            for (int64_t resident : {1L, 256L, 768L})
                for (double per : {84.0, 148.0, 1144.0, 6300.0})
                    for (double m = 1; m < 1.2e12; m *= 1.9) {
                        const int64_t M = std::min<int64_t>(static_cast<int64_t>(m), 1L << 40);
                        const GradPlan g = grad_plan_of(groups, step, resident, 8, M, per, kGradDrawBudget);
                        bad += g.slice_len % step != 0 || g.n_slices * g.slice_len < M || (g.n_slices - 1) * g.slice_len >= M;
                        bad += g.pass < 1 || (g.pass < M && g.pass % g.slice_len != 0) || g.pass > kGradPassDraws;
                        bad += (g.pass + g.slice_len - 1) / g.slice_len > 65535;
                        bad += static_cast<double>(g.pass) * per > static_cast<double>(kGradDrawBudget);
                        for (size_t budget : {size_t(1), size_t(1) << 24, size_t(200) << 30}) {
                            const GradPlan o = grad_plan_of(groups, step, resident, 8, M, per, budget);
                            bad += o.slice_len != g.slice_len || o.n_slices != g.n_slices || o.pass > kGradPassDraws;
                            bad += (o.pass + o.slice_len - 1) / o.slice_len > 65535;
                            bad += static_cast<double>(o.pass) * per > std::max<double>(budget, o.slice_len * per);
                        }
                        int64_t n = (8 * resident + groups - 1) / groups;
                        n = std::max<int64_t>(1, std::min<int64_t>({n, (M + step - 1) / step, 65528}));
                        if (n >= 8) n = (n + 7) / 8 * 8;
                        const int64_t len = ((M + n - 1) / n + step - 1) / step * step;
                        const bool fits = len <= kGradPassDraws && len * per <= static_cast<double>(kGradDrawBudget);
                        if (fits) bad += len != g.slice_len;
                        (fits ? kept : cut) += 1;
                    }
    std::printf("%ld %ld %ld\\n", bad, kept, cut);""")
    assert bad == 0 and kept > 0 and cut > 0


def test_slices_within_the_window(tmp_path):
    """Slices no longer than the window (in whole steps) unless the partial sums' bound
    is reached; calls within it anyway keep their slices (counted: both)."""
    bad, kept, cut, bound = _run(tmp_path, """
    long bad = 0, kept = 0, cut = 0, bound = 0;
    for (int64_t groups : {1L, 128L, 512L, 8192L, 1L << 20})
        for (int64_t window : {650L, 4369L, 65536L})
            for (int64_t most : {0L, 3L, 40L, 100000L})
                for (int64_t M = 1; M < 200000000; M = M * 3 + 1) {
                    const GradPlan a = grad_plan_of(groups, 64, 768, 8, M, 700.0, kGradDrawBudget);
                    const GradPlan b = grad_plan_of(groups, 64, 768, 8, M, 700.0, kGradDrawBudget, window, most);
                    const int64_t w = (window + 63) / 64 * 64;
                    bad += b.n_slices * b.slice_len < M || (b.n_slices - 1) * b.slice_len >= M || b.slice_len > a.slice_len;
                    if (a.slice_len <= window) { bad += b.slice_len != a.slice_len; ++kept; }
                    else if (most >= (M + window - 1) / window) { bad += b.slice_len > w; ++cut; }
                    else { bad += b.n_slices > std::max(a.n_slices, (most + 7) / 8 * 8); ++bound; }
                }
    std::printf("%ld %ld %ld %ld\\n", bad, kept, cut, bound);""")
    assert bad == 0 and kept > 0 and cut > 0 and bound > 0
