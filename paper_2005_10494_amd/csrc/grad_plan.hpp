// How a gradient call over B points and M draws splits its draws: slices (a
// workgroup takes one slice of draws and one row of points), and passes (whole
// slices whose draws are in device memory together).  Host arithmetic only.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace bmd {

constexpr size_t kGradDrawBudget = size_t(4) << 30;        // bytes of draws that a pass may hold
constexpr int64_t kGradPassDraws = int64_t(1) << 28;       // draws of a pass: the kernel's byte offsets have 32 bits

struct GradPlan {
    int64_t n_slices, slice_len;
    int64_t pass;   // draws of a pass: M, or whole slices
};

// groups: rows of points; step: draws a workgroup has in flight (slices are whole
// steps); resident: workgroups the chip holds at once; rounds of them the call
// is cut into; per_draw: bytes of a draw; budget: bytes of a pass.
// window, most (0: none): slices of at most `window` draws, as far as `most` slices
// allow.
// Many groups fill the chip by themselves and would take few, long slices, so a
// slice is also bounded by what one pass may hold: by kGradDrawBudget whatever
// `budget` is, so that the slices, and with them the order of the sums, do not
// depend on it (a budget below one slice holds one slice).
inline GradPlan grad_plan_of(int64_t groups, int64_t step, int64_t resident, int64_t rounds, int64_t M, double per_draw,
                             size_t budget, int64_t window = 0, int64_t most = 0) {
    const int64_t fits = static_cast<int64_t>(static_cast<double>(kGradDrawBudget) / per_draw);
    const int64_t longest = std::max<int64_t>(1, std::min(fits, kGradPassDraws) / step) * step;
    int64_t n = (rounds * resident + groups - 1) / groups;
    n = std::max<int64_t>(1, std::min<int64_t>({n, (M + step - 1) / step, 65528}));
    if (window > 0) n = std::max(n, std::min(most, (M + window - 1) / window));
    n = std::max(n, (M + longest - 1) / longest);
    if (n >= 8) n = (n + 7) / 8 * 8;   // the XCDs take slices in turn
    int64_t len = (M + n - 1) / n;
    len = (len + step - 1) / step * step;   // at most `longest`, itself whole steps
    int64_t slices = static_cast<int64_t>(static_cast<double>(budget) / (per_draw * static_cast<double>(len)));
    slices = std::max<int64_t>(1, std::min(slices, kGradPassDraws / len));
    return {(M + len - 1) / len, len, std::min(M, slices * len)};
}

// Whether a call of plan g may read the draws that the call before it on the
// same M left: only if that call made all of them in one pass (`left`), and only
// in a single pass of its own.  Two calls of different point counts have slices of
// different lengths, hence passes of different lengths: one may need several passes
// (and leave the last, laid out for its own length) where the other needs one.
inline bool grad_draws_ready(bool left, const GradPlan& g, int64_t M) { return left && g.pass >= M; }
inline bool grad_leaves_draws(const GradPlan& g, int64_t M) { return g.pass >= M; }

}  // namespace bmd
