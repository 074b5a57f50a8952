// Generated by gen_exp2_fit.py; do not edit.
// 2^f = sum_(i=0..11) c_i f^i on |f| <= 1/2, c_0 first; against 40-digit values the
// polynomial is within 1.97e-17 relative, its double-precision evaluation within 1.14e-16.
#pragma once

namespace bmd {
constexpr int kExp2Deg = 11;
constexpr double kExp2Fit[kExp2Deg + 1] = {
    0x1.0000000000000p+0,  // 1
    0x1.62e42fefa39efp-1,  // 0.69314718055994529
    0x1.ebfbdff82c598p-3,  // 0.24022650695910097
    0x1.c6b08d704a0c2p-5,  // 0.055504108664821597
    0x1.3b2ab6fba1ddap-7,  // 0.0096181291076068882
    0x1.5d87fe78a5276p-10,  // 0.0013333558146416936
    0x1.430913096fd9fp-13,  // 0.0001540353044173605
    0x1.ffcbfc670dcd4p-17,  // 1.5252733829836119e-05
    0x1.62bfd47773353p-20,  // 1.3215442587921689e-06
    0x1.b524fae627834p-24,  // 1.0178062445845774e-07
    0x1.e6063f7217bc6p-28,  // 7.0725859492692234e-09
    0x1.e9d3fe3952179p-32,  // 4.4549605981865186e-10
};
}  // namespace bmd
