// Generated by fit_fp32_math.py; do not edit.
// R = erfcx(a/sqrt2)/2 ~= P(v)/Q(v), v = kappa a, a in [0, 40]: max rel err 2.06e-08 (fp64 eval), 4.58e-07 (fp32 eval).
// z = -Phi^-1(q) ~= P(s)/Q(s), s = sqrt(-log2 q): max abs err 1.35e-07 (fp64), rel 3.07e-06 (fp32).
// z for s in [34, 1100] ~= P(s)/Q(s): max rel err 3.62e-08 (fp64), 3.26e-07 (fp32).
#pragma once
static constexpr double kPhiScale = 0.8493218002880191;   // kappa = sqrt(log2(e) / 2)
static constexpr float kRP[5] = {0x1.0000000000000p-1f, 0x1.15227e0000000p-1f, 0x1.1b43c80000000p-2f, 0x1.3533f20000000p-4f, 0x1.399e880000000p-7f};
static constexpr float kRQ[6] = {0x1.0000000000000p+0f, 0x1.02d0c80000000p+1f, 0x1.c276b40000000p+0f, 0x1.ac63a80000000p-1f, 0x1.c849400000000p-3f, 0x1.cecbd40000000p-6f};
static constexpr float kZP[6] = {-0x1.95e0160000000p+1f, -0x1.1765860000000p+3f, 0x1.02295e0000000p+2f, 0x1.a567fa0000000p+2f, 0x1.3e07120000000p+0f, 0x1.54009e0000000p-5f};
static constexpr float kZQ[5] = {0x1.0000000000000p+0f, 0x1.8920c00000000p+2f, 0x1.6ef04e0000000p+2f, 0x1.0e300c0000000p+0f, 0x1.20c3180000000p-5f};
static constexpr float kZPW[4] = {-0x1.e0170e0000000p-1f, 0x1.28dbb20000000p+0f, 0x1.3ea9e60000000p-2f, 0x1.cddafe0000000p-9f};
static constexpr float kZQW[3] = {0x1.0000000000000p+0f, 0x1.0ea71e0000000p-2f, 0x1.88437e0000000p-9f};
