// Standard normal pairs from one Philox block (Box-Muller), for the noise of
// the Euler-Maruyama scheme (Sec. 2.1.3 eq. (EMx)/(EMy)) and of the initial
// law.  The random bits are laid out so that both uniforms come out of two
// integer operations:
//
//   u = (k + 1/2) 2^-52,  k = (w0 >> 12) 2^32 + w1            u in (0, 1)
//   t = (i + f) / 128,    i = bits 4..11 of w2,
//                         f = ((w2 >> 12) 2^32 + w3) 2^-52     t in [0, 2)
//   z0 = sqrt(-2 ln u) cos(pi t),  z1 = sqrt(-2 ln u) sin(pi t).
//
// 1 + k 2^-52 and 1 + f are doubles whose high word is 0x3FF00000 | (w >> 12)
// and whose low word is a whole 32-bit word, so each costs one funnel shift.
//
// -2 ln u (table of 1024 pairs, Tang-style reduction):
//   u = m 2^e with m in [1/2, 1); c_i = 1/2 + (i + 1/2)/2048 for the cell i
//   of m (its top 10 mantissa bits), R_i = RN(1/c_i), g = m R_i - 1 with
//   |g| <= 2^-11; -2 ln u = -2 e ln 2 + 2 ln R_i - 2 ln(1 + g), the last term
//   as g (-2 + g - 2g^2/3 + g^3/2 - 2g^4/5) (the next term, g^6/3, is below
//   2^-57 of 2|g|).  The top cell uses R = 1 exactly, so g = m - 1 is exact
//   and -2 ln u keeps full relative accuracy as u -> 1.
// sin and cos of pi t (table of 256 pairs):
//   t = a_i + b/128 with a_i = (i + 1/2)/128 and b = (1 + f) - 3/2 exact in
//   [-1/2, 1/2); with h = pi/128, sin(h b) to b^5 and cos(h b) - 1 to b^6
//   (truncation below 1e-17), then the angle-addition formulas against the
//   tabulated sin(pi a_i), cos(pi a_i).
//
// The tables (pr_noise_tables.inc, written by gen_noise_tables.py) sit in
// LDS during a kernel: every block fills its copy with load_noise_tab()
// before its first normal.  The same code runs on the host against the
// host copy of the tables, for the tests.
#pragma once

#include <cstdint>

#include "pr_fastmath.hpp"

namespace pr {

#include "pr_noise_tables.inc"

struct alignas(16) TabPair {
    double a, b;
};

struct NoiseTab {
    TabPair sc[256];   // sin(pi a_i), cos(pi a_i)
    TabPair lg[1024];  // R_i, 2 ln R_i
};
constexpr int kNoiseTabDoubles = 2560;

static __constant__ double kNoiseTabDev[kNoiseTabDoubles] = {
#define PR_NOISE_TABLE_ENTRIES
#include "pr_noise_tables.inc"
#undef PR_NOISE_TABLE_ENTRIES
};

// 0x3FF00000 | (w >> 12): high word of the double 1 + (w >> 12) 2^-20.
__host__ __device__ __forceinline__ uint32_t unit_high_word(uint32_t w) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_alignbit(0x3FFu, w, 12u);
#else
    return 0x3FF00000u | (w >> 12);
#endif
}

__host__ __device__ __forceinline__ double double_of_words(uint32_t hi, uint32_t lo) {
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// -2 ln u for u in (0, 1); positive for every such u.
__host__ __device__ __forceinline__ double neg2_ln(double u, const TabPair *lg) {
#pragma clang fp contract(off)
    int e;
    const double m = mantissa_exponent(u, e);  // [1/2, 1)
    const uint32_t hi = (uint32_t)(__builtin_bit_cast(uint64_t, m) >> 32);
    const TabPair t = lg[(hi >> 10) & 1023u];
    const double g = __builtin_fma(m, t.a, -1.0);
    double q = __builtin_fma(-0.4, g, 0.5);
    q = __builtin_fma(q, g, -2.0 / 3.0);
    q = __builtin_fma(q, g, 1.0);
    q = __builtin_fma(q, g, -2.0);
    const double s = __builtin_fma(g, q, t.b);  // 2 ln R_i - 2 ln(1 + g)
    return __builtin_fma((double)e, kMinus2Ln2, s);
}

// sin(pi t) -> s, cos(pi t) -> c for t = (i + f)/128 given by words w2, w3.
__host__ __device__ __forceinline__ void sincos_cell(uint32_t w2, uint32_t w3, const TabPair *sc,
                                                     double &s, double &c) {
#pragma clang fp contract(off)
    const TabPair t = sc[(w2 >> 4) & 255u];
    const double b = double_of_words(unit_high_word(w2), w3) - 1.5;
    const double b2 = b * b;
    double ps = __builtin_fma(kSinP5, b2, kSinP3);
    ps = __builtin_fma(ps, b2, kSinP1);
    const double sb = b * ps;  // sin(h b)
    double pc = __builtin_fma(kCosQ6, b2, kCosQ4);
    pc = __builtin_fma(pc, b2, kCosQ2);
    const double cm1 = b2 * pc;  // cos(h b) - 1
    s = __builtin_fma(t.a, cm1, __builtin_fma(t.b, sb, t.a));
    c = __builtin_fma(t.b, cm1, __builtin_fma(-t.a, sb, t.b));
}

// The normal pair of one block of words.
__host__ __device__ __forceinline__ void normal_pair_of_words(uint32_t w0, uint32_t w1, uint32_t w2,
                                                              uint32_t w3, const NoiseTab &tab,
                                                              double &z0, double &z1) {
#pragma clang fp contract(off)
    // 1 + k 2^-52 - (1 - 2^-53) = (k + 1/2) 2^-52, exact
    const double u = double_of_words(unit_high_word(w0), w1) - 0x1.fffffffffffffp-1;
    const double r = sqrt_positive(neg2_ln(u, tab.lg));
    double s, c;
    sincos_cell(w2, w3, tab.sc, s, c);
    z0 = r * c;
    z1 = r * s;
}

// Every thread of the (one-dimensional) block calls this before its first
// normal, and before any early exit.
__device__ __forceinline__ void load_noise_tab(NoiseTab &tab) {
    double *d = reinterpret_cast<double *>(&tab);
    for (int i = (int)threadIdx.x; i < kNoiseTabDoubles; i += (int)blockDim.x) d[i] = kNoiseTabDev[i];
    __syncthreads();
}

// FP32 pair with the same bits at single precision: u from the top 24 bits of
// w0 (rounded to single), the angle from bits 4..31 of w2, by the table of
// 256 pairs above in single precision.
//   -2 ln u: the hardware's base-2 logarithm (1 ulp, also next to u = 1) times
//   -2 ln 2 in two parts; 2^-100 keeps the root's seed finite at u = 1.
//   sin(h b) to b^3 and cos(h b) - 1 to b^2 (truncation below 1e-9), b exact.
// 26 vector operations and two transcendental ones per pair, against 44 for
// logf, sqrtf and sincospif, whose angle is also rounded (t to 24 bits).
struct alignas(8) TabPairF {
    float a, b;
};
struct NoiseTabF {
    TabPairF sc[256];
};

__device__ __forceinline__ void load_noise_tab(NoiseTabF &tab) {
    float *d = reinterpret_cast<float *>(&tab);
    for (int i = (int)threadIdx.x; i < 512; i += (int)blockDim.x) d[i] = (float)kNoiseTabDev[i];
    __syncthreads();
}

__device__ __forceinline__ void normal_pair_of_words_f32(uint32_t w0, uint32_t w2, const NoiseTabF &tab, float &z0,
                                                         float &z1) {
#pragma clang fp contract(off)
    constexpr float M2LN2 = -0x1.62e43p+0f, M2LN2_LO = (float)(kMinus2Ln2 - (double)M2LN2);
    const float u = __builtin_fmaf((float)(w0 >> 8), 0x1p-24f, 0x1p-25f);
    const float l2 = __builtin_amdgcn_logf(u);
    const float L = __builtin_fmaf(l2, M2LN2, __builtin_fmaf(l2, M2LN2_LO, 0x1p-100f));
    const float y = __builtin_amdgcn_rsqf(L);
    float r = L * y;
    r = __builtin_fmaf(__builtin_fmaf(-r, r, L), 0.5f * y, r);
    const TabPairF t = tab.sc[(w2 >> 4) & 255u];
    const float b = __builtin_fmaf((float)(w2 >> 12), 0x1p-20f, -0.5f);
    const float b2 = b * b;
    const float sb = b * __builtin_fmaf((float)kSinP3, b2, (float)kSinP1);
    const float cm1 = (float)kCosQ2 * b2;
    const float ds = __builtin_fmaf(t.b, sb, t.a * cm1), dc = __builtin_fmaf(-t.a, sb, t.b * cm1);
    z0 = __builtin_fmaf(r, dc, r * t.b);
    z1 = __builtin_fmaf(r, ds, r * t.a);
}

}  // namespace pr
