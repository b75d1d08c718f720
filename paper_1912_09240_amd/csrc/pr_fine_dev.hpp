// Device side of the fine propagator shared by the single-instance and the
// batched launches: the scheme's coefficients and one Euler-Maruyama step
// (Sec. 2.1.3 eq. (EMx)/(EMy)) of one particle with its in-kernel normals.
#pragma once

#include <cmath>

#include "pr_internal.hpp"

namespace pr {

// Parameters of the scheme, precomputed on the host.
template <typename T>
struct EmCoef {
    T a3, a1, al;  // -dt times the drift coefficients of X: c3 x^3 + c1 x + lam (x - ybar)
    T rate;        // dt / eps
    T sx;          // sqrt(2 dt / beta)
    T sy;          // sqrt(2 dt / (beta eps))
};

// The normals' tables in LDS, by precision.
template <typename T>
struct TabOf {
    using type = NoiseTab;
};
template <>
struct TabOf<float> {
    using type = NoiseTabF;
};

__device__ __forceinline__ double fmaf_t(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fmaf_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// One Euler-Maruyama update of one particle from its normals z, drift at the
// old state.  Fused multiply-adds written out, everything else unfused, so
// that every kernel that inlines it produces the same bits:
//   x' = x - dt lam (x - ybar) - dt (c1 + c3 x^2) x + sx z0
template <int D, typename T>
__device__ __forceinline__ void em_update(T &x, T (&y)[D], const T (&a)[D], const EmCoef<T> &c, const T *z) {
#pragma clang fp contract(off)
    T ybar;
    if constexpr (D == 1) {
        ybar = y[0];
    } else {
        T s = (T)0;
#pragma unroll
        for (int i = 0; i < D; ++i) s += y[i];
        ybar = s / (T)D;
    }
    const T d = x - ybar;
    const T x2 = x * x;
    const T cx = fmaf_t(c.a3, x2, c.a1);
    T t = fmaf_t(c.al, d, x);
    t = fmaf_t(cx, x, t);
    const T xn = fmaf_t(c.sx, z[0], t);
    if constexpr (D == 1) {
        // y' = y + (dt/eps) (x - y) + sy z1
        y[0] = fmaf_t(c.sy, z[1], fmaf_t(c.rate, d, y[0]));
    } else {
#pragma unroll
        for (int i = 0; i < D; ++i) y[i] = fmaf_t(c.sy, z[i + 1], fmaf_t(-c.rate, y[i] - a[i] * x, y[i]));
    }
    x = xn;
}

// One step of one particle with its normals generated in place.
template <int D, typename T>
__device__ __forceinline__ void em_step(T &x, T (&y)[D], const T (&a)[D], const EmCoef<T> &c,
                                        const typename TabOf<T>::type &tab, Key key, uint32_t inst, uint32_t m,
                                        uint32_t p) {
    constexpr int NP = (D + 2) / 2;  // pairs of normals for 1 + D components
    T z[2 * NP];
#pragma unroll
    for (int j = 0; j < NP; ++j)
        box_muller(noise_block(key, inst, 0u, m, p, (uint32_t)j), tab, z[2 * j], z[2 * j + 1]);
    em_update<D, T>(x, y, a, c, z);
}

// ---------------------------------------------------------------------------
// Steps of few particles (d = 1, FP64).  A wave that steps its particles alone
// waits through the generator's and the transform's latencies every step
// (about 900 clocks per step of two particles, however few instructions it
// issues); with few waves per SIMD nothing fills the wait.  The normals do not
// depend on the state, so SPLIT_PROD waves generate them ahead, SPLIT_AHEAD
// steps each per round, into one of two LDS buffers while one wave runs the
// update's own short chain over the other.
// ---------------------------------------------------------------------------
constexpr int SPLIT_PROD = 7;
constexpr int SPLIT_AHEAD = 2;
constexpr int SPLIT_ROUND = SPLIT_PROD * SPLIT_AHEAD;  // steps per round
constexpr int SPLIT_THREADS = 64 * (SPLIT_PROD + 1);

struct SplitLds {
    NoiseTab tab;
    TabPair z[2][SPLIT_ROUND][64];
};

// Runs step(i, z0, z1) for i = 0..steps-1 on the last wave of the block, in
// order, with the normals of particle p (one per lane) at global step m0 + i.
// Every thread of the block calls it (tab loaded); all waves meet at a barrier
// per round and at the end.
template <class Step>
__device__ __forceinline__ void split_steps(SplitLds &L, Key key, uint32_t inst, uint32_t m0, uint32_t steps,
                                            uint32_t p, Step step) {
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = (int)(threadIdx.x & 63);
    const uint32_t rounds = (steps + SPLIT_ROUND - 1) / SPLIT_ROUND;
    auto produce = [&](uint32_t r) {
#pragma unroll
        for (int u = 0; u < SPLIT_AHEAD; ++u) {
            const uint32_t i = (uint32_t)(wave * SPLIT_AHEAD + u);  // past the last step: generated, not used
            TabPair z;
            box_muller(noise_block(key, inst, 0u, m0 + r * SPLIT_ROUND + i, p, 0u), L.tab, z.a, z.b);
            L.z[r & 1u][i][lane] = z;
        }
    };
    if (wave < SPLIT_PROD && rounds > 0) produce(0);
    for (uint32_t r = 0; r < rounds; ++r) {
        __syncthreads();  // round r is there, round r - 1's buffer is free
        if (wave < SPLIT_PROD) {
            if (r + 1 < rounds) produce(r + 1);
        } else {
            const uint32_t left = steps - r * SPLIT_ROUND;
            if (left >= SPLIT_ROUND) {
#pragma unroll
                for (uint32_t i = 0; i < SPLIT_ROUND; ++i) {
                    const TabPair z = L.z[r & 1u][i][lane];
                    step(r * SPLIT_ROUND + i, z.a, z.b);
                }
            } else {
                for (uint32_t i = 0; i < left; ++i) {
                    const TabPair z = L.z[r & 1u][i][lane];
                    step(r * SPLIT_ROUND + i, z.a, z.b);
                }
            }
        }
    }
    __syncthreads();
}

template <typename T>
inline EmCoef<T> make_coef(const pr_sde *s, double dt) {
    EmCoef<T> c;
    c.a3 = (T)(-dt * s->c3);
    c.a1 = (T)(-dt * s->c1);
    c.al = (T)(-dt * s->lambda);
    c.rate = (T)(dt / s->eps);
    c.sx = (T)std::sqrt(2.0 * dt / s->beta);
    c.sy = (T)std::sqrt(2.0 * dt / (s->beta * s->eps));
    return c;
}

}  // namespace pr
