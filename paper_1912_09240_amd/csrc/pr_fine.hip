// Fine propagator: initial ensemble and Euler-Maruyama over all slices at once
// (Sec. 2.1.3 eq. (EMx)/(EMy), Sec. 3.2.1).  One thread owns one particle of
// one slice and keeps its state in registers for the whole slice; the
// normal increments come from the counter-based generator, so no random
// state is stored and a slice recomputed later sees the same numbers.
#include "pr_fine_dev.hpp"
#include "pr_internal.hpp"

namespace pr {

// With a fast part in R^32 the unrolled FP64 step would take all 256 VGPRs
// (one wave per SIMD); asking for 3 blocks per CU makes the compiler fit it
// in 168 with a few spilled values, which runs 1.5x faster (FP32: 4 blocks,
// 128 VGPRs: 32 x 2^20 particles x 16 steps 14.1 ms, 15.3 with its own 180; 4 x
// 10^4 x 100 steps, a wave per SIMD or less, 314 us and 271).
// MANY: groups of 256 particles per block, one after the other.
template <int D, typename T, bool MANY>
__global__ void __launch_bounds__(256, (D >= 32 ? (sizeof(T) == 4 ? 4 : 3) : 1))
fine_kernel(const T *xin, const T *yin, T *xout, T *yout, int64_t n, int slice_first, int64_t S, int N, EmCoef<T> c,
            const double *__restrict__ a_dev, Key key, uint32_t inst, int groups) {
    __shared__ typename TabOf<T>::type tab;
    load_noise_tab(tab);
    const int s = blockIdx.y;
    const int sl = slice_first + s;
    // the slice's step range is the block's: keep it in scalar registers so
    // that the step loop's compare runs on the scalar unit
    const int64_t m0 = uniform_i64(slice_begin(S, N, sl));
    const int64_t m1 = uniform_i64(slice_begin(S, N, sl + 1));
    T a[D];
#pragma unroll
    for (int i = 0; i < D; ++i) a[i] = a_dev ? (T)a_dev[i] : (T)1;

    // 32-bit step counter (the generator's counter word is 32 bits wide);
    // unrolled twice where the registers allow (a large fast part would spill)
    constexpr int UNROLL = D <= 4 ? 2 : 1;
    const uint32_t mb = (uint32_t)m0, steps = (uint32_t)(m1 - m0);
#pragma unroll 1
    for (int g = 0; g < (MANY ? groups : 1); ++g) {
        // waves past the last particle end here; single threads past it step the
        // first one: behind a return for them the compiler no longer overlaps two
        // unrolled steps (d = 2, 5 x 10^4 particles, 100 steps: 49 us, 56 with
        // such a return)
        const int64_t p = ((int64_t)blockIdx.x * (MANY ? groups : 1) + g) * blockDim.x + threadIdx.x, pc = p < n ? p : 0;
        if (uniform_i64(p - (int64_t)(threadIdx.x & 63)) >= n) return;
        T x = xin[(int64_t)s * n + pc], y[D];
#pragma unroll
        for (int i = 0; i < D; ++i) y[i] = yin[((int64_t)s * D + i) * n + pc];
#pragma unroll UNROLL
        for (uint32_t i = 0; i < steps; ++i) em_step<D, T>(x, y, a, c, tab, key, inst, mb + i, (uint32_t)p);
        if (p >= n) return;
        xout[(int64_t)s * n + p] = x;
#pragma unroll
        for (int i = 0; i < D; ++i) yout[((int64_t)s * D + i) * n + p] = y[i];
    }
}

// Few particles (d = 1, FP64): 64 per block, their normals generated ahead by
// the block's other waves.  The same bits as fine_kernel.
__global__ void __launch_bounds__(SPLIT_THREADS) fine_split_kernel(const double *xin, const double *yin, double *xout,
                                                                   double *yout, int64_t n, int slice_first,
                                                                   int64_t S, int N, EmCoef<double> c, Key key,
                                                                   uint32_t inst) {
    __shared__ SplitLds L;
    load_noise_tab(L.tab);
    const int s = blockIdx.y, sl = slice_first + s;
    const int64_t m0 = uniform_i64(slice_begin(S, N, sl));
    const int64_t m1 = uniform_i64(slice_begin(S, N, sl + 1));
    const int64_t p = (int64_t)blockIdx.x * 64 + (threadIdx.x & 63), pc = (int64_t)s * n + (p < n ? p : 0);
    double x = xin[pc], y[1] = {yin[pc]};
    const double a[1] = {1.0};
    split_steps(L, key, inst, (uint32_t)m0, (uint32_t)(m1 - m0), (uint32_t)p, [&](uint32_t, double z0, double z1) {
        const double z[2] = {z0, z1};
        em_update<1, double>(x, y, a, c, z);
    });
    if (threadIdx.x >= 64 * SPLIT_PROD && p < n) {
        xout[pc] = x;
        yout[pc] = y[0];
    }
}

template <int D, typename T>
__global__ void __launch_bounds__(256) init_kernel(T *__restrict__ x, T *__restrict__ y, int64_t n,
                                                   const double *__restrict__ a_dev, double sd_y,
                                                   Key key, uint32_t inst) {
    __shared__ NoiseTab tab;
    load_noise_tab(tab);
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    constexpr int NP = (D + 2) / 2;
    double z[2 * NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) box_muller(noise_block(key, inst, 1u, 0u, (uint32_t)p, (uint32_t)j), tab, z[2 * j], z[2 * j + 1]);
    const double x0 = 0.5 * z[0];
    x[p] = (T)x0;
#pragma unroll
    for (int i = 0; i < D; ++i) {
        const double ai = a_dev ? a_dev[i] : 1.0;
        y[(int64_t)i * n + p] = (T)(ai * x0 + sd_y * z[i + 1]);
    }
}

__global__ void coupling_kernel(double *a, int d, Key key, uint32_t inst) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= d) return;
    double u1, u2;
    uniforms53(noise_block(key, inst, 2u, 0u, (uint32_t)i, 0u), u1, u2);
    a[i] = 0.5 + u2;
}

// Whether the normals are generated ahead (d = 1, FP64): while the blocks of 64
// particles find room on the chip at once (three per CU, 49152 particles), and
// beyond one block per CU only for slices long enough to repay the blocks'
// start (the tables are filled per 64 instead of per 256 particles).
// Blocks of fewer than 64 particles (short ensembles in many slices) count as
// full ones.  Measured in us with / without, 100 steps: 10^4 particles 9.6 / 25, 40,000
// 20.7 / 25.1, 48,000 21.8 / 25.2, 60,000 25.9 / 25.5, 100,000 41.8 / 37.7;
// 20 steps: 10^4 7.4 / 8.8, 20,000 8.8 / 8.7, 40,000 11.5 / 8.5; 40 steps:
// 40,000 13.1 / 12.6; 1000 steps: 10^4 58 / 208; one step: 10^4 11.8 / 11.0; 16384
// slices of one particle, one step: 288 / 137.
static bool normals_ahead(int64_t n, int64_t slices, int64_t steps) {
    const int64_t particles = (n + 63) / 64 * 64 * slices;
    return steps >= 4 && (particles <= 16384 || (particles <= 49152 && steps >= 48));
}

template <int D, typename T>
static int launch_fine(const pr_sde *sde, const pr_schedule *sch, uint64_t seed, uint32_t inst,
                       int64_t n, int slice_first, int slice_count, const void *xi, const void *yi, void *x,
                       void *y, hipStream_t st) {
    if constexpr (D == 1 && sizeof(T) == 8) {
        if (normals_ahead(n, slice_count, sch->total_steps / sch->n_slices)) {
            const dim3 grid((unsigned)((n + 63) / 64), (unsigned)slice_count);
            hipLaunchKernelGGL(fine_split_kernel, grid, dim3(SPLIT_THREADS), 0, st, (const double *)xi,
                               (const double *)yi, (double *)x, (double *)y, n, slice_first, sch->total_steps,
                               sch->n_slices, make_coef<double>(sde, sch->dt), make_key(seed), inst);
            PR_LAUNCHED();
            return PR_OK;
        }
    }
    // One particle per thread: two take the same time where the chip is full
    // (64 x 2^20 particles: 221.8 ms both) and up to 1.8 times as long where it
    // is not (40,000 particles: 45 us, one 25 us; 100,000: 45.5 and 37.7).
    const int64_t groups = D == 1 ? groups_per_block((n + 255) / 256, slice_count, sch->total_steps / sch->n_slices) : 1;
    dim3 grid((unsigned)(((n + 255) / 256 + groups - 1) / groups), (unsigned)slice_count);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, (const T *)xi, (const T *)yi, (T *)x, (T *)y, n,
                           slice_first, sch->total_steps, sch->n_slices, make_coef<T>(sde, sch->dt), sde->a,
                           make_key(seed), inst, (int)groups);
    };
    if constexpr (D == 1) {
        if (groups > 1) launch(fine_kernel<D, T, true>);
        else launch(fine_kernel<D, T, false>);
    } else {
        launch(fine_kernel<D, T, false>);
    }
    PR_LAUNCHED();
    return PR_OK;
}

template <typename T>
static int dispatch_fine(const pr_sde *sde, const pr_schedule *sch, uint64_t seed, uint32_t inst,
                         int64_t n, int sf, int sc, const void *xi, const void *yi, void *x, void *y,
                         hipStream_t st) {
    switch (sde->d_fast) {
        case 1: return launch_fine<1, T>(sde, sch, seed, inst, n, sf, sc, xi, yi, x, y, st);
        case 2: return launch_fine<2, T>(sde, sch, seed, inst, n, sf, sc, xi, yi, x, y, st);
        case 3: return launch_fine<3, T>(sde, sch, seed, inst, n, sf, sc, xi, yi, x, y, st);
        case 4: return launch_fine<4, T>(sde, sch, seed, inst, n, sf, sc, xi, yi, x, y, st);
        case 8: return launch_fine<8, T>(sde, sch, seed, inst, n, sf, sc, xi, yi, x, y, st);
        case 16: return launch_fine<16, T>(sde, sch, seed, inst, n, sf, sc, xi, yi, x, y, st);
        case 32: return launch_fine<32, T>(sde, sch, seed, inst, n, sf, sc, xi, yi, x, y, st);
    }
    set_error("d_fast = %d not served", sde->d_fast);
    return PR_E_UNSUPPORTED;
}

template <int D, typename T>
static int launch_init(const pr_sde *sde, uint64_t seed, uint32_t inst, int64_t n, void *x, void *y,
                       hipStream_t st) {
    dim3 grid((unsigned)((n + 255) / 256));
    hipLaunchKernelGGL((init_kernel<D, T>), grid, dim3(256), 0, st, (T *)x, (T *)y, n, sde->a,
                       1.0 / std::sqrt(sde->beta), make_key(seed), inst);
    PR_LAUNCHED();
    return PR_OK;
}

template <typename T>
static int dispatch_init(const pr_sde *sde, uint64_t seed, uint32_t inst, int64_t n, void *x, void *y,
                         hipStream_t st) {
    switch (sde->d_fast) {
        case 1: return launch_init<1, T>(sde, seed, inst, n, x, y, st);
        case 2: return launch_init<2, T>(sde, seed, inst, n, x, y, st);
        case 3: return launch_init<3, T>(sde, seed, inst, n, x, y, st);
        case 4: return launch_init<4, T>(sde, seed, inst, n, x, y, st);
        case 8: return launch_init<8, T>(sde, seed, inst, n, x, y, st);
        case 16: return launch_init<16, T>(sde, seed, inst, n, x, y, st);
        case 32: return launch_init<32, T>(sde, seed, inst, n, x, y, st);
    }
    set_error("d_fast = %d not served", sde->d_fast);
    return PR_E_UNSUPPORTED;
}

// Host-side entry used by the parareal driver (validation done by caller).
int fine_propagate(const pr_sde *sde, const pr_schedule *sch, uint64_t seed, uint32_t inst, int64_t n,
                   int slice_first, int slice_count, const void *xi, const void *yi, void *x, void *y,
                   hipStream_t st) {
    if (slice_count == 0 || n == 0) return PR_OK;
    if (sde->precision == PR_F64)
        return dispatch_fine<double>(sde, sch, seed, inst, n, slice_first, slice_count, xi, yi, x, y, st);
    return dispatch_fine<float>(sde, sch, seed, inst, n, slice_first, slice_count, xi, yi, x, y, st);
}

int init_ensemble(const pr_sde *sde, uint64_t seed, uint32_t inst, int64_t n, void *x, void *y, hipStream_t st) {
    if (n == 0) return PR_OK;
    if (sde->precision == PR_F64) return dispatch_init<double>(sde, seed, inst, n, x, y, st);
    return dispatch_init<float>(sde, seed, inst, n, x, y, st);
}

}  // namespace pr

using namespace pr;

extern "C" int pr_draw_coupling(uint64_t seed, uint32_t instance, int d, double *a, void *stream) {
    clear_error();
    PR_REQUIRE(d >= 1 && a != nullptr, "need d >= 1 and a != NULL");
    hipLaunchKernelGGL(coupling_kernel, dim3((d + 63) / 64), dim3(64), 0, as_stream(stream), a, d,
                       make_key(seed), instance);
    PR_LAUNCHED();
    return PR_OK;
}

extern "C" int pr_init_ensemble(const pr_sde *sde, uint64_t seed, uint32_t instance, int64_t n,
                                void *x, void *y, void *stream) {
    clear_error();
    PR_CHECK(check_sde(sde));
    PR_REQUIRE(n >= 0 && n <= 0xFFFFFFFFll, "n must be in [0, 2^32)");
    PR_REQUIRE(n == 0 || (x != nullptr && y != nullptr), "x and y must be non-NULL");
    return init_ensemble(sde, seed, instance, n, x, y, as_stream(stream));
}

extern "C" int pr_fine_propagate(const pr_sde *sde, const pr_schedule *sched, uint64_t seed,
                                 uint32_t instance, int64_t n, int slice_first, int slice_count,
                                 void *x, void *y, void *stream) {
    clear_error();
    PR_CHECK(check_sde(sde));
    PR_CHECK(check_schedule(sched));
    PR_REQUIRE(n >= 0 && n <= 0xFFFFFFFFll, "n must be in [0, 2^32)");
    PR_REQUIRE(slice_first >= 0 && slice_count >= 0 && slice_first + slice_count <= sched->n_slices,
               "slices [%d, %d) outside [0, %d)", slice_first, slice_first + slice_count, sched->n_slices);
    PR_REQUIRE(slice_count <= 65535, "at most 65535 slices per call");
    PR_REQUIRE(n == 0 || slice_count == 0 || (x != nullptr && y != nullptr), "x and y must be non-NULL");
    return fine_propagate(sde, sched, seed, instance, n, slice_first, slice_count, x, y, x, y, as_stream(stream));
}
