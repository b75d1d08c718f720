// Pathwise adjoint of the Euler-Maruyama ensemble (d = 1, FP64) with respect
// to theta = (lambda, eps, beta, c3): reverse-mode differentiation of
//   x' = x - dt (c3 x^3 + c1 x + lambda (x - y)) + sx z0,  sx = sqrt(2 dt / beta)
//   y' = y - (dt/eps) (y - x) + sy z1,                     sy = sqrt(2 dt / (beta eps))
// with the noise z held fixed (common random numbers), including the
// dependence of the initial law Y0 = X0 + beta^-1/2 z on beta.
//
// Memory plan: the forward pass stores the state every E steps (E = 256 for
// the differentiated workload; with E <= 8 the checkpoints are the tapes'
// starts and the first recomputation below drops out).
// The reverse kernel walks every particle through the segments backwards.
// For one segment it recomputes the E steps once, writing the state every
// AD_SUB = 8 steps to a small global scratch; then for each 8-step
// sub-segment, last first, it recomputes the 8 states into registers and
// runs the reverse recursion over them.  Every recomputed step is the fine
// propagator's own Euler-Maruyama step (em_step), so the checkpoints and the
// replayed states carry the bits of pr_fine_propagate.  The noise increments
// sx z0, sy z1 of a step are recovered from two consecutive states, so the
// reverse recursion itself needs no random numbers.  Up to four seed vectors
// (observables) are carried at once, giving up to four rows of the Jacobian
// in one sweep.
#include "pr_fine_dev.hpp"
#include "pr_internal.hpp"

namespace pr {

// Steps per register tape and threads per block.  The reverse sweep is bound
// by instruction issue: two Euler-Maruyama steps (77 vector operations each)
// and the recursion (50 with four seeds) per step, two waves per SIMD in 208
// registers.  4 seeds, 2^20 particles x 10,000 steps, E = 256: 74 -> 62 ms
// with the recursion in 50 instead of 65 operations, whole tapes without
// branches and no recomputation behind the last sub-segment's start (forward
// 25 ms).  Held to 168 or 128 registers it spills (85 and 120 ms with the
// forward pass, against 85); tapes of 4 and 16 steps 92 and 103.
constexpr int AD_SUB = 8;
constexpr int AD_THREADS = 256;

struct AdCoef {
    double j3, j1;    // dx'/dx = j3 x^2 + j1
    double jxy, jyy;  // dx'/dy, dy'/dy (dy'/dx = dt/eps)
    double e1, e2;    // dy'/deps = e1 (x - y) + e2 sy z1
    double dt, inv2b;
};

// One step of the fine propagator (eq. (EMx)/(EMy), d = 1, FP64).
__device__ __forceinline__ void em_step_d1(double &x, double &y, const EmCoef<double> &ec, const NoiseTab &tab,
                                           Key key, uint32_t inst, uint32_t m, uint32_t p) {
    const double a1[1] = {1.0};
    double yv[1] = {y};
    em_step<1, double>(x, yv, a1, ec, tab, key, inst, m, p);
    y = yv[0];
}

// Forward over all steps [0, S) with checkpoints, one particle per thread
// (as the fine propagator).  MANY: groups of 256 particles per block, one after
// the other.
template <bool MANY>
__global__ void __launch_bounds__(256) fwd_ckpt_kernel(double *__restrict__ x, double *__restrict__ y, int64_t n,
                                                       int64_t S, int every, double *__restrict__ ckpt,
                                                       EmCoef<double> ec, Key key, uint32_t inst, int groups) {
    __shared__ NoiseTab tab;
    load_noise_tab(tab);
#pragma unroll 1
    for (int g = 0; g < (MANY ? groups : 1); ++g) {
        const int64_t p = ((int64_t)blockIdx.x * (MANY ? groups : 1) + g) * blockDim.x + threadIdx.x;
        if (p >= n) return;
        double xv = x[p], yv = y[p];
        int64_t cidx = 0;
        for (int64_t m0 = 0; m0 < S; m0 += every, ++cidx) {
            ckpt[(cidx * 2) * n + p] = xv;
            ckpt[(cidx * 2 + 1) * n + p] = yv;
            const int64_t m1 = m0 + every < S ? m0 + every : S;
            // 32-bit step counter (the generator's counter word is 32 bits wide)
            const uint32_t mb = (uint32_t)m0, steps = (uint32_t)(m1 - m0);
#pragma unroll 2
            for (uint32_t i = 0; i < steps; ++i) em_step_d1(xv, yv, ec, tab, key, inst, mb + i, (uint32_t)p);
        }
        x[p] = xv;
        y[p] = yv;
    }
}

// One sub-segment of the reverse sweep: the L <= AD_SUB steps from ms are
// replayed from (x0, y0) into a register tape, then the recursion runs over
// them backwards.  FULL: L = AD_SUB, without a branch between the steps (the
// replayed steps' noise is independent and interleaves).
//
// The recursion accumulates, with d = x - y and the step's increments
// xi_x = sx z0, xi_y = sy z1,
//   g0 += ax d,  g1 += ay (-d dt/eps^2 - xi_y/(2 eps)),
//   g2 += ax xi_x + ay xi_y,  g3 += ax x^3
// (the constant factors of the derivatives are applied once, at the end): 9
// fused operations per step and seed beside 14 that the seeds share.
template <int NS, bool FULL>
__device__ __forceinline__ void reverse_sub(double (&ax)[NS], double (&ay)[NS], double (&g)[NS][4], double x0,
                                            double y0, int L, uint32_t ms, uint32_t p, const AdCoef &c,
                                            const EmCoef<double> &ec, const NoiseTab &tab, Key key, uint32_t inst) {
    double tx[AD_SUB + 1], ty[AD_SUB + 1];
    tx[0] = x0;
    ty[0] = y0;
#pragma unroll
    for (int i = 0; i < AD_SUB; ++i) {
        double a = tx[i], b = ty[i];
        if (FULL || i < L) em_step_d1(a, b, ec, tab, key, inst, ms + (uint32_t)i, p);
        tx[i + 1] = a;
        ty[i + 1] = b;
    }
#pragma unroll
    for (int i = AD_SUB - 1; i >= 0; --i) {
        if (!FULL && i >= L) continue;
        const double x = tx[i], y = ty[i];
        const double d = x - y, x2 = x * x, x3 = x2 * x;
        // the step's deterministic part, as em_update has it
        double t = fmaf_t(ec.al, d, x);
        t = fmaf_t(fmaf_t(ec.a3, x2, ec.a1), x, t);
        const double xi_x = tx[i + 1] - t;
        const double xi_y = ty[i + 1] - fmaf_t(ec.rate, d, y);
        const double jxx = fmaf_t(c.j3, x2, c.j1);  // 1 - dt (3 c3 x^2 + c1 + lam)
        const double de = fmaf_t(c.e1, d, c.e2 * xi_y);
#pragma unroll
        for (int k = 0; k < NS; ++k) {
            g[k][0] = fmaf_t(ax[k], d, g[k][0]);
            g[k][1] = fmaf_t(ay[k], de, g[k][1]);
            g[k][2] = fmaf_t(ax[k], xi_x, fmaf_t(ay[k], xi_y, g[k][2]));
            g[k][3] = fmaf_t(ax[k], x3, g[k][3]);
            const double nax = fmaf_t(ax[k], jxx, ay[k] * ec.rate);
            ay[k] = fmaf_t(ax[k], c.jxy, ay[k] * c.jyy);
            ax[k] = nax;
        }
    }
}

template <int NS>
__global__ void __launch_bounds__(AD_THREADS)
adjoint_kernel(const double *__restrict__ ckpt, int n_ckpt, int every, int64_t n, int64_t S,
               const double *__restrict__ seed_x, const double *__restrict__ seed_y, int from_initial,
               double *__restrict__ sub, double *__restrict__ part, AdCoef c, EmCoef<double> ec, Key key,
               uint32_t inst) {
    __shared__ NoiseTab tab;
    load_noise_tab(tab);
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool live = p < n;
    const int64_t pc = live ? p : 0;
    double ax[NS], ay[NS], g[NS][4];
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        ax[k] = live ? seed_x[(int64_t)k * n + pc] : 0.0;
        ay[k] = (live && seed_y) ? seed_y[(int64_t)k * n + pc] : 0.0;
#pragma unroll
        for (int t = 0; t < 4; ++t) g[k][t] = 0.0;
    }
    if (live) {
        for (int seg = n_ckpt - 1; seg >= 0; --seg) {
            const int64_t m0 = (int64_t)seg * every;
            const int64_t m1 = m0 + every < S ? m0 + every : S;
            // level 1: states every AD_SUB steps of this segment into the
            // scratch, up to the start of the last sub-segment; a segment
            // of at most AD_SUB steps is one tape, which starts from the
            // checkpoint itself (checkpoints that close trade memory for
            // this whole recomputation)
            const int nsub = (int)((m1 - m0 + AD_SUB - 1) / AD_SUB);
            double nxs = ckpt[(2 * (int64_t)seg) * n + p], nys = ckpt[(2 * (int64_t)seg + 1) * n + p];
            for (int j = 0; j < nsub - 1; ++j) {
                sub[(2 * (int64_t)j) * n + p] = nxs;
                sub[(2 * (int64_t)j + 1) * n + p] = nys;
                const uint32_t ms = (uint32_t)(m0 + (int64_t)j * AD_SUB);
#pragma unroll 2
                for (uint32_t i = 0; i < (uint32_t)AD_SUB; ++i)
                    em_step_d1(nxs, nys, ec, tab, key, inst, ms + i, (uint32_t)p);
            }
            // level 2: each sub-segment, last first; the start of the next
            // one is loaded while this one is replayed
            for (int j = nsub - 1; j >= 0; --j) {
                const int64_t ms = m0 + (int64_t)j * AD_SUB;
                const int L = (int)((m1 - ms) < AD_SUB ? (m1 - ms) : AD_SUB);
                const double x0 = nxs, y0 = nys;
                if (j > 0) {
                    nxs = sub[(2 * (int64_t)(j - 1)) * n + p];
                    nys = sub[(2 * (int64_t)(j - 1) + 1) * n + p];
                }
                if (L == AD_SUB)
                    reverse_sub<NS, true>(ax, ay, g, x0, y0, L, (uint32_t)ms, (uint32_t)p, c, ec, tab, key, inst);
                else
                    reverse_sub<NS, false>(ax, ay, g, x0, y0, L, (uint32_t)ms, (uint32_t)p, c, ec, tab, key, inst);
            }
        }
#pragma unroll
        for (int k = 0; k < NS; ++k) {
            g[k][0] *= -c.dt;     // dx'/dlambda = -dt (x - y)
            g[k][2] *= -c.inv2b;  // d(sx z0)/dbeta = -xi_x / (2 beta), the same for y
            g[k][3] *= -c.dt;     // dx'/dc3 = -dt x^3
        }
        if (from_initial) {
            // Y0 = X0 + beta^-1/2 z  =>  dY0/dbeta = -(Y0 - X0) / (2 beta)
            const double dy0 = -(ckpt[n + p] - ckpt[p]) * c.inv2b;
#pragma unroll
            for (int k = 0; k < NS; ++k) g[k][2] += ay[k] * dy0;
        }
    }
    // block reduction in a fixed order
    __shared__ double red[AD_THREADS / 64][NS * 4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NS; ++k)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            double v = live ? g[k][t] : 0.0;
            for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
            if (lane == 0) red[wave][k * 4 + t] = v;
        }
    __syncthreads();
    if (threadIdx.x < NS * 4) {
        double v = 0.0;
        for (int w = 0; w < AD_THREADS / 64; ++w) v += red[w][threadIdx.x];
        part[(int64_t)blockIdx.x * NS * 4 + threadIdx.x] = v;
    }
}

__global__ void __launch_bounds__(256) adjoint_reduce(const double *__restrict__ part, int nblk, int width, double *__restrict__ grad) {
    // one block per output element; eight loads in flight per thread
    const int e = blockIdx.x;
    double s = 0.0;
    int64_t b = threadIdx.x;
    for (; b + 7 * 256 < nblk; b += 8 * 256) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = part[(b + u * 256) * width + e];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; b < nblk; b += 256) s += part[b * width + e];
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
    __shared__ double w[4];
    if ((threadIdx.x & 63) == 0) w[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) grad[e] = (w[0] + w[1]) + (w[2] + w[3]);
}

static AdCoef make_adcoef(const pr_sde *s, double dt) {
    AdCoef c;
    c.j3 = -3.0 * dt * s->c3;
    c.j1 = 1.0 - dt * (s->c1 + s->lambda);
    c.jxy = dt * s->lambda;
    c.jyy = 1.0 - dt / s->eps;
    c.e1 = -dt / (s->eps * s->eps);
    c.e2 = -0.5 / s->eps;
    c.dt = dt;
    c.inv2b = 0.5 / s->beta;
    return c;
}

static int n_checkpoints(int64_t S, int every) { return (int)((S + every - 1) / every); }

size_t adjoint_ws(int64_t n, int every, int n_seed) {
    const int64_t nblk = (n + AD_THREADS - 1) / AD_THREADS;
    const int nsub = (every + AD_SUB - 1) / AD_SUB;
    return sizeof(double) * ((size_t)2 * nsub * n + (size_t)nblk * n_seed * 4) + 512;
}

// Observables of the slow variable and their pathwise seeds (ranks frozen):
// obs[0] = mean x^2, seed 2 x_p / n; obs[1+a] = midpoint (Hazen) quantile at
// alpha_a = (1-f) x_(r) + f x_(r+1), seed (1-f) at particle perm[r], f at
// perm[r+1].  Every block works out the quantiles' one or two particles and
// weights, and its threads write their own particles' seeds: bound by the
// (1 + n_alpha) n values written (2^20 particles, 3 quantiles: 682 -> 10 us
// against one block that filled the rows before it set the weights).
constexpr int OBS_THREADS = 256;

__global__ void __launch_bounds__(OBS_THREADS)
observables_kernel(const double *__restrict__ x, const double *__restrict__ xs, const uint32_t *__restrict__ perm,
                   const double *__restrict__ mom, int64_t n, double a0, double a1, double a2, int n_alpha,
                   double *__restrict__ obs, double *__restrict__ seed) {
#pragma clang fp contract(off)
    __shared__ int64_t at[3][2];  // particles with a weight (-1: none)
    __shared__ double wt[3][2];
    if (blockIdx.x == 0 && threadIdx.x == 0) obs[0] = mom[1];
    if ((int)threadIdx.x < n_alpha) {
        const int a = threadIdx.x;
        const double t = (a == 0 ? a0 : a == 1 ? a1 : a2) * (double)n - 0.5;
        double v;
        int64_t r0, r1 = -1;
        double w0 = 1.0, w1 = 0.0;
        if (t <= 0.0) {
            r0 = 0;
            v = xs[0];
        } else if (t >= (double)(n - 1)) {
            r0 = n - 1;
            v = xs[n - 1];
        } else {
            r0 = (int64_t)floor(t);
            r1 = r0 + 1;
            const double f = t - (double)r0;
            v = xs[r0] + f * (xs[r1] - xs[r0]);
            v = v < xs[r1] ? v : xs[r1];
            w0 = 1.0 - f;
            w1 = f;
        }
        if (blockIdx.x == 0) obs[1 + a] = v;
        at[a][0] = perm[r0];
        at[a][1] = r1 >= 0 ? (int64_t)perm[r1] : -1;
        wt[a][0] = w0;
        wt[a][1] = w1;
    }
    if (!seed) return;
    __syncthreads();
    for (int64_t p = (int64_t)blockIdx.x * OBS_THREADS + threadIdx.x; p < n; p += (int64_t)gridDim.x * OBS_THREADS) {
        seed[p] = 2.0 * x[p] / (double)n;
        for (int a = 0; a < n_alpha; ++a)
            seed[(int64_t)(1 + a) * n + p] = p == at[a][0] ? wt[a][0] : p == at[a][1] ? wt[a][1] : 0.0;
    }
}

size_t observables_ws(int64_t n) {
    return restrict_ws(n, 1, PR_F64) + sizeof(double) * (size_t)n + sizeof(uint32_t) * (size_t)n + 4096;
}

}  // namespace pr

using namespace pr;

extern "C" size_t pr_observables_workspace_size(int64_t n) { return n > 0 ? observables_ws(n) : 4096; }

extern "C" int pr_observables(const double *x, int64_t n, const double *alpha, int n_alpha, double *obs,
                              double *seed_x, void *ws, size_t ws_bytes, void *stream) {
    clear_error();
    PR_REQUIRE(n >= 1 && n <= 0xFFFFFFFFll, "n must be in [1, 2^32)");
    PR_REQUIRE(n_alpha >= 0 && n_alpha <= 3, "n_alpha must be in [0, 3]");
    PR_REQUIRE(n_alpha == 0 || alpha != nullptr, "alpha must be non-NULL");
    for (int a = 0; a < n_alpha; ++a) PR_REQUIRE(alpha[a] >= 0.0 && alpha[a] <= 1.0, "alpha must be in [0, 1]");
    PR_REQUIRE(x && obs && ws, "x, obs and ws must be non-NULL");
    if (ws_bytes < observables_ws(n)) {
        set_error("workspace too small: %zu < %zu bytes", ws_bytes, observables_ws(n));
        return PR_E_NOMEM;
    }
    hipStream_t st = as_stream(stream);
    char *b = (char *)(((uintptr_t)ws + 255) & ~(uintptr_t)255);
    double *mom = (double *)b;            // 4
    double *q = mom + 4;                  // 2
    double *xs = mom + 8;                 // n
    uint32_t *perm = (uint32_t *)(xs + n);  // n
    void *rws = (void *)(((uintptr_t)(perm + n) + 255) & ~(uintptr_t)255);
    PR_CHECK(restrict_quantiles(x, PR_F64, n, 1, 1, nullptr, q, nullptr, perm, xs, mom, nullptr, rws, st));
    const double a0 = n_alpha > 0 ? alpha[0] : 0.0, a1 = n_alpha > 1 ? alpha[1] : 0.0,
                 a2 = n_alpha > 2 ? alpha[2] : 0.0;
    const int64_t obs_blocks = seed_x ? (n + OBS_THREADS - 1) / OBS_THREADS : 1;
    hipLaunchKernelGGL(observables_kernel, dim3((unsigned)(obs_blocks < 8192 ? obs_blocks : 8192)), dim3(OBS_THREADS), 0,
                       st, x, (const double *)xs, (const uint32_t *)perm,
                       (const double *)mom, n, a0, a1, a2, n_alpha, obs, seed_x);
    PR_LAUNCHED();
    return PR_OK;
}

static int check_adjoint_sde(const pr_sde *sde) {
    PR_CHECK(check_sde(sde));
    if (sde->d_fast != 1 || sde->precision != PR_F64 || sde->a != nullptr) {
        set_error("the adjoint serves d_fast = 1, FP64, a = NULL");
        return PR_E_UNSUPPORTED;
    }
    return PR_OK;
}

extern "C" int pr_fine_checkpoint(const pr_sde *sde, const pr_schedule *sched, uint64_t seed, uint32_t instance,
                                  int64_t n, void *x, void *y, double *ckpt, int ckpt_every, void *stream) {
    clear_error();
    PR_CHECK(check_adjoint_sde(sde));
    PR_CHECK(check_schedule(sched));
    PR_REQUIRE(n >= 1 && n <= 0xFFFFFFFFll, "n must be in [1, 2^32)");
    PR_REQUIRE(ckpt_every >= 1 && ckpt_every <= 1 << 20, "ckpt_every must be in [1, 2^20]");
    PR_REQUIRE(x && y && ckpt, "x, y and ckpt must be non-NULL");
    const int64_t groups = groups_per_block((n + 255) / 256, 1, sched->total_steps);
    auto kernel = groups > 1 ? fwd_ckpt_kernel<true> : fwd_ckpt_kernel<false>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(((n + 255) / 256 + groups - 1) / groups)), dim3(256), 0,
                       as_stream(stream), (double *)x, (double *)y, n, sched->total_steps, ckpt_every, ckpt,
                       make_coef<double>(sde, sched->dt), make_key(seed), instance, (int)groups);
    PR_LAUNCHED();
    return PR_OK;
}

extern "C" size_t pr_adjoint_workspace_size(int64_t n, int ckpt_every, int n_seed) {
    if (n <= 0 || ckpt_every <= 0 || n_seed <= 0) return 512;
    return adjoint_ws(n, ckpt_every, n_seed);
}

extern "C" int pr_fine_adjoint(const pr_sde *sde, const pr_schedule *sched, uint64_t seed, uint32_t instance,
                               int64_t n, const double *ckpt, int ckpt_every, const double *seed_x,
                               const double *seed_y, int n_seed, int from_initial, double *grad, void *ws,
                               size_t ws_bytes, void *stream) {
    clear_error();
    PR_CHECK(check_adjoint_sde(sde));
    PR_CHECK(check_schedule(sched));
    PR_REQUIRE(n >= 1 && n <= 0xFFFFFFFFll, "n must be in [1, 2^32)");
    PR_REQUIRE(ckpt_every >= 1 && ckpt_every <= 1 << 20, "ckpt_every must be in [1, 2^20]");
    PR_REQUIRE(n_seed >= 1 && n_seed <= 4, "n_seed must be in [1, 4]");
    PR_REQUIRE(ckpt && seed_x && grad && ws, "ckpt, seed_x, grad and ws must be non-NULL");
    if (ws_bytes < adjoint_ws(n, ckpt_every, n_seed)) {
        set_error("workspace too small: %zu < %zu bytes", ws_bytes, adjoint_ws(n, ckpt_every, n_seed));
        return PR_E_NOMEM;
    }
    const int nck = n_checkpoints(sched->total_steps, ckpt_every);
    const int64_t nblk = (n + AD_THREADS - 1) / AD_THREADS;
    double *base = (double *)(((uintptr_t)ws + 255) & ~(uintptr_t)255);
    const int nsub = (ckpt_every + AD_SUB - 1) / AD_SUB;
    double *sub = base;
    double *part = base + (size_t)2 * nsub * n;
    hipStream_t st = as_stream(stream);
    const AdCoef c = make_adcoef(sde, sched->dt);
    const EmCoef<double> ec = make_coef<double>(sde, sched->dt);
    const dim3 grid((unsigned)nblk);
    switch (n_seed) {
        case 1: hipLaunchKernelGGL(adjoint_kernel<1>, grid, dim3(AD_THREADS), 0, st, ckpt, nck, ckpt_every, n,
                                   sched->total_steps, seed_x, seed_y, from_initial, sub, part, c, ec, make_key(seed),
                                   instance); break;
        case 2: hipLaunchKernelGGL(adjoint_kernel<2>, grid, dim3(AD_THREADS), 0, st, ckpt, nck, ckpt_every, n,
                                   sched->total_steps, seed_x, seed_y, from_initial, sub, part, c, ec, make_key(seed),
                                   instance); break;
        case 3: hipLaunchKernelGGL(adjoint_kernel<3>, grid, dim3(AD_THREADS), 0, st, ckpt, nck, ckpt_every, n,
                                   sched->total_steps, seed_x, seed_y, from_initial, sub, part, c, ec, make_key(seed),
                                   instance); break;
        default: hipLaunchKernelGGL(adjoint_kernel<4>, grid, dim3(AD_THREADS), 0, st, ckpt, nck, ckpt_every, n,
                                    sched->total_steps, seed_x, seed_y, from_initial, sub, part, c, ec, make_key(seed),
                                    instance); break;
    }
    PR_LAUNCHED();
    hipLaunchKernelGGL(adjoint_reduce, dim3(n_seed * 4), dim3(256), 0, st, (const double *)part, (int)nblk,
                       n_seed * 4, grad);
    PR_LAUNCHED();
    return PR_OK;
}
