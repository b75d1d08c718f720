// Dense exponentials E(tau) = exp(A tau) of tridiagonal generators
// (Sec. 2.2.2), by uniformisation and squaring.
//
// With L = max_i |A[i][i]| and P = I + A / L (entries >= 0, columns summing
// to 1), exp(A t) = sum_k w_k P^k with the Poisson weights w_k of mean L t.
// For L t <= 64 the sum has at most ~165 terms above 1e-25, and row r of P^k
// lives on the columns r-k..r+k: one wave forms a whole row of the sum in
// registers (expm_rows), no dense product and no cancellation.  A longer time
// is halved s times to a mean <= 64 and the result squared s times, with
// FP64 matrix instructions (expm_gemm); a factor's band bounds the k range of
// the early squarings.  Slice lengths of one generator differ by single steps,
// so the longer exponential is the short one times exp(A (tau' - tau)), whose
// band is narrow: one more product instead of a second chain of squarings.
//
// 1024 cells, mean 6.0e3 (64 slices of T = 10): 7 squarings and one banded
// product for both slice lengths.  The scheme before this one (degree-24
// Taylor polynomial by 23 dense products, then 14 squarings, per length, in
// 64x64 VALU tiles at 9 TFLOP/s) took 17.9 ms with its set-up.
#include <algorithm>
#include <cmath>

#include "pr_expm.hpp"

namespace pr {

constexpr int EX_PER = 6;               // columns per lane
constexpr int EX_HALF = 191;            // columns of the window before the row's own
constexpr int EX_TERMS = EX_HALF - 1;   // most terms of one sum
constexpr double EX_MEAN = 64.0;        // most expected jumps of one sum
constexpr int EX_K = 16;                // k depth of a product's LDS stage

struct RowJob {  // out = sum_k w[k] P_gen^k
    double *out;
    int gen, w0, terms, pad;
};
struct GemmJob {  // C = A B; A[i][j] = 0 for |i-j| > ba, B likewise with bb
    const double *A, *B;
    double *C;
    int ba, bb;
};

// The lane's neighbours along the wave (0 beyond its ends).
__device__ __forceinline__ double from_lane_below(double v) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, 0x138, 0xF, 0xF, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), 0x138, 0xF, 0xF, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ double from_lane_above(double v) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, 0x130, 0xF, 0xF, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), 0x130, 0xF, 0xF, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// One wave per row.  coef: per generator [4][n], the entries of column j of
// P: the diagonal in two parts (high, low), P[j-1][j], P[j+1][j].  Latency
// bound: every term depends on the last (30 fused multiply-adds per lane and
// two lane shifts, ~150 clocks); one wave per SIMD at 1024 rows.
__global__ void __launch_bounds__(256) expm_rows(const RowJob *__restrict__ jobs, const double *__restrict__ coef,
                                                 const double *__restrict__ weights, int n) {
    const RowJob J = jobs[blockIdx.y];
    const int r = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6), lane = (int)(threadIdx.x & 63);
    if (r >= n) return;
    const double *c = coef + (size_t)J.gen * 4 * n;
    const double *w = weights + J.w0;
    const int j0 = r - EX_HALF + lane * EX_PER;
    double sh[EX_PER], sl[EX_PER], fl[EX_PER], fr[EX_PER], u[EX_PER], acc[EX_PER];
#pragma unroll
    for (int i = 0; i < EX_PER; ++i) {
        const int j = j0 + i;
        const bool in = j >= 0 && j < n;
        const int jc = in ? j : 0;
        sh[i] = in ? c[jc] : 0.0;
        sl[i] = in ? c[n + jc] : 0.0;
        fl[i] = in ? c[2 * n + jc] : 0.0;
        fr[i] = in ? c[3 * n + jc] : 0.0;
        u[i] = j == r ? 1.0 : 0.0;
        acc[i] = w[0] * u[i];
    }
    for (int k = 1; k < J.terms; ++k) {
        const double wk = w[k];
        const double below = from_lane_below(u[EX_PER - 1]), above = from_lane_above(u[0]);
        double t[EX_PER];
#pragma unroll
        for (int i = 0; i < EX_PER; ++i) {
            const double ul = i > 0 ? u[i - 1] : below, ur = i + 1 < EX_PER ? u[i + 1] : above;
            t[i] = fma(sh[i], u[i], fma(sl[i], u[i], fma(fl[i], ul, fr[i] * ur)));
        }
#pragma unroll
        for (int i = 0; i < EX_PER; ++i) {
            u[i] = t[i];
            acc[i] = fma(wk, t[i], acc[i]);
        }
    }
    double *o = J.out + (int64_t)r * n;
#pragma unroll
    for (int i = 0; i < EX_PER; ++i) {
        const int j = j0 + i;
        if (j >= 0 && j < n) o[j] = acc[i];
    }
    // the rest of the row is zero
    for (int j = lane; j < r - EX_HALF; j += 64) o[j] = 0.0;
    for (int j = r - EX_HALF + 64 * EX_PER + lane; j < n; j += 64) o[j] = 0.0;
}

typedef double f64x4 __attribute__((ext_vector_type(4)));

// C = A B (n x n, row-major) for the jobs of one step (blockIdx.z), one
// 32W x 32W tile per block of NW waves, each 16W x 16WC of it in 16x16x4
// FP64 matrix instructions.  Operand lanes: A[l%16][l/16], B[l/16][l%16];
// result register r of lane l: row 4 r + l/16, column l%16.
// Matrix rate bound: 64 clocks per instruction and SIMD, 27 us for a full
// 1024^3 product (256 blocks of W = 2, one per CU).  Two waves per SIMD hide
// the LDS reads: 8 waves take 44 us on average over the 8 products of 1024
// cells (the first two banded), 4 waves of 32x32 took 58 us.  W = 1 keeps 4x
// as many blocks where W = 2 would leave most CUs idle (200 cells: 49 blocks,
// 16 otherwise).
template <int W, int NW>
__global__ void __launch_bounds__(64 * NW) expm_gemm(const GemmJob *__restrict__ jobs, int n) {
    constexpr int T = 32 * W, NT = 64 * NW, PER = T * EX_K / NT;
    constexpr int WC = 4 * W * W / NW / W;  // 16-column tiles per wave (W rows of them)
    __shared__ double As[2][EX_K][T + 2], Bs[2][EX_K][T + 2];
    const GemmJob J = jobs[blockIdx.z];
    const int row0 = (int)blockIdx.y * T, col0 = (int)blockIdx.x * T;
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wr = (wave / (NW / 2)) * 16 * W, wc = (wave % (NW / 2)) * 16 * WC, li = lane & 15, lk = lane >> 4;
    // k with A[row][k] and B[k][col] both inside their bands
    const int ka = max(0, max(row0 - J.ba, col0 - J.bb)) & ~(EX_K - 1);
    const int kb = min(n, min(row0 + T + J.ba, col0 + T + J.bb));
    f64x4 acc[W][WC];
#pragma unroll
    for (int i = 0; i < W; ++i)
#pragma unroll
        for (int j = 0; j < WC; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
    double ra[PER], rb[PER];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const int id = tid + e * NT;
            const int ar = row0 + id / EX_K, ac = k0 + id % EX_K;
            ra[e] = (ar < n && ac < n) ? J.A[(int64_t)ar * n + ac] : 0.0;
            const int br = k0 + id / T, bc = col0 + id % T;
            rb[e] = (br < n && bc < n) ? J.B[(int64_t)br * n + bc] : 0.0;
        }
    };
    auto stage = [&](int b) {
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const int id = tid + e * NT;
            As[b][id % EX_K][id / EX_K] = ra[e];
            Bs[b][id / T][id % T] = rb[e];
        }
    };
    if (ka < kb) {
        fetch(ka);
        stage(0);
        int b = 0;
        for (int k0 = ka; k0 < kb; k0 += EX_K, b ^= 1) {
            __syncthreads();  // stage b is filled, stage b ^ 1 has been read
            const bool more = k0 + EX_K < kb;
            if (more) fetch(k0 + EX_K);
#pragma unroll
            for (int kk = 0; kk < EX_K; kk += 4) {
                double a[W], v[WC];
#pragma unroll
                for (int i = 0; i < W; ++i) a[i] = As[b][kk + lk][wr + 16 * i + li];
#pragma unroll
                for (int j = 0; j < WC; ++j) v[j] = Bs[b][kk + lk][wc + 16 * j + li];
#pragma unroll
                for (int i = 0; i < W; ++i)
#pragma unroll
                    for (int j = 0; j < WC; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], v[j], acc[i][j], 0, 0, 0);
            }
            if (more) stage(b ^ 1);
        }
    }
#pragma unroll
    for (int i = 0; i < W; ++i)
#pragma unroll
        for (int j = 0; j < WC; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = row0 + wr + 16 * i + 4 * r + lk, col = col0 + wc + 16 * j + li;
                if (row < n && col < n) J.C[(int64_t)row * n + col] = acc[i][j][r];
            }
}

namespace {

// Poisson weights of mean m (m <= EX_MEAN) down to 1e-25, appended to w.
int append_weights(double m, std::vector<double> &w) {
    long double t = expl(-(long double)m);
    int k = 0;
    w.push_back((double)t);
    while (++k < EX_TERMS) {
        t = t * (long double)m / (long double)k;
        if ((long double)k > (long double)m && t < 1e-25L) break;
        w.push_back((double)t);
    }
    return k;
}

}  // namespace

int build_expms(const std::vector<Tridiag> &gens, const std::vector<ExpmReq> &reqs, int n, double *out,
                hipStream_t st) {
    const int G = (int)gens.size(), R = (int)reqs.size();
    if (R == 0) return PR_OK;
    const int64_t nn = (int64_t)n * n;
    // jump chain of every generator
    std::vector<double> coef((size_t)G * 4 * n), rate(G);
    for (int g = 0; g < G; ++g) {
        const Tridiag &A = gens[g];
        double L = 0.0;
        for (int j = 0; j < n; ++j) L = A.di[j] < -L ? -A.di[j] : (A.di[j] != A.di[j] ? A.di[j] : L);
        rate[g] = L;
        double *c = coef.data() + (size_t)g * 4 * n;
        for (int j = 0; j < n; ++j) {
            const double pl = (j > 0 && L > 0.0) ? A.up[j - 1] / L : 0.0;
            const double pr = (j + 1 < n && L > 0.0) ? A.lo[j + 1] / L : 0.0;
            const long double stay = 1.0L - (long double)pl - (long double)pr;
            c[j] = (double)stay;
            c[n + j] = (double)(stay - (long double)c[j]);
            c[2 * n + j] = pl;
            c[3 * n + j] = pr;
        }
    }
    // squarings of each request; whether it is its base times a narrow factor
    std::vector<int> sq(R, 0), base(R, -1);
    for (int e = 0; e < R; ++e) {
        const double mean = rate[reqs[e].gen] * reqs[e].tau;
        while (sq[e] < 1100 && std::ldexp(mean, -sq[e]) > EX_MEAN) ++sq[e];
    }
    for (int e = 0; e < R; ++e) {
        const int b = reqs[e].base;
        if (b < 0) continue;
        const double d = reqs[e].tau - reqs[b].tau;
        if (d >= 0.0 && sq[b] > 0 && rate[reqs[e].gen] * d <= EX_MEAN) base[e] = b;
    }
    // one spare matrix per request of a chunk; a request's base is in its
    // chunk or an earlier one, whose results are final
    const int chunk = (int)std::max<int64_t>(2, std::min<int64_t>(R, ((int64_t)256 << 20) / (8 * nn)));
    std::vector<int> order;
    for (int e = 0; e < R; ++e)
        if (base[e] < 0) order.push_back(e);
    for (int e = 0; e < R; ++e)
        if (base[e] >= 0) order.push_back(e);
    std::vector<double> weights;
    std::vector<RowJob> rows;
    std::vector<GemmJob> gemms;
    struct Step {
        int row0, nrows;               // row jobs
        std::vector<int> g0, ng;       // products, launch by launch
    };
    std::vector<Step> steps;
    const int spare_n = std::min(chunk, R);
    // operands by request; addresses are filled in once the memory is there
    struct Ref {
        int e, slot;  // request's own matrix (slot < 0) or spare matrix
    };
    std::vector<Ref> row_ref;
    std::vector<Ref> ga, gb, gc;
    for (int o0 = 0; o0 < R; o0 += chunk) {
        const int o1 = std::min(R, o0 + chunk);
        Step S;
        S.row0 = (int)rows.size();
        int most = 0;
        std::vector<int> band(o1 - o0, 0);
        for (int o = o0; o < o1; ++o) {
            const int e = order[o], g = reqs[e].gen;
            const double t = base[e] >= 0 ? reqs[e].tau - reqs[base[e]].tau : std::ldexp(reqs[e].tau, -sq[e]);
            const int w0 = (int)weights.size();
            const int terms = append_weights(rate[g] * t, weights);
            band[o - o0] = terms - 1;
            // the last product must end in the request's own matrix
            const int products = base[e] >= 0 ? 1 : sq[e];
            rows.push_back(RowJob{nullptr, g, w0, terms, 0});
            row_ref.push_back(Ref{e, products % 2 ? o - o0 : -1});
            most = std::max(most, base[e] >= 0 ? 0 : sq[e]);
        }
        S.nrows = (int)rows.size() - S.row0;
        for (int i = 0; i < most; ++i) {
            S.g0.push_back((int)gemms.size());
            for (int o = o0; o < o1; ++o) {
                const int e = order[o];
                if (base[e] >= 0 || sq[e] <= i) continue;
                const int64_t bw = std::min<int64_t>(n, (int64_t)band[o - o0] << std::min(i, 20));
                gemms.push_back(GemmJob{nullptr, nullptr, nullptr, (int)bw, (int)bw});
                const bool in_spare = (sq[e] - i) % 2 != 0;
                const Ref src{e, in_spare ? o - o0 : -1}, dst{e, in_spare ? -1 : o - o0};
                ga.push_back(src);
                gb.push_back(src);
                gc.push_back(dst);
            }
            S.ng.push_back((int)gemms.size() - S.g0.back());
        }
        S.g0.push_back((int)gemms.size());
        for (int o = o0; o < o1; ++o) {
            const int e = order[o];
            if (base[e] < 0) continue;
            gemms.push_back(GemmJob{nullptr, nullptr, nullptr, band[o - o0], n});
            ga.push_back(Ref{e, o - o0});
            gb.push_back(Ref{base[e], -1});
            gc.push_back(Ref{e, -1});
        }
        S.ng.push_back((int)gemms.size() - S.g0.back());
        steps.push_back(S);
    }
    auto up256 = [](size_t b) { return (b + 255) & ~(size_t)255; };
    const size_t o_w = up256(sizeof(double) * coef.size()), o_r = o_w + up256(sizeof(double) * weights.size());
    const size_t o_g = o_r + up256(sizeof(RowJob) * rows.size()), o_s = o_g + up256(sizeof(GemmJob) * gemms.size());
    char *mem = nullptr;
    if (hipMalloc((void **)&mem, o_s + sizeof(double) * (size_t)nn * spare_n) != hipSuccess) {
        set_error("device allocation of the exponential workspace failed");
        return PR_E_NOMEM;
    }
    auto at = [&](const Ref &r) { return r.slot < 0 ? out + nn * r.e : (double *)(mem + o_s) + nn * r.slot; };
    for (size_t i = 0; i < rows.size(); ++i) rows[i].out = at(row_ref[i]);
    for (size_t i = 0; i < gemms.size(); ++i) {
        gemms[i].A = at(ga[i]);
        gemms[i].B = at(gb[i]);
        gemms[i].C = at(gc[i]);
    }
    std::vector<char> host(o_s, 0);
    std::copy((const char *)coef.data(), (const char *)(coef.data() + coef.size()), host.data());
    std::copy((const char *)weights.data(), (const char *)(weights.data() + weights.size()), host.data() + o_w);
    std::copy((const char *)rows.data(), (const char *)(rows.data() + rows.size()), host.data() + o_r);
    std::copy((const char *)gemms.data(), (const char *)(gemms.data() + gemms.size()), host.data() + o_g);
    auto run = [&]() -> int {
        PR_HIP(hipMemcpyAsync(mem, host.data(), o_s, hipMemcpyHostToDevice, st));
        const RowJob *d_rows = (const RowJob *)(mem + o_r);
        const GemmJob *d_gemms = (const GemmJob *)(mem + o_g);
        constexpr int MAXZ = 32768;
        for (const Step &S : steps) {
            for (int z = 0; z < S.nrows; z += MAXZ) {
                hipLaunchKernelGGL(expm_rows, dim3((unsigned)((n + 3) / 4), (unsigned)std::min(MAXZ, S.nrows - z)),
                                   dim3(256), 0, st, d_rows + S.row0 + z, (const double *)mem,
                                   (const double *)(mem + o_w), n);
                PR_LAUNCHED();
            }
            for (size_t i = 0; i < S.g0.size(); ++i)
                for (int z = 0; z < S.ng[i]; z += MAXZ) {
                    const unsigned nz = (unsigned)std::min(MAXZ, S.ng[i] - z);
                    const GemmJob *jobs = d_gemms + S.g0[i] + z;
                    const unsigned t2 = (unsigned)((n + 63) / 64), t1 = (unsigned)((n + 31) / 32);
                    if ((uint64_t)t2 * t2 * nz >= 128)
                        hipLaunchKernelGGL((expm_gemm<2, 8>), dim3(t2, t2, nz), dim3(512), 0, st, jobs, n);
                    else
                        hipLaunchKernelGGL((expm_gemm<1, 4>), dim3(t1, t1, nz), dim3(256), 0, st, jobs, n);
                    PR_LAUNCHED();
                }
        }
        PR_HIP(hipStreamSynchronize(st));
        return PR_OK;
    };
    const int s = run();
    (void)hipFree(mem);
    return s;
}

}  // namespace pr
