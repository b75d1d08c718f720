// Dense exponentials E(tau) = exp(A tau) of tridiagonal generators
// (Sec. 2.2.2), by scaling and squaring: X = A tau / 2^s with ||X||_1 <= 1, the
// degree-24 Taylor polynomial by Horner's rule, then s squarings.
//
// X is tridiagonal, so a column of the polynomial needs no other column and
// has at most 49 entries: one wave forms it in registers (expm_taylor), where
// dense products would take 23 of the 37 products.  The squarings run on FP64
// matrix instructions (expm_gemm), all requests of a step in one launch; the
// bands of the factors (24, 48, 96, ... on either side) bound their k ranges.
// Both sum every entry in the order of a dense product over ascending k (a
// matrix instruction adds its four products one after the other, each
// rounded, as measured against chains of fma), and exact zeros change no
// sum, so the entries do not depend on the tile sizes or the bands.
//
// 1024 cells, 64 slices of T = 10 (two slice lengths, 14 squarings each),
// with one coarse pass: 1.14 ms; 37 products per length in 64x64 VALU tiles at
// 9 TFLOP/s took 17.8 ms.
#include <algorithm>
#include <cmath>

#include "pr_expm.hpp"

namespace pr {

constexpr int EX_DEG = 24;  // ||X|| <= 1: truncation below 1/25! ~ 6e-26
constexpr int EX_K = 16;    // k depth of a product's LDS stage

struct TaylorJob {  // out = the polynomial of scale * A_gen
    double *out;
    double scale;
    int gen, pad;
};
struct GemmJob {  // C = A B; A[i][j] = 0 for |i-j| > ba, B likewise with bb
    const double *A, *B;
    double *C;
    int ba, bb;
};

__global__ void __launch_bounds__(256) expm_clear(const TaylorJob *__restrict__ jobs, int64_t nn) {
    double *o = jobs[blockIdx.y].out;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < nn; i += (int64_t)gridDim.x * 256) o[i] = 0.0;
}

// One wave per column c, lane l its row c - 31 + l (the polynomial reaches
// rows c - 24 .. c + 24).  gens: per generator [3][n], the entries A[r][r-1],
// A[r][r], A[r][r+1] of row r.  Latency bound: every step depends on the last.
__global__ void __launch_bounds__(256) expm_taylor(const TaylorJob *__restrict__ jobs,
                                                   const double *__restrict__ gens, int n) {
#pragma clang fp contract(off)
    const TaylorJob J = jobs[blockIdx.y];
    const int c = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6), lane = (int)(threadIdx.x & 63);
    if (c >= n) return;
    const double *g = gens + (size_t)J.gen * 3 * n;
    const int r = c - 31 + lane;
    const bool in = r >= 0 && r < n;
    const double lo = in ? g[r] * J.scale : 0.0, di = in ? g[n + r] * J.scale : 0.0;
    const double up = in ? g[2 * n + r] * J.scale : 0.0;
    const double one = r == c ? 1.0 : 0.0;
    // I + X / 24, then R <- I + X R / k
    double R = fma(r == c ? di : (r == c - 1 ? up : (r == c + 1 ? lo : 0.0)), 1.0 / EX_DEG, one);
    for (int k = EX_DEG - 1; k >= 1; --k) {
        const double below = __shfl_up(R, 1), above = __shfl_down(R, 1);  // rows r - 1 and r + 1
        double a = fma(lo, lane > 0 ? below : 0.0, 0.0);
        a = fma(di, R, a);
        a = fma(up, lane < 63 ? above : 0.0, a);
        R = fma(1.0 / k, a, one);
    }
    if (in && r >= c - EX_DEG && r <= c + EX_DEG) J.out[(int64_t)r * n + c] = R;
}

typedef double f64x4 __attribute__((ext_vector_type(4)));
struct alignas(8) Pair {  // 16 bytes at a multiple of 8 (rows of an odd length)
    double a, b;
};

// C = A B (n x n, row-major) for the jobs of one step (blockIdx.z), one
// 32W x 32W tile per block of NW waves, each 16W x 16WC of it in 16x16x4
// FP64 matrix instructions.  Operand lanes: A[l%16][l/16], B[l/16][l%16];
// result register r of lane l: row 4 r + l/16, column l%16.
// Matrix rate bound: 64 clocks per instruction and SIMD, 27 us for a full
// 1024^3 product, which takes 45 us (two at once: 90 us, 47 TFLOP/s).  Two
// waves per SIMD and block hide the LDS reads (four waves of 32x32 per block
// took 58 us where eight of 32x16 took 44), pairs of elements per load keep
// the address arithmetic off the matrix pipe (100 -> 90 us); stages twice as
// deep gave nothing.  Two stages on their way in registers: creation at 1024
// cells 1.15 -> 1.12 ms, at 333 (rows at the edge read element by element) 202
// -> 170 us, at 200 140 -> 126 us; four and six gave nothing more, nor did
// reads of clamped pairs in place of the edge's branches (1.20 ms at 1024).  W = 1 keeps 4x as many blocks where W = 2 would leave
// most CUs idle (200 cells: 49 blocks, 16 otherwise).
template <int W, int NW>
__global__ void __launch_bounds__(64 * NW) expm_gemm(const GemmJob *__restrict__ jobs, int n) {
    constexpr int T = 32 * W;
    constexpr int AHEAD = 2;  // stages on their way in registers, even (a stage's buffer is its parity)
    static_assert(AHEAD % 2 == 0, "buffers by parity");
    static_assert(T * EX_K == 2 * 64 * NW, "a stage is one pair of each factor per thread");
    constexpr int WC = 4 * W * W / NW / W;  // 16-column tiles per wave (W rows of them)
    // strides that put the two k of a half wave's operand reads on different
    // banks (A by rows of 18 doubles, B by rows whose length is 16 mod 32)
    __shared__ double As[2][T][EX_K + 2], Bs[2][EX_K][T + 16];
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
    // this thread's pairs of a stage: row ar, k ac of A; k br, column bc of B
    const int ar = tid / (EX_K / 2), ac = tid % (EX_K / 2) * 2, br = tid / (T / 2), bc = tid % (T / 2) * 2;
    const bool inner = row0 + T <= n && col0 + T <= n;
    const double *pa = J.A + (int64_t)min(row0 + ar, n - 1) * n, *pb = J.B + col0 + bc;
    Pair fa[AHEAD], fb[AHEAD];
    auto fetch = [&](Pair &ra, Pair &rb, int k0) {
        if (inner && k0 + EX_K <= n) {
            ra = *(const Pair *)(pa + k0 + ac);
            rb = *(const Pair *)(pb + (int64_t)(k0 + br) * n);
        } else {  // the matrix's edge, element by element
            const bool okr = row0 + ar < n, okk = k0 + br < n;
            ra.a = okr && k0 + ac < n ? pa[k0 + ac] : 0.0;
            ra.b = okr && k0 + ac + 1 < n ? pa[k0 + ac + 1] : 0.0;
            rb.a = okk && col0 + bc < n ? pb[(int64_t)(k0 + br) * n] : 0.0;
            rb.b = okk && col0 + bc + 1 < n ? pb[(int64_t)(k0 + br) * n + 1] : 0.0;
        }
    };
    auto step = [&](int b, const Pair &ra, const Pair &rb) {
        As[b][ar][ac] = ra.a;
        As[b][ar][ac + 1] = ra.b;
        Bs[b][br][bc] = rb.a;
        Bs[b][br][bc + 1] = rb.b;
    };
    auto multiply = [&](int b) {
#pragma unroll
        for (int kk = 0; kk < EX_K; kk += 4) {
            double a[W], v[WC];
#pragma unroll
            for (int i = 0; i < W; ++i) a[i] = As[b][wr + 16 * i + li][kk + lk];
#pragma unroll
            for (int j = 0; j < WC; ++j) v[j] = Bs[b][kk + lk][wc + 16 * j + li];
#pragma unroll
            for (int i = 0; i < W; ++i)
#pragma unroll
                for (int j = 0; j < WC; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], v[j], acc[i][j], 0, 0, 0);
        }
    };
#pragma unroll
    for (int d = 0; d < AHEAD; ++d) fetch(fa[d], fb[d], ka + d * EX_K);
    // a stage goes to the buffer that was read two stages ago (its readers have
    // passed the last stage's barrier)
    for (int k0 = ka; k0 < kb; k0 += AHEAD * EX_K)
#pragma unroll
        for (int d = 0; d < AHEAD; ++d) {
            const int k = k0 + d * EX_K;
            if (k >= kb) break;
            step(d & 1, fa[d], fb[d]);
            fetch(fa[d], fb[d], k + AHEAD * EX_K);
            __syncthreads();
            multiply(d & 1);
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

int build_expms(const std::vector<Tridiag> &gens, const std::vector<ExpmReq> &reqs, int n, double *out,
                hipStream_t st) {
    const int G = (int)gens.size(), R = (int)reqs.size();
    if (R == 0) return PR_OK;
    const int64_t nn = (int64_t)n * n;
    std::vector<double> tri;
    std::vector<double> norm1(G, 0.0);  // largest column sum of |A|
    for (int g = 0; g < G; ++g) {
        const Tridiag &A = gens[g];
        for (const std::vector<double> *v : {&A.lo, &A.di, &A.up}) tri.insert(tri.end(), v->begin(), v->end());
        for (int c = 0; c < n; ++c) {
            double s = std::fabs(A.di[c]);
            if (c > 0) s += std::fabs(A.up[c - 1]);
            if (c + 1 < n) s += std::fabs(A.lo[c + 1]);
            norm1[g] = std::max(norm1[g], s);
        }
    }
    // squarings; every request alternates between its own matrix and a spare
    // one and ends in its own
    std::vector<int> sq(R, 0);
    int most = 0;
    for (int e = 0; e < R; ++e) {
        const double norm = norm1[reqs[e].gen] * reqs[e].tau;
        while (norm / std::ldexp(1.0, sq[e]) > 1.0) ++sq[e];
        most = std::max(most, sq[e]);
    }
    // as many requests at once as 256 MiB of spare matrices serve, two at least
    const int chunk = (int)std::min<int64_t>(R, std::max<int64_t>(2, ((int64_t)256 << 20) / (8 * nn)));
    auto up256 = [](size_t b) { return (b + 255) & ~(size_t)255; };
    size_t products = 0;
    for (int s : sq) products += s;
    const size_t o_t = up256(sizeof(double) * tri.size()), o_g = o_t + up256(sizeof(TaylorJob) * R);
    const size_t o_s = o_g + up256(sizeof(GemmJob) * std::max<size_t>(1, products));
    char *mem = nullptr;
    if (hipMalloc((void **)&mem, o_s + sizeof(double) * (size_t)nn * chunk) != hipSuccess) {
        set_error("device allocation of the exponential workspace failed");
        return PR_E_NOMEM;
    }
    std::vector<char> host(o_s, 0);
    std::copy((const char *)tri.data(), (const char *)(tri.data() + tri.size()), host.data());
    TaylorJob *tj = (TaylorJob *)(host.data() + o_t);
    GemmJob *gj = (GemmJob *)(host.data() + o_g);
    struct Launch {
        int first, count;
    };
    std::vector<std::vector<Launch>> steps;  // products of every chunk, squaring by squaring
    int ng = 0;
    for (int e0 = 0; e0 < R; e0 += chunk) {
        const int e1 = std::min(R, e0 + chunk);
        auto at = [&](int e, bool spare) {
            return spare ? (double *)(mem + o_s) + nn * (e - e0) : out + nn * e;
        };
        steps.emplace_back();
        for (int e = e0; e < e1; ++e)
            tj[e] = TaylorJob{at(e, sq[e] % 2 != 0), reqs[e].tau / std::ldexp(1.0, sq[e]), reqs[e].gen, 0};
        for (int i = 0; i < most; ++i) {
            const int first = ng;
            for (int e = e0; e < e1; ++e) {
                if (sq[e] <= i) continue;
                const bool spare = (sq[e] - i) % 2 != 0;
                const int band = (int)std::min<int64_t>(n, (int64_t)EX_DEG << std::min(i, 20));
                gj[ng++] = GemmJob{at(e, spare), at(e, spare), at(e, !spare), band, band};
            }
            if (ng > first) steps.back().push_back(Launch{first, ng - first});
        }
    }
    auto run = [&]() -> int {
        PR_HIP(hipMemcpyAsync(mem, host.data(), o_s, hipMemcpyHostToDevice, st));
        const TaylorJob *d_t = (const TaylorJob *)(mem + o_t);
        const GemmJob *d_g = (const GemmJob *)(mem + o_g);
        constexpr int MAXZ = 32768;
        const unsigned t2 = (unsigned)((n + 63) / 64), t1 = (unsigned)((n + 31) / 32);
        for (int e0 = 0, ci = 0; e0 < R; e0 += chunk, ++ci) {
            const int e1 = std::min(R, e0 + chunk);
            for (int e = e0; e < e1; e += MAXZ) {
                const unsigned cnt = (unsigned)std::min(MAXZ, e1 - e);
                const unsigned cb = (unsigned)std::min<int64_t>((nn + 1023) / 1024, 1024);
                hipLaunchKernelGGL(expm_clear, dim3(cb, cnt), dim3(256), 0, st, d_t + e, nn);
                PR_LAUNCHED();
                hipLaunchKernelGGL(expm_taylor, dim3((unsigned)((n + 3) / 4), cnt), dim3(256), 0, st, d_t + e,
                                   (const double *)mem, n);
                PR_LAUNCHED();
            }
            for (const Launch &l : steps[ci])
                for (int z = 0; z < l.count; z += MAXZ) {
                    const unsigned nz = (unsigned)std::min(MAXZ, l.count - z);
                    if ((uint64_t)t2 * t2 * nz >= 128)
                        hipLaunchKernelGGL((expm_gemm<2, 8>), dim3(t2, t2, nz), dim3(512), 0, st, d_g + l.first + z, n);
                    else
                        hipLaunchKernelGGL((expm_gemm<1, 4>), dim3(t1, t1, nz), dim3(256), 0, st, d_g + l.first + z, n);
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
