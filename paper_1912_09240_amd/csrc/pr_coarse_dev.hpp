// Device helpers of the coarse propagator shared by the single-instance and
// the batched drivers: the piecewise-linear cdf of a knot vector (Sec. 4.4,
// eq. (discr_cdf) read on the quantile side), its inverse on cell masses
// with the flat-stretch midpoint rule, and pool-adjacent-violators.
#pragma once

#include "pr_internal.hpp"

namespace pr {

// Row-vector products.  A lane takes the elements lane, lane + 64, ..., in
// that order.  Elements past the end are read at the last one and not used:
// a load behind a condition would wait for the one before.
//
// The lane's shares of R rows at once (row k at rows[k]); the loads of U
// elements of all R rows are issued before any of them is used.  The sums do
// not depend on R and U.
template <int R, int U>
__device__ __forceinline__ void lane_rows_dot(const double *const *rows, const double *v, int n, int lane,
                                              double *acc) {
#pragma unroll
    for (int k = 0; k < R; ++k) acc[k] = 0.0;
    for (int j0 = lane; j0 < n; j0 += 64 * U) {
        double e[R][U];
#pragma unroll
        for (int k = 0; k < R; ++k)
#pragma unroll
            for (int u = 0; u < U; ++u) e[k][u] = rows[k][min(j0 + u * 64, n - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = j0 + u * 64;
            const double vj = v[min(j, n - 1)];
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const double t = fma(e[k][u], vj, acc[k]);
                acc[k] = j < n ? t : acc[k];
            }
        }
    }
}

// The lane's share of one row.
__device__ __forceinline__ double lane_row_dot(const double *__restrict__ row, const double *v, int n, int lane) {
    const double *rows[1] = {row};
    double acc[1];
    lane_rows_dot<1, 8>(rows, v, n, lane, acc);
    return acc[0];
}

// One 32-bit word from the lane that a DPP control selects.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)b, CTRL, 0xF, 0xF, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)(b >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Sum over the wave, the same additions as the butterfly v += v[lane ^ off] for
// off = 32, 16, 8, 4, 2, 1, in every lane: the first two by swapping halves and
// rows between two copies, the others by rotations inside rows of 16 (after
// the step for 8 the row has period 8, and so on, so a rotation by off reads
// the value of lane ^ off).  No LDS: the butterfly's twelve ds_bpermute per
// row took most of a link's product E rho.
__device__ __forceinline__ double wave_sum(double v) {
#pragma clang fp contract(off)
    {
        const long long b = __double_as_longlong(v);
        const auto l = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
        const auto h = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
        v = __longlong_as_double((long long)(((unsigned long long)h[0] << 32) | l[0])) +
            __longlong_as_double((long long)(((unsigned long long)h[1] << 32) | l[1]));
    }
    {
        const long long b = __double_as_longlong(v);
        const auto l = __builtin_amdgcn_permlane16_swap((unsigned)b, (unsigned)b, false, false);
        const auto h = __builtin_amdgcn_permlane16_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
        v = __longlong_as_double((long long)(((unsigned long long)h[0] << 32) | l[0])) +
            __longlong_as_double((long long)(((unsigned long long)h[1] << 32) | l[1]));
    }
    v += dpp_f64<0x128>(v);  // row_ror:8
    v += dpp_f64<0x124>(v);
    v += dpp_f64<0x122>(v);
    v += dpp_f64<0x121>(v);
    return v;
}

// ---------------------------------------------------------------------------
// Knots -> cell masses (H).  c(x) = 0 for x <= q_0, 1 for x > q_Q, else
// (j + (x - q_j)/(q_{j+1} - q_j))/Q with j the largest index with q_j < x
// (a repeated knot is a jump; c(x) = P(X < x)).  rho_i = c(x_{i+1}) - c(x_i),
// the mass beyond the grid going to the end cells.
// ---------------------------------------------------------------------------
struct GridDev {
    int cells, nq;
    double lo, h;
};

__device__ __forceinline__ double edge_at(const GridDev &g, int i) {
#pragma clang fp contract(off)
    return g.lo + (double)i * g.h;
}

__device__ inline double cdf_knots(const double *q, int nq, double x) {
#pragma clang fp contract(off)
    if (x <= q[0]) return 0.0;
    if (x > q[nq]) return 1.0;
    int lo = 0, hi = nq;  // q[lo] < x <= q[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (q[mid] < x) lo = mid;
        else hi = mid;
    }
    const double t = (x - q[lo]) / (q[lo + 1] - q[lo]);
    return ((double)lo + t) / (double)nq;
}

// The value of v in lane l (uniform l) of the wave.
__device__ __forceinline__ double lane_value(double v, int l) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, l);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), l);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Cell masses -> knots (Qf) of the piecewise-linear cdf with cumulative
// masses C_i (left to right); level p_j C_I.  A level hit on a flat stretch
// gives its midpoint; the end knots are the grid ends.  Runs inside one
// block; C must hold cells + 1 doubles of LDS.
// MAX_PER: cells of a run at most, 16 for any grid, less where the caller knows
// that it has no more than 64 MAX_PER cells.
template <int MAX_PER = 16>
__device__ inline void masses_to_knots_block(const double *rho, double *C, const GridDev &g, double *q) {
#pragma clang fp contract(off)
    // Cumulative masses by one wave, in three nested levels: every lane sums its
    // own run of consecutive masses, the runs' totals are summed along groups
    // of 8 lanes, the groups' totals along the wave, and C_{i+1} = start of the
    // group + (start of the run in it + sum inside the run).  The start of the
    // next run or group is the last value of this one and every sum is
    // non-decreasing, so C is, and constant over cells without mass, as a
    // single running sum would be (the searches below rely on both); 16 + 7 + 8
    // dependent additions per 1024 cells instead of 1024.
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        if (lane == 0) C[0] = 0.0;
        double carry = 0.0;
        for (int base = 0; base < g.cells; base += 1024) {
            const int m = min(1024, g.cells - base), per = (m + 63) >> 6;
            double v[MAX_PER], run = 0.0;
#pragma unroll
            for (int i = 0; i < MAX_PER; ++i) {
                const int idx = lane * per + i;
                v[i] = (i < per && idx < m) ? rho[base + idx] : 0.0;
            }
#pragma unroll
            for (int i = 0; i < MAX_PER; ++i)
                if (i < per) {
                    run = run + v[i];
                    v[i] = run;
                }
            // inclusive sums of the totals along the group: lane l commits in
            // step l mod 8, when the lane before it is final
            double inc = run;
#pragma unroll
            for (int l = 1; l < 8; ++l) {
                const double t = dpp_f64<0x111>(inc) + run;  // row_shr:1
                inc = (lane & 7) == l ? t : inc;
            }
            const double before = dpp_f64<0x111>(inc);
            const double in_group = (lane & 7) == 0 ? 0.0 : before;
            double start = carry;
#pragma unroll
            for (int w = 0; w < 8; ++w) {
                carry = carry + lane_value(inc, 8 * w + 7);
                start = (lane >> 3) > w ? carry : start;
            }
#pragma unroll
            for (int i = 0; i < MAX_PER; ++i) {
                const int idx = lane * per + i;
                if (i < per && idx < m) C[base + idx + 1] = start + (in_group + v[i]);
            }
        }
    }
    __syncthreads();
    const double tot = C[g.cells];
    for (int j = threadIdx.x; j <= g.nq; j += blockDim.x) {
        double v;
        if (j == 0) {
            v = edge_at(g, 0);
        } else if (j == g.nq) {
            v = edge_at(g, g.cells);
        } else {
            const double ct = ((double)j / (double)g.nq) * tot;
            int lo = -1, hi = g.cells;  // first i with C_i >= ct: C[lo] < ct <= C[hi]
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (C[mid] >= ct) hi = mid;
                else lo = mid;
            }
            const int i1 = hi;
            if (C[i1] > ct) {
                const int i = i1 - 1;
                const double e0 = edge_at(g, i), e1 = edge_at(g, i + 1);
                double x = e0 + (ct - C[i]) / rho[i] * g.h;
                x = x > e0 ? x : e0;
                v = x < e1 ? x : e1;
            } else {
                int lo2 = i1, hi2 = g.cells + 1;  // last i with C_i <= ct: C[lo2] <= ct < C[hi2]
                while (hi2 - lo2 > 1) {
                    const int mid = (lo2 + hi2) >> 1;
                    if (C[mid] <= ct) lo2 = mid;
                    else hi2 = mid;
                }
                v = 0.5 * (edge_at(g, i1) + edge_at(g, lo2));
            }
        }
        q[j] = v;
    }
}

// Whether the rounded mean a/ca exceeds the rounded mean b/cb (counts >= 1).
// Where the cross products a*cb and b*ca differ by more than 2^-49 of their
// magnitudes (plus 2^-1000), the exact means differ by more than 2^-50 of
// theirs, more than the two roundings of the divisions can close, so the
// rounded means compare as the exact ones do; otherwise (and for inf or NaN)
// both divisions are taken and compared.  The result is that of comparing
// the two rounded quotients in every case.
__host__ __device__ inline bool mean_above(double a, int ca, double b, int cb) {
#pragma clang fp contract(off)
    const double x = a * (double)cb, y = b * (double)ca;
    const double d = x - y, tol = (fabs(x) + fabs(y)) * 0x1p-49 + 0x1p-1000;
    if (d > tol) return true;
    if (-d > tol) return false;
    return a / (double)ca > b / (double)cb;
}

// Pool-adjacent-violators (equal weights) over the stretch [lo, hi) of v
// alone, as if it started the input, with the same additions and the same
// outcome of every comparison as the textbook stack form: a new value starts
// a pool (sum s, count c); while the pool below has a larger rounded mean
// S/C it is merged (s = s + S, c = c + C).  vio: the violations v[j] >
// v[j+1] inside the stretch, increasing (positions absolute, at least one).
//
// The pool on top (T) and the pool just below it (B) are held in registers;
// of the pools under T only those of more than one value are stored, in
// position order, at S[lo + k] and SC[lo + k] = start << 16 | count (B, when
// it has more than one value, is the last of them); a pool of one value is
// read back from v.  A run of values that each merge into T (a decreasing
// run) thus touches only v.  When T is a single value, nothing merges until
// the next violation: the values in between stay single pools and are
// skipped.  Returns the number of stored pools.  *fm receives the smallest
// of the means that the pool holding lo takes (v[lo] first, then after
// every merge that reaches lo): the values the serial pass over a longer
// input would compare with the mean of the last pool before the stretch.
// *lm receives the mean of the pool holding hi - 1.
//
// Run by a whole wave, every lane with the same arguments and the same scalar
// steps on the same values.  Bound by one wave's instructions and branches, about
// 500 clocks a step; a step's two comparisons (T's mean against the next value,
// B's against T's with that value) are taken together, and the pool below B (A) is
// read from LDS as soon as it is known, not when B has been merged.  Where values
// have merged into T alone several times in a row, the wave takes the run ahead at
// once: lane j adds v[i + j] to T's sum after the lanes before it, in the
// serial order, and checks the two comparisons the serial pass would make for that
// value; the longest prefix of lanes that pass is committed (windows of 8 values,
// doubling up to 64 while whole windows pass), so that a decreasing run of L
// values costs about L / 64 windows.  A window costs as much as five steps, so it
// is taken after PAVA_RUN merges, and after one where the last run would have
// repaid that (1025 values, us, with a window at every second merge / always after
// four / so: noise 426 / 384 / 373, runs of three 569 / 398 / 381, of seven 251 / 394
// / 274, of forty 130 / 170 / 148).
//
// Lanes: the wave's own lanes, or 64 lanes in one host thread (PavaHostLanes), so
// that the host runs every step the kernels run.
constexpr int PAVA_RUN = 4;

struct PavaWaveLanes {
    using Value = double;  // one per lane
    static __device__ __forceinline__ int lane() { return (int)(threadIdx.x & 63); }
    // f(lane) for every lane; lanes' values through of(x, lane)
    template <class F>
    static __device__ __forceinline__ void each(F f) {
        f(lane());
    }
    static __device__ __forceinline__ double &of(Value &x, int) { return x; }
    template <class F>
    static __device__ __forceinline__ uint64_t ballot(F f) {
        return __ballot(f(lane()));
    }
    static __device__ __forceinline__ double value(const Value &x, int l) { return lane_value(x, l); }
    static __device__ __forceinline__ double smallest(Value x) {
        for (int off = 32; off >= 1; off >>= 1) {
            const double o = __shfl_xor(x, off);
            x = o < x ? o : x;
        }
        return x;
    }
};

struct PavaHostLanes {
    struct Value {
        double x[64];
    };
    template <class F>
    static inline void each(F f) {
        for (int l = 0; l < 64; ++l) f(l);
    }
    static inline double &of(Value &x, int l) { return x.x[l]; }
    template <class F>
    static inline uint64_t ballot(F f) {
        uint64_t m = 0;
        for (int l = 0; l < 64; ++l) m |= (uint64_t)(f(l) ? 1 : 0) << l;
        return m;
    }
    static inline double value(const Value &x, int l) { return x.x[l]; }
    static inline double smallest(const Value &x) {
        double m = x.x[0];
        for (double o : x.x) m = o < m ? o : m;
        return m;
    }
};

template <class Lanes>
__host__ __device__ inline int pava_range(const double *v, int lo, int hi, const int *vio, int nv, double *S, int *SC,
                                          double *fm, double *lm) {
#pragma clang fp contract(off)
    int nb = 0, vi = 0, win = 8, run = 0, need = PAVA_RUN;
    double fmin_ = v[lo];
    int i = vio[0];
    double tS = v[i], bS = 0.0;
    int tC = 1, tSt = i, bC = 1, bSt = i - 1;
    if (i > lo) bS = v[i - 1];
    // the pool below B as loaded: the last stored one under B, and the value
    // before B, which is a pool of its own unless that pool ends there
    int aSC = 0, aN = 0;
    double aS = 0.0, aV = 0.0;
    auto load_a = [&]() {
        aN = nb - (bC > 1 ? 1 : 0);  // stored pools under B
        const int k = lo + (aN > 0 ? aN - 1 : 0);
        aSC = SC[k];
        aS = S[k];
        aV = v[bSt > lo ? bSt - 1 : lo];
    };
    load_a();
    ++i;
    double vcur = v[i < hi ? i : hi - 1];
    while (i < hi) {
        if (tC == 1) {
            // first violation at or after i - 1 (a decreasing run leaves a
            // long stretch of consumed ones behind): 64 entries per look
            int at = vi < nv ? vio[vi] : hi;
            if (at < i - 1) {
                while (true) {
                    const uint64_t bm =
                        Lanes::ballot([&](int lane) { return vi + lane >= nv || vio[vi + lane] >= i - 1; });
                    if (bm) {
                        vi += __builtin_ctzll(bm);
                        break;
                    }
                    vi += 64;
                }
                if (vi > nv) vi = nv;
                at = vi < nv ? vio[vi] : hi;
            }
            if (vi == nv) break;  // non-decreasing from v[i-1] on
            if (at > i - 1) {
                tSt = at;
                tS = v[at];
                bSt = at - 1;  // a single value: the values since i - 1 stay single
                bS = v[at - 1];
                bC = 1;
                load_a();
                i = at + 1;
                vcur = v[i];
            }
        }
        const bool into = mean_above(tS, tC, vcur, 1);
        const double s1 = vcur + tS;
        const bool onto = tSt != lo && mean_above(bS, bC, s1, tC + 1);
        if (into && !onto) {
            if (tC == 1 || run < need) {
                vcur = v[i + 1 < hi ? i + 1 : i];  // the next value
                tS = s1;
                ++tC;
                ++i;
                ++run;
                win = 8;
                if (tSt == lo) {
                    const double m = tS / (double)tC;
                    if (m < fmin_) fmin_ = m;
                }
                continue;
            }
            const int m = hi - i < win ? hi - i : win;
            typename Lanes::Value ve, acc, prev;  // T's sum before and after each lane's value
            Lanes::each([&](int lane) {
                Lanes::of(ve, lane) = lane < m ? v[i + lane] : 0.0;  // one load for the window
                Lanes::of(acc, lane) = Lanes::of(prev, lane) = tS;
            });
            for (int k = 0; k < m; ++k) {
                const double vk = Lanes::value(ve, k);
                Lanes::each([&](int lane) {
                    if (k <= lane) {
                        Lanes::of(prev, lane) = Lanes::of(acc, lane);
                        Lanes::of(acc, lane) = vk + Lanes::of(acc, lane);
                    }
                });
            }
            const uint64_t bad = Lanes::ballot([&](int lane) {
                const int cb = tC + lane;
                return !(lane < m && mean_above(Lanes::of(prev, lane), cb, Lanes::of(ve, lane), 1) &&
                         (tSt == lo || !mean_above(bS, bC, Lanes::of(acc, lane), cb + 1)));
            });
            const int f = bad ? __builtin_ctzll(bad) : 64;  // >= 1: lane 0 passes
            if (tSt == lo) {
                typename Lanes::Value mean;
                Lanes::each([&](int lane) {
                    Lanes::of(mean, lane) = lane < f ? Lanes::of(acc, lane) / (double)(tC + lane + 1) : INFINITY;
                });
                const double mm = Lanes::smallest(mean);
                if (mm < fmin_) fmin_ = mm;
            }
            tS = Lanes::value(acc, f - 1);
            tC += f;
            i += f;
            run += f;
            need = run > PAVA_RUN + 1 ? 1 : PAVA_RUN;
            if (f < m) run = 0;
            win = f == m ? (win < 64 ? 2 * win : 64) : 8;
            vcur = v[i < hi ? i : hi - 1];
            continue;
        }
        run = 0;
        const double s0 = vcur;
        vcur = v[i + 1 < hi ? i + 1 : i];
        if (into) {
            double s = s1;
            int c = tC + 1, st = tSt;
            do {  // B's mean is above
                s = s + bS;
                c = c + bC;
                st = bSt;
                if (bC > 1) --nb;  // B was the last stored pool
                if (st == lo) {
                    const double m = s / (double)c;
                    if (m < fmin_) fmin_ = m;
                    break;
                }
                if (aN > 0 && (aSC >> 16) + (aSC & 0xFFFF) == st) {
                    bS = aS;
                    bC = aSC & 0xFFFF;
                    bSt = aSC >> 16;
                } else {
                    bS = aV;
                    bC = 1;
                    bSt = st - 1;
                }
                load_a();
            } while (mean_above(bS, bC, s, c));
            tS = s;
            tC = c;
            tSt = st;
        } else {
            if (tC > 1) {
                S[lo + nb] = tS;
                SC[lo + nb] = (tSt << 16) | tC;
                ++nb;
            }
            bS = tS;
            bC = tC;
            bSt = tSt;
            load_a();
            tS = s0;
            tC = 1;
            tSt = i;
        }
        ++i;
    }
    *lm = (i - 1 == hi - 1) ? tS / (double)tC : v[hi - 1];
    if (tC > 1) {
        S[lo + nb] = tS;
        SC[lo + nb] = (tSt << 16) | tC;
        ++nb;
    }
    *fm = fmin_;
    return nb;
}

__device__ inline int pava_wave_range(const double *v, int lo, int hi, const int *vio, int nv, double *S, int *SC,
                                      double *fm, double *lm) {
    return pava_range<PavaWaveLanes>(v, lo, hi, vio, nv, S, SC, fm, lm);
}

// The same on the host.
inline int pava_sparse_range(const double *v, int lo, int hi, const int *vio, int nv, double *S, int *SC, double *fm,
                             double *lm) {
    return pava_range<PavaHostLanes>(v, lo, hi, vio, nv, S, SC, fm, lm);
}

// The same over the whole input v[0..L).
inline void pava_sparse(const double *v, int L, const int *vio, int nv, double *S, int *SC, int *npools) {
    double fm, lm;
    *npools = pava_sparse_range(v, 0, L, vio, nv, S, SC, &fm, &lm);
}

// Pool-adjacent-violators over v[0..L) by the whole block from its known
// violations vio[0..nv) (increasing), with the arithmetic of the serial
// stack form.  The input is cut where every value before is below every
// value after (no pool can reach across such a cut); the stretches between
// cuts that hold violations run pava_wave_range, one wave each.  Where
// the last pool of a stretch has a mean above a value the first pool of the
// next one takes (rounding can put a pool's mean above its largest value),
// the serial pass would have merged across the cut: those cuts are dropped
// and the stretches run again, until no cut is crossed -- then the pools are
// those of the serial pass, sums and means bit for bit.  At most PAVA_MAXC
// stretches (neighbours beyond that are joined).  LDS: S [L] doubles, SC [L]
// ints (first the last cut at or before every position), and the stretch
// tables.
constexpr int PAVA_MAXC = 512;

struct PavaChunks {
    int cb[PAVA_MAXC + 1];  // stretch bounds
    int fv[PAVA_MAXC + 1];  // first violation of each stretch
    int np[PAVA_MAXC];      // stored pools of each stretch
    int pst[PAVA_MAXC + 1];  // number of the first of them over all stretches
    double fm[PAVA_MAXC], lm[PAVA_MAXC];
    double wmax[16], wmin[16];
    int nc, drop, wsum[16];
};

__device__ inline void pava_block_chunked(double *v, int L, const int *vio, int nv, double *S, int *SC,
                                          PavaChunks &pc) {
    const int nt = (int)blockDim.x, tid = (int)threadIdx.x;
    const int lane = tid & 63, w = tid >> 6;
    // Cuts: positions b with max(v[0..b)) < min(v[b..L)), where no pool can
    // reach across.  Every thread takes a contiguous run of the values.
    const int per = (L + nt - 1) / nt;
    const int j0 = min(tid * per, L), j1 = min(j0 + per, L);
    {
        double cmax = -INFINITY, cmin = INFINITY;
        for (int j = j0; j < j1; ++j) {
            cmax = fmax(cmax, v[j]);
            cmin = fmin(cmin, v[j]);
        }
        // exclusive prefix max and exclusive suffix min over the threads' runs
        double pmx = cmax, smn = cmin;
        for (int off = 1; off < 64; off <<= 1) {
            const double u = __shfl_up(pmx, off), d = __shfl_down(smn, off);
            if (lane >= off) pmx = fmax(pmx, u);
            if (lane + off < 64) smn = fmin(smn, d);
        }
        if (lane == 63) pc.wmax[w] = pmx;
        if (lane == 0) pc.wmin[w] = smn;
        __syncthreads();
        double before = __shfl_up(pmx, 1), after = __shfl_down(smn, 1);
        if (lane == 0) before = -INFINITY;
        if (lane == 63) after = INFINITY;
        for (int k = 0; k < nt / 64; ++k) {
            if (k < w) before = fmax(before, pc.wmax[k]);
            if (k > w) after = fmin(after, pc.wmin[k]);
        }
        // cut flags of the run: SC[b] = b at a cut, else 0
        double run_max = before;
        for (int b = j0; b < j1; ++b) {
            double suf = after;
            for (int j = j1 - 1; j >= b; --j) suf = fmin(suf, v[j]);
            SC[b] = (b > 0 && run_max < suf) ? b : 0;
            run_max = fmax(run_max, v[b]);
        }
        __syncthreads();
        // SC[j] = the last cut at or before j: inclusive prefix max
        int rmx = 0;
        for (int j = j0; j < j1; ++j) rmx = max(rmx, SC[j]);
        int inc = rmx;
        for (int off = 1; off < 64; off <<= 1) {
            const int u = __shfl_up(inc, off);
            if (lane >= off) inc = max(inc, u);
        }
        if (lane == 63) pc.wsum[w] = inc;
        __syncthreads();
        int carry = __shfl_up(inc, 1);
        if (lane == 0) carry = 0;
        for (int k = 0; k < w; ++k) carry = max(carry, pc.wsum[k]);
        for (int j = j0; j < j1; ++j) {
            carry = max(carry, SC[j]);
            SC[j] = carry;
        }
        __syncthreads();
    }
    // stretches: a new one at every violation whose last cut differs from its
    // predecessor's; at most PAVA_MAXC of them, evenly
    {
        const int fper = (nv + nt - 1) / nt;
        const int f0 = tid * fper, f1 = min(f0 + fper, nv);
        int cnt = 0;
        for (int f = f0; f < f1; ++f) cnt += (f == 0 || SC[vio[f]] != SC[vio[f - 1]]) ? 1 : 0;
        int inc = cnt;
        for (int off = 1; off < 64; off <<= 1) {
            const int t = __shfl_up(inc, off);
            if (lane >= off) inc += t;
        }
        if (lane == 63) pc.wsum[w] = inc;
        __syncthreads();
        int base = inc - cnt, total = 0;
        for (int k = 0; k < nt / 64; ++k) {
            if (k < w) base += pc.wsum[k];
            total += pc.wsum[k];
        }
        const int stride = (total + PAVA_MAXC - 1) / PAVA_MAXC;
        for (int f = f0; f < f1; ++f)
            if (f == 0 || SC[vio[f]] != SC[vio[f - 1]]) {
                if (base % stride == 0) {
                    const int k = base / stride;
                    pc.fv[k] = f;
                    pc.cb[k] = f == 0 ? 0 : SC[vio[f]];
                }
                ++base;
            }
        __syncthreads();
        if (tid == 0) {
            const int nc = (total + stride - 1) / stride;
            pc.nc = nc;
            pc.cb[nc] = L;
            pc.fv[nc] = nv;
        }
        __syncthreads();
    }
    while (true) {
        const int nc = pc.nc;
        for (int k = w; k < nc; k += nt / 64) {  // one wave per stretch
            double fm, lm;
            const int np = pava_wave_range(v, pc.cb[k], pc.cb[k + 1], vio + pc.fv[k],
                                                   pc.fv[k + 1] - pc.fv[k], S, SC, &fm, &lm);
            if (lane == 0) {
                pc.np[k] = np;
                pc.fm[k] = fm;
                pc.lm[k] = lm;
            }
        }
        __syncthreads();
        // keep cut k (1 <= k < nc) unless the serial pass would cross it
        const int per = (nc + nt - 1) / nt;
        const int k0 = tid * per, k1 = min(k0 + per, nc);
        int cnt = 0;
        for (int k = k0; k < k1; ++k) cnt += (k == 0 || !(pc.lm[k - 1] > pc.fm[k])) ? 1 : 0;
        int inc = cnt;
        for (int off = 1; off < 64; off <<= 1) {
            const int t = __shfl_up(inc, off);
            if (lane >= off) inc += t;
        }
        if (lane == 63) pc.wsum[w] = inc;
        __syncthreads();
        int base = inc - cnt, total = 0;
        for (int k = 0; k < nt / 64; ++k) {
            if (k < w) base += pc.wsum[k];
            total += pc.wsum[k];
        }
        if (total == nc) break;  // every cut holds (uniform: total is the block's sum)
        // compact the kept cuts in place: kept cut k moves to base <= k, so
        // read every kept value before any write
        int keep_cb[8], keep_fv[8], nk = 0;
        for (int k = k0; k < k1 && nk < 8; ++k)
            if (k == 0 || !(pc.lm[k - 1] > pc.fm[k])) {
                keep_cb[nk] = pc.cb[k];
                keep_fv[nk] = pc.fv[k];
                ++nk;
            }
        __syncthreads();
        for (int t = 0; t < nk; ++t) {
            pc.cb[base + t] = keep_cb[t];
            pc.fv[base + t] = keep_fv[t];
        }
        if (tid == 0) {
            pc.nc = total;
            pc.cb[total] = L;
            pc.fv[total] = nv;
        }
        __syncthreads();
    }
    // write the means of the stored pools of every stretch, one wave per
    // pool: the pools numbered through an exclusive scan of their counts
    const int nc = pc.nc;
    {
        const int per = (nc + nt - 1) / nt;
        const int k0 = min(tid * per, nc), k1 = min(k0 + per, nc);
        int cnt = 0;
        for (int k = k0; k < k1; ++k) cnt += pc.np[k];
        int inc = cnt;
        for (int off = 1; off < 64; off <<= 1) {
            const int t = __shfl_up(inc, off);
            if (lane >= off) inc += t;
        }
        if (lane == 63) pc.wsum[w] = inc;
        __syncthreads();
        int base = inc - cnt, total = 0;
        for (int k = 0; k < nt / 64; ++k) {
            if (k < w) base += pc.wsum[k];
            total += pc.wsum[k];
        }
        for (int k = k0; k < k1; ++k) {
            pc.pst[k] = base;
            base += pc.np[k];
        }
        if (tid == 0) pc.pst[nc] = total;
        __syncthreads();
    }
    const int total = pc.pst[nc], wl = min(64, nt - 64 * w);  // lanes of this wave
    for (int g = w; g < total; g += (nt + 63) / 64) {
        int a = 0, b = nc;  // the stretch holding pool g: pst[a] <= g < pst[b]
        while (b - a > 1) {
            const int mid = (a + b) >> 1;
            if (pc.pst[mid] <= g) a = mid;
            else b = mid;
        }
        const int idx = pc.cb[a] + (g - pc.pst[a]);
        const int cq = SC[idx] & 0xFFFF, st = SC[idx] >> 16;
        const double mean = S[idx] / (double)cq;
        for (int t = lane; t < cq; t += wl) v[st + t] = mean;
    }
    __syncthreads();
}

// Pool-adjacent-violators over v[0..L) (L < 65536) by the whole block, with
// the arithmetic of the serial stack form: the violations v[j] > v[j+1] are found
// in parallel; without any, v is already the result; otherwise one wave
// builds the pools and the block writes their means.  LDS:
// S [L] doubles, SC and vio [L] ints.  Every thread of the block calls it.
__device__ inline void pava_block(double *v, int L, double *S, int *SC, int *vio) {
#pragma clang fp contract(off)
    __shared__ int wsum[16], npools;
    const int nt = (int)blockDim.x, nw = (nt + 63) / 64;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    // the violations in order, nt indices at a time
    int nbad = 0;
    for (int j0 = 0; j0 < L - 1; j0 += nt) {
        const int j = j0 + (int)threadIdx.x;
        const bool bad = j < L - 1 && v[j] > v[j + 1];
        const uint64_t all = __ballot(bad);
        if (j0) __syncthreads();  // the last round's counts have been read
        if (lane == 0) wsum[w] = __popcll(all);
        __syncthreads();
        int at = nbad + __popcll(all & ((1ull << lane) - 1ull));
        for (int k = 0; k < nw; ++k) {
            at += k < w ? wsum[k] : 0;
            nbad += wsum[k];
        }
        if (bad) vio[at] = j;
    }
    if (nbad == 0) return;
    __syncthreads();
    if (w == 0) {  // the whole first wave runs the pass
        double fm, lm;
        const int np = pava_wave_range(v, 0, L, vio, nbad, S, SC, &fm, &lm);
        if (lane == 0) npools = np;
    }
    __syncthreads();
    const int wl = min(64, nt - 64 * w);  // lanes of this wave
    for (int q = w; q < npools; q += (nt + 63) / 64) {  // one wave per pool
        const int cq = SC[q] & 0xFFFF, st = SC[q] >> 16;
        const double mean = S[q] / (double)cq;
        for (int t = lane; t < cq; t += wl) v[st + t] = mean;
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------
// One link of a serial chain by one block: qc (LDS, the knots q^n) becomes
// J(C_n(q^n), q_f, q_c^*), or C_n(q^n) without qf.  Es: E of the slice, En: E of
// the next link (any E behind the last).  lds: chain_lds() bytes.  Every thread
// of the block calls it; the result is complete when it returns.
//
// The product E rho is spread over the block's 16 waves, row r on wave r mod
// 16, in groups of CHAIN_ROWS rows per wave.  STREAM (rows of at most 256
// cells): the next group of rows is always on its way in registers while one is
// multiplied, behind the last of a link the first of the next one, which does
// not depend on the knots and arrives while these are worked out.  What bounds
// the product is the one CU's rate of loads, one per wave and 16 clocks: in
// loads of 8 bytes per lane, a reduction per row, it took 17800 of a link's
// 28000 clocks (200 cells, 100 knots), with the next rows on their way 17000, in
// loads of 16 bytes 9400 of 18500.  The rest is latency: the knots' searches, the
// masses' running sum and the monotone repair.  Longer rows are loaded four at
// a time as they are needed.
// ---------------------------------------------------------------------------
constexpr int CHAIN_THREADS = 1024;
constexpr int CHAIN_ROWS = 4;
constexpr int CHAIN_STREAM_CELLS = 256;

// Two groups of a wave's rows of E in registers (rows of at most 256 cells).
// Half a wave holds a row: its lane l the elements 2 l + 64 u and 2 l + 1 + 64 u,
// in loads of 16 bytes (a CU issues one load per wave and 16 clocks, of 8 or of
// 16 bytes per lane).  The sums are those of lane_row_dot and wave_sum: lane c
// there takes the elements c + 64 u.
struct ChainStream {
    typedef double Pair __attribute__((ext_vector_type(2)));
    typedef double Pair8 __attribute__((ext_vector_type(2), aligned(8)));  // as it lies in E
    Pair e[2][CHAIN_ROWS / 2][4];

    // Rows k = 2 p + half of group grp: (grp CHAIN_ROWS + k) 16 + wave.  Rows past
    // the end are read at the last one, elements past it at the pair from the last
    // one on (E has one more element behind its last row): no load waits behind
    // a condition.
    __device__ __forceinline__ void load(int b, const double *E, int cells, int grp) {
        // in scalar registers, and known to be global memory
        using Global = const __attribute__((address_space(1))) char *;
        const Global base = (Global)uniform_i64((int64_t)E);
        const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = (int)(threadIdx.x & 63);
#pragma unroll
        for (int p = 0; p < CHAIN_ROWS / 2; ++p) {
            const int r = (grp * CHAIN_ROWS + 2 * p + (lane >> 5)) * (CHAIN_THREADS / 64) + wave;
            const uint32_t row = (uint32_t)min(r, cells - 1) * (uint32_t)cells;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t off = 8u * (row + (uint32_t)min(2 * (lane & 31) + 64 * u, cells - 1));
                e[b][p][u] = *(const __attribute__((address_space(1))) Pair8 *)(base + off);
            }
        }
    }
    // rho2 = max(E rho, 0) for group grp in slot b; v: the lane's elements of
    // rho, 0 past the end.
    __device__ __forceinline__ void apply(int b, const Pair *v, int cells, int grp, double *rho2) const {
#pragma clang fp contract(off)
        const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = (int)(threadIdx.x & 63);
        Pair acc[2];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            acc[p] = Pair{0.0, 0.0};
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                acc[p].x = fma(e[b][p][u].x, v[u].x, acc[p].x);
                acc[p].y = fma(e[b][p][u].y, v[u].y, acc[p].y);
            }
        }
        // elements c ^ 32: the other row of 16 lanes, the two pairs' side by side
        auto fold = [](double x, double y) {
            const long long p = __double_as_longlong(x), q = __double_as_longlong(y);
            const auto l = __builtin_amdgcn_permlane16_swap((unsigned)p, (unsigned)q, false, false);
            const auto h = __builtin_amdgcn_permlane16_swap((unsigned)(p >> 32), (unsigned)(q >> 32), false, false);
            return __longlong_as_double((long long)(((unsigned long long)h[0] << 32) | l[0])) +
                   __longlong_as_double((long long)(((unsigned long long)h[1] << 32) | l[1]));
        };
        Pair w{fold(acc[0].x, acc[1].x), fold(acc[0].y, acc[1].y)};
        w.x += dpp_f64<0x128>(w.x);  // c ^ 16: row_ror:8
        w.y += dpp_f64<0x128>(w.y);
        w.x += dpp_f64<0x124>(w.x);
        w.y += dpp_f64<0x124>(w.y);
        w.x += dpp_f64<0x122>(w.x);
        w.y += dpp_f64<0x122>(w.y);
        w.x += dpp_f64<0x121>(w.x);
        w.y += dpp_f64<0x121>(w.y);
        const double sum = w.x + w.y;  // c ^ 1
        const int t = lane >> 4, k = ((t & 1) << 1) | (t >> 1);
        const int r = (grp * CHAIN_ROWS + k) * (CHAIN_THREADS / 64) + wave;
        if ((lane & 15) == 0 && r < cells) rho2[r] = sum > 0.0 ? sum : 0.0;
    }
    __device__ __forceinline__ void start(const double *E, int cells) { load(0, E, cells, 0); }
    __device__ __forceinline__ void product(const double *Es, const double *En, const double *rho, int cells,
                                            double *rho2) {
        const int lane = (int)(threadIdx.x & 63);
        Pair v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = 2 * (lane & 31) + 64 * u;
            const double a = rho[min(j, cells - 1)], b = rho[min(j + 1, cells - 1)];
            v[u] = Pair{j < cells ? a : 0.0, j + 1 < cells ? b : 0.0};
        }
        // groups in pairs: 2 for up to 128 rows, else 4
        const int groups = cells <= 2 * CHAIN_ROWS * (CHAIN_THREADS / 64) ? 2 : 4;
#pragma unroll 1
        for (int grp = 0; grp < groups; grp += 2) {
            const bool last = grp + 2 >= groups;
            load(1, Es, cells, grp + 1);
            apply(0, v, cells, grp, rho2);
            load(0, last ? En : Es, cells, last ? 0 : grp + 2);
            apply(1, v, cells, grp + 1, rho2);
        }
    }
};
static_assert(CHAIN_ROWS == 4, "the fold puts two pairs of rows side by side");

inline size_t chain_lds(const GridDev &g) {
    return sizeof(double) * (2 * (g.nq + 1) + 4 * g.cells + 2) + 2 * sizeof(int) * (g.nq + 1);
}

template <bool STREAM>
__device__ __forceinline__ void chain_link(ChainStream &stream, const double *__restrict__ Es,
                                           const double *__restrict__ En, const double *__restrict__ qf,
                                           const double *__restrict__ qcs, const GridDev &g, double *lds) {
#pragma clang fp contract(off)
    const int Q1 = g.nq + 1;
    double *qc = lds;               // Q1: current knots
    double *c = qc + Q1;            // cells + 1
    double *rho = c + g.cells + 1;  // cells
    double *rho2 = rho + g.cells;   // cells
    double *C = rho2 + g.cells;     // cells + 1
    double *S = C + g.cells + 1;    // Q1
    int *SC = (int *)(S + Q1);      // Q1
    int *vio = SC + Q1;             // Q1
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = (int)(blockDim.x >> 6);
    // the link's other inputs, wanted at its end, on their way from the start
    const int j0 = threadIdx.x;
    const double f0 = qf && j0 < Q1 ? qf[j0] : 0.0, s0 = qf && j0 < Q1 ? qcs[j0] : 0.0;
    for (int i = 1 + threadIdx.x; i < g.cells; i += blockDim.x) c[i] = cdf_knots(qc, g.nq, edge_at(g, i));
    __syncthreads();
    for (int i = threadIdx.x; i < g.cells; i += blockDim.x)
        rho[i] = (i == 0) ? c[1] : (i == g.cells - 1) ? 1.0 - c[g.cells - 1] : c[i + 1] - c[i];
    __syncthreads();
    if constexpr (STREAM) {
        stream.product(Es, En, rho, g.cells, rho2);
    } else {
        for (int r0 = wave; r0 < g.cells; r0 += nw * CHAIN_ROWS) {
            const double *rows[CHAIN_ROWS];
            double acc[CHAIN_ROWS];
#pragma unroll
            for (int k = 0; k < CHAIN_ROWS; ++k) {
                const int r = r0 + k * nw;
                rows[k] = Es + (int64_t)(r < g.cells ? r : r0) * g.cells;
            }
            lane_rows_dot<CHAIN_ROWS, 4>(rows, rho, g.cells, lane, acc);
#pragma unroll
            for (int k = 0; k < CHAIN_ROWS; ++k) {
                const double a = wave_sum(acc[k]);
                const int r = r0 + k * nw;
                if (lane == 0 && r < g.cells) rho2[r] = a > 0.0 ? a : 0.0;
            }
        }
    }
    __syncthreads();
    masses_to_knots_block<STREAM ? CHAIN_STREAM_CELLS / 64 : 16>(rho2, C, g, qc);
    __syncthreads();
    if (qf) {
        if (j0 < Q1) qc[j0] = f0 + (qc[j0] - s0);
        for (int j = j0 + blockDim.x; j < Q1; j += blockDim.x) qc[j] = qf[j] + (qc[j] - qcs[j]);
        __syncthreads();
        pava_block(qc, Q1, S, SC, vio);
    }
}

}  // namespace pr
