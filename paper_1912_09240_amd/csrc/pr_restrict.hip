// Restriction to the empirical quantile function (Sec. 3.2.2, Sec. 4.4):
// a segmented sort of the slow coordinates of many ensembles (one segment
// per ensemble, equal or unequal lengths) by (key, particle), followed by
// the midpoint (Hazen) knots; the moments (eq. (MCestimator)) and the cell
// histogram (eq. (binning)) are fused into the first read of the values.
// Ensembles of up to 2^20 + 2^16 keys take the splitter sort (sample,
// buckets, one LDS sort per bucket; described with its kernels below); longer
// ones the radix sort.
//
// Radix sort design (HBM bound): 8-bit digits, one pass per byte of the
// orderable key.  A pass is
//   count   digit histogram of every tile (ITEMS x 256 keys),
//   rowscan one wave per (segment, digit) -- one block per segment in the
//           segment-table layout: exclusive prefix of that digit's tile
//           counts and the digit total of the segment,
//   scatter stable rank of every key inside its tile (each wave ranks its
//           keys in order with ballot-built peer masks), exclusive scan of
//           the digit totals, then the tile is staged in LDS in digit order
//           and every digit run is written to HBM as a contiguous burst.
// Equal digits keep tile order, so every pass is stable and the sort orders
// by (key, particle).  The first pass reads FP64 (or FP32) values directly
// and generates the particle index as payload; the last pass writes the
// outputs asked for (rank by scatter, perm and sorted values in order).  A
// sort that only needs knots carries no payload.  64-bit keys run only the
// four passes over their high halves, then a fix-up pass (rs_fixup) that
// orders every run of equal high halves and writes the last pass's outputs
// (the ranks of a segment table through a staging buffer instead of stores to
// random addresses, rs_rank_bucket and rs_rank_place); the complete sort
// follows, guarded by a flag that the fix-up raises only for a run longer than
// it handles.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "pr_internal.hpp"

namespace pr {

constexpr int RS_THREADS = 256;
constexpr int RS_WAVES = RS_THREADS / 64;
constexpr int RS_RADIX = 256;
constexpr int RS_ITEMS = 16;  // keys per thread and tile (tiles of RS_THREADS x RS_ITEMS keys)
constexpr int RK_SHIFT = 12;  // bits of a place in a tile

template <typename K> struct KeyTraits;
template <> struct KeyTraits<uint64_t> { using V = double; static constexpr int passes = 8; };
template <> struct KeyTraits<uint32_t> { using V = float;  static constexpr int passes = 4; };

// Key buffer (0 or 1) of the workspace that holds the sorted keys when a
// sort ends: 64-bit keys end in buffer 0 (the fix-up after the passes over
// the high halves, or the complete sort arranged to end there), 32-bit keys
// in the buffer the last of their 4 passes writes.
template <typename K>
constexpr int sorted_buffer() { return std::is_same<K, uint64_t>::value ? 0 : 1; }

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Exclusive prefix of one value per thread over a 256-thread block.
__device__ __forceinline__ uint32_t block_exclusive_256(uint32_t v, uint32_t *wtot) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t inc = v;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t t = __shfl_up(inc, off);
        if (lane >= off) inc += t;
    }
    if (lane == 63) wtot[wave] = inc;
    __syncthreads();
    uint32_t pre = 0;
    for (int w = 0; w < wave; ++w) pre += wtot[w];
    __syncthreads();
    return pre + inc - v;
}

struct HistArgs {
    uint32_t *hist;  // [segments][cells] or NULL
    int cells;
    double lo, inv_h;
};

struct TileRef {
    int seg, blk, nblk;
    int64_t base, n, tile0;
};

// Tile processed by block b of nb.  Blocks are handed to the 8 XCDs round
// robin (block b runs on XCD b mod 8) and every XCD has its own L2, so each
// XCD takes one contiguous range of tiles: neighbouring tiles share cache
// lines of the per-tile count columns and of the digit runs they write, and
// those lines then fill up in one L2 instead of being written partially from
// several.
__device__ __forceinline__ int64_t xcd_tile(int64_t b, int64_t nb) {
    constexpr int64_t X = 8;
    const int64_t q = nb / X, r = nb % X;
    const int64_t x = b % X, i = b / X;
    return x < r ? x * (q + 1) + i : r * (q + 1) + (x - r) * q + i;
}

template <bool VAR>
__device__ __forceinline__ TileRef tile_ref(const SortLayout &L, int64_t t) {
    TileRef r;
    if constexpr (VAR) {
        r.seg = L.tile_seg[t];
        const SortSeg s = L.segs[r.seg];
        r.blk = (int)(t - s.tile0);
        r.nblk = s.nblk;
        r.base = s.base;
        r.n = s.n;
        r.tile0 = s.tile0;
    } else {
        r.seg = (int)(t / L.nblk);
        r.blk = (int)(t % L.nblk);
        r.nblk = L.nblk;
        r.base = (int64_t)r.seg * L.n;
        r.n = L.n;
        r.tile0 = (int64_t)r.seg * L.nblk;
    }
    return r;
}

template <bool VAR>
__device__ __forceinline__ void seg_ref(const SortLayout &L, int s, int64_t &base, int64_t &n, int64_t &tile0,
                                        int &nblk, int &qrow) {
    if constexpr (VAR) {
        const SortSeg g = L.segs[s];
        base = g.base;
        n = g.n;
        tile0 = g.tile0;
        nblk = g.nblk;
        qrow = g.qrow;
    } else {
        base = (int64_t)s * L.n;
        n = L.n;
        tile0 = (int64_t)s * L.nblk;
        nblk = L.nblk;
        qrow = s;
    }
}

// ---------------------------------------------------------------------------
// Count.
// ---------------------------------------------------------------------------
template <typename K, int ITEMS, bool FIRST, bool VAR>
__global__ void __launch_bounds__(RS_THREADS)
rs_count(const void *__restrict__ src, int shift, SortLayout L, uint32_t *__restrict__ counts,
         double *__restrict__ mom_part, HistArgs ha) {
    using V = typename KeyTraits<K>::V;
    constexpr int WAVE_KEYS = 64 * ITEMS, TILE = RS_THREADS * ITEMS;
    // two copies of every wave's histogram (even and odd lanes) halve the
    // same-address serialisation of the LDS atomics when few digits occur
    __shared__ uint32_t h[RS_WAVES][2][RS_RADIX];
    __shared__ double wsum[RS_WAVES][4];
    extern __shared__ uint32_t cell_h[];
    if (L.guard && *L.guard == 0) return;
    const TileRef T = tile_ref<VAR>(L, xcd_tile(blockIdx.x, gridDim.x));
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    for (int i = tid; i < RS_WAVES * 2 * RS_RADIX; i += RS_THREADS) (&h[0][0][0])[i] = 0;
    const bool do_hist = FIRST && ha.hist != nullptr;
    if (do_hist)
        for (int i = tid; i < ha.cells; i += RS_THREADS) cell_h[i] = 0;
    __syncthreads();
    const int64_t t0 = (int64_t)T.blk * TILE + wave * WAVE_KEYS;
    // all loads of the tile first, so that they are in flight together
    using In = typename std::conditional<FIRST, V, K>::type;
    In in[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int64_t idx = t0 + i * 64 + lane;
        in[i] = idx < T.n ? ((const In *)src)[T.base + idx] : (In)0;
    }
    double s1 = 0, s2 = 0, s3 = 0, s4 = 0;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int64_t idx = t0 + i * 64 + lane;
        if (idx < T.n) {
            K key;
            if constexpr (FIRST) {
                const V v = in[i];
                key = key_of(v);
                const double xv = (double)v;
                const double x2 = xv * xv;
                s1 += xv;
                s2 += x2;
                s3 += x2 * xv;
                s4 += x2 * x2;
                if (do_hist) {
                    double c = floor((xv - ha.lo) * ha.inv_h);
                    c = fmin(fmax(c, 0.0), (double)(ha.cells - 1));
                    atomicAdd(&cell_h[(int)c], 1u);
                }
            } else {
                key = in[i];
            }
            atomicAdd(&h[wave][lane & 1][(uint32_t)(key >> shift) & 0xFFu], 1u);
        }
    }
    if (FIRST && mom_part != nullptr) {
        for (int off = 32; off >= 1; off >>= 1) {  // fixed butterfly
            s1 += __shfl_xor(s1, off);
            s2 += __shfl_xor(s2, off);
            s3 += __shfl_xor(s3, off);
            s4 += __shfl_xor(s4, off);
        }
        if (lane == 0) {
            wsum[wave][0] = s1;
            wsum[wave][1] = s2;
            wsum[wave][2] = s3;
            wsum[wave][3] = s4;
        }
    }
    __syncthreads();
    {
        const int d = tid;  // RS_THREADS == RS_RADIX
        uint32_t c = 0;
#pragma unroll
        for (int w = 0; w < RS_WAVES; ++w) c += h[w][0][d] + h[w][1][d];
        counts[T.tile0 * RS_RADIX + (int64_t)d * T.nblk + T.blk] = c;
    }
    if (FIRST && mom_part != nullptr && tid < 4) {
        double t = 0;
        for (int w = 0; w < RS_WAVES; ++w) t += wsum[w][tid];
        mom_part[(T.tile0 + T.blk) * 4 + tid] = t;
    }
    if (do_hist)
        for (int i = tid; i < ha.cells; i += RS_THREADS)
            if (cell_h[i]) atomicAdd(&ha.hist[(int64_t)T.seg * ha.cells + i], cell_h[i]);
}

// ---------------------------------------------------------------------------
// Row scan: one wave per (segment, digit).
// ---------------------------------------------------------------------------
template <bool VAR>
__global__ void __launch_bounds__(256) rs_rowscan(uint32_t *__restrict__ counts, uint32_t *__restrict__ totals,
                                                  SortLayout L) {
    if (L.guard && *L.guard == 0) return;
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= (int64_t)L.nseg * RS_RADIX) return;
    const int lane = threadIdx.x & 63;
    const int s = (int)(row >> 8), d = (int)(row & 255);
    int64_t base, n, tile0;
    int nblk, qrow;
    seg_ref<VAR>(L, s, base, n, tile0, nblk, qrow);
    uint32_t *c = counts + tile0 * RS_RADIX + (int64_t)d * nblk;
    uint32_t carry = 0;
    for (int c0 = 0; c0 < nblk; c0 += 64) {
        const int i = c0 + lane;
        const uint32_t v = i < nblk ? c[i] : 0u;
        uint32_t inc = v;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t t = __shfl_up(inc, off);
            if (lane >= off) inc += t;
        }
        if (i < nblk) c[i] = carry + inc - v;
        carry += __shfl(inc, 63);
    }
    if (lane == 0) totals[(int64_t)s * RS_RADIX + d] = carry;
}

// Row scan for many short segments (the segment-table layout): one block per
// segment, one thread per digit walking that digit's tile counts, so that a
// launch has one block per segment instead of one wave per (segment, digit).
template <bool VAR>
__global__ void __launch_bounds__(256) rs_rowscan_seg(uint32_t *__restrict__ counts, uint32_t *__restrict__ totals,
                                                      SortLayout L) {
    if (L.guard && *L.guard == 0) return;
    const int s = blockIdx.x, d = threadIdx.x;  // RS_RADIX threads
    int64_t base, n, tile0;
    int nblk, qrow;
    seg_ref<VAR>(L, s, base, n, tile0, nblk, qrow);
    uint32_t *c = counts + tile0 * RS_RADIX + (int64_t)d * nblk;
    uint32_t carry = 0;
    for (int b = 0; b < nblk; ++b) {
        const uint32_t v = c[b];
        c[b] = carry;
        carry += v;
    }
    totals[(int64_t)s * RS_RADIX + d] = carry;
}

// ---------------------------------------------------------------------------
// Scatter.
// ---------------------------------------------------------------------------
template <typename K, int ITEMS, bool FIRST, bool LAST, bool PAYLOAD, bool VAR>
__global__ void __launch_bounds__(RS_THREADS)
rs_scatter(const void *__restrict__ src, const uint32_t *__restrict__ vals_in, K *__restrict__ keys_out,
           uint32_t *__restrict__ vals_out, const uint32_t *__restrict__ counts,
           const uint32_t *__restrict__ totals, int shift, SortLayout L, uint32_t *__restrict__ rank_out,
           uint32_t *__restrict__ perm_out, double *__restrict__ xs_out) {
    using V = typename KeyTraits<K>::V;
    constexpr int WAVE_KEYS = 64 * ITEMS, TILE = RS_THREADS * ITEMS;
    __shared__ uint32_t wcnt[RS_WAVES][RS_RADIX];
    __shared__ uint32_t wbase[RS_WAVES][RS_RADIX];
    __shared__ uint32_t gdelta[RS_RADIX];
    __shared__ uint32_t wtot[RS_WAVES];
    __shared__ K stage[TILE];  // keys, then (reused) payload

    if (L.guard && *L.guard == 0) return;
    const TileRef T = tile_ref<VAR>(L, xcd_tile(blockIdx.x, gridDim.x));
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int64_t t0 = (int64_t)T.blk * TILE + wave * WAVE_KEYS;
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));

    for (int i = lane; i < RS_RADIX; i += 64) wcnt[wave][i] = 0;
    wave_sync();

    K key[ITEMS];
    uint32_t val[ITEMS];
    uint32_t rnk[ITEMS];
    // all loads of the tile first, so that they are in flight together (a
    // conversion next to each load made every load wait for the one before)
    using In = typename std::conditional<FIRST, V, K>::type;
    In in[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int64_t idx = t0 + i * 64 + lane;
        in[i] = idx < T.n ? ((const In *)src)[T.base + idx] : (In)0;
        val[i] = 0;
        if constexpr (PAYLOAD && !FIRST)
            if (idx < T.n) val[i] = vals_in[T.base + idx];
    }
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int64_t idx = t0 + i * 64 + lane;
        key[i] = 0;
        if (idx < T.n) {
            if constexpr (FIRST) {
                key[i] = key_of(in[i]);
                val[i] = (uint32_t)idx;
            } else {
                key[i] = in[i];
            }
        }
    }
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const bool valid = t0 + i * 64 + lane < T.n;
        const uint32_t d = (uint32_t)(key[i] >> shift) & 0xFFu;
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bal = __ballot(bit);
            peers &= bit ? bal : ~bal;
        }
        uint32_t base = 0;
        if (valid) base = wcnt[wave][d];
        rnk[i] = base + (uint32_t)__popcll(peers & lt);
        wave_sync();
        if (valid && lane == 63 - __clzll(peers)) wcnt[wave][d] = base + (uint32_t)__popcll(peers);
        wave_sync();
    }
    __syncthreads();
    {
        const int d = tid;
        uint32_t c[RS_WAVES], tot = 0;
#pragma unroll
        for (int w = 0; w < RS_WAVES; ++w) {
            c[w] = wcnt[w][d];
            tot += c[w];
        }
        const uint32_t lstart = block_exclusive_256(tot, wtot);
        const uint32_t dbase = block_exclusive_256(totals[(int64_t)T.seg * RS_RADIX + d], wtot);
        uint32_t acc = lstart;
#pragma unroll
        for (int w = 0; w < RS_WAVES; ++w) {
            wbase[w][d] = acc;
            acc += c[w];
        }
        gdelta[d] = dbase + counts[T.tile0 * RS_RADIX + (int64_t)d * T.nblk + T.blk] - lstart;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        if (t0 + i * 64 + lane < T.n) {
            const uint32_t d = (uint32_t)(key[i] >> shift) & 0xFFu;
            stage[wbase[wave][d] + rnk[i]] = key[i];
        }
    }
    __syncthreads();
    const int64_t rem = T.n - (int64_t)T.blk * TILE;
    const int tile_n = rem < TILE ? (int)rem : TILE;
    uint32_t gpos[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int j = tid + r * RS_THREADS;
        gpos[r] = 0xFFFFFFFFu;
        if (j < tile_n) {
            const K k = stage[j];
            const uint32_t g = (uint32_t)j + gdelta[(uint32_t)(k >> shift) & 0xFFu];
            if ((int64_t)g < T.n) {  // always true for a consistent scan
                gpos[r] = g;
                keys_out[T.base + g] = k;
                if (LAST && xs_out) xs_out[T.base + g] = value_of(k);
            }
        }
    }
    if constexpr (PAYLOAD) {
        __syncthreads();
        uint32_t *sv = (uint32_t *)stage;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            if (t0 + i * 64 + lane < T.n) {
                const uint32_t d = (uint32_t)(key[i] >> shift) & 0xFFu;
                sv[wbase[wave][d] + rnk[i]] = val[i];
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) {
            const int j = tid + r * RS_THREADS;
            if (j < tile_n && gpos[r] != 0xFFFFFFFFu) {
                const uint32_t v = sv[j];
                if (!LAST) {
                    vals_out[T.base + gpos[r]] = v;
                } else if ((int64_t)v < T.n) {
                    if (rank_out) rank_out[T.base + v] = gpos[r];
                    if (perm_out) perm_out[T.base + gpos[r]] = v;
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Splitter sort of ensembles of up to SS_MAX_N keys (equal lengths or a
// segment table): the keys of every ensemble are first distributed over
// ss_buckets(n) buckets (about 4096 keys each) by splitters drawn from a
// sample, then every bucket is ordered on its own in LDS.  An ensemble of at
// most SS_BIG keys (segment table: SS_CAP) is one bucket, read from the values
// themselves.
//   ss_sample       ss_runs() runs of SS_RUN keys per ensemble, one per block,
//                   each sorted and thinned to SS_KEEP keys;
//   ss_splitters    the thinned runs merged; splitter b is the merged key at
//                   the fraction b / ss_buckets(n);
//   ss_count        bucket histogram of every tile and the bucket of every
//                   key (one byte; the moments and the cell histogram fused
//                   into this first read of the values);
//   ss_rowscan(_seg) tile offsets and bucket totals;
//   ss_scatter      stable scatter of the keys into the buckets, and where
//                   every particle's key went: its bucket and its place among
//                   the tile's keys in bucket order;
//   ss_bucket_sort  one block per bucket: the keys go to value sub-buckets
//                   (linear in the value between the bucket's bounds, which
//                   keeps the order), every key counts the keys of its
//                   sub-bucket that precede it by (key, slot), and the bucket
//                   leaves in order, with the rank of every slot; where a
//                   sub-bucket is crowded (ties, outliers, values of many
//                   magnitudes), the bucket goes by the digits of its keys
//                   instead, in LDS as well;
//   ss_left         the buckets of SS_CAP..SS_BIG keys the same way, one block
//                   per CU, and longer ones by digits in global memory (not
//                   launched for ensembles of one bucket, which fit a block);
//   ss_finish       the rank of every particle from that of its slot (a tile's
//                   particles of one bucket hold neighbouring slots: the ranks
//                   are read as runs and put in particle order in LDS, none is
//                   stored to a random address); the knots and moments.
// The scatter is stable, so slots of equal keys are in particle order and the
// particles need not travel with the keys (only the permutation, where asked
// for, moves them).  Bytes per FP64 key with ranks: 62, of which the key's read
// and the rank's write (12) cannot be avoided.
//
// 64 FP64 ensembles of 2^20 (ranks, knots): 1.16 ms -- bucket sort 0.46 (20
// bytes per key, 2.9 TB/s; LDS), scatter 0.35 (4.0 TB/s), ranks 0.19, count
// 0.16, sample and splitters 0.06, what is left 0.05.  The scheme before it
// (splitters as means of the runs' quantiles, particles carried along, ranks
// staged by particle block, a complete guarded radix sort behind) took 1.37 ms
// where every bucket fitted and 5.70 ms where one did not, as for ensembles in
// two narrow wells.  33 FP32 ensembles of 99,991: 98 us (four radix passes:
// 170 us).  10 FP64 ensembles of 10^4: one kernel, 29 us (about forty
// launches of radix passes, fix-up and their guarded repetition: 160 us).
// ---------------------------------------------------------------------------
constexpr int SS_B = 256;
constexpr int SS_MAX_RUNS = 16;
constexpr int SS_RUN = 1024;                // sampled keys of a run
constexpr int SS_LIST = 64;                // of them sorted by one wave
constexpr int SS_KEEP = 256;                // of them kept
constexpr int SS_BT = 1024;                 // threads of a bucket block
constexpr int SS_IT = 7;                    // keys per thread of a bucket block
constexpr int SS_CAP = SS_BT * SS_IT;       // 7168: two bucket blocks share a CU's LDS
constexpr int SS_IT_BIG = 14;
constexpr int SS_BIG = SS_BT * SS_IT_BIG;   // 14336: one block takes 156 KiB of it
// Keys of a value sub-bucket above which the bucket goes by digits: the
// counting's time grows with them and with the keys per thread, that of the
// digits only with the latter.  FP32, 8 ensembles of 2^20 of 20,000 values (52 keys
// each): 396 us counted, 359 by digits; FP64, 64 of them: 2.63 and 3.48 ms.  HERE, FP64
// ensembles of one bucket, which wait for one block and not for the chip: with
// the line of the others 7168 keys of 140 values take 144 us instead of 90, 1000
// half of which are zero 69 instead of 25.
template <typename K, bool HERE>
constexpr uint32_t ss_crowded(uint32_t size) {
    return (sizeof(K) == 8 && !HERE ? 160u : 42u) << (size <= 1024 ? 2 : size <= 2048 ? 1 : 0);
}
// Above this the SS_B buckets average more than 4352 keys.  A bucket spans 64
// samples and its two splitters are each a few samples off (thinned runs): its
// size has a standard deviation of about 16 %, so one bucket in tens of
// thousands passes SS_CAP and none SS_BIG.
constexpr int64_t SS_MAX_N = ((int64_t)1 << 20) + ((int64_t)1 << 16);
// From here on a batch of unequal ensembles times both sorts.
constexpr int64_t SS_LARGE_N = (int64_t)1 << 16;
static_assert(SS_B == RS_RADIX, "buckets take the place of a radix pass's digits");
static_assert(SS_RUN == 4 * SS_KEEP && SS_RUN == 16 * SS_LIST, "a run's lists and its kept keys");

// Buckets of an ensemble of n keys: one where it fits a block, else one per
// tile of 4096, at most SS_B.  Equal ensembles are one bucket up to SS_BIG keys
// (10 of 10^4 keys: one kernel instead of seven), those of a segment table up
// to SS_CAP: the others' distribution is launched in any case, and above SS_CAP
// they would wait for one of 256 blocks in ss_left (637 segments of 2^12 to
// 2^15 keys: that took 156 us, now 10).
template <bool VAR>
__host__ __device__ __forceinline__ int ss_buckets(int64_t n) {
    if (n <= (VAR ? SS_CAP : SS_BIG)) return 1;
    const int64_t b = (n + RS_THREADS * RS_ITEMS - 1) / (RS_THREADS * RS_ITEMS);
    return b > SS_B ? SS_B : (int)b;
}
// Runs sampled of an ensemble with nb buckets: 64 samples per bucket, a power
// of two.
__host__ __device__ __forceinline__ int ss_runs(int nb) {
    int r = 1;
    while (r < SS_MAX_RUNS && 16 * r < nb) r <<= 1;
    return r;
}

// Bucket search.  The bucket of a key is the number of splitters
// sp[1..SS_B-1] at or below it, except that a key equal to a repeated splitter
// goes one below the last of them, so that the bucket between the two holds
// nothing else; it is non-decreasing in the key.  The search starts from a
// table over cells of equal width between the first and last splitters: the
// cell is non-decreasing in the value, so a splitter of a lower cell is below
// the key and one of a higher cell above it, and only the splitters of the
// key's own cell are left (one or none for smooth values, where eight steps
// over all of them would wait for LDS eight times).
constexpr int SS_CELLS = 1024;

template <typename K>
struct BucketSearch {
    K sp[SS_B];
    uint16_t first[SS_CELLS + 1];  // splitters 1.. in cells below
    double lo, scale;
    int nb;

    __device__ __forceinline__ int cell(K key) const {
        const double t = (value_of(key) - lo) * scale;
        if (t != t) return (key >> (8 * sizeof(K) - 1)) ? SS_CELLS - 1 : 0;  // NaN, or infinities: by the sign
        return t >= (double)SS_CELLS ? SS_CELLS - 1 : (t > 0.0 ? (int)t : 0);
    }
    // Called by a whole block; ready after the caller's next barrier.
    __device__ __forceinline__ void load(const K *split, int buckets) {
        const int tid = (int)threadIdx.x, nt = (int)blockDim.x;
        for (int i = tid; i < SS_B; i += nt) sp[i] = split[i];
        if (tid == 0) {
            nb = buckets;
            const double a = value_of(split[1]), b = value_of(split[buckets - 1]), w = b - a;
            lo = a;
            scale = (w > 0.0 && w <= 1.79e308) ? (double)SS_CELLS / w : 0.0;
        }
        __syncthreads();
        // splitter i (1..nb-1) fills the entries of the cells after its
        // predecessor's up to its own, the last one also those behind it
        for (int i = 1 + tid; i < buckets; i += nt) {
            const int c0 = i == 1 ? -1 : cell(sp[i - 1]), c1 = cell(sp[i]);
            for (int c = c0 + 1; c <= c1; ++c) first[c] = (uint16_t)(i - 1);
            if (i == buckets - 1)
                for (int c = c1 + 1; c <= SS_CELLS; ++c) first[c] = (uint16_t)i;
        }
    }
    __device__ __forceinline__ uint32_t operator()(K key) const {
        const int c = cell(key);
        int b = first[c], hi = first[c + 1];  // splitters 1..b are below the key, hi + 1.. above
        while (b < hi) {
            const int mid = (b + hi + 1) >> 1;
            if (sp[mid] <= key) b = mid;
            else hi = mid - 1;
        }
        if (b > 1 && sp[b] == key && sp[b - 1] == key) --b;
        return (uint32_t)b;
    }
};

// Whether bucket d of nb holds copies of one value only, by their splitters.  The
// scatter then writes it where the sorted keys go, and the rank of every slot
// is the slot's own number: nothing is left of it for a block of its own, however
// long it is (2^20 + 2^16 equal FP32 keys: 272 -> 89 us, FP64 399 -> 110).
template <typename K>
__device__ __forceinline__ bool one_value(const K *split, int d, int nb) {
    return d > 0 && d + 1 < nb && split[d] == split[d + 1];
}

// Merge of the sorted lists of len keys in a[0..m) (m / len a power of two)
// into out, pairs of neighbouring lists: a key's place is its index plus the
// number of the partner list's keys before it, equal keys of the first list
// before those of the second.  Called by a whole block.
template <typename K>
__device__ __forceinline__ void merge_pairs(const K *a, K *out, int m, int len) {
    for (int i = (int)threadIdx.x; i < m; i += (int)blockDim.x) {
        const int list = i / len, in = i % len;
        const K k = a[i], *o = a + (list ^ 1) * len;
        const bool first = (list & 1) == 0;
        int lo = 0, hi = len;  // o[0..lo) precede k
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (o[mid] < k || (!first && o[mid] == k)) lo = mid + 1;
            else hi = mid;
        }
        out[(list >> 1) * 2 * len + in + lo] = k;
    }
}

// One run: SS_RUN keys at positions spread over the ensemble, one in every
// n / (runs SS_RUN) at a place taken from a hash (a fixed stride could meet a
// period of the particles).  Every thread counts its wave's keys below its
// own, the sixteen lists are merged.
template <typename K, bool VAR>
__global__ void __launch_bounds__(SS_RUN)
ss_sample(const void *__restrict__ x, SortLayout L, int most_runs, K *__restrict__ runq) {
    using V = typename KeyTraits<K>::V;
    __shared__ K sk[2][SS_RUN];
    if (L.guard && *L.guard == 0) return;
    const int r = (int)blockIdx.x % most_runs, s = (int)blockIdx.x / most_runs, t = threadIdx.x;
    int64_t base, n, tile0;
    int nblk, qrow;
    seg_ref<VAR>(L, s, base, n, tile0, nblk, qrow);
    const int nb = ss_buckets<VAR>(n), runs = ss_runs(nb);
    if (nb == 1 || r >= runs) return;
    const uint32_t g = (uint32_t)(r * SS_RUN + t);
    uint32_t h = (g + 0x9E3779B9u * (uint32_t)s) * 0x85EBCA6Bu;
    h ^= h >> 15;
    h *= 0xC2B2AE35u;
    h ^= h >> 16;
    const uint64_t at = ((((uint64_t)g << 16) + (h & 0xFFFFu)) * (uint64_t)n) / ((uint64_t)(runs * SS_RUN) << 16);
    const K k = key_of(((const V *)x)[base + (int64_t)at]);
    sk[0][t] = k;
    __syncthreads();
    const int q0 = t & ~(SS_LIST - 1), in = t - q0;
    int below = 0;
#pragma unroll 8
    for (int j = 0; j < SS_LIST; ++j) {
        const K o = sk[0][q0 + j];
        below += (o < k || (o == k && j < in)) ? 1 : 0;
    }
    sk[1][q0 + below] = k;
    __syncthreads();
    int cur = 1;
    for (int len = SS_LIST; len < SS_RUN; len <<= 1, cur ^= 1) {
        merge_pairs(sk[cur], sk[cur ^ 1], SS_RUN, len);
        __syncthreads();
    }
    if (t < SS_KEEP) runq[((int64_t)s * SS_MAX_RUNS + r) * SS_KEEP + t] = sk[cur][4 * t + 2];
}

// The kept keys of the runs merged, then the splitters.  Splitters past the
// last bucket are the largest key; the place of splitter 0, which bounds
// nothing, says whether any bucket holds one value (see one_value).
template <typename K, bool VAR>
__global__ void __launch_bounds__(1024)
ss_splitters(const K *__restrict__ runq, SortLayout L, K *__restrict__ split) {
    __shared__ K buf[2][SS_MAX_RUNS * SS_KEEP];
    if (L.guard && *L.guard == 0) return;
    const int s = blockIdx.x, t = threadIdx.x;
    int64_t base, n, tile0;
    int nblk, qrow;
    seg_ref<VAR>(L, s, base, n, tile0, nblk, qrow);
    const int nb = ss_buckets<VAR>(n);
    if (nb == 1) return;
    const int M = ss_runs(nb) * SS_KEEP;
    for (int i = t; i < M; i += 1024) buf[0][i] = runq[(int64_t)s * SS_MAX_RUNS * SS_KEEP + i];
    __syncthreads();
    int cur = 0;
    for (int len = SS_KEEP; len < M; len <<= 1, cur ^= 1) {
        merge_pairs(buf[cur], buf[cur ^ 1], M, len);
        __syncthreads();
    }
    auto at = [&](int b) { return b < nb ? buf[cur][(int)((int64_t)b * M / nb)] : ~(K)0; };
    const bool twice = t > 0 && t + 1 < nb && at(t) == at(t + 1);
    const int any = __syncthreads_or(twice);
    if (t < SS_B) split[(int64_t)s * SS_B + t] = t == 0 ? (K)(any ? 1 : 0) : at(t);
}

// The tiles of the radix passes (RS_THREADS x RS_ITEMS keys) are taken by
// twice the threads with half the keys each in the splitter sort's
// per-key passes.
constexpr int SC_THREADS = 2 * RS_THREADS;
constexpr int SC_WAVES = SC_THREADS / 64;

template <typename K, bool VAR>
__global__ void __launch_bounds__(SC_THREADS)
ss_count(const void *__restrict__ src, const K *__restrict__ split, SortLayout L, uint32_t *__restrict__ counts,
         double *__restrict__ mom_part, HistArgs ha, uint32_t *__restrict__ bucket) {
    using V = typename KeyTraits<K>::V;
    constexpr int TILE = RS_THREADS * RS_ITEMS, ITEMS = TILE / SC_THREADS, WAVE_KEYS = 64 * ITEMS;
    __shared__ uint32_t h[SC_WAVES][2][RS_RADIX];
    __shared__ double wsum[SC_WAVES][4];
    __shared__ BucketSearch<K> bucket_of;
    extern __shared__ uint32_t cell_h[];
    if (L.guard && *L.guard == 0) return;
    const TileRef T = tile_ref<VAR>(L, xcd_tile(blockIdx.x, gridDim.x));
    const int nb = ss_buckets<VAR>(T.n);
    const bool do_hist = ha.hist != nullptr;
    if (nb == 1 && !do_hist && mom_part == nullptr) return;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    for (int i = tid; i < SC_WAVES * 2 * RS_RADIX; i += SC_THREADS) (&h[0][0][0])[i] = 0;
    if (nb > 1) bucket_of.load(split + (int64_t)T.seg * SS_B, nb);
    if (do_hist)
        for (int i = tid; i < ha.cells; i += SC_THREADS) cell_h[i] = 0;
    __syncthreads();
    const int64_t t0 = (int64_t)T.blk * TILE + wave * WAVE_KEYS;
    V in[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int64_t idx = t0 + i * 64 + lane;
        in[i] = idx < T.n ? ((const V *)src)[T.base + idx] : (V)0;
    }
    if (nb > 1) {
        // every key's bucket first (loads of LDS only, so the searches of the
        // tile's keys overlap), then the counting; one byte per key for the
        // scatter, at the head of the tile's own stretch of the slots
        uint32_t bk[ITEMS];
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) bk[i] = bucket_of(key_of(in[i]));
        uint8_t *bb = bucket ? (uint8_t *)(bucket + T.base + (int64_t)T.blk * TILE) : nullptr;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const int64_t idx = t0 + i * 64 + lane;
            if (idx < T.n) {
                if (bb) bb[wave * WAVE_KEYS + i * 64 + lane] = (uint8_t)bk[i];
                atomicAdd(&h[wave][lane & 1][bk[i]], 1u);
            }
        }
    }
    if (do_hist || mom_part != nullptr) {
        double s1 = 0, s2 = 0, s3 = 0, s4 = 0;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const int64_t idx = t0 + i * 64 + lane;
            if (idx < T.n) {
                const double xv = (double)in[i];
                const double x2 = xv * xv;
                s1 += xv;
                s2 += x2;
                s3 += x2 * xv;
                s4 += x2 * x2;
                if (do_hist) {
                    double c = floor((xv - ha.lo) * ha.inv_h);
                    c = fmin(fmax(c, 0.0), (double)(ha.cells - 1));
                    atomicAdd(&cell_h[(int)c], 1u);
                }
            }
        }
        for (int off = 32; off >= 1; off >>= 1) {  // fixed butterfly
            s1 += __shfl_xor(s1, off);
            s2 += __shfl_xor(s2, off);
            s3 += __shfl_xor(s3, off);
            s4 += __shfl_xor(s4, off);
        }
        if (lane == 0) {
            wsum[wave][0] = s1;
            wsum[wave][1] = s2;
            wsum[wave][2] = s3;
            wsum[wave][3] = s4;
        }
    }
    __syncthreads();
    if (tid < nb && nb > 1) {
        const int d = tid;
        uint32_t c = 0;
#pragma unroll
        for (int w = 0; w < SC_WAVES; ++w) c += h[w][0][d] + h[w][1][d];
        counts[T.tile0 * RS_RADIX + (int64_t)d * T.nblk + T.blk] = c;
    }
    if (mom_part != nullptr && tid < 4) {
        double t = 0;
        for (int w = 0; w < SC_WAVES; ++w) t += wsum[w][tid];
        mom_part[(T.tile0 + T.blk) * 4 + tid] = t;
    }
    if (do_hist)
        for (int i = tid; i < ha.cells; i += SC_THREADS)
            if (cell_h[i]) atomicAdd(&ha.hist[(int64_t)T.seg * ha.cells + i], cell_h[i]);
}

// Exclusive prefix of every bucket's tile counts and the bucket totals: one
// wave per (ensemble, bucket), or one thread of a block per ensemble where
// the ensembles are many and short (the segment-table layout).
__global__ void __launch_bounds__(256) ss_rowscan(uint32_t *__restrict__ counts, uint32_t *__restrict__ totals,
                                                  SortLayout L) {
    if (L.guard && *L.guard == 0) return;
    const int d = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (d >= ss_buckets<false>(L.n)) return;
    uint32_t *c = counts + (int64_t)blockIdx.y * L.nblk * RS_RADIX + (int64_t)d * L.nblk;
    uint32_t carry = 0;
    for (int c0 = 0; c0 < L.nblk; c0 += 64) {
        const int i = c0 + lane;
        const uint32_t v = i < L.nblk ? c[i] : 0u;
        uint32_t inc = v;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t t = __shfl_up(inc, off);
            if (lane >= off) inc += t;
        }
        if (i < L.nblk) c[i] = carry + inc - v;
        carry += __shfl(inc, 63);
    }
    if (lane == 0) totals[(int64_t)blockIdx.y * RS_RADIX + d] = carry;
}

__global__ void __launch_bounds__(SS_B) ss_rowscan_seg(uint32_t *__restrict__ counts, uint32_t *__restrict__ totals,
                                                       SortLayout L) {
    if (L.guard && *L.guard == 0) return;
    const SortSeg g = L.segs[blockIdx.x];
    const int d = threadIdx.x, nb = ss_buckets<true>(g.n);
    if (nb == 1 || d >= nb) return;
    uint32_t *c = counts + g.tile0 * RS_RADIX + (int64_t)d * g.nblk;
    uint32_t carry = 0;
    for (int b = 0; b < g.nblk; ++b) {
        const uint32_t v = c[b];
        c[b] = carry;
        carry += v;
    }
    totals[(int64_t)blockIdx.x * RS_RADIX + d] = carry;
}

// Exclusive prefix of one value per thread over a block of NT threads.
template <int NT>
__device__ __forceinline__ uint32_t block_exclusive(uint32_t v, uint32_t *wtot) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t inc = v;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t t = __shfl_up(inc, off);
        if (lane >= off) inc += t;
    }
    if (lane == 63) wtot[wave] = inc;
    __syncthreads();
    uint32_t pre = 0;
    for (int w = 0; w < wave; ++w) pre += wtot[w];
    __syncthreads();
    return pre + inc - v;
}

// Lanes of the wave whose 8-bit digit equals this lane's, among the valid ones:
// peers & ~(ballot(bit) ^ bit) over the bits, one three-input operation per half.
__device__ __forceinline__ uint64_t digit_peers(uint32_t d, bool valid) {
    const uint64_t all = __ballot(valid);
    uint32_t lo = (uint32_t)all, hi = (uint32_t)(all >> 32);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const uint32_t bit = 0u - ((d >> b) & 1u);
        const uint64_t bal = __ballot(bit != 0u);
        lo = (uint32_t)__builtin_amdgcn_bitop3_b32((int)lo, (int)(uint32_t)bal, (int)bit, 0x90);
        hi = (uint32_t)__builtin_amdgcn_bitop3_b32((int)hi, (int)(uint32_t)(bal >> 32), (int)bit, 0x90);
    }
    return ((uint64_t)hi << 32) | lo;
}

// Stable scatter of the keys into the buckets.  Every wave ranks its keys in
// order with ballot-built peer masks, the tile is staged in LDS in bucket
// order and every bucket's run leaves as a contiguous burst.  slots receives
// the bucket and the staged place of every particle (in the array the stored
// buckets were read from), pv (only for the permutation) the particle of
// every slot.
template <typename K, bool VAR>
__global__ void __launch_bounds__(SC_THREADS)
ss_scatter(const void *__restrict__ src, const uint32_t *bucket, const K *__restrict__ split,
           K *__restrict__ keys_out, K *__restrict__ sorted, double *__restrict__ xs, uint32_t *slots,
           uint32_t *__restrict__ pv, const uint32_t *__restrict__ counts, const uint32_t *__restrict__ totals,
           SortLayout L, uint32_t *__restrict__ bstart) {
    using V = typename KeyTraits<K>::V;
    constexpr int TILE = RS_THREADS * RS_ITEMS, ITEMS = TILE / SC_THREADS, WAVE_KEYS = 64 * ITEMS;
    __shared__ uint32_t wcnt[SC_WAVES][RS_RADIX];  // keys of a wave's bucket, then its first place in the tile
    __shared__ uint32_t gdelta[RS_RADIX];
    __shared__ bool same[RS_RADIX];
    __shared__ uint32_t wtot[SC_WAVES];
    __shared__ alignas(16) K stage[TILE];
    __shared__ uint8_t sdig[TILE];
    static_assert(sizeof(BucketSearch<K>) <= sizeof(stage), "the search fits the staging area");
    BucketSearch<K> *bucket_of = reinterpret_cast<BucketSearch<K> *>(stage);
    if (L.guard && *L.guard == 0) return;
    const TileRef T = tile_ref<VAR>(L, xcd_tile(blockIdx.x, gridDim.x));
    const int nb = ss_buckets<VAR>(T.n);
    if (nb == 1) return;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int64_t t0 = (int64_t)T.blk * TILE + wave * WAVE_KEYS;
    const uint64_t lt = (1ull << lane) - 1ull;
    for (int i = lane; i < RS_RADIX; i += 64) wcnt[wave][i] = 0;
    const bool any_same = split[(int64_t)T.seg * SS_B] != 0;
    const bool stored = bucket != nullptr;
    if (!stored) {  // no stored buckets: searched again, from the staging area
        bucket_of->load(split + (int64_t)T.seg * SS_B, nb);
        __syncthreads();
    }
    V in[ITEMS];
    uint32_t dig[ITEMS];
    const uint8_t *bb = stored ? (const uint8_t *)(bucket + T.base + (int64_t)T.blk * TILE) : nullptr;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int64_t idx = t0 + i * 64 + lane;
        in[i] = idx < T.n ? ((const V *)src)[T.base + idx] : (V)0;
        dig[i] = (stored && idx < T.n) ? (uint32_t)bb[wave * WAVE_KEYS + i * 64 + lane] : 0u;
    }
    if (!stored) {
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) dig[i] = (*bucket_of)(key_of(in[i]));
    }
    wave_sync();
    uint32_t rnk[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const bool valid = t0 + i * 64 + lane < T.n;
        const uint64_t peers = digit_peers(dig[i], valid);
        uint32_t before = 0;
        if (valid) before = wcnt[wave][dig[i]];
        rnk[i] = before + (uint32_t)__popcll(peers & lt);
        wave_sync();
        if (valid && lane == 63 - __clzll(peers)) wcnt[wave][dig[i]] = before + (uint32_t)__popcll(peers);
        wave_sync();
    }
    __syncthreads();
    {
        // one thread per bucket; the other half adds zeros to the scans
        const int d = tid & (RS_RADIX - 1);
        const bool own = tid < nb;
        uint32_t tot = 0;
        if (own)
#pragma unroll
            for (int w = 0; w < SC_WAVES; ++w) tot += wcnt[w][d];
        const uint32_t ls = block_exclusive<SC_THREADS>(own ? tot : 0u, wtot);
        const uint32_t dbase = block_exclusive<SC_THREADS>(own ? totals[(int64_t)T.seg * RS_RADIX + d] : 0u, wtot);
        if (own) {
            uint32_t acc = ls;
#pragma unroll
            for (int w = 0; w < SC_WAVES; ++w) {
                const uint32_t c = wcnt[w][d];
                wcnt[w][d] = acc;
                acc += c;
            }
            gdelta[d] = dbase + counts[T.tile0 * RS_RADIX + (int64_t)d * T.nblk + T.blk] - ls;
            if (any_same) same[d] = one_value(split + (int64_t)T.seg * SS_B, d, nb);
            if (T.blk == 0) bstart[(int64_t)T.seg * RS_RADIX + d] = dbase;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int64_t idx = t0 + i * 64 + lane;
        if (idx < T.n) {
            rnk[i] += wcnt[wave][dig[i]];
            stage[rnk[i]] = key_of(in[i]);
            sdig[rnk[i]] = (uint8_t)dig[i];
            if (slots) slots[T.base + idx] = (dig[i] << RK_SHIFT) | rnk[i];
        }
    }
    __syncthreads();
    const int64_t rem = T.n - (int64_t)T.blk * TILE;
    const int tile_n = rem < TILE ? (int)rem : TILE;
    uint32_t gpos[ITEMS];
    auto leave = [&](auto mixed) {  // mixed: some bucket's keys go where the sorted ones do
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) {
            const int j = tid + r * SC_THREADS;
            gpos[r] = 0xFFFFFFFFu;
            if (j < tile_n) {
                const uint32_t d = sdig[j], g = (uint32_t)j + gdelta[d];
                if ((int64_t)g < T.n) {  // always true for a consistent scan
                    gpos[r] = g;
                    K *to = keys_out;
                    if constexpr (mixed) {
                        if (same[d]) {
                            to = sorted;
                            if (xs) xs[T.base + g] = value_of(stage[j]);
                        }
                    }
                    to[T.base + g] = stage[j];
                }
            }
        }
    };
    if (any_same) leave(std::true_type{});
    else leave(std::false_type{});
    if (!pv) return;
    __syncthreads();
    uint32_t *sv = (uint32_t *)stage;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
        if (t0 + i * 64 + lane < T.n) sv[rnk[i]] = (uint32_t)(t0 + i * 64 + lane);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int j = tid + r * SC_THREADS;
        if (j < tile_n && gpos[r] != 0xFFFFFFFFu) pv[T.base + gpos[r]] = sv[j];
    }
}

// Midpoint knot at level j / nq of n keys in order.
template <typename K>
__device__ __forceinline__ double knot_of(const K *s, int64_t n, int j, int nq) {
#pragma clang fp contract(off)
    const double t = (double)((int64_t)j * n) / (double)nq - 0.5;
    if (t <= 0.0) return value_of(s[0]);
    if (t >= (double)(n - 1)) return value_of(s[n - 1]);
    const int64_t r = (int64_t)floor(t);
    const double f = t - (double)r;
    const double a = value_of(s[r]), b = value_of(s[r + 1]);
    const double v = a + f * (b - a);
    return v < b ? v : b;
}

enum BucketLeft : uint32_t { BL_NONE = 0, BL_BIG = 1, BL_CROWDED = 2, BL_LONG = 3 };

// Moments of an ensemble from its tiles' sums, by the block's first wave.
__device__ __forceinline__ void moments_of(const double *part, int64_t tile0, int nblk, int64_t n, double *mom) {
    const int lane = threadIdx.x;
    if (lane >= 64) return;
    for (int m = 0; m < 4; ++m) {
        double s = 0;
        for (int b = lane; b < nblk; b += 64) s += part[(tile0 + b) * 4 + m];
        for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
        if (lane == 0) mom[m] = s / (double)n;
    }
}

// Where a bucket's keys come from and what becomes of them.
template <typename K>
struct BucketArgs {
    const void *x;           // values: the input of an ensemble that is one bucket
    K *skeys;                // scattered keys: the input otherwise
    const uint32_t *totals, *bstart;
    const K *split;
    K *keys_out;             // sorted keys
    uint32_t *frank;         // rank of every slot, or NULL
    uint32_t *rank;          // rank of every particle (written here for one-bucket ensembles), or NULL
    uint32_t *perm;          // in: particle of every slot; out: in order; or NULL
    uint32_t *tmp;           // 4 bytes per key free for a bucket's use until ss_finish, or NULL without payload
    double *xs;              // sorted values, or NULL
    double *q;               // knots (written here for one-bucket ensembles)
    uint32_t *left;          // one word per tile: what is left to do (BucketLeft)
    int nq;
};

struct BucketRef {
    int64_t sbase, sn;       // the ensemble
    uint32_t start, size;    // the bucket in it
    int seg, b, nb, qrow;
};

template <typename K, bool VAR>
__device__ __forceinline__ BucketRef bucket_ref(const SortLayout &L, const BucketArgs<K> &A, int64_t tile) {
    const TileRef T = tile_ref<VAR>(L, tile);
    BucketRef R;
    R.seg = T.seg;
    R.b = T.blk;
    R.sbase = T.base;
    R.sn = T.n;
    R.nb = ss_buckets<VAR>(T.n);
    if constexpr (VAR) R.qrow = L.segs[T.seg].qrow;
    else R.qrow = T.seg;
    R.start = 0;
    R.size = 0;
    if (R.b < R.nb) {
        R.size = R.nb == 1 ? (uint32_t)R.sn : A.totals[(int64_t)R.seg * SS_B + R.b];
        R.start = R.nb == 1 ? 0u : A.bstart[(int64_t)R.seg * SS_B + R.b];
    }
    return R;
}

// Reduction of one value per thread over a block of SS_BT.
template <typename V, typename Op>
__device__ __forceinline__ V ss_block_reduce(V v, V *red, Op op) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int off = 32; off >= 1; off >>= 1) v = op(v, (V)__shfl_xor(v, off));
    if (lane == 0) red[wave] = v;
    __syncthreads();
    V r = red[0];
    for (int w = 1; w < SS_BT / 64; ++w) r = op(r, red[w]);
    __syncthreads();
    return r;
}

// One bucket by one block, IT keys per thread; says in left[tile] what is
// left of it.
template <typename K, int IT>
struct BucketLds {
    K sk[SS_BT * IT];
    K redk[SS_BT / 64];
    // value sub-buckets: a power of two, about as many as half the keys the
    // block takes; two 16-bit counts per word, turned into starts in place
    static constexpr int SUB = IT <= 7 ? 4096 : 8192;
    union {
        uint32_t count[SUB / 2];
        uint16_t start[SUB + 2];
    };
    uint32_t red32[SS_BT / 64];
    int too_big;
    uint16_t spos[SS_BT * IT];     // slot of the key in the bucket's input
    // by digits: a word of every key in slot order, the slots in the order so far
    // and the next, a place per slot; 64-bit keys' own array has room for more
    // than the words
    uint16_t more[sizeof(K) == 4 ? 2 * SS_BT * IT : 2];
    __device__ __forceinline__ uint32_t *words() { return reinterpret_cast<uint32_t *>(sk); }
    __device__ __forceinline__ uint16_t *slots(int b) {
        if constexpr (sizeof(K) == 4) return b ? more : spos;
        else return reinterpret_cast<uint16_t *>(words() + SS_BT * IT) + b * (SS_BT * IT);
    }
    __device__ __forceinline__ uint16_t *places() {
        if constexpr (sizeof(K) == 4) return more + SS_BT * IT;
        else return spos;
    }
};
// two bucket blocks per CU, and the largest alone (with ss_left's list) in one
constexpr size_t CU_LDS = 160 << 10;
static_assert(2 * sizeof(BucketLds<uint64_t, SS_IT>) <= CU_LDS && 2 * sizeof(BucketLds<uint32_t, SS_IT>) <= CU_LDS,
              "two blocks of SS_CAP keys share a CU");
static_assert(sizeof(BucketLds<uint64_t, SS_IT_BIG>) + 2 * SS_BT + 64 <= CU_LDS &&
                  sizeof(BucketLds<uint32_t, SS_IT_BIG>) + 2 * SS_BT + 64 <= CU_LDS,
              "a block of SS_BIG keys and its list of tiles fit a CU");

// The slots in S.slots(cur) into the order of their words, by the bytes in
// which the words differ at all (diff), least significant first: every wave ranks
// its consecutive slots in order with ballot-built peer masks, so every pass is
// stable.  Returns the buffer that holds the result.  Bound by the ranking's
// vector operations, about 60 per key and pass, and the LDS reads before them;
// held in loops, not unrolled, which leaves the kernels around it their registers.
// Called by the whole block, behind a barrier; ends with one.
template <typename Lds>
__device__ __forceinline__ int slots_by_digits(Lds &S, int tid, int cur, uint32_t size, uint32_t diff) {
    constexpr int NW = SS_BT / 64;
    static_assert(NW * RS_RADIX <= Lds::SUB, "the counts take the sub-buckets' place");
    uint16_t(*wcnt)[RS_RADIX] = reinterpret_cast<uint16_t(*)[RS_RADIX]>(S.count);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const uint64_t lt = (1ull << lane) - 1ull;
    const uint32_t per = (size + SS_BT - 1) / SS_BT, p0 = wave * per * 64 + lane, p1 = min(size, (wave + 1) * per * 64);
    const uint32_t *word = S.words();
    uint16_t *place = S.places();
#pragma unroll 1
    for (int shift = 0; shift < 32; shift += 8) {
        if (((diff >> shift) & 0xFFu) == 0) continue;
        const uint16_t *in = S.slots(cur);
        uint16_t *out = S.slots(cur ^ 1);
        cur ^= 1;
        for (int i = lane; i < RS_RADIX / 2; i += 64) reinterpret_cast<uint32_t *>(wcnt[wave])[i] = 0;
        wave_sync();
        uint32_t next = p0 < p1 ? word[in[p0]] : 0u;  // read ahead of the ranking
#pragma unroll 1
        for (uint32_t i = 0, p = p0; i < per; ++i, p += 64) {
            const bool valid = p < p1;
            const uint32_t d = (next >> shift) & 0xFFu;
            next = word[in[min(p + 64, size - 1)]];
            const uint64_t peers = digit_peers(d, valid);
            const uint32_t before = wcnt[wave][d];
            if (valid) place[p] = (uint16_t)(before + (uint32_t)__popcll(peers & lt));
            wave_sync();
            if (valid && lane == 63 - __clzll(peers)) wcnt[wave][d] = (uint16_t)(before + (uint32_t)__popcll(peers));
            wave_sync();
        }
        __syncthreads();
        uint32_t tot = 0;
        if (tid < RS_RADIX)
            for (int v = 0; v < NW; ++v) tot += wcnt[v][tid];
        uint32_t at = block_exclusive<SS_BT>(tot, S.red32);
        if (tid < RS_RADIX)
            for (int v = 0; v < NW; ++v) {
                const uint32_t c = wcnt[v][tid];
                wcnt[v][tid] = (uint16_t)at;
                at += c;
            }
        __syncthreads();
#pragma unroll 4
        for (uint32_t p = p0; p < p1; p += 64) {
            const uint16_t slot = in[p];
            out[wcnt[wave][(word[slot] >> shift) & 0xFFu] + place[p]] = slot;
        }
        __syncthreads();
    }
    return cur;
}

// The slots of a bucket in key order, whatever the values (ties, far outliers,
// values of many magnitudes or not finite).  64-bit keys are sorted by 32 bits
// from the highest in which any two differ on; what is left are short runs of
// equal words, put in order by one thread each.  Only where a longer run is out of
// order do the passes over both halves run.  diff: the bits in which keys differ;
// key(slot) reads one.  Returns the buffer that holds the slots.
template <typename K, int IT, typename Key>
__device__ __forceinline__ int bucket_digits(BucketLds<K, IT> &S, int tid, uint32_t size, K diff, Key key) {
    constexpr uint32_t RUN = 32;
    uint32_t *word = S.words();
    const int top = sizeof(K) == 8 && (uint64_t)diff >> 32 ? 32 - __builtin_clzll((unsigned long long)diff) : 0;
    int cur = 0;
#pragma unroll 1
    for (int round = 0; round < 3; ++round) {
        const int shift = round == 0 ? top : (round == 1 ? 0 : 32);
        for (uint32_t i = tid; i < size; i += SS_BT) {
            word[i] = (uint32_t)((uint64_t)key(i) >> shift);
            if (round < 2) S.slots(cur)[i] = (uint16_t)i;
        }
        __syncthreads();
        cur = slots_by_digits(S, tid, cur, size, (uint32_t)((uint64_t)diff >> shift));
        if (round == 1) continue;
        if (round == 2 || (diff & (((K)1 << top) - 1)) == 0) break;  // the words tell the keys apart
        uint16_t *slot = S.slots(cur);
        for (uint32_t p = tid; p + 1 < size; p += SS_BT) {
            const uint32_t v = word[slot[p]];
            if (word[slot[p + 1]] != v || (p > 0 && word[slot[p - 1]] == v)) continue;
            uint32_t e = p + 2;  // the run [p, e)
            while (e < size && e - p <= RUN && word[slot[e]] == v) ++e;
            if (e - p > RUN) continue;
            for (uint32_t i = p + 1; i < e; ++i) {
                const uint16_t s = slot[i];
                const K k = key(s);
                uint32_t j = i;
                for (; j > p && key(slot[j - 1]) > k; --j) slot[j] = slot[j - 1];
                slot[j] = s;
            }
        }
        __syncthreads();
        for (uint32_t p = tid; p + 1 < size; p += SS_BT)
            if (word[slot[p]] == word[slot[p + 1]] && key(slot[p]) > key(slot[p + 1])) S.too_big = 2;
        __syncthreads();
        if (S.too_big != 2) break;
    }
    return cur;
}

// The bucket by digits, with its outputs.
template <typename K, int IT>
__device__ __forceinline__ void bucket_by_digits_in_lds(const BucketArgs<K> &A, const BucketRef &R,
                                                        BucketLds<K, IT> &S) {
    using V = typename KeyTraits<K>::V;
    int tid = threadIdx.x;
    int64_t base = uniform_i64(R.sbase + R.start);
    uint32_t size = (uint32_t)__builtin_amdgcn_readfirstlane((int)R.size);
    // no address or bound is kept from the code before, whose registers it would take
    asm volatile("" : "+v"(tid), "+s"(base), "+s"(size));
    auto key = [&](uint32_t i) { return R.nb == 1 ? key_of(((const V *)A.x)[base + i]) : A.skeys[base + i]; };
    K diff = 0;  // the bits in which any two keys differ
    const K k0 = key(0);
    for (uint32_t i0 = tid; i0 < size; i0 += 4 * SS_BT) {
        K k[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) k[u] = key(i0 + u * SS_BT < size ? i0 + u * SS_BT : i0);
#pragma unroll
        for (int u = 0; u < 4; ++u) diff |= k[u] ^ k0;
    }
    diff = (K)uniform_i64((int64_t)ss_block_reduce<K>(diff, S.redk, [](K a, K c) { return (K)(a | c); }));
    const uint16_t *slot = S.slots(bucket_digits<K, IT>(S, tid, size, diff, key));
#pragma unroll 4
    for (uint32_t i = tid; i < size; i += SS_BT) {
        const K ok = key(slot[i]);
        A.keys_out[base + i] = ok;
        if (A.xs) A.xs[base + i] = value_of(ok);
    }
    uint16_t *place = S.places();
    if (A.rank) {
        uint32_t *rank = R.nb == 1 ? A.rank : A.frank;
        for (uint32_t i = tid; i < size; i += SS_BT) place[slot[i]] = (uint16_t)i;
        __syncthreads();
        for (uint32_t i = tid; i < size; i += SS_BT) rank[base + i] = R.start + place[i];
    }
    __syncthreads();  // the sorted keys are written, the words are free
    if (R.nb == 1)
        for (int j = tid; j <= A.nq; j += SS_BT)
            A.q[(int64_t)R.qrow * (A.nq + 1) + j] = knot_of<K>(A.keys_out + base, R.sn, j, A.nq);
    if (!A.perm) return;
    uint32_t *sv = S.words();
    for (uint32_t i = tid; i < size; i += SS_BT) sv[i] = R.nb == 1 ? (uint32_t)slot[i] : A.perm[base + slot[i]];
    __syncthreads();
    for (uint32_t i = tid; i < size; i += SS_BT) A.perm[base + i] = sv[i];
}

// HERE: also where a sub-bucket is crowded (else left).  ALIKE: without ranks and
// permutation equal keys are alike, and a crowded sub-bucket of one value is in
// order as its keys were counted (twentieths of a normal, knots of 16 ensembles of
// 200,000: FP32 205 -> 147 us, FP64 257 -> 171 us); only crowded ones of several
// values need the digits.  In a kernel of its own: with ranks the code for it costs
// every bucket registers (33 FP32 ensembles of 99,991: 30 -> 33 us).
template <typename K, bool VAR, int IT, bool HERE, bool ALIKE>
__device__ __forceinline__ void bucket_by_block(const BucketArgs<K> &A, const SortLayout &L, int64_t tile,
                                                BucketLds<K, IT> &S) {
    using V = typename KeyTraits<K>::V;
    constexpr int CAP = SS_BT * IT, SUB = BucketLds<K, IT>::SUB, PER = SUB / 2 / SS_BT;
    constexpr uint32_t NONE = ~0u;
    const BucketRef R = bucket_ref<K, VAR>(L, A, tile);
    const int tid = threadIdx.x;
    const uint32_t size = R.size;
    if (size == 0 || size > (uint32_t)CAP) {
        const bool done = size == 0 || one_value(A.split + (int64_t)R.seg * SS_B, R.b, R.nb);
        if (tid == 0) A.left[tile] = done ? BL_NONE : (size <= (uint32_t)SS_BIG ? BL_BIG : BL_LONG);
        return;
    }
    // the splitters on either side, on their way with the keys
    const bool inside = R.b > 0 && R.b < R.nb - 1;
    K kmin = inside ? A.split[(int64_t)R.seg * SS_B + R.b] : ~(K)0;
    K kmax = inside ? A.split[(int64_t)R.seg * SS_B + R.b + 1] : (K)0;
    if (HERE && tid == 0) A.left[tile] = BL_NONE;
    const int64_t base = R.sbase + R.start;
    for (int i = tid; i < SUB / 2; i += SS_BT) S.count[i] = 0;
    if (tid == 0) S.too_big = 0;
    K k[IT];
#pragma unroll
    for (int i = 0; i < IT; ++i) {
        const uint32_t idx = (uint32_t)tid + (uint32_t)i * SS_BT;
        if (R.nb == 1) {
            const V v = idx < size ? ((const V *)A.x)[base + idx] : (V)0;
            k[i] = key_of(v);
        } else {
            k[i] = idx < size ? A.skeys[base + idx] : ~(K)0;
        }
    }
    // bounds of the bucket's values: its splitters inside, its extremes at
    // the two ends of the ensemble
    if (inside && kmin == kmax) {  // one value: the scatter has written it
        if (!HERE && tid == 0) A.left[tile] = BL_NONE;
        return;
    }
    if (!inside) {
#pragma unroll
        for (int i = 0; i < IT; ++i)
            if ((uint32_t)tid + (uint32_t)i * SS_BT < size) {
                kmin = k[i] < kmin ? k[i] : kmin;
                kmax = k[i] > kmax ? k[i] : kmax;
            }
        kmin = ss_block_reduce<K>(kmin, S.redk, [](K a, K c) { return a < c ? a : c; });
        kmax = ss_block_reduce<K>(kmax, S.redk, [](K a, K c) { return a > c ? a : c; });
    }
    // value sub-buckets: floor((x - lo) SUB / (hi - lo)) is non-decreasing
    // in x (every rounded operation is), so they keep the order; equal values
    // share one.  Bounds that are not finite put every key in one.
    const double lo = value_of(kmin), hi = value_of(kmax);
    const double span = hi - lo;
    const double scale = (span > 0.0 && span <= 1.79e308) ? (double)SUB / span : 0.0;
    __syncthreads();
    // per key: its sub-bucket (low half) and its number among the keys counted
    // there, then its place in sub-bucket order, then its final place
    uint32_t w[IT];
#pragma unroll
    for (int i = 0; i < IT; ++i) {
        w[i] = NONE;
        if ((uint32_t)tid + (uint32_t)i * SS_BT < size) {
            const double t = (value_of(k[i]) - lo) * scale;
            w[i] = (uint32_t)(t >= (double)SUB ? SUB - 1 : (t > 0.0 ? (int)t : 0));
        }
    }
#pragma unroll
    for (int i = 0; i < IT; ++i)
        if (w[i] != NONE) {
            const uint32_t sh = 16 * (w[i] & 1);
            w[i] |= ((atomicAdd(&S.count[w[i] >> 1], 1u << sh) >> sh) & 0xFFFFu) << 16;
        }
    __syncthreads();
    // exclusive scan of the sub-bucket counts (2 PER per thread), their maximum
    {
        uint32_t c[2 * PER], sum = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const uint32_t two = S.count[tid * PER + i];
            c[2 * i] = two & 0xFFFFu;
            c[2 * i + 1] = two >> 16;
            sum += c[2 * i] + c[2 * i + 1];
            if (max(c[2 * i], c[2 * i + 1]) > ss_crowded<K, HERE>(size)) S.too_big = 1;
        }
        const int lane = tid & 63, wave = tid >> 6;
        uint32_t inc = sum;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t t = __shfl_up(inc, off);
            if (lane >= off) inc += t;
        }
        if (lane == 63) S.red32[wave] = inc;
        __syncthreads();
        uint32_t e = inc - sum;
        for (int v = 0; v < wave; ++v) e += S.red32[v];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            S.count[tid * PER + i] = e | ((e + c[2 * i]) << 16);
            e += c[2 * i] + c[2 * i + 1];
        }
        if (tid == SS_BT - 1) S.start[SUB] = (uint16_t)size;
        __syncthreads();
    }
    const bool crowded = S.too_big != 0;
    if constexpr (!ALIKE) {
        if (!HERE && tid == 0) A.left[tile] = crowded ? BL_CROWDED : BL_NONE;
        if (__builtin_expect(crowded, 0)) {  // and no register of the code below is spilled for it
            if constexpr (HERE) bucket_by_digits_in_lds<K, IT>(A, R, S);
            return;
        }
    }
#pragma unroll
    for (int i = 0; i < IT; ++i)
        if (w[i] != NONE) {
            const uint32_t at = S.start[w[i] & 0xFFFFu] + (w[i] >> 16);
            S.sk[at] = k[i];
            S.spos[at] = (uint16_t)((uint32_t)tid + (uint32_t)i * SS_BT);
            w[i] = (w[i] & 0xFFFFu) | (at << 16);
        }
    uint32_t alike = 0;  // a bit per key: its sub-bucket holds one value
    if constexpr (ALIKE) {
        if (__builtin_expect(crowded, 0)) {
            // the top bit of its first key's slot: another value is in the sub-bucket
            constexpr uint16_t MIXED = 0x8000;
            static_assert(CAP <= MIXED, "slots leave their top bit");
            __syncthreads();
#pragma unroll
            for (int i = 0; i < IT; ++i)
                if (w[i] != NONE) {
                    const uint32_t a = S.start[w[i] & 0xFFFFu];
                    if (S.sk[a] != k[i]) S.spos[a] = S.spos[a] | MIXED;  // any number of threads, the same word
                }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < IT; ++i)
                if (w[i] != NONE) {
                    const uint32_t a = S.start[w[i] & 0xFFFFu], e = S.start[(w[i] & 0xFFFFu) + 1];
                    if (!(S.spos[a] & MIXED)) alike |= 1u << i;
                    else if (e - a > ss_crowded<uint32_t, HERE>(SS_CAP)) S.too_big = 4;
                }
            __syncthreads();
            if (S.too_big == 4) {
                if (!HERE && tid == 0) A.left[tile] = BL_CROWDED;
                if constexpr (HERE) bucket_by_digits_in_lds<K, IT>(A, R, S);
                return;
            }
#pragma unroll
            for (int i = 0; i < IT; ++i)
                if (w[i] != NONE) S.spos[w[i] >> 16] = S.spos[w[i] >> 16] & (uint16_t)~MIXED;
        }
        if (!HERE && tid == 0) A.left[tile] = BL_NONE;
    }
    __syncthreads();
    // place: the keys of the sub-bucket before this one by (key, slot)
#pragma unroll
    for (int i = 0; i < IT; ++i) {
        if (w[i] != NONE) {
            const uint32_t idx = (uint32_t)tid + (uint32_t)i * SS_BT;
            const uint32_t a = S.start[w[i] & 0xFFFFu], e = S.start[(w[i] & 0xFFFFu) + 1], me = w[i] >> 16;
            // four entries per step, their LDS loads in flight together; the
            // steps past the end read the key's own place, which never counts.
            // Input slots are read only for equal keys.
            const bool several = e - a > 1 && !(ALIKE && ((alike >> i) & 1u));
            uint32_t r = ALIKE && !several ? me : a;
            for (uint32_t j = several ? a : e; j < e; j += 4) {
                K kj[4];
                uint32_t jj[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    jj[u] = j + u < e ? j + u : me;
                    kj[u] = S.sk[jj[u]];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (kj[u] < k[i]) ++r;
                    else if (kj[u] == k[i] && jj[u] != me && S.spos[jj[u]] < idx) ++r;
                }
            }
            w[i] = r;
        }
    }
    // the ranks in slot order from the registers; the keys pass through LDS
    // to their final places and leave in order
    uint32_t *frank = (R.nb == 1 || !A.rank) ? A.rank : A.frank;
    if (frank) {
#pragma unroll
        for (int i = 0; i < IT; ++i)
            if (w[i] != NONE) frank[base + tid + i * SS_BT] = R.start + w[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < IT; ++i)
        if (w[i] != NONE) S.sk[w[i]] = k[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < IT; ++i) {
        const uint32_t idx = (uint32_t)tid + (uint32_t)i * SS_BT;
        if (idx < size) {
            const K ok = S.sk[idx];
            A.keys_out[base + idx] = ok;
            if (A.xs) A.xs[base + idx] = value_of(ok);
        }
    }
    if (R.nb == 1)
        for (int j = tid; j <= A.nq; j += SS_BT)
            A.q[(int64_t)R.qrow * (A.nq + 1) + j] = knot_of<K>(S.sk, R.sn, j, A.nq);
    if (!A.perm) return;
    // the particles, by way of LDS (in the keys' own array)
    uint32_t v[IT];
#pragma unroll
    for (int i = 0; i < IT; ++i) {
        const uint32_t idx = (uint32_t)tid + (uint32_t)i * SS_BT;
        v[i] = idx < size ? (R.nb == 1 ? idx : A.perm[base + idx]) : 0u;
    }
    __syncthreads();
    uint32_t *sv = reinterpret_cast<uint32_t *>(S.sk);
#pragma unroll
    for (int i = 0; i < IT; ++i)
        if (w[i] != NONE) sv[w[i]] = v[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < IT; ++i) {
        const uint32_t idx = (uint32_t)tid + (uint32_t)i * SS_BT;
        if (idx < size) A.perm[base + idx] = sv[idx];
    }
}

// With SS_IT keys per thread two blocks share a CU, which leaves FP64 no registers
// for the digits in the same kernel (64 ensembles of 2^20: 1.26 ms, 1.41 with
// them); up to SS_WHOLE ensembles of one such bucket each one block per CU is
// enough, and nothing is left for another launch (64 of 1000 keys 17.7 us, 23.0 in
// two launches).
constexpr int SS_WHOLE = 256;

template <typename K, bool VAR, int IT, bool HERE, bool ALIKE>
__global__ void __launch_bounds__(SS_BT, IT <= SS_IT && (!HERE || (sizeof(K) == 4 && !ALIKE)) ? 8 : 4)
ss_bucket_sort(BucketArgs<K> A, SortLayout L) {
    if (L.guard && *L.guard == 0) return;
    __shared__ BucketLds<K, IT> S;
    bucket_by_block<K, VAR, IT, HERE, ALIKE>(A, L, xcd_tile(blockIdx.x, gridDim.x), S);
}

// Tile j of this block's share.  Neighbouring ensembles mostly leave the same
// bucket, so the share is skewed.
__device__ __forceinline__ int64_t shared_tile(int64_t j) {
    return j * gridDim.x + (blockIdx.x + 37 * j) % gridDim.x;
}

// The tiles of the block's share whose word is want, among the SS_BT of chunk
// c: their numbers in the chunk in list, their count returned.
__device__ __forceinline__ int tiles_left(const uint32_t *left, int64_t tiles, int64_t c, uint32_t want,
                                          uint16_t *list, int *count) {
    __syncthreads();  // the last list has been read
    if (threadIdx.x == 0) *count = 0;
    __syncthreads();
    const int64_t t = shared_tile(c * SS_BT + threadIdx.x);
    if (t < tiles && left[t] == want) list[atomicAdd(count, 1)] = (uint16_t)threadIdx.x;
    __syncthreads();
    return *count;
}

// A bucket of more than SS_BIG keys, one of several of its ensemble.  One block
// orders it in global memory by the digits in which its keys differ at all,
// least significant first; every pass is stable, so equal keys stay in slot
// order.  The keys alternate between the scattered and the sorted keys'
// stretches (the first pass reads the scattered ones), their slots between tmp
// and frank.
template <typename K>
struct DigitsLds {
    K redk[SS_BT / 64];
    uint32_t wcnt[SS_BT / 64][RS_RADIX];
    uint32_t dbase[RS_RADIX];
    uint32_t wtot[SS_BT / 64];
};

template <typename K, bool VAR>
__device__ __forceinline__ void bucket_by_digits(const BucketArgs<K> &A, const SortLayout &L, int64_t tile,
                                                 DigitsLds<K> &S) {
    constexpr int NW = SS_BT / 64, IT = 4, STEP = SS_BT * IT;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const uint64_t lt = (1ull << lane) - 1ull;
    const BucketRef R = bucket_ref<K, VAR>(L, A, tile);
    const int64_t base = R.sbase + R.start, size = R.size;
    const bool payload = A.tmp != nullptr;
    K *buf[2] = {A.skeys + base, A.keys_out + base};
    uint32_t *pos[2] = {payload ? A.tmp + base : nullptr, payload ? A.frank + base : nullptr};
    // the first buffer holds the keys; the digits in which they differ (eight
    // loads in flight per thread: one block reads the whole bucket)
    K diff = 0;
    const K k0 = buf[0][0];
    for (int64_t i0 = tid; i0 < size; i0 += 8 * SS_BT) {
        K k[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int64_t i = i0 + u * SS_BT < size ? i0 + u * SS_BT : i0;
            k[u] = buf[0][i];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) diff |= k[u] ^ k0;
    }
    diff = ss_block_reduce<K>(diff, S.redk, [](K a, K c) { return (K)(a | c); });
    if (diff == 0) {  // one value: already in order, slot by slot
        for (int64_t i = tid; i < size; i += SS_BT) {
            buf[1][i] = k0;
            if (A.rank) A.frank[base + i] = R.start + (uint32_t)i;
            if (A.xs) A.xs[base + i] = value_of(k0);
        }
        return;
    }
    if (payload)
        for (int64_t i = tid; i < size; i += SS_BT) pos[0][i] = (uint32_t)i;
    __syncthreads();
    int cur = 0;
    for (int shift = 0; shift < (int)sizeof(K) * 8; shift += 8) {
        if (((diff >> shift) & (K)0xFF) == 0) continue;
        const K *in = buf[cur];
        K *out = buf[cur ^ 1];
        const uint32_t *pin = pos[cur];
        uint32_t *pout = pos[cur ^ 1];
        // digit totals, then where each digit's keys go next
        if (tid < RS_RADIX) S.dbase[tid] = 0;
        __syncthreads();
        for (int64_t i = tid; i < size; i += SS_BT) atomicAdd(&S.dbase[(uint32_t)(in[i] >> shift) & 0xFFu], 1u);
        __syncthreads();
        const uint32_t e = block_exclusive<SS_BT>(tid < RS_RADIX ? S.dbase[tid] : 0u, S.wtot);
        if (tid < RS_RADIX) S.dbase[tid] = e;
        for (int64_t t0 = 0; t0 < size; t0 += STEP) {
            for (int i = lane; i < RS_RADIX; i += 64) S.wcnt[wave][i] = 0;
            wave_sync();
            K k[IT];
            uint32_t rnk[IT];
#pragma unroll
            for (int i = 0; i < IT; ++i) {
                const int64_t idx = t0 + wave * (64 * IT) + i * 64 + lane;
                const bool valid = idx < size;
                k[i] = valid ? in[idx] : (K)0;
                const uint32_t d = (uint32_t)(k[i] >> shift) & 0xFFu;
                const uint64_t peers = digit_peers(d, valid);
                const uint32_t before = valid ? S.wcnt[wave][d] : 0u;
                rnk[i] = before + (uint32_t)__popcll(peers & lt);
                wave_sync();
                if (valid && lane == 63 - __clzll(peers)) S.wcnt[wave][d] = before + (uint32_t)__popcll(peers);
                wave_sync();
            }
            __syncthreads();
            if (tid < RS_RADIX) {
                uint32_t acc = S.dbase[tid];
                for (int w = 0; w < NW; ++w) {
                    const uint32_t c = S.wcnt[w][tid];
                    S.wcnt[w][tid] = acc;
                    acc += c;
                }
                S.dbase[tid] = acc;
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < IT; ++i) {
                const int64_t idx = t0 + wave * (64 * IT) + i * 64 + lane;
                if (idx < size) {
                    const uint32_t to = S.wcnt[wave][(uint32_t)(k[i] >> shift) & 0xFFu] + rnk[i];
                    if ((int64_t)to < size) {  // always true: the digit totals sum to size
                        out[to] = k[i];
                        if (payload) pout[to] = pin[idx];
                    }
                }
            }
            __syncthreads();
        }
        cur ^= 1;
    }
    if (cur == 0)
        for (int64_t i = tid; i < size; i += SS_BT) buf[1][i] = buf[0][i];
    if (payload && cur == 1)
        for (int64_t i = tid; i < size; i += SS_BT) pos[0][i] = pos[1][i];
    __syncthreads();
    if (A.xs)
        for (int64_t i = tid; i < size; i += SS_BT) A.xs[base + i] = value_of(buf[1][i]);
    if (payload) {
        // pos[0] holds the slots in key order (in the rank array, where
        // ranks are asked for)
        if (A.perm) {
            for (int64_t i = tid; i < size; i += SS_BT) pos[1][i] = A.perm[base + pos[0][i]];
            __syncthreads();
            for (int64_t i = tid; i < size; i += SS_BT) A.perm[base + i] = pos[1][i];
            __syncthreads();
        }
        if (A.rank)
            for (int64_t i = tid; i < size; i += SS_BT) pos[1][pos[0][i]] = R.start + (uint32_t)i;
    }
}

// What ss_bucket_sort left: the buckets of SS_CAP..SS_BIG keys by one block
// with most of a CU's LDS, then the longer ones.
template <typename K, bool VAR, bool ALIKE>
__global__ void __launch_bounds__(SS_BT) ss_left(BucketArgs<K> A, SortLayout L, int64_t tiles) {
    union Lds {
        BucketLds<K, SS_IT_BIG> bucket;
        DigitsLds<K> digits;
    };
    __shared__ Lds S;
    __shared__ uint16_t list[SS_BT];
    __shared__ int count;
    if (L.guard && *L.guard == 0) return;
    for (int64_t c = 0; c * SS_BT * gridDim.x < tiles; ++c) {
        const int big = tiles_left(A.left, tiles, c, BL_BIG, list, &count);
        for (int i = 0; i < big; ++i) {
            bucket_by_block<K, VAR, SS_IT_BIG, true, ALIKE>(A, L, shared_tile(c * SS_BT + list[i]), S.bucket);
            __syncthreads();
        }
        const int crowded = tiles_left(A.left, tiles, c, BL_CROWDED, list, &count);
        for (int i = 0; i < crowded; ++i) {
            if (threadIdx.x == 0) S.bucket.too_big = 0;  // the last bucket's
            bucket_by_digits_in_lds<K, SS_IT_BIG>(A, bucket_ref<K, VAR>(L, A, shared_tile(c * SS_BT + list[i])), S.bucket);
            __syncthreads();
        }
        const int longer = tiles_left(A.left, tiles, c, BL_LONG, list, &count);
        for (int i = 0; i < longer; ++i) {
            bucket_by_digits<K, VAR>(A, L, shared_tile(c * SS_BT + list[i]), S.digits);
            __syncthreads();
        }
    }
}

// Rank of every particle from the rank of its slot: the block stages the
// bucket of every place of its tile, reads the ranks of those places' slots
// (runs of neighbouring slots, one per bucket) into LDS and writes them in
// particle order.
template <typename K, bool VAR>
__device__ __forceinline__ void ranks_of_tile(const uint32_t *slots, const uint32_t *frank, const uint32_t *counts,
                                              const uint32_t *totals, const uint32_t *bstart, const K *split,
                                              const SortLayout &L, int64_t tile, uint32_t *rank) {
    constexpr int TILE = RS_THREADS * RS_ITEMS, ITEMS = TILE / SC_THREADS;
    __shared__ uint8_t sdig[TILE];
    __shared__ uint32_t sr[TILE];
    __shared__ uint32_t gdelta[SS_B], wtot[SC_WAVES];
    __shared__ bool same[SS_B];
    const TileRef T = tile_ref<VAR>(L, tile);
    const int nb = ss_buckets<VAR>(T.n), tid = threadIdx.x;
    if (nb == 1) return;
    const bool any_same = split[(int64_t)T.seg * SS_B] != 0;
    const int64_t t0 = (int64_t)T.blk * TILE;
    const int tile_n = T.n - t0 < TILE ? (int)(T.n - t0) : TILE;
    uint32_t s[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int p = tid + i * SC_THREADS;
        s[i] = p < tile_n ? slots[T.base + t0 + p] : ~0u;
    }
    uint32_t mine = 0, at = 0;  // the tile's keys of bucket tid, the slot of the first
    if (tid < nb) {
        const uint32_t *c = counts + T.tile0 * RS_RADIX + (int64_t)tid * T.nblk + T.blk;
        const uint32_t end = T.blk + 1 < T.nblk ? c[1] : totals[(int64_t)T.seg * SS_B + tid];
        mine = end - c[0];
        at = bstart[(int64_t)T.seg * SS_B + tid] + c[0];
    }
    const uint32_t ls = block_exclusive<SC_THREADS>(mine, wtot);
    if (tid < nb) {
        gdelta[tid] = at - ls;
        if (any_same) same[tid] = one_value(split + (int64_t)T.seg * SS_B, tid, nb);
    }
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
        if (s[i] != ~0u) sdig[s[i] & (TILE - 1)] = (uint8_t)(s[i] >> RK_SHIFT);
    __syncthreads();
    uint32_t r[ITEMS];
    auto ranks = [&](auto mixed) {  // mixed: some bucket's slots are their own ranks
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const int j = tid + i * SC_THREADS;
            const uint32_t g = j < tile_n ? (uint32_t)j + gdelta[sdig[j]] : ~0u;
            r[i] = g;
            if constexpr (mixed) {
                if ((int64_t)g < T.n && !same[sdig[j]]) r[i] = frank[T.base + g];
            } else {
                r[i] = (int64_t)g < T.n ? frank[T.base + g] : 0u;
            }
        }
    };
    if (any_same) ranks(std::true_type{});
    else ranks(std::false_type{});
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) sr[tid + i * SC_THREADS] = r[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
        if (s[i] != ~0u) rank[T.base + t0 + tid + i * SC_THREADS] = sr[s[i] & (TILE - 1)];
}

// Blocks [0, nseg): the knots (sorted != NULL) and the moments (part != NULL)
// of an ensemble; the others, where ranks are asked for: those of a tile.
template <typename K, bool VAR>
__global__ void __launch_bounds__(SC_THREADS)
ss_finish(const K *__restrict__ sorted, int nq, double *__restrict__ q, const double *__restrict__ part,
          double *__restrict__ mom, const uint32_t *__restrict__ slots, const uint32_t *__restrict__ frank,
          const uint32_t *__restrict__ counts, const uint32_t *__restrict__ totals,
          const uint32_t *__restrict__ bstart, const K *__restrict__ split, SortLayout L,
          uint32_t *__restrict__ rank) {
    if (L.guard && *L.guard == 0) return;
    if ((int64_t)blockIdx.x >= L.nseg) {
        ranks_of_tile<K, VAR>(slots, frank, counts, totals, bstart, split, L,
                              xcd_tile((int64_t)blockIdx.x - L.nseg, (int64_t)gridDim.x - L.nseg), rank);
        return;
    }
    int64_t base, n, tile0;
    int nblk, qrow;
    seg_ref<VAR>(L, blockIdx.x, base, n, tile0, nblk, qrow);
    if (sorted)
        for (int j = threadIdx.x; j <= nq; j += blockDim.x)
            q[(int64_t)qrow * (nq + 1) + j] = knot_of<K>(sorted + base, n, j, nq);
    if (part) moments_of(part, tile0, nblk, n, mom + (int64_t)qrow * 4);
}

// ---------------------------------------------------------------------------
// Fix-up after the passes over the high 32 bits of 64-bit keys.  The keys
// are then ordered by their high halves, and among equal high halves by
// particle (the passes are stable), so a run of equal high halves needs
// only its own order by the full key, ties by position.  Every key finds the
// run around it in the tile's keys (staged in LDS with FIX_MAX + 1 keys on
// either side), counts the keys of the run that precede it in that order,
// and goes to its final place with the rank, perm and sorted-value outputs
// of the last pass.  A run longer than FIX_MAX sets *flag: the complete sort
// then runs (guarded by the flag) and redoes every output.
// ---------------------------------------------------------------------------
constexpr int FIX_MAX = 64;
constexpr int FIX_HALO = FIX_MAX + 1;
constexpr int FIX_NEAR = 4;

template <bool VAR, bool PAYLOAD>
__global__ void __launch_bounds__(RS_THREADS)
rs_fixup(const uint64_t *__restrict__ keys_in, const uint32_t *__restrict__ vals_in, uint64_t *__restrict__ keys_out,
         SortLayout L, uint32_t *__restrict__ rank_out, uint32_t *__restrict__ perm_out, double *__restrict__ xs_out,
         int *__restrict__ flag) {
    constexpr int TILE = RS_THREADS * RS_ITEMS;
    __shared__ uint64_t sk[TILE + 2 * FIX_HALO];
    if (L.guard && *L.guard == 0) return;
    const TileRef T = tile_ref<VAR>(L, xcd_tile(blockIdx.x, gridDim.x));
    const uint64_t *k = keys_in + T.base;
    const int64_t n = T.n, t0 = (int64_t)T.blk * TILE;
    // sk[j] = k[t0 - FIX_HALO + j] where that position exists; all loads
    // first, so that they are in flight together
    constexpr int SK = TILE + 2 * FIX_HALO, SK_PER = (SK + RS_THREADS - 1) / RS_THREADS;
    uint64_t ld[SK_PER];
#pragma unroll
    for (int r = 0; r < SK_PER; ++r) {
        const int j = (int)threadIdx.x + r * RS_THREADS;
        const int64_t q = t0 - FIX_HALO + j;
        ld[r] = (j < SK && q >= 0 && q < n) ? k[q] : 0ull;
    }
#pragma unroll
    for (int r = 0; r < SK_PER; ++r) {
        const int j = (int)threadIdx.x + r * RS_THREADS;
        if (j < SK) sk[j] = ld[r];
    }
    __syncthreads();
    bool too_long = false;
    // final places first, then all stores of the tile's keys at once
    int64_t pos[RS_ITEMS];
    uint64_t key[RS_ITEMS];
#pragma unroll
    for (int i = 0; i < RS_ITEMS; ++i) {
        const int64_t p = t0 + (int64_t)i * RS_THREADS + threadIdx.x;
        pos[i] = -1;
        key[i] = 0;
        if (p < n) {
            const int j = (int)(p - t0) + FIX_HALO;  // p in sk
            const uint64_t kp = sk[j];
            const uint32_t hp = (uint32_t)(kp >> 32);
            // the run [p - back, p + fwd] of equal high halves, up to FIX_MAX keys on
            // either side: the first few key by key, the rest in halving steps (the
            // high halves are in order; all of a long run key by key took more
            // than a quarter of the whole sort)
            const int bmax = (int)min((int64_t)FIX_MAX, p), fmax = (int)min((int64_t)FIX_MAX, n - 1 - p);
            int back = 0, fwd = 0;
            while (back < FIX_NEAR && back < bmax && (uint32_t)(sk[j - back - 1] >> 32) == hp) ++back;
            if (back == FIX_NEAR)
                for (int step = FIX_MAX / 2; step > 0; step >>= 1)
                    if (back + step <= bmax && (uint32_t)(sk[j - back - step] >> 32) == hp) back += step;
            while (fwd < FIX_NEAR && fwd < fmax && (uint32_t)(sk[j + fwd + 1] >> 32) == hp) ++fwd;
            if (fwd == FIX_NEAR)
                for (int step = FIX_MAX / 2; step > 0; step >>= 1)
                    if (fwd + step <= fmax && (uint32_t)(sk[j + fwd + step] >> 32) == hp) fwd += step;
            key[i] = kp;
            if (back + fwd + 1 > FIX_MAX) {
                too_long = true;
            } else if (back + fwd == 0) {
                pos[i] = p;
            } else {
                int r = 0;
                for (int b = -back; b <= fwd; ++b) {
                    const uint64_t kb = sk[j + b];
                    r += (kb < kp || (kb == kp && b < 0)) ? 1 : 0;
                }
                pos[i] = p - back + r;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < RS_ITEMS; ++i) {
        if (pos[i] >= 0) {
            keys_out[T.base + pos[i]] = key[i];
            if (xs_out) xs_out[T.base + pos[i]] = value_of(key[i]);
        }
    }
    if constexpr (PAYLOAD) {
        uint32_t val[RS_ITEMS];
#pragma unroll
        for (int i = 0; i < RS_ITEMS; ++i)
            val[i] = pos[i] >= 0 ? vals_in[T.base + t0 + (int64_t)i * RS_THREADS + threadIdx.x] : 0u;
#pragma unroll
        for (int i = 0; i < RS_ITEMS; ++i) {
            if (pos[i] >= 0) {
                if (rank_out && (int64_t)val[i] < n) rank_out[T.base + val[i]] = (uint32_t)pos[i];
                if (perm_out) perm_out[T.base + pos[i]] = val[i];
            }
        }
    }
    if (too_long) *flag = 1;
}

// ---------------------------------------------------------------------------
// Ranks from the permutation (sorted position -> particle) without stores to
// random addresses: a 4-byte store at a random index leaves its cache line
// partly written, and the line then costs a whole memory sector.  Instead
//   rs_rank_bucket  every tile of the permutation groups its (position,
//                   particle) pairs by the block of TILE particles the
//                   particle belongs to and appends each group, as one
//                   contiguous run, to that block's region of a staging
//                   buffer (the region has one slot per particle of the
//                   block; a cursor per block hands out the slots),
//   rs_rank_place   every block of TILE particles takes its region, places
//                   the ranks in LDS and writes them out in particle order.
// A pair packs the position (below 2^20) and the particle's offset in its
// block (below 2^12) into 32 bits, so segment tables of up to 2^20 keys per
// segment take this path (ensembles of equal lengths come to the radix passes
// only with more).  Both kernels return at once where the fix-up raised its
// flag (the complete sort then writes the ranks).
// ---------------------------------------------------------------------------
constexpr int64_t RK_MAX_N = (int64_t)1 << 20;
static_assert((1 << RK_SHIFT) == RS_THREADS * RS_ITEMS, "a block of particles is one tile");
static_assert(RS_THREADS == RS_RADIX, "one thread per particle block of a segment");

__global__ void __launch_bounds__(RS_THREADS)
rs_rank_bucket(const uint32_t *__restrict__ perm, SortLayout L, uint32_t *__restrict__ cursor,
               uint32_t *__restrict__ staged, const int *__restrict__ flag) {
    constexpr int TILE = RS_THREADS * RS_ITEMS;
    __shared__ uint32_t cnt[RS_RADIX], lofs[RS_RADIX], gofs[RS_RADIX], wtot[RS_WAVES];
    __shared__ uint32_t stage[TILE];
    __shared__ uint8_t sblk[TILE];
    if ((L.guard && *L.guard == 0) || *flag != 0) return;
    const TileRef T = tile_ref<true>(L, xcd_tile(blockIdx.x, gridDim.x));
    const int tid = threadIdx.x;
    cnt[tid] = 0;
    __syncthreads();
    const int64_t t0 = (int64_t)T.blk * TILE;
    uint32_t p[RS_ITEMS];
#pragma unroll
    for (int i = 0; i < RS_ITEMS; ++i) {
        const int64_t pos = t0 + (int64_t)i * RS_THREADS + tid;
        p[i] = pos < T.n ? perm[T.base + pos] : 0xFFFFFFFFu;
    }
    uint32_t slot[RS_ITEMS];
#pragma unroll
    for (int i = 0; i < RS_ITEMS; ++i)
        if ((int64_t)p[i] < T.n) slot[i] = atomicAdd(&cnt[p[i] >> RK_SHIFT], 1u);
    __syncthreads();
    const uint32_t c = cnt[tid];
    lofs[tid] = block_exclusive_256(c, wtot);
    if (c != 0) gofs[tid] = atomicAdd(&cursor[T.tile0 + tid], c);  // c != 0 only for blocks of this segment
    __syncthreads();
#pragma unroll
    for (int i = 0; i < RS_ITEMS; ++i) {
        if ((int64_t)p[i] < T.n) {
            const uint32_t b = p[i] >> RK_SHIFT, j = lofs[b] + slot[i];
            const uint32_t pos = (uint32_t)(t0 + i * RS_THREADS + tid);
            stage[j] = (pos << RK_SHIFT) | (p[i] & (TILE - 1));
            sblk[j] = (uint8_t)b;
        }
    }
    __syncthreads();
    const uint32_t total = lofs[RS_RADIX - 1] + cnt[RS_RADIX - 1];
    for (uint32_t j = tid; j < total; j += RS_THREADS) {
        const uint32_t b = sblk[j];
        const int64_t b0 = (int64_t)b << RK_SHIFT;
        const int64_t bn = T.n - b0 < TILE ? T.n - b0 : TILE;
        const uint32_t s = gofs[b] + (j - lofs[b]);
        if ((int64_t)s < bn) staged[T.base + b0 + s] = stage[j];
    }
}

__global__ void __launch_bounds__(RS_THREADS)
rs_rank_place(const uint32_t *__restrict__ staged, SortLayout L, uint32_t *__restrict__ rank_out,
              const int *__restrict__ flag) {
    constexpr int TILE = RS_THREADS * RS_ITEMS;
    __shared__ uint32_t r[TILE];
    if ((L.guard && *L.guard == 0) || *flag != 0) return;
    const TileRef T = tile_ref<true>(L, xcd_tile(blockIdx.x, gridDim.x));
    const int64_t b0 = (int64_t)T.blk * TILE;
    const int bn = (int)(T.n - b0 < TILE ? T.n - b0 : TILE);
    uint32_t e[RS_ITEMS];
#pragma unroll
    for (int i = 0; i < RS_ITEMS; ++i) {
        const int j = i * RS_THREADS + threadIdx.x;
        e[i] = j < bn ? staged[T.base + b0 + j] : 0xFFFFFFFFu;
    }
#pragma unroll
    for (int i = 0; i < RS_ITEMS; ++i)
        if (i * RS_THREADS + (int)threadIdx.x < bn && (int)(e[i] & (TILE - 1)) < bn) r[e[i] & (TILE - 1)] = e[i] >> RK_SHIFT;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < RS_ITEMS; ++i) {
        const int j = i * RS_THREADS + threadIdx.x;
        if (j < bn) rank_out[T.base + b0 + j] = r[j];
    }
}

// ---------------------------------------------------------------------------
// Knots (midpoint convention) from the sorted keys; moment totals.
// ---------------------------------------------------------------------------
template <typename K, bool VAR>
__global__ void rs_knots(const K *__restrict__ sorted, SortLayout L, int nq, double *__restrict__ q) {
    if (L.guard && *L.guard == 0) return;
    int64_t base, n, tile0;
    int nblk, qrow;
    seg_ref<VAR>(L, blockIdx.x, base, n, tile0, nblk, qrow);
    const K *s = sorted + base;
    for (int j = threadIdx.x; j <= nq; j += blockDim.x) q[(int64_t)qrow * (nq + 1) + j] = knot_of<K>(s, n, j, nq);
}

template <bool VAR>
__global__ void rs_moments(const double *__restrict__ part, SortLayout L, double *__restrict__ mom) {
    if (L.guard && *L.guard == 0) return;
    int64_t base, n, tile0;
    int nblk, qrow;
    seg_ref<VAR>(L, blockIdx.x, base, n, tile0, nblk, qrow);
    moments_of(part, tile0, nblk, n, mom + (int64_t)qrow * 4);
}

__global__ void zero_u32(uint32_t *p, int64_t count) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

// ---------------------------------------------------------------------------
// Knots of matched ensembles from the sort of their priors.
//
// Matching moves every prior value by a smooth function of its rank, so the
// matched values taken in the prior's rank order, z_r = M(xs_r) (xs the
// sorted prior), are nearly sorted.  A position c is a cut where every z
// before it is below every z from it on, in key order (c = 0 and c = n are
// cuts); between neighbouring cuts a <= r < b the order statistics of ranks
// a..b-1 are z_a..z_{b-1} sorted.  The order statistic of rank r is thus the
// key of rank r - a among the few values between the cuts around r.  The
// maxima before and minima after every chunk of 64 ranks come from one
// streaming pass and a scan; inside a chunk, from wave scans.
// ---------------------------------------------------------------------------
constexpr int MK_REACH = 8;  // chunks searched on either side of a rank for a cut

template <typename K>
__device__ __forceinline__ K shfl_key(K v, int src) {
    return (K)__shfl((unsigned long long)v, src);
}

// Key of the matched value of the prior with key kp at rank r.
template <typename K>
__device__ __forceinline__ K matched_key(K kp, int64_t r, const double *dk, double nd, double Q) {
    using V = typename KeyTraits<K>::V;
    return key_of(matched_value<V>((V)value_of(kp), (uint64_t)r, dk, nd, Q));
}

// Arguments of the matched-knot kernels.  Equal lengths (segs == NULL):
// ensemble s holds keys [s n, s n + n) and knot rows s of qt, qp (strides
// qts, qps) and q.  Unequal lengths: the segment table.
struct MkArgs {
    const void *sorted;  // the sorted keys
    int64_t n, nch, ngr;  // equal lengths: ranks, chunks, groups per ensemble
    const double *qt, *qp;
    int64_t qts, qps;
    double *q;
    const MkSeg *segs;
    const int *group_seg;
    void *pre, *suf, *gx, *gn;  // extremes: [chunks], [chunks], [groups], [groups]
    int nq;
    int *flag;     // raised where some ensemble's knots need the sort
    int *segflag;  // unequal lengths: one flag per ensemble, or NULL
};

// One ensemble as the kernels see it.
struct MkRef {
    int64_t base, n, nch, ngr, ch0, gr0;
    const double *qt, *qp;
    double *q;
};

template <bool VAR>
__device__ __forceinline__ MkRef mk_ref(const MkArgs &A, int s) {
    MkRef R;
    if constexpr (VAR) {
        const MkSeg g = A.segs[s];
        R.base = g.base;
        R.n = g.n;
        R.nch = (g.n + 63) / 64;
        R.ngr = (R.nch + 63) / 64;
        R.ch0 = g.ch0;
        R.gr0 = g.gr0;
        R.qt = A.qt + (int64_t)g.qt_row * (A.nq + 1);
        R.qp = A.qp + (int64_t)g.qp_row * (A.nq + 1);
        R.q = A.q + (int64_t)g.q_row * (A.nq + 1);
    } else {
        R.base = s * A.n;
        R.n = A.n;
        R.nch = A.nch;
        R.ngr = A.ngr;
        R.ch0 = s * A.nch;
        R.gr0 = s * A.ngr;
        R.qt = A.qt + s * A.qts;
        R.qp = A.qp + s * A.qps;
        R.q = A.q + (int64_t)s * (A.nq + 1);
    }
    return R;
}

__device__ __forceinline__ void load_dk(double *dk, const MkRef &R, int nq) {
    for (int j = threadIdx.x; j <= nq; j += blockDim.x) dk[j] = R.qt[j] - R.qp[j];
    __syncthreads();
}

// Chunk and group extremes.  A group is 64 chunks (4096 ranks, one block of
// 256 threads, 4 consecutive ranks per thread and pass).  For every chunk c
// of group g: pre[c] = largest key of the chunks of g before c, suf[c] =
// smallest key of the chunks of g from c on; gx[g], gn[g] = largest and
// smallest key of g (turned into the values over the groups before g and
// from g on by mk_scan).
constexpr int MK_GROUP = 64;

template <typename K, bool VAR>
__global__ void __launch_bounds__(256) mk_extremes(MkArgs A) {
    extern __shared__ double dk[];
    __shared__ K cx[MK_GROUP], cn[MK_GROUP];
    int seg;
    int64_t g;
    if constexpr (VAR) {
        seg = A.group_seg[blockIdx.x];
        g = (int64_t)blockIdx.x - A.segs[seg].gr0;
    } else {
        seg = blockIdx.y;
        g = blockIdx.x;
    }
    const MkRef R = mk_ref<VAR>(A, seg);
    load_dk(dk, R, A.nq);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const K *sorted = (const K *)A.sorted + R.base;
    const int64_t n = R.n;
    const double nd = (double)n, Q = (double)A.nq;
    // all sixteen loads of a thread first, so that they are in flight together
    K v[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t e0 = g * (MK_GROUP * 64) + w * 1024 + i * 256 + 4 * lane;
#pragma unroll
        for (int t = 0; t < 4; ++t) v[i][t] = e0 + t < n ? sorted[e0 + t] : (K)0;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        // ranks e0..e0+3 of chunk 16 w + 4 i + lane / 16 of the group
        const int64_t e0 = g * (MK_GROUP * 64) + w * 1024 + i * 256 + 4 * lane;
        K kx = 0, kn = ~(K)0;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if (e0 + t < n) {
                const K z = matched_key<K>(v[i][t], e0 + t, dk, nd, Q);
                kx = z > kx ? z : kx;
                kn = z < kn ? z : kn;
            }
        }
        for (int off = 1; off < 16; off <<= 1) {  // over the 16 lanes of the chunk
            const K ox = (K)__shfl_xor((unsigned long long)kx, off), on = (K)__shfl_xor((unsigned long long)kn, off);
            kx = ox > kx ? ox : kx;
            kn = on < kn ? on : kn;
        }
        if ((lane & 15) == 0) {
            cx[w * 16 + i * 4 + (lane >> 4)] = kx;
            cn[w * 16 + i * 4 + (lane >> 4)] = kn;
        }
    }
    __syncthreads();
    if (w == 0) {
        // lane = chunk of the group: exclusive prefix max, inclusive suffix min
        const K x = cx[lane], m = cn[lane];
        K px = x, sn = m;
        for (int off = 1; off < 64; off <<= 1) {
            const K u = shfl_key(px, lane >= off ? lane - off : lane);
            const K d = shfl_key(sn, lane + off < 64 ? lane + off : lane);
            px = u > px ? u : px;
            sn = d < sn ? d : sn;
        }
        K ex = shfl_key(px, lane > 0 ? lane - 1 : 0);
        if (lane == 0) ex = 0;
        const int64_t c = g * MK_GROUP + lane;
        if (c < R.nch) {
            ((K *)A.pre)[R.ch0 + c] = ex;
            ((K *)A.suf)[R.ch0 + c] = sn;
        }
        if (lane == 63) ((K *)A.gx)[R.gr0 + g] = px;
        if (lane == 0) ((K *)A.gn)[R.gr0 + g] = sn;
    }
}

// Per ensemble (one block of 256): gx[g] <- largest key of the groups before
// g, gn[g] <- smallest key of the groups from g on.
template <typename K, bool VAR>
__global__ void __launch_bounds__(256) mk_scan(MkArgs A) {
    __shared__ K wmx[4], wmn[4];
    const MkRef R = mk_ref<VAR>(A, blockIdx.x);
    const int64_t ngr = R.ngr;
    K *gx = (K *)A.gx + R.gr0, *gn = (K *)A.gn + R.gr0;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t per = (ngr + 255) / 256;
    const int64_t g0 = tid * per < ngr ? tid * per : ngr, g1 = g0 + per < ngr ? g0 + per : ngr;
    K lx = 0, ln = ~(K)0;
    for (int64_t g = g0; g < g1; ++g) {
        lx = gx[g] > lx ? gx[g] : lx;
        ln = gn[g] < ln ? gn[g] : ln;
    }
    K px = lx, sn = ln;
    for (int off = 1; off < 64; off <<= 1) {
        const K u = shfl_key(px, lane >= off ? lane - off : lane);
        const K d = shfl_key(sn, lane + off < 64 ? lane + off : lane);
        px = u > px ? u : px;
        sn = d < sn ? d : sn;
    }
    if (lane == 63) wmx[w] = px;
    if (lane == 0) wmn[w] = sn;
    __syncthreads();
    K ex = shfl_key(px, lane > 0 ? lane - 1 : 0);
    if (lane == 0) ex = 0;
    K es = shfl_key(sn, lane < 63 ? lane + 1 : 63);
    if (lane == 63) es = ~(K)0;
    for (int k = 0; k < 4; ++k) {
        if (k < w) ex = wmx[k] > ex ? wmx[k] : ex;
        if (k > w) es = wmn[k] < es ? wmn[k] : es;
    }
    for (int64_t g = g0; g < g1; ++g) {
        const K v = gx[g];
        gx[g] = ex;
        ex = v > ex ? v : ex;
    }
    for (int64_t g = g1 - 1; g >= g0; --g) {
        es = gn[g] < es ? gn[g] : es;
        gn[g] = es;
    }
}

// The extremes one ensemble's cut tests read.
template <typename K>
struct MkExt {
    const K *pre, *suf, *gx, *gn;
    int64_t nch, ngr;
    // largest key of the chunks before c
    __device__ K before(int64_t c) const {
        const K a = pre[c], b = gx[c / MK_GROUP];
        return a > b ? a : b;
    }
    // smallest key of the chunks from c on (c <= nch)
    __device__ K from(int64_t c) const {
        if (c >= nch) return ~(K)0;
        const int64_t g = c / MK_GROUP;
        const K a = suf[c], b = g + 1 < ngr ? gn[g + 1] : ~(K)0;
        return a < b ? a : b;
    }
};

// Cut flags of the positions 64c + lane of chunk c (the wave).
template <typename K>
__device__ __forceinline__ uint64_t chunk_cuts(const K *sorted, int64_t n, const MkExt<K> &E, int64_t c,
                                               const double *dk, double nd, double Q, int lane) {
    const int64_t p = c * 64 + lane;
    K kx = 0, kn = ~(K)0;
    if (p < n) {
        kx = matched_key<K>(sorted[p], p, dk, nd, Q);
        kn = kx;
    }
    K px = kx, sn = kn;  // inclusive prefix max, inclusive suffix min inside the chunk
    for (int off = 1; off < 64; off <<= 1) {
        const K u = shfl_key(px, lane >= off ? lane - off : lane);
        const K d = shfl_key(sn, lane + off < 64 ? lane + off : lane);
        px = u > px ? u : px;
        sn = d < sn ? d : sn;
    }
    K before = shfl_key(px, lane > 0 ? lane - 1 : 0);
    if (lane == 0) before = 0;
    const K b0 = E.before(c);
    before = b0 > before ? b0 : before;
    const K a0 = E.from(c + 1);
    const K from = a0 < sn ? a0 : sn;
    const bool cut = p == 0 || p == n || (p < n && before <= from);
    return __ballot(cut);
}

// Key of the order statistic of rank r (the wave); sets *flag (and the
// ensemble's flag when there is one) where the cuts around r are not found
// within MK_REACH chunks or lie more than 64 ranks apart.
template <typename K>
__device__ K order_stat(const K *sorted, int64_t n, const MkExt<K> &E, int64_t r, const double *dk, double nd,
                        double Q, int lane, int *flag, int *segflag) {
    const int64_t nch = E.nch;
    const int64_t c = r / 64;
    const int off = (int)(r - c * 64);
    const uint64_t mc = chunk_cuts<K>(sorted, n, E, c, dk, nd, Q, lane);
    int64_t a = -1, b = -1;
    uint64_t m = mc & (off == 63 ? ~0ull : ((2ull << off) - 1));  // positions <= r
    if (m) a = c * 64 + 63 - __builtin_clzll(m);
    for (int64_t cc = c - 1; a < 0 && cc >= 0 && cc >= c - MK_REACH; --cc) {
        m = chunk_cuts<K>(sorted, n, E, cc, dk, nd, Q, lane);
        if (m) a = cc * 64 + 63 - __builtin_clzll(m);
    }
    m = off == 63 ? 0ull : mc & ~((2ull << off) - 1);  // positions > r
    if (m) b = c * 64 + __builtin_ctzll(m);
    for (int64_t cc = c + 1; b < 0 && cc <= c + MK_REACH; ++cc) {
        if (cc >= nch) {
            b = n;
            break;
        }
        m = chunk_cuts<K>(sorted, n, E, cc, dk, nd, Q, lane);
        if (m) b = cc * 64 + __builtin_ctzll(m);
    }
    if (a < 0 || b < 0 || b - a > 64) {
        if (lane == 0) {
            *flag = 1;
            if (segflag) *segflag = 1;
        }
        return 0;
    }
    // rank r - a among z_a..z_{b-1}: count the smaller keys (ties by position)
    const int ms = (int)(b - a);
    const K w = lane < ms ? matched_key<K>(sorted[a + lane], a + lane, dk, nd, Q) : ~(K)0;
    int below = 0;
    for (int l = 0; l < ms; ++l) {
        const K o = shfl_key(w, l);
        below += (o < w || (o == w && l < lane)) ? 1 : 0;
    }
    const uint64_t sel = __ballot(lane < ms && below == (int)(r - a));
    return shfl_key(w, __builtin_ctzll(sel));
}

// Midpoint (Hazen) knots of every matched ensemble, the arithmetic of
// rs_knots on the order statistics: one wave per knot.
template <typename K, bool VAR>
__global__ void __launch_bounds__(256) mk_knots(MkArgs A) {
#pragma clang fp contract(off)
    extern __shared__ double dk[];
    const MkRef R = mk_ref<VAR>(A, blockIdx.y);
    load_dk(dk, R, A.nq);
    const int nq = A.nq;
    const int j = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (j > nq) return;
    const int lane = threadIdx.x & 63;
    const int64_t n = R.n;
    const K *sorted = (const K *)A.sorted + R.base;
    const MkExt<K> E{(const K *)A.pre + R.ch0, (const K *)A.suf + R.ch0, (const K *)A.gx + R.gr0,
                     (const K *)A.gn + R.gr0, R.nch, R.ngr};
    int *flag = A.flag;
    int *segflag = (VAR && A.segflag) ? A.segflag + blockIdx.y : nullptr;
    const double nd = (double)n, Q = (double)nq;
    const double t = (double)((int64_t)j * n) / (double)nq - 0.5;
    double v;
    if (t <= 0.0) {
        v = value_of(order_stat<K>(sorted, n, E, 0, dk, nd, Q, lane, flag, segflag));
    } else if (t >= (double)(n - 1)) {
        v = value_of(order_stat<K>(sorted, n, E, n - 1, dk, nd, Q, lane, flag, segflag));
    } else {
        const int64_t r = (int64_t)floor(t);
        const double f = t - (double)r;
        const double a = value_of(order_stat<K>(sorted, n, E, r, dk, nd, Q, lane, flag, segflag));
        const double b = value_of(order_stat<K>(sorted, n, E, r + 1, dk, nd, Q, lane, flag, segflag));
        v = a + f * (b - a);
        v = v < b ? v : b;
    }
    if (lane == 0) R.q[j] = v;
}

// ---------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------
static size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

int64_t sort_tiles(int64_t n) {
    const int64_t tile = (int64_t)RS_THREADS * RS_ITEMS;
    return (n + tile - 1) / tile;
}

size_t sort_ws_bytes(int64_t total_keys, int64_t total_tiles, int nseg, int precision, bool payload) {
    const size_t ks = precision == PR_F32 ? 4 : 8;
    size_t b = align256(total_keys * ks) * 2 + align256((size_t)total_tiles * RS_RADIX * 4) +
               align256((size_t)nseg * RS_RADIX * 4) + align256((size_t)total_tiles * 4 * 8) + 256 + 256 +
               align256((size_t)nseg * (SS_B * (8 + 4) + 8 * SS_MAX_RUNS * SS_KEEP));
    if (payload) b += align256(total_keys * 4) * 2;
    return b;
}

bool splitter_sorts(int64_t n) { return n <= SS_MAX_N; }
bool splitter_tuned(int64_t n) { return n >= SS_LARGE_N && n <= SS_MAX_N; }

size_t restrict_ws(int64_t n, int k, int precision) {
    return sort_ws_bytes((int64_t)n * k, sort_tiles(n) * k, k, precision, true);
}

template <typename K, bool VAR>
static int sort_impl(const void *x, const SortLayout &L, int64_t total_keys, int64_t total_tiles, int nq,
                     const pr_grid *hg, double *q, uint32_t *rank, uint32_t *perm, double *xs, double *mom,
                     uint32_t *hist, void *ws, hipStream_t st) {
    constexpr int ITEMS = RS_ITEMS;
    const bool payload = rank || perm;
    char *p = (char *)(((uintptr_t)ws + 255) & ~(uintptr_t)255);
    K *keys[2];
    uint32_t *vals[2] = {nullptr, nullptr};
    keys[0] = (K *)p; p += align256(total_keys * sizeof(K));
    keys[1] = (K *)p; p += align256(total_keys * sizeof(K));
    uint32_t *counts = (uint32_t *)p; p += align256((size_t)total_tiles * RS_RADIX * 4);
    uint32_t *totals = (uint32_t *)p; p += align256((size_t)L.nseg * RS_RADIX * 4);
    double *mom_part = (double *)p; p += align256((size_t)total_tiles * 4 * 8);
    if (payload) {
        vals[0] = (uint32_t *)p; p += align256(total_keys * 4);
        vals[1] = (uint32_t *)p;
    }
    HistArgs ha{hist, 0, 0.0, 0.0};
    size_t cell_lds = 0;
    if (hist) {
        ha.cells = hg->n_cells;
        ha.lo = hg->x_lo;
        ha.inv_h = (double)hg->n_cells / (hg->x_hi - hg->x_lo);
        cell_lds = (size_t)hg->n_cells * 4;
        const int64_t cnt = (int64_t)L.nseg * hg->n_cells;
        const int64_t blocks = (cnt + 255) / 256 < 1024 ? (cnt + 255) / 256 : 1024;
        hipLaunchKernelGGL(zero_u32, dim3((unsigned)blocks), dim3(256), 0, st, hist, cnt);
        PR_LAUNCHED();
    }
    int *flag = (int *)p;  // 256 bytes after the payload (or the moment) buffers
    if (payload) flag = (int *)((char *)vals[1] + align256(total_keys * 4));
    K *split = (K *)((char *)flag + 256);                               // splitters, [nseg][SS_B]
    uint32_t *bstart = (uint32_t *)(split + (size_t)L.nseg * SS_B);     // bucket starts, [nseg][SS_B]
    K *runq = (K *)(bstart + (size_t)L.nseg * SS_B);                    // thinned runs, [nseg][SS_MAX_RUNS SS_KEEP]
    const dim3 grid((unsigned)total_tiles);
    const dim3 rows((unsigned)(((int64_t)L.nseg * RS_RADIX + 3) / 4));
    const int64_t max_n = VAR ? L.max_n : L.n;
    // One LSD pass over the byte at shift: keys[in] -> keys[out] (pass 0
    // reads the values), with the statistics on the first read and the rank,
    // perm and sorted-value outputs on the last pass.
    auto pass = [&](const SortLayout &LL, int shift, bool first, bool last, int in, int out, bool stats) -> int {
        if (first)
            hipLaunchKernelGGL((rs_count<K, ITEMS, true, VAR>), grid, dim3(RS_THREADS), stats ? cell_lds : 0, st, x,
                               shift, LL, counts, (stats && mom) ? mom_part : nullptr,
                               stats ? ha : HistArgs{nullptr, 0, 0.0, 0.0});
        else
            hipLaunchKernelGGL((rs_count<K, ITEMS, false, VAR>), grid, dim3(RS_THREADS), 0, st,
                               (const void *)keys[in], shift, LL, counts, nullptr, HistArgs{nullptr, 0, 0.0, 0.0});
        PR_LAUNCHED();
        if constexpr (VAR)
            hipLaunchKernelGGL((rs_rowscan_seg<VAR>), dim3((unsigned)LL.nseg), dim3(RS_RADIX), 0, st, counts, totals,
                               LL);
        else
            hipLaunchKernelGGL((rs_rowscan<VAR>), rows, dim3(256), 0, st, counts, totals, LL);
        PR_LAUNCHED();
#define PR_SCATTER(FIRST, LAST, PAY, SRC, VIN, VOUT)                                                            \
    hipLaunchKernelGGL((rs_scatter<K, ITEMS, FIRST, LAST, PAY, VAR>), grid, dim3(RS_THREADS), 0, st, SRC, VIN,     \
                       keys[out], VOUT, (const uint32_t *)counts, (const uint32_t *)totals, shift, LL,         \
                       LAST ? rank : nullptr, LAST ? perm : nullptr, LAST ? xs : nullptr)
        if (payload) {
            if (first) PR_SCATTER(true, false, true, x, nullptr, vals[out]);
            else if (!last) PR_SCATTER(false, false, true, (const void *)keys[in], vals[in], vals[out]);
            else PR_SCATTER(false, true, true, (const void *)keys[in], vals[in], nullptr);
        } else {
            if (first) PR_SCATTER(true, false, false, x, nullptr, nullptr);
            else if (!last) PR_SCATTER(false, false, false, (const void *)keys[in], nullptr, nullptr);
            else PR_SCATTER(false, true, false, (const void *)keys[in], nullptr, nullptr);
        }
#undef PR_SCATTER
        PR_LAUNCHED();
        return PR_OK;
    };
    constexpr int P = KeyTraits<K>::passes;
    const bool splitter = !L.radix && max_n > 0 && max_n <= SS_MAX_N;
    const bool many = max_n > (VAR ? SS_CAP : SS_BIG);  // some ensemble is more than one bucket
    if (splitter) {
        K *skeys = keys[1 - sorted_buffer<K>()], *out = keys[sorted_buffer<K>()];
        const int nb = ss_buckets<VAR>(max_n), runs = ss_runs(nb);
        if (many) {
            hipLaunchKernelGGL((ss_sample<K, VAR>), dim3((unsigned)(runs * L.nseg)), dim3(SS_RUN), 0, st, x, L, runs,
                               runq);
            PR_LAUNCHED();
            hipLaunchKernelGGL((ss_splitters<K, VAR>), dim3((unsigned)L.nseg), dim3(1024), 0, st, (const K *)runq, L,
                               split);
            PR_LAUNCHED();
        }
        if (many || mom || hist) {
            hipLaunchKernelGGL((ss_count<K, VAR>), grid, dim3(SC_THREADS), cell_lds, st, x, (const K *)split, L,
                               counts, mom ? mom_part : nullptr, ha, vals[0]);
            PR_LAUNCHED();
        }
        if (many) {
            if constexpr (VAR)
                hipLaunchKernelGGL(ss_rowscan_seg, dim3((unsigned)L.nseg), dim3(SS_B), 0, st, counts, totals, L);
            else
                hipLaunchKernelGGL(ss_rowscan, dim3((unsigned)((nb + 3) / 4), (unsigned)L.nseg), dim3(256), 0, st,
                                   counts, totals, L);
            PR_LAUNCHED();
            hipLaunchKernelGGL((ss_scatter<K, VAR>), grid, dim3(SC_THREADS), 0, st, x, (const uint32_t *)vals[0],
                               (const K *)split, skeys, out, xs, rank ? vals[0] : nullptr, perm,
                               (const uint32_t *)counts, (const uint32_t *)totals, L, bstart);
            PR_LAUNCHED();
        }
        // the ranks' final array is free until ss_finish writes it, the
        // runs' since the splitters were taken
        const BucketArgs<K> A{x, skeys, totals, bstart, split, out, vals[1], rank, perm,
                              payload ? (rank ? rank : vals[0]) : nullptr, xs, q, (uint32_t *)runq, nq};
        const bool big = !VAR && !many && max_n > SS_CAP;  // ensembles of one bucket above SS_CAP
        const bool whole = !many && L.nseg <= SS_WHOLE;
        // many small FP32 ensembles: crowded ones in the same launch, all by digits
        const bool alike = !payload && (sizeof(K) == 8 || many || whole);
        const bool here = big || whole || (sizeof(K) == 4 && !alike);
        auto sort = [&](auto al) {
            constexpr bool AL = decltype(al)::value;
            if (big) {
                if constexpr (!VAR)
                    hipLaunchKernelGGL((ss_bucket_sort<K, VAR, SS_IT_BIG, true, AL>), grid, dim3(SS_BT), 0, st, A, L);
            } else if (here)
                hipLaunchKernelGGL((ss_bucket_sort<K, VAR, SS_IT, true, AL>), grid, dim3(SS_BT), 0, st, A, L);
            else
                hipLaunchKernelGGL((ss_bucket_sort<K, VAR, SS_IT, false, AL>), grid, dim3(SS_BT), 0, st, A, L);
            PR_LAUNCHED();
            if (many || !here) {
                hipLaunchKernelGGL((ss_left<K, VAR, AL>), dim3((unsigned)std::min<int64_t>(total_tiles, 256)),
                                   dim3(SS_BT), 0, st, A, L, total_tiles);
                PR_LAUNCHED();
            }
            return PR_OK;
        };
        PR_CHECK(alike ? sort(std::true_type{}) : sort(std::false_type{}));
        if (many || mom) {
            const int64_t blocks = L.nseg + (many && rank ? total_tiles : 0);
            hipLaunchKernelGGL((ss_finish<K, VAR>), dim3((unsigned)blocks), dim3(SC_THREADS), 0, st,
                               many ? (const K *)out : nullptr, nq, q, mom ? (const double *)mom_part : nullptr, mom,
                               (const uint32_t *)vals[0], (const uint32_t *)vals[1], (const uint32_t *)counts,
                               (const uint32_t *)totals, (const uint32_t *)bstart, (const K *)split, L, rank);
            PR_LAUNCHED();
        }
    } else if constexpr (std::is_same<K, uint64_t>::value) {
        // the high 32 bits (passes 4..7, ending in buffer 1), the fix-up of
        // runs of equal high halves into buffer 0, and the complete sort
        // (also ending in buffer 0) only where a run is too long for it
        for (int j = 0; j < 4; ++j) PR_CHECK(pass(L, 32 + 8 * j, j == 0, false, (j + 1) & 1, j & 1, true));
        hipLaunchKernelGGL(zero_u32, dim3(1), dim3(64), 0, st, (uint32_t *)flag, (int64_t)1);
        PR_LAUNCHED();
        // a segment table's ranks through the staging buffer (vals[1], free
        // once the fix-up has read it) where every segment fits the packing,
        // the fix-up then writing the permutation in order (into vals[0]
        // unless asked for) instead of the ranks; the complete sort behind it
        // keeps storing the ranks itself
        const bool staged_ranks = VAR && rank != nullptr && max_n > 0 && max_n <= RK_MAX_N;
        uint32_t *perm_fix = perm ? perm : (staged_ranks ? vals[0] : nullptr);
        if (payload)
            hipLaunchKernelGGL((rs_fixup<VAR, true>), grid, dim3(RS_THREADS), 0, st, (const uint64_t *)keys[1],
                               (const uint32_t *)vals[1], (uint64_t *)keys[0], L, staged_ranks ? nullptr : rank,
                               perm_fix, xs, flag);
        else
            hipLaunchKernelGGL((rs_fixup<VAR, false>), grid, dim3(RS_THREADS), 0, st, (const uint64_t *)keys[1],
                               (const uint32_t *)nullptr, (uint64_t *)keys[0], L, rank, perm, xs, flag);
        PR_LAUNCHED();
        if constexpr (VAR) {
            if (staged_ranks) {
                const int64_t zb = (total_tiles + 255) / 256 < 1024 ? (total_tiles + 255) / 256 : 1024;
                hipLaunchKernelGGL(zero_u32, dim3((unsigned)zb), dim3(256), 0, st, counts, total_tiles);
                PR_LAUNCHED();
                hipLaunchKernelGGL(rs_rank_bucket, grid, dim3(RS_THREADS), 0, st, (const uint32_t *)perm_fix, L, counts,
                                   vals[1], (const int *)flag);
                PR_LAUNCHED();
                hipLaunchKernelGGL(rs_rank_place, grid, dim3(RS_THREADS), 0, st, (const uint32_t *)vals[1], L, rank,
                                   (const int *)flag);
                PR_LAUNCHED();
            }
        }
        SortLayout LG = L;
        LG.guard = flag;
        for (int j = 0; j < P; ++j) PR_CHECK(pass(LG, 8 * j, j == 0, j == P - 1, j & 1, (j + 1) & 1, false));
    } else {
        for (int j = 0; j < P; ++j) PR_CHECK(pass(L, 8 * j, j == 0, j == P - 1, (j + 1) & 1, j & 1, true));
    }
    if (splitter) return PR_OK;
    hipLaunchKernelGGL((rs_knots<K, VAR>), dim3(L.nseg), dim3(128), 0, st, (const K *)keys[sorted_buffer<K>()], L, nq,
                       q);
    PR_LAUNCHED();
    if (mom) {
        hipLaunchKernelGGL((rs_moments<VAR>), dim3(L.nseg), dim3(64), 0, st, (const double *)mom_part, L, mom);
        PR_LAUNCHED();
    }
    return PR_OK;
}

int restrict_quantiles(const void *x, int precision, int64_t n, int k, int nq, const pr_grid *hg, double *q,
                       uint32_t *rank, uint32_t *perm, double *xs, double *mom, uint32_t *hist, void *ws,
                       hipStream_t st) {
    SortLayout L{n, (int)sort_tiles(n), k, nullptr, nullptr};
    const int64_t tiles = (int64_t)L.nblk * k;
    if (precision == PR_F64)
        return sort_impl<uint64_t, false>(x, L, n * k, tiles, nq, hg, q, rank, perm, xs, mom, hist, ws, st);
    return sort_impl<uint32_t, false>(x, L, n * k, tiles, nq, hg, q, rank, perm, xs, mom, hist, ws, st);
}

int restrict_knots_guarded(const void *x, int precision, int64_t n, int k, int nq, double *q, void *ws,
                           const int *guard, hipStream_t st) {
    SortLayout L{n, (int)sort_tiles(n), k, nullptr, nullptr, guard};
    const int64_t tiles = (int64_t)L.nblk * k;
    if (precision == PR_F64)
        return sort_impl<uint64_t, false>(x, L, n * k, tiles, nq, nullptr, q, nullptr, nullptr, nullptr, nullptr,
                                          nullptr, ws, st);
    return sort_impl<uint32_t, false>(x, L, n * k, tiles, nq, nullptr, q, nullptr, nullptr, nullptr, nullptr,
                                      nullptr, ws, st);
}

int restrict_segments(const double *x, const SortLayout &L, int64_t total_keys, int64_t total_tiles, int nq,
                      double *q, uint32_t *rank, void *ws, hipStream_t st) {
    return sort_impl<uint64_t, true>(x, L, total_keys, total_tiles, nq, nullptr, q, rank, nullptr, nullptr, nullptr,
                                     nullptr, ws, st);
}


template <typename K, bool VAR>
static int launch_matched_knots(const MkArgs &A, unsigned ngroups_or_x, int nseg, hipStream_t st) {
    const size_t lds = (size_t)(A.nq + 1) * sizeof(double);
    hipLaunchKernelGGL(zero_u32, dim3(1), dim3(64), 0, st, (uint32_t *)A.flag, (int64_t)1);
    PR_LAUNCHED();
    if (A.segflag) {
        hipLaunchKernelGGL(zero_u32, dim3((unsigned)((nseg + 255) / 256)), dim3(256), 0, st, (uint32_t *)A.segflag,
                           (int64_t)nseg);
        PR_LAUNCHED();
    }
    const dim3 eg = VAR ? dim3(ngroups_or_x) : dim3(ngroups_or_x, (unsigned)nseg);
    hipLaunchKernelGGL((mk_extremes<K, VAR>), eg, dim3(256), lds, st, A);
    PR_LAUNCHED();
    hipLaunchKernelGGL((mk_scan<K, VAR>), dim3((unsigned)nseg), dim3(256), 0, st, A);
    PR_LAUNCHED();
    hipLaunchKernelGGL((mk_knots<K, VAR>), dim3((unsigned)((A.nq + 1 + 3) / 4), (unsigned)nseg), dim3(256), lds, st,
                       A);
    PR_LAUNCHED();
    return PR_OK;
}

// The workspace as sort_impl lays it out: two key buffers of kb bytes, the
// sorted keys in the one the last pass wrote; the other is free scratch.
template <typename K>
static void key_buffers(const void *ws, size_t kb, const void **sorted, void **scratch) {
    char *p = (char *)(((uintptr_t)ws + 255) & ~(uintptr_t)255);
    constexpr int last = sorted_buffer<K>();
    *sorted = p + last * kb;
    *scratch = p + (1 - last) * kb;
}

template <typename K>
static int matched_knots_impl(const void *ws, int64_t n, int k, int nq, const double *qt, int64_t qts,
                              const double *qp, int64_t qps, double *q, int *flag, hipStream_t st) {
    const size_t kb = align256((size_t)n * k * sizeof(K));
    const int64_t nch = (n + 63) / 64, ngr = (nch + MK_GROUP - 1) / MK_GROUP;
    if ((size_t)2 * (nch + ngr) * k * sizeof(K) > kb) return PR_E_UNSUPPORTED;
    const void *sorted;
    void *scratch;
    key_buffers<K>(ws, kb, &sorted, &scratch);
    K *pre = (K *)scratch, *suf = pre + nch * k, *gx = suf + nch * k, *gn = gx + ngr * k;
    const MkArgs A{sorted, n, nch, ngr, qt, qp, qts, qps, q, nullptr, nullptr, pre, suf, gx, gn, nq, flag, nullptr};
    return launch_matched_knots<K, false>(A, (unsigned)ngr, k, st);
}

int matched_knots_segments(const void *ws, int64_t total_keys, int nseg, const MkSeg *segs, const int *group_seg,
                           int64_t total_chunks, int64_t total_groups, int nq, const double *qt, const double *qp,
                           double *q, int *flag, int *segflag, hipStream_t st) {
    const size_t kb = align256((size_t)total_keys * sizeof(uint64_t));
    if ((size_t)2 * (total_chunks + total_groups) * sizeof(uint64_t) > kb) return PR_E_UNSUPPORTED;
    const void *sorted;
    void *scratch;
    key_buffers<uint64_t>(ws, kb, &sorted, &scratch);
    uint64_t *pre = (uint64_t *)scratch, *suf = pre + total_chunks, *gx = suf + total_chunks,
             *gn = gx + total_groups;
    const MkArgs A{sorted, 0, 0, 0, qt, qp, 0, 0, q, segs, group_seg, pre, suf, gx, gn, nq, flag, segflag};
    return launch_matched_knots<uint64_t, true>(A, (unsigned)total_groups, nseg, st);
}

int matched_knots(const void *ws, int precision, int64_t n, int k, int nq, const double *qt, int64_t qt_stride,
                  const double *qp, int64_t qp_stride, double *q, int *flag, hipStream_t st) {
    if (precision == PR_F64)
        return matched_knots_impl<uint64_t>(ws, n, k, nq, qt, qt_stride, qp, qp_stride, q, flag, st);
    return matched_knots_impl<uint32_t>(ws, n, k, nq, qt, qt_stride, qp, qp_stride, q, flag, st);
}
}  // namespace pr

using namespace pr;

extern "C" size_t pr_restrict_workspace_size(int64_t n, int k, int precision) {
    if (n <= 0 || k <= 0) return 256;
    return restrict_ws(n, k, precision);
}

extern "C" int pr_restrict_quantiles(const void *x, int precision, int64_t n, int k, int n_q,
                                     const pr_grid *hist_grid, double *q, uint32_t *rank, uint32_t *perm,
                                     double *x_sorted, double *moments, uint32_t *hist, void *ws,
                                     size_t ws_bytes, void *stream) {
    clear_error();
    PR_REQUIRE(valid_precision(precision), "precision must be 64 or 32");
    PR_REQUIRE(n >= 1 && n <= 0xFFFFFFFFll, "n must be in [1, 2^32)");
    PR_REQUIRE(k >= 1 && k <= 65535, "k must be in [1, 65535]");
    PR_REQUIRE(n_q >= 1 && n_q <= 1 << 20, "n_q must be in [1, 2^20]");
    PR_REQUIRE(x != nullptr && q != nullptr && ws != nullptr, "x, q and ws must be non-NULL");
    PR_REQUIRE((int64_t)n * k <= 0x7FFFFFFFFFFFll, "n * k too large");
    if (hist) {
        PR_REQUIRE(hist_grid != nullptr, "hist requires hist_grid");
        PR_REQUIRE(hist_grid->n_cells >= 1 && hist_grid->n_cells <= 8192 && hist_grid->x_lo < hist_grid->x_hi,
                   "hist_grid must have 1..8192 cells and x_lo < x_hi");
    }
    if (ws_bytes < restrict_ws(n, k, precision)) {
        set_error("workspace too small: %zu < %zu bytes", ws_bytes, restrict_ws(n, k, precision));
        return PR_E_NOMEM;
    }
    return restrict_quantiles(x, precision, n, k, n_q, hist_grid, q, rank, perm, x_sorted, moments, hist, ws,
                              as_stream(stream));
}

// ---------------------------------------------------------------------------
// Restriction without allocation: the workspace is a file-scope device array
// of PR_STATIC_SCRATCH_BYTES (one copy per GPU, held until the process ends).
// Host code never passes the array's name to a kernel: its device address on
// the current GPU is taken once per device with hipGetSymbolAddress and kept.
// ---------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[PR_STATIC_SCRATCH_BYTES];

namespace pr {
namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

int scratch_on_current_device(void **out) {
    int dev = 0;
    PR_HIP(hipGetDevice(&dev));
    PR_REQUIRE(dev >= 0 && dev < kMaxDevices, "device %d outside the %d devices served", dev, kMaxDevices);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || ptr == nullptr) {
            set_error("hipGetSymbolAddress of the static scratch failed: %s", hipGetErrorString(e));
            return PR_E_HIP;
        }
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return PR_OK;
}
}  // namespace
}  // namespace pr

extern "C" int pr_restrict_quantiles_static(const void *x, int precision, int64_t n, int k, int n_q,
                                            const pr_grid *hist_grid, double *q, uint32_t *rank, uint32_t *perm,
                                            double *x_sorted, double *moments, uint32_t *hist, void *stream) {
    clear_error();
    PR_REQUIRE(valid_precision(precision), "precision must be 64 or 32");
    PR_REQUIRE(n >= 1 && n <= 0xFFFFFFFFll, "n must be in [1, 2^32)");
    PR_REQUIRE(k >= 1 && k <= 65535, "k must be in [1, 65535]");
    PR_REQUIRE(n_q >= 1 && n_q <= 1 << 20, "n_q must be in [1, 2^20]");
    PR_REQUIRE(x != nullptr && q != nullptr, "x and q must be non-NULL");
    if (hist) {
        PR_REQUIRE(hist_grid != nullptr, "hist requires hist_grid");
        PR_REQUIRE(hist_grid->n_cells >= 1 && hist_grid->n_cells <= 8192 && hist_grid->x_lo < hist_grid->x_hi,
                   "hist_grid must have 1..8192 cells and x_lo < x_hi");
    }
    const size_t need = restrict_ws(n, k, precision);
    if (need > (size_t)PR_STATIC_SCRATCH_BYTES) {
        set_error("n * k = %lld keys need %zu bytes of scratch; the static scratch holds %zu",
                  (long long)n * k, need, (size_t)PR_STATIC_SCRATCH_BYTES);
        return PR_E_NOMEM;
    }
    void *ws = nullptr;
    PR_CHECK(scratch_on_current_device(&ws));
    return restrict_quantiles(x, precision, n, k, n_q, hist_grid, q, rank, perm, x_sorted, moments, hist, ws,
                              as_stream(stream));
}

extern "C" int pr_match_knots(const double *q_target, const double *q_prior, int64_t n, int k, int n_q,
                              int precision, void *ws, size_t ws_bytes, double *q_out, int *flag, void *stream) {
    clear_error();
    PR_REQUIRE(valid_precision(precision), "precision must be 64 or 32");
    PR_REQUIRE(n >= 1 && n <= 0xFFFFFFFFll, "n must be in [1, 2^32)");
    PR_REQUIRE(k >= 1 && k <= 65535, "k must be in [1, 65535]");
    PR_REQUIRE(n_q >= 1 && n_q <= 8191, "n_q must be in [1, 8191]");
    PR_REQUIRE(q_target && q_prior && ws && q_out && flag, "pointers must be non-NULL");
    if (ws_bytes < restrict_ws(n, k, precision)) {
        set_error("workspace too small: %zu < %zu bytes", ws_bytes, restrict_ws(n, k, precision));
        return PR_E_NOMEM;
    }
    const int rc = matched_knots(ws, precision, n, k, n_q, q_target, n_q + 1, q_prior, n_q + 1, q_out, flag,
                                 as_stream(stream));
    if (rc == PR_E_UNSUPPORTED) set_error("n = %lld is too small for the workspace to hold the chunk extremes",
                                          (long long)n);
    return rc;
}
