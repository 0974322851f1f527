// Row analysis and binning (the work estimate of Section 2: flops(A,B)
// counts scalar multiplications; Gustavson's cost is O(flops + nnz + m + n),
// Section 3).  For each row i of A, restricted to the inner window
// [k_lo, k_hi):
//   a_beg[i], a_end[i]  index range of A's stored entries inside the window
//   flops[i]            sum over those entries k of nnz(B(k,:))
//   maxb[i]             max over those k of nnz(B(k,:))  (a lower bound of nnz(C(i,:)))
//   bin[i]              the accumulator class the row is sent to
// Rows with at most LONG_ROW entries are handled by 16-lane groups, longer ones
// by a wave and those above HUB_ROW by their whole workgroup, so no wave walks
// a hub row alone.
#pragma once
#include "common.hpp"

namespace spg {

struct BinParams {
    int32_t small_max_flops;  // <= 64
    int32_t hash_max_flops;   // symbolic hash limit
    int32_t hash_max_nnz;     // numeric hash limit
    int32_t dense_ok;         // symbolic LDS bitmap allowed (n <= 2^19)
    int32_t rank_max_log2;    // numeric rank-space accumulator: largest capacity (log2), 0 = off
    int32_t chunk_counts;     // the bitmap pass records per-chunk counts for the numeric chunks
    int32_t chunk_min_nnz;    // rows with chunk counts and more outputs than this take rank chunks
    int32_t heap_max_lists;   // rows with at most this many A entries ...
    int32_t heap_max_flops;   // ... and products take the k-way merge (heap) bin; 0 = off
    int64_t ncols;            // n
};

constexpr int NBINS = 17;
constexpr int BIN_EMPTY = 0, BIN_TINY = 1, BIN_SMALL = 2, BIN_HASH0 = 3, BIN_DENSE = 12;
constexpr int BIN_DENSE_PAR = 11;  // numeric: column chunks of one row in parallel
constexpr int BIN_RANK0 = 13;  // rank-space accumulator, capacity 4096 << (b - BIN_RANK0)
constexpr int BIN_HEAP = 16;   // k-way merge of the row's few B rows (both passes)
constexpr int RANK_MIN_LOG2 = 12;
constexpr int LONG_ROW = 128, HUB_ROW = 2048;
constexpr int HASH_MIN_LOG2 = 7;  // 128 slots

__device__ inline int ceil_log2_i64(int64_t x) {
    return x <= 1 ? 0 : 64 - __clzll((unsigned long long)(x - 1));
}

// Symbolic bin from the row's work.
__device__ inline int sym_bin(int64_t flops, int64_t annz, const BinParams& bp) {
    if (flops == 0) return BIN_EMPTY;
    if (annz == 1) return BIN_TINY;
    if (flops <= bp.small_max_flops) return BIN_SMALL;
    if (annz <= bp.heap_max_lists && flops <= bp.heap_max_flops) return BIN_HEAP;
    // a bitmap over all n columns costs n/32 words to clear and count; use it
    // once the row's products outnumber that, or once a hash table would not fit
    bool bitmap_cheaper = bp.dense_ok && flops * 32 >= bp.ncols;
    if (flops <= bp.hash_max_flops && !bitmap_cheaper) {  // larger rows: bitmap, in blocks if n is large
        // at most 3/4 of the slots in use (the row's distinct columns are at most its products)
        int lg = ceil_log2_i64((4 * flops + 2) / 3);
        if (lg < HASH_MIN_LOG2) lg = HASH_MIN_LOG2;
        return BIN_HASH0 + (lg - HASH_MIN_LOG2);
    }
    return BIN_DENSE;
}

// Numeric bin from the exact output count.  Rows whose symbolic pass kept
// a full-width bitmap (sym_dense) reuse it: their values accumulate in LDS
// indexed by output rank when the count fits the largest capacity.
__device__ inline int num_bin(int64_t flops, int64_t annz, int64_t cnt, bool sym_dense,
                              const BinParams& bp) {
    if (cnt == 0) return BIN_EMPTY;
    if (annz == 1) return BIN_TINY;
    if (flops <= bp.small_max_flops) return BIN_SMALL;
    if (annz <= bp.heap_max_lists && flops <= bp.heap_max_flops) return BIN_HEAP;  // as in the symbolic pass
    if (sym_dense && bp.rank_max_log2 && cnt <= (1ll << bp.rank_max_log2)) {
        int lg = ceil_log2_i64(cnt);
        if (lg < RANK_MIN_LOG2) lg = RANK_MIN_LOG2;
        return BIN_RANK0 + (lg - RANK_MIN_LOG2);
    }
    // rows with a saved bitmap and chunk counts may take rank chunks before
    // the largest hash tables
    const bool chunks_ok = sym_dense && bp.chunk_counts;
    const int64_t hash_lim = chunks_ok ? bp.chunk_min_nnz : bp.hash_max_nnz;
    if (cnt <= hash_lim) {
        int lg = ceil_log2_i64((4 * cnt + 2) / 3);  // at most 3/4 of the slots in use
        if (lg < HASH_MIN_LOG2) lg = HASH_MIN_LOG2;
        return BIN_HASH0 + (lg - HASH_MIN_LOG2);
    }
    return chunks_ok ? BIN_DENSE_PAR : BIN_DENSE;
}

// Work of a bin's kernel, from the counts of a classification ([0, NBINS) rows,
// [NBINS, 2 NBINS) products).
inline double bin_work(const int64_t* counts, int bin) {
    return (double)counts[NBINS + bin] + 32.0 * (double)counts[bin];
}

// Whether a pass is spread over the helper streams at all, from the counts of a
// classification that launches a kernel for every bin with rows from first_bin on.
// A fork and a join cost ten calls on the host and waits between the GPU's queues,
// 20 to 50 us a pass; what they save is the latency of each further kernel, which is
// that of a few rows however many it has: a bin's share of the work says little.
// So: from six kernels on (power-law matrices; uniform ones and stencils have
// fewer), and not for few products.
// Gain of four streams over one, whole products of random graphs of 1M to 400M
// products, us by symbolic kernels: two to four -69 to -42, five -50 to -21, six -96
// to 57, seven and more -26 to 193 (R-MAT scale 16, eight: 1948 -> 1924; the
// rectangular boolean product, seven: 516 -> 470).
constexpr int64_t FORK_MIN_PRODUCTS = 1 << 20;
constexpr int FORK_MIN_KERNELS = 6;
inline bool worth_forking(const int64_t* counts, int first_bin) {
    int64_t products = 0;
    int kernels = 0;
    for (int b = BIN_TINY; b < NBINS; ++b) {
        products += counts[NBINS + b];
        kernels += b >= first_bin && counts[b] > 0;
    }
    return products >= FORK_MIN_PRODUCTS && kernels >= FORK_MIN_KERNELS;
}
// The numeric pass: spread where the symbolic pass was (one serial pass after one
// that was spread was slower than either alone: ER 21,083 x 55,716 x 32,369 230 us
// both spread, 243 neither, 272 the symbolic pass only), and also where its own
// kernels, besides the copies of rows of one A entry, are as many and the three kinds
// with a bitmap's ranks (rank chunks, two capacities of whole rows) share its work:
// their workgroups, which the LDS limits, overlap well.  The heavy rows of a product
// with predicted sizes, all of them symbolic bitmap rows, whole call on one stream and
// on several: R-MAT scale 16, 16 entries a row (78, 15 and 7% of the work) 2331 / 2158
// us, 8 a row (51, 29, 17%) 1431 / 1337, scale 15 (57, 28, 14%) 986 / 940.  Hash and
// rank kernels of few rows lose: R-MAT 13,550 x 20,699 x 9387 225 / 275 us, two rank
// kernels SSCA 12,249 243 / 293.
constexpr double HEAVY_SHARE = 0.05;
inline bool worth_forking_numeric(const int64_t* counts, bool symbolic_spread) {
    if (symbolic_spread) return true;
    if (!worth_forking(counts, BIN_SMALL)) return false;
    double total = 0;
    for (int b = BIN_TINY; b < NBINS; ++b) total += bin_work(counts, b);
    int heavy = 0;
    for (int b : {BIN_DENSE_PAR, BIN_RANK0, BIN_RANK0 + 1, BIN_RANK0 + 2})
        heavy += bin_work(counts, b) >= HEAVY_SHARE * total;
    return heavy >= 3;
}

// The rows of one bin, located on the device: the per-bin row counts (the
// lists of the bins below b come first in `lists`).  Kernels launched this
// way stride over the bin's rows, so their launches need no host copy of
// the counts (the grid only sizes the parallelism).
struct BinRef {
    const int64_t* counts;
    const int32_t* lists;
    int32_t bin;
    __device__ inline void locate(const int32_t*& rows, int64_t& n) const {
        int64_t off = 0;
        for (int x = 0; x < bin; ++x) off += counts[x];
        rows = lists + off;
        n = counts[bin];
    }
};

// Rows of a bin over workgroups: row r goes to workgroup r mod gridDim.x.
// body(r, i) gets the position r in the bin list and the row i; it may use
// barriers (all threads call it).
template <class Body>
__device__ inline void for_each_bin_row(const BinRef& ref, Body body) {
    const int32_t* rows;
    int64_t n;
    ref.locate(rows, n);
    for (int64_t r = blockIdx.x; r < n; r += gridDim.x) {
        body(r, (int64_t)rows[r]);
        __syncthreads();  // the row is done with the LDS
    }
}

// Longest-processing-time order of the row lists of a run of consecutive
// bins [b_lo, b_hi): within each bin, rows with more products first, so that
// the heaviest workgroups start early and the end of a launch is not held up
// by a large row that started last.  The classification counts the rows of
// those bins by (bin, work class) and the scatter places them by it; 256 work
// classes per bin, 8 per power of two of the products (rows within about 12%
// of each other share a class).
constexpr int LPT_KEYS = 256;
constexpr int LPT_MAX_BINS = 5;
__device__ inline int lpt_class(int64_t w) {
    if (w < 1) w = 1;
    const int e = 63 - __clzll((unsigned long long)w);  // floor(log2 w)
    const int frac = e >= 3 ? (int)((w >> (e - 3)) & 7) : (int)((w << (3 - e)) & 7);
    const int k = e * 8 + frac;
    return LPT_KEYS - 1 - (k < LPT_KEYS - 1 ? k : LPT_KEYS - 1);  // more work: smaller class
}
struct OrderedBins {
    int32_t b_lo, b_hi;  // none when equal
    int32_t* hist;       // rows by key, (b_hi - b_lo) LPT_KEYS of them
    const int64_t* work;
    __host__ __device__ bool has(int b) const { return b >= b_lo && b < b_hi; }
    __device__ int key(int b, int64_t w) const { return (b - b_lo) * LPT_KEYS + lpt_class(w); }
    __host__ __device__ int keys() const { return (b_hi - b_lo) * LPT_KEYS; }
};

struct RowInfoOut {
    int64_t* a_beg;
    int64_t* a_end;
    int64_t* flops;
    int32_t* maxb;
    uint8_t* bin;
    int64_t* cnt;        // symbolic counts (c_row_ptr + 1); EMPTY/TINY rows written here
    int64_t* bin_stats;  // [3][NBINS]: rows, flops, A entries
    unsigned long long* max_flops;  // largest flops_i over the rows (one value)
    OrderedBins order;
};

__device__ inline int64_t lower_bound_col(const int32_t* col, int64_t lo, int64_t hi, int64_t key) {
    while (lo < hi) {
        int64_t mid = (lo + hi) >> 1;
        if ((int64_t)col[mid] < key) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// Per-workgroup statistics of a classification, added to the global ones once.
// Device-wide atomics on a few addresses serialize across the XCDs (about 2 ns
// each), so the classification grids are kept to few, large workgroups.
constexpr int CLASS_NT = 1024;
template <int NV>
struct ClassLds {
    int32_t rows[NBINS];
    unsigned long long v[NV][NBINS];
    unsigned long long fmax;
    int32_t lpt[LPT_KEYS * LPT_MAX_BINS];

    __device__ void clear(const OrderedBins& o) {
        if (threadIdx.x < NBINS) {
            rows[threadIdx.x] = 0;
            for (int x = 0; x < NV; ++x) v[x][threadIdx.x] = 0;
        }
        if (threadIdx.x == 0) fmax = 0;
        for (int k = threadIdx.x; k < o.keys(); k += CLASS_NT) lpt[k] = 0;
        __syncthreads();
    }
    __device__ void flush(const OrderedBins& o, int64_t* stats, unsigned long long* max_flops) {
        __syncthreads();
        if (threadIdx.x < NBINS && rows[threadIdx.x]) {
            const int b = threadIdx.x;
            atomicAdd((unsigned long long*)&stats[b], (unsigned long long)rows[b]);
            for (int x = 0; x < NV; ++x) atomicAdd((unsigned long long*)&stats[(x + 1) * NBINS + b], v[x][b]);
        }
        if (max_flops && threadIdx.x == 0 && fmax) atomicMax(max_flops, fmax);
        for (int k = threadIdx.x; k < o.keys(); k += CLASS_NT)
            if (lpt[k]) atomicAdd(&o.hist[k], lpt[k]);
    }
};

__device__ inline void finish_row(int64_t i, int64_t beg, int64_t end, int64_t f, int32_t mb,
                                  const BinParams& bp, const RowInfoOut& o, ClassLds<2>& c) {
    o.a_beg[i] = beg;
    o.a_end[i] = end;
    o.flops[i] = f;
    o.maxb[i] = mb;
    int b = sym_bin(f, end - beg, bp);
    o.bin[i] = (uint8_t)b;
    if (b == BIN_EMPTY) o.cnt[i] = 0;
    else if (b == BIN_TINY) o.cnt[i] = f;  // nnz(C(i,:)) = nnz(B(k,:)) exactly
    atomicAdd(&c.rows[b], 1);
    atomicAdd(&c.v[0][b], (unsigned long long)f);
    atomicAdd(&c.v[1][b], (unsigned long long)(end - beg));
    if (o.order.has(b)) atomicAdd(&c.lpt[o.order.key(b, f)], 1);
}

// Products and longest B row of A's entries lb + t, lb + t + stride, ... < le, four in flight.
__device__ inline void walk_entries(const Csr& A, const Csr& B, int64_t lb, int64_t le, int t, int stride, int64_t& f,
                                    int32_t& mb) {
    constexpr int U = 4;
    f = 0;
    mb = 0;
    for (int64_t p0 = lb + t; p0 < le; p0 += U * stride) {
        int64_t k[U], l[U];
#pragma unroll
        for (int u = 0; u < U; ++u) k[u] = p0 + u * stride < le ? (int64_t)A.col[p0 + u * stride] : -1;
#pragma unroll
        for (int u = 0; u < U; ++u) l[u] = k[u] >= 0 ? B.rp[k[u] + 1] - B.rp[k[u]] : 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            f += l[u];
            mb = l[u] > mb ? (int32_t)l[u] : mb;
        }
    }
}

// 1024 threads = 64 groups of 16 lanes; a group takes two rows at a time, so
// that the dependent loads (row extent, A columns, B row extents) of both are
// in flight together.  Bound by that latency: at most 512 workgroups (every
// wave slot once, few statistics atomics), no barrier in the loop.
// Runs of 2^run_log2 rows (4 to 64) are dealt out to the workgroups one after
// another, so that long rows that lie side by side go to different ones: 64 rows
// of 50,000 entries among 200,000 of 4, symbolic call 1745 us by runs of 64, 860
// by 16, 645 by 4.  1000 rows of 3000 entries: 355 us on the 16 workgroups that
// their number asks for, 153 on 250 (rowinfo_grid).
constexpr int ROWINFO_RUN = 4;  // the shortest: a wave's rows
__global__ void __launch_bounds__(CLASS_NT) k_rowinfo(Csr A, Csr B, int64_t k_lo, int64_t k_hi, int full_window,
                                                      int run_log2, BinParams bp, RowInfoOut o) {
    constexpr int G = 16, NG = CLASS_NT / G, R = 2, E = 2;  // lanes a row, groups, rows a group, entries a lane
    constexpr int HUBS = 512;
    __shared__ ClassLds<2> c;
    __shared__ int32_t s_hub[HUBS];
    __shared__ int32_t s_nhub;
    __shared__ int64_t s_f[CLASS_NT / SPG_WAVE];
    __shared__ int32_t s_mb[CLASS_NT / SPG_WAVE];
    if (threadIdx.x == 0) s_nhub = 0;
    c.clear(o.order);
    const int g = threadIdx.x / G, gl = threadIdx.x % G, lane = lane_id();
    unsigned long long fmax = 0;
    auto finish = [&](int64_t i, int64_t beg, int64_t end, int64_t f, int32_t mb) {
        finish_row(i, beg, end, f, mb, bp, o, c);
        fmax = (unsigned long long)f > fmax ? (unsigned long long)f : fmax;
    };
    auto window = [&](int64_t& beg, int64_t& end) {
        if (full_window) return;
        // the A row is sorted by column: binary search the window edges
        beg = lower_bound_col(A.col, beg, end, k_lo);
        end = lower_bound_col(A.col, beg, end, k_hi);
    };
    const int64_t step = (int64_t)gridDim.x * NG;
    // the wave's first row of a step, and the group's of the wave's rows
    const int g0 = g & ~(SPG_WAVE / G - 1), gr = g - g0, run = 1 << run_log2;
    const int64_t first = (((int64_t)(g0 >> run_log2) * gridDim.x + blockIdx.x) << run_log2) + (g0 & (run - 1));
    for (int64_t i0 = first; i0 < A.nrows; i0 += R * step) {
        int64_t beg[R], end[R], f[R];
        int32_t mb[R];
        bool active[R];
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const int64_t i = i0 + u * step + gr;
            active[u] = i < A.nrows;
            beg[u] = active[u] ? A.rp[i] : 0;
            end[u] = active[u] ? A.rp[i + 1] : 0;
            f[u] = 0;
            mb[u] = 0;
        }
        uint64_t longs[R];  // the wave's groups with a long row (a bit per lane of them)
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const bool is_long = end[u] - beg[u] > LONG_ROW;
            bool hub = false;
            if (is_long && gl == 0 && end[u] - beg[u] > HUB_ROW) {
                const int slot = atomicAdd(&s_nhub, 1);
                if (slot < HUBS) {  // (past the queue's end: by the wave)
                    s_hub[slot] = (int32_t)(i0 + u * step + gr);
                    hub = true;
                }
            }
            longs[u] = __builtin_amdgcn_ballot_w64(is_long && gl == 0 && !hub);
            if (is_long) active[u] = false;
        }
        int64_t most = 0;
#pragma unroll
        for (int u = 0; u < R; ++u) most = active[u] && end[u] - beg[u] > most ? end[u] - beg[u] : most;
        // the whole row is read and entries outside the window are dropped
        // (two binary searches are a chain of dependent loads)
        int32_t below[R] = {}, inside[R] = {};
        for (int64_t x = gl; x < most; x += G * E) {
            int64_t k[R][E], l0[R][E], l1[R][E];
#pragma unroll
            for (int u = 0; u < R; ++u)
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const int64_t p = beg[u] + x + e * G;
                    k[u][e] = active[u] && p < end[u] ? (int64_t)A.col[p] : -1;
                }
            if (!full_window) {
#pragma unroll
                for (int u = 0; u < R; ++u)
#pragma unroll
                    for (int e = 0; e < E; ++e) {
                        below[u] += k[u][e] >= 0 && k[u][e] < k_lo;
                        if (k[u][e] < k_lo || k[u][e] >= k_hi) k[u][e] = -1;
                        inside[u] += k[u][e] >= 0;
                    }
            }
#pragma unroll
            for (int u = 0; u < R; ++u)
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    l0[u][e] = k[u][e] >= 0 ? B.rp[k[u][e]] : 0;
                    l1[u][e] = k[u][e] >= 0 ? B.rp[k[u][e] + 1] : 0;
                }
#pragma unroll
            for (int u = 0; u < R; ++u)
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const int64_t l = l1[u][e] - l0[u][e];
                    f[u] += l;
                    mb[u] = l > mb[u] ? (int32_t)l : mb[u];
                }
        }
        if (!full_window) {
#pragma unroll
            for (int u = 0; u < R; ++u) {
#pragma unroll
                for (int d = G / 2; d > 0; d >>= 1) {
                    below[u] += lane_xor(below[u], d);
                    inside[u] += lane_xor(inside[u], d);
                }
                if (active[u]) {
                    beg[u] += below[u];
                    end[u] = beg[u] + inside[u];
                }
            }
        }
#pragma unroll
        for (int u = 0; u < R; ++u) {
            // reduce inside the 16-lane group (xor offsets < 16 stay in the group)
#pragma unroll
            for (int d = G / 2; d > 0; d >>= 1) {
                f[u] += lane_xor(f[u], d);
                const int32_t o2 = lane_xor(mb[u], d);
                mb[u] = o2 > mb[u] ? o2 : mb[u];
            }
            if (active[u] && gl == 0) finish(i0 + u * step + gr, beg[u], end[u], f[u], mb[u]);
            for (uint64_t m = longs[u]; m; m &= m - 1) {
                const int l = __builtin_ctzll(m);
                int64_t lb = lane_get(beg[u], l), le = lane_get(end[u], l);
                window(lb, le);
                int64_t lf;
                int32_t lm;
                walk_entries(A, B, lb, le, lane, SPG_WAVE, lf, lm);
                lf = wave_reduce_add(lf);
                lm = wave_reduce_max(lm);
                if (lane == l) finish(i0 + u * step + gr, lb, le, lf, lm);
            }
        }
    }
    __syncthreads();
    const int nhub = s_nhub < HUBS ? s_nhub : HUBS;
    for (int q = 0; q < nhub; ++q) {
        const int64_t i = s_hub[q];
        int64_t lb = A.rp[i], le = A.rp[i + 1];
        window(lb, le);
        int64_t lf;
        int32_t lm;
        walk_entries(A, B, lb, le, threadIdx.x, CLASS_NT, lf, lm);
        lf = wave_reduce_add(lf);
        lm = wave_reduce_max(lm);
        const int w = threadIdx.x / SPG_WAVE;
        if (lane == 0) {
            s_f[w] = lf;
            s_mb[w] = lm;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            int64_t tf = 0;
            int32_t tm = 0;
            for (int x = 0; x < CLASS_NT / SPG_WAVE; ++x) {
                tf += s_f[x];
                tm = s_mb[x] > tm ? s_mb[x] : tm;
            }
            finish(i, lb, le, tf, tm);
        }
        __syncthreads();
    }
    fmax = wave_reduce_max(fmax);
    if (lane == 0 && fmax) atomicMax(&c.fmax, fmax);
    c.flush(o.order, o.bin_stats, o.max_flops);
}

// Numeric classification from exact counts, and the sums of the counts per
// tile of CLASS_NT rows for the scan that follows (k_scan_scatter).  cnt[i] =
// outputs of row i.  A bitmap row keeps its rank paths only if the symbolic
// pass saved its bitmap (heavy_idx >= 0; NULL = no bitmaps saved).
__global__ void __launch_bounds__(CLASS_NT) k_num_classify(int64_t m, const int64_t* cnt, const int64_t* a_beg,
                                                           const int64_t* a_end, const int64_t* flops, BinParams bp,
                                                           const int32_t* heavy_idx, uint8_t* bin, int64_t* bin_stats,
                                                           OrderedBins order, int64_t* tile_sums) {
    __shared__ ClassLds<3> c;
    __shared__ int64_t red[CLASS_NT / SPG_WAVE + 1];
    c.clear(order);
    for (int64_t t0 = (int64_t)blockIdx.x * CLASS_NT; t0 < m; t0 += (int64_t)gridDim.x * CLASS_NT) {
        const int64_t i = t0 + threadIdx.x;
        int64_t n = 0;
        if (i < m) {
            n = cnt[i];
            const int64_t an = a_end[i] - a_beg[i];
            const int64_t f = flops[i];
            const bool saved = bin[i] == BIN_DENSE && heavy_idx && heavy_idx[i] >= 0;
            const int b = num_bin(f, an, n, saved, bp);
            bin[i] = (uint8_t)b;
            atomicAdd(&c.rows[b], 1);
            atomicAdd(&c.v[0][b], (unsigned long long)f);
            atomicAdd(&c.v[1][b], (unsigned long long)an);
            atomicAdd(&c.v[2][b], (unsigned long long)n);
            if (order.has(b)) atomicAdd(&c.lpt[order.key(b, f)], 1);
        }
        int64_t total;
        (void)block_exclusive_scan<CLASS_NT, int64_t>(n, &total, red);
        if (threadIdx.x == 0) tile_sums[t0 / CLASS_NT] = total;
    }
    c.flush(order, bin_stats, nullptr);
}

// Counting-sort scatter of a tile's rows (one per thread, b < 0: none) into
// per-bin lists: the list of bin b starts at the sum of the counts of the bins
// below it (counts[0..NBINS)); a run of ordered bins is placed by its keys.
// cursor[NBINS + order.keys()] must be zero before the first tile.
struct ScatterLds {
    int32_t cnt[NBINS + LPT_KEYS * LPT_MAX_BINS];
    int32_t base[NBINS + LPT_KEYS * LPT_MAX_BINS];
    int32_t red[CLASS_NT / SPG_WAVE + 1];
};
__device__ inline void scatter_tile(int64_t i, int b, const int64_t* counts, const OrderedBins& order, int32_t* cursor,
                                    int32_t* lists, ScatterLds& S) {
    const int nk = order.keys();
    for (int k = threadIdx.x; k < NBINS + nk; k += CLASS_NT) S.cnt[k] = 0;
    if (threadIdx.x < NBINS) {
        int64_t off = 0;
        for (int x = 0; x < (int)threadIdx.x; ++x) off += counts[x];
        S.base[threadIdx.x] = (int32_t)off;
    }
    __syncthreads();
    if (nk > 0) {  // starts of the keys: a scan of their counts from the run's first bin
        constexpr int PER = (LPT_KEYS * LPT_MAX_BINS + CLASS_NT - 1) / CLASS_NT;
        int32_t h[PER], part = 0;
#pragma unroll
        for (int x = 0; x < PER; ++x) {
            const int k = threadIdx.x * PER + x;
            h[x] = k < nk ? order.hist[k] : 0;
            part += h[x];
        }
        int32_t total;
        int32_t run = block_exclusive_scan<CLASS_NT, int32_t>(part, &total, S.red) + S.base[order.b_lo];
#pragma unroll
        for (int x = 0; x < PER; ++x) {
            const int k = threadIdx.x * PER + x;
            if (k < nk) S.base[NBINS + k] = run;
            run += h[x];
        }
    }
    int key = 0, local = 0;
    if (b >= 0) {
        key = order.has(b) ? NBINS + order.key(b, order.work[i]) : b;
        local = atomicAdd(&S.cnt[key], 1);
    }
    __syncthreads();
    for (int k = threadIdx.x; k < NBINS + nk; k += CLASS_NT)
        if (S.cnt[k]) S.base[k] += atomicAdd(&cursor[k], S.cnt[k]);
    __syncthreads();
    if (b >= 0) lists[S.base[key] + local] = (int32_t)i;
}

// host (optional, pinned): receives words of the statistics
__global__ void __launch_bounds__(CLASS_NT) k_bin_scatter(int64_t m, const uint8_t* bin, const int64_t* counts,
                                                          OrderedBins order, int32_t* cursor, int32_t* lists,
                                                          const int64_t* stats, int32_t words, int64_t* host) {
    __shared__ ScatterLds S;
    if (host && blockIdx.x == 0)
        for (int t = threadIdx.x; t < words; t += CLASS_NT)
            __hip_atomic_store(&host[t], stats[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    const int64_t i = (int64_t)blockIdx.x * CLASS_NT + threadIdx.x;
    scatter_tile(i, i < m ? (int)bin[i] : -1, counts, order, cursor, lists, S);
}

// Row pointers and bin lists after k_num_classify, one tile per workgroup:
// rp[0] = 0, rp[i + 1] = inclusive sum of the counts, in place (rp[i + 1] holds
// row i's count; each workgroup sums the tiles before its own itself), and
// the tile's rows into the lists.  host (optional, pinned): receives words of
// the statistics, then nnz(C).
__global__ void __launch_bounds__(CLASS_NT) k_scan_scatter(int64_t m, int64_t* rp, const int64_t* tile_sums,
                                                           const uint8_t* bin, const int64_t* counts, OrderedBins order,
                                                           int32_t* cursor, int32_t* lists, const int64_t* stats,
                                                           int32_t words, int64_t* host) {
    __shared__ ScatterLds S;
    __shared__ int64_t red[CLASS_NT / SPG_WAVE + 1];
    const int64_t i = (int64_t)blockIdx.x * CLASS_NT + threadIdx.x;
    int64_t before = 0;
    for (int64_t t = threadIdx.x; t < (int64_t)blockIdx.x; t += CLASS_NT) before += tile_sums[t];
    const int64_t n = i < m ? rp[i + 1] : 0;
    int64_t base, total;
    (void)block_exclusive_scan<CLASS_NT, int64_t>(before, &base, red);
    const int64_t pre = block_exclusive_scan<CLASS_NT, int64_t>(n, &total, red);
    if (i < m) rp[i + 1] = base + pre + n;
    if (i == 0) rp[0] = 0;
    if (host) {
        if (blockIdx.x == 0)
            for (int t = threadIdx.x; t < words; t += CLASS_NT)
                __hip_atomic_store(&host[t], stats[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        if (i == m - 1) __hip_atomic_store(&host[words], base + pre + n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    scatter_tile(i, i < m ? (int)bin[i] : -1, counts, order, cursor, lists, S);
}

}  // namespace spg
