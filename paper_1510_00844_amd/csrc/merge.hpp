// Multiway merge with reduction (Section 4.3; LocalMerge of Algorithm 2):
// out = entry-wise semiring sum of c layers of equal shape.  Row i of the
// output is the sorted union of the c sorted segments layer_l(i,:), with
// values of equal columns combined in ascending layer order.  The paper
// merges with a heap per thread over a split of the column range; here:
//   SORT   (merge_sorts) rows of 65 ... MS_LMAX entries whose columns
//          span less than RS_SPAN_MAX: one wave per row sorts the entries
//          by column and layer (rowsort.hpp) and folds equal columns in
//          ascending layer order
//   WAVE   rows of at most KW_LMAX entries over at most 8 layers: one
//          wave per row, the column range split over the 64 lanes and each
//          lane merging its range of the c segments (kway.hpp), staged in LDS
//   SMALL  (merge_sorts) rows of <= 64 entries: a wave sort of
//          (column, position)
//   RANK   65 ... 4096 entries: a workgroup places each entry by binary
//          searches in the other layers' segments, staged in LDS
//   DENSE  longer rows: a workgroup sweeping column chunks with an LDS dense
//          accumulator, each layer's chunk range found by binary search (the
//          column-range split of Section 4.3)
#pragma once
#include "kway.hpp"
#include "rowsort.hpp"
#include "products.hpp"
#include "rowinfo.hpp"

namespace spg {

struct LayerDesc {
    const int64_t* rp;
    const int32_t* col;
    const void* val;
};

constexpr int MERGE_MAX_LAYERS = 64;

// The layers, passed by value as a kernel argument (no device copy).
struct LayerSet {
    LayerDesc d[MERGE_MAX_LAYERS];
};

// merge bins by total row length L over the layers
constexpr int MBIN_EMPTY = 0, MBIN_WAVE = 1, MBIN_SMALL = 2, MBIN_R256 = 3, MBIN_R1K = 4, MBIN_R4K = 5,
              MBIN_DENSE = 6, MBIN_SORT = 7;
constexpr int MBINS = 8;

// the SORT bin's rows
constexpr int MS_LMAX = RS_MAX;
constexpr int64_t MS_SPAN_MAX = RS_SPAN_MAX;
constexpr int MERGE_LDS_MAX = 4096;

// layers the wave k-way merge takes (it costs O(c) instructions per output)
constexpr int MERGE_KWAY_MAX_LAYERS = 8;

// Whether rows are sorted: rows of up to 64 entries by the register sort, longer
// ones whose columns pack (see RS_SPAN_MAX) by the row sort.  Never up to four
// layers, always above eight.  The cost of the k-way sweep grows with the layers
// (ER scale 18, 256 entries a row, count and fill, swept / sorted: two layers 0.93
// / 0.86 ms, four 1.01 / 0.87, eight 1.52 / 0.89).  Up to four, what the sort gains
// on many uniform rows it loses on few of them (ER scale 14, four layers: 141 / 161
// us) and on rows of mixed lengths (SSCA scale 11 162 / 193, scale 15 761 / 781),
// where it needs bins of its own.  From five to eight the two bins also need
// enough rows to hide their latency and their launches; eight layers, swept /
// sorted: 256 entries a row (ER) 8192 rows 144 / 154 us, 16384 187 / 177, 32768
// 268 / 219; 16 a row 4096 rows 71 / 74, 8192 80 / 77, 16384 97 / 84; and where
// the mean row is longer than the sweep takes (SSCA, G500), few rows are sorted at
// all: 2048 rows 269 / 300, 16384 526 / 544, 65536 2602 / 2597.
inline bool merge_sorts(int32_t c, int64_t m, int64_t entries) {
    if (c <= 4 || c > MERGE_KWAY_MAX_LAYERS) return c > 4;
    if (entries > KW_LMAX * m) return false;
    return m >= (entries <= SPG_WAVE * m ? 1 << 13 : 1 << 14);
}

__device__ inline int merge_bin(int64_t L, int c, bool sorts) {
    if (L == 0) return MBIN_EMPTY;
    if (L <= SPG_WAVE && sorts) return MBIN_SMALL;
    if (L <= KW_LMAX && c <= MERGE_KWAY_MAX_LAYERS) return MBIN_WAVE;
    if (L <= 256) return MBIN_R256;
    if (L <= 1024) return MBIN_R1K;
    if (L <= MERGE_LDS_MAX) return MBIN_R4K;
    return MBIN_DENSE;
}

// packs: every span of the n columns packs (n <= MS_SPAN_MAX), so no column is
// read (the two ends of every segment were most of this kernel's time: 67 -> 28
// us for 16 layers of 262,144 rows).
__global__ void __launch_bounds__(256) k_merge_rowinfo(int64_t m, int32_t c, LayerSet layers, int sorts, int packs,
                                                       int64_t* total_len, uint8_t* bin,
                                                       int64_t* bin_stats) {
    __shared__ int s_hist[NBINS];
    __shared__ int64_t s_len[NBINS];
    if (threadIdx.x < NBINS) {
        s_hist[threadIdx.x] = 0;
        s_len[threadIdx.x] = 0;
    }
    __syncthreads();
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < m; i += (int64_t)gridDim.x * 256) {
        int64_t L = 0;
        for (int l = 0; l < c; ++l) L += layers.d[l].rp[i + 1] - layers.d[l].rp[i];
        total_len[i] = L;
        int b = merge_bin(L, c, sorts != 0);
        if (sorts && L > SPG_WAVE && L <= MS_LMAX) {  // the bucket sort, if the columns pack
            int32_t mn = packs ? 0 : 0x7fffffff, mx = packs ? 0 : -1;
            for (int l = 0; l < c && !packs; ++l) {
                const int64_t rs = layers.d[l].rp[i], re = layers.d[l].rp[i + 1];
                if (re > rs) {
                    const int32_t a = layers.d[l].col[rs], z = layers.d[l].col[re - 1];
                    mn = a < mn ? a : mn;
                    mx = z > mx ? z : mx;
                }
            }
            if ((int64_t)mx - mn < MS_SPAN_MAX) b = MBIN_SORT;
        }
        bin[i] = (uint8_t)b;
        atomicAdd(&s_hist[b], 1);
        atomicAdd((unsigned long long*)&s_len[b], (unsigned long long)L);
    }
    __syncthreads();
    if (threadIdx.x < NBINS && s_hist[threadIdx.x]) {
        atomicAdd((unsigned long long*)&bin_stats[threadIdx.x], (unsigned long long)s_hist[threadIdx.x]);
        atomicAdd((unsigned long long*)&bin_stats[NBINS + threadIdx.x], (unsigned long long)s_len[threadIdx.x]);
    }
}

// One wave per row (4 per workgroup), the rows of the bin located on the
// device.  cnt != nullptr: count pass; otherwise fill pass at out_rp.
template <int SR, int KMAX, bool FILL>
__global__ void __launch_bounds__(256) k_merge_kway(int32_t c, LayerSet layers, BinRef ref, int64_t* cnt,
                                                    const int64_t* out_rp, int32_t* out_col, void* out_val) {
    typedef typename Sr<SR>::acc_t V;
    __shared__ KwLds<V, FILL> lds[4];
    KwLds<V, FILL>& W = lds[threadIdx.x >> 6];
    const int32_t* rows;
    int64_t n;
    ref.locate(rows, n);
    const int lane = lane_id();
    for (int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); r < n; r += (int64_t)gridDim.x * 4) {
        const int64_t i = rows[r];
        KwList<V> lst{nullptr, nullptr, 0, 0, Sr<SR>::zero()};
        if (lane < c) {
            const int64_t rs = layers.d[lane].rp[i];
            lst.colp = layers.d[lane].col;
            lst.valp = layers.d[lane].val;
            lst.start = rs;
            lst.len = (int32_t)(layers.d[lane].rp[i + 1] - rs);
        }
        const int32_t L = wave_reduce_add(lst.len);
        const int32_t got = kway_merge_wave<SR, KMAX, FILL, false>(lst, c, L, W, out_col, out_val,
                                                                   FILL ? out_rp[i] : 0);
        if (!FILL && lane == 0) cnt[i] = got;
        wave_lds_sync();  // the staged row is read before the next one overwrites it
    }
}

// The flat order of a merge row (layer 0's segment, then layer 1's, ...) over
// a wave: lane l < c holds layer l's segment; entry x of the flat order lies in
// the last non-empty layer that starts at or before it.
struct MergeRow {
    int32_t off;          // first entry of the lane's layer
    int32_t L;            // entries (wave-uniform)
    const int32_t* colp;  // entry x of the layer: colp[x], valp[x]
    int64_t rel;          // ... = arrays of the layer at rel + x
    const void* valp;
};
__device__ inline MergeRow merge_row(const LayerSet& layers, int32_t c, int64_t i) {
    const int lane = lane_id();
    MergeRow m{0, 0, nullptr, 0, nullptr};
    int64_t rs = 0;
    int32_t len = 0;
    if (lane < c) {
        rs = layers.d[lane].rp[i];
        len = (int32_t)(layers.d[lane].rp[i + 1] - rs);
        m.colp = layers.d[lane].col;
        m.valp = layers.d[lane].val;
    }
    const int32_t incl = wave_inclusive_scan_add(len);
    m.off = len > 0 ? incl - len : -1;  // (empty layers own no entry)
    m.L = __builtin_amdgcn_readlane(incl, SPG_WAVE - 1);
    m.rel = rs - (incl - len);
    if (m.colp) m.colp += m.rel;
    return m;
}
// Layer of entry x = u * 64 + lane of each step: the lane of every non-empty
// layer is marked (a byte; NU * 64 of them in the wave's LDS) at its first
// entry, and a running maximum of the marks gives each entry its layer (a
// search over the layers took log2(c) lane exchanges a step).
template <int NU>
__device__ inline void merge_layers_of(const MergeRow& m, uint8_t* marks, int32_t (&l)[NU]) {
    const int lane = lane_id();
#pragma unroll
    for (int t = 0; t < NU / 4; ++t)
        if (t * 4 * SPG_WAVE < m.L) reinterpret_cast<uint32_t*>(marks)[t * SPG_WAVE + lane] = 0;
    wave_lds_sync();
    if (m.off >= 0) marks[m.off] = (uint8_t)lane;
    wave_lds_sync();
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        if (u * SPG_WAVE >= m.L) break;
        l[u] = marks[u * SPG_WAVE + lane];
    }
    int32_t carry = 0;
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        if (u * SPG_WAVE >= m.L) break;
        const int32_t x = wave_inclusive_scan_max(l[u]);
        l[u] = x > carry ? x : carry;
        carry = __builtin_amdgcn_readlane(l[u], SPG_WAVE - 1);
    }
    wave_lds_sync();  // the marks are read before their bytes are used again
}

// Count pass of the WAVE and SORT bins (rows of at most MS_LMAX entries):
// counting needs no order, so the row's columns are inserted into an LDS
// hash set of MC_SLOTS slots (at most half full), one wave per row, and
// each new column counts once.  Every lane then clears the slots it
// filled, so the set is empty again for the wave's next row.
constexpr int MC_LOG2 = 10;
constexpr int MC_SLOTS = 1 << MC_LOG2;
static_assert(MC_SLOTS >= 2 * MS_LMAX && MS_LMAX >= KW_LMAX, "the hash count takes both bins' rows");

__global__ void __launch_bounds__(256) k_merge_count_hash(int32_t c, LayerSet layers, BinRef ref, int64_t* cnt) {
    constexpr int NU = MS_LMAX / SPG_WAVE;
    __shared__ int32_t tab[4][MC_SLOTS];
    __shared__ __align__(4) uint8_t marks[4][MS_LMAX];
    int32_t* T = tab[threadIdx.x >> 6];
    const int lane = lane_id();
    for (int t = lane; t < MC_SLOTS; t += SPG_WAVE) T[t] = -1;
    wave_lds_sync();
    const int32_t* rows;
    int64_t n;
    ref.locate(rows, n);
    for (int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); r < n; r += (int64_t)gridDim.x * 4) {
        const int64_t i = rows[r];
        const MergeRow m = merge_row(layers, c, i);
        const int32_t L = m.L;
        int32_t l[NU], col[NU], used[NU];
        merge_layers_of<NU>(m, marks[threadIdx.x >> 6], l);
        int32_t mine = 0;
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            used[u] = -1;
            if (u * SPG_WAVE >= L) break;
            const int32_t x = u * SPG_WAVE + lane;
            const int32_t* cp = (const int32_t*)(intptr_t)lane_get((int64_t)(intptr_t)m.colp, l[u]);
            col[u] = cp[x < L ? x : L - 1];
        }
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            if (u * SPG_WAVE >= L) break;
            pin(col[u]);
            if (u * SPG_WAVE + lane < L) {
                uint32_t h = hash_slot(col[u], MC_LOG2);
                while (true) {  // ends: the set is at most half full
                    const int32_t old = atomicCAS(&T[h], -1, col[u]);
                    if (old == -1) {
                        ++mine;
                        used[u] = (int32_t)h;
                        break;
                    }
                    if (old == col[u]) break;
                    h = (h + 1) & (MC_SLOTS - 1);
                }
            }
        }
        const int32_t tot = wave_reduce_add(mine);
        if (lane == 0) cnt[i] = tot;
        wave_lds_sync();  // every insertion is done before the set is cleared
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            if (u * SPG_WAVE >= L) break;
            if (used[u] >= 0) T[used[u]] = -1;
        }
        wave_lds_sync();
    }
}

// One wave per row of the SORT bin (4 per workgroup): the row's entries in the
// flat order (equal columns in ascending layer order), sorted and folded by
// rowsort.hpp, its columns and values four steps in flight.  Bound by latency
// at 5 waves per SIMD: the register limit of launch bounds (96 instead of 108,
// no spill) took the 16-layer merge from 1.17 to 1.06 ms, where 80 registers
// spilled and took 1.12; now 0.95 (16 layers of 262,144 rows: this kernel 519 us,
// 550 VALU instructions a row).
template <int SR>
__global__ void __launch_bounds__(256, 5) k_merge_sort(int32_t c, LayerSet layers, BinRef ref, const int64_t* out_rp,
                                                    int32_t* out_col, void* out_val) {
    typedef Sr<SR> S;
    typedef typename S::acc_t V;
    constexpr int NU = MS_LMAX / SPG_WAVE;
    __shared__ RowSortLds<V, NU> lds[4];
    RowSortLds<V, NU>& W = lds[threadIdx.x >> 6];
    const int32_t* rows;
    int64_t n;
    ref.locate(rows, n);
    const int lane = lane_id();
    for (int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); r < n; r += (int64_t)gridDim.x * 4) {
        const int64_t i = rows[r];
        const MergeRow m = merge_row(layers, c, i);
        const int32_t L = m.L;
        const int64_t o = out_rp[i];
        const int32_t room = (int32_t)(out_rp[i + 1] - o);
        int32_t l[NU], col[NU];
        merge_layers_of<NU>(m, reinterpret_cast<uint8_t*>(W.key), l);
        W.bcnt[lane] = 0;
        constexpr int U = 4;
#pragma unroll
        for (int u0 = 0; u0 < NU; u0 += U) {
            if (u0 * SPG_WAVE >= L) break;
            V v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if ((u0 + u) * SPG_WAVE >= L) break;
                const int32_t x = (u0 + u) * SPG_WAVE + lane;
                const int32_t y = x < L ? x : L - 1;
                const int32_t* cp = (const int32_t*)(intptr_t)lane_get((int64_t)(intptr_t)m.colp, l[u0 + u]);
                const void* vp = (const void*)(intptr_t)lane_get((int64_t)(intptr_t)m.valp, l[u0 + u]);
                // (taken by every lane: boolean layers may have no value array, and
                // an exchange inside that test would read lanes that it switches off)
                const int64_t q = lane_get(m.rel, l[u0 + u]) + y;
                col[u0 + u] = cp[y];
                v[u] = S::load(vp, q);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if ((u0 + u) * SPG_WAVE >= L) break;
                pin(col[u0 + u]);
                pin(v[u]);
                const int32_t x = (u0 + u) * SPG_WAVE + lane;
                if (x < L) W.val[x] = v[u];
            }
        }
        int32_t cmin = 0x7fffffff, cmax = -1;
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            if (u * SPG_WAVE >= L) break;
            cmin = col[u] < cmin ? col[u] : cmin;
            cmax = col[u] > cmax ? col[u] : cmax;
        }
        cmin = __builtin_amdgcn_readfirstlane(wave_all(cmin, [](int32_t x, int32_t y) { return x < y ? x : y; }));
        cmax = __builtin_amdgcn_readfirstlane(wave_all(cmax, [](int32_t x, int32_t y) { return x > y ? x : y; }));
        wave_lds_sync();
        wave_sort_row(W, L, cmin, cmax, col, nullptr);
        (void)wave_fold_row<SR, NU>(W, L, cmin, out_col, out_val, o, room);
        wave_lds_sync();  // the row's LDS is read before the next row overwrites it
    }
}

// cnt != nullptr: count pass; otherwise fill pass into out_rp/out_col/out_val.
template <int SR>
__global__ void __launch_bounds__(256) k_merge_small(int32_t c, LayerSet layers_, BinRef ref, int64_t* cnt,
                                                     const int64_t* out_rp, int32_t* out_col,
                                                     void* out_val) {
    typedef Sr<SR> S;
    typedef typename S::acc_t V;
    const LayerDesc* layers = layers_.d;
    const int32_t* rows;
    int64_t nrows;
    ref.locate(rows, nrows);
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    for (int64_t r = (int64_t)blockIdx.x * 4 + wv; r < nrows; r += (int64_t)gridDim.x * 4) {
    const int64_t i = rows[r];
    const int lane = lane_id();
    int pos = 0, my_l = -1;
    int64_t my_q = 0;
    for (int l = 0; l < c; ++l) {
        const int64_t rs = layers[l].rp[i];
        const int len = (int)(layers[l].rp[i + 1] - rs);
        if (lane >= pos && lane < pos + len) {
            my_l = l;
            my_q = rs + (lane - pos);
        }
        pos += len;
    }
    uint64_t key = ~0ull;
    V v = S::zero();
    if (my_l >= 0) {
        key = ((uint64_t)(uint32_t)layers[my_l].col[my_q] << 6) | (uint64_t)lane;
        if (!cnt) v = S::load(layers[my_l].val, my_q);
    }
    key = wave_bitonic_sort_u64(key);
    const uint32_t col = (uint32_t)(key >> 6);
    v = __shfl(v, (int)(key & 63), SPG_WAVE);
    const uint64_t heads = wave_fold_sorted<SR>(col, v, pos);
    if (cnt) {
        if (lane == 0) cnt[i] = __popcll(heads);
        continue;
    }
    if ((heads >> lane) & 1) {
        const int64_t o = out_rp[i] + lanes_below(heads);
        out_col[o] = (int32_t)col;
        if (out_val) S::store(out_val, o, v);
    }
    }
}

// first index in [lo, hi) of the sorted s with s[idx] >= x (lower) or > x (upper)
__device__ inline int seg_lower(const int32_t* s, int lo, int hi, int32_t x) {
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (s[mid] < x) lo = mid + 1; else hi = mid;
    }
    return lo;
}
__device__ inline int seg_upper(const int32_t* s, int lo, int hi, int32_t x) {
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (s[mid] <= x) lo = mid + 1; else hi = mid;
    }
    return lo;
}
// layer of staged entry x: largest l < c with soff[l] <= x
__device__ inline int layer_of(const int32_t* soff, int c, int x) {
    int lo = 0, hi = c;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (soff[mid] <= x) lo = mid; else hi = mid;
    }
    return lo;
}

// One workgroup per row of 65..cap entries.  The row's c segments are
// staged back to back in LDS (scol).  Count pass: an entry opens a new
// column unless an earlier layer holds the same column.  Fill pass: the
// entry's place in the merged order is its index in its own segment plus,
// for every other layer, the entries of that layer with smaller columns
// (and, for earlier layers, equal ones), so equal columns end up adjacent in
// ascending layer order; the runs are then folded left to right.
// Dynamic LDS: cap values (fill pass), cap staged columns, cap merged
// columns (fill pass).
template <int SR, int NT>
__global__ void __launch_bounds__(NT) k_merge_rank(int32_t c, LayerSet layers_, BinRef ref,
                                                   const int64_t* total_len, int32_t cap, int64_t* cnt,
                                                   const int64_t* out_rp, int32_t* out_col, void* out_val) {
    typedef Sr<SR> S;
    typedef typename S::acc_t V;
    const LayerDesc* layers = layers_.d;
    extern __shared__ uint64_t dyn[];
    V* mval = reinterpret_cast<V*>(dyn);
    int32_t* scol = cnt ? reinterpret_cast<int32_t*>(dyn) : reinterpret_cast<int32_t*>(mval + cap);
    int32_t* mcol = scol + cap;
    __shared__ int32_t soff[MERGE_MAX_LAYERS + 1];
    __shared__ int64_t srs[MERGE_MAX_LAYERS];
    __shared__ int32_t red[NT / SPG_WAVE + 1];
    for_each_bin_row(ref, [&](int64_t, int64_t i) {
    const int L = (int)total_len[i];
    if (threadIdx.x < SPG_WAVE) {  // c <= 64 segment lengths, scanned by one wave
        const int l = threadIdx.x;
        int len = 0;
        if (l < c) {
            const int64_t rs = layers[l].rp[i];
            len = (int)(layers[l].rp[i + 1] - rs);
            srs[l] = rs;
        }
        const int incl = wave_inclusive_scan_add(len);
        if (l < c) soff[l + 1] = incl;
        if (l == 0) soff[0] = 0;
    }
    __syncthreads();
    for (int x = threadIdx.x; x < L; x += NT) {
        const int l = layer_of(soff, c, x);
        scol[x] = layers[l].col[srs[l] + (x - soff[l])];
    }
    __syncthreads();
    if (cnt) {
        int32_t mine = 0;
        for (int x = threadIdx.x; x < L; x += NT) {
            const int l = layer_of(soff, c, x);
            const int32_t col = scol[x];
            bool fresh = true;
            for (int l2 = 0; l2 < l && fresh; ++l2) {
                const int q = seg_lower(scol, soff[l2], soff[l2 + 1], col);
                fresh = !(q < soff[l2 + 1] && scol[q] == col);
            }
            mine += fresh ? 1 : 0;
        }
        const int32_t tot = block_reduce_add<NT, int32_t>(mine, red);
        if (threadIdx.x == 0) cnt[i] = tot;
        return;
    }
    for (int x = threadIdx.x; x < L; x += NT) {
        const int l = layer_of(soff, c, x);
        const int32_t col = scol[x];
        int pos = x - soff[l];
        for (int l2 = 0; l2 < c; ++l2) {
            if (l2 == l) continue;
            const int lo = soff[l2], hi = soff[l2 + 1];
            pos += (l2 < l ? seg_upper(scol, lo, hi, col) : seg_lower(scol, lo, hi, col)) - lo;
        }
        mcol[pos] = col;
        if (out_val) mval[pos] = S::load(layers[l].val, srs[l] + (x - soff[l]));
    }
    __syncthreads();
    // heads over a contiguous range of merged positions per thread
    const int per = (L + NT - 1) / NT;
    const int q0 = threadIdx.x * per;
    const int q1 = q0 + per < L ? q0 + per : L;
    int32_t mine = 0;
    for (int q = q0; q < q1; ++q) mine += (q == 0 || mcol[q - 1] != mcol[q]) ? 1 : 0;
    int32_t total;
    int32_t rank = block_exclusive_scan<NT, int32_t>(mine, &total, red);
    const int64_t o = out_rp[i];
    for (int q = q0; q < q1; ++q) {
        if (q == 0 || mcol[q - 1] != mcol[q]) {
            const int32_t col = mcol[q];
            out_col[o + rank] = col;
            if (out_val) {
                V acc = mval[q];
                for (int y = q + 1; y < L && mcol[y] == col; ++y) acc = S::add(acc, mval[y]);
                S::store(out_val, o + rank, acc);
            }
            ++rank;
        }
    }
    });
}

// Rows above the rank path: a workgroup sweeps column chunks of W; within a
// chunk the layers are added one after the other (a layer holds a column
// at most once, so its entries go to distinct accumulators without atomics,
// and a barrier orders the layers), so equal columns combine in ascending
// layer order.  Each layer's chunk range is found by binary search (the
// column-range split of Section 4.3).
template <int SR, int NT, int W>
__global__ void __launch_bounds__(NT) k_merge_dense(int32_t c, LayerSet layers_, BinRef ref, int64_t ncols, int64_t* cnt,
                                                    const int64_t* out_rp, int32_t* out_col,
                                                    void* out_val) {
    typedef Sr<SR> S;
    typedef typename S::acc_t V;
    constexpr int NWD = W / 32;
    const LayerDesc* layers = layers_.d;
    __shared__ V acc[W];
    __shared__ uint32_t bits[NWD];
    __shared__ int32_t wpre[NWD];
    __shared__ int64_t s_lo[MERGE_MAX_LAYERS], s_hi[MERGE_MAX_LAYERS];
    __shared__ int32_t red[NT / SPG_WAVE + 1];
    const int P = (int)((ncols + W - 1) / W);
    for_each_bin_row(ref, [&](int64_t, int64_t i) {
    int64_t off = cnt ? 0 : out_rp[i];
    int64_t count = 0;
    for (int ch = 0; ch < P; ++ch) {
        for (int t = threadIdx.x; t < W; t += NT) acc[t] = S::zero();
        for (int t = threadIdx.x; t < NWD; t += NT) bits[t] = 0u;
        const int64_t cbase = (int64_t)ch * W;
        if (threadIdx.x < c) {  // each layer's entries inside the chunk
            const int l = threadIdx.x;
            const int64_t rs = layers[l].rp[i], re = layers[l].rp[i + 1];
            const int64_t lo = lower_bound_col(layers[l].col, rs, re, cbase);
            s_lo[l] = lo;
            s_hi[l] = lower_bound_col(layers[l].col, lo, re, cbase + W);
        }
        __syncthreads();
        for (int l = 0; l < c; ++l) {
            for (int64_t q = s_lo[l] + threadIdx.x; q < s_hi[l]; q += NT) {
                const int32_t j = (int32_t)(layers[l].col[q] - cbase);
                const uint32_t b = 1u << (j & 31);
                if (!cnt) {
                    const V v = S::load(layers[l].val, q);
                    acc[j] = (bits[j >> 5] & b) ? S::add(acc[j], v) : v;
                }
                atomicOr(&bits[j >> 5], b);
            }
            __syncthreads();  // layer l complete before layer l + 1
        }
        constexpr int WPT = (NWD + NT - 1) / NT;
        int32_t wc[WPT];
        int32_t sum = 0;
#pragma unroll
        for (int x = 0; x < WPT; ++x) {
            int w = threadIdx.x * WPT + x;
            wc[x] = w < NWD ? __popc(bits[w]) : 0;
            sum += wc[x];
        }
        int32_t chunk_total;
        int32_t pre = block_exclusive_scan<NT, int32_t>(sum, &chunk_total, red);
#pragma unroll
        for (int x = 0; x < WPT; ++x) {
            int w = threadIdx.x * WPT + x;
            if (w < NWD) wpre[w] = pre;
            pre += wc[x];
        }
        __syncthreads();
        if (!cnt && chunk_total) {
            for (int j = threadIdx.x; j < W; j += NT) {
                const uint32_t wbits = bits[j >> 5];
                const uint32_t b = 1u << (j & 31);
                if (wbits & b) {
                    const int64_t o = off + wpre[j >> 5] + __popc(wbits & (b - 1));
                    out_col[o] = (int32_t)(cbase + j);
                    if (out_val) S::store(out_val, o, acc[j]);
                }
            }
        }
        off += chunk_total;
        count += chunk_total;
        __syncthreads();
    }
    if (cnt && threadIdx.x == 0) cnt[i] = count;
    });
}

}  // namespace spg
