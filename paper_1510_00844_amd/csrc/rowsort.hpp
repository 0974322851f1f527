// One row's (column, value) entries sorted and folded by one wave, without a
// hash table: the accumulator of product rows of up to 512 products and of
// merge rows of up to 512 entries.
//
// Entry x of the row (its position in the order equal columns are added in:
// ascending k for a product, ascending layer for a merge) lies in LDS as a
// column and a value.  It becomes the key (column - cmin) << RS_XBITS | x; the
// keys are counted into 64 buckets of equal column width (bucket = (column -
// cmin) * 64 / span in FP32, monotone), placed bucket by bucket, and every
// lane sorts its own bucket in registers with a sorting network.  Columns in
// clusters overflow the networks; product rows of a span that a bitmap in the
// keys' place can hold then take buckets of equal numbers of columns, the others
// a bitonic sort of the whole row.  12 runs of 32 neighbouring columns a row, in
// a window of 12,000 (262,144 rows): numeric kernel 1867 us by the whole-row
// sort, 961 by the ranks, 896 hashed, where the hash table orders its outputs by
// such a bitmap too; in 190,000 (131,072 rows): 907 by the whole-row sort, 3117
// hashed.  Equal columns are then neighbours in ascending x, so the fold adds them
// in that order, and the output positions are counted by ballots: consecutive
// lanes write consecutive outputs.
//
// Bound by instruction issue (a few hundred VALU instructions a row), so
// everything is done per entry of the row, not per slot of a table: a row of
// 256 entries is four steps, where the 512-slot table it took before cost eight
// to clear, eight to compact and a probe loop per product (ER scale 18, 210K
// rows of 270 products: 1248 -> 609 VALU instructions a row, 598 -> 427 us, now
// at 6.3 TB/s past L2: the lines of the short B rows are used in part).
#pragma once
#include "common.hpp"

namespace spg {

constexpr int RS_XBITS = 9;
constexpr int RS_MAX = 1 << RS_XBITS;                  // entries of a row
constexpr int64_t RS_SPAN_MAX = 1ll << (32 - RS_XBITS);  // columns it may span
constexpr int RS_PAD = 16;                             // keys a network may read past the row

template <typename V, int NU>
struct RowSortLds {
    uint32_t key[NU * SPG_WAVE + RS_PAD];
    V val[NU * SPG_WAVE];
    int32_t bcnt[SPG_WAVE];
};

// Batcher's odd-even merge sort of a[0, N) ascending (every comparator leaves
// the smaller key at the lower index, so N need not be a power of two).
template <int N>
__device__ inline void sort_network(uint32_t (&a)[N]) {
#pragma unroll
    for (int p = 1; p < N; p *= 2)
#pragma unroll
        for (int k = p; k >= 1; k /= 2)
#pragma unroll
            for (int j = k % p; j + k < N; j += 2 * k)
#pragma unroll
                for (int i = 0; i < k; ++i)
                    if (i + j + k < N && (i + j) / (2 * p) == (i + j + k) / (2 * p)) {
                        const uint32_t lo = a[i + j] < a[i + j + k] ? a[i + j] : a[i + j + k];
                        const uint32_t hi = a[i + j] < a[i + j + k] ? a[i + j + k] : a[i + j];
                        a[i + j] = lo;
                        a[i + j + k] = hi;
                    }
}

// Sorts the calling lane's bucket keys[off, off + n), n <= N <= RS_PAD.
template <int N>
__device__ inline void sort_bucket(uint32_t* keys, int32_t off, int32_t n) {
    static_assert(N <= RS_PAD, "reads stay inside the padding");
    uint32_t a[N];
#pragma unroll
    for (int u = 0; u < N; ++u) a[u] = keys[off + u];
#pragma unroll
    for (int u = 0; u < N; ++u) a[u] = u < n ? a[u] : 0xffffffffu;
    sort_network<N>(a);
#pragma unroll
    for (int u = 0; u < N; ++u)
        if (u < n) keys[off + u] = a[u];
}

// Counts the row's entries (bucket_of(u): step u's bucket) into W.bcnt, which
// is clear, and sorts them if the largest bucket fits a network: the keys key_of(u)
// are placed bucket by bucket and every lane sorts its own.  false: not sorted.
// Counted first, then placed by a second atomic that returns the place: keeping
// each entry's place in between costs registers, and so waves.
template <int NU, typename V, class BucketOf, class KeyOf>
__device__ inline bool wave_sort_by_buckets(RowSortLds<V, NU>& W, int32_t L, BucketOf bucket_of, KeyOf key_of) {
    const int lane = lane_id();
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        if (u * SPG_WAVE >= L) break;
        if (u * SPG_WAVE + lane < L) atomicAdd(&W.bcnt[bucket_of(u)], 1);
    }
    wave_lds_sync();
    const int32_t mine = W.bcnt[lane];
    const int32_t off = wave_inclusive_scan_add(mine) - mine;
    const int32_t most =
        __builtin_amdgcn_readfirstlane(wave_all(mine, [](int32_t x, int32_t y) { return x > y ? x : y; }));
    wave_lds_sync();  // every lane has its count
    if (most > RS_PAD) return false;
    W.bcnt[lane] = off;
    wave_lds_sync();
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        if (u * SPG_WAVE >= L) break;
        if (u * SPG_WAVE + lane < L) W.key[atomicAdd(&W.bcnt[bucket_of(u)], 1)] = key_of(u);
    }
    wave_lds_sync();
    if (most <= 8) sort_bucket<8>(W.key, off, mine);
    else if (most <= 12) sort_bucket<12>(W.key, off, mine);
    else sort_bucket<16>(W.key, off, mine);
    return true;
}

// Sorts entries x < L (0 < L <= NU * 64), col[u] the column of entry u * 64 +
// lane, that span fewer than RS_SPAN_MAX columns from cmin to cmax, into W.key.
// W.bcnt is clear; W.key may be overwritten.  pfx (optional): NU * 32 words for the
// ranks of clustered columns.
template <int NU, typename V>
__device__ inline void wave_sort_row(RowSortLds<V, NU>& W, int32_t L, int32_t cmin, int32_t cmax,
                                     const int32_t (&col)[NU], uint16_t* pfx) {
    const int lane = lane_id();
    auto key_of = [&](int u) { return ((uint32_t)(col[u] - cmin) << RS_XBITS) | (uint32_t)(u * SPG_WAVE + lane); };
    const float bscale = (float)SPG_WAVE / ((float)(uint32_t)(cmax - cmin) + 1.0f);
    bool done = wave_sort_by_buckets(W, L, [&](int u) {
        const int32_t t = (int32_t)((float)(uint32_t)(col[u] - cmin) * bscale);
        return t < SPG_WAVE - 1 ? t : SPG_WAVE - 1;
    }, key_of);
    // Clustered columns overfill some of the buckets of equal width.  Where a
    // bitmap of the span fits W.key, a column's rank among the row's columns
    // makes buckets of equal numbers of columns instead.
    const int32_t nw = ((cmax - cmin) >> 5) + 1;
    if (!done && pfx && nw <= NU * SPG_WAVE) {
        static_assert(NU % 2 == 0, "a prefix for every two words");
        W.bcnt[lane] = 0;
#pragma unroll
        for (int k = 0; k < NU; ++k) W.key[k * SPG_WAVE + lane] = 0;
        wave_lds_sync();
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            if (u * SPG_WAVE >= L) break;
            const int32_t d = col[u] - cmin;
            if (u * SPG_WAVE + lane < L) atomicOr(&W.key[d >> 5], 1u << (d & 31));
        }
        wave_lds_sync();
        int32_t two[NU / 2], sum = 0;  // set bits of this lane's pairs of words
#pragma unroll
        for (int k = 0; k < NU / 2; ++k) {
            two[k] = __popc(W.key[lane * NU + 2 * k]) + __popc(W.key[lane * NU + 2 * k + 1]);
            sum += two[k];
        }
        const int32_t incl = wave_inclusive_scan_add(sum);
        int32_t run = incl - sum;
#pragma unroll
        for (int k = 0; k < NU / 2; ++k) {
            pfx[lane * (NU / 2) + k] = (uint16_t)run;
            run += two[k];
        }
        wave_lds_sync();
        const float rscale = (float)SPG_WAVE / (float)__builtin_amdgcn_readlane(incl, SPG_WAVE - 1);
        uint32_t b[NU];  // the entries' buckets
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            if (u * SPG_WAVE >= L) break;
            const int32_t d = col[u] - cmin, w = d >> 5;
            const uint32_t below = W.key[w] & ((1u << (d & 31)) - 1u), before = W.key[w & ~1];
            const int32_t rank = (int32_t)pfx[w >> 1] + __popc(below) + ((w & 1) ? __popc(before) : 0);
            const int32_t t = (int32_t)((float)rank * rscale);
            b[u] = t < SPG_WAVE - 1 ? t : SPG_WAVE - 1;
        }
        wave_lds_sync();  // the bitmap is read before keys overwrite it
        done = wave_sort_by_buckets(W, L, [&](int u) { return b[u]; }, key_of);
    }
    if (!done) {  // the wave sorts the row whole
        int P = SPG_WAVE;
        while (P < L) P <<= 1;
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int32_t x = u * SPG_WAVE + lane;
            if (x < L) W.key[x] = key_of(u);
            else if (x < P) W.key[x] = 0xffffffffu;
        }
        wave_lds_sync();
        wave_lds_bitonic_u32(W.key, P);
    }
    wave_lds_sync();
}

// Clears the bucket counts and reads the row's columns and their span.
template <int NU, typename V>
__device__ inline void wave_row_span(RowSortLds<V, NU>& W, int32_t L, int32_t (&col)[NU], int32_t& cmin, int32_t& cmax) {
    const int lane = lane_id();
    W.bcnt[lane] = 0;
    cmin = 0x7fffffff;
    cmax = -1;
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        if (u * SPG_WAVE >= L) break;
        const int32_t x = u * SPG_WAVE + lane;
        col[u] = (int32_t)W.key[x < L ? x : L - 1];
    }
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        if (u * SPG_WAVE >= L) break;
        cmin = col[u] < cmin ? col[u] : cmin;
        cmax = col[u] > cmax ? col[u] : cmax;
    }
    cmin = __builtin_amdgcn_readfirstlane(wave_all(cmin, [](int32_t x, int32_t y) { return x < y ? x : y; }));
    cmax = __builtin_amdgcn_readfirstlane(wave_all(cmax, [](int32_t x, int32_t y) { return x > y ? x : y; }));
    wave_lds_sync();  // the columns are read before keys overwrite them
}

// Folds the sorted row and writes it from position o on, at most `room`
// outputs; returns their number.
template <int SR, int NU>
__device__ inline int32_t wave_fold_row(const RowSortLds<typename Sr<SR>::acc_t, NU>& W, int32_t L, int32_t cmin,
                                        int32_t* out_col, void* out_val, int64_t o, int32_t room) {
    typedef Sr<SR> S;
    typedef typename S::acc_t V;
    constexpr uint32_t XMASK = (1u << RS_XBITS) - 1;
    const int lane = lane_id();
    constexpr int U = NU < 4 ? NU : 4;  // steps whose LDS reads are in flight together
    int32_t before = 0;
#pragma unroll
    for (int u0 = 0; u0 < NU; u0 += U) {
        if (u0 * SPG_WAVE >= L) break;
        uint32_t key[U], prev[U];
        V v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int32_t x = (u0 + u) * SPG_WAVE + lane;
            const int32_t y = x < L ? x : L - 1;
            key[u] = W.key[y];
            prev[u] = W.key[y > 0 ? y - 1 : 0];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = W.val[key[u] & XMASK];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int32_t s = (u0 + u) * SPG_WAVE;
            if (s >= L) break;
            const int32_t y = s + lane;
            const uint32_t c = key[u] >> RS_XBITS;
            const bool head = y < L && (y == 0 || (prev[u] >> RS_XBITS) != c);
            const uint64_t heads = __builtin_amdgcn_ballot_w64(head);
            // a later entry of the run in the next lane (or past this step)
            const int32_t left = L - s;  // entries from this step on
            const uint64_t full = left >= SPG_WAVE ? ~0ull : (1ull << left) - 1;
            const uint64_t more = (~heads & full) >> 1 | (left > SPG_WAVE ? 1ull << 63 : 0);
            if (more) {
                if (head && ((more >> lane) & 1))
                    for (int32_t z = y + 1; z < L; ++z) {
                        const uint32_t kz = W.key[z];
                        if ((kz >> RS_XBITS) != c) break;
                        v[u] = S::add(v[u], W.val[kz & XMASK]);
                    }
            }
            const int32_t r = before + lanes_below(heads);
            if (head && r < room) {
                out_col[o + r] = cmin + (int32_t)c;
                if (out_val) S::store(out_val, o + r, v[u]);
            }
            before += __popcll(heads);
        }
    }
    return before;
}

}  // namespace spg
