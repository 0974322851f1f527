// Numeric phase: C(i,j) = (+)-sum over stored A(i,k), k in window, of
// A(i,k) (x) B(k,j), written as canonical CSR rows sorted by column
// (Section 5.1.1) at the offsets the symbolic phase produced.  Bins:
//   TINY   one A entry: C(i,:) = a (x) B(k,:), already sorted (no accumulator)
//   SMALL  <= 64 products: one wave per row; products sorted across the wave
//          by (column, product order), equal columns folded left to right,
//          which is ascending k (the order of Algorithm 1)
//   HASH   rows of few products per output in the bins of up to 384 outputs: a
//          wave sorts the products (rowsort.hpp); otherwise
//          workgroup per row: LDS open-addressing table sized >= 4/3 slots per
//          output, semiring add by LDS atomics, then compaction and an LDS
//          bitonic sort by column
//   RANK   rows whose symbolic pass kept an n-bit bitmap: the bitmap is
//          reloaded, each word gets the count of set bits before it, c_col is
//          written straight from the bitmap, and values accumulate in LDS at
//          index rank(j) = set bits below column j, i.e. directly in output
//          order (a sparse accumulator compressed to the row's own columns)
//   DENSE  workgroup per row sweeping column chunks of W: an LDS dense
//          accumulator plus occupancy bitmap per chunk (the sparse
//          accumulator of Section 3, blocked by columns so it fits LDS);
//          the bitmap scan emits columns in order, so no sort is needed.
#pragma once
#include "products.hpp"
#include "rowinfo.hpp"
#include "rowsort.hpp"
#include "symbolic.hpp"

namespace spg {

// Where a row's output goes: its count is rp[i+1] - rp[i]; it starts at
// pos[i] when pos is given (rows of a gathered sub-product written straight
// into the full product), else at rp[i].
struct OutRows {
    const int64_t* rp;
    const int64_t* pos;
    __host__ __device__ OutRows(const int64_t* r, const int64_t* p = nullptr) : rp(r), pos(p) {}
    __device__ int64_t off(int64_t i) const { return pos ? pos[i] : rp[i]; }
    __device__ int64_t count(int64_t i) const { return rp[i + 1] - rp[i]; }
};

// Rows of one A entry in the window: C(i,:) = a * B(k,:), a copy.  Each row
// takes G lanes (256 / G rows per workgroup): with G = 16 a wave keeps the
// dependent loads (row, A entry, B row extent) of four rows in flight, for
// bins whose B rows are short (most lanes of a whole wave would idle); G =
// 64 (a wave per row) for long B rows (R-MAT hubs), where 16 lanes would
// need four times the steps.
template <int SR, int G>
__global__ void __launch_bounds__(256) k_num_tiny(Csr A, Csr B, const int32_t* rows, int32_t nrows,
                                                  const int64_t* a_beg, OutRows c_rp,
                                                  int32_t* c_col, void* c_val) {
    typedef Sr<SR> S;
    static_assert(G == 16 || G == 32 || G == 64, "lanes per row");
    const int r = blockIdx.x * (256 / G) + (int)(threadIdx.x / G);
    if (r >= nrows) return;  // no barriers below
    const int g = (int)(threadIdx.x % G);
    const int64_t i = rows[r];
    const int64_t p = a_beg[i];
    const int64_t k = A.col[p];
    const typename S::acc_t a = S::load(A.val, p);
    const int64_t bs = B.rp[k], be = B.rp[k + 1];
    const int64_t off = c_rp.off(i) - bs;
    // four strides of the row loaded before any is stored, so the loads of
    // a long B row overlap instead of waiting one stride at a time
    constexpr int U = 4;
    for (int64_t q0 = bs; q0 < be; q0 += U * G) {
        int32_t cc[U];
        typename S::acc_t vv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t q = q0 + u * G + g;
            cc[u] = 0;
            vv[u] = S::zero();
            if (q < be) {
                cc[u] = B.col[q];
                if (c_val) vv[u] = S::load(B.val, q);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t q = q0 + u * G + g;
            if (q < be) {
                c_col[off + q] = cc[u];
                if (c_val) S::store(c_val, off + q, S::mul(a, vv[u]));
            }
        }
    }
}

// cnt_out (optional) receives each row's output count.  4 waves per block,
// SMALL_ROWS rows per wave (their loads in flight together; four rows measured
// 2 to 3 % slower than two).
//
// It was bound by instruction issue (81 % of the vector slots): a search of six
// lane exchanges for each product's segment, 64-bit addresses of the windows per
// lane, one row's sort after another's, and a fold that shifted columns, values
// and validity and compared them at every step.  Now the segments are marked,
// the wave's rows are scalars, the sorts run side by side and end at the row's
// size, and a fold step is a shift and an add: 350 -> 170 vector instructions a
// row; the two products of 64 grids of 16^3 ... 64^3 points 700 -> 530 us, at 3.5
// TB/s past L2, bound by latency at full occupancy.
template <int SR>
__global__ void __launch_bounds__(256) k_num_small(Csr A, Csr B, const int32_t* rows, int32_t nrows,
                                                   const int64_t* a_beg, const int64_t* a_end,
                                                   OutRows c_rp, int32_t* c_col, void* c_val,
                                                   int64_t* cnt_out) {
    typedef Sr<SR> S;
    typedef typename S::acc_t V;
    // the wave's number as a scalar: its rows' windows are then scalar loads
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t w = (int64_t)blockIdx.x * 4 + wv;
    if (w * SMALL_ROWS >= nrows) return;  // whole wave leaves; no block barriers below
    const int lane = lane_id();
    __shared__ uint8_t s_mark[4][SMALL_ROWS * SPG_WAVE];
    V vals[SMALL_ROWS];
    uint32_t key[SMALL_ROWS];  // columns, then (32-bit sort) columns and product order
    int64_t row[SMALL_ROWS];
    int n[SMALL_ROWS];
    for_small_rows(A, B, rows, nrows, w, a_beg, a_end, s_mark[wv], n,
                   [&](int u, int64_t i, bool have, int64_t p, int64_t q) {
        row[u] = i;
        vals[u] = S::zero();
        key[u] = ~0u;
        if (have) {
            vals[u] = S::mul(S::load(A.val, p), S::load(B.val, q));
            key[u] = (uint32_t)B.col[q];
        }
    });
    int order[SMALL_ROWS];  // the product this lane takes after the sort
    // (column, lane) fits 32 bits below 2^26 - 1 columns (the all-ones key stays
    // the empty lane's): the cheaper 32-bit sort of all rows together
    if (B.ncols < (1ll << 26) - 1) {
        int most = 0;
#pragma unroll
        for (int u = 0; u < SMALL_ROWS; ++u) {
            key[u] = lane < n[u] ? key[u] << 6 | (uint32_t)lane : ~0u;
            most = n[u] > most ? n[u] : most;
        }
        wave_bitonic_sort_u32(key, most);
#pragma unroll
        for (int u = 0; u < SMALL_ROWS; ++u) {
            order[u] = (int)(key[u] & 63);
            key[u] >>= 6;
        }
    } else {
#pragma unroll
        for (int u = 0; u < SMALL_ROWS; ++u) {
            const uint64_t k = wave_bitonic_sort_u64(lane < n[u] ? (uint64_t)key[u] << 6 | (uint64_t)lane : ~0ull);
            order[u] = (int)(k & 63);
            key[u] = (uint32_t)(k >> 6);
        }
    }
#pragma unroll
    for (int u = 0; u < SMALL_ROWS; ++u) {
        if (w * SMALL_ROWS + u >= nrows) break;
        V v = __shfl(vals[u], order[u], SPG_WAVE);  // value travels with its key
        const uint64_t heads = wave_fold_sorted<SR>(key[u], v, n[u]);
        if (__builtin_amdgcn_inverse_ballot_w64(heads)) {
            const int64_t o = c_rp.off(row[u]) + lanes_below(heads);
            c_col[o] = (int32_t)key[u];
            if (c_val) S::store(c_val, o, v);
        }
        if (cnt_out && lane == 0) cnt_out[row[u]] = __popcll(heads);
    }
}

// A row of the one-wave hash bins by sorting (rowsort.hpp): f products, at
// most 64 NU.  Each batch of 64 A entries is scanned, the lane of every
// non-empty B segment is marked at its first product, and a running maximum of
// the marks gives each product its segment.
template <int SR, int NU>
__device__ inline void num_sort_row(const Csr& A, const Csr& B, int64_t beg, int64_t end, int32_t f,
                                    RowSortLds<typename Sr<SR>::acc_t, NU>& W, uint8_t* marks, int32_t* c_col,
                                    void* c_val, int64_t o, int32_t room) {
    typedef Sr<SR> S;
    typedef typename S::acc_t V;
    const int lane = lane_id();
    int32_t pos = 0;  // products of the batches before
    for (int64_t base = beg; base < end && pos < f; base += SPG_WAVE) {
        const int64_t p = base + lane;
        int64_t bs = 0;
        int32_t len = 0;
        V av = S::zero();
        if (p < end) {
            const int64_t k = A.col[p];
            bs = B.rp[k];
            len = (int32_t)(B.rp[k + 1] - bs);
            av = S::load(A.val, p);
        }
        const int32_t inc = wave_inclusive_scan_add(len);
        int32_t nb = __builtin_amdgcn_readlane(inc, SPG_WAVE - 1);
        nb = nb < f - pos ? nb : f - pos;  // (f counts them all: a guard for inputs changed since)
        const int32_t off = inc - len;
        const int64_t rel = bs - off;
#pragma unroll
        for (int t = 0; t < NU / 4 + 1; ++t)
            if (t * SPG_WAVE + lane < NU * SPG_WAVE / 4) reinterpret_cast<uint32_t*>(marks)[t * SPG_WAVE + lane] = 0;
        wave_lds_sync();
        if (len > 0 && off < nb) marks[off] = (uint8_t)lane;
        wave_lds_sync();
        // four steps of gathers in flight (more cost registers, so waves)
        constexpr int U = NU < 4 ? NU : 4;
        int32_t carry = 0;
#pragma unroll
        for (int u0 = 0; u0 < NU; u0 += U) {
            if (u0 * SPG_WAVE >= nb) break;
            int32_t mark[U];
            V a[U];
            BEntry<V> e[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int32_t x = (u0 + u) * SPG_WAVE + lane;
                mark[u] = marks[x < nb ? x : nb - 1];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                int32_t l = wave_inclusive_scan_max(mark[u]);
                l = l > carry ? l : carry;
                carry = __builtin_amdgcn_readlane(l, SPG_WAVE - 1);
                const int32_t x = (u0 + u) * SPG_WAVE + lane;
                const int64_t q = lane_get(rel, l) + (x < nb ? x : nb - 1);
                a[u] = lane_get(av, l);
                e[u] = BEntry<V>{B.col[q], S::load(B.val, q)};
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                pin(e[u]);
                const int32_t x = (u0 + u) * SPG_WAVE + lane;
                if (x < nb) {
                    W.key[pos + x] = (uint32_t)e[u].col;
                    W.val[pos + x] = S::mul(a[u], e[u].val);
                }
            }
        }
        pos += nb;
        wave_lds_sync();
    }
    if (pos == 0) return;
    int32_t col[NU], cmin, cmax;
    wave_row_span(W, pos, col, cmin, cmax);
    wave_sort_row(W, pos, cmin, cmax, col, reinterpret_cast<uint16_t*>(marks));  // (the marks are done with)
    (void)wave_fold_row<SR, NU>(W, pos, cmin, c_col, c_val, o, room);
}

// cnt_out (optional) receives each row's output count; a count above the
// slot c_rp.count(i) means the slot overflowed (only then is the output
// incomplete).
template <int SR, int NT, int LOG2T>
__global__ void __launch_bounds__(NT) k_num_hash(Csr A, Csr B, const int32_t* rows,
                                                 const int64_t* a_beg, const int64_t* a_end,
                                                 const int64_t* flops, OutRows c_rp, int32_t* c_col, void* c_val,
                                                 int64_t* cnt_out) {
    typedef Sr<SR> S;
    typedef typename S::acc_t V;
    constexpr int T = 1 << LOG2T;
    constexpr int PER = T / NT;  // table slots owned by a thread during compaction
    static_assert(PER >= 1, "table smaller than block");
    // 8 bytes a slot whatever the value type: the full sort below keeps up
    // to T keys of 8 bytes there
    struct Table {
        uint64_t val[T];
        int32_t key[T];
    };
    constexpr bool SORT = NT == SPG_WAVE;  // the one-wave bins sort most rows instead
    constexpr int NU = SORT ? T / SPG_WAVE : 1;  // steps of 64 products a row may sort
    union Lds {
        Table table;
        RowSortLds<V, NU> sort;
        __device__ Lds() {}
    };
    __shared__ Lds lds;
    int32_t* tkey = lds.table.key;
    uint64_t* tval_store = lds.table.val;
    V* tval = reinterpret_cast<V*>(tval_store);
    __shared__ ProductLds<NT> L;
    __shared__ int32_t red[NT / SPG_WAVE + 1];
    __shared__ int32_t mm[2 * (NT / SPG_WAVE)];
    __shared__ V s_av[NT];
    __shared__ int32_t s_bucket[NT];
    __shared__ __align__(4) uint8_t s_mark[SORT ? (T > 4 * SPG_WAVE ? T : 4 * SPG_WAVE) : 4];
    const int64_t i = rows[blockIdx.x];
    if constexpr (SORT) {
        // Sorting costs by the product, the table by the slot and the output, so
        // rows of up to 64 NU products and three per two outputs are sorted.  64
        // grids restricted by MIS-2 aggregates (R^T A has two products per output),
        // batched: 0.94 ms; with four per output sorted 0.99, with nine per eight
        // 0.94; uniform matrices the same.
        const int64_t f = flops[i], n = c_rp.count(i);
        if (!cnt_out && f <= NU * SPG_WAVE && f <= n + n / 2 && B.ncols <= RS_SPAN_MAX) {
            num_sort_row<SR, NU>(A, B, a_beg[i], a_end[i], (int32_t)f, lds.sort, s_mark, c_col, c_val, c_rp.off(i),
                                 (int32_t)n);
            return;
        }
    }
    for (int t = threadIdx.x; t < T; t += NT) {
        tkey[t] = EMPTY_KEY;
        tval[t] = S::zero();
    }
    __syncthreads();
    // the table has >= 4/3 slots per output of the symbolic count, so a
    // probe ends within T steps; the cap only guards inputs that changed
    // between the two phases
    auto insert = [&](int32_t j, V v) {
        uint32_t h = hash_slot(j, LOG2T);
        for (int probes = 0; probes < T; ++probes) {
            int32_t cur = __hip_atomic_load(&tkey[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (cur == EMPTY_KEY) {
                int32_t old = atomicCAS(&tkey[h], EMPTY_KEY, j);
                cur = old == EMPTY_KEY ? j : old;
            }
            if (cur == j) {
                S::lds_add(&tval[h], v);
                break;
            }
            h = (h + 1) & (T - 1);
        }
    };
    if constexpr (NT == SPG_WAVE) {
        // one wave: the lane search needs no block-wide enumeration
        wave_products<4, V>(
            a_beg[i], a_end[i], s_mark,
            [&](int64_t p, int64_t& bs, int32_t& len, V& av) {
                const int64_t k = A.col[p];
                bs = B.rp[k];
                len = (int32_t)(B.rp[k + 1] - bs);
                av = S::load(A.val, p);
            },
            [&](int64_t q) { return BEntry<V>{B.col[q], S::load(B.val, q)}; },
            [&](V av, const BEntry<V>& x) { insert(x.col, S::mul(av, x.val)); });
        __syncthreads();  // every insertion lands before the table is read
    } else {
        for_each_product_u<NT, 4>(
            a_beg[i], a_end[i], L,
            [&](int64_t p, int64_t& bs, int32_t& len) {
                int64_t k = A.col[p];
                bs = B.rp[k];
                len = (int32_t)(B.rp[k + 1] - bs);
            },
            [&](int t, int64_t p) { s_av[t] = S::load(A.val, p); },
            [&](int64_t q) { return BEntry<V>{B.col[q], S::load(B.val, q)}; },
            [&](int t, const BEntry<V>& x) { insert(x.col, S::mul(s_av[t], x.val)); });
    }
    // compaction: slots [t*PER, (t+1)*PER) -> registers
    int32_t rk[PER];
    V rv[PER];
    int32_t mine = 0;
#pragma unroll
    for (int s = 0; s < PER; ++s) {
        rk[s] = tkey[threadIdx.x * PER + s];
        rv[s] = tval[threadIdx.x * PER + s];
        mine += rk[s] != EMPTY_KEY;
    }
    __syncthreads();  // every slot is in registers before the table is reused
    int32_t cnt;
    int32_t pos = block_exclusive_scan<NT, int32_t>(mine, &cnt, red);
    const int64_t o = c_rp.off(i);
    const int32_t cnt_sym = (int32_t)c_rp.count(i);
    if (cnt_out && threadIdx.x == 0) cnt_out[i] = cnt;
    if (cnt_out && cnt > cnt_sym) return;  // slot overflow: the row is redone exactly
    // Output order.  When the row's columns span few enough bitmap words, the
    // rank of a column is the popcount of the bitmap below it (prefix of
    // per-word popcounts): no sort.  Otherwise sort (column, slot) keys.
    int32_t kmin = 0x7fffffff, kmax = -1;
#pragma unroll
    for (int s = 0; s < PER; ++s) {
        if (rk[s] != EMPTY_KEY) {
            kmin = rk[s] < kmin ? rk[s] : kmin;
            kmax = rk[s] > kmax ? rk[s] : kmax;
        }
    }
    block_min_max<NT, int32_t>(kmin, kmax, mm);
    const int32_t nw = kmax >= kmin ? ((kmax - kmin) >> 5) + 1 : 0;
    if (nw > 0 && nw <= T && nw <= 8 * cnt + 64) {
        uint32_t* bm = reinterpret_cast<uint32_t*>(tkey);
        int32_t* wp = reinterpret_cast<int32_t*>(tval);
        for (int w = threadIdx.x; w < nw; w += NT) bm[w] = 0u;
        __syncthreads();
#pragma unroll
        for (int s = 0; s < PER; ++s) {
            if (rk[s] != EMPTY_KEY) {
                const int32_t j = rk[s] - kmin;
                atomicOr(&bm[j >> 5], 1u << (j & 31));
            }
        }
        __syncthreads();
        const int wpt = (nw + NT - 1) / NT;
        const int w0 = threadIdx.x * wpt;
        int32_t part = 0;
        for (int w = w0; w < w0 + wpt && w < nw; ++w) part += __popc(bm[w]);
        int32_t dummy;
        int32_t run = block_exclusive_scan<NT, int32_t>(part, &dummy, red);
        for (int w = w0; w < w0 + wpt && w < nw; ++w) {
            wp[w] = run;
            run += __popc(bm[w]);
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < PER; ++s) {
            if (rk[s] != EMPTY_KEY) {
                const int32_t j = rk[s] - kmin;
                const int32_t w = j >> 5;
                const int32_t rank = wp[w] + __popc(bm[w] & ((1u << (j & 31)) - 1u));
                if (rank < cnt_sym) {
                    c_col[o + rank] = rk[s];
                    if (c_val) S::store(c_val, o + rank, rv[s]);
                }
            }
        }
        return;
    }
    // Wide spans: NT buckets of (nearly) equal column width, one per thread.
    // The entries are counted per bucket, placed bucket by bucket, and each
    // thread sorts its own bucket (insertion sort); then the row is written in
    // order.  Falls back to the full sort below when some bucket holds more
    // than 32.  The bucket of a column is (column - kmin) * NT / span in FP32,
    // truncated and clamped to NT - 1: every step of that is monotone, so the
    // buckets follow column order, and it costs a multiply where an integer
    // division by the width would cost a few dozen instructions per entry.
    if (cnt <= T) {
        const float bscale = (float)NT / (float)((int64_t)kmax - kmin + 1);
        auto bucket_of = [&](int32_t key) {
            const int32_t b = (int32_t)((float)(uint32_t)(key - kmin) * bscale);
            return b < NT - 1 ? b : NT - 1;
        };
        s_bucket[threadIdx.x] = 0;
        __syncthreads();
        int32_t bl[PER];
#pragma unroll
        for (int s = 0; s < PER; ++s)
            bl[s] = rk[s] != EMPTY_KEY ? atomicAdd(&s_bucket[bucket_of(rk[s])], 1) : 0;
        __syncthreads();
        const int32_t mycnt = s_bucket[threadIdx.x];
        int32_t bmin = mycnt, bmax = mycnt;
        block_min_max<NT, int32_t>(bmin, bmax, mm);
        if (bmax <= 32) {
            int32_t tot;
            const int32_t boff = block_exclusive_scan<NT, int32_t>(mycnt, &tot, red);
            s_bucket[threadIdx.x] = boff;
            __syncthreads();
            const int32_t nout = cnt < cnt_sym ? cnt : cnt_sym;
            // Columns that fit beside a slot index in 32 bits: each entry
            // becomes the key (column - kmin) << LOG2T | slot, the values stay
            // in the table, and every thread sorts its bucket's keys in
            // registers with a sorting network (two instructions per
            // comparator, no LDS round trips).  Buckets of 17 to 32 take a
            // network only in the kernels of 16 slots per thread, where they
            // are common; elsewhere its registers would cost waves.
            constexpr int NET_MAX = PER >= 16 ? 32 : 16;
            if (bmax <= NET_MAX && cnt > 0 && (int64_t)kmax - kmin < (1ll << (32 - LOG2T))) {
#pragma unroll
                for (int s = 0; s < PER; ++s) {
                    if (rk[s] != EMPTY_KEY) {
                        const int32_t q = s_bucket[bucket_of(rk[s])] + bl[s];
                        tkey[q] = (int32_t)(((uint32_t)(rk[s] - kmin) << LOG2T) | (uint32_t)(threadIdx.x * PER + s));
                    }
                }
                __syncthreads();
                uint32_t* pk = reinterpret_cast<uint32_t*>(tkey);
                if (bmax <= 8) bucket_sort_net<8>(pk, boff, mycnt, T);
                else if (NET_MAX == 16 || bmax <= 16) bucket_sort_net<16>(pk, boff, mycnt, T);
                else bucket_sort_net<NET_MAX>(pk, boff, mycnt, T);
                __syncthreads();
                for (int t = threadIdx.x; t < nout; t += NT) {
                    const uint32_t key = (uint32_t)tkey[t];
                    c_col[o + t] = kmin + (int32_t)(key >> LOG2T);
                    if (c_val) S::store(c_val, o + t, tval[key & (T - 1)]);
                }
                return;
            }
#pragma unroll
            for (int s = 0; s < PER; ++s) {
                if (rk[s] != EMPTY_KEY) {
                    const int32_t q = s_bucket[bucket_of(rk[s])] + bl[s];
                    tkey[q] = rk[s];
                    tval[q] = rv[s];
                }
            }
            __syncthreads();
            for (int x = boff + 1; x < boff + mycnt; ++x) {
                const int32_t kx = tkey[x];
                const V vx = tval[x];
                int y = x - 1;
                while (y >= boff && tkey[y] > kx) {
                    tkey[y + 1] = tkey[y];
                    tval[y + 1] = tval[y];
                    --y;
                }
                tkey[y + 1] = kx;
                tval[y + 1] = vx;
            }
            __syncthreads();
            for (int t = threadIdx.x; t < nout; t += NT) {
                c_col[o + t] = tkey[t];
                if (c_val) S::store(c_val, o + t, tval[t]);
            }
            return;
        }
        __syncthreads();
    }
    // Full sort: (column, compact index) keys sorted in the value storage
    // (up to T keys of 8 bytes); the sorted order gives each compact index
    // its rank (in tkey's bytes), and every thread writes its own entries,
    // whose values never left its registers, at their ranks.
    uint64_t* skey = tval_store;
    int32_t* rank_of = tkey;
    int32_t posv[PER];
#pragma unroll
    for (int s = 0; s < PER; ++s) {
        posv[s] = -1;
        if (rk[s] != EMPTY_KEY) {
            posv[s] = pos;
            skey[pos] = ((uint64_t)(uint32_t)rk[s] << 32) | (uint64_t)pos;
            ++pos;
        }
    }
    int P = 1;
    while (P < cnt) P <<= 1;
    for (int t = cnt + threadIdx.x; t < P; t += NT) skey[t] = ~0ull;
    __syncthreads();
    block_bitonic_sort<NT>(skey, P);
    for (int t = threadIdx.x; t < cnt; t += NT) rank_of[(int32_t)(skey[t] & 0xffffffffu)] = t;
    __syncthreads();
#pragma unroll
    for (int s = 0; s < PER; ++s) {
        if (posv[s] >= 0) {
            const int32_t rank = rank_of[posv[s]];
            if (rank < cnt_sym) {
                c_col[o + rank] = rk[s];
                if (c_val) S::store(c_val, o + rank, rv[s]);
            }
        }
    }
}

// Column split table for the dense sweep: split[k*(P+1)+c] = offset inside
// B(k,:) of the first entry with column >= c*W (c = 0..P).
__global__ void __launch_bounds__(256) k_split_table(Csr B, int32_t W, int32_t P, int32_t* split) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t total = B.nrows * (int64_t)(P + 1);
    if (idx >= total) return;
    const int64_t k = idx / (P + 1);
    const int c = (int)(idx - k * (P + 1));
    const int64_t rs = B.rp[k], re = B.rp[k + 1];
    int64_t r;
    if (c == 0) r = rs;
    else if (c == P) r = re;
    else r = lower_bound_col(B.col, rs, re, (int64_t)c * W);
    split[idx] = (int32_t)(r - rs);
}

// Rows without a saved bitmap (n above the LDS bitmap): one workgroup per
// row sweeps the P column chunks of W columns in order, accumulating each
// chunk densely in LDS and emitting it in column order.
template <int SR, int NT, int W, int GM>
__global__ void __launch_bounds__(NT) k_num_dense(Csr A, Csr B, const int32_t* rows, int64_t nrows,
                                                  const int64_t* a_beg, const int64_t* a_end,
                                                  const int32_t* split, int32_t P,
                                                  OutRows c_rp, int32_t* c_col, void* c_val) {
    typedef Sr<SR> S;
    typedef typename S::acc_t V;
    constexpr int NWD = W / 32;
    static_assert(NWD <= NT, "one bitmap word per thread at most");
    __shared__ V acc[W];
    __shared__ uint32_t bits[NWD];
    __shared__ V s_av[NT];
    __shared__ ProductLds<NT> L;
    __shared__ int32_t red[NT / SPG_WAVE + 1];
    // the accumulator is cleared once; emission resets exactly the slots it
    // reads, so later chunks (and later work items) start from zero again
    for (int t = threadIdx.x; t < W; t += NT) acc[t] = S::zero();
    for (int t = threadIdx.x; t < NWD; t += NT) bits[t] = 0u;
    // grid-stride over the rows, so the grid stays small
    for (int64_t item = blockIdx.x; item < nrows; item += gridDim.x) {
    const int64_t i = rows[item];
    const int64_t beg = a_beg[i], end = a_end[i];
    int64_t off = c_rp.off(i);
    const int64_t row_end = off + c_rp.count(i);
    const int c_first = 0, c_last = P;
    // Rows with at most one batch of entries in the window keep their A entry (column
    // k, start of B(k,:), position reached in B(k,:)) in registers across
    // the chunks, so each chunk costs one split-table load per entry.
    const bool single = end - beg <= ProductLds<NT>::EB;
    int64_t my_k = 0, my_rs = 0;
    int32_t my_cur = 0;
    V my_av = S::zero();
    if (single && beg + (int64_t)threadIdx.x < end) {
        const int64_t p = beg + threadIdx.x;
        my_k = A.col[p];
        my_rs = B.rp[my_k];
        my_av = S::load(A.val, p);
    }
    __syncthreads();
    for (int c = c_first; c < c_last; ++c) {
        const int32_t cbase = c * W;
        for_each_product_gm<NT, GM>(
            beg, end, L,
            [&](int64_t p, int64_t& bs, int32_t& len) {
                if (single) {
                    const int32_t nxt = P > 1 ? split[my_k * (P + 1) + c + 1] : (int32_t)(B.rp[my_k + 1] - my_rs);
                    bs = my_rs + my_cur;
                    len = nxt - my_cur;
                    my_cur = nxt;
                } else {
                    const int64_t k = A.col[p];
                    const int64_t rs = B.rp[k];
                    if (P > 1) {
                        const int32_t* sp = split + k * (P + 1) + c;
                        bs = rs + sp[0];
                        len = sp[1] - sp[0];
                    } else {
                        bs = rs;
                        len = (int32_t)(B.rp[k + 1] - rs);
                    }
                }
            },
            [&](int t, int64_t p) { s_av[t] = single ? my_av : S::load(A.val, p); },
            [&](int64_t q) { return BEntry<V>{B.col[q], S::load(B.val, q)}; },
            [&](int t, const BEntry<V>& x) {
                const int32_t j = x.col - cbase;
                S::lds_add(&acc[j], S::mul(s_av[t], x.val));
                atomicOr(&bits[j >> 5], 1u << (j & 31));
            });
        // thread t owns bitmap word t: prefix of popcounts, then its set bits
        const uint32_t wbits = threadIdx.x < NWD ? bits[threadIdx.x] : 0u;
        int32_t chunk_total;
        int32_t pre = block_exclusive_scan<NT, int32_t>(__popc(wbits), &chunk_total, red);
        if (wbits) {
            int64_t o = off + pre;
            uint32_t wb = wbits;
            while (wb) {
                const int b = __ffs(wb) - 1;
                wb &= wb - 1;
                const int j = threadIdx.x * 32 + b;
                if (o < row_end) {
                    c_col[o] = cbase + j;
                    if (c_val) S::store(c_val, o, acc[j]);
                }
                acc[j] = S::zero();
                ++o;
            }
            bits[threadIdx.x] = 0u;
        }
        off += chunk_total;
        __syncthreads();
    }
    }
}

__device__ inline int32_t uniform32(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ inline int64_t uniform64(int64_t v) {
    return (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)((uint64_t)v >> 32)) << 32) |
                     (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v));
}
// A bitmap's words spread over a workgroup, at most KW per thread: wave w
// holds the 64 keff words from 64 keff w, word k of a lane 64 k further, so
// the loads are coalesced and a wave's words are consecutive.
template <int NT, int KW>
__device__ inline void fetch_words(const uint32_t* src, int nw, uint32_t* wv) {
    const int keff = nw < NT * KW ? (nw + NT - 1) / NT : KW;
    const int w0 = (int)(threadIdx.x / SPG_WAVE) * SPG_WAVE * keff + lane_id();
#pragma unroll
    for (int k = 0; k < KW; ++k) {
        const int w = w0 + k * SPG_WAVE;
        wv[k] = k < keff && w < nw ? __builtin_nontemporal_load(src + w) : 0u;
    }
}

// Ranks of a bitmap of nw words (at most 65535 set bits): bits[w] = word w,
// pfx[w] = set bits of all earlier words, and stage[r] = the column cbase +
// 32 w + b of the r-th set bit.  wv holds the words' first NT KW (from
// fetch_words); more are fetched here.  The counts are scanned in registers
// (a wave's words are consecutive), so one exchange of the wave totals through
// tot (NT / 64 words of LDS) is all that the waves wait for.  Contains
// barriers; the results are visible after the next one.
template <int NT, int KW>
__device__ inline void rank_words(const uint32_t* src, int nw, uint32_t* wv, uint32_t* bits, uint16_t* pfx,
                                  int32_t* stage, int32_t cbase, int32_t* tot) {
    constexpr int NW = NT / SPG_WAVE;
    const int lane = lane_id();
    const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / SPG_WAVE));
    int32_t before = 0;
    for (int t0 = 0; t0 < nw; t0 += NT * KW) {
        const int tw = nw - t0;
        const int keff = tw < NT * KW ? (tw + NT - 1) / NT : KW;
        if (t0 > 0) {
            fetch_words<NT, KW>(src + t0, tw, wv);
            __syncthreads();  // the last tile's totals are read
        }
        int32_t pre[KW], run = 0;
#pragma unroll
        for (int k = 0; k < KW; ++k) {
            if (k >= keff) break;
            const int32_t pc = __popc(wv[k]);
            const int32_t inc = wave_inclusive_scan_add(pc);
            pre[k] = run + inc - pc;
            run += __builtin_amdgcn_readlane(inc, SPG_WAVE - 1);
        }
        if (lane == 0) tot[wid] = run;
        __syncthreads();
        const int32_t wt = lane < NW ? tot[lane] : 0;
        const int32_t ws = wave_inclusive_scan_add(wt);
        const int32_t wbase = before + __builtin_amdgcn_readlane(ws - wt, wid);
        before += __builtin_amdgcn_readlane(ws, NW - 1);
        const int w0 = t0 + wid * SPG_WAVE * keff + lane;
#pragma unroll
        for (int k = 0; k < KW; ++k) {
            const int w = w0 + k * SPG_WAVE;
            if (k >= keff) break;
            if (w >= nw) break;
            uint32_t b = wv[k];
            int32_t r = wbase + pre[k];
            bits[w] = b;
            pfx[w] = (uint16_t)r;
            const int32_t c = cbase + w * 32;
            while (b) {
                stage[r++] = c + __builtin_ctz(b);
                b &= b - 1;
            }
        }
    }
}

// The staged columns to out[0, cnt), consecutive threads on consecutive
// positions, leaving the accumulators acc[0, cnt), whose bytes held them, zero.
template <int NT, typename V>
__device__ inline void write_staged_cols(V* acc, int32_t cnt, int32_t* out) {
    const int32_t* stage = reinterpret_cast<const int32_t*>(acc);
    // accumulator e holds staged positions [K e, K e + K): one thread reads
    // them, stores them (one store when all K are outputs) and clears the
    // accumulator; four of them are read before any is stored
    constexpr int K = (int)(sizeof(V) / sizeof(int32_t));
    static_assert(K == 1 || K == 2, "4- or 8-byte accumulators");
    constexpr int U = 4;
    for (int e0 = threadIdx.x; K * e0 < cnt; e0 += U * NT) {
        int32_t c[U][K];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int r = K * (e0 + u * NT) + k;
                c[u][k] = stage[r < cnt ? r : 0];
            }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = K * (e0 + u * NT);
            if (r + K <= cnt) {
#pragma unroll
                for (int k = 0; k < K; ++k) __builtin_nontemporal_store(c[u][k], out + r + k);
            } else if (r < cnt) {
                __builtin_nontemporal_store(c[u][0], out + r);
            }
        }
    }
    __syncthreads();  // every staged column is read
    for (int e = threadIdx.x; e < cnt; e += NT) acc[e] = V(0);
}

// The accumulators acc[0, cnt) to out[off, off + cnt), four read before any
// is stored.
template <int SR, int NT>
__device__ inline void write_values(const typename Sr<SR>::acc_t* acc, int32_t cnt, void* out, int64_t off) {
    typedef typename Sr<SR>::acc_t V;
    constexpr int U = 4;
    for (int r0 = threadIdx.x; r0 < cnt; r0 += U * NT) {
        V v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = acc[r0 + u * NT < cnt ? r0 + u * NT : 0];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (r0 + u * NT < cnt) Sr<SR>::store_stream(out, off + r0 + u * NT, v[u]);
    }
}

// Dynamic LDS: `cap` accumulators, then nwords bitmap words and their 16-bit
// prefixes (6 bytes per 32 columns: with 8, the packed words kept a third
// workgroup per CU out at 65536 columns and 4096 outputs).
template <int SR, int NT, int GM>
__global__ void __launch_bounds__(NT) k_num_rank(Csr A, Csr B, const int32_t* rows,
                                                 const int64_t* a_beg, const int64_t* a_end,
                                                 const uint32_t* bm_save, const int32_t* heavy_idx,
                                                 int32_t nwords, int32_t cap, OutRows c_rp, int32_t* c_col,
                                                 void* c_val) {
    typedef Sr<SR> S;
    typedef typename S::acc_t V;
    constexpr int KW = 4;  // bitmap words per thread held in registers
    extern __shared__ uint64_t dyn[];
    V* acc = reinterpret_cast<V*>(dyn);
    uint32_t* bits = reinterpret_cast<uint32_t*>(acc + cap);
    uint16_t* pfx = reinterpret_cast<uint16_t*>(bits + nwords);
    __shared__ V s_av[ProductLds<NT>::EB];
    __shared__ ProductLds<NT> L;
    __shared__ int32_t tot[NT / SPG_WAVE];
    const int64_t i = rows[blockIdx.x];
    const int64_t off = c_rp.off(i);
    const int32_t cnt = (int32_t)c_rp.count(i);
    const uint32_t* src = bm_save + (int64_t)heavy_idx[i] * nwords;
    uint32_t wv[KW];
    fetch_words<NT, KW>(src, nwords, wv);
    rank_words<NT, KW>(src, nwords, wv, bits, pfx, reinterpret_cast<int32_t*>(acc), 0, tot);
    __syncthreads();
    write_staged_cols<NT>(acc, cnt, c_col + off);
    __syncthreads();
    for_each_product_gm<NT, GM>(
        a_beg[i], a_end[i], L,
        [&](int64_t p, int64_t& bs, int32_t& len) {
            int64_t k = A.col[p];
            bs = B.rp[k];
            len = (int32_t)(B.rp[k + 1] - bs);
        },
        [&](int t, int64_t p) { s_av[t] = S::load(A.val, p); },
        [&](int64_t q) { return BEntry<V>{B.col[q], S::load(B.val, q)}; },
        [&](int t, const BEntry<V>& x) {
            const uint32_t j = (uint32_t)x.col;
            const int32_t rank = (int32_t)pfx[j >> 5] + __popc(bits[j >> 5] & ((1u << (j & 31)) - 1u));
            return BEntry<V>{rank, S::mul(s_av[t], x.val)};
        },
        [&](const BEntry<V>& y) {
            if (y.col < cnt) S::lds_add(&acc[y.col], y.val);
        });
    if (c_val) write_values<SR, NT>(acc, cnt, c_val, off);
}

// static LDS of k_num_rank<*, 512> and <*, 1024> (A values, product offsets, scan scratch), with margin
constexpr int RANK_STATIC_LDS = (int)(8 * 512 + sizeof(ProductLds<512>) + 4 * 16 + 256);
constexpr int RANK_STATIC_LDS_1024 = (int)(8 * 1024 + sizeof(ProductLds<1024>) + 4 * 32 + 256);

// Threads of k_num_rank at `lds` bytes of dynamic LDS: what the option asks for,
// or (0) 512, and 1024 where a CU holds only one workgroup of 512.
inline int rank_threads(int32_t rank_block, int64_t lds, int64_t max_lds) {
    const bool one = 2 * (lds + RANK_STATIC_LDS) > max_lds;
    const bool wide = rank_block == 1024 || (rank_block == 0 && one);
    return wide && lds + RANK_STATIC_LDS_1024 <= max_lds ? 1024 : 512;
}

// Rank chunks: the rows of the bitmap pass that are too large for the
// per-row rank kernel.  A row's column chunks of W columns (counts recorded
// by the bitmap pass) are grouped greedily into items of at most RC outputs
// and at most G chunks; an item accumulates in LDS at index = rank inside
// the item, with its B segments taken from the split table.
struct RankItem {
    int32_t row;    // the row
    int32_t slot;   // its saved bitmap
    int32_t c0, c1; // chunk range [c0, c1)
    int32_t cnt;    // outputs of the item
    int32_t annz;   // the row's A entries
    int64_t a_beg;  // the first of them
    int64_t roff;   // outputs of the row before the item
};

__device__ inline RankItem uniform_item(const RankItem& x) {
    return RankItem{uniform32(x.row), uniform32(x.slot), uniform32(x.c0), uniform32(x.c1), uniform32(x.cnt),
                    uniform32(x.annz), uniform64(x.a_beg), uniform64(x.roff)};
}

// Size of the rank-chunk items: at most RC outputs over at most G chunks of W
// columns, so that an item holds about RC outputs at the bin's mean density
// (cnnz outputs over nr rows of `chunks` chunks).  An item's fixed work (its
// bitmap, its A entries' B segments, its barriers) and the partly used cache
// lines at both ends of each B segment weigh less the larger it is, so RC
// grows from 4096 (at least W: a chunk may be full) as long as the same
// number of workgroups fits a CU's LDS.  R-MAT scale 19 (G = 26): RC 4096
// 53.4 ms, 5120 49.6, 5376 with one workgroup per CU 71.5 (whole product);
// scale 16: 4096 and 4608 the same.  Integer arithmetic, so the host (sizing
// the launch) and the device (forming the items) agree.
constexpr int RANKC_NT = 512;
constexpr int64_t RANKC_STATIC_LDS = (int64_t)(8 * ProductLds<RANKC_NT>::EB + sizeof(ProductLds<RANKC_NT>) +
                                               4 * (RANKC_NT / SPG_WAVE) + sizeof(RankItem)) + 64;
// the dynamic LDS their kernel may take: declared to the runtime, and what bounds an item's size
__host__ __device__ inline int64_t rankc_dyn_lds(int64_t max_lds) { return max_lds - RANKC_STATIC_LDS; }
struct RankShape {
    int32_t RC, G;
};
__host__ __device__ inline RankShape rankc_shape(int64_t nr, int64_t cnnz, int32_t chunks, int32_t chunk_group, int32_t W,
                                                 int64_t max_lds) {
    auto group = [&](int64_t RC) {
        int64_t G = cnnz > 0 ? (2 * RC * nr * chunks + cnnz) / (2 * cnnz) : chunks;
        if (G > chunks) G = chunks;
        if (G > chunk_group) G = chunk_group;
        return G < 1 ? (int64_t)1 : G;
    };
    auto lds = [&](int64_t RC, int64_t G) { return RC * 8 + G * (W / 32) * 6 + RANKC_STATIC_LDS; };
    int64_t RC = W > 4096 ? W : 4096;
    int64_t G = group(RC);
    while (G > 1 && lds(RC, G) > max_lds) --G;
    int64_t wg = max_lds / lds(RC, G);  // workgroups per CU, at most 4 by their threads
    if (wg < 1) wg = 1;
    if (wg > 4) wg = 4;
    constexpr int64_t STEP = 512;
    while (G < chunks && G < chunk_group && RC + STEP < 65536 && lds(RC + STEP, group(RC + STEP)) * wg <= max_lds) {
        RC += STEP;
        G = group(RC);
    }
    return RankShape{(int32_t)RC, (int32_t)G};
}

// Work items of the rank-chunk bin, located on the device (counts of the
// numeric classification): each row's chunks grouped greedily into items
// of at most RC outputs and G chunks.
__global__ void __launch_bounds__(256) k_rank_items(BinRef ref, const int64_t* a_beg, const int64_t* a_end,
                                                    const int32_t* heavy_idx, const int32_t* chunk_cnt,
                                                    int32_t P, int32_t chunk_group, int32_t W, int64_t max_lds,
                                                    const int64_t* cnnz_of_bin,
                                                    RankItem* items, int32_t* nitems) {
    __shared__ int32_t tmp[256 / SPG_WAVE + 1];
    __shared__ int32_t s_base;
    const int32_t* rows;
    int64_t nrows;
    ref.locate(rows, nrows);
    const RankShape shape = rankc_shape(nrows, *cnnz_of_bin, P, chunk_group, W, max_lds);
    const int32_t RC = shape.RC, G = shape.G;
    for (int64_t r0 = (int64_t)blockIdx.x * 256; r0 < nrows; r0 += (int64_t)gridDim.x * 256) {
        const int64_t r = r0 + threadIdx.x;
        const int32_t row = r < nrows ? rows[r] : 0;
        const int32_t bslot = r < nrows ? heavy_idx[row] : 0;
        const int32_t* cc = r < nrows ? chunk_cnt + (int64_t)bslot * P : nullptr;
        const int64_t ab = r < nrows ? a_beg[row] : 0;
        const int32_t an = r < nrows ? (int32_t)(a_end[row] - ab) : 0;
        // the greedy grouping of the row's chunks, walked twice: to count the
        // items (one global add per workgroup reserves their slots), then to
        // write them; eight counts are loaded before any is looked at
        auto walk = [&](auto emit) {
            int64_t roff = 0;
            int c0 = 0;
            int32_t n = 0;  // outputs of chunks [c0, c)
            auto close = [&](int c1) {
                if (n > 0) emit(c0, c1, n, roff);
                roff += n;
                n = 0;
                c0 = c1;
            };
            for (int cb = 0; cb < P; cb += 8) {
                int32_t v[8];
#pragma unroll
                for (int x = 0; x < 8; ++x) v[x] = cb + x < P ? cc[cb + x] : 0;
#pragma unroll
                for (int x = 0; x < 8; ++x) {
                    const int c = cb + x;
                    if (c >= P) break;
                    // (the host keeps RC >= W, so a chunk alone always fits)
                    if (c > c0 && (c - c0 >= G || n + v[x] > RC)) close(c);
                    n += v[x];
                }
            }
            close(P);
        };
        int32_t mine = 0;
        if (cc) walk([&](int, int, int32_t, int64_t) { ++mine; });
        int32_t total;
        int32_t slot = block_exclusive_scan<256, int32_t>(mine, &total, tmp);
        if (threadIdx.x == 0) s_base = total ? atomicAdd(nitems, total) : 0;
        __syncthreads();
        slot += s_base;
        if (cc) walk([&](int c0, int c1, int32_t n, int64_t roff) { items[slot++] = RankItem{row, bslot, c0, c1, n, an, ab, roff}; });
        __syncthreads();
    }
}

// Dynamic LDS: RC values, then G*W/32 bitmap words and their 16-bit prefixes.
// The item after the current one is fetched ahead: its bitmap words and the
// A entries of its first batch are in registers, and the item after that on
// its way to LDS, before the current item's products are gathered.
// Bound by the traffic past L2 where B exceeds it and by latency elsewhere:
// R-MAT scale 19 (7.6G products, B = 96 MB) 45.6 -> 27.2 ms alone at 6.4 TB/s
// past L2 (copy rate 5.1); scale 16 (303M products) 1.13 -> 0.70 ms.  Before,
// an item began with four dependent loads, its ranks with a serial walk over
// LDS words, and each step that crossed segments with LDS reads; stores of C
// that stayed in L2 displaced B (1.97 -> 1.91 ms for the scale-16 product).
// Larger workgroups (768 and 1024 threads) gained nothing.
// Workgroup b runs on XCD b mod 8; blocks of `run` consecutive items go to one
// XCD, whose L2 then serves the lines that a row's items share (the ends of
// their B segments, the split table).
template <int SR, int NT, int GM, int KW>
__global__ void __launch_bounds__(NT) k_num_rankc(Csr A, Csr B, int32_t W, const uint32_t* bm_save, int32_t nwords,
                                                  const int32_t* split, int32_t P, const RankItem* items,
                                                  const int32_t* nitems, int32_t run, int32_t RC, int32_t G, OutRows c_rp,
                                                  int32_t* c_col, void* c_val) {
    typedef Sr<SR> S;
    typedef typename S::acc_t V;
    const int WPC = W / 32;  // bitmap words per chunk
    extern __shared__ uint64_t dyn[];
    V* acc = reinterpret_cast<V*>(dyn);                      // RC
    uint32_t* bits = reinterpret_cast<uint32_t*>(acc + RC);  // G * WPC
    uint16_t* pfx = reinterpret_cast<uint16_t*>(bits + G * WPC);
    constexpr int EB = ProductLds<NT>::EB;
    __shared__ V s_av[EB];
    __shared__ ProductLds<NT> L;
    __shared__ int32_t tot[NT / SPG_WAVE];
    __shared__ RankItem s_next;
    constexpr int ITEM_WORDS = (int)(sizeof(RankItem) / 4);
    const int wid = uniform32((int)(threadIdx.x / SPG_WAVE));
    const int32_t total_items = *nitems;
    const int32_t xx = blockIdx.x & 7, xs = gridDim.x >> 3;
    int32_t pos = blockIdx.x >> 3;
    auto item_at = [&](int32_t q) { return (q / run * 8 + xx) * run + q % run; };
    if (item_at(pos) >= total_items) return;
    // the last chunk of a row may be partial (n not a multiple of W): the
    // saved bitmap ends at nwords, so no word past it is read (columns of
    // the missing words are >= n and never looked up)
    auto words_of = [&](const RankItem& x) {
        const int full = (x.c1 - x.c0) * WPC, left = nwords - x.c0 * WPC;
        return full < left ? full : left;
    };
    auto bits_of = [&](const RankItem& x) { return bm_save + (int64_t)x.slot * nwords + (int64_t)x.c0 * WPC; };
    uint32_t wv[KW];
    int32_t ak = 0;
    V av = S::zero();
    int64_t noff = 0;
    auto fetch = [&](const RankItem& x) {
        fetch_words<NT, KW>(bits_of(x), words_of(x), wv);
        ak = 0;
        if ((int)threadIdx.x < x.annz) {
            const int64_t p = x.a_beg + threadIdx.x;
            ak = A.col[p];
            av = S::load(A.val, p);
        }
        noff = c_rp.off(x.row);
    };
    // word t of the item at position q, in thread t (the first item where q is past the list)
    auto item_word = [&](int32_t q) {
        const int32_t it = item_at(q);
        return (int)threadIdx.x < ITEM_WORDS
                   ? reinterpret_cast<const int32_t*>(items + (it < total_items ? it : 0))[threadIdx.x]
                   : 0;
    };
    auto put_item = [&](int32_t w) {
        if ((int)threadIdx.x < ITEM_WORDS) reinterpret_cast<int32_t*>(&s_next)[threadIdx.x] = w;
    };
    RankItem item = uniform_item(items[item_at(pos)]);
    fetch(item);
    put_item(item_word(pos + xs));
    __syncthreads();
    while (true) {
        const int c0 = item.c0, c1 = item.c1;
        const int32_t cnt = item.cnt < RC ? item.cnt : RC;
        const int32_t cbase = c0 * W;
        // B segment of an A entry: the B row's start, and the chunk range's
        // ends inside it (one chunk covers all columns without a split table)
        auto segment = [&](int64_t k, int64_t& rs, int64_t& lo, int64_t& hi) {
            rs = B.rp[k];
            if (split) {
                lo = split[k * (P + 1) + c0];
                hi = split[k * (P + 1) + c1];
            } else {
                lo = 0;
                hi = B.rp[k + 1] - rs;
            }
        };
        // loaded by whole waves (lanes without an entry: B row 0) and combined
        // only after the bitmap's ranks are laid out
        int64_t rs0 = 0, lo0 = 0, hi0 = 0;
        if (wid * SPG_WAVE < item.annz) segment(ak, rs0, lo0, hi0);
        const V av0 = av;
        const int64_t off = uniform64(noff) + item.roff;
        const RankItem next = uniform_item(s_next);
        pos += xs;
        const bool more = item_at(pos) < total_items;
        rank_words<NT, KW>(bits_of(item), words_of(item), wv, bits, pfx, reinterpret_cast<int32_t*>(acc), cbase, tot);
        __syncthreads();
        write_staged_cols<NT>(acc, cnt, c_col + off);
        if (more) fetch(next);
        const int32_t nw = item_word(pos + xs);
        __syncthreads();
        const int64_t first_end = item.a_beg + EB;
        for_each_product_gm<NT, GM>(
            item.a_beg, item.a_beg + item.annz, L,
            [&](int64_t p, int64_t& bs, int32_t& len) {
                int64_t rs = rs0, lo = lo0, hi = hi0;
                if (p >= first_end) segment(A.col[p], rs, lo, hi);
                bs = rs + lo;
                len = (int32_t)(hi - lo);
            },
            [&](int t, int64_t p) { s_av[t] = p < first_end ? av0 : S::load(A.val, p); },
            [&](int64_t q) { return BEntry<V>{B.col[q], S::load(B.val, q)}; },
            [&](int t, const BEntry<V>& x) {
                const uint32_t j = (uint32_t)(x.col - cbase);
                const int32_t rank = (int32_t)pfx[j >> 5] + __popc(bits[j >> 5] & ((1u << (j & 31)) - 1u));
                return BEntry<V>{rank, S::mul(s_av[t], x.val)};
            },
            [&](const BEntry<V>& y) {
                if (y.col < RC) S::lds_add(&acc[y.col], y.val);
            });
        if (c_val)
            write_values<SR, NT>(acc, cnt, c_val, off);
        if (!more) break;
        put_item(nw);
        __syncthreads();
        item = next;
    }
}

}  // namespace spg
