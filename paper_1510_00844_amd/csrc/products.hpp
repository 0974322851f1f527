// Enumerating the scalar products of one output row inside a workgroup.
//
// Row i of C gathers, for every stored A(i,k) in the window, the stored
// entries of B(k,:) (the row form of Algorithm 1).  B rows differ wildly in
// length (R-MAT hubs), so a batch of A entries is turned into a flat index
// space of products with a workgroup prefix sum of their B-segment lengths,
// and every wave (or thread) takes an equal contiguous range of that space (a
// merge path over the segment offsets).  No thread walks a long B row alone
// and no product pays for a search over all segments.
#pragma once
#include <cstdint>
#include "common.hpp"

namespace spg {

// A batch holds at most EB A entries, one per thread of the first EB threads.
// In workgroups of 512 or more threads the last wave brings none: the 20 bytes
// an entry (its value in the caller's LDS included) then leave room for a
// third workgroup per CU beside 4096 FP64 accumulators and a 65536-column
// bitmap (54.1 KB of 54.6).
template <int NT>
struct ProductLds {
    static constexpr int EB = NT >= 512 ? NT - SPG_WAVE : NT;
    int32_t off[EB + 1];        // first product of each segment, then their number
    int64_t bstart[EB];         // first B index of each segment
    int32_t tmp[2 * (NT / SPG_WAVE) + 1];
};

// seg(p, &bstart, &len): B index range [bstart, bstart+len) for A entry p.
// pre(t, p): called once per A entry of the batch before the products (for
// staging per-entry data in LDS at place t).  load(q) reads B entry q;
// apply(t, x) takes a product.  All threads of the block must call these.

// Thread-contiguous variant: thread t walks products [t*per, (t+1)*per).
template <int NT, int U, class Seg, class Pre, class Load, class Apply>
__device__ inline void for_each_product_t(int64_t a_beg, int64_t a_end, ProductLds<NT>& L, Seg seg,
                                          Pre pre, Load load, Apply apply) {
    typedef decltype(load((int64_t)0)) X;
    constexpr int EB = ProductLds<NT>::EB;
    for (int64_t base = a_beg; base < a_end; base += EB) {
        const int64_t p = base + threadIdx.x;
        int64_t bs = 0;
        int32_t len = 0;
        if ((int)threadIdx.x < EB && p < a_end) {
            seg(p, bs, len);
            pre((int)threadIdx.x, p);
        }
        int32_t total;
        int32_t off = block_exclusive_scan<NT, int32_t>(len, &total, L.tmp);
        if ((int)threadIdx.x < EB) {
            L.off[threadIdx.x] = off;
            L.bstart[threadIdx.x] = bs;
        }
        if (threadIdx.x == 0) L.off[EB] = total;
        __syncthreads();
        const int32_t per = (total + NT - 1) / NT;
        int32_t f = (int32_t)threadIdx.x * per;
        const int32_t fend = f + per < total ? f + per : total;
        if (f < fend) {
            int t = 0, hi = EB;
            while (hi - t > 1) {
                int mid = (t + hi) >> 1;
                if (L.off[mid] <= f) t = mid; else hi = mid;
            }
            int32_t seg_end = L.off[t + 1];
            int64_t q = L.bstart[t] + (f - L.off[t]);
            for (; f < fend; f += U) {
                int64_t qq[U];
                int tt[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (f + u < fend) {
                        while (f + u >= seg_end) {
                            ++t;
                            seg_end = L.off[t + 1];
                            q = L.bstart[t];
                        }
                        qq[u] = q++;
                        tt[u] = t;
                    }
                }
                X x[U];
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (f + u < fend) x[u] = load(qq[u]);
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (f + u < fend) apply(tt[u], x[u]);
            }
        }
        __syncthreads();
    }
}

// 64-bit value of lane l (l wave-uniform).
__device__ inline int64_t readlane_i64(int64_t v, int l) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), l);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// The 64 consecutive segments [base, base + 64) of a batch (all non-empty),
// one per lane: the registers a wave locates its products with.  `last` is
// the first product past the window (INT32_MAX when no segment lies past it).
struct SegWindow {
    int32_t base;  // wave-uniform
    int32_t last;  // wave-uniform
    int32_t off;   // first product of segment base + lane (INT32_MAX past the batch)
    int64_t rel;   // B index of product f of the segment = rel + f
};

template <int NT>
__device__ inline void load_window(const ProductLds<NT>& L, int32_t base, int32_t nseg, SegWindow& w) {
    const int j = base + lane_id();
    w.base = base;
    w.off = INT32_MAX;
    w.rel = 0;
    if (j < nseg) {
        w.off = L.off[j];
        w.rel = L.bstart[j] - w.off;
    }
    w.last = base + SPG_WAVE < nseg ? __builtin_amdgcn_readfirstlane(L.off[base + SPG_WAVE]) : INT32_MAX;
}

// A loaded B entry and its segment.
template <typename X>
struct SlotEntry {
    int t;
    X x;
};
template <typename X>
__device__ inline void pin(SlotEntry<X>&) {}  // its parts are pinned when loaded

// Same enumeration, mapped for coalesced gathers: each wave takes an equal
// contiguous range of the batch's products and its lanes take consecutive
// products, 64 at a time, so one load instruction reads 64 neighbouring B
// entries.  Empty segments are dropped when the batch is laid out in LDS
// (pre(t, p) gets the place t of A entry p among the others), so the starts
// strictly increase.  The wave holds a window of 64 segments in registers and
// the segment it is in (its lane of the window, its end, and the offset that
// turns a product number into a B index) in scalar registers.  A step inside
// that segment needs nothing else.  A step that crosses segment ends sets one
// bit per start in a scalar mask; the bits at or below a lane count the
// segments to move on, and two lane exchanges fetch that segment's offset.
// The window is read from LDS once per 64 segments: the steps of a range are
// a serial chain, and an LDS round trip in each of them would stand in front
// of every round of gathers.
// U steps are gathered (`load(q)`) before any is looked up (`look(t, x)`, the
// LDS reads a product needs), and all are looked up before any is committed
// (`commit(y)`), so each lane keeps U loads and U look-ups in flight.  Lanes
// past the range load and look up its last product and commit nothing.
// With COAL = false each thread instead takes its own contiguous range of
// products (one search per thread, U consecutive products per step): lanes
// then touch different segments, which spreads LDS atomics over more
// addresses at the price of uncoalesced gathers.
template <int NT, int U, bool COAL = true, bool DB = false, class Seg, class Pre, class Load, class Look, class Commit>
__device__ inline void for_each_product_lc(int64_t a_beg, int64_t a_end, ProductLds<NT>& L, Seg seg, Pre pre, Load load,
                                           Look look, Commit commit) {
    typedef decltype(load((int64_t)0)) X;
    typedef decltype(look(0, load((int64_t)0))) Y;
    if constexpr (!COAL) {
        for_each_product_t<NT, U>(a_beg, a_end, L, seg, pre, load, [&](int t, const X& x) { commit(look(t, x)); });
        return;
    }
    // segment starts inside one step up to which the scalar loop is used
    constexpr int LOOP_MAX = 32;
    constexpr int NW = NT / SPG_WAVE;
    constexpr int EB = ProductLds<NT>::EB;
    static_assert(NT % SPG_WAVE == 0 && NW <= SPG_WAVE, "whole waves");
    const int lane = lane_id();
    // wave-uniform values live in scalar registers (readfirstlane), so the
    // step bookkeeping below is scalar work and scalar branches
    const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / SPG_WAVE));
    for (int64_t base = a_beg; base < a_end; base += EB) {
        const int64_t p = base + threadIdx.x;
        int64_t bs = 0;
        int32_t len = 0;
        if ((int)threadIdx.x < EB && p < a_end) seg(p, bs, len);
        // products and non-empty segments before this thread's, and in all
        const int32_t inc = wave_inclusive_scan_add(len);
        const uint64_t full = __builtin_amdgcn_ballot_w64(len > 0);
        if (lane == SPG_WAVE - 1) {
            L.tmp[wid] = inc;
            L.tmp[NW + wid] = __popcll(full);
        }
        __syncthreads();
        const int32_t wlen = lane < NW ? L.tmp[lane] : 0, wseg = lane < NW ? L.tmp[NW + lane] : 0;
        const int32_t plen = wave_inclusive_scan_add(wlen), pseg = wave_inclusive_scan_add(wseg);
        const int32_t tot = __builtin_amdgcn_readlane(plen, NW - 1);
        const int32_t nseg = __builtin_amdgcn_readlane(pseg, NW - 1);
        const int32_t len_before = __builtin_amdgcn_readlane(plen - wlen, wid);
        const int32_t seg_before = __builtin_amdgcn_readlane(pseg - wseg, wid);
        if (len > 0) {
            const int t = seg_before + lanes_below(full);
            L.off[t] = len_before + inc - len;
            L.bstart[t] = bs;
            pre(t, p);
        }
        if (threadIdx.x == 0) L.off[nseg] = tot;
        __syncthreads();
        const int32_t span = (tot + NW - 1) / NW;
        const int32_t f0 = wid * span;
        const int32_t f1 = f0 + span < tot ? f0 + span : tot;
        if (f0 < f1) {
            // the window of the range start: every NW-th segment probed at
            // once (off[0] = 0 <= f0), then the last one starting at or before f0
            const int32_t probe = lane * NW < nseg ? L.off[lane * NW] : INT32_MAX;
            SegWindow w;
            load_window<NT>(L, (63 - __builtin_clzll(__builtin_amdgcn_ballot_w64(probe <= f0))) * NW, nseg, w);
            int cur = 0;  // the current segment's lane
            int64_t cur_rel = 0;
            int32_t cur_end = 0;
            auto enter = [&](int l) {
                cur = l;
                cur_rel = readlane_i64(w.rel, l);
                cur_end = l < SPG_WAVE - 1 ? __builtin_amdgcn_readlane(w.off, l + 1) : w.last;
            };
            enter(63 - __builtin_clzll(__builtin_amdgcn_ballot_w64(w.off <= f0)));
            // segment t and B entry q of this lane's product in the step that
            // starts at product fs (fs < f1); moves the segment state forward
            auto locate = [&](int32_t fs, int& t, int64_t& q) {
                const int32_t flast = fs + SPG_WAVE - 1 < f1 ? fs + SPG_WAVE - 1 : f1 - 1;
                const int32_t f = fs + lane < flast ? fs + lane : flast;
                t = w.base + cur;
                int64_t rel = cur_rel;
                if (flast >= cur_end) {
                    const int n = __popcll(__builtin_amdgcn_ballot_w64(w.off <= flast)) - 1;  // last start's lane
                    if (flast < w.last && n - cur <= LOOP_MAX) {
                        uint64_t starts = 0;
                        for (int l = cur + 1; l <= n; ++l)
                            starts |= 1ull << (__builtin_amdgcn_readlane(w.off, l) - fs);
                        const int l = cur + (int)(starts & 1) + lanes_below(starts >> 1);
                        t = w.base + l;
                        rel = lane_get(w.rel, l);
                        enter(n);
                    } else {
                        // many starts (short B rows), or past the window: each
                        // lane searches the batch, and the window moves on
                        int lo = w.base, hi = nseg;
                        while (hi - lo > 1) {
                            const int mid = (lo + hi) >> 1;
                            if (L.off[mid] <= f) lo = mid; else hi = mid;
                        }
                        t = lo;
                        rel = L.bstart[lo] - L.off[lo];
                        load_window<NT>(L, __builtin_amdgcn_readlane(lo, SPG_WAVE - 1), nseg, w);
                        enter(0);
                    }
                }
                q = rel + f;
            };
            auto fetch = [&](int32_t fb, X* x, int* tt) {
                int64_t qq[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int32_t fs = fb + u * SPG_WAVE;
                    // steps past the range repeat the last located product
                    if (fs < f1) {
                        locate(fs, tt[u], qq[u]);
                    } else if (u > 0) {
                        tt[u] = tt[u - 1];
                        qq[u] = qq[u - 1];
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u) x[u] = load(qq[u]);
            };
            auto drain = [&](int32_t fb, X* x, const int* tt) {
                Y y[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    pin(x[u]);
                    y[u] = look(tt[u], x[u]);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    pin(y[u]);
                    if (fb + u * SPG_WAVE + lane < f1) commit(y[u]);
                }
            };
            constexpr int32_t R = SPG_WAVE * U;
            X xa[U];
            int ta[U];
            if constexpr (!DB) {
                for (int32_t fb = f0; fb < f1; fb += R) {
                    fetch(fb, xa, ta);
                    drain(fb, xa, ta);
                }
            } else {
                // two rounds in flight: the gathers of the next round are
                // issued before the products of the current one are applied
                // (more registers, fewer waves: pays when the gathers miss L2)
                X xb[U];
                int tb[U];
                fetch(f0, xa, ta);
                for (int32_t fb = f0; fb < f1; fb += 2 * R) {
                    if (fb + R < f1) fetch(fb + R, xb, tb);
                    drain(fb, xa, ta);
                    if (fb + R >= f1) break;
                    if (fb + 2 * R < f1) fetch(fb + 2 * R, xa, ta);
                    drain(fb + R, xb, tb);
                }
            }
        }
        __syncthreads();
    }
}

// The same with one step per product: apply(t, x).
template <int NT, int U, bool COAL = true, bool DB = false, class Seg, class Pre, class Load, class Apply>
__device__ inline void for_each_product_u(int64_t a_beg, int64_t a_end, ProductLds<NT>& L, Seg seg, Pre pre, Load load,
                                          Apply apply) {
    typedef decltype(load((int64_t)0)) X;
    for_each_product_lc<NT, U, COAL, DB>(
        a_beg, a_end, L, seg, pre, load, [](int t, const X& x) { return SlotEntry<X>{t, x}; },
        [&](const SlotEntry<X>& y) { apply(y.t, y.x); });
}

// Gather mode of the heavy-row kernels (a tuning choice):
//   0: coalesced, 4 steps in flight   1: coalesced, 8 steps in flight
//   2: per-thread ranges, 4 in flight 3: per-thread ranges, 8 in flight
//   4: coalesced, two rounds of 4 steps in flight (double-buffered)
template <int NT, int GM, class Seg, class Pre, class Load, class Look, class Commit>
__device__ inline void for_each_product_gm(int64_t a_beg, int64_t a_end, ProductLds<NT>& L, Seg seg,
                                           Pre pre, Load load, Look look, Commit commit) {
    constexpr int U = GM == 1 || GM == 3 ? 8 : 4;
    for_each_product_lc<NT, U, GM != 2 && GM != 3, GM == 4>(a_beg, a_end, L, seg, pre, load, look, commit);
}
template <int NT, int GM, class Seg, class Pre, class Load, class Apply>
__device__ inline void for_each_product_gm(int64_t a_beg, int64_t a_end, ProductLds<NT>& L, Seg seg,
                                           Pre pre, Load load, Apply apply) {
    constexpr int U = GM == 1 || GM == 3 ? 8 : 4;
    for_each_product_u<NT, U, GM != 2 && GM != 3, GM == 4>(a_beg, a_end, L, seg, pre, load, apply);
}

// The products of one row by one wave, for rows whose products are few or
// whose B rows are short (no workgroup-wide enumeration, no barriers).  The
// row's A entries are taken 64 at a time: seg(p, bs, len, pa) gives lane
// p - base its B segment and a per-entry payload pa (the A value); a wave
// scan of the lengths gives the segment offsets.  The products are taken in
// rounds of U steps of 64: the lane of every non-empty segment is marked in
// LDS (64 U bytes of the wave's own) at the segment's first product of the
// round, and a running maximum of the marks over the round gives each product
// its segment (a binary search across the lanes took six exchanges a step).
// Each lane issues its U gathers (load(q)) before applying any (apply(pa, x)),
// so U loads are in flight.
template <int U, typename PA, class Seg, class Load, class Apply>
__device__ inline void wave_products(int64_t beg, int64_t end, uint8_t* marks, Seg seg, Load load, Apply apply) {
    typedef decltype(load((int64_t)0)) X;
    const int lane = lane_id();
    for (int64_t base = beg; base < end; base += SPG_WAVE) {
        const int64_t p = base + lane;
        int64_t bs = 0;
        int32_t len = 0;
        PA pa{};
        if (p < end) seg(p, bs, len, pa);
        const int32_t incl = wave_inclusive_scan_add(len);
        const int32_t off = incl - len;
        const int64_t rel = bs - off;
        const int32_t nb = __builtin_amdgcn_readlane(incl, SPG_WAVE - 1);
        for (int32_t x0 = 0; x0 < nb; x0 += SPG_WAVE * U) {
            static_assert(U == 4, "a word of marks per lane");
            reinterpret_cast<uint32_t*>(marks)[lane] = 0;
            wave_lds_sync();
            // a segment that began before the round is marked at its start
            const int32_t first = off > x0 ? off : x0;
            if (first < incl && first < x0 + SPG_WAVE * U) marks[first - x0] = (uint8_t)lane;
            wave_lds_sync();
            int32_t m[U];
#pragma unroll
            for (int u = 0; u < U; ++u) m[u] = marks[u * SPG_WAVE + lane];
            wave_lds_sync();  // read before the next round clears them
            PA a[U];
            X v[U];
            int32_t carry = 0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                int32_t l = wave_inclusive_scan_max(m[u]);
                l = l > carry ? l : carry;
                carry = __builtin_amdgcn_readlane(l, SPG_WAVE - 1);
                const int32_t x = x0 + u * SPG_WAVE + lane;
                // products past the batch load its last one and apply nothing
                const int64_t q = lane_get(rel, l) + (x < nb ? x : nb - 1);
                a[u] = lane_get(pa, l);
                v[u] = load(q);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                pin(v[u]);
                if (x0 + u * SPG_WAVE + lane < nb) apply(a[u], v[u]);
            }
        }
    }
}

}  // namespace spg
