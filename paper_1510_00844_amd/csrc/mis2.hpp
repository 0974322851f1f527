// Distance-2 maximal independent sets and the aggregation that builds a
// restriction operator from them (Section 5.3, Algorithm 3).  Vectors are
// dense on the device: an absent entry of the algorithm's sparse vectors is
// the largest 64-bit key (or a zero flag).  Every row operation uses 8 lanes
// per row, so rows of any length are handled and short rows (stencils)
// still fill the waves.
#pragma once
#include "common.hpp"

namespace spg {

constexpr uint64_t MIS_ABSENT = ~0ull;
constexpr int MIS_LANES = 8;  // lanes per row

// SplitMix64 (Steele, Lea, Flood): the output for generator state x, i.e.
// the state advanced by the golden gamma and passed through the mixer.
__device__ inline uint64_t splitmix64_output(uint64_t x) {
    uint64_t z = x + 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Round-r key of vertex v: random high half, the vertex id as the low half
// (keys never tie).
__device__ inline uint64_t mis_key(uint64_t seed, int32_t round, int64_t v) {
    const uint64_t h = splitmix64_output(seed ^ (((uint64_t)(uint32_t)round << 32) | (uint64_t)v));
    return (h & 0xFFFFFFFF00000000ull) | (uint64_t)v;
}

// Key by which an unassigned vertex v ranks an assigned neighbour u.
__device__ inline uint64_t choice_key(uint64_t seed, int64_t v, int64_t u) {
    return splitmix64_output(seed ^ 0x5DEECE66D2B9A1F3ull ^ (((uint64_t)v << 32) | (uint64_t)u));
}

template <typename T, class Op>
__device__ inline T group_reduce(T v, Op op) {
#pragma unroll
    for (int d = MIS_LANES / 2; d > 0; d >>= 1) v = op(v, __shfl_xor(v, d, SPG_WAVE));
    return v;
}

// The four kernels of a round return at once when the round before left no
// candidate (*live == 0), so rounds can be queued without reading the flag
// back.  They are bound by the latency of the gathers; candidates are one byte
// each and their keys are computed where they are read (a 64-bit mixer costs
// less than gathering 8 bytes instead of 1), and rows whose result is settled
// (no candidate) gather nothing.  7-point grid of 75^3 points, six rounds: the
// last kernel 804 -> 25 us (it counted the remaining candidates with an atomic
// per wave on one address; a flag is enough), the others 240 -> 165 us.

// y(i) = min over stored A(i,j) of the candidates' keys x(j)   (semiring (min, select2nd))
__global__ void __launch_bounds__(256) k_mis_row_min(Csr A, const uint8_t* cand, uint64_t seed, int32_t round,
                                                     const int32_t* live, uint64_t* y) {
    if (*live == 0) return;
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) / MIS_LANES;
    const int gl = threadIdx.x % MIS_LANES;
    uint64_t m = MIS_ABSENT;
    if (i < A.nrows)
        for (int64_t p = A.rp[i] + gl; p < A.rp[i + 1]; p += MIS_LANES) {
            const int64_t j = A.col[p];
            if (cand[j]) {
                const uint64_t t = mis_key(seed, round, j);
                m = t < m ? t : m;
            }
        }
    m = group_reduce(m, [](uint64_t a, uint64_t b) { return a < b ? a : b; });
    if (i < A.nrows && gl == 0) y[i] = m;
}

// Second hop and selection: minadj = min(m1(i), min over A(i,j) of m1(j));
// a candidate whose key is not larger joins (newS).  It stops being a
// candidate in the pruning (the row minima of this round are read there no more).
__global__ void __launch_bounds__(256) k_mis_select(Csr A, const uint8_t* cand, uint64_t seed, int32_t round,
                                                    const int32_t* live, const uint64_t* m1, uint8_t* news) {
    if (*live == 0) return;
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) / MIS_LANES;
    const int gl = threadIdx.x % MIS_LANES;
    const bool c = i < A.nrows && cand[i] != 0;
    uint64_t m = MIS_ABSENT;
    if (c)
        for (int64_t p = A.rp[i] + gl; p < A.rp[i + 1]; p += MIS_LANES) {
            const uint64_t t = m1[A.col[p]];
            m = t < m ? t : m;
        }
    m = group_reduce(m, [](uint64_t a, uint64_t b) { return a < b ? a : b; });
    if (i < A.nrows && gl == 0) {
        bool joins = false;
        if (c) {
            const uint64_t mn = m1[i] < m ? m1[i] : m;
            joins = mis_key(seed, round, i) <= mn;
        }
        news[i] = joins ? 1 : 0;
    }
}

// y(i) = OR over stored A(i,j) of x(j)
__global__ void __launch_bounds__(256) k_mis_row_any(Csr A, const int32_t* live, const uint8_t* x, uint8_t* y) {
    if (*live == 0) return;
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) / MIS_LANES;
    const int gl = threadIdx.x % MIS_LANES;
    int hit = 0;
    if (i < A.nrows)
        for (int64_t p = A.rp[i] + gl; p < A.rp[i + 1] && !hit; p += MIS_LANES) hit = x[A.col[p]] ? 1 : 0;
    hit = group_reduce(hit, [](int a, int b) { return a | b; });
    if (i < A.nrows && gl == 0) y[i] = (uint8_t)hit;
}

// Second hop of the new vertices' neighbourhood, pruning of the candidates
// (the new vertices among them), MIS-2 update, and *left = 1 when a candidate
// remains.
__global__ void __launch_bounds__(256) k_mis_prune(Csr A, const int32_t* live, const uint8_t* a1, const uint8_t* news,
                                                   uint8_t* cand, uint8_t* in_mis, int32_t* left) {
    if (*live == 0) return;
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) / MIS_LANES;
    const int gl = threadIdx.x % MIS_LANES;
    const bool c = i < A.nrows && cand[i] != 0;
    int hit = 0;
    if (c)
        for (int64_t p = A.rp[i] + gl; p < A.rp[i + 1] && !hit; p += MIS_LANES) hit = a1[A.col[p]] ? 1 : 0;
    hit = group_reduce(hit, [](int a, int b) { return a | b; });
    bool stays = false;
    if (c && gl == 0) {
        const bool joined = news[i] != 0;
        if (joined) in_mis[i] = 1;
        stays = !(joined || hit || a1[i]);
        if (!stays) cand[i] = 0;
    }
    if (__ballot(stays) && lane_id() == 0) *left = 1;
}

// flags[v + 1] = in_mis(v), for the exclusive scan that numbers the roots
__global__ void __launch_bounds__(256) k_mis_flags(int64_t n, const uint8_t* in_mis, int64_t* flags) {
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (v < n) flags[v + 1] = in_mis[v] ? 1 : 0;
}

// Roots take their number; their neighbours join them (a vertex is adjacent
// to at most one root); others stay -1.
__global__ void __launch_bounds__(256) k_agg_roots(Csr A, const uint8_t* in_mis, const int64_t* root_id,
                                                   int32_t* agg1) {
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) / MIS_LANES;
    const int gl = threadIdx.x % MIS_LANES;
    int64_t r = -1;
    if (i < A.nrows && !in_mis[i])
        for (int64_t p = A.rp[i] + gl; p < A.rp[i + 1]; p += MIS_LANES) {
            const int64_t j = A.col[p];
            if (in_mis[j]) r = j > r ? j : r;
        }
    r = group_reduce(r, [](int64_t a, int64_t b) { return a > b ? a : b; });
    if (i < A.nrows && gl == 0) agg1[i] = in_mis[i] ? (int32_t)root_id[i] : (r >= 0 ? (int32_t)root_id[r] : -1);
}

// Unassigned vertices join the assigned neighbour with the smallest
// (choice key, neighbour) pair; *unassigned counts any left over.
__global__ void __launch_bounds__(256) k_agg_rest(Csr A, const int32_t* agg1, uint64_t seed, int32_t* agg,
                                                  int32_t* unassigned) {
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) / MIS_LANES;
    const int gl = threadIdx.x % MIS_LANES;
    const bool need = i < A.nrows && agg1[i] < 0;
    uint64_t bk = MIS_ABSENT;
    int64_t bj = -1;
    if (need)
        for (int64_t p = A.rp[i] + gl; p < A.rp[i + 1]; p += MIS_LANES) {
            const int64_t j = A.col[p];
            if (agg1[j] < 0) continue;
            const uint64_t k = choice_key(seed, i, j);
            if (bj < 0 || k < bk || (k == bk && j < bj)) {
                bk = k;
                bj = j;
            }
        }
#pragma unroll
    for (int d = MIS_LANES / 2; d > 0; d >>= 1) {
        const uint64_t ok = __shfl_xor(bk, d, SPG_WAVE);
        const int64_t oj = __shfl_xor(bj, d, SPG_WAVE);
        if (oj >= 0 && (bj < 0 || ok < bk || (ok == bk && oj < bj))) {
            bk = ok;
            bj = oj;
        }
    }
    if (i < A.nrows && gl == 0) {
        const int32_t a = need ? (bj >= 0 ? agg1[bj] : -1) : agg1[i];
        agg[i] = a;
        if (a < 0) atomicAdd(unassigned, 1);
    }
}

// R (n x n_agg): one entry per row at the aggregate; counts of R^T's rows.
template <int SR>
__global__ void __launch_bounds__(256) k_restrict_rows(int64_t n, const int32_t* agg, int64_t* r_rp, int32_t* r_col,
                                                       void* r_val, int64_t* rt_cnt) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i > n) return;
    r_rp[i] = i;
    if (i == n) return;
    r_col[i] = agg[i];
    if (r_val) {
        if (SR == SR_F64) ((double*)r_val)[i] = 1.0;
        else if (SR == SR_I64) ((int64_t*)r_val)[i] = 1;
        else ((uint8_t*)r_val)[i] = 1;
    }
    atomicAdd((unsigned long long*)&rt_cnt[agg[i] + 1], 1ull);
}

// R^T: vertex i goes to row agg(i) (any order; rows are sorted afterwards).
template <int SR>
__global__ void __launch_bounds__(256) k_restrict_cols(int64_t n, const int32_t* agg, const int64_t* rt_rp,
                                                       int64_t* cursor, int32_t* rt_col, void* rt_val) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int32_t a = agg[i];
    const int64_t q = rt_rp[a] + (int64_t)atomicAdd((unsigned long long*)&cursor[a], 1ull);
    rt_col[q] = (int32_t)i;
    if (rt_val) {
        if (SR == SR_F64) ((double*)rt_val)[q] = 1.0;
        else if (SR == SR_I64) ((int64_t*)rt_val)[q] = 1;
        else ((uint8_t*)rt_val)[q] = 1;
    }
}

// Sort each row's column indices (values are all equal).  Rows of up to 64
// entries by a wave each in registers, up to SRC_WAVE in the wave's own LDS, four
// rows per workgroup; the longer rows have a kernel of their own (with their LDS
// in the same kernel only five waves fitted a CU: 53 -> 9 us for 75^3 points).
constexpr int SRC_WAVE = 256;
constexpr int SRC_MAX = 4096;  // longest row

__global__ void __launch_bounds__(256) k_sort_row_cols(int64_t nrows, const int64_t* rp, int32_t* col) {
    __shared__ uint32_t s_keys[4][SRC_WAVE];
    const int wv = threadIdx.x / SPG_WAVE;
    const int64_t r = (int64_t)blockIdx.x * 4 + wv;
    if (r >= nrows) return;  // whole waves; no block barriers below
    const int64_t s = rp[r];
    const int64_t len = rp[r + 1] - s;
    if (len > SRC_WAVE) return;
    const int lane = lane_id();
    if (len <= SPG_WAVE) {
        const uint32_t k = wave_bitonic_sort_u32(lane < len ? (uint32_t)col[s + lane] : 0xffffffffu, (int)len);
        if (lane < len) col[s + lane] = (int32_t)k;
        return;
    }
    uint32_t* keys = s_keys[wv];
    const int P = len <= 2 * SPG_WAVE ? 2 * SPG_WAVE : SRC_WAVE;
    for (int t = lane; t < P; t += SPG_WAVE) keys[t] = t < len ? (uint32_t)col[s + t] : 0xffffffffu;
    wave_lds_sync();
    wave_lds_bitonic_u32(keys, P);
    for (int t = lane; t < len; t += SPG_WAVE) col[s + t] = (int32_t)keys[t];
}

// The longer rows, a workgroup each; *too_long counts rows above SRC_MAX.  Every
// workgroup looks at the rows that lie gridDim.x apart from its own number on, 64
// at a time, so that neighbouring long rows go to different workgroups.  With 64
// neighbouring rows to a workgroup one after another, the whole call took 5.61 ms
// for 64 aggregates of 4096 and 0.43 ms for 1000 of 100; so 0.77 and 0.11 ms.
__global__ void __launch_bounds__(256) k_sort_long_row_cols(int64_t nrows, const int64_t* rp, int32_t* col,
                                                            int32_t* too_long) {
    __shared__ uint32_t keys[SRC_MAX];
    __shared__ uint64_t s_long;
    const int64_t step = gridDim.x;
    for (int64_t r0 = blockIdx.x; r0 < nrows; r0 += SPG_WAVE * step) {
        if (threadIdx.x < SPG_WAVE) {
            const int64_t r = r0 + threadIdx.x * step;
            const uint64_t m = __ballot(r < nrows && rp[r + 1] - rp[r] > SRC_WAVE);
            if (threadIdx.x == 0) s_long = m;
        }
        __syncthreads();
        for (uint64_t m = s_long; m; m &= m - 1) {
            const int64_t r = r0 + __builtin_ctzll(m) * step;
            const int64_t s = rp[r];
            const int64_t len = rp[r + 1] - s;
            if (len > SRC_MAX) {
                if (threadIdx.x == 0) atomicAdd(too_long, 1);
                continue;
            }
            int P = 2 * SRC_WAVE;
            while (P < len) P <<= 1;
            for (int t = threadIdx.x; t < P; t += 256) keys[t] = t < len ? (uint32_t)col[s + t] : 0xffffffffu;
            __syncthreads();
            block_bitonic_sort<256>(keys, P);
            for (int t = threadIdx.x; t < len; t += 256) col[s + t] = (int32_t)keys[t];
            __syncthreads();  // the row is done with the LDS
        }
        __syncthreads();  // s_long is read
    }
}

}  // namespace spg
