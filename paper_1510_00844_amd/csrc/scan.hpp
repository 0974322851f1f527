// Device prefix sum of int64 row counts into CSR row pointers: in place over
// rp[1..m] (inclusive), with rp[0] = 0.  Two launches: per-tile sums, then
// per-tile scans in which every workgroup adds up the tiles before its own
// (up to SCAN_SELF tiles; above that a launch in between scans the sums).  The
// arrays are short, so what they cost is launches: three launches and a fill
// took 21 us where two take 10 (65,536 rows).
#pragma once
#include "common.hpp"

namespace spg {

constexpr int SCAN_NT = 1024;
constexpr int SCAN_PER = 4;
constexpr int SCAN_TILE = SCAN_NT * SCAN_PER;
constexpr int64_t SCAN_SELF = 4096;

__global__ void __launch_bounds__(SCAN_NT) k_scan_tiles(const int64_t* in, int64_t n, int64_t* tile_sums) {
    __shared__ int64_t red[SCAN_NT / SPG_WAVE + 1];
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + threadIdx.x;
    int64_t s = 0;
#pragma unroll
    for (int x = 0; x < SCAN_PER; ++x)
        if (base + x * SCAN_NT < n) s += in[base + x * SCAN_NT];
    int64_t total = block_reduce_add<SCAN_NT, int64_t>(s, red);
    if (threadIdx.x == 0) tile_sums[blockIdx.x] = total;
}

// Exclusive scan of ntiles sums in place by one workgroup.
__global__ void __launch_bounds__(SCAN_NT) k_scan_top(int64_t* tile_sums, int64_t ntiles) {
    __shared__ int64_t red[SCAN_NT / SPG_WAVE + 1];
    int64_t carry = 0;
    for (int64_t base = 0; base < ntiles; base += SCAN_NT) {
        const int64_t idx = base + threadIdx.x;
        const int64_t v = idx < ntiles ? tile_sums[idx] : 0;
        int64_t total;
        const int64_t ex = block_exclusive_scan<SCAN_NT, int64_t>(v, &total, red);
        if (idx < ntiles) tile_sums[idx] = ex + carry;
        carry += total;
    }
}

// rp[x + 1] = sums of the tiles before + inclusive prefix inside the tile, in
// place; rp[0] = 0.  scanned: tile_sums holds the tiles' offsets already.
__global__ void __launch_bounds__(SCAN_NT) k_scan_apply(int64_t* rp, int64_t n, const int64_t* tile_sums, int scanned) {
    __shared__ int64_t red[SCAN_NT / SPG_WAVE + 1];
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_PER;
    int64_t* cnt = rp + 1;
    int64_t before = 0;
    if (scanned) before = threadIdx.x == 0 ? tile_sums[blockIdx.x] : 0;
    else
        for (int64_t t = threadIdx.x; t < (int64_t)blockIdx.x; t += SCAN_NT) before += tile_sums[t];
    int64_t v[SCAN_PER];
    int64_t s = 0;
#pragma unroll
    for (int x = 0; x < SCAN_PER; ++x) {
        v[x] = base + x < n ? cnt[base + x] : 0;
        s += v[x];
    }
    int64_t off, total;
    (void)block_exclusive_scan<SCAN_NT, int64_t>(before, &off, red);
    int64_t pre = block_exclusive_scan<SCAN_NT, int64_t>(s, &total, red) + off;
#pragma unroll
    for (int x = 0; x < SCAN_PER; ++x) {
        pre += v[x];
        if (base + x < n) cnt[base + x] = pre;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) rp[0] = 0;
}

}  // namespace spg
