// Batched products: many independent instances are multiplied as one
// block-diagonal product.  The instances' CSR matrices are copied side by
// side into one CSR (row pointers shifted by the entries before the
// instance, column indices shifted by the columns before it), so every
// row-binned launch covers the rows of all instances at once and the
// binning balances uneven instances.  Results are split back per instance.
// Used for the Galerkin products R^T A R of multigrid restriction (the
// restriction experiments of Section 5.3), one instance per grid.
#pragma once
#include "common.hpp"

namespace spg {

struct BatchDesc {
    const int64_t* rp;
    const int32_t* col;
    const void* val;
    int64_t nrows;
    int64_t row_off;  // first row of the instance in the batch
    int64_t nz_off;   // first entry of the instance in the batch
    int64_t col_off;  // first column of the instance in the batch
};

// Largest b with d[b].row_off <= r (instances with no rows share the
// offset of the next instance and are skipped).
__device__ inline int find_instance(const BatchDesc* d, int32_t nb, int64_t r) {
    int lo = 0, hi = nb;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (d[mid].row_off <= r) lo = mid; else hi = mid;
    }
    return lo;
}

constexpr int BATCH_LDS_MAX = 1024;  // instances whose offsets fit the LDS tables

__device__ inline int find_sorted(const int64_t* off, int32_t nb, int64_t x) {
    int lo = 0, hi = nb;  // largest b with off[b] <= x
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (off[mid] <= x) lo = mid; else hi = mid;
    }
    return lo;
}

// The batch's row pointers (shifted by the entries before the row's instance)
// and entries (columns shifted by the columns before it, values copied).  vw =
// value bytes (8 or 1; 0 = no values); structure = 0: the row pointers and
// columns are in place from an earlier call with the same instances and only
// the values are copied.
//
// Bound by memory, so the entries are taken BATCH_TILE at a time with the loads
// of a thread in flight together: one search per tile, and where the tile lies
// in one instance (nearly always) one base address for all of it.  Three
// operands of 64 grids of 16^3 ... 64^3 points, values only: 275 us with a
// search and one load at a time per thread, 155 so.
constexpr int BATCH_U = 8;
constexpr int BATCH_TILE = 256 * BATCH_U;

template <typename V>
__device__ inline void assemble_entries(const BatchDesc* d, int32_t nb, const int64_t* s_nz, bool lds, int64_t base,
                                        int64_t nnz, bool structure, int32_t* col, V* val) {
    auto first = [&](int b) { return lds ? s_nz[b] : d[b].nz_off; };
    int b = 0;  // the tile's first entry: the same address for every thread
    if (lds) {
        b = find_sorted(s_nz, nb, base);
    } else {
        for (int lo = 0, hi = nb; hi - lo > 1; b = lo) {
            const int mid = (lo + hi) >> 1;
            if (d[mid].nz_off <= base) lo = mid; else hi = mid;
        }
    }
    const int64_t tile_end = base + BATCH_TILE < nnz ? base + BATCH_TILE : nnz;
    int64_t x[BATCH_U];
    V v[BATCH_U];
    int32_t c[BATCH_U];
    if (tile_end - base == BATCH_TILE && (b + 1 == nb || first(b + 1) >= tile_end)) {
        const BatchDesc& D = d[b];
        const int64_t e = base - D.nz_off + D.rp[0] + threadIdx.x;
        const V* sv = (const V*)D.val;
#pragma unroll
        for (int u = 0; u < BATCH_U; ++u) {
            if (structure) c[u] = D.col[e + u * 256];
            if (val) v[u] = sv ? sv[e + u * 256] : V(1);
        }
#pragma unroll
        for (int u = 0; u < BATCH_U; ++u) {
            x[u] = base + u * 256 + threadIdx.x;
            if (structure) col[x[u]] = (int32_t)(c[u] + D.col_off);
            if (val) val[x[u]] = v[u];
        }
        return;
    }
#pragma unroll
    for (int u = 0; u < BATCH_U; ++u) {
        x[u] = base + u * 256 + threadIdx.x;
        if (x[u] >= tile_end) break;
        while (b + 1 < nb && first(b + 1) <= x[u]) ++b;
        const BatchDesc& D = d[b];
        const int64_t e = x[u] - D.nz_off + D.rp[0];
        if (structure) col[x[u]] = (int32_t)(D.col[e] + D.col_off);
        if (val) val[x[u]] = D.val ? ((const V*)D.val)[e] : V(1);
    }
}

__global__ void __launch_bounds__(256) k_batch_assemble(const BatchDesc* d, int32_t nb, int64_t rows, int64_t nnz,
                                                        int32_t vw, int32_t structure, int64_t* rp, int32_t* col,
                                                        void* val) {
    // the instances' first entries and rows, staged for the searches
    __shared__ int64_t s_row[BATCH_LDS_MAX], s_nz[BATCH_LDS_MAX];
    const bool lds = nb <= BATCH_LDS_MAX;
    if (lds)
        for (int b = threadIdx.x; b < nb; b += 256) {
            s_row[b] = d[b].row_off;
            s_nz[b] = d[b].nz_off;
        }
    __syncthreads();
    if (structure)
        for (int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x; x <= rows; x += (int64_t)gridDim.x * 256) {
            if (x == rows) {
                rp[rows] = nnz;
            } else {
                const BatchDesc& D = d[lds ? find_sorted(s_row, nb, x) : find_instance(d, nb, x)];
                rp[x] = D.nz_off + (D.rp[x - D.row_off] - D.rp[0]);
            }
        }
    for (int64_t base = (int64_t)blockIdx.x * BATCH_TILE; base < nnz; base += (int64_t)gridDim.x * BATCH_TILE) {
        if (vw == 8) assemble_entries<uint64_t>(d, nb, s_nz, lds, base, nnz, structure, col, (uint64_t*)val);
        else assemble_entries<uint8_t>(d, nb, s_nz, lds, base, nnz, structure, col, vw == 1 ? (uint8_t*)val : nullptr);
    }
}

// Split the batch product back: per-instance row pointers starting at 0
// (instance b's rows at out_rp[row_off_b + b ...]) and column indices made
// local to the instance (in place).
__global__ void __launch_bounds__(256) k_batch_split(const BatchDesc* d, int32_t nb, int64_t rows, const int64_t* rp,
                                                     int32_t* col, int64_t* out_rp) {
    const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (r >= rows) return;
    const int b = find_instance(d, nb, r);
    const BatchDesc& D = d[b];
    const int64_t i = r - D.row_off;
    const int64_t base = rp[D.row_off];
    out_rp[D.row_off + b + i] = rp[r] - base;
    if (i == D.nrows - 1) out_rp[D.row_off + b + i + 1] = rp[r + 1] - base;
    for (int64_t p = rp[r]; p < rp[r + 1]; ++p) col[p] = (int32_t)(col[p] - D.col_off);
}

}  // namespace spg
