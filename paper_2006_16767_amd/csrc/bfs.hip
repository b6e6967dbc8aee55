// Breadth-first search driver: every level is one adaptive (OR, AND)
// SpMSpV of the frontier (the application the paper evaluates its kernels
// in, Section 7), so the kernel follows the frontier's density from level
// to level. A level's product y = A (x) f marks every vertex with an edge
// from the frontier; the update kernel keeps the unvisited ones, labels
// them and appends them to the next frontier. When the frontier's edges
// outweigh the unexplored ones, a level can instead run the masked pull
// kernel, which reads only the rows of unvisited vertices and stops each at
// its first frontier neighbour.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.hpp"
#include "frontier.hpp"
#include "internal.hpp"

namespace spx {

// Level L appends into counter L & 1 and clears the other one for level L + 1
// (the host has read it before level L is enqueued, on the same stream).
//
// level = -1 except the source (0); the frontier is the source, as a list
// and as a bitvector; the counter of level 0 holds {1 vertex, out-degree of
// the source}, the other one is cleared.
__global__ __launch_bounds__(kBlock) void k_bfs_seed(int32_t n, int32_t source, const int32_t* __restrict__ col_ptr,
                                                     int32_t* __restrict__ level, int32_t* __restrict__ frontier,
                                                     uint32_t* __restrict__ bits, Counters c) {
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x; v < n; v += stride)
        level[v] = v == source ? 0 : -1;
    const int64_t words = ceil_div((int64_t)n, 32);
    for (int64_t w = (int64_t)blockIdx.x * kBlock + threadIdx.x; w < words; w += stride)
        bits[w] = w == source >> 5 ? 1u << (source & 31) : 0u;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        frontier[0] = source;
        const Count seed = ((Count)(uint32_t)(col_ptr[source + 1] - col_ptr[source]) << 32) | 1ull;
        *c.count = seed;
        *c.clear = 0;
        *c.done = 0;
        __hip_atomic_store(c.host, seed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// Vertices reached by the product and not labelled yet get level L and go
// to the next frontier. Thread t of a chunk owns its 8 consecutive vertices.
__global__ __launch_bounds__(kWideBlock) void k_bfs_update(int32_t n, const uint8_t* __restrict__ y, int32_t L,
                                                       const int32_t* __restrict__ col_ptr,
                                                       int32_t* __restrict__ level, int32_t* __restrict__ next,
                                                       uint32_t* __restrict__ next_bits, Counters c) {
    __shared__ Count tmp[kWideBlock / kWave];
    if (blockIdx.x == 0 && threadIdx.x == 0) *c.clear = 0;
    for (int64_t base = (int64_t)blockIdx.x * kWideChunk; base < n; base += (int64_t)gridDim.x * kWideChunk) {
        const int64_t v0 = base + (int64_t)threadIdx.x * kVpt;
        uint64_t yy = 0;
        if (v0 + kVpt <= n) {
            yy = *(const uint64_t*)(y + v0);  // y is 256-byte aligned and v0 a multiple of 8
        } else {
            for (int j = 0; v0 + j < n; ++j) yy |= (uint64_t)(y[v0 + j] != 0) << (8 * j);
        }
        uint32_t reached = 0;
#pragma unroll
        for (int j = 0; j < kVpt; ++j) reached |= (uint32_t)(((yy >> (8 * j)) & 0xffu) != 0) << j;
        uint32_t deg = 0;
        const uint32_t mask = label_unvisited(reached, v0, n, L, col_ptr, level, &deg);
        write_bits(mask, v0, n, next_bits);
        block_append<kWideBlock>(mask, v0, deg, next, c.count, tmp);
    }
    publish_count(c);
}

// Masked pull (the row-major expansion restricted to the unvisited rows,
// with early exit). Row i of A lists the vertices with an edge into i; an
// unvisited i joins level L at its first entry in the frontier's
// bitvector (written by the previous level). Per chunk of kPullChunk rows:
//   A. each thread takes rows strided by the workgroup size (coalesced)
//      and tests their first two entries, all loads independent;
//   B. the rows still open are listed in LDS and scanned by kPullLanes lanes
//      each, four entries per lane and step, stopping at the first hit;
//   C. threads label and append 8 consecutive rows' hits each.
// Rows of visited vertices are not read.
//
// Bound by the chain level, row_ptr, col_idx, bitvector: 16 and 11 us for the
// two pulled levels of a search of the R-MAT graph of 2^20 vertices (16 edges
// each), 22 and 18 us with 256 threads to 2048 rows, a branch around each
// vertex's loads and a wave per open row.
constexpr int kPullChunk = 4096;
constexpr int kPullLanes = 16;
__device__ __forceinline__ bool in_bits(const uint32_t* __restrict__ bits, int32_t c) {
    return (bits[c >> 5] >> (c & 31)) & 1u;
}

__global__ __launch_bounds__(kWideBlock) void k_bfs_pull(int32_t n, const int32_t* __restrict__ row_ptr,
                                                     const int32_t* __restrict__ col_idx,
                                                     const uint32_t* __restrict__ bits, int32_t L,
                                                     const int32_t* __restrict__ col_ptr,
                                                     int32_t* __restrict__ level, int32_t* __restrict__ next,
                                                     uint32_t* __restrict__ next_bits, Counters c) {
    constexpr int kPer = kPullChunk / kWideBlock;
    __shared__ alignas(8) uint8_t hit[kPullChunk];
    if (blockIdx.x == 0 && threadIdx.x == 0) *c.clear = 0;
    __shared__ int16_t open[kPullChunk];
    __shared__ int n_open;
    __shared__ Count tmp[kWideBlock / kWave];
    for (int64_t base = (int64_t)blockIdx.x * kPullChunk; base < n; base += (int64_t)gridDim.x * kPullChunk) {
        if (threadIdx.x == 0) n_open = 0;
        __syncthreads();
        // A: no branch around a load, so that each step's are in flight together
        int32_t lv[kPer], k0[kPer], k1[kPer], c0[kPer], c1[kPer];
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int64_t r = base + j * kWideBlock + threadIdx.x;
            lv[j] = r < n ? level[r] : 0;
        }
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int64_t r = lv[j] < 0 ? base + j * kWideBlock + threadIdx.x : 0;
            k0[j] = row_ptr[r];
            k1[j] = row_ptr[r + 1];
        }
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            if (lv[j] >= 0) k1[j] = k0[j];
            c0[j] = col_idx[k1[j] > k0[j] ? k0[j] : 0];  // a level with out-edges to pull: nnz > 0
            c1[j] = col_idx[k1[j] > k0[j] + 1 ? k0[j] + 1 : 0];
        }
        uint32_t w0[kPer], w1[kPer];
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            w0[j] = bits[c0[j] >> 5];
            w1[j] = bits[c1[j] >> 5];
        }
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const bool h = (k1[j] > k0[j] && ((w0[j] >> (c0[j] & 31)) & 1u)) ||
                           (k1[j] > k0[j] + 1 && ((w1[j] >> (c1[j] & 31)) & 1u));
            const int p = j * kWideBlock + threadIdx.x;
            hit[p] = h;
            if (!h && k1[j] > k0[j] + 2) open[atomicAdd(&n_open, 1)] = (int16_t)p;
        }
        __syncthreads();
        // B
        const int no = n_open, lane = threadIdx.x % kPullLanes;
        for (int q = threadIdx.x / kPullLanes; q < no; q += kWideBlock / kPullLanes) {
            const int p = open[q];
            const int64_t r = base + p;
            const int32_t e = row_ptr[r + 1];
            bool found = false;
            for (int32_t kb = row_ptr[r] + 2; kb < e && !found; kb += 4 * kPullLanes) {
                bool h = false;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int32_t k = kb + u * kPullLanes + lane;
                    h |= k < e && in_bits(bits, col_idx[min(k, e - 1)]);
                }
                found = (__ballot(h) >> (lane_id() - lane)) & ((1ull << kPullLanes) - 1ull);
            }
            if (found && lane == 0) hit[p] = 1;
        }
        __syncthreads();
        // C
        const int64_t v0 = base + (int64_t)threadIdx.x * kVpt;
        uint32_t mask = 0, deg = 0;
        if (threadIdx.x < kPullChunk / kVpt) {
            const uint64_t h = *(const uint64_t*)(hit + threadIdx.x * kVpt);
#pragma unroll
            for (int j = 0; j < kVpt; ++j) {
                if ((h >> (8 * j)) & 1u) {
                    level[v0 + j] = L;
                    mask |= 1u << j;
                }
            }
            if (mask) deg = degrees(mask, v0, n, col_ptr);
        }
        write_bits(mask, threadIdx.x < kPullChunk / kVpt ? v0 : n, n, next_bits);
        block_append<kWideBlock>(mask, v0, deg, next, c.count, tmp);
    }
    publish_count(c);
}

spx_status launch_bfs_seed(int32_t n, int32_t source, const int32_t* col_ptr, int32_t* level, int32_t* frontier,
                           uint32_t* bits, void* count, void* host, hipStream_t s) {
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(ceil_div(n, kBlock), 4096));
    k_bfs_seed<<<grid, kBlock, 0, s>>>(n, source, col_ptr, level, frontier, bits, counters_of(count, 0, host));
    SPX_HIP(hipGetLastError());
    return SPX_OK;
}

spx_status launch_bfs_update(int32_t n, const uint8_t* y, int32_t L, const int32_t* col_ptr, int32_t* level,
                             int32_t* next, uint32_t* next_bits, void* count, void* host, hipStream_t s) {
    if ((uintptr_t)y % 8) return fail(SPX_ERR_ARG, "breadth-first search: product buffer must be 8-byte aligned");
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(ceil_div(n, kWideChunk), 2048));
    k_bfs_update<<<grid, kWideBlock, 0, s>>>(n, y, L, col_ptr, level, next, next_bits,
                                           counters_of(count, L, host));
    SPX_HIP(hipGetLastError());
    return SPX_OK;
}

spx_status launch_bfs_pull(int32_t n, const int32_t* row_ptr, const int32_t* col_idx, const uint32_t* bits,
                           int32_t L, const int32_t* col_ptr, int32_t* level, int32_t* next, uint32_t* next_bits,
                           void* count, void* host, hipStream_t s) {
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(ceil_div(n, kPullChunk), 2048));
    k_bfs_pull<<<grid, kWideBlock, 0, s>>>(n, row_ptr, col_idx, bits, L, col_ptr, level, next, next_bits,
                                       counters_of(count, L, host));
    SPX_HIP(hipGetLastError());
    return SPX_OK;
}

}  // namespace spx
