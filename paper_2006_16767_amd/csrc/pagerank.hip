// Incremental PageRank driver (the second application the paper evaluates
// its kernels in, Section 7): residual push, where every round propagates
// only the vertices whose residual is above a threshold, so the product's
// input starts dense and thins out round by round, and run() follows it.
//
// Stored entry (i, j) is an edge j -> i of weight a_ij >= 0; the walk
// leaves j along (i, j) with probability a_ij / W_j, W_j = sum of column j.
// State: residual r (starts at (1 - d)/n) and rank p (starts at 0). A round
// (k_pr_select) folds the previous product into r (r += d y), moves every
// active residual (|r_v| > eps) into p_v, clears it, and appends the
// active vertices with W_v > 0 to the sparse input x_v = r_v / W_v of the
// next product y = A x, as a dense vector, so that no conversion runs before
// a row-major kernel, and as a list unless that product is row-major.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.hpp"
#include "frontier.hpp"
#include "internal.hpp"

namespace spx {

// bad gets bit 0 if a stored weight is negative (one atomic per wave that
// sees one). The column sums themselves are a product: W = A^T 1.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_pr_negcheck(int64_t nnz, const T* __restrict__ vals,
                                                        uint32_t* __restrict__ bad) {
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    bool neg = false;
    for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < nnz; k += stride) neg |= vals[k] < (T)0;
    if (__ballot(neg) && lane_id() == 0) atomicOr(bad, 1u);
}

// v = 1 everywhere (the x of W = A^T 1).
template <typename T>
__global__ __launch_bounds__(kBlock) void k_pr_ones(int32_t n, T* __restrict__ v) {
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += stride) v[i] = (T)1;
}

// r = r0 everywhere, p = 0, and the dense x buffer of round 0 zeroed.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_pr_init(int32_t n, T r0, T* __restrict__ r, T* __restrict__ p,
                                                    T* __restrict__ xd0) {
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x; v < n; v += stride) {
        r[v] = r0;
        p[v] = (T)0;
        xd0[v] = (T)0;
    }
}

// One round. y = nullptr on the first round (no product yet). The counter
// gets {entries of x (low), their column lengths (high), i.e. the
// nnz_s of the next product}; the other counter is zeroed for the next round.
// x goes dense into xd_fill at position map[v] (the column order of the
// row-major copy; v itself when map is null): xd_fill was zeroed by the
// previous round, and this round zeroes xd_clear for the next one (two buffers
// alternate, each zeroed while the other is in use). LIST: x also as a list
// (x_idx, x_val), for a product that may be column-major. r += d y is rounded
// as a product and then a sum (no fused multiply-add), the order the
// definition states.
//
// Bound by its 42 MB, by the scattered stores of x and by latency (three steps
// of loads, then the counter): 12.9 us with every one of 2^20 vertices active,
// 8 to 10 once the frontier thins out. Half the vertices per workgroup and no
// list in the row-major rounds took a ranking of the R-MAT graph of 2^20
// vertices (66 rounds) from 4902 to 4856 us.
constexpr int kSelVpt = 4;
constexpr int kSelChunk = kWideBlock * kSelVpt;

// The first tile whose last row is row or a later one. Every lane of the wave
// must call it with the same row.
__device__ __forceinline__ int first_tile_from(const Carries& c, int64_t row) {
    int lo = 0, hi = c.tiles;
    while (lo < hi) {
        const int step = (hi - lo + kWave - 1) / kWave;
        const int t = lo + lane_id() * step;
        const uint64_t at = __ballot(t >= hi || c.part[2 * t + 2] >= row);
        const int f = at ? __ffsll((unsigned long long)at) - 1 : kWave;
        hi = min(hi, lo + f * step);
        lo = f > 0 ? lo + (f - 1) * step + 1 : lo;
    }
    return lo;
}

template <typename T, bool LIST>
__global__ __launch_bounds__(kWideBlock) void k_pr_select(int32_t n, T d, T eps, const T* __restrict__ y,
                                                      Carries carries,
                                                      T* __restrict__ r, T* __restrict__ p,
                                                      const T* __restrict__ W, const int32_t* __restrict__ col_ptr,
                                                      const int32_t* __restrict__ map, int32_t* __restrict__ x_idx,
                                                      T* __restrict__ x_val, T* __restrict__ xd_fill,
                                                      T* __restrict__ xd_clear, Counters c) {
#pragma clang fp contract(off)
    __shared__ Count tmp[kWideBlock / kWave];
    __shared__ T s_add[kSelChunk];
    __shared__ int s_tile[2];
    if (blockIdx.x == 0 && threadIdx.x == 0) *c.clear = 0;
    for (int64_t base = (int64_t)blockIdx.x * kSelChunk; base < n; base += (int64_t)gridDim.x * kSelChunk) {
        const int64_t v0 = base + (int64_t)threadIdx.x * kSelVpt;
        // all loads of a phase are independent, so they are in flight together
        T rv[kSelVpt], wv[kSelVpt], xv[kSelVpt];
        load_run(r, v0, n, rv);
        load_run(W, v0, n, wv);
        if (y) {
            T yv[kSelVpt];
            load_run(y, v0, n, yv);
            if (carries.tiles) {
                // what rows of the chunk that span tiles still lack, added in
                // tile order by the thread of a row's first tile
                if (wave_id() < 2) {
                    const int t = first_tile_from(carries, base + wave_id() * kSelChunk);
                    if (lane_id() == 0) s_tile[wave_id()] = t;
                }
#pragma unroll
                for (int j = 0; j < kSelVpt; ++j) s_add[threadIdx.x * kSelVpt + j] = (T)0;
                __syncthreads();
                for (int t = s_tile[0] + (int)threadIdx.x; t < s_tile[1]; t += kWideBlock) {
                    const int row = carries.row[t];
                    if (row < 0 || (t > 0 && carries.row[t - 1] == row)) continue;
                    T sum = (T)0;
                    for (int u = t; u < carries.tiles && carries.row[u] == row; ++u)
                        sum = sum + ((const T*)carries.val)[u];
                    s_add[row - base] = sum;
                }
                __syncthreads();
#pragma unroll
                for (int j = 0; j < kSelVpt; ++j) yv[j] = yv[j] + s_add[threadIdx.x * kSelVpt + j];
            }
#pragma unroll
            for (int j = 0; j < kSelVpt; ++j) {
                const T dy = d * yv[j];
                rv[j] = rv[j] + dy;
            }
        }
        uint32_t act = 0;
#pragma unroll
        for (int j = 0; j < kSelVpt; ++j)
            if (v0 + j < n && (rv[j] > eps || rv[j] < -eps)) act |= 1u << j;
        uint32_t mask = 0, ns = 0;
#pragma unroll
        for (int j = 0; j < kSelVpt; ++j) xv[j] = (T)0;
        if (act) {
            // the rank, the column pointers and the map of the thread's
            // vertices only when one of them is active
            T pv[kSelVpt];
            int32_t cp[kSelVpt], mp[kSelVpt];
            load_run(p, v0, n, pv);
            load_run(col_ptr, v0, (int64_t)n + 1, cp);
            const int32_t end = v0 + kSelVpt <= n ? col_ptr[v0 + kSelVpt] : 0;
            if (map) load_run(map, v0, n, mp);
#pragma unroll
            for (int j = 0; j < kSelVpt; ++j) {
                if (!((act >> j) & 1u)) continue;
                pv[j] = pv[j] + rv[j];
                if (wv[j] > (T)0) {
                    mask |= 1u << j;
                    xv[j] = rv[j] / wv[j];
                    ns += (uint32_t)((j + 1 < kSelVpt ? cp[j + 1] : end) - cp[j]);
                    xd_fill[map ? mp[j] : v0 + j] = xv[j];
                }
                rv[j] = (T)0;
            }
            store_run(p, v0, n, pv);
        }
        if (y || act) store_run(r, v0, n, rv);
        const T zero[kSelVpt] = {};
        store_run(xd_clear, v0, n, zero);
        if constexpr (LIST)
            block_append<kWideBlock>(mask, ns, c.count, tmp, [&](uint32_t slot, int j) {
                x_idx[slot] = (int32_t)(v0 + j);
                x_val[slot] = xv[j];
            });
        else
            block_count<kWideBlock>(mask, ns, c.count, tmp);
    }
    publish_count(c);
}

// r += d y (the product of the last round, when the rounds stop at the
// product limit).
template <typename T>
__global__ __launch_bounds__(kBlock) void k_pr_fold(int32_t n, T d, const T* __restrict__ y, T* __restrict__ r) {
#pragma clang fp contract(off)
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x; v < n; v += stride) {
        const T dy = d * y[v];
        r[v] = r[v] + dy;
    }
}

static int flat_grid(int32_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>(ceil_div(n, kBlock), 4096)); }

template <typename T>
static spx_status pr_t(const PrArgs& a, hipStream_t s) {
    switch (a.stage) {
        case PR_NEGCHECK: {
            const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(ceil_div(a.nnz, kBlock), 4096));
            k_pr_negcheck<T><<<grid, kBlock, 0, s>>>(a.nnz, (const T*)a.vals_csc, a.bad);
            break;
        }
        case PR_ONES:
            k_pr_ones<T><<<flat_grid(a.n), kBlock, 0, s>>>(a.n, (T*)a.ones);
            break;
        case PR_INIT:
            k_pr_init<T><<<flat_grid(a.n), kBlock, 0, s>>>(a.n, (T)((1.0 - a.damping) / a.n), (T*)a.r, (T*)a.p,
                                                           (T*)a.xd[0]);
            break;
        case PR_SELECT: {
            const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(ceil_div(a.n, kSelChunk), 2048));
            const auto kernel = a.list ? k_pr_select<T, true> : k_pr_select<T, false>;
            kernel<<<grid, kWideBlock, 0, s>>>(a.n, (T)a.damping, (T)a.eps, (const T*)a.y, a.carries, (T*)a.r, (T*)a.p,
                                               (const T*)a.W, a.col_ptr, a.map, a.x_idx, (T*)a.x_val,
                                               (T*)a.xd[a.round & 1], (T*)a.xd[(a.round + 1) & 1],
                                               counters_of(a.count, a.round, a.host));
            break;
        }
        case PR_FOLD:
            k_pr_fold<T><<<flat_grid(a.n), kBlock, 0, s>>>(a.n, (T)a.damping, (const T*)a.y, (T*)a.r);
            break;
        default:
            return fail(SPX_ERR_ARG, "PageRank: unknown stage");
    }
    SPX_HIP(hipGetLastError());
    return SPX_OK;
}

spx_status launch_pagerank(const PrArgs& a, hipStream_t s) {
    if (a.n <= 0) return SPX_OK;
    if (a.dtype == SPX_F32) return pr_t<float>(a, s);
    if (a.dtype == SPX_F64) return pr_t<double>(a, s);
    return fail(SPX_ERR_DTYPE, "PageRank supports F32 and F64");
}

}  // namespace spx
