// Frontier appends shared by the graph drivers (breadth-first search and
// PageRank): a workgroup owns consecutive vertices, 8 per thread,
// and appends the ones it selects to an output list with one atomic on a
// packed counter.
#pragma once

#include <hip/hip_runtime.h>

#include "common.hpp"

namespace spx {

// A counter is one 64-bit word of two halves that are added together: the
// low half counts the vertices appended to the list, the high half holds a
// per-driver sum (both drivers: the column lengths of the appended
// vertices, i.e. nnz_s of the next product). Neither half can carry into the other (both stay below
// 2^31), so one atomic add updates both.
using Count = unsigned long long;

// The drivers' counter words in device memory: two counters that alternate
// between rounds (round k appends into count[k & 1] and clears the other one),
// and a cache line further the workgroups of the running kernel that have
// finished. host: a pinned word that takes the round's total.
struct Counters {
    Count* count;
    Count* clear;
    uint32_t* done;
    Count* host;
};
constexpr Count kNoCount = ~0ull;  // in the pinned word: not written yet

inline Counters counters_of(void* words, int32_t round, void* host) {
    Count* c = (Count*)words;
    return Counters{c + (round & 1), c + ((round + 1) & 1), (uint32_t*)(c + 16), (Count*)host};
}

// The workgroup has added its share: the last one to come here stores the
// total to the pinned word, which the host polls. (A copy of the counter and a
// stream synchronization per round cost 4 us and 20 to 30 us until the next
// launch.) The word itself is all that the host reads, and kernels see each
// other's data by stream order, so there is no fence, only the wait for the
// workgroup's own add.
__device__ __forceinline__ void publish_count(const Counters& c) {
    if (threadIdx.x != 0) return;
    __builtin_amdgcn_s_waitcnt(0);
    asm volatile("" ::: "memory");
    if (atomicAdd(c.done, 1u) + 1 == gridDim.x) {
        *c.done = 0;
        __hip_atomic_store(c.host, atomicAdd(c.count, 0ull), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// Vertices per thread: a workgroup owns NT * kVpt consecutive vertices and
// appends the ones it selects with a single atomic on the counter. Atomics
// on one word serialize (about 12 ns each on this GPU, so one per wave
// costs more than the rest of a level on a large frontier, and even one
// per 256-thread workgroup costs about 6 µs at n = 2^20): the streaming
// kernels therefore run 1024-thread workgroups (kWideBlock), the same
// threads in a quarter of the atomics.
constexpr int kVpt = 8;
constexpr int kWideBlock = 1024;
constexpr int kWideChunk = kWideBlock * kVpt;

// Inclusive prefix sum across an NT-thread workgroup; tmp holds NT / 64
// elements of LDS; *total gets the workgroup total. Contains __syncthreads.
template <int NT, typename T>
__device__ __forceinline__ T block_scan_nt(T v, T* tmp, T* total) {
    constexpr int W = NT / kWave;
    T w = wave_incl_scan(v);
    if (lane_id() == kWave - 1) tmp[wave_id()] = w;
    __syncthreads();
    T pre = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < W; ++i) {
        const T t = tmp[i];
        if (i < wave_id()) pre += t;
        tot += t;
    }
    __syncthreads();
    *total = tot;
    return w + pre;
}

// N consecutive values from v0, as 16-byte loads and stores of 4-byte aligned
// words (which is what a global access of that width needs); element by
// element at the tail.
struct __attribute__((packed, aligned(4))) Words4 {
    uint32_t w[4];
};

template <int N, typename T>
__device__ __forceinline__ void load_run(const T* __restrict__ a, int64_t v0, int64_t n, T (&o)[N]) {
    if (v0 + N <= n) {
        static_assert(N * sizeof(T) % 16 == 0);
        Words4 w[N * sizeof(T) / 16];
#pragma unroll
        for (int u = 0; u < (int)(N * sizeof(T) / 16); ++u) w[u] = ((const Words4*)(a + v0))[u];
        __builtin_memcpy(o, w, sizeof(o));
    } else {
#pragma unroll
        for (int j = 0; j < N; ++j) o[j] = v0 + j < n ? a[v0 + j] : (T)0;
    }
}

template <int N, typename T>
__device__ __forceinline__ void store_run(T* __restrict__ a, int64_t v0, int64_t n, const T (&o)[N]) {
    if (v0 + N <= n) {
        Words4 w[N * sizeof(T) / 16];
        __builtin_memcpy(w, o, sizeof(o));
#pragma unroll
        for (int u = 0; u < (int)(N * sizeof(T) / 16); ++u) ((Words4*)(a + v0))[u] = w[u];
    } else {
#pragma unroll
        for (int j = 0; j < N; ++j)
            if (v0 + j < n) a[v0 + j] = o[j];
    }
}

// The workgroup's share of the counter without a list: {popcount of mask,
// high} summed, one atomic whose result nothing waits for. Contains
// __syncthreads; tmp: NT / 64 words of LDS.
template <int NT>
__device__ __forceinline__ void block_count(uint32_t mask, uint32_t high, Count* __restrict__ count, Count* tmp) {
    Count total;
    block_scan_nt<NT, Count>(((Count)high << 32) | (Count)__popc(mask), tmp, &total);
    if (threadIdx.x == 0 && total) atomicAdd(count, total);
}

// Thread t holds the candidates v0 + j for the set bits j of mask, and
// high, its share of the counter's high half. The workgroup (NT threads)
// reserves one range of the list and calls emit(slot, j) for each
// candidate, slots ascending with the vertex. Contains __syncthreads;
// every thread of the workgroup must call it. tmp: NT / 64 words of LDS.
template <int NT, typename Emit>
__device__ __forceinline__ void block_append(uint32_t mask, uint32_t high, Count* __restrict__ count, Count* tmp,
                                             Emit emit) {
    const Count mine = ((Count)high << 32) | (Count)__popc(mask);
    Count total;
    const Count incl = block_scan_nt<NT, Count>(mine, tmp, &total);
    __shared__ Count base;
    if (threadIdx.x == 0) base = total ? atomicAdd(count, total) : 0ull;
    __syncthreads();
    uint32_t slot = (uint32_t)base + (uint32_t)(incl - mine);
    while (mask) {
        const int j = __ffs(mask) - 1;
        mask &= mask - 1;
        emit(slot++, j);
    }
    __syncthreads();  // base is reused by the next chunk
}

// The vertex list form: next[slot] = v0 + j.
template <int NT>
__device__ __forceinline__ void block_append(uint32_t mask, int64_t v0, uint32_t high, int32_t* __restrict__ next,
                                             Count* __restrict__ count, Count* tmp) {
    block_append<NT>(mask, high, count, tmp, [&](uint32_t slot, int j) { next[slot] = (int32_t)(v0 + j); });
}

// The column lengths of the vertices v0 + j with bit j of mask set.
__device__ __forceinline__ uint32_t degrees(uint32_t mask, int64_t v0, int32_t n, const int32_t* __restrict__ col_ptr) {
    int32_t cp[kVpt];
    load_run(col_ptr, v0, (int64_t)n + 1, cp);
    const int32_t end = v0 + kVpt <= n ? col_ptr[v0 + kVpt] : 0;
    uint32_t deg = 0;
#pragma unroll
    for (int j = 0; j < kVpt; ++j)
        if ((mask >> j) & 1u) deg += (uint32_t)((j + 1 < kVpt ? cp[j + 1] : end) - cp[j]);
    return deg;
}

// Breadth-first search: of the vertices v0 + j with bit j of reached set, the
// unvisited ones get level L; returned as a mask, *deg their column lengths.
// The levels are loaded together, then the column pointers together (one
// vertex after the other is up to eight round trips of each).
__device__ __forceinline__ uint32_t label_unvisited(uint32_t reached, int64_t v0, int32_t n, int32_t L,
                                                    const int32_t* __restrict__ col_ptr, int32_t* __restrict__ level,
                                                    uint32_t* deg) {
    uint32_t mask = 0;
    *deg = 0;
    if (!reached) return 0;
    int32_t lv[kVpt];
    load_run(level, v0, n, lv);
#pragma unroll
    for (int j = 0; j < kVpt; ++j) {
        if (((reached >> j) & 1u) && v0 + j < n && lv[j] < 0) {
            lv[j] = L;
            mask |= 1u << j;
        }
    }
    if (mask) {
        store_run(level, v0, n, lv);
        *deg = degrees(mask, v0, n, col_ptr);
    }
    return mask;
}

// Writes the next frontier's bitvector for the 8 consecutive vertices
// v0.. of every thread (v0 a multiple of 8): the four threads of one
// 32-bit word are neighbouring lanes. Every lane of the wave must call it.
__device__ __forceinline__ void write_bits(uint32_t mask8, int64_t v0, int32_t n, uint32_t* __restrict__ bits) {
    const uint32_t b1 = __shfl_down(mask8, 1, kWave), b2 = __shfl_down(mask8, 2, kWave),
                   b3 = __shfl_down(mask8, 3, kWave);
    if ((threadIdx.x & 3) == 0 && v0 < n) bits[v0 >> 5] = mask8 | b1 << 8 | b2 << 16 | b3 << 24;
}

}  // namespace spx
