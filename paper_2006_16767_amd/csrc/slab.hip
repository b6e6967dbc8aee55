// The pruned layer's products with the dense operand held in LDS: a batch of
// dense rows times A (or its transpose), and the gradient of A's values.
//
//   k_slab_gather  out[b, j]  = sum over the entries k of segment j of
//                  vals[k] * in[b, idx[k]]: the forward (segments = rows of A,
//                  in = X) and dX (segments = columns, in = G)
//   k_slab_dots    dvals[k] = sum_b G[b, row k] * X[b, col k]
//
// Per stored entry and batch row these need one value of the dense operand,
// at a random place. Gathering it from L2 (a B-minor copy, a row of B values
// per entry) moves 4 B bytes per entry through the L2 and the address path:
// 860 MB for the 16384 x 4096 layer at 5 % and B = 64, 57 us at 15 TB/s. Here
// a workgroup holds a slab of the operand in LDS, slab_cols(W) columns of a few
// batch rows (32 bytes a column: 8 FP32 or 4 FP64 batch rows, one or two
// 16-byte LDS reads per entry), built from the B-major operand itself (no
// B-minor copy), and streams the segments' indices and values past it. The
// matrix is then read once per 8 batch rows instead of once, 64 instead of
// 264 bytes per entry; the workgroups that read the same segments for the
// other batch rows are neighbours on one XCD, so those reads meet in its L2.
//
// 16 lanes walk a segment, four segments per wave in lockstep, four entries
// per lane at a time with the next four (of the segment, or the first of the
// next one) already in flight. The bound is the LDS: random 32-byte columns
// meet on the same banks about twice as often as they would in order. Odd
// lanes read the second half of a column first, so that the two reads of a
// wave use all banks.
//
// A lane's running sum takes at most kFoldRounds additions: then the 16 lanes'
// sums are added as a tree and go to the segment's sum in LDS, where a slab
// (slab_cols(W) distinct indices) adds at most slab_cols(W) / (16 kFoldRounds)
// of them. In one chain a row that fills a slab would take 256 or 512
// additions, 1.5e-5 or 3.1e-5 of sum |a x| at worst in FP32; so it is 72 or 76,
// 4.5e-6 (4096 and 8192 entries). Rows of that length take 3 to 13 % longer for
// it (200000 x 4096 with 411 full rows, FP32: B = 8 63.6 us against 58.4, B = 64
// 340 against 329), rows below 1024 entries up to 1 % (16384 x 4096 at 5 %, B = 64:
// 27.3 against 27.1).
#include <algorithm>
#include <utility>

#include "common.hpp"
#include "csr_tile.hpp"
#include "internal.hpp"

namespace spx {

constexpr int kSlabThreads = 1024;
constexpr int kSlabLanes = 16;                            // lanes per segment: a DPP row
constexpr int kSlabGroups = kSlabThreads / kSlabLanes;    // segments in flight per workgroup
constexpr int kSlabU = 4;                                 // entries per lane and step
constexpr int kSlabStep = kSlabLanes * kSlabU;
constexpr int kSlabFold = kFoldRounds / kSlabU;           // steps between folds
constexpr int kSlabBytes = 128 * 1024;                    // of the CU's 160 KiB
constexpr int kSlabMaxSegs = 512;                         // segments per workgroup

// columns of a slab of 16-byte (W = 1) or 32-byte (W = 2) columns
constexpr int slab_cols(int W) { return kSlabBytes / (16 * W); }

template <int CTRL>
__device__ __forceinline__ int dpp_word(int v) {
    return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true);
}

template <int CTRL, typename T>
__device__ __forceinline__ T dpp(T v) {
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(T, dpp_word<CTRL>(__builtin_bit_cast(int, v)));
    } else {
        const uint64_t u = __builtin_bit_cast(uint64_t, v);
        const uint32_t lo = (uint32_t)dpp_word<CTRL>((int)(uint32_t)u);
        const uint32_t hi = (uint32_t)dpp_word<CTRL>((int)(uint32_t)(u >> 32));
        return __builtin_bit_cast(T, ((uint64_t)hi << 32) | lo);
    }
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E;      // quad_perm
constexpr int kDppRor4 = 0x124, kDppRor8 = 0x128;    // rotations of a row of 16 lanes
constexpr int kDppBcast = 0x150;                     // row_newbcast: lane n of the row to all

template <typename T>
struct alignas(16) SlabVec {
    static constexpr int E = 16 / sizeof(T);  // values per 16-byte LDS read
    T v[E];
};

// One slab: columns [c0, c0 + cb) of batch rows b0 .. b0 + NB - 1 of in (B x
// N), first into registers (so that the next slab loads while this one is in
// use), then to LDS; rows past B are zeros. Column cb of the slab is all
// zeros: the place that lanes without an entry read.
template <typename T, int W>
struct SlabLoad {
    static constexpr int E = SlabVec<T>::E, NB = W * E;
    static constexpr int kPer = slab_cols(W) / kSlabThreads;
    T r[kPer][NB];
    __device__ __forceinline__ void load(const T* __restrict__ in, int64_t N, int32_t B, int32_t b0, int32_t c0,
                                         int32_t cb) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            // past the columns, and for rows past B, the load returns 0
            const auto row = buffer_of(in + (int64_t)(b0 + b) * N + c0, b0 + b < B ? cb * (int)sizeof(T) : 0);
#pragma unroll
            for (int p = 0; p < kPer; ++p)
                r[p][b] = buffer_value<T>(row, (p * kSlabThreads + (int)threadIdx.x) * (int)sizeof(T));
        }
    }
    __device__ __forceinline__ void store(char* slab, int32_t cb) const {
        const int par = threadIdx.x & 1;
#pragma unroll
        for (int p = 0; p < kPer; ++p) {
            const int c = p * kSlabThreads + (int)threadIdx.x;
            if (c < cb) {
                if constexpr (W == 2) {
                    // odd lanes store their second half first (bank use)
                    SlabVec<T> a, b;
#pragma unroll
                    for (int e = 0; e < E; ++e) {
                        a.v[e] = par ? r[p][E + e] : r[p][e];
                        b.v[e] = par ? r[p][e] : r[p][E + e];
                    }
                    *(SlabVec<T>*)(slab + (c << 5) + (par << 4)) = a;
                    *(SlabVec<T>*)(slab + (c << 5) + ((par ^ 1) << 4)) = b;
                } else {
                    SlabVec<T> a;
#pragma unroll
                    for (int e = 0; e < E; ++e) a.v[e] = r[p][e];
                    *(SlabVec<T>*)(slab + (c << 4)) = a;
                }
            }
        }
        if (threadIdx.x < (unsigned)W) {
            SlabVec<T> z;
#pragma unroll
            for (int e = 0; e < E; ++e) z.v[e] = (T)0;
            *(SlabVec<T>*)(slab + (int64_t)cb * 16 * W + threadIdx.x * 16) = z;
        }
    }
};

// Byte offset of column c of the slab; for W = 2, of its half of the lane's
// parity (par16 = 16 for odd lanes), which p[0] then holds, p[1] the other.
template <int W>
__device__ __forceinline__ int slab_at(int c, int par16) {
    return W == 2 ? (c << 5) | par16 : c << 4;
}
template <typename T, int W>
__device__ __forceinline__ void slab_read(const char* slab, int at, SlabVec<T> (&p)[W]) {
    p[0] = *(const SlabVec<T>*)(slab + at);
    if constexpr (W == 2) p[1] = *(const SlabVec<T>*)(slab + (at ^ 16));
}

// The 16 lanes' sums a[w][e] of a segment folded: every lane ends with E / 2
// full sums, of batch rows slab_fold_row(lane) .. + E / 2 - 1.
template <typename T, int W>
__device__ __forceinline__ void slab_fold(const T (&a)[W][SlabVec<T>::E], T (&out)[SlabVec<T>::E / 2]) {
    constexpr int E = SlabVec<T>::E;
    const int lane = lane_id();
    T v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        v[e] = a[0][e];
        // the neighbour's second half is this lane's first
        if constexpr (W == 2) v[e] += dpp<kDppXor1>(a[1][e]);
    }
    const bool hi = lane & W;  // bit 1 for W = 2, bit 0 for W = 1
    constexpr int ctrl = W == 2 ? kDppXor2 : kDppXor1;
#pragma unroll
    for (int i = 0; i < E / 2; ++i) {
        T s = (hi ? v[i + E / 2] : v[i]) + dpp<ctrl>(hi ? v[i] : v[i + E / 2]);
        if constexpr (W == 1) s += dpp<kDppXor2>(s);
        s += dpp<kDppRor4>(s);
        out[i] = s + dpp<kDppRor8>(s);
    }
}
template <typename T, int W>
__device__ __forceinline__ int slab_fold_row(int lane) {
    constexpr int E = SlabVec<T>::E;
    return W == 2 ? (lane & 1) * E + ((lane >> 1) & 1) * (E / 2) : (lane & 1) * (E / 2);
}

// The first entry of a segment (of [lo, hi)) whose index is at or past c; its
// indices ascend.
__device__ __forceinline__ int first_from(const int32_t* __restrict__ idx, int lo, int hi, int c) {
    while (lo < hi) {
        const int mid = lo + (hi - lo) / 2;
        if (idx[mid] < c)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

// LDS of a gather workgroup: the slab and its zero column, then the sums of
// the segments, NB + 1 values apart.
template <typename T, int W>
static size_t slab_gather_lds(int32_t cb, int32_t segs) {
    return (size_t)(cb + 1) * 16 * W + (size_t)segs * (W * SlabVec<T>::E + 1) * sizeof(T);
}

// Workgroup = (segments [tile * st, + st), batch rows [chunk * NB, + NB)).
// The operand's N columns come as nblk slabs of cb; with nblk > 1 the
// segments' indices ascend and part[blk * nseg + j] is the first entry of
// segment j at or past column blk * cb (blk < nblk); without the table (PART =
// false) it is searched for.
template <typename T, int W, bool PART>
__global__ __launch_bounds__(kSlabThreads) void k_slab_gather(int32_t nseg, int32_t N, int32_t nnz, int32_t B,
                                                              int32_t st, int32_t nchunk, int32_t nblk, int32_t cb,
                                                              const int32_t* __restrict__ seg_ptr,
                                                              const int32_t* __restrict__ part,
                                                              const int32_t* __restrict__ idx,
                                                              const T* __restrict__ vals, const T* __restrict__ in,
                                                              T* __restrict__ out) {
    constexpr int E = SlabVec<T>::E, NB = W * E, kRow = NB + 1;
    extern __shared__ __align__(16) char s_raw[];
    const int64_t t = xcd_tile(blockIdx.x, gridDim.x);
    const int32_t tile = (int32_t)(t / nchunk), b0 = (int32_t)(t % nchunk) * NB;
    const int32_t j0 = tile * st;
    const int32_t ns = min(st, nseg - j0);
    char* slab = s_raw;
    T* sums = (T*)(s_raw + (size_t)(cb + 1) * 16 * W);
    const int lane = lane_id();
    const int g = lane % kSlabLanes, par16 = (lane & 1) << 4;
    const int s0 = threadIdx.x / kSlabLanes;
    const int rounds = (ns + kSlabGroups - 1) / kSlabGroups;
    const auto bidx = buffer_of(idx, nnz * 4), bval = buffer_of(vals, nnz * (int)sizeof(T));
    SlabLoad<T, W> next;
    next.load(in, N, B, b0, 0, min(cb, N));
    // the wave's walk, slab after slab, kSlabGroups segments at a time: the
    // bounds run two rounds ahead and the entries one step, across slabs too
    // (only the LDS reads depend on the slab)
    int pblk = 0, pr = 0;  // the round whose bounds are read next
    auto advance = [&](int& k0, int& k1) {
        const int s = pr * kSlabGroups + s0;
        k0 = k1 = 0;
        if (pblk < nblk && s < ns) {
            const int64_t j = j0 + s;
            if constexpr (PART) {
                k0 = pblk > 0 ? part[(int64_t)pblk * nseg + j] : seg_ptr[j];
                k1 = pblk + 1 < nblk ? part[(int64_t)(pblk + 1) * nseg + j] : seg_ptr[j + 1];
            } else {
                k0 = seg_ptr[j];
                k1 = seg_ptr[j + 1];
                if (pblk > 0) k0 = first_from(idx, k0, k1, pblk * cb);
                if (pblk + 1 < nblk) k1 = first_from(idx, k0, k1, (pblk + 1) * cb);
            }
        }
        if (++pr == rounds) {
            pr = 0;
            ++pblk;
        }
    };
    auto fetch = [&](int k, int (&c)[kSlabU], T (&v)[kSlabU]) {
#pragma unroll
        for (int u = 0; u < kSlabU; ++u) {
            c[u] = buffer_value<int>(bidx, (k + g + u * kSlabLanes) * 4);
            v[u] = buffer_value<T>(bval, (k + g + u * kSlabLanes) * (int)sizeof(T));
        }
    };
    int ka, kb, kc, kd;
    advance(ka, kb);
    advance(kc, kd);
    int c[kSlabU];
    T v[kSlabU];
    fetch(ka, c, v);
    for (int blk = 0; blk < nblk; ++blk) {
        const int32_t c0 = blk * cb;
        const int32_t width = min(cb, N - c0);
        if (blk > 0) __syncthreads();  // the last slab has been read
        next.store(slab, width);
        __syncthreads();
        if (blk + 1 < nblk) next.load(in, N, B, b0, c0 + cb, min(cb, N - c0 - cb));
        for (int r = 0; r < rounds; ++r) {
            int ke, kf;
            advance(ke, kf);
            int k = ka;
            bool more, first = blk == 0;
            do {
                T acc[W][E];
#pragma unroll
                for (int w = 0; w < W; ++w)
#pragma unroll
                    for (int e = 0; e < E; ++e) acc[w][e] = (T)0;
                int left = kSlabFold;
                do {
                    more = __any(k + kSlabStep < kb);  // uniform over the wave
                    // entries past the end read the zero column with value 0
                    SlabVec<T> p[kSlabU][W];
                    T a[kSlabU];
#pragma unroll
                    for (int u = 0; u < kSlabU; ++u) {
                        const bool on = k + g + u * kSlabLanes < kb;
                        slab_read<T, W>(slab, slab_at<W>(on ? c[u] - c0 : width, par16), p[u]);
                        a[u] = on ? v[u] : (T)0;
                    }
                    fetch(more ? k + kSlabStep : kc, c, v);
#pragma unroll
                    for (int u = 0; u < kSlabU; ++u)
#pragma unroll
                        for (int w = 0; w < W; ++w)
#pragma unroll
                            for (int e = 0; e < E; ++e) acc[w][e] = fma_t(a[u], p[u][w].v[e], acc[w][e]);
                    k += kSlabStep;
                } while (more && --left);
                T f[E / 2];
                slab_fold<T, W>(acc, f);
                const int s = r * kSlabGroups + s0;
                if (g < 2 * W && s < ns) {
                    T* o = sums + s * kRow + slab_fold_row<T, W>(lane);
#pragma unroll
                    for (int i = 0; i < E / 2; ++i) o[i] = first ? f[i] : o[i] + f[i];
                }
                first = false;
            } while (more);
            ka = kc;
            kb = kd;
            kc = ke;
            kd = kf;
        }
    }
    __syncthreads();
    const int nb = min(NB, B - b0);
    for (int i = threadIdx.x; i < ns * nb; i += kSlabThreads) {
        const int b = i / ns, s = i - b * ns;
        out[(int64_t)(b0 + b) * nseg + j0 + s] = sums[s * kRow + b];
    }
}

// dvals, the columns cut instead of the batch: a workgroup's slab holds all
// batch rows of a chunk (LPE lanes of E values: 64, 16 or 4 FP32 ones) for
// cols = kDotsBytes / (16 LPE) columns, so that every stored entry is read
// once, by the workgroup (rows [tile * st, + st), its block of columns), and
// its gradient written once. 16 lanes (a DPP row) take a row's entries of
// the block, 16 at a time, 16 / LPE per step: entry l of the 16 is loaded by
// lane l, its LDS address goes to the lanes of its group by a DPP broadcast,
// each lane multiplies its batch rows' values of G (in registers for the
// row), and a fold leaves entry l's sum with lane l. The column's 16-byte
// pieces are permuted by its number (dots_at), so that neither the slab's
// writes (a wave writes one piece of 64 columns) nor its reads (LPE = 16: the
// 256 bytes of 4 columns) meet on banks. part[i * m + r] is the first entry
// of row r at or past column i * kDotsGrain (columns ascend within a row); PART
// as above.
constexpr int kDotsBytes = 128 * 1024;
constexpr int kDotsGrain = 512;

template <int LPE>
constexpr int dots_cols() {
    return kDotsBytes / (16 * LPE);
}

// byte offset of piece 0 of column c; piece i is at the offset xor i * 16
template <int LPE>
__device__ __forceinline__ int dots_at(int c) {
    return c * (16 * LPE) ^ (((c / (16 / LPE)) & (LPE - 1)) << 4);
}

// v[t] summed over the LPE lanes of each group, for the 16 / P entries t of
// every lane's group; lane l of the row ends with entry l's sum.
template <int LPE, typename T>
__device__ __forceinline__ T dots_fold(const T (&v)[LPE]) {
    const int lane = lane_id();
    if constexpr (LPE == 1) {
        return v[0];
    } else {
        const bool h0 = lane & 1, h1 = lane & 2;
        T out = (T)0;
#pragma unroll
        for (int q = 0; q < LPE / 4; ++q) {
            const T a = (h0 ? v[4 * q + 1] : v[4 * q]) + dpp<kDppXor1>(h0 ? v[4 * q] : v[4 * q + 1]);
            const T b = (h0 ? v[4 * q + 3] : v[4 * q + 2]) + dpp<kDppXor1>(h0 ? v[4 * q + 2] : v[4 * q + 3]);
            T s = (h1 ? b : a) + dpp<kDppXor2>(h1 ? a : b);
            if constexpr (LPE == 16) {
                s += dpp<kDppRor4>(s);
                s += dpp<kDppRor8>(s);
                out = ((lane >> 2) & 3) == q ? s : out;
            } else {
                out = s;
            }
        }
        return out;
    }
}

// lane t of the group's loaded word, to all its lanes
template <int LPE, int t>
__device__ __forceinline__ int dots_bcast(int v) {
    if constexpr (LPE == 16) return dpp_word<kDppBcast + t>(v);
    if constexpr (LPE == 4) return dpp_word<0x55 * t>(v);
    return v;
}

template <typename T, int LPE, int... t>
__device__ __forceinline__ T dots_step(const char* slab, int at, int mine, const T (&gv)[SlabVec<T>::E],
                                       std::integer_sequence<int, t...>) {
    constexpr int E = SlabVec<T>::E;
    T v[LPE];
    auto one = [&](int tt, int a) {
        const SlabVec<T> x = *(const SlabVec<T>*)(slab + (a ^ mine));
        T s = gv[0] * x.v[0];
#pragma unroll
        for (int e = 1; e < E; ++e) s = fma_t(gv[e], x.v[e], s);
        v[tt] = s;
    };
    (one(t, dots_bcast<LPE, t>(at)), ...);
    return dots_fold<LPE, T>(v);
}

template <typename T, int LPE, bool PART>
__global__ __launch_bounds__(kSlabThreads) void k_slab_dots(int32_t m, int32_t n, int32_t nnz, int32_t B, int32_t st,
                                                            int32_t nblk, const int32_t* __restrict__ row_ptr,
                                                            const int32_t* __restrict__ part,
                                                            const int32_t* __restrict__ col_idx,
                                                            const T* __restrict__ G, const T* __restrict__ X,
                                                            T* __restrict__ dvals) {
    constexpr int E = SlabVec<T>::E, NB = LPE * E;
    constexpr int cols = dots_cols<LPE>(), grains = cols / kDotsGrain;
    extern __shared__ __align__(16) char s_raw[];
    char* slab = s_raw;
    const int64_t t = xcd_tile(blockIdx.x, gridDim.x);
    const int32_t tile = (int32_t)(t / nblk), blk = (int32_t)(t % nblk);
    const int32_t j0 = tile * st, c0 = blk * cols;
    const int32_t ns = min(st, m - j0), width = min(cols, n - c0);
    const int g = lane_id() % kSlabLanes;
    const int mine = (g % LPE) << 4;
    const int s0 = threadIdx.x / kSlabLanes;
    const int rounds = (ns + kSlabGroups - 1) / kSlabGroups;
    const auto bidx = buffer_of(col_idx, nnz * 4);
    for (int32_t b0 = 0; b0 < B; b0 += NB) {
        if (b0 > 0) __syncthreads();
        // the slab: a thread takes E batch rows of one column at a time (the
        // lanes of a wave 64 neighbouring columns), all loads before the stores
        constexpr int kPer = LPE * cols / kSlabThreads;
        SlabVec<T> x[kPer];
#pragma unroll
        for (int p = 0; p < kPer; ++p) {
            const int q = p * kSlabThreads + (int)threadIdx.x;
            const int c = q % cols, i = __builtin_amdgcn_readfirstlane(q / cols);
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int b = b0 + i * E + e;
                x[p].v[e] = buffer_value<T>(buffer_of(X + (int64_t)b * n + c0, b < B ? width * (int)sizeof(T) : 0),
                                            c * (int)sizeof(T));
            }
        }
#pragma unroll
        for (int p = 0; p < kPer; ++p) {
            const int q = p * kSlabThreads + (int)threadIdx.x;
            const int c = q % cols, i = q / cols;
            if (c < width) *(SlabVec<T>*)(slab + (dots_at<LPE>(c) ^ (i << 4))) = x[p];
        }
        // a row's bounds in the block and its values of G, one round ahead;
        // its first 16 column indices too
        auto bounds = [&](int r, int& k0, int& k1, T (&gv)[E]) {
            const int s = r * kSlabGroups + s0;
            k0 = k1 = 0;
#pragma unroll
            for (int e = 0; e < E; ++e) gv[e] = (T)0;
            if (s < ns) {
                const int64_t j = j0 + s;
                if constexpr (PART) {
                    const int32_t p = blk * grains;
                    k0 = blk > 0 ? part[p * (int64_t)m + j] : row_ptr[j];
                    k1 = blk + 1 < nblk ? part[(p + grains) * (int64_t)m + j] : row_ptr[j + 1];
                } else {
                    k0 = row_ptr[j];
                    k1 = row_ptr[j + 1];
                    if (blk > 0) k0 = first_from(col_idx, k0, k1, c0);
                    if (blk + 1 < nblk) k1 = first_from(col_idx, k0, k1, c0 + cols);
                }
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const int b = b0 + (g % LPE) * E + e;
                    if (b < B) gv[e] = G[(int64_t)b * m + j];
                }
            }
        };
        int ka, kb, kc, kd;
        T ga[E], gc[E];
        bounds(0, ka, kb, ga);
        bounds(1, kc, kd, gc);
        int c = buffer_value<int>(bidx, (ka + g) * 4);
        __syncthreads();
        for (int r = 0; r < rounds; ++r) {
            int ke, kf;
            T ge[E];
            bounds(r + 2, ke, kf, ge);
            int k = ka;
            bool more;
            do {
                more = __any(k + kSlabLanes < kb);  // uniform over the wave
                const bool on = k + g < kb;
                const int at = on ? dots_at<LPE>(c - c0) : 0;
                c = buffer_value<int>(bidx, ((more ? k + kSlabLanes : kc) + g) * 4);
                const T s = dots_step<T, LPE>(slab, at, mine, ga, std::make_integer_sequence<int, LPE>{});
                if (on) dvals[k + g] = b0 > 0 ? dvals[k + g] + s : s;
                k += kSlabLanes;
            } while (more);
            ka = kc;
            kb = kd;
            kc = ke;
            kd = kf;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                ga[e] = gc[e];
                gc[e] = ge[e];
            }
        }
    }
}

// part[blk * nseg + j]: the first entry of segment j whose index is at or
// past blk * cb (the indices ascend within a segment).
__global__ __launch_bounds__(kBlock) void k_slab_part(int32_t nseg, int32_t nblk, int32_t cb,
                                                      const int32_t* __restrict__ seg_ptr,
                                                      const int32_t* __restrict__ idx, int32_t* __restrict__ part) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= (int64_t)nseg * nblk) return;
    const int32_t blk = (int32_t)(i / nseg), j = (int32_t)(i % nseg);
    part[i] = first_from(idx, seg_ptr[j], seg_ptr[j + 1], blk * cb);
}

// ------------------------------------------------------------------ host
SlabBlocks slab_blocks(int32_t N) {
    SlabBlocks b;
    b.nblk = (int32_t)std::max<int64_t>(1, ceil_div(N, slab_cols(2)));
    b.cb = (int32_t)ceil_div(std::max(N, 1), b.nblk);
    return b;
}

SlabBlocks dots_blocks(int32_t n) {
    SlabBlocks b;
    b.nblk = (int32_t)std::max<int64_t>(1, ceil_div(n, kDotsGrain));
    b.cb = kDotsGrain;
    return b;
}

spx_status slab_part_build(int32_t nseg, const SlabBlocks& b, const int32_t* seg_ptr, const int32_t* idx,
                           int32_t* part, hipStream_t s) {
    k_slab_part<<<(unsigned)ceil_div((int64_t)nseg * b.nblk, kBlock), kBlock, 0, s>>>(nseg, b.nblk, b.cb, seg_ptr,
                                                                                      idx, part);
    SPX_HIP(hipGetLastError());
    return SPX_OK;
}

// Mean entries a segment must have per slab: below it the segment's share of
// a workgroup is its bounds, its fold and idle lanes.
constexpr double kSlabMinEntries = 8.0;

// 16-byte columns for few batch rows, and for operands of up to twice the
// columns
template <typename T>
static int slab_width(int32_t N, int32_t B) {
    constexpr int E = SlabVec<T>::E;
    if (N > slab_cols(1)) return 0;
    return N > slab_cols(2) || B <= E ? 1 : 2;
}

// the entries' arrays are addressed by 32-bit byte offsets
static bool slab_addresses(int32_t nnz, int dtype) { return (int64_t)nnz * (dtype == SPX_F64 ? 8 : 4) < (int64_t(1) << 31); }

// Segments per workgroup and batch rows per workgroup of the gather.
struct SlabTiling {
    int32_t st, nchunk;
};
static SlabTiling slab_tiling(int32_t nseg, int32_t B, int NB, int cus) {
    SlabTiling t;
    t.nchunk = (int32_t)ceil_div(B, NB);
    // about a workgroup per CU (the slab fills its LDS), and enough segments
    // in each for its 64 groups
    const int64_t want = std::max<int64_t>(1, cus / t.nchunk);
    t.st = (int32_t)std::min<int64_t>(kSlabMaxSegs, std::max<int64_t>(kSlabGroups, ceil_div(nseg, want)));
    return t;
}

// Whether the gather through slabs of cb columns is the faster one, by what
// the two take in us on a chip of 256 CUs. The slab kernel works by
// workgroups, one per CU: for each slab a fill, then rounds of 64 segments that
// cost at least a step of 64 entries each, again for every 4 to 8 FP32 (2 to 4
// FP64) batch rows. The gather from L2 (k_seg_gather behind a transpose) has a
// wave per segment and 64 batch rows, whatever the batch: its entries at the
// chip's rate, or one segment's chain where there are few; past 8 MB the
// B-minor copy no longer lies in the L2s. The constants are a fit to 2368
// products (forward with 256 to 8192 columns, dX over 1 to 64 slabs, 8 to 512
// entries per segment and slab, B = 1 to 256, both types). The rule takes the
// slabs where they are more than 6 % slower in 25 of them (22 % at most); the
// mean alone (from 8 entries on) did in 529. L2 gather against slabs: 300000 x 4096
// with 8 entries a row, FP32, 74 against 184 us at B = 64 and 65 against 31 at
// B = 8; 100000 x 4096 at B = 64, FP32, 40 / 73 us with 16 entries a row, 98 /
// 79 with 64; FP64 100 / 155 with 32, 363 / 225 with 128; dX of 262144 x 4096
// (64 slabs) at B = 1, FP32, 48 / 140 us with 8 entries a row, 193 / 163 with 32.
static bool slab_gather_pays(int32_t nseg, int32_t N, int32_t nnz, int32_t B, int es, int W, int32_t nblk, int32_t cb) {
    constexpr int kCus = 256;
    const SlabTiling t = slab_tiling(nseg, B, W * 16 / es, kCus);
    const double grid = (double)ceil_div(nseg, t.st) * t.nchunk;
    const double rounds = (double)ceil_div(std::min(t.st, nseg), kSlabGroups);
    const double len = (double)nnz / nseg;
    const double steps = std::max(1.0, len / nblk / kSlabStep + 0.25);
    const double fill = 0.88 + 0.95 * W * cb / slab_cols(2);
    const double round = 0.2 + (0.06 * (4 + es) + 0.2 * W) * steps;
    const double slab_us = 4.5 + std::max(1.0, grid / kCus) * nblk * (fill + rounds * round);
    const double in_mb = (double)N * B * es * 1e-6;
    const double far = std::min(1.0, std::max(0.0, (in_mb - 8.0) / 24.0));
    const double rate_us = nseg * (0.08 + 0.013 * (es / 4) * len * (1.0 + 0.28 * far)) * 1e-3;
    const double l2_us = 10.4 + 0.5 * in_mb + (double)ceil_div(B, kWave) * std::max(rate_us, 0.11 * len);
    return slab_us < l2_us;
}

bool slab_gather_fits(int32_t nseg, int32_t N, int32_t nnz, int32_t B, int dtype, const SlabBlocks* blocks) {
    if (nseg <= 0 || N <= 0 || B <= 0 || !slab_addresses(nnz, dtype)) return false;
    const int es = dtype == SPX_F64 ? 8 : 4;
    const int32_t nblk = blocks ? blocks->nblk : 1, cb = blocks ? blocks->cb : N;
    const int W = es == 8 ? slab_width<double>(cb, B) : slab_width<float>(cb, B);
    return W > 0 && (double)nnz >= kSlabMinEntries * (double)nseg * nblk &&
           slab_gather_pays(nseg, N, nnz, B, es, W, nblk, cb);
}

// lanes that hold an entry's batch rows
static int dots_lanes(int32_t B, int dtype) {
    const int E = dtype == SPX_F64 ? 2 : 4;
    return B <= E ? 1 : B <= 4 * E ? 4 : 16;
}

// Segments (rows) per workgroup of the gradient of the values.
static int32_t dots_rows(int32_t m, int32_t nblk, int cus) {
    return (int32_t)std::max<int64_t>(kSlabGroups, ceil_div(m, std::max(1, cus / nblk)));
}

// With more batch rows than a slab holds a workgroup passes over its entries
// again, adding to what it stored, and there are no more workgroups for it: it
// takes half a chip of them and 16 entries per row and block to beat the
// gather from L2, which spreads every batch over the chip (FP32 at B = 256,
// gather against slabs in us: 2000 x 256 with 256 entries a row, 32 workgroups,
// 61 / 86; 2000 x 1024 with 32, 64 workgroups, 17 / 24; 16384 x 1024 with 16, 8
// to a block, 33 / 36; 16384 x 1024 with 32, 46 / 37; 2000 x 4096 with 128, 43 /
// 26. FP64 at B = 64: 2000 x 256 with 256, 37 / 57; 100000 x 256 with 16, 80 /
// 37). With the batch in one slab the slabs were the faster ones in all of
// 1110 products measured.
bool slab_dots_fits(int32_t m, int32_t n, int32_t nnz, int32_t B, int dtype) {
    if (m <= 0 || n <= 0 || B <= 0 || !slab_addresses(nnz, dtype)) return false;
    constexpr int kCus = 256;
    const int lanes = dots_lanes(B, dtype);
    const int32_t nblk = (int32_t)ceil_div(n, kDotsBytes / (16 * lanes));
    const bool again = B > lanes * (dtype == SPX_F64 ? 2 : 4);
    if (again && ceil_div(m, dots_rows(m, nblk, kCus)) * nblk < kCus / 2) return false;
    // and the table of bounds stays below the index array
    return (double)nnz >= (again ? 2 : 1) * kSlabMinEntries * (double)m * nblk &&
           nnz >= (int64_t)m * ceil_div(n, kDotsGrain);
}

static spx_status slab_cus(int* cus) {
    int dev = 0;
    SPX_HIP(hipGetDevice(&dev));
    SPX_HIP(hipDeviceGetAttribute(cus, hipDeviceAttributeMultiprocessorCount, dev));
    *cus = std::max(*cus, 1);
    return SPX_OK;
}

template <typename T, int W>
static spx_status slab_gather_w(int32_t nseg, int32_t N, int32_t nnz, int32_t B, const SlabBlocks& b, const int32_t* seg_ptr,
                                const int32_t* part, const int32_t* idx, const T* vals, const T* in, T* out,
                                hipStream_t s) {
    int cus = 0;
    SPX_TRY(slab_cus(&cus));
    const auto [st, nchunk] = slab_tiling(nseg, B, W * SlabVec<T>::E, cus);
    const int64_t grid = ceil_div(nseg, st) * nchunk;
    if (grid > 0x7fffffff) return fail(SPX_ERR_SHAPE, "batch gather: too many batch rows");
    const size_t lds = slab_gather_lds<T, W>(b.cb, st);
    const auto kernel = part || b.nblk == 1 ? k_slab_gather<T, W, true> : k_slab_gather<T, W, false>;
    SPX_HIP(hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    kernel<<<(unsigned)grid, kSlabThreads, lds, s>>>(nseg, N, nnz, B, st, nchunk, b.nblk, b.cb, seg_ptr, part, idx,
                                                     vals, in, out);
    SPX_HIP(hipGetLastError());
    return SPX_OK;
}

template <typename T>
static spx_status slab_gather_t(int32_t nseg, int32_t N, int32_t nnz, int32_t B, const SlabBlocks* blocks, const int32_t* seg_ptr,
                                const int32_t* part, const int32_t* idx, const void* vals, const void* in, void* out,
                                hipStream_t s) {
    const SlabBlocks b = blocks ? *blocks : SlabBlocks{1, N};
    if (slab_width<T>(b.cb, B) == 2)
        return slab_gather_w<T, 2>(nseg, N, nnz, B, b, seg_ptr, part, idx, (const T*)vals, (const T*)in, (T*)out, s);
    return slab_gather_w<T, 1>(nseg, N, nnz, B, b, seg_ptr, part, idx, (const T*)vals, (const T*)in, (T*)out, s);
}

spx_status slab_gather(int32_t nseg, int32_t N, int32_t nnz, int32_t B, int dtype, const SlabBlocks* blocks, const int32_t* seg_ptr,
                       const int32_t* part, const int32_t* idx, const void* vals, const void* in, void* out,
                       hipStream_t s) {
    if (dtype == SPX_F32) return slab_gather_t<float>(nseg, N, nnz, B, blocks, seg_ptr, part, idx, vals, in, out, s);
    return slab_gather_t<double>(nseg, N, nnz, B, blocks, seg_ptr, part, idx, vals, in, out, s);
}

template <typename T, int LPE>
static spx_status slab_dots_l(int32_t m, int32_t n, int32_t nnz, int32_t B, const int32_t* row_ptr,
                              const int32_t* part, const int32_t* col_idx, const void* G, const void* X, void* dvals,
                              hipStream_t s) {
    int cus = 0;
    SPX_TRY(slab_cus(&cus));
    const int32_t nblk = (int32_t)ceil_div(n, dots_cols<LPE>());
    const int32_t st = dots_rows(m, nblk, cus);
    const int64_t grid = ceil_div(m, st) * nblk;
    if (grid > 0x7fffffff) return fail(SPX_ERR_SHAPE, "dvals: too many blocks");
    const size_t lds = (size_t)std::min(n, dots_cols<LPE>()) * 16 * LPE;
    const auto kernel = part || nblk == 1 ? k_slab_dots<T, LPE, true> : k_slab_dots<T, LPE, false>;
    SPX_HIP(hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kDotsBytes));
    // the permuted pieces of the last columns stay within their column
    kernel<<<(unsigned)grid, kSlabThreads, lds, s>>>(m, n, nnz, B, st, nblk, row_ptr, part, col_idx, (const T*)G,
                                                     (const T*)X, (T*)dvals);
    SPX_HIP(hipGetLastError());
    return SPX_OK;
}

template <typename T>
static spx_status slab_dots_t(int32_t m, int32_t n, int32_t nnz, int32_t B, int dtype, const int32_t* row_ptr,
                              const int32_t* part, const int32_t* col_idx, const void* G, const void* X, void* dvals,
                              hipStream_t s) {
    switch (dots_lanes(B, dtype)) {
        case 1: return slab_dots_l<T, 1>(m, n, nnz, B, row_ptr, part, col_idx, G, X, dvals, s);
        case 4: return slab_dots_l<T, 4>(m, n, nnz, B, row_ptr, part, col_idx, G, X, dvals, s);
        default: return slab_dots_l<T, 16>(m, n, nnz, B, row_ptr, part, col_idx, G, X, dvals, s);
    }
}

spx_status slab_dots(int32_t m, int32_t n, int32_t nnz, int32_t B, int dtype, const int32_t* row_ptr,
                     const int32_t* part, const int32_t* col_idx, const void* G, const void* X, void* dvals,
                     hipStream_t s) {
    if (dtype == SPX_F32) return slab_dots_t<float>(m, n, nnz, B, dtype, row_ptr, part, col_idx, G, X, dvals, s);
    return slab_dots_t<double>(m, n, nnz, B, dtype, row_ptr, part, col_idx, G, X, dvals, s);
}

}  // namespace spx
