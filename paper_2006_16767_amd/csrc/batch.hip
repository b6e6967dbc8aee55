// Batched SpMSpV: B sparse vectors of uneven sparsity, the plan of every
// vector chosen on the device.
//
//  k_batch_plan        one workgroup per vector: the decision trees evaluated on
//                      the Table 1 features (matrix features + nnz_x,
//                      x_sparsity, and where a tree reads them nnz_s and
//                      m_sparsity, from the lengths of the columns it selects)
//  k_batch_scan        deals the vectors that share passes over A out to groups
//                      and puts the others in order, the longest first
//  k_batch_slabs       the groups' vectors as dense slabs X^T (n rows = columns
//                      of A, one slot per vector, a cache line per row)
//  k_batch_stray       vectors whose indices do not ascend, into their slots
//  k_batch_fused       walks A once per group
//  k_batch_rows        every other vector, column-major by blocks of rows: a
//                      block of its Y in LDS, the selected columns' entries
//                      added there
//
// Groups: a vector whose plan is row-major (SpMV or CSR SpMSpV, any value type
// but BOOL), or whose entries reach kFusedMinXSparsity of n, joins a group that
// shares one pass over A: 32 vectors of 4-byte values, 16 of 8-byte ones.
// k_batch_fused walks work units of A for each group (at most fused_unit_nnz
// entries of at most kFusedUnitRows whole rows, or a piece of a longer row), a
// wave per unit. Pieces of split rows are added to Y with atomics (their rows
// of Y are zeroed beforehand); every other row is written once. Non-support
// entries meet zeros in the slab, so the bitvector validation of CSR SpMSpV
// becomes a product with zero.
//
// Where the table of column segments would be too large (batch_row_blocks),
// and for BOOL, k_batch_phase<A|B|C> runs the vectors of no group instead:
// persistent workgroups pop the items of one phase until its queue is drained
// (every workgroup exits once the queue head passes the item count):
//   A: row-major plans scatter x into the vector's bitvector / value slots;
//      column-major plans zero the vector's row of Y
//   B: one merge-path tile (or one row/entry chunk of the direct
//      distribution) of the vector's kernel
//   C: row-major balanced fix-up of tile carries, and the self-cleaning of
//      the bitvector / value slots (they are zero when a run starts)
// Items of one phase never wait for each other: the ordering between phases
// is the kernel boundary. Column-major plans write back with device atomics
// (the sort and bucket write-backs need per-vector pair buffers sized by
// nnz_s, which the host does not know without a sync).
//
// The kernels follow each other on the caller's stream. (The groups' walk on a
// stream of its own beside the other vectors': 1186 against 1035 us for 512
// vectors on R-MAT 2^18, since each starves the other of wave slots.)
#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.hpp"
#include "csc_tile.hpp"
#include "csr_tile.hpp"
#include "internal.hpp"

namespace spx {

constexpr int kBatchTile = 2048;     // merge tile (row-major and column-major)
constexpr int kFillChunk = 65536;    // rows of Y zeroed per phase-A item
constexpr int kScatterChunk = 2048;  // x entries scattered / cleared per item
constexpr int kCscDirectEntries = 64;
constexpr int kCscDirectLanes = 4;
// A fused group: the vectors whose values fill a 128-byte slab row (one cache
// line), 32 of 4-byte values, 16 of 8-byte ones.
constexpr int kSlabRow = 128;
template <int DT>
constexpr int group_size() {
    return kSlabRow / (int)sizeof(typename SR<DT>::X);
}
// a column-major vector this dense joins a fused group
constexpr double kFusedMinXSparsity = 0.02;
constexpr int kSplitZeroRows = 64;  // split rows of Y zeroed per item

constexpr int32_t kJoins = -2;  // BatchPlan::gslot until k_batch_scan deals the slots

struct BatchPlan {
    int32_t pattern, dist, wb, lanes;
    int32_t nnz_x, base;
    int32_t nA, nB, nC;
    int32_t gslot;  // slot in the fused groups, -1 if in none
    int64_t nnz_s;
};

struct BatchDev {
    int32_t m, n, nnz;
    const int32_t* row_ptr;
    const int32_t* col_idx;
    const void* vals;
    const int32_t* col_ptr;
    const int32_t* row_idx;
    const void* vals_csc;
    const int32_t* part;
    int64_t tiles_mat;
    int32_t B;
    int64_t cap_nnz_x;  // capacity of the per-entry arrays (host bound of vec_ptr[B])
    const int32_t* vec_ptr;
    const int32_t* idx;
    const void* val;
    void* Y;
    const DevSelector* sel;
    int32_t row_lanes;  // lanes per row of the row-major direct distribution
    // workspace
    BatchPlan* plans;
    int32_t* offs;    // 3 x (B + 1)
    int32_t* totals;  // 4 (with segs only [0]: the end of gvec)
    int32_t* queue;   // queue heads of the phases, [3] = err of the last run
    int32_t* err;     // of this run, cleared by k_batch_scan
    int32_t* excl_all;  // cap_nnz_x + B
    uint32_t* bits_all;  // B x nwords
    void* xd_all;        // B x n values
    int32_t* carry_row_all;  // B x tiles_mat
    void* carry_val_all;     // B x tiles_mat accumulators
    int64_t nwords;
    // fused row-major groups
    const int4* units;        // {first row, end row, first entry, end entry}
    int32_t nunits;
    const int32_t* split_rows;  // rows cut into several units
    int32_t nsplit;
    const int32_t* segs;  // the columns' first entries in each block of rows (null: k_batch_phase runs the rest)
    int32_t nblk;
    int32_t* gcount;  // vectors in groups
    int32_t* heads;   // of the queues of work units, 128 bytes apart
    int32_t* stray;   // a flag per vector: k_batch_slabs met an entry outside its tile
    int32_t* gvec;    // slot -> vector, behind the groups' slots the other vectors for k_batch_rows
    void* xt_all;     // a slab of (n + 1) x group_size values per group, row n zero
};

__device__ __forceinline__ int dev_tree_eval(const DevTree& t, const double* f) {
    int i = 0;
    for (int guard = 0; guard < 64 && i >= 0 && i < t.n; ++guard) {
        if (t.cls[i] >= 0) return t.cls[i];
        const int fi = t.feat[i];
        i = (fi >= 0 && fi < F_COUNT && f[fi] <= t.thr[i]) ? t.left[i] : t.right[i];
    }
    return 0;
}

// ------------------------------------------------------------------ plan
template <int DT>
__global__ __launch_bounds__(kBlock) void k_batch_plan(BatchDev a) {
    __shared__ int32_t s_tmp[kWavesPerBlock];
    const int b = blockIdx.x;
    const int base = a.vec_ptr[b];
    const int nx = a.vec_ptr[b + 1] - base;
    if (base < 0 || nx < 0 || (int64_t)a.vec_ptr[a.B] > a.cap_nnz_x || nx > a.n) {
        // vec_ptr disagrees with the capacity the host sized: no work, flag it
        if (threadIdx.x == 0) {
            BatchPlan z{};
            a.plans[b] = z;
            atomicOr(a.err, 2);
        }
        return;
    }
    int32_t* excl = a.segs ? nullptr : a.excl_all + base + b;
    const int32_t* idx = a.idx + base;
    const DevSelector& S = *a.sel;
    __shared__ int s_fuse;
    // host-known features first: a vector that joins a fused group or runs by
    // blocks of rows needs no prefix of its column lengths (unless the trees
    // read nnz_s)
    if (threadIdx.x == 0) {
        int fuse = 0;
        if (a.segs && nx == 0) {
            fuse = 2;
        } else if (DT != SPX_BOOL && a.units != nullptr && nx > 0 && !S.needs_nnz_s) {
            double f[F_COUNT];
            for (int i = 0; i < 9; ++i) f[i] = S.mfeat[i];
            f[9] = nx;
            f[10] = a.n > 0 ? (double)nx / a.n : 0.0;
            f[11] = f[12] = f[13] = 0.0;
            f[F_COUNTED] = 0.0;
            int pat = dev_tree_eval(S.t[0], f);
            if (pat < 0 || pat > 2) pat = 0;
            fuse = pat != SPX_PAT_CSC_SPMSPV || f[10] >= kFusedMinXSparsity ? 1 : (a.segs ? 2 : 0);
        }
        s_fuse = fuse;
    }
    __syncthreads();
    if (s_fuse) {
        if (threadIdx.x == 0) {
            BatchPlan p{};
            p.pattern = s_fuse == 1 ? SPX_PAT_SPMV : SPX_PAT_CSC_SPMSPV;
            p.dist = SPX_DIST_BALANCED;
            p.wb = SPX_WB_NONE;
            p.lanes = a.row_lanes;
            p.nnz_x = nx;
            p.base = base;
            p.nnz_s = -1;
            p.gslot = s_fuse == 1 ? kJoins : -1;
            a.plans[b] = p;
        }
        return;
    }
    constexpr int kIpt = 8;
    int32_t carry = 0;
    for (int c0 = 0; c0 < nx; c0 += kBlock * kIpt) {
        int32_t len[kIpt];
        int32_t sum = 0;
#pragma unroll
        for (int i = 0; i < kIpt; ++i) {
            const int e = c0 + threadIdx.x * kIpt + i;
            len[i] = 0;
            if (e < nx) {
                const int j = idx[e];
                len[i] = a.col_ptr[j + 1] - a.col_ptr[j];
            }
            sum += len[i];
        }
        int32_t tot;
        const int32_t incl = block_incl_scan(sum, s_tmp, &tot);
        int32_t run = carry + incl - sum;
#pragma unroll
        for (int i = 0; i < kIpt; ++i) {
            const int e = c0 + threadIdx.x * kIpt + i;
            if (excl && e < nx) excl[e] = run;
            run += len[i];
        }
        carry += tot;
    }
    if (threadIdx.x != 0) return;
    if (excl) excl[nx] = carry;
    double f[F_COUNT];
    for (int i = 0; i < 9; ++i) f[i] = S.mfeat[i];
    f[9] = nx;
    f[10] = a.n > 0 ? (double)nx / a.n : 0.0;
    f[11] = carry;
    f[12] = a.nnz > 0 ? (double)carry / a.nnz : 0.0;
    f[13] = (double)carry / (double)(nx > 0 ? nx : 1);
    f[F_COUNTED] = 1.0;
    BatchPlan p;
    p.pattern = dev_tree_eval(S.t[0], f);
    if (p.pattern < 0 || p.pattern > 2) p.pattern = 0;
    p.gslot = -1;
    const bool fusable = DT != SPX_BOOL && a.units != nullptr && nx > 0;
    if (fusable && (p.pattern != SPX_PAT_CSC_SPMSPV || f[10] >= kFusedMinXSparsity)) {
        if (p.pattern == SPX_PAT_CSC_SPMSPV) p.pattern = SPX_PAT_SPMV;
        p.gslot = kJoins;
    }
    p.dist = dev_tree_eval(S.t[1 + p.pattern], f) == SPX_DIST_BALANCED ? SPX_DIST_BALANCED : SPX_DIST_DIRECT;
    p.wb = p.pattern == SPX_PAT_CSC_SPMSPV ? SPX_WB_ATOMIC : SPX_WB_NONE;
    p.lanes = a.row_lanes;
    p.nnz_x = nx;
    p.base = base;
    p.nnz_s = carry;
    if (p.gslot == kJoins || a.segs) {
        p.nA = p.nB = p.nC = 0;
    } else if (p.pattern == SPX_PAT_CSC_SPMSPV) {
        p.nA = (int32_t)ceil_div(a.m, kFillChunk);
        p.nB = p.dist == SPX_DIST_BALANCED ? (int32_t)ceil_div((int64_t)nx + carry, kBatchTile)
                                           : (int32_t)ceil_div(nx, kCscDirectEntries);
        p.nC = 0;
    } else {
        const int64_t rows_per_item = (int64_t)(kBlock / a.row_lanes) * 8;
        p.nA = (int32_t)ceil_div(nx, kScatterChunk);
        p.nB = p.dist == SPX_DIST_BALANCED ? (int32_t)a.tiles_mat : (int32_t)ceil_div(a.m, rows_per_item);
        p.nC = (p.dist == SPX_DIST_BALANCED ? 1 : 0) + (int32_t)ceil_div(nx, kScatterChunk);
    }
    a.plans[b] = p;
}

// ------------------------------------------------------------------ queue
// One ordered queue per phase, and the vectors of the fused groups in their
// order in the batch.
__global__ __launch_bounds__(kBlock) void k_batch_scan(BatchDev a) {
    __shared__ int32_t s_tmp[kWavesPerBlock];
    if (threadIdx.x == 0) {
        a.queue[3] = *a.err;
        *a.err = 0;
    }
    int32_t count = 0;
    for (int c0 = 0; c0 < a.B; c0 += kBlock) {
        const int b = c0 + threadIdx.x;
        const bool joins = b < a.B && a.plans[b].gslot == kJoins;
        int32_t tot;
        const int32_t incl = block_incl_scan(joins ? 1 : 0, s_tmp, &tot);
        if (joins) {
            const int slot = count + incl - 1;
            a.plans[b].gslot = slot;
            a.gvec[slot] = b;
            a.stray[b] = 0;
        }
        count += tot;
    }
    if (threadIdx.x == 0) *a.gcount = count;
    if (a.segs) {
        // the others behind them, the longest first (four bins per octave), so
        // that no long one starts when the rest is done
        constexpr int kBins = 128;
        __shared__ int32_t s_bin[kBins];
        auto bin_of = [](const BatchPlan& p) {
            const int k = (int)(__float_as_uint((float)max(p.nnz_x, 1)) >> 21) - (127 << 2);
            return kBins - 1 - min(k, kBins - 1);
        };
        for (int i = threadIdx.x; i < kBins; i += kBlock) s_bin[i] = 0;
        __syncthreads();  // and the slots of the groups are dealt
        auto rest = [&](int b) { return a.plans[b].gslot < 0; };
        for (int b = threadIdx.x; b < a.B; b += kBlock)
            if (rest(b)) atomicAdd(&s_bin[bin_of(a.plans[b])], 1);
        __syncthreads();
        const int v = threadIdx.x < kBins ? s_bin[threadIdx.x] : 0;
        int32_t tot;
        const int32_t incl = block_incl_scan(v, s_tmp, &tot);
        if (threadIdx.x < kBins) s_bin[threadIdx.x] = count + incl - v;
        if (threadIdx.x == 0) a.totals[0] = count + tot;  // without those that were refused
        __syncthreads();
        for (int b = threadIdx.x; b < a.B; b += kBlock)
            if (rest(b)) a.gvec[atomicAdd(&s_bin[bin_of(a.plans[b])], 1)] = b;
    }
    if (threadIdx.x < 8) a.heads[threadIdx.x * 32] = 0;
    if (a.segs) return;  // no queues
    for (int ph = 0; ph < 3; ++ph) {
        int32_t* off = a.offs + ph * (a.B + 1);
        int32_t carry = 0;
        for (int c0 = 0; c0 < a.B; c0 += kBlock) {
            const int b = c0 + threadIdx.x;
            int32_t v = 0;
            if (b < a.B) v = ph == 0 ? a.plans[b].nA : (ph == 1 ? a.plans[b].nB : a.plans[b].nC);
            int32_t tot;
            const int32_t incl = block_incl_scan(v, s_tmp, &tot);
            if (b < a.B) off[b] = carry + incl - v;
            carry += tot;
        }
        if (threadIdx.x == 0) {
            off[a.B] = carry;
            a.totals[ph] = carry;
        }
        __syncthreads();
    }
    if (threadIdx.x < 3) a.queue[threadIdx.x] = 0;
}

// ------------------------------------------------------------------ persistent
template <int DT>
union BatchLds {
    CsrTileLds<DT, kBatchTile> csr;
    CscTileLds<DT> csc;
};

// last b with off[b] <= item (off has B + 1 entries, non-decreasing)
__device__ __forceinline__ int find_vector(const int32_t* off, int B, int item) {
    int lo = 0, hi = B - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (off[mid] <= item)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

template <int DT, int L>
__device__ __forceinline__ void batch_rows_direct(const BatchDev& a, int64_t r0, int64_t r1, bool valid,
                                                  const typename SR<DT>::X* xd, const uint32_t* bits,
                                                  typename SR<DT>::Y* y) {
    using S = SR<DT>;
    const auto* vals = (const typename S::V*)a.vals;
    constexpr int G = kBlock / L;
    const int g = threadIdx.x / L, lane = threadIdx.x % L;
    for (int64_t row = r0 + g; row < r1; row += G) {
        const int k0 = a.row_ptr[row], k1 = a.row_ptr[row + 1];
        ChunkedAcc<DT, 4> acc;  // a partial sum per load slot: bounded chains on hub rows
        int k = k0 + lane;
        for (; k + 3 * L < k1; k += 4 * L) {
            int c[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) c[u] = a.col_idx[k + u * L];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (!valid || test_bit(bits, c[u]))
                    acc.part[u] = S::fma(S::val(vals, k + u * L), S::xval(xd, c[u]), acc.part[u]);
            acc.end_round();
        }
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            const int kk = k + u * L;
            if (kk < k1) {
                const int c = a.col_idx[kk];
                if (!valid || test_bit(bits, c)) acc.part[u] = S::fma(S::val(vals, kk), S::xval(xd, c), acc.part[u]);
            }
        }
        const typename S::Acc sum = group_reduce<DT, L>(acc.total());
        if (lane == 0) y[row] = S::out(sum);
    }
}

// Lane q's value, read into a scalar register (q uniform).
template <typename T>
__device__ __forceinline__ T lane_value(T v, int q) {
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(T, __builtin_amdgcn_readlane(__builtin_bit_cast(int32_t, v), q));
    } else {
        const uint64_t u = __builtin_bit_cast(uint64_t, v);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int32_t)(uint32_t)u, q);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int32_t)(uint32_t)(u >> 32), q);
        return __builtin_bit_cast(T, ((uint64_t)hi << 32) | lo);
    }
}

// 16 bytes of a slab row: the values of a lane's vectors.
template <typename X>
struct alignas(16) SlotVals {
    static constexpr int E = 16 / sizeof(X);
    X v[E];
};

// The groups' slabs, a tile of kSlabCols slab rows per step of a workgroup:
// where the tile's columns begin and end in each vector by search, its entries
// into LDS, whole lines out. Entries that are not where an ascending index
// list would have them flag their vector: every entry lies in the range of at
// least one tile (a tile ends where the next one begins), so k_batch_stray can
// put the flagged vectors right. Past the tiles: items that zero
// kSplitZeroRows split rows of Y for a group's vectors.
//
// Bound by the slab's bytes: 120 us (2.9 TB/s) for the 217
// vectors of density 2 % and more (14M entries) on R-MAT 2^18. Scattered
// stores to slabs kept zero between runs took 240 us with the zeroing of the
// other vectors' Y, and 112 us for clearing them again: a 4-byte store per
// entry and pass is an L2 request each, and neither pass can run beside the
// products.
constexpr int kSlabCols = 256;

template <int DT>
__global__ __launch_bounds__(kBlock) void k_batch_slabs(BatchDev a) {
    if constexpr (DT != SPX_BOOL) {  // BOOL vectors never join a group
        using X = typename SR<DT>::X;
        constexpr int GS = group_size<DT>(), E = SlotVals<X>::E;
        constexpr int kPitch = GS + 1;  // rows on different banks
        __shared__ X s_x[kSlabCols * kPitch];
        __shared__ int32_t s_vec[GS], s_at[GS], s_start[GS + 1];
        const int count = *a.gcount;
        const int64_t G = ceil_div(count, GS), T = ceil_div((int64_t)a.n + 1, kSlabCols);
        const int64_t zper = ceil_div(a.nsplit, kSplitZeroRows);
        const auto* val = (const X*)a.val;
        for (int64_t i = blockIdx.x; i < G * (T + zper); i += gridDim.x) {
            if (i >= G * T) {
                const int g = (int)((i - G * T) / zper);
                const int s0 = (int)((i - G * T) % zper) * kSplitZeroRows;
                const int ns = min(kSplitZeroRows, a.nsplit - s0);
                const int nvec = min(GS, count - g * GS);
                for (int t = threadIdx.x; t < ns * nvec; t += kBlock)
                    ((typename SR<DT>::Y*)a.Y)[(int64_t)a.gvec[g * GS + t % nvec] * a.m + a.split_rows[s0 + t / nvec]] =
                        (typename SR<DT>::Y)0;
                continue;
            }
            // an XCD's workgroups take neighbouring tiles: they share lines of
            // the sparser vectors
            const int64_t t = xcd_tile(i, G * T);
            const int g = (int)(t / T);
            const int c0 = (int)(t % T) * kSlabCols;
            const int rows = (int)min((int64_t)kSlabCols, (int64_t)a.n + 1 - c0);
            const int nvec = min(GS, count - g * GS);
            for (int e = threadIdx.x; e < kSlabCols * kPitch; e += kBlock) s_x[e] = (X)0;
            // eight lanes search a vector's list for the first entries that
            // are not below c0 and c0 + kSlabCols, nine ways a step
            const int v = threadIdx.x >> 3, l = threadIdx.x & 7;
            const bool mine = v < nvec;
            const int b = mine ? a.gvec[g * GS + v] : 0;
            const int base = mine ? a.vec_ptr[b] : 0;
            const int nx = mine ? a.vec_ptr[b + 1] - base : 0;
            const int32_t* idx = a.idx + base;
            int lo[2] = {0, 0}, hi[2] = {c0 == 0 ? 0 : nx, nx};
            if (c0 + rows > a.n) lo[1] = nx;
            while (__any(lo[0] < hi[0] || lo[1] < hi[1])) {
                int at[2], col[2];
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const int w = hi[k] - lo[k];
                    at[k] = lo[k] + (w >= 9 ? (l + 1) * (w / 9) : min(l, w - 1));
                    col[k] = w > 0 ? idx[at[k]] : 0;
                }
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const uint32_t m = (uint32_t)(__ballot(col[k] >= c0 + k * kSlabCols) >> (lane_id() & 56)) & 255u;
                    const int f = m ? __ffs(m) - 1 : 8;
                    const int up = __shfl(at[k], (lane_id() & 56) | min(f, 7), kWave);
                    const int below = __shfl(at[k], (lane_id() & 56) | max(f - 1, 0), kWave);
                    if (hi[k] > lo[k]) {
                        if (f < 8) hi[k] = up;
                        if (f > 0) lo[k] = below + 1;
                    }
                }
            }
            if (v < GS && l == 0) {
                s_vec[v] = b;
                s_start[v + 1] = max(0, lo[1] - lo[0]);
                s_at[v] = base + lo[0];
            }
            if (threadIdx.x == 0) s_start[0] = 0;
            __syncthreads();
            if (threadIdx.x < kWave) {
                int sum = threadIdx.x < GS ? s_start[threadIdx.x + 1] : 0;
                for (int d = 1; d < GS; d <<= 1) {
                    const int o = __shfl_up(sum, d, kWave);
                    if ((int)threadIdx.x >= d) sum += o;
                }
                if (threadIdx.x < GS) s_start[threadIdx.x + 1] = sum;
            }
            __syncthreads();
            const int total = s_start[GS];
            constexpr int kPer = 8;
            for (int e0 = threadIdx.x; e0 < total; e0 += kPer * kBlock) {
                int u[kPer], c[kPer];
                X x[kPer];
#pragma unroll
                for (int q = 0; q < kPer; ++q) {
                    const int e = min(e0 + q * kBlock, total - 1);
                    int w = 0;
#pragma unroll
                    for (int d = GS / 2; d > 0; d >>= 1)
                        if (s_start[w + d] <= e) w += d;
                    u[q] = w;
                    const int at = s_at[w] + e - s_start[w];
                    c[q] = a.idx[at];
                    x[q] = val[at];
                }
#pragma unroll
                for (int q = 0; q < kPer; ++q) {
                    const int r = c[q] - c0;
                    if (r >= 0 && r < rows && c[q] < a.n)
                        s_x[r * kPitch + u[q]] = x[q];
                    else
                        a.stray[s_vec[u[q]]] = 1;
                }
            }
            __syncthreads();
            auto* xt = (SlotVals<X>*)((X*)a.xt_all + ((int64_t)g * (a.n + 1) + c0) * GS);
#pragma unroll
            for (int q = 0; q < kSlabCols * 8 / kBlock; ++q) {
                const int e = q * kBlock + threadIdx.x;
                SlotVals<X> o;
#pragma unroll
                for (int k = 0; k < E; ++k) o.v[k] = s_x[(e >> 3) * kPitch + (e & 7) * E + k];
                if ((e >> 3) < rows) xt[e] = o;
            }
            __syncthreads();
        }
    }
}

// The flagged vectors' entries into their slots, in any order: a workgroup per
// slot of the groups.
template <int DT>
__global__ __launch_bounds__(kBlock) void k_batch_stray(BatchDev a) {
    if constexpr (DT != SPX_BOOL) {
        using X = typename SR<DT>::X;
        constexpr int GS = group_size<DT>();
        const int slot = blockIdx.x;
        if (slot >= *a.gcount) return;
        const int b = a.gvec[slot];
        if (!a.stray[b]) return;
        auto* xt = (X*)a.xt_all + (int64_t)(slot / GS) * (a.n + 1) * GS + slot % GS;
        for (int e = a.vec_ptr[b] + threadIdx.x; e < a.vec_ptr[b + 1]; e += kBlock)
            if (a.idx[e] >= 0 && a.idx[e] < a.n) xt[(int64_t)a.idx[e] * GS] = ((const X*)a.val)[e];
    }
}

// A wave's LDS in the fused walk: a unit's entries; for an entry that ends a
// row, where the row's sums go (kNoEnd for the others); the rows' sums, slot by
// slot, until they are stored. A row's 16-byte pieces are permuted by the row,
// so that the rows of one slot lie on different banks.
template <int DT>
constexpr int kUnitNnz = fused_unit_nnz((int)sizeof(typename SR<DT>::X));
template <int DT>
struct FusedEntry {
    int32_t col;
    typename SR<DT>::V val;
};
constexpr int kFusedSteps = 4;  // gathers in flight, twice
template <int DT>
struct FusedLds {
    alignas(16) typename SR<DT>::Acc sums[kFusedUnitRows * group_size<DT>()];
    // lane group h's entries from h * (len + 1), its ends from h * (len + 8):
    // the eight lane groups read from different banks
    alignas(16) uint16_t end[kUnitNnz<DT> + 8 * 8];
    FusedEntry<DT> e[kUnitNnz<DT> + 8];
    FusedEntry<DT> none[kFusedSteps];  // past the last step: the slab's zero row
    int64_t y[group_size<DT>()];  // where the vectors' Y begin
};
constexpr uint32_t kNoEnd = 0xffff;

// One work unit of A for the vectors of fused group g. Eight lanes hold the
// group's slots, 16 bytes each; the wave's eight lane groups each walk an eighth of the unit's
// entries, the next kFusedSteps gathers in flight while it adds the last ones (a
// gather reads eight whole slab rows, a cache line each). A lane group that passes a row's end leaves the
// row's sum (or the last piece of it) in LDS; the pieces of rows that run on
// into the next eighth are added at the end, in order. Then the unit's rows go
// out together, one run of consecutive rows per vector. A piece of a split row
// adds its sums to Y with atomics.
//
// 527 us for the seven groups of 217 vectors on R-MAT 2^18 (7.6M entries: 53M
// gathered lines, 100 G lines/s, 55 % of them from L2). With units of 512
// entries it took 587: 330 of that is what the units took without the gathers
// (90 of it the stores of Y, in lines that units share), and lines that all come
// from L2 would have saved 65. Longer units store longer runs of rows, but hold
// more LDS: 256 entries 725 us, 640 538, 768 527 (12 waves per CU), 1024 602.
// Two vectors per lane (512-byte gathers, three times the slab per group) took
// 1066 us beside the other vectors' walk; eight entries of one row per step, the
// lane groups' sums added at every row's end, twice the instructions; the next
// unit's entries loaded ahead gave nothing (602 against 588 us).
template <int DT, bool BUF>
__device__ __forceinline__ void batch_fused_unit(const BatchDev& a, int g, int32_t unit, FusedLds<DT>& L) {
    using S = SR<DT>;
    using X = typename S::X;
    using V = typename S::V;
    using Acc = typename S::Acc;
    constexpr int E = SlotVals<X>::E, GS = group_size<DT>();
    const int4 u = a.units[unit];
    const int r0 = u.x, nrows = u.y - u.x, k0 = u.z, cnt = u.w - u.z;
    const int lane = lane_id();
    const int q = lane >> 3, piece = (lane & 7) * 16;
    const int nvec = min(GS, *a.gcount - g * GS);
    const char* xt = (const char*)a.xt_all + (int64_t)g * (a.n + 1) * kSlabRow;
    const auto rsrc = buffer_of(xt, BUF ? (int)((int64_t)(a.n + 1) * kSlabRow) : 0);
    auto load = [&](int c) {
        if constexpr (BUF)
            return __builtin_bit_cast(SlotVals<X>, __builtin_amdgcn_raw_buffer_load_b128(rsrc, c * kSlabRow | piece, 0, 0));
        else
            return *(const SlotVals<X>*)(xt + (int64_t)c * kSlabRow + piece);
    };
    // lane i holds the end of row r0 + i - 1 in the unit's entries
    int rp = lane <= nrows ? a.row_ptr[r0 + lane] - k0 : 0;
    const bool split = nrows == 1 && (lane_value(rp, 0) != 0 || lane_value(rp, 1) != cnt);
    if (split) rp = lane == 0 ? 0 : cnt;
    if (lane < GS) L.y[lane] = lane < nvec ? (int64_t)a.gvec[g * GS + lane] * a.m : 0;
    // A streams through once per group: non-temporal, so that L2 keeps the
    // slab rows the gathers re-read
    constexpr int kPer = kUnitNnz<DT> / kWave;
    FusedEntry<DT> in[kPer];
#pragma unroll
    for (int p = 0; p < kPer; ++p) {
        const int i = p * kWave + lane;
        // past the unit's end: value 0 and the slab's zero row
        in[p].col = i < cnt ? __builtin_nontemporal_load(a.col_idx + k0 + i) : a.n;
        in[p].val = i < cnt ? __builtin_nontemporal_load((const V*)a.vals + k0 + i) : (V)0;
    }
    SlotVals<Acc> z;
#pragma unroll
    for (int e = 0; e < E; ++e) z.v[e] = S::zero();
    for (int i = lane; i < nrows * 8; i += kWave) *(SlotVals<Acc>*)(L.sums + i * E) = z;
    // lane group h takes the entries from h * len on; inv finds i / len for
    // i < 1024
    const int len = ((cnt + 7) / 8 + 2 * kFusedSteps - 1) / (2 * kFusedSteps) * (2 * kFusedSteps);
    const uint32_t inv = len > 0 ? ((1u << 20) + len - 1) / len : 0;
    auto group_of = [&](int i) { return (int)(((uint32_t)i * inv) >> 20); };
    // of row r, the lane's piece of its sums
    auto sums_at = [&](int r) { return r * 8 * 16 + ((r & 7) << 4); };
#pragma unroll
    for (int p = 0; p < kPer; ++p) {
        const int i = p * kWave + lane;
        if (i < 8 * len) L.e[i + group_of(i)] = in[p];
    }
    if (lane < kFusedSteps) L.none[lane] = FusedEntry<DT>{a.n, (V)0};
    for (int i = lane; i < len + 8; i += kWave) ((uint4*)L.end)[i] = uint4{~0u, ~0u, ~0u, ~0u};
    const int row_end = __shfl_down(rp, 1, kWave);  // of row lane, for lane < nrows
    const bool some = lane < nrows && row_end > rp;
    __builtin_amdgcn_wave_barrier();
    if (some) L.end[row_end - 1 + 8 * group_of(row_end - 1)] = (uint16_t)sums_at(lane);
    __builtin_amdgcn_wave_barrier();
    auto sums = [&](uint32_t at) { return (SlotVals<Acc>*)((char*)L.sums + (at ^ piece)); };
    SlotVals<Acc> acc = z;
    const FusedEntry<DT>* mine = L.e + q * (len + 1);
    const uint16_t* ends = L.end + q * (len + 8);
    struct Steps {
        FusedEntry<DT> e[kFusedSteps];
        SlotVals<X> x[kFusedSteps];
    } A, B;
    auto fetch = [&](Steps& s, const FusedEntry<DT>* from) {
#pragma unroll
        for (int t = 0; t < kFusedSteps; ++t) s.e[t] = from[t];
#pragma unroll
        for (int t = 0; t < kFusedSteps; ++t) s.x[t] = load(s.e[t].col);
    };
    auto use = [&](const Steps& s, uint32_t end01, uint32_t end23) {
#pragma unroll
        for (int t = 0; t < kFusedSteps; ++t) {
#pragma unroll
            for (int i = 0; i < E; ++i) acc.v[i] = S::fma(s.e[t].val, s.x[t].v[i], acc.v[i]);
            const uint32_t end = ((t < 2 ? end01 : end23) >> (t % 2 * 16)) & 0xffffu;
            if (end != kNoEnd) {
                *sums(end) = acc;
                acc = z;
            }
        }
    };
    static_assert(kFusedSteps == 4, "two words of ends per step");
    // a unit of empty rows has no entry in LDS to fetch
    fetch(A, len > 0 ? mine : L.none);
    for (int t0 = 0; t0 < len; t0 += 2 * kFusedSteps) {
        fetch(B, mine + t0 + kFusedSteps);
        const uint4 end = *(const uint4*)(ends + t0);
        use(A, end.x, end.y);
        fetch(A, t0 + 2 * kFusedSteps < len ? mine + t0 + 2 * kFusedSteps : L.none);
        use(B, end.z, end.w);
    }
    __builtin_amdgcn_wave_barrier();
    // the row that runs on past a lane group's eighth
    for (int h = 0; h < 8; ++h) {
        const int e = min((h + 1) * len, cnt);
        const uint64_t m = __ballot(some && rp < e && e < row_end);
        if (m == 0 || h * len >= cnt) continue;
        if (q == h) {
            SlotVals<Acc>* to = sums(sums_at(__ffsll((unsigned long long)m) - 1));
            SlotVals<Acc> sum = *to;
#pragma unroll
            for (int i = 0; i < E; ++i) sum.v[i] = S::add(sum.v[i], acc.v[i]);
            *to = sum;
        }
    }
    __builtin_amdgcn_wave_barrier();
    auto sum_of = [&](int r, int v) {
        return *(const Acc*)((const char*)L.sums + ((sums_at(r) ^ (v / E * 16)) | v % E * (int)sizeof(Acc)));
    };
    auto* Y = (typename S::Y*)a.Y + r0;
    if (split) {
        if (lane < nvec) S::atomic_add(Y + L.y[lane], sum_of(0, lane));
    } else {
        const int rr = lane % kFusedUnitRows;
        for (int v = lane / kFusedUnitRows; v < nvec; v += kWave / kFusedUnitRows)
            if (rr < nrows) __builtin_nontemporal_store(S::out(sum_of(rr, v)), Y + (L.y[v] + rr));
    }
    __builtin_amdgcn_wave_barrier();
}

// The fused groups' work, one group after the other: units from eight queues
// (a workgroup's by its number, which goes round the XCDs), one ahead of the
// walk. (One queue per group and no unit ahead: the pops, atomics on one
// word, took 890 us in all against 652 for units dealt round the waves; dealt
// out, the last wave is 15 % behind. Units in runs of 64 on one XCD, whose
// rows of Y share cache lines: 691. Each XCD at a group of its own: no faster
// either, since every L2 sees the same share of a slab.)
constexpr int kFusedQueues = 8;

template <int DT, bool BUF>
__global__ __launch_bounds__(kBlock) void k_batch_fused(BatchDev a) {
    if constexpr (DT != SPX_BOOL) {  // BOOL vectors never join a group
        __shared__ FusedLds<DT> s_lds[kWavesPerBlock];
        FusedLds<DT>& L = s_lds[__builtin_amdgcn_readfirstlane(wave_id())];
        const int64_t total = ceil_div(*a.gcount, group_size<DT>()) * a.nunits;
        const int x = blockIdx.x % kFusedQueues;
        auto pop = [&] { return lane_id() == 0 ? atomicAdd(a.heads + x * 32, 1) : 0; };
        int next = pop();
        for (;;) {
            const int64_t i = (int64_t)__builtin_amdgcn_readfirstlane(next) * kFusedQueues + x;
            if (i >= total) break;
            next = pop();
            const int g = (int)(i / a.nunits);
            batch_fused_unit<DT, BUF>(a, g, (int)(i - (int64_t)g * a.nunits), L);
        }
    }
}

// The vectors of no group, by blocks of rows: a workgroup holds kRowsBytes of
// one vector's Y in LDS, adds the products of the selected columns' entries in
// those rows to it there, and stores it. A column's entries ascend by row, so a
// block's are one segment, found in a table (k_segs). A thread reads one
// segment's bounds; then the wave takes its 64 segments as one run of entries,
// 64 at a step. The blocks of one vector follow each other on one XCD: they
// read neighbouring segments, in the same cache lines.
//
// Bound by the chain from index to segment to entries, by its cache lines
// (three per segment, 14M) and by Y: 150 us for the 295 vectors below a density
// of 2 % on R-MAT 2^18 (4.7M segments of 1.8 entries on average, of 13 in the
// first block; 310 MB of Y), 190 when the vectors came in the batch's order and
// the last long one ran on alone. 55 of it is zeroing and storing Y; 16 are adds
// to one row by several lanes. In the batch's order, four lanes to a segment
// and a wave to a long one took 219 us (where all segments are short it is 5 %
// faster), 512 threads 252; 128 KB of Y per workgroup 182. Atomics into Y took
// 760 us, and 54 us for zeroing Y before: the chip does 21 G scattered
// atomics/s, from one XCD or all.
constexpr int kRowsBytes = 65536;
constexpr int kRowsThreads = 1024;
constexpr int kRowsSteps = 4;

// Lane dst / 4 gets the value (ds_permute moves words).
template <typename T>
__device__ __forceinline__ T permute_to(int dst, T v) {
    uint32_t w[sizeof(T) / 4];
    __builtin_memcpy(w, &v, sizeof(T));
#pragma unroll
    for (int i = 0; i < (int)(sizeof(T) / 4); ++i) w[i] = (uint32_t)__builtin_amdgcn_ds_permute(dst, (int)w[i]);
    __builtin_memcpy(&v, w, sizeof(T));
    return v;
}

template <int DT>
__global__ __launch_bounds__(kRowsThreads) void k_batch_rows(BatchDev a, int32_t b0) {
    if constexpr (DT != SPX_BOOL) {
        using S = SR<DT>;
        using Acc = typename S::Acc;
        extern __shared__ __align__(16) char s_raw[];
        __shared__ unsigned long long s_starts[kRowsThreads / kWave][kRowsSteps];
        Acc* y = (Acc*)s_raw;
        constexpr int R = kRowsBytes / (int)sizeof(Acc);
        const int i = blockIdx.x / 8;
        const int at = *a.gcount + b0 + i / a.nblk * 8 + (int)(blockIdx.x % 8), blk = i % a.nblk;
        if (at >= a.totals[0]) return;
        const int b = a.gvec[at];
        const BatchPlan p = a.plans[b];
        for (int r = threadIdx.x; r < kRowsBytes / 16; r += kRowsThreads) ((uint4*)s_raw)[r] = uint4{0, 0, 0, 0};
        __syncthreads();
        const int32_t* __restrict__ idx = a.idx + p.base;
        const auto* __restrict__ xv = (const typename S::X*)a.val + p.base;
        const auto* __restrict__ vals = (const typename S::V*)a.vals_csc;
        const int r0 = blk * R, lane = lane_id();
        unsigned long long* starts = s_starts[wave_id()];
        for (int c0 = 0; c0 < p.nnz_x; c0 += kRowsThreads) {
            const int e = c0 + threadIdx.x;
            int k0 = 0, len = 0;
            typename S::X x = (typename S::X)0;
            if (e < p.nnz_x) {
                const int32_t* t = a.segs + (int64_t)idx[e] * a.nblk + blk;
                k0 = t[0];
                len = t[1] - k0;
                x = xv[e];
            }
            // the wave's segments end to end: position p of the run belongs to
            // the last non-empty segment that starts at or before it, found
            // as a rank in the bits of the starts (kRowsSteps words of 64
            // positions at a time); first, the non-empty segments side by side
            const uint64_t some = __ballot(len > 0);
            const int at = __popcll(some & ((1ull << lane) - 1ull));
            const int incl = wave_incl_scan(len);
            const int total = __shfl(incl, kWave - 1, kWave);
            const int dst = (len > 0 ? at : kWave - 1) * 4;
            int start = incl - len, shift = k0 - start;  // entry = position + shift
            if (__popcll(some) < kWave) {  // else they are
                const int n0 = __popcll(some);
                start = __builtin_amdgcn_ds_permute(dst, start);
                shift = __builtin_amdgcn_ds_permute(dst, shift);
                x = permute_to(dst, x);
                if (lane >= n0) start = total;
            }
            int before = 0;
            for (int p0 = 0; p0 < total; p0 += kRowsSteps * kWave) {
                if (lane < kRowsSteps) starts[lane] = 0;
                __builtin_amdgcn_wave_barrier();
                const int o = start - p0;
                if (o >= 0 && o < kRowsSteps * kWave && start < total)
                    atomicOr(&starts[o / kWave], 1ull << (o % kWave));
                __builtin_amdgcn_wave_barrier();
                int row[kRowsSteps], k[kRowsSteps];
                typename S::X xs[kRowsSteps];
                typename S::V v[kRowsSteps];
#pragma unroll
                for (int t = 0; t < kRowsSteps; ++t) {
                    const uint64_t w = starts[t];
                    const int rank = before + __popcll(w & (~0ull >> (kWave - 1 - lane))) - 1;
                    before += __popcll(w);
                    const int p = p0 + t * kWave + lane;
                    k[t] = min(p, total - 1) + __shfl(shift, rank, kWave);
                    xs[t] = __shfl(x, rank, kWave);
                }
#pragma unroll
                for (int t = 0; t < kRowsSteps; ++t) {
                    row[t] = a.row_idx[k[t]];
                    v[t] = vals[k[t]];
                }
#pragma unroll
                for (int t = 0; t < kRowsSteps; ++t)
                    if (p0 + t * kWave + lane < total) S::lds_atomic_add(&y[row[t] - r0], S::mul(v[t], xs[t]));
            }
        }
        __syncthreads();
        const int nr = min(R, a.m - r0);
        auto* out = (typename S::Y*)a.Y + (int64_t)b * a.m + r0;
        for (int r = threadIdx.x; r < nr; r += kRowsThreads) __builtin_nontemporal_store(S::out(y[r]), out + r);
    }
}

// The first entry of column j in rows from block k on, at j * nblk + k; nnz at
// the end, so that each entry of the table ends the segment before it.
__global__ __launch_bounds__(kBlock) void k_segs(int64_t total, int32_t nblk, int32_t rows, int32_t nnz,
                                                 const int32_t* __restrict__ col_ptr,
                                                 const int32_t* __restrict__ row_idx, int32_t* __restrict__ segs) {
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i <= total; i += (int64_t)gridDim.x * kBlock) {
        if (i == total) {
            segs[i] = nnz;
            continue;
        }
        const int64_t j = i / nblk;
        const int64_t from = (i - j * nblk) * rows;
        int lo = col_ptr[j], hi = from ? col_ptr[j + 1] : lo;
        while (lo < hi) {
            const int mid = lo + ((hi - lo) >> 1);
            if (row_idx[mid] < from)
                lo = mid + 1;
            else
                hi = mid;
        }
        segs[i] = lo;
    }
}

template <int DT, int PH>
__global__ __launch_bounds__(kBlock) void k_batch_phase(BatchDev a) {
    using S = SR<DT>;
    using Acc = typename S::Acc;
    __shared__ BatchLds<DT> L;
    __shared__ int32_t s_item;
    // the phase's item offsets per vector, in LDS when they fit (the vector
    // of an item is found by a binary search over them)
    constexpr int kOffLds = 2048;
    __shared__ int32_t s_voff[kOffLds];
    const int32_t total = a.totals[PH];
    constexpr int ph = PH;
    const bool off_in_lds = a.B + 1 <= kOffLds;
    if (off_in_lds)
        for (int i = threadIdx.x; i <= a.B; i += kBlock) s_voff[i] = a.offs[ph * (a.B + 1) + i];
    const auto* vals = (const typename S::V*)a.vals;
    const auto* vals_csc = (const typename S::V*)a.vals_csc;
    const auto* xval_all = (const typename S::X*)a.val;
    for (;;) {
        if (threadIdx.x == 0) s_item = atomicAdd(a.queue + PH, 1);
        __syncthreads();
        const int item = s_item;
        __syncthreads();
        if (item >= total) break;
        const int32_t* off = a.offs + ph * (a.B + 1);
        const int b = find_vector(off_in_lds ? s_voff : off, a.B, item);
        const int j = item - off[b];
        const BatchPlan p = a.plans[b];
        auto* Yb = (typename S::Y*)a.Y + (int64_t)b * a.m;
        uint32_t* bits = a.bits_all + (int64_t)b * a.nwords;
        auto* xd = S::kVals ? (typename S::X*)a.xd_all + (int64_t)b * a.n : (typename S::X*)nullptr;
        const int32_t* idx = a.idx + p.base;
        const typename S::X* xv = S::kVals ? xval_all + p.base : nullptr;
        const bool csc = p.pattern == SPX_PAT_CSC_SPMSPV;
        if constexpr (PH == 0) {
            if (csc) {
                const int64_t r0 = (int64_t)j * kFillChunk;
                const int64_t r1 = std::min<int64_t>(r0 + kFillChunk, a.m);
                for (int64_t r = r0 + threadIdx.x; r < r1; r += kBlock) Yb[r] = (typename S::Y)0;
            } else {
                const int e1 = std::min(p.nnz_x, (j + 1) * kScatterChunk);
                for (int e = j * kScatterChunk + threadIdx.x; e < e1; e += kBlock) {
                    const int c = idx[e];
                    atomicOr(&bits[c >> 5], 1u << (c & 31));
                    if constexpr (S::kVals) xd[c] = xv[e];
                }
            }
        } else if constexpr (PH == 1) {
            if (csc) {
                const int32_t* excl = a.excl_all + p.base + b;
                if (p.dist == SPX_DIST_BALANCED) {
                    csc_merge_tile<DT>(j, p.nnz_x, p.nnz_s, idx, xv, a.col_ptr, a.row_idx, vals_csc, Excl{excl, nullptr},
                                       EmitAtomic<DT>{Yb}, L.csc);
                } else {
                    const int e = j * kCscDirectEntries + threadIdx.x / kCscDirectLanes;
                    if (e < p.nnz_x)
                        csc_direct_entry<DT, kCscDirectLanes>(e, threadIdx.x % kCscDirectLanes, idx, xv, a.col_ptr,
                                                              a.row_idx, vals_csc, Excl{nullptr, nullptr},
                                                              EmitAtomic<DT>{Yb});
                }
            } else {
                const bool valid = p.pattern == SPX_PAT_CSR_SPMSPV || DT == SPX_BOOL;
                if (p.dist == SPX_DIST_BALANCED) {
                    int32_t* crow = a.carry_row_all + (int64_t)b * a.tiles_mat;
                    Acc* cval = (Acc*)a.carry_val_all + (int64_t)b * a.tiles_mat;
                    if (valid)
                        csr_merge_tile<DT, true, kBatchTile>(j, a.m, a.row_ptr, a.col_idx, vals, xd, bits, Yb, a.part,
                                                             crow, cval, L.csr);
                    else
                        csr_merge_tile<DT, false, kBatchTile>(j, a.m, a.row_ptr, a.col_idx, vals, xd, bits, Yb, a.part,
                                                              crow, cval, L.csr);
                } else {
                    const int64_t rpi = (int64_t)(kBlock / p.lanes) * 8;
                    const int64_t r0 = (int64_t)j * rpi, r1 = std::min<int64_t>(r0 + rpi, a.m);
                    switch (p.lanes) {
                        case 1: batch_rows_direct<DT, 1>(a, r0, r1, valid, xd, bits, Yb); break;
                        case 2: batch_rows_direct<DT, 2>(a, r0, r1, valid, xd, bits, Yb); break;
                        case 4: batch_rows_direct<DT, 4>(a, r0, r1, valid, xd, bits, Yb); break;
                        case 8: batch_rows_direct<DT, 8>(a, r0, r1, valid, xd, bits, Yb); break;
                        case 16: batch_rows_direct<DT, 16>(a, r0, r1, valid, xd, bits, Yb); break;
                        case 32: batch_rows_direct<DT, 32>(a, r0, r1, valid, xd, bits, Yb); break;
                        default: batch_rows_direct<DT, 64>(a, r0, r1, valid, xd, bits, Yb); break;
                    }
                }
            }
        } else {
            int jj = j;
            if (p.dist == SPX_DIST_BALANCED) {
                if (jj == 0) {
                    csr_merge_fixup_range<DT>(threadIdx.x, kBlock, a.tiles_mat, a.carry_row_all + (int64_t)b * a.tiles_mat,
                                              (const Acc*)a.carry_val_all + (int64_t)b * a.tiles_mat, Yb);
                }
                --jj;
            }
            if (jj >= 0) {
                const int e1 = std::min(p.nnz_x, (jj + 1) * kScatterChunk);
                for (int e = jj * kScatterChunk + threadIdx.x; e < e1; e += kBlock) {
                    const int c = idx[e];
                    bits[c >> 5] = 0u;
                    if constexpr (S::kVals) xd[c] = (typename S::X)0;
                }
            }
        }
    }
}

// ------------------------------------------------------------------ host side
// Blocks of rows of a column-major vector's Y, or 0 where its products go to Y
// with atomics. By blocks is faster down to an entry in eight segments (128
// vectors of density 1 % on 2^18 x 2^18, float32: 77 against 134 us with 2
// entries per row, 89 against 246 with 8, 129 against 623 with 32; density
// 0.05 %: 42 against 95 us); beyond that the table of segments is more than
// four times A.
int32_t batch_row_blocks(int32_t m, int32_t n, int64_t nnz, int dtype) {
    if (dtype == SPX_BOOL || m <= 0 || n <= 0) return 0;
    const int64_t nblk = ceil_div(m, kRowsBytes / (dtype == SPX_F64 ? 8 : 4));
    return n * nblk <= 8 * nnz && n * nblk < ((int64_t)1 << 31) ? (int32_t)nblk : 0;
}

spx_status batch_build_segs(const spx_csr& A, const int32_t* col_ptr, const int32_t* row_idx, int32_t nblk,
                            int32_t* segs, hipStream_t s) {
    const int64_t total = (int64_t)A.n * nblk;
    k_segs<<<(unsigned)std::min<int64_t>(ceil_div(total + 1, kBlock), 65536), kBlock, 0, s>>>(
        total, nblk, kRowsBytes / (A.dtype == SPX_F64 ? 8 : 4), A.nnz, col_ptr, row_idx, segs);
    SPX_HIP(hipGetLastError());
    return SPX_OK;
}

static void batch_layout(int32_t m, int32_t n, int dtype, int32_t B, int64_t cap_nnz_x, int64_t tiles_mat,
                         bool by_rows, BatchDev* d, char* base, size_t* bytes) {
    Sizer z;
    size_t off[20];
    int k = 0;
    auto take = [&](size_t n_bytes) {
        z.used = align_up(z.used, 256);
        off[k++] = z.used;
        z.used += align_up(n_bytes, 256);
    };
    const int vs = std::max(1, value_size(dtype));
    const int as = dtype == SPX_F64 ? 8 : 4;
    const int64_t nwords = ceil_div(n, 32) + 1;
    const int32_t vB = by_rows ? 0 : B;  // vectors that k_batch_phase may run
    take(sizeof(BatchPlan) * (size_t)B);                 // 0 plans
    take(4 * (size_t)3 * (B + 1));                       // 1 offs
    take(4 * 4);                                          // 2 totals
    take(4 * 8);                                          // 3 queue heads, err of the last run, err
    take(4);                                              // 4 vectors in groups
    take(by_rows ? 0 : 4 * (size_t)(cap_nnz_x + B));      // 5 excl
    take(4 * (size_t)vB * nwords);                        // 6 bits (self-cleaning)
    take((size_t)vs * vB * (size_t)n);                    // 7 xd (self-cleaning)
    take(4 * (size_t)vB * tiles_mat);                     // 8 carry rows
    take((size_t)as * vB * tiles_mat);                    // 9 carry values
    take(4 * (size_t)B);                                  // 10 group slot -> vector
    const int64_t gsize = kSlabRow / (vs == 8 ? 8 : 4);
    take((size_t)kSlabRow * ceil_div(B, gsize) * ((size_t)n + 1));  // 11 group slabs
    take(8 * 128);                                        // 12 queue heads of the groups' walk
    take(4 * (size_t)B);                                  // 13 the vectors' stray flags
    *bytes = z.used;
    if (!d || !base) return;
    d->plans = (BatchPlan*)(base + off[0]);
    d->offs = (int32_t*)(base + off[1]);
    d->totals = (int32_t*)(base + off[2]);
    d->queue = (int32_t*)(base + off[3]);
    d->err = d->queue + 4;
    d->excl_all = (int32_t*)(base + off[5]);
    d->bits_all = (uint32_t*)(base + off[6]);
    d->xd_all = base + off[7];
    d->carry_row_all = (int32_t*)(base + off[8]);
    d->carry_val_all = base + off[9];
    d->nwords = nwords;
    d->gcount = (int32_t*)(base + off[4]);
    d->heads = (int32_t*)(base + off[12]);
    d->stray = (int32_t*)(base + off[13]);
    d->gvec = (int32_t*)(base + off[10]);
    d->xt_all = base + off[11];
}

size_t batch_ws_size(int32_t m, int32_t n, int dtype, int32_t B, int64_t cap_nnz_x, int64_t tiles_mat,
                     bool by_rows, size_t* zero_from, size_t* zero_bytes) {
    size_t bytes = 0;
    batch_layout(m, n, dtype, B, cap_nnz_x, tiles_mat, by_rows, nullptr, nullptr, &bytes);
    // the whole workspace is zeroed at allocation; only the bitvector and
    // value slots rely on it (they are self-cleaning afterwards)
    if (zero_from) *zero_from = 0;
    if (zero_bytes) *zero_bytes = bytes;
    return bytes;
}

spx_status launch_batch(const BatchLaunch& L, void* ws, size_t ws_bytes, hipStream_t s, int32_t** err_dev) {
    BatchDev d{};
    d.m = L.csr.m;
    d.n = L.csr.n;
    d.nnz = L.csr.nnz;
    d.row_ptr = L.csr.row_ptr;
    d.col_idx = L.csr.col_idx;
    d.vals = L.csr.vals;
    d.col_ptr = L.col_ptr;
    d.row_idx = L.row_idx;
    d.vals_csc = L.vals_csc;
    d.part = L.part;
    d.tiles_mat = L.tiles_mat;
    d.B = L.B;
    d.cap_nnz_x = L.cap_nnz_x;
    d.vec_ptr = L.vec_ptr;
    d.idx = L.idx;
    d.val = L.val;
    d.Y = L.Y;
    d.sel = L.sel;
    d.row_lanes = L.row_lanes;
    d.units = (const int4*)L.units;
    d.nunits = L.nunits;
    d.split_rows = L.split_rows;
    d.nsplit = L.nsplit;
    d.segs = L.segs;
    d.nblk = L.nblk;
    size_t need = 0;
    // laid out for the capacity, not for this call's B: the parts that are kept
    // zero between runs stay where they are
    batch_layout(d.m, d.n, L.csr.dtype, L.cap_B, L.cap_nnz_x, L.tiles_mat, L.segs != nullptr, &d, (char*)ws, &need);
    if (need > ws_bytes) return fail(SPX_ERR_WORKSPACE, "run_batch: workspace too small");
    if (err_dev) *err_dev = d.queue + 3;
    if (L.B == 0) return SPX_OK;
    // a group's slab addressed by 32-bit buffer offsets when it fits
    const bool slab_buf = (int64_t)(d.n + (int64_t)1) * kSlabRow < ((int64_t)1 << 31);
    // the walk's grid is what stays resident at once, a multiple of the XCDs
    auto resident = [&](const void* fn) {
        int per_cu = *L.fused_per_cu;
        if (per_cu == 0) {
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, kBlock, 0) != hipSuccess || per_cu < 1)
                per_cu = 1;
            *L.fused_per_cu = per_cu;
        }
        return (unsigned)std::max(1, L.persistent_grid / 4) * (unsigned)per_cu;
    };
    // vectors per launch of k_batch_rows: a grid holds fewer than 2^32 threads
    const int32_t rows_step = (int32_t)std::max<int64_t>(8, ((1 << 21) / std::max(1, d.nblk)) & ~7);
    const bool fused = L.csr.dtype != SPX_BOOL && d.units && d.nunits > 0;
    switch (L.csr.dtype) {
#define SPX_DT(DT)                                                                                    \
    case DT:                                                                                          \
        k_batch_plan<DT><<<L.B, kBlock, 0, s>>>(d);                                                   \
        k_batch_scan<<<1, kBlock, 0, s>>>(d);                                                         \
        if (fused) {                                                                                  \
            k_batch_slabs<DT><<<L.persistent_grid, kBlock, 0, s>>>(d);                                \
            k_batch_stray<DT><<<L.B, kBlock, 0, s>>>(d);                                              \
            if (slab_buf)                                                                             \
                k_batch_fused<DT, true><<<resident((const void*)k_batch_fused<DT, true>), kBlock, 0, s>>>(d);\
            else                                                                                      \
                k_batch_fused<DT, false><<<resident((const void*)k_batch_fused<DT, false>), kBlock, 0, s>>>(d);\
        }                                                                                             \
        if (d.segs) {                                                                                 \
            SPX_HIP(hipFuncSetAttribute((const void*)k_batch_rows<DT>,                                \
                                        hipFuncAttributeMaxDynamicSharedMemorySize, kRowsBytes));     \
            for (int32_t b0 = 0; b0 < L.B; b0 += std::min(rows_step, L.B - b0))                       \
                k_batch_rows<DT><<<(unsigned)(ceil_div(std::min(rows_step, L.B - b0), 8) * 8 * d.nblk), \
                                   kRowsThreads, kRowsBytes, s>>>(d, b0);                             \
        } else {                                                                                      \
            k_batch_phase<DT, 0><<<L.persistent_grid, kBlock, 0, s>>>(d);                             \
            k_batch_phase<DT, 1><<<L.persistent_grid, kBlock, 0, s>>>(d);                             \
            k_batch_phase<DT, 2><<<L.persistent_grid, kBlock, 0, s>>>(d);                             \
        }                                                                                             \
        break;
        SPX_DT(SPX_F32)
        SPX_DT(SPX_F64)
        SPX_DT(SPX_I32)
        SPX_DT(SPX_BOOL)
#undef SPX_DT
        default:
            return fail(SPX_ERR_DTYPE, "run_batch: dtype");
    }
    SPX_HIP(hipGetLastError());
    return SPX_OK;
}

void upload_tree(const Tree& t, DevTree* out) {
    const int n = std::min<int>((int)t.cls.size(), kDevTreeNodes);
    out->n = n;
    for (int i = 0; i < n; ++i) {
        out->feat[i] = t.feat[i];
        out->thr[i] = t.thr[i];
        out->left[i] = t.left[i];
        out->right[i] = t.right[i];
        out->cls[i] = t.cls[i];
    }
}

}  // namespace spx
