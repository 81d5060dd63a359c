// gemv.hip -- y = h W^T for gfx950 (wave64): the vector-unit forms (one to four rows of h, and every fp32
// shape), the matrix-core forms (five rows and more), and the forms that carry an RMSNorm in front and
// elementwise kernels behind in the same dispatch (kernels.h, "merged dispatches").
//
// Built with -ffp-contract=off: fused multiply-adds appear only where written.
#include "device.h"

namespace pgk {
namespace {

// ---- GEMV ------------------------------------------------------------------------------------------
// Ask for every kernel argument in one batch of scalar loads.  Left alone, the compiler fetches `n`
// for the early-exit test first and the pointers only behind it: two dependent trips to the kernel
// argument buffer (cold in the scalar cache at every launch) before the first weight load goes out,
// about 0.4 us on a 3 us kernel.
__device__ __forceinline__ void args_up_front(const GemvArgs& p) {
    asm volatile("" ::"s"(p.out), "s"(p.W), "s"(p.h), "s"(p.rows), "s"(p.n), "s"(p.cols), "s"(p.row_groups));
}

// Memory-bound: every weight is read exactly once.  One wave computes R output columns (R weight
// rows): per chunk of 4 * 64 vectors of the row it issues all R * 4 weight loads (non-temporal:
// streamed, no reuse) and the 4 loads of its slice of h before the first multiply, accumulates in
// fp32 in a fixed order, and reduces across the wave.  No MFMA: at batch 1 there is no reuse to
// feed a matrix core.  Row-shape classes RS (from cols alone): 0 = cols is a whole number of
// chunks (no bounds handling at all), 1 = a whole number of vectors, 2 = ragged.
constexpr int kGemvChunk = 4;   // vectors per lane per chunk

template <typename T, int RS, bool AL, bool NT>
__device__ __forceinline__ void gemv_issue(const T* row, int nfull, int v, unsigned* w) {
    constexpr int NV = Vec<T, 16>::NV;
    if constexpr (RS == 0) load_vec<T, 16, AL, NT>(row + (size_t)v * NV, w);
    else row_vec_issue<T, AL, NT>(row, nfull, v, w);
}
template <typename T, int RS>
__device__ __forceinline__ void gemv_fix(const T* row, int cols, int nfull, int v, unsigned* w) {
    if constexpr (RS != 0) row_vec_fix<T, RS == 2>(row, cols, nfull, v, w);
}

template <typename T, int R, int RS, bool AL>
__device__ __forceinline__ void gemv_body(const T* W, const T* h, T* y, int n, int cols, int j0, int lane) {
    constexpr int NV = Vec<T, 16>::NV;
    const int nfull = cols / NV;
    const int nvec = (cols + NV - 1) / NV;
    float acc[R];
    const T* wrow[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
        acc[r] = 0.f;
        wrow[r] = W + (size_t)((j0 + r < n) ? j0 + r : n - 1) * cols;   // a ragged last group re-reads the last row
    }
    for (int v0 = 0; v0 < nvec; v0 += 64 * kGemvChunk) {
        unsigned ww[R][kGemvChunk][4], wh[kGemvChunk][4];
        if (RS != 2 || nfull > 0) {
#pragma unroll
            for (int r = 0; r < R; r++)
#pragma unroll
                for (int u = 0; u < kGemvChunk; u++) gemv_issue<T, RS, AL, true>(wrow[r], nfull, v0 + u * 64 + lane, ww[r][u]);
#pragma unroll
            for (int u = 0; u < kGemvChunk; u++) gemv_issue<T, RS, AL, false>(h, nfull, v0 + u * 64 + lane, wh[u]);
        }
#pragma unroll
        for (int u = 0; u < kGemvChunk; u++) gemv_fix<T, RS>(h, cols, nfull, v0 + u * 64 + lane, wh[u]);
#pragma unroll
        for (int r = 0; r < R; r++)
#pragma unroll
            for (int u = 0; u < kGemvChunk; u++) {
                gemv_fix<T, RS>(wrow[r], cols, nfull, v0 + u * 64 + lane, ww[r][u]);
                acc[r] = dot_acc<T>(ww[r][u], wh[u], acc[r]);
            }
    }
#pragma unroll
    for (int r = 0; r < R; r++) {
        const float s = wave_sum(acc[r]);
        if (lane == 0 && j0 + r < n) store_elem(y + j0 + r, s);
    }
}

template <typename T, int IND, int R, int RS>
__global__ __launch_bounds__(kBlock) void k_gemv(GemvArgs p) {
    args_up_front(p);
    const T* W = static_cast<const T*>(resolve<(IND & 1) != 0>(p.W));
    const T* h = static_cast<const T*>(resolve<(IND & 2) != 0>(p.h));
    T* y = static_cast<T*>(p.out);
    const int lane = threadIdx.x & 63;
    const int j0 = (blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6)) * R;
    if (j0 >= p.n) return;   // whole wave leaves together
    // row starts of W stay aligned only if cols is a multiple of the vector
    const bool al = RS != 2 && aligned_to(W, 16) && aligned_to(h, 16);
    if (__builtin_expect(al, 1)) gemv_body<T, R, RS, true>(W, h, y, p.n, p.cols, j0, lane);
    else gemv_body<T, R, RS, false>(W, h, y, p.n, p.cols, j0, lane);
}

// The same for rows of exactly one chunk (2048 bf16 or 1024 fp32 columns -- the decode chain's shape)
// and one or two rows of h: instead of every wave fetching all of h, lane t of the workgroup fetches
// vector t of each row once and the four waves share it through LDS.  That takes 12 KB (one row of h)
// or 24 KB (two) of cache traffic per workgroup off the load path the weights come in by (3.16 ->
// 3.07 us per launch at 2048 x 2048, one row); h is asked for before the weights, so the exchange is
// over long before the first weight arrives.  Same lanes, same products, same order as gemv_body and
// gemvb_body: the results are bit-identical.
static_assert(kBlock == 64 * kGemvChunk, "one vector of h per lane of the workgroup");
template <typename T, int R, int RB, bool AL>
__device__ __forceinline__ void gemv_body_shared(const T* W, const T* h, T* y, int n, int j0, int lane, int tid, v4u* hs /* [RB][kBlock] */) {
    constexpr int NV = Vec<T, 16>::NV;
    constexpr int kCols = 64 * kGemvChunk * NV;
    unsigned hv[RB][4], ww[R][kGemvChunk][4], wh[RB][kGemvChunk][4];
#pragma unroll
    for (int rr = 0; rr < RB; rr++) load_vec<T, 16, AL, false>(h + (size_t)rr * kCols + (size_t)tid * NV, hv[rr]);
    __builtin_amdgcn_sched_barrier(0);   // h first: loads come back in the order they were issued
#pragma unroll
    for (int r = 0; r < R; r++) {
        const T* wrow = W + (size_t)((j0 + r < n) ? j0 + r : n - 1) * kCols;   // a ragged last group re-reads the last row
#pragma unroll
        for (int u = 0; u < kGemvChunk; u++) load_vec<T, 16, AL, true>(wrow + (size_t)(u * 64 + lane) * NV, ww[r][u]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int rr = 0; rr < RB; rr++) hs[rr * kBlock + tid] = v4u{hv[rr][0], hv[rr][1], hv[rr][2], hv[rr][3]};
    __syncthreads();      // every wave of the workgroup gets here: none leaves early
#pragma unroll
    for (int rr = 0; rr < RB; rr++)
#pragma unroll
        for (int u = 0; u < kGemvChunk; u++) {
            const v4u t = hs[rr * kBlock + u * 64 + lane];
            wh[rr][u][0] = t.x; wh[rr][u][1] = t.y; wh[rr][u][2] = t.z; wh[rr][u][3] = t.w;
        }
    float acc[R][RB];
#pragma unroll
    for (int r = 0; r < R; r++)
#pragma unroll
        for (int rr = 0; rr < RB; rr++) {
            acc[r][rr] = 0.f;
#pragma unroll
            for (int u = 0; u < kGemvChunk; u++) acc[r][rr] = dot_acc<T>(ww[r][u], wh[rr][u], acc[r][rr]);
        }
#pragma unroll
    for (int rr = 0; rr < RB; rr++)
#pragma unroll
        for (int r = 0; r < R; r++) {
            const float sum = wave_sum(acc[r][rr]);
            if (lane == 0 && j0 + r < n) store_elem(y + (size_t)rr * n + j0 + r, sum);
        }
}

// RB = rows of h: 1 to 4
template <typename T, int IND, int R, int RB>
__global__ __launch_bounds__(kBlock) void k_gemv_shared(GemvArgs p) {
    args_up_front(p);
    const T* W = static_cast<const T*>(resolve<(IND & 1) != 0>(p.W));
    const T* h = static_cast<const T*>(resolve<(IND & 2) != 0>(p.h));
    T* y = static_cast<T*>(p.out);
    __shared__ v4u hs[RB * kBlock];
    const int tid = threadIdx.x, lane = tid & 63;
    const int j0 = (blockIdx.x * (kBlock / 64) + (tid >> 6)) * R;
    const bool al = aligned_to(W, 16) && aligned_to(h, 16);
    if (__builtin_expect(al, 1)) gemv_body_shared<T, R, RB, true>(W, h, y, p.n, j0, lane, tid, hs);
    else gemv_body_shared<T, R, RB, false>(W, h, y, p.n, j0, lane, tid, hs);
}

// Batched (rows > 1) on the vector units: one wave per R output columns, as in the one-row kernel;
// the R weight chunks stay in registers while the rows of h (from cache) stream past them,
// RB rows at a time (RB = 2 when there are only two rows: a clamped row would be loaded and summed
// for nothing).
template <typename T, int R, int RB, int RS, bool AL>
__device__ __forceinline__ void gemvb_body(const T* W, const T* h, T* y, int rows, int n, int cols, int j0, int lane) {
    constexpr int NV = Vec<T, 16>::NV;
    const int nfull = cols / NV;
    const int nvec = (cols + NV - 1) / NV;
    const T* wrow[R];
#pragma unroll
    for (int r = 0; r < R; r++) wrow[r] = W + (size_t)((j0 + r < n) ? j0 + r : n - 1) * cols;   // a ragged last group re-reads the last row
    for (int r0 = 0; r0 < rows; r0 += RB) {
        float acc[R][RB];
        const T* hrow[RB];
#pragma unroll
        for (int rr = 0; rr < RB; rr++) {
#pragma unroll
            for (int r = 0; r < R; r++) acc[r][rr] = 0.f;
            hrow[rr] = h + (size_t)((r0 + rr < rows) ? r0 + rr : rows - 1) * cols;
        }
        for (int v0 = 0; v0 < nvec; v0 += 64 * kGemvChunk) {
            unsigned ww[R][kGemvChunk][4], wh[RB][kGemvChunk][4];
            if (RS != 2 || nfull > 0) {
#pragma unroll
                for (int r = 0; r < R; r++)
#pragma unroll
                    for (int u = 0; u < kGemvChunk; u++) gemv_issue<T, RS, AL, true>(wrow[r], nfull, v0 + u * 64 + lane, ww[r][u]);
#pragma unroll
                for (int rr = 0; rr < RB; rr++)
#pragma unroll
                    for (int u = 0; u < kGemvChunk; u++) gemv_issue<T, RS, AL, false>(hrow[rr], nfull, v0 + u * 64 + lane, wh[rr][u]);
            }
#pragma unroll
            for (int r = 0; r < R; r++)
#pragma unroll
                for (int u = 0; u < kGemvChunk; u++) gemv_fix<T, RS>(wrow[r], cols, nfull, v0 + u * 64 + lane, ww[r][u]);
#pragma unroll
            for (int rr = 0; rr < RB; rr++)
#pragma unroll
                for (int u = 0; u < kGemvChunk; u++) {
                    gemv_fix<T, RS>(hrow[rr], cols, nfull, v0 + u * 64 + lane, wh[rr][u]);
#pragma unroll
                    for (int r = 0; r < R; r++) acc[r][rr] = dot_acc<T>(ww[r][u], wh[rr][u], acc[r][rr]);
                }
        }
#pragma unroll
        for (int rr = 0; rr < RB; rr++)
#pragma unroll
            for (int r = 0; r < R; r++) {
                const float s = wave_sum(acc[r][rr]);
                if (lane == 0 && r0 + rr < rows && j0 + r < n) store_elem(y + (size_t)(r0 + rr) * n + j0 + r, s);
            }
    }
}

template <typename T, int IND, int R, int RB, int RS>
__global__ __launch_bounds__(kBlock) void k_gemv_batched(GemvArgs p) {
    args_up_front(p);
    const T* W = static_cast<const T*>(resolve<(IND & 1) != 0>(p.W));
    const T* h = static_cast<const T*>(resolve<(IND & 2) != 0>(p.h));
    T* y = static_cast<T*>(p.out);
    const int lane = threadIdx.x & 63;
    const int j0 = (blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6)) * R;
    if (j0 >= p.n) return;
    const bool al = RS != 2 && aligned_to(W, 16) && aligned_to(h, 16);
    if (__builtin_expect(al, 1)) gemvb_body<T, R, RB, RS, true>(W, h, y, p.rows, p.n, p.cols, j0, lane);
    else gemvb_body<T, R, RB, RS, false>(W, h, y, p.rows, p.n, p.cols, j0, lane);
}

// Batched bf16 with whole 16-byte vectors per row: y[rows, n] = h[rows, cols] * W[n, cols]^T is a
// dense contraction once rows > 1, so it goes to the matrix cores (v_mfma_f32_16x16x32_bf16, fp32
// accumulate).  Still weight-streaming bound up to rows ~ 128: every weight is read once from HBM.
//   - a workgroup owns 16 output columns and one group of 16-row tiles of h; the grid is
//     (column blocks) x (row groups), column block fastest, so that the row groups of one column
//     block land on the same XCD (workgroups go to the 8 XCDs round-robin) and all but the first find
//     the weights in its L2;
//   - its 4 waves split K: of every 8 consecutive 32-wide K-steps wave w takes steps 2w and 2w+1 (128
//     contiguous bytes of each row), 16 steps per 2048 columns;
//   - a fragment (A: lane l holds row l & 15, B: column l & 15; the 8 consecutive k's of chunk l >> 4
//     of a step) read straight from global memory would touch 16 rows x 64 bytes per instruction, all
//     4 KB apart: half cache lines, one cache channel (measured: 0.3 - 1.1 us slower per launch).
//     Instead each wave loads its own K-slices of 16 rows -- a tile of h, or the weights of the 16
//     columns -- row by row (one row = 8 x 128 contiguous bytes per instruction) and transposes them
//     through its private slice of LDS into fragment order.  The weight fragments stay in registers
//     when cols <= 2048 (SINGLE) and are re-read per tile (from cache) otherwise; the next tile's rows
//     of h are in flight while the matrix cores work on this one.  LDS slot (lane of the load) holds 16 rows x 16 bytes and is padded to 272
//     bytes so that 16 consecutive lanes hit all banks.  74 KB of LDS per workgroup: two fit a CU, and
//     one's staging overlaps the other's multiplies;
//   - rows beyond the batch re-read the last row and are never stored;
//   - per tile the 4 waves' partial sums meet in LDS and are added in a fixed order; lane l of a tile
//     holds column (l & 15), rows 4 * (l >> 4) .. + 3.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
constexpr int kMmSteps = 16;        // K-steps per wave per super-chunk (4 waves x 16 steps x 32 = 2048 columns)
constexpr int kMmSlotBytes = 272;   // 16 rows x 16 B + 16 B of padding
constexpr int kMmWaveLds = 64 * kMmSlotBytes;   // one wave's staging area: one tile, 64 slots
constexpr int kMmMaxRowGroups = 4;
constexpr int kMmWideRows = 81;     // rows from which the 32-column form is used (measured: the 16-column form is faster up to 5 tiles of rows, slower from 6)

// k offset of the 16-byte chunk that lane `l` of wave `wave` loads from a row (super-chunk at step s0);
// the same chunk is fragment step l >> 2, k-chunk l & 3 of that wave.
__device__ __forceinline__ int mm_k0(int s0, int wave, int l) {
    return (s0 + (l >> 3) * 8 + wave * 2 + ((l >> 2) & 1)) * 32 + (l & 3) * 8;
}

// 16 rows of a row-major matrix (a tile of h, or the weights of 16 output columns), this wave's
// K-slices: one row per instruction; rows beyond the matrix repeat its last row
template <bool FULL, bool AL, int NR = 16>
__device__ __forceinline__ void mm_load_rows(const bf16_t* h, int rows, int cols, int r0, int s0, int wave, int lane, unsigned (*g)[4]) {
    const int k0 = mm_k0(s0, wave, lane);
    const int koff = (FULL || k0 < cols) ? k0 : 0;      // an out-of-range chunk is read from column 0 and zeroed on both sides later
#pragma unroll
    for (int r = 0; r < NR; r++) {
        const int R = r0 + r < rows ? r0 + r : rows - 1;
        load_vec_global<bf16_t, AL, false>(h + (size_t)R * cols + koff, g[r]);     // global outright: see load_vec_global
    }
}

// LDS operations of one wave execute in order: these writes cannot overtake the previous tile's reads
template <int NR = 16>
__device__ __forceinline__ void mm_stage(char* lds /* this wave's */, int lane, const unsigned (*g)[4]) {
#pragma unroll
    for (int r = 0; r < NR; r++) {
        v4u t;
        t.x = g[r][0]; t.y = g[r][1]; t.z = g[r][2]; t.w = g[r][3];
        *reinterpret_cast<v4u*>(lds + lane * kMmSlotBytes + r * 16) = t;
    }
}

// fragment (step i, k-chunk lane >> 4, row or column lane & 15) of the tile staged in `lds`
__device__ __forceinline__ void mm_read_frags(const char* lds, int lane, v4u* f) {
#pragma unroll
    for (int i = 0; i < kMmSteps; i++)
        f[i] = *reinterpret_cast<const v4u*>(lds + (i * 4 + (lane >> 4)) * kMmSlotBytes + (lane & 15) * 16);
}
// chunks beyond cols are zeroed on both sides (the loads fetched column 0 in their place): zeroing the
// weight side alone would turn an Inf or NaN of h[:, 0:8] into NaN in every output (0 * Inf)
template <bool FULL>
__device__ __forceinline__ void mm_zero_tail(v4u* b, int cols, int s0, int wave, int kq) {
    if constexpr (!FULL) {
#pragma unroll
        for (int i = 0; i < kMmSteps; i++)      // cols is a multiple of 8: a chunk is all in or all out
            if ((s0 + (i >> 1) * 8 + wave * 2 + (i & 1)) * 32 + kq * 8 >= cols) b[i] = v4u{0u, 0u, 0u, 0u};
    }
}
__device__ __forceinline__ void mm_mfma(const v4u* a, const v4u* b, f32x4& acc) {
#pragma unroll
    for (int i = 0; i < kMmSteps; i++)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[i]), __builtin_bit_cast(bf16x8, b[i]), acc, 0, 0, 0);
}

// What becomes of a finished tile.  All four waves share the output stage: a lane is given NE consecutive
// rows of one column -- begin(r, j, ok) before the partial sums are exchanged (or earlier), put(k, v) for
// each of its sums, end().
// MmStore: the stand-alone kernels -- each sum is rounded and stored.
template <int NE>
struct MmStore {
    static constexpr bool kEarly = false;
    bf16_t* y;
    int rows, n;
    size_t at = 0;
    int r = 0;
    bool col_ok = false;
    __device__ __forceinline__ void prepare() {}
    __device__ __forceinline__ void begin(int r_, int j, bool ok) { r = r_; col_ok = ok; at = (size_t)r_ * n + j; }
    __device__ __forceinline__ void put(int k, float v) { if (col_ok && r + k < rows) store_elem(y + at + (size_t)k * n, v); }
    __device__ __forceinline__ void end() {}
};
// MmEpilogue: the kernels that follow the GEMV in the chain, element for element, ride along (kernels.h,
// GemvEpiArgs): prepare() reads their table out of the kernel arguments and resolves pointer-table slots --
// the bodies call it once their weight loads are on their way, as k_gemv_rows does, so that nothing but
// the first 64 bytes of the arguments stands between the start of the kernel and those loads; begin() asks
// for the operands, so that they arrive while the tile is staged and multiplied and the partial sums are
// exchanged; end() plays the kernels on the lane's outputs, rounding to bf16 after each as the stand-alone
// kernels do, with the GELU as the only branch.
// EARLY (the narrow forms, whose few loads leave the operands' latency exposed): begin() comes right behind the
// weight loads and always issues the same number of loads -- an operand that comes from a register slot is
// fetched from the GEMV's own output buffer instead and ignored -- so that every wait on the rows and weights
// knows exactly how many younger loads are outstanding.  Otherwise the loads are conditional, which the compiler
// cannot count (a wait for an older load placed behind them would wait for more than it needs), and begin() comes
// once the rows and weights of the tile have been taken out of their registers, in front of the multiplies.
template <int NE, bool EARLY>
struct MmEpilogue {
    static constexpr bool kEarly = EARLY;
    static constexpr int P = kEpiMaxPhases;
    bf16_t* y;
    int rows, n;
    unsigned head;
    int n_epi;
    const void PG_CONSTANT* ka;   // the kernel-argument segment (a GemvEpiArgs)
    float eps = 0.f;              // the prologue's, read with the table
    const bf16_t* q0[P];        // operand addresses, pointer-table slots resolved; null: comes from a register slot
    const bf16_t* q1[P];
    bf16_t* outs[P];
    unsigned ms[P], metas[P], inds[P];
    bool plain = true;          // EARLY: no operand has a broadcast period
    bool decoder = false;       // the kernels are GELU of the GEMV's result, then one or two adds with an operand from memory
    // per call
    unsigned idx[NE];
    bool ok[NE];
    unsigned ld0[P][NE], ld1[P][NE];
    float v[NE];
    __device__ __forceinline__ void prepare() {
        static_assert(P == 3, "the argument batch names every phase");
        using SlotPtr = const void* const PG_CONSTANT*;
        const void* a0[P];
        const void* a1[P];
        {   // through the segment's address made opaque: otherwise the compiler moves these loads (invariant
            // memory) to the top of the kernel, in front of the weight loads
            const GemvEpiArgs PG_CONSTANT* kp = (const GemvEpiArgs PG_CONSTANT*)ka;
            asm volatile("" : "+s"(kp));
            eps = kp->eps;
#pragma unroll
            for (int i = 0; i < P; i++) {
                a0[i] = kp->ph[i].in0; a1[i] = kp->ph[i].in1; outs[i] = static_cast<bf16_t*>(kp->ph[i].out);
                ms[i] = kp->ph[i].m; metas[i] = kp->ph[i].meta; inds[i] = kp->ph[i].ind;
            }
            asm volatile("" : "+s"(eps),
                              "+s"(a0[0]), "+s"(a1[0]), "+s"(outs[0]), "+s"(ms[0]), "+s"(metas[0]), "+s"(inds[0]),
                              "+s"(a0[1]), "+s"(a1[1]), "+s"(outs[1]), "+s"(ms[1]), "+s"(metas[1]), "+s"(inds[1]),
                              "+s"(a0[2]), "+s"(a1[2]), "+s"(outs[2]), "+s"(ms[2]), "+s"(metas[2]), "+s"(inds[2]));
        }
        bool f0[P], f1[P], s0[P], s1[P];
        unsigned any = 0;
#pragma unroll
        for (int i = 0; i < P; i++) {
            const unsigned mt = metas[i];
            f0[i] = ((mt >> 8) & 0xffu) == kMergeFromMemory;
            f1[i] = (mt & 0xffu) != kGelu && ((mt >> 16) & 0xffu) == kMergeFromMemory;
            s0[i] = f0[i] && (inds[i] & 1u);
            s1[i] = f1[i] && (inds[i] & 2u);
            any |= (f0[i] ? inds[i] & 1u : 0u) | (f1[i] ? inds[i] & 2u : 0u);
        }
        any = __builtin_amdgcn_readfirstlane(any);
        asm volatile("" : "+s"(any));       // keeps what follows behind the weight loads
        {   // the decoder block's tail, recognised here so that end() runs it straight through (see k_gemv_rows)
            auto add_of = [](unsigned mt, unsigned q) {
                const unsigned a = (mt >> 8) & 0xffu, b = (mt >> 16) & 0xffu;
                return (mt & 0xffu) == (unsigned)kAdd && ((a == q && b == kMergeFromMemory) || (a == kMergeFromMemory && b == q));
            };
            const unsigned hq = (head >> 8) & 0xffu, d0 = metas[0] >> 24, d1 = metas[1] >> 24;
            decoder = (n_epi == 2 || n_epi == 3) && (metas[0] & 0xffu) == (unsigned)kGelu && ((metas[0] >> 8) & 0xffu) == hq &&
                      add_of(metas[1], d0) && (n_epi == 2 || add_of(metas[2], d1));
        }
        if (any) {                           // some operand is a pointer-table slot: all in one batch, without branches
            auto slot_addr = [&](const void* q, bool is_slot) -> SlotPtr { return is_slot ? (SlotPtr)(uintptr_t)q : (SlotPtr)ka; };
            SlotPtr at0[P], at1[P];
            const void* t0[P];
            const void* t1[P];
#pragma unroll
            for (int i = 0; i < P; i++) { at0[i] = slot_addr(a0[i], s0[i]); at1[i] = slot_addr(a1[i], s1[i]); }
#pragma unroll
            for (int i = 0; i < P; i++) { t0[i] = *at0[i]; t1[i] = *at1[i]; }
            asm volatile("" : "+s"(t0[0]), "+s"(t1[0]), "+s"(t0[1]), "+s"(t1[1]), "+s"(t0[2]), "+s"(t1[2]));
#pragma unroll
            for (int i = 0; i < P; i++) {
                if (s0[i]) a0[i] = t0[i];
                if (s1[i]) a1[i] = t1[i];
            }
        }
        if constexpr (EARLY) {
            const unsigned total = (unsigned)rows * (unsigned)n;
            plain = true;
#pragma unroll
            for (int i = 0; i < P; i++) {
                q0[i] = f0[i] ? static_cast<const bf16_t*>(a0[i]) : y;
                q1[i] = f1[i] ? static_cast<const bf16_t*>(a1[i]) : y;
                ms[i] = f1[i] ? ms[i] : total;
                plain = plain && ms[i] == total;
            }
        } else {
#pragma unroll
            for (int i = 0; i < P; i++) {
                q0[i] = f0[i] ? static_cast<const bf16_t*>(a0[i]) : nullptr;
                q1[i] = f1[i] ? static_cast<const bf16_t*>(a1[i]) : nullptr;
#pragma unroll
                for (int k = 0; k < NE; k++) ld0[i][k] = ld1[i][k] = 0u;
            }
        }
    }
    __device__ __forceinline__ void begin(int r, int j, bool col_ok) {
        const unsigned total = (unsigned)rows * (unsigned)n;
#pragma unroll
        for (int e = 0; e < NE; e++) {
            ok[e] = col_ok && r + e < rows;
            idx[e] = ok[e] ? (unsigned)(r + e) * (unsigned)n + (unsigned)j : 0u;
        }
        if constexpr (EARLY) {
            if (__builtin_expect(plain, 1)) {      // the usual case, one branch for all
#pragma unroll
                for (int i = 0; i < P; i++)
#pragma unroll
                    for (int e = 0; e < NE; e++) {
                        ld0[i][e] = load_raw_global_at(q0[i], idx[e]);
                        ld1[i][e] = load_raw_global_at(q1[i], idx[e]);
                    }
            } else {
#pragma unroll
                for (int i = 0; i < P; i++)
#pragma unroll
                    for (int e = 0; e < NE; e++) {
                        ld0[i][e] = load_raw_global_at(q0[i], idx[e]);
                        ld1[i][e] = load_raw_global_at(q1[i], idx[e] % ms[i]);
                    }
            }
        } else {
#pragma unroll
            for (int i = 0; i < P; i++) {
                if (i < n_epi && q0[i]) {
#pragma unroll
                    for (int e = 0; e < NE; e++) ld0[i][e] = load_raw_global_at(q0[i], idx[e]);
                }
                if (i < n_epi && q1[i]) {
                    const unsigned m = ms[i];
#pragma unroll
                    for (int e = 0; e < NE; e++) ld1[i][e] = load_raw_global_at(q1[i], m == total ? idx[e] : idx[e] % m);
                }
            }
        }
    }
    __device__ __forceinline__ void put(int e, float sum) { v[e] = sum; }
    __device__ __forceinline__ void end() {
        unsigned bits[NE];
        float slot[kMergeSlots][NE];
        __builtin_amdgcn_s_waitcnt(0x0F70);      // vmcnt(0): every operand, before the first store (see k_gemv_rows)
#pragma unroll
        for (int e = 0; e < NE; e++) {
            bits[e] = f32_to_bf16(v[e]);
            if (ok[e] && (head & kEpiHeadStore)) *(unsigned short PG_GLOBAL*)(uintptr_t)(y + idx[e]) = (unsigned short)bits[e];
        }
        if (__builtin_expect(decoder, 1)) {
            // the same kernels with the same arithmetic and roundings, operands known: GELU of the GEMV's rounded result,
            // then each add takes the value before it and its operand from memory, in the order its descriptor names
            const bool mf1 = ((metas[1] >> 8) & 0xffu) == kMergeFromMemory, mf2 = ((metas[2] >> 8) & 0xffu) == kMergeFromMemory;
#pragma unroll
            for (int e = 0; e < NE; e++) {
                float val = ew_apply<kGelu, false>(from_raw<bf16_t>(bits[e]), 0.f);
                unsigned b = f32_to_bf16(val);
                if (ok[e] && (inds[0] & kEpiStore)) *(unsigned short PG_GLOBAL*)(uintptr_t)(outs[0] + idx[e]) = (unsigned short)b;
                val = from_raw<bf16_t>(b);
                {
                    const float fa = mf1 ? from_raw<bf16_t>(ld0[1][e]) : val, fb = mf1 ? val : from_raw<bf16_t>(ld1[1][e]);
                    b = f32_to_bf16(ew_apply<kAdd, false>(fa, fb));
                    if (ok[e] && (inds[1] & kEpiStore)) *(unsigned short PG_GLOBAL*)(uintptr_t)(outs[1] + idx[e]) = (unsigned short)b;
                    val = from_raw<bf16_t>(b);
                }
                if (n_epi == 3) {
                    const float fa = mf2 ? from_raw<bf16_t>(ld0[2][e]) : val, fb = mf2 ? val : from_raw<bf16_t>(ld1[2][e]);
                    b = f32_to_bf16(ew_apply<kAdd, false>(fa, fb));
                    if (ok[e] && (inds[2] & kEpiStore)) *(unsigned short PG_GLOBAL*)(uintptr_t)(outs[2] + idx[e]) = (unsigned short)b;
                }
            }
            return;
        }
        {
            const unsigned dst = (head >> 8) & 0xffu;
#pragma unroll
            for (int q = 0; q < kMergeSlots; q++)
#pragma unroll
                for (int e = 0; e < NE; e++) slot[q][e] = dst == (unsigned)q ? from_raw<bf16_t>(bits[e]) : 0.f;
        }
#pragma unroll
        for (int i = 0; i < P; i++) {
            if (i >= n_epi) break;
            const unsigned mt = metas[i], ind = inds[i];
            const unsigned op = mt & 0xffu, src0 = (mt >> 8) & 0xffu, src1 = (mt >> 16) & 0xffu, dst = mt >> 24;
            float fa[NE], fb[NE], fo[NE];
#pragma unroll
            for (int e = 0; e < NE; e++) {
                fa[e] = from_raw<bf16_t>(ld0[i][e]);
                fb[e] = from_raw<bf16_t>(ld1[i][e]);
#pragma unroll
                for (int q = 0; q < kMergeSlots; q++) {
                    if (src0 == (unsigned)q) fa[e] = slot[q][e];
                    if (src1 == (unsigned)q) fb[e] = slot[q][e];
                }
            }
            if (op == kGelu) {
#pragma unroll
                for (int e = 0; e < NE; e++) fo[e] = ew_apply<kGelu, false>(fa[e], 0.f);
            } else {
#pragma unroll
                for (int e = 0; e < NE; e++) {
                    const float sum = ew_apply<kAdd, false>(fa[e], fb[e]), prod = ew_apply<kMul, false>(fa[e], fb[e]);
                    fo[e] = op == kAdd ? sum : prod;
                }
            }
#pragma unroll
            for (int e = 0; e < NE; e++) {
                bits[e] = f32_to_bf16(fo[e]);
                if (ok[e] && (ind & kEpiStore)) *(unsigned short PG_GLOBAL*)(uintptr_t)(outs[i] + idx[e]) = (unsigned short)bits[e];
#pragma unroll
                for (int q = 0; q < kMergeSlots; q++)
                    if (dst == (unsigned)q) slot[q][e] = from_raw<bf16_t>(bits[e]);
            }
        }
    }
};

// where the output stage of the 16-column forms puts a lane: wave w takes row w of the four that an
// accumulator lane holds
template <int NC = 16, class Emit>
__device__ __forceinline__ void mm_emit_begin(Emit& emit, int n, int r0, int j0, int wave, int lane) {
    emit.begin(r0 + (lane >> 4) * 4 + wave, j0 + (lane & 15), j0 + (lane & 15) < n && (NC == 16 || (lane & 15) < NC));
}
// sum the 4 waves' partial tiles in a fixed order and hand rows r0 .. r0 + 15 of the 16 columns at j0 to `emit`
// (mm_emit_begin has been called for this tile)
template <class Emit>
__device__ __forceinline__ void mm_reduce_store(float* red, f32x4 acc, Emit& emit, int wave, int lane) {
    // A matrix-core result may not be read by an LDS write until the instruction has drained (up to
    // 19 wait states for the longest forms).  The compiler inserts those itself inside a block, but
    // it was seen to omit them when the last multiply of a K loop and this write sit in different
    // blocks (loop exit): the write then stored a stale accumulator.  32 idle cycles, tied to `acc`
    // so that they stay between the two, make it independent of that.
    asm volatile("s_nop 15\n\ts_nop 15" : "+v"(acc));
    float* dst = red + ((size_t)wave * 64 + lane) * 4;
    dst[0] = acc.x; dst[1] = acc.y; dst[2] = acc.z; dst[3] = acc.w;
    __syncthreads();
    {
        const int e = wave;
        const float p0 = red[((size_t)0 * 64 + lane) * 4 + e], p1 = red[((size_t)1 * 64 + lane) * 4 + e];
        const float p2 = red[((size_t)2 * 64 + lane) * 4 + e], p3 = red[((size_t)3 * 64 + lane) * 4 + e];
        emit.put(0, ((p0 + p1) + p2) + p3);
    }
    __syncthreads();      // `red` is free again
    emit.end();
}

// mm_rmsnorm_rows is defined with the narrow form below
template <int NRH>
__device__ __forceinline__ void mm_rmsnorm_rows(unsigned (*g)[4], const unsigned* wg, float eps, bf16_t* hstore, int rows, int wave, int lane, float* scratch);

// PRO (SINGLE, FULL, one tile of rows per workgroup -- rows < kMmWideRows): h points at the rows to normalise,
// the workgroups of column block 0 store the normalised rows to hstore (see mm_rmsnorm_rows).
template <bool FULL, bool SINGLE, bool AL, bool PRO = false, class Emit>
__device__ __forceinline__ void gemm_mfma_body(const bf16_t* W, const bf16_t* h, Emit& emit, int rows, int n, int cols, int row_groups,
                                               char* stage /* LDS: 4 x kMmWaveLds */, float* red /* LDS: [4 waves][64 lanes][4] */,
                                               const bf16_t* gain = nullptr, const float& eps = 0.f /* read by emit.prepare() */, bf16_t* hstore = nullptr) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int kq = lane >> 4;
    const int ncb = (n + 15) / 16;
    const int cb = blockIdx.x % ncb, rg = blockIdx.x / ncb;
    const int ntiles = (rows + 15) / 16, per = (ntiles + row_groups - 1) / row_groups;
    const int t0 = rg * per, t1 = (t0 + per < ntiles) ? t0 + per : ntiles;
    if (t0 >= t1) return;                                  // whole workgroup: nothing waits on it
    const int j0 = cb * 16;
    char* lds = stage + wave * kMmWaveLds;
    unsigned g[16][4], gw[16][4];
    v4u a[kMmSteps], b[kMmSteps];
    if constexpr (SINGLE) {
        // The h rows (from L2) are asked for before the weights (from HBM): loads return in order, so
        // the tile is staged and its fragments are back in registers while the weights are still on
        // their way; then the same LDS slice takes the weights.  The weight fragments stay in registers
        // for all tiles of the workgroup, and a later tile's rows are in flight across the multiplies
        // of the one before.
        mm_load_rows<FULL, AL>(h, rows, cols, t0 * 16, 0, wave, lane, g);
        unsigned wg[4] = {0u, 0u, 0u, 0u};
        if constexpr (PRO) load_vec_global<bf16_t, AL, false>(gain + mm_k0(0, wave, lane), wg);   // before the weights: loads come back in order
        mm_load_rows<FULL, AL>(W, n, cols, j0, 0, wave, lane, gw);
        emit.prepare();                                      // the epilogue's table right behind the weight loads
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        if constexpr (PRO) {
            static_assert(FULL && SINGLE, "the prologue exists for rows of 2048 columns");
            bf16_t* tile_store = (hstore && cb == 0) ? hstore + (size_t)t0 * 16 * (32 * 4 * kMmSteps) : nullptr;
            mm_rmsnorm_rows<16>(g, wg, eps, tile_store, rows - t0 * 16, wave, lane, reinterpret_cast<float*>(stage));
            lds_barrier();        // the sums are read: the staging area takes the rows now
        }
        mm_stage(lds, lane, g);
        mm_read_frags(lds, lane, a);
        mm_zero_tail<FULL>(a, cols, 0, wave, kq);
        if (t1 - t0 > 1) mm_load_rows<FULL, AL>(h, rows, cols, (t0 + 1) * 16, 0, wave, lane, g);
        mm_stage(lds, lane, gw);
        mm_read_frags(lds, lane, b);
        mm_zero_tail<FULL>(b, cols, 0, wave, kq);
        __builtin_amdgcn_sched_barrier(0);   // all fragment reads before the first multiply, not one LDS latency per pair
        mm_emit_begin(emit, n, t0 * 16, j0, wave, lane);
        mm_mfma(a, b, acc);
        mm_reduce_store(red, acc, emit, wave, lane);
#pragma unroll 1
        for (int t = t0 + 1; t < t1; t++) {
            acc = f32x4{0.f, 0.f, 0.f, 0.f};
            mm_stage(lds, lane, g);
            if (t + 1 < t1) mm_load_rows<FULL, AL>(h, rows, cols, (t + 1) * 16, 0, wave, lane, g);
            mm_read_frags(lds, lane, a);
            mm_zero_tail<FULL>(a, cols, 0, wave, kq);
            __builtin_amdgcn_sched_barrier(0);
            mm_emit_begin(emit, n, t * 16, j0, wave, lane);
            mm_mfma(a, b, acc);
            mm_reduce_store(red, acc, emit, wave, lane);
        }
    } else {
        emit.prepare();
#pragma unroll 1
        for (int t = t0; t < t1; t++) {
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
            for (int s0 = 0; s0 * 32 < cols; s0 += 4 * kMmSteps) {
                mm_load_rows<FULL, AL>(h, rows, cols, t * 16, s0, wave, lane, g);
                mm_load_rows<FULL, AL>(W, n, cols, j0, s0, wave, lane, gw);
                mm_stage(lds, lane, g);
                mm_read_frags(lds, lane, a);
                mm_zero_tail<FULL>(a, cols, s0, wave, kq);
                mm_stage(lds, lane, gw);
                mm_read_frags(lds, lane, b);
                mm_zero_tail<FULL>(b, cols, s0, wave, kq);
                __builtin_amdgcn_sched_barrier(0);
                mm_mfma(a, b, acc);
            }
            mm_emit_begin(emit, n, t * 16, j0, wave, lane);
            mm_reduce_store(red, acc, emit, wave, lane);
        }
    }
}

// Narrow form for one tile of rows (rows <= 16) and cols <= 2048: 8 output columns per workgroup, so
// that 2048 columns make 256 workgroups and every CU pulls weights (a loads-only kernel takes in the
// same bytes 0.35 us faster from 256 CUs than from 128); half of each multiply is idle, which costs
// nothing here.  Only the 8 weight rows are loaded and staged: fragment columns 8-15 are whatever the
// slot held before and their results are never stored.  NRH = 8 (4) when rows <= 8 (4): the absent
// rows of the tile are not loaded either.  With two tiles of rows (8 columns x 2 tiles = 512
// workgroups, measured) it loses to the 16-column form: 5.7 against 4.9 us at 32 rows.
// RMSNorm of the rows the narrow form has just loaded, as a prologue (FULL, 2048 columns): lane (wave, l)
// holds 16-byte chunk c of every row, where c runs over all 256 chunks of a row across the workgroup, but
// not in lane order.  The stand-alone kernel's sums must be reproduced bit for bit: per chunk the fused
// sum of squares in element order (any lane can do that); then the stand-alone kernel's reduction, which
// is a tree of fixed shape over the chunk sums in chunk order -- wave_sum adds neighbours, then pairs of
// pairs, of quads, of eights (a floating-point add does not care which operand is which), then the four
// sixteens in order, and the four wave sums in order.  Here the chunk sums go to LDS in chunk order and
// the workgroup's 16 * NRH subtrees of sixteen leaves are spread over its lanes, one each; lane r < NRH
// then finishes row r (four sixteens per wave sum, four wave sums) and turns the total into the row's
// scale; every lane scales its own chunks: (x * scale) * gain, one rounding.  `scratch`: NRH * 336 + NRH
// floats of LDS that nothing else uses until the rows are staged.  hstore: this workgroup also stores the rows.
template <int NRH>
__device__ __forceinline__ void mm_rmsnorm_rows(unsigned (*g)[4], const unsigned* wg /* the lane's chunk of the gain */, float eps, bf16_t* hstore,
                                                int rows, int wave, int lane, float* scratch) {
    constexpr int kCols = 32 * 4 * kMmSteps;
    constexpr int kRow = 256 + 64;             // a row of chunk sums, 8 floats of padding after every 32: the lanes of a wave hold
                                               // chunks 32 apart, which would otherwise all fall into the same eight banks
    const int tid = wave * 64 + lane;
    const int k0 = mm_k0(0, wave, lane);
    float* sq = scratch;                       // [NRH][kRow]: chunk sums in chunk order
    float* six = scratch + NRH * kRow;         // [NRH][16]: sums of sixteen chunks
    float* scale = six + NRH * 16;             // [NRH]
    auto at = [](int c) { return c + 8 * (c >> 5); };
    float fx[NRH][8];
#pragma unroll
    for (int r = 0; r < NRH; r++) {
        Vec<bf16_t, 16>::unpack(g[r], fx[r]);
        float acc = 0.f;
#pragma unroll
        for (int e = 0; e < 8; e++) acc = __builtin_fmaf(fx[r][e], fx[r][e], acc);
        sq[r * kRow + at(k0 >> 3)] = acc;
    }
    lds_barrier();
    if (tid < 16 * NRH) {                      // subtree tid: row tid / 16, chunks 16 * (tid % 16) .. + 15
        const f32x4* leaf = reinterpret_cast<const f32x4*>(sq + (tid >> 4) * kRow + at((tid & 15) * 16));
        const f32x4 l0 = leaf[0], l1 = leaf[1], l2 = leaf[2], l3 = leaf[3];
        const float q0 = (l0.x + l0.y) + (l0.z + l0.w), q1 = (l1.x + l1.y) + (l1.z + l1.w);
        const float q2 = (l2.x + l2.y) + (l2.z + l2.w), q3 = (l3.x + l3.y) + (l3.z + l3.w);
        six[tid] = (q0 + q1) + (q2 + q3);
    }
    lds_barrier();
    if (tid < NRH) {
        const f32x4* sx = reinterpret_cast<const f32x4*>(six + tid * 16);
        float wsum[4];
#pragma unroll
        for (int w = 0; w < 4; w++) wsum[w] = ((sx[w].x + sx[w].y) + sx[w].z) + sx[w].w;
        const float total = ((wsum[0] + wsum[1]) + wsum[2]) + wsum[3];
        scale[tid] = 1.0f / sqrtf(total / (float)kCols + eps);
    }
    lds_barrier();
    float fg[8];
    Vec<bf16_t, 16>::unpack(wg, fg);
#pragma unroll
    for (int r = 0; r < NRH; r++) {
        float fo[8];
        const float sc = scale[r];
#pragma unroll
        for (int e = 0; e < 8; e++) fo[e] = (fx[r][e] * sc) * fg[e];
        Vec<bf16_t, 16>::pack(fo, g[r]);
    }
    if (hstore) {
#pragma unroll
        for (int r = 0; r < NRH; r++)
            if (r < rows) store_vec_global(hstore + (size_t)r * kCols + k0, g[r]);
    }
}

template <bool FULL, bool AL, int NRH, bool PRO = false, class Emit>
__device__ __forceinline__ void gemm_mfma_narrow_body(const bf16_t* W, const bf16_t* h, Emit& emit, int rows, int n, int cols,
                                                      char* stage, float* red, const bf16_t* gain = nullptr, const float& eps = 0.f /* read by emit.prepare() */,
                                                      bf16_t* hstore = nullptr) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int kq = lane >> 4;
    const int j0 = blockIdx.x * 8, r0 = 0;
    char* lds = stage + wave * kMmWaveLds;
    unsigned g[NRH][4], gw[8][4];
    v4u a[kMmSteps], b[kMmSteps];
    mm_load_rows<FULL, AL, NRH>(h, rows, cols, r0, 0, wave, lane, g);      // with a prologue: the rows to normalise
    unsigned wg[4] = {0u, 0u, 0u, 0u};
    if constexpr (PRO) load_vec_global<bf16_t, AL, false>(gain + mm_k0(0, wave, lane), wg);   // before the weights: loads come back in order
    mm_load_rows<FULL, AL, 8>(W, n, cols, j0, 0, wave, lane, gw);
    emit.prepare();                                          // the epilogue's table right behind the weight loads
    if constexpr (Emit::kEarly) mm_emit_begin<8>(emit, n, r0, j0, wave, lane);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    if constexpr (PRO) {
        static_assert(FULL, "the prologue exists for rows of 2048 columns");
        static_assert((NRH * 336 + NRH) * sizeof(float) <= 4 * kMmWaveLds, "the prologue's sums fit the staging area");
        mm_rmsnorm_rows<NRH>(g, wg, eps, hstore, rows, wave, lane, reinterpret_cast<float*>(stage));
        lds_barrier();        // the sums are read: the staging area takes the rows now
    }
    mm_stage<NRH>(lds, lane, g);
    mm_read_frags(lds, lane, a);
    mm_zero_tail<FULL>(a, cols, 0, wave, kq);
    mm_stage<8>(lds, lane, gw);
    mm_read_frags(lds, lane, b);
    mm_zero_tail<FULL>(b, cols, 0, wave, kq);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!Emit::kEarly) mm_emit_begin<8>(emit, n, r0, j0, wave, lane);
    mm_mfma(a, b, acc);
    mm_reduce_store(red, acc, emit, wave, lane);
}

template <int IND, bool FULL, int NRH>
__global__ __launch_bounds__(kBlock, 2) void k_gemm_mfma_bf16_narrow(GemvArgs p) {
    const bf16_t* W = static_cast<const bf16_t*>(resolve<(IND & 1) != 0>(p.W));
    const bf16_t* h = static_cast<const bf16_t*>(resolve<(IND & 2) != 0>(p.h));
    bf16_t* y = static_cast<bf16_t*>(p.out);
    MmStore<1> emit{y, p.rows, p.n};
    __shared__ __attribute__((aligned(16))) char stage[4 * kMmWaveLds];
    __shared__ float red[4 * 64 * 4];
    const bool al = aligned_to(W, 16) && aligned_to(h, 16);
    if (__builtin_expect(al, 1)) gemm_mfma_narrow_body<FULL, true, NRH>(W, h, emit, p.rows, p.n, p.cols, stage, red);
    else gemm_mfma_narrow_body<FULL, false, NRH>(W, h, emit, p.rows, p.n, p.cols, stage, red);
}

// Wide form for many rows and cols == 2048: 32 output columns per workgroup, i.e. two sets of weight
// fragments and two accumulators against every staged tile of h, which halves the h traffic per
// output (the bound once there are many rows).  One workgroup per CU (the fragments of 32 columns do not fit
// the register budget of two), waves 0 and 1 each finish one 16-column half.
template <bool AL, class Emit>
__device__ __forceinline__ void gemm_mfma_wide_body(const bf16_t* W, const bf16_t* h, Emit& emit, int rows, int n, int cols, int row_groups,
                                                    char* stage, float* red /* LDS: [2 halves][4 waves][64 lanes][4] */) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int ncb = (n + 31) / 32;
    const int cb = blockIdx.x % ncb, rg = blockIdx.x / ncb;
    const int ntiles = (rows + 15) / 16, per = (ntiles + row_groups - 1) / row_groups;
    const int t0 = rg * per, t1 = (t0 + per < ntiles) ? t0 + per : ntiles;
    if (t0 >= t1) return;
    const int j0 = cb * 32;
    char* lds = stage + wave * kMmWaveLds;
    unsigned g[16][4], gw0[16][4], gw1[16][4];
    v4u a[kMmSteps], b0[kMmSteps], b1[kMmSteps];
    mm_load_rows<true, AL>(h, rows, cols, t0 * 16, 0, wave, lane, g);
    mm_load_rows<true, AL>(W, n, cols, j0, 0, wave, lane, gw0);
    mm_load_rows<true, AL>(W, n, cols, j0 + 16, 0, wave, lane, gw1);
    emit.prepare();      // the epilogue's table right behind the weight loads
    mm_stage(lds, lane, g);
    mm_read_frags(lds, lane, a);
    if (t1 - t0 > 1) mm_load_rows<true, AL>(h, rows, cols, (t0 + 1) * 16, 0, wave, lane, g);
    mm_stage(lds, lane, gw0);
    mm_read_frags(lds, lane, b0);
    mm_stage(lds, lane, gw1);
    mm_read_frags(lds, lane, b1);
    for (int t = t0;;) {
        f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
        __builtin_amdgcn_sched_barrier(0);
        // output stage: wave w finishes rows 2 * (w >> 1), + 1 of each accumulator lane's four, in 16-column half w & 1
        emit.begin(t * 16 + (lane >> 4) * 4 + (wave >> 1) * 2, j0 + (wave & 1) * 16 + (lane & 15), j0 + (wave & 1) * 16 + (lane & 15) < n);
#pragma unroll
        for (int i = 0; i < kMmSteps; i++) {
            acc0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[i]), __builtin_bit_cast(bf16x8, b0[i]), acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[i]), __builtin_bit_cast(bf16x8, b1[i]), acc1, 0, 0, 0);
        }
        asm volatile("s_nop 15\n\ts_nop 15" : "+v"(acc0), "+v"(acc1));   // see mm_reduce_store
        float* d0 = red + ((size_t)(0 * 4 + wave) * 64 + lane) * 4;
        float* d1 = red + ((size_t)(1 * 4 + wave) * 64 + lane) * 4;
        d0[0] = acc0.x; d0[1] = acc0.y; d0[2] = acc0.z; d0[3] = acc0.w;
        d1[0] = acc1.x; d1[1] = acc1.y; d1[2] = acc1.z; d1[3] = acc1.w;
        __syncthreads();
        {
            const float* src = red + (size_t)(wave & 1) * 4 * 64 * 4;
#pragma unroll
            for (int k = 0; k < 2; k++) {
                const int e = (wave >> 1) * 2 + k;
                const float p0 = src[((size_t)0 * 64 + lane) * 4 + e], p1 = src[((size_t)1 * 64 + lane) * 4 + e];
                const float p2 = src[((size_t)2 * 64 + lane) * 4 + e], p3 = src[((size_t)3 * 64 + lane) * 4 + e];
                emit.put(k, ((p0 + p1) + p2) + p3);
            }
        }
        __syncthreads();
        emit.end();
        if (++t >= t1) break;
        mm_stage(lds, lane, g);
        if (t + 1 < t1) mm_load_rows<true, AL>(h, rows, cols, (t + 1) * 16, 0, wave, lane, g);
        mm_read_frags(lds, lane, a);
    }
}

template <int IND>
__global__ __launch_bounds__(kBlock, 1) void k_gemm_mfma_bf16_wide(GemvArgs p) {
    const bf16_t* W = static_cast<const bf16_t*>(resolve<(IND & 1) != 0>(p.W));
    const bf16_t* h = static_cast<const bf16_t*>(resolve<(IND & 2) != 0>(p.h));
    bf16_t* y = static_cast<bf16_t*>(p.out);
    MmStore<2> emit{y, p.rows, p.n};
    __shared__ __attribute__((aligned(16))) char stage[4 * kMmWaveLds];
    __shared__ float red[2 * 4 * 64 * 4];
    const bool al = aligned_to(W, 16) && aligned_to(h, 16);
    if (__builtin_expect(al, 1)) gemm_mfma_wide_body<true>(W, h, emit, p.rows, p.n, p.cols, p.row_groups, stage, red);
    else gemm_mfma_wide_body<false>(W, h, emit, p.rows, p.n, p.cols, p.row_groups, stage, red);
}

template <int IND, bool FULL, bool SINGLE>
__global__ __launch_bounds__(kBlock, 2) void k_gemm_mfma_bf16(GemvArgs p) {
    const bf16_t* W = static_cast<const bf16_t*>(resolve<(IND & 1) != 0>(p.W));
    const bf16_t* h = static_cast<const bf16_t*>(resolve<(IND & 2) != 0>(p.h));
    bf16_t* y = static_cast<bf16_t*>(p.out);
    MmStore<1> emit{y, p.rows, p.n};
    __shared__ __attribute__((aligned(16))) char stage[4 * kMmWaveLds];
    __shared__ float red[4 * 64 * 4];
    const bool al = aligned_to(W, 16) && aligned_to(h, 16);   // rows keep the alignment: cols is a multiple of 8
    if (__builtin_expect(al, 1)) gemm_mfma_body<FULL, SINGLE, true>(W, h, emit, p.rows, p.n, p.cols, p.row_groups, stage, red);
    else gemm_mfma_body<FULL, SINGLE, false>(W, h, emit, p.rows, p.n, p.cols, p.row_groups, stage, red);
}

// The matrix-core forms with an elementwise epilogue (kernels.h, GemvEpiArgs; no prologue): the same bodies,
// with MmEpilogue in place of the plain store.  Only for rows of 2048 columns.  FORM 0: narrow, 8 rows of h
// loaded; 1: narrow, 16; 2: 16 columns per workgroup, one pass over K; 3: wide.
template <int FORM, bool PRO = false>
__global__ __launch_bounds__(kBlock, (FORM == 3 || PRO) ? 1 : 2) void k_gemm_mfma_epilogue(GemvEpiArgs p) {
    static_assert(!PRO || FORM <= 2, "a prologue exists for the forms with one tile of rows per workgroup");
    // As in k_gemv_rows: the first 64 bytes of the arguments hold everything that is needed before the
    // loads of h and the weights can go out, and only those are waited for here, in one batch of scalar loads;
    // the epilogue's table and eps are read once the weights are on their way (MmEpilogue::prepare).
    static_assert(offsetof(GemvEpiArgs, gain) + sizeof(void*) == 64, "what the kernel needs first sits in the first 64 bytes");
    const void* Wa = p.g.W;
    const void* ha = p.g.h;
    bf16_t* y = static_cast<bf16_t*>(p.g.out);
    int rows = p.g.rows, n = p.g.n, cols = p.g.cols, row_groups = p.g.row_groups;
    unsigned head = p.head;
    int n_epi = p.n_epi;
    const void* xa = p.x;
    const void* ga = p.gain;
    asm volatile("" : "+s"(Wa), "+s"(ha), "+s"(y), "+s"(rows), "+s"(n), "+s"(cols), "+s"(row_groups), "+s"(head), "+s"(n_epi), "+s"(xa), "+s"(ga));
    const void PG_CONSTANT* const ka = (const void PG_CONSTANT*)__builtin_amdgcn_kernarg_segment_ptr();   // a readable address for a load whose result is not used
    using SlotPtr = const void* const PG_CONSTANT*;
    auto slot_addr = [&](const void* q, bool is_slot) -> SlotPtr { return is_slot ? (SlotPtr)(uintptr_t)q : (SlotPtr)ka; };
    // with a prologue the GEMV's input is computed from x and the gain; p.g.h is where the normalised rows are stored
    if (head & (1u | (PRO ? kEpiXSlot | kEpiGainSlot : 2u))) {      // some operand is a pointer-table slot: all in one batch, without branches
        const bool sw = head & 1u, sh = head & (PRO ? kEpiXSlot : 2u), sg = PRO && (head & kEpiGainSlot);
        SlotPtr aw = slot_addr(Wa, sw), ah = slot_addr(PRO ? xa : ha, sh), ag = slot_addr(ga, sg);
        const void* tw = *aw;
        const void* th = *ah;
        const void* tg = PRO ? *ag : nullptr;
        asm volatile("" : "+s"(tw), "+s"(th), "+s"(tg));
        if (sw) Wa = tw;
        if (sh) { if (PRO) xa = th; else ha = th; }
        if (sg) ga = tg;
    }
    const bf16_t* W = static_cast<const bf16_t*>(Wa);
    const bf16_t* h = static_cast<const bf16_t*>(PRO ? xa : ha);
    const bf16_t* gain = PRO ? static_cast<const bf16_t*>(ga) : nullptr;
    // the narrow forms have one workgroup per column block: the first stores; the 16-column form picks its column block 0 itself
    bf16_t* hstore = (PRO && (head & kEpiStoreH) && (FORM == 2 || blockIdx.x == 0)) ? static_cast<bf16_t*>(const_cast<void*>(ha)) : nullptr;
    __shared__ __attribute__((aligned(16))) char stage[4 * kMmWaveLds];
    __shared__ float red[(FORM == 3 ? 2 : 1) * 4 * 64 * 4];
    MmEpilogue<FORM == 3 ? 2 : 1, FORM <= 1> emit;
    emit.y = y; emit.rows = rows; emit.n = n; emit.head = head; emit.n_epi = n_epi; emit.ka = ka;
    const bool al = aligned_to(W, 16) && aligned_to(h, 16) && (!PRO || aligned_to(gain, 16));
    if constexpr (FORM == 0) {
        if (__builtin_expect(al, 1)) gemm_mfma_narrow_body<true, true, 8, PRO>(W, h, emit, rows, n, cols, stage, red, gain, emit.eps, hstore);
        else gemm_mfma_narrow_body<true, false, 8, PRO>(W, h, emit, rows, n, cols, stage, red, gain, emit.eps, hstore);
    } else if constexpr (FORM == 1) {
        if (__builtin_expect(al, 1)) gemm_mfma_narrow_body<true, true, 16, PRO>(W, h, emit, rows, n, cols, stage, red, gain, emit.eps, hstore);
        else gemm_mfma_narrow_body<true, false, 16, PRO>(W, h, emit, rows, n, cols, stage, red, gain, emit.eps, hstore);
    } else if constexpr (FORM == 2) {
        if (__builtin_expect(al, 1)) gemm_mfma_body<true, true, true, PRO>(W, h, emit, rows, n, cols, row_groups, stage, red, gain, emit.eps, hstore);
        else gemm_mfma_body<true, true, false, PRO>(W, h, emit, rows, n, cols, row_groups, stage, red, gain, emit.eps, hstore);
    } else {
        if (__builtin_expect(al, 1)) gemm_mfma_wide_body<true>(W, h, emit, rows, n, cols, row_groups, stage, red);
        else gemm_mfma_wide_body<false>(W, h, emit, rows, n, cols, row_groups, stage, red);
    }
}

// ---- one to four rows of h, rows of any width: the sums, and in front of them optionally the RMSNorm ------
// bf16.  A wave computes R output columns (R weight rows of up to U * 64 vectors, U per lane); h is fetched once per
// workgroup (lane t vectors t, t + 256, ..., asked for before the weights) and shared by the four waves through
// LDS.  Every load of the wave is in flight before the first wait.  Same products in the same order as gemv_body
// and gemvb_body.
// What bounds it: at 2048 columns and below the latency of one dispatch (1.55 us of graph node, then x from memory,
// the reduction, the weights, the tail, the store), not bytes; the sums of all rows and columns are therefore
// reduced together (wave_sums) and the rows' scales worked out side by side.  From about 4096 columns on, the
// weights: 4096 x 4096 at four rows takes 9.8 us with its node, 3.4 TB/s.  Decode chains with one dispatch per
// sub-block against the four to five they took before, us per iteration: 520 columns, 3 rows, 120 sub-blocks
// 1108 -> 440; 4096 columns, 4 rows, 30 sub-blocks 504 -> 294; 2048 columns, 1 row, 120 sub-blocks 439 -> 431 (this
// width was merged already; the rest is the scalar row addresses and the common reduction).
// EXACT: a row is exactly 512 * U columns.  Otherwise rows end anywhere: a vector that reaches past
// the end is fetched from the row's last eight columns instead (no load leaves the row, whatever its alignment:
// vector loads here take any element boundary) and shifted into place, zeros behind.
// PRO: h is not loaded but computed here -- `h` points at the rows x to normalise, `gain` and `eps` are
// RMSNorm's; the arithmetic is rms_body's (fused multiply-add sum of squares in element order over the lane's
// vectors, wave_sum, the four wave sums added in a fixed order through LDS, 1 / sqrt(mean + eps), (x * scale) *
// gain, one rounding), and what lane t computes goes where lane t's vectors of h would have gone.
// hstore != nullptr: this workgroup also stores the rows there.
// `after_issue()` runs once every weight load of the wave has been asked for (the kernel reads the epilogue's
// table and asks for its operands there: every instruction in front of the weight loads delays the whole kernel
// -- asking for the epilogue's operands first, so that they would be back before the weights, measured 0.17 us
// slower per launch); sums[rr * R + r] receives the lane's part of the dot products.
// (eps by reference: the kernel reads it from its arguments inside the hook.)
template <bool NT>
__device__ __forceinline__ void load_any(const bf16_t* base /* uniform */, unsigned elem, unsigned* w) {
    const v4u_any PG_GLOBAL* q = (const v4u_any PG_GLOBAL*)((const bf16_t PG_GLOBAL*)(uintptr_t)base + elem);
    v4u t;
    if constexpr (NT) t = __builtin_nontemporal_load(q);
    else t = *q;
    w[0] = t.x; w[1] = t.y; w[2] = t.z; w[3] = t.w;
}
// vector v of a row of `cols` >= 8 elements: where it is fetched ...
template <bool EXACT>
__device__ __forceinline__ unsigned span_at(int cols, int v) {
    if constexpr (EXACT) return (unsigned)v * 8u;
    const int at = v * 8;
    return (unsigned)(at < cols - 8 ? at : cols - 8);
}
// ... and what becomes of it: elements past the row's end are zeros
template <bool EXACT>
__device__ __forceinline__ void span_fix(int cols, int v, unsigned* w) {
    if constexpr (!EXACT) {
        const int over = v * 8 + 8 - cols;
        if (over > 0) {                                  // the fetched vector lies `over` elements before its place
            const unsigned s = (unsigned)(over < 8 ? over : 8);
            if (s & 1u) { w[0] = (w[0] >> 16) | (w[1] << 16); w[1] = (w[1] >> 16) | (w[2] << 16); w[2] = (w[2] >> 16) | (w[3] << 16); w[3] >>= 16; }
            if (s & 2u) { w[0] = w[1]; w[1] = w[2]; w[2] = w[3]; w[3] = 0u; }
            if (s & 4u) { w[0] = w[2]; w[1] = w[3]; w[2] = w[3] = 0u; }
            if (s & 8u) w[0] = w[1] = w[2] = w[3] = 0u;
        }
    }
}
__device__ __forceinline__ void span_store(bf16_t* row, int cols, int v, const unsigned* w) {
    if (v * 8 + 8 <= cols) {
        *(v4u_any PG_GLOBAL*)(uintptr_t)(row + (size_t)v * 8) = v4u{w[0], w[1], w[2], w[3]};
    } else {
#pragma unroll
        for (int e = 0; e < 8; e++)
            if (v * 8 + e < cols) *(unsigned short PG_GLOBAL*)(uintptr_t)(row + (size_t)v * 8 + e) = (unsigned short)(w[e / 2] >> (16 * (e & 1)));
    }
}

template <int R, int RB, int U, bool EXACT, bool PRO, class Hook>
__device__ __forceinline__ void gemv_rows_sums(const bf16_t* W, const bf16_t* h, int n, int cols, int j0 /* uniform */, int lane, int tid, v4u* hs /* [RB][U * 64] */,
                                               Hook after_issue, float (&sums)[R * RB],
                                               const bf16_t* gain, const float& eps, bf16_t* hstore, f32x4* part /* [4]: four wave sums per row */) {
    constexpr int KC = (U + 3) / 4;                      // vectors per lane of the workgroup
    if constexpr (EXACT) cols = 512 * U;
    // vector c of lane tid exists for every lane unless U is no multiple of four: then the last waves have none of the last
    auto mine = [&](int c) { return U % 4 == 0 || c < KC - 1 || tid < 64 * (U % 4); };
    unsigned hv[RB][KC][4], wg[KC][4], ww[R][U][4];
#pragma unroll
    for (int rr = 0; rr < RB; rr++)
#pragma unroll
        for (int c = 0; c < KC; c++) load_any<false>(h + (size_t)rr * cols, mine(c) ? span_at<EXACT>(cols, c * kBlock + tid) : 0u, hv[rr][c]);
    if constexpr (PRO)
#pragma unroll
        for (int c = 0; c < KC; c++) load_any<false>(gain, mine(c) ? span_at<EXACT>(cols, c * kBlock + tid) : 0u, wg[c]);
    __builtin_amdgcn_sched_barrier(0);   // h first: loads come back in the order they were issued
#pragma unroll
    for (int r = 0; r < R; r++) {
        const bf16_t* wrow = W + (size_t)((j0 + r < n) ? j0 + r : n - 1) * cols;   // a ragged last group re-reads the last row
#pragma unroll
        for (int u = 0; u < U; u++) load_any<true>(wrow, span_at<EXACT>(cols, u * 64 + lane), ww[r][u]);
    }
    __builtin_amdgcn_sched_barrier(0);
    after_issue();
#pragma unroll
    for (int rr = 0; rr < RB; rr++)
#pragma unroll
        for (int c = 0; c < KC; c++) {
            span_fix<EXACT>(cols, c * kBlock + tid, hv[rr][c]);
            if (!mine(c)) hv[rr][c][0] = hv[rr][c][1] = hv[rr][c][2] = hv[rr][c][3] = 0u;
        }
    if constexpr (PRO) {
        // every row's sum of squares first, then one barrier for all rows (a row of partial sums per row of x), and one
        // square root and division for all rows: lane r works out row r's scale (each row's own took 0.1 us)
        float sq[RB];
#pragma unroll
        for (int rr = 0; rr < RB; rr++) {
            sq[rr] = 0.f;
#pragma unroll
            for (int c = 0; c < KC; c++) {
                float fx[8];
                Vec<bf16_t, 16>::unpack(hv[rr][c], fx);
#pragma unroll
                for (int e = 0; e < 8; e++) sq[rr] = __builtin_fmaf(fx[e], fx[e], sq[rr]);
            }
        }
        float wsum;
        if constexpr (RB == 1) wsum = wave_sum(sq[0]);
        else wsum = wave_sums<RB>(sq, lane);
        if (lane < RB) reinterpret_cast<float*>(part)[lane * (kBlock / 64) + (tid >> 6)] = wsum;      // sums_index(lane) == lane here
        lds_barrier();
        const f32x4 p4 = part[lane & 3];           // rows beyond RB: nothing reads what comes of them
        const float total = ((p4.x + p4.y) + p4.z) + p4.w;
        const float my_scale = 1.0f / sqrtf(total / (float)cols + eps);
#pragma unroll
        for (int rr = 0; rr < RB; rr++) {
            const float scale = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_scale), rr));
#pragma unroll
            for (int c = 0; c < KC; c++) {
                float fx[8], fg[8], fo[8];
                Vec<bf16_t, 16>::unpack(hv[rr][c], fx);
                if (rr == 0) span_fix<EXACT>(cols, c * kBlock + tid, wg[c]);
                Vec<bf16_t, 16>::unpack(wg[c], fg);
#pragma unroll
                for (int e = 0; e < 8; e++) fo[e] = (fx[e] * scale) * fg[e];
                Vec<bf16_t, 16>::pack(fo, hv[rr][c]);
            }
        }
    }
#pragma unroll
    for (int rr = 0; rr < RB; rr++)
#pragma unroll
        for (int c = 0; c < KC; c++) if (mine(c)) hs[rr * (U * 64) + c * kBlock + tid] = v4u{hv[rr][c][0], hv[rr][c][1], hv[rr][c][2], hv[rr][c][3]};
    lds_barrier();        // every wave of the workgroup gets here: none leaves early
    if constexpr (PRO) {  // after the barrier: nothing waits for these stores
        if (hstore)
#pragma unroll
            for (int rr = 0; rr < RB; rr++)
#pragma unroll
                for (int c = 0; c < KC; c++) {
                    if (!mine(c)) continue;
                    if constexpr (EXACT) store_vec_global(hstore + (size_t)rr * cols + (size_t)(c * kBlock + tid) * 8, hv[rr][c]);
                    else span_store(hstore + (size_t)rr * cols, cols, c * kBlock + tid, hv[rr][c]);
                }
    }
#pragma unroll
    for (int e = 0; e < R * RB; e++) sums[e] = 0.f;
#pragma unroll
    for (int u = 0; u < U; u++) {
        unsigned wh[RB][4];
#pragma unroll
        for (int rr = 0; rr < RB; rr++) {
            const v4u t = hs[rr * (U * 64) + u * 64 + lane];
            wh[rr][0] = t.x; wh[rr][1] = t.y; wh[rr][2] = t.z; wh[rr][3] = t.w;
        }
#pragma unroll
        for (int r = 0; r < R; r++) {
            span_fix<EXACT>(cols, u * 64 + lane, ww[r][u]);
#pragma unroll
            for (int rr = 0; rr < RB; rr++) sums[rr * R + r] = dot_acc<bf16_t>(ww[r][u], wh[rr], sums[rr * R + r]);
        }
    }
}

// GEMV with an elementwise epilogue: one lane of each wave per output e (row e / R of h, column j0 + e % R) plays it
// through the kernels that follow (see kernels.h; none of them: the plain GEMV).
template <int R, int RB, int U, bool EXACT, bool PRO>
__global__ __launch_bounds__(kBlock) void k_gemv_rows(GemvEpiArgs p) {
    constexpr int P = kEpiMaxPhases;
    // The GEMV's own arguments first, in one batch of scalar loads (see args_up_front): nothing else stands
    // between the start of the kernel and the weight loads.  The epilogue's table is read once those are on
    // their way (`fetch`), and kept in scalar registers from then on.
    // The first 64 bytes of the arguments hold everything that is needed before the weight loads can go out,
    // and only those are waited for here, in one batch of scalar loads (see args_up_front; the start of the
    // argument buffer arrives in under 0.1 us, the lines behind it take 0.3 us more).  The epilogue's table
    // and eps are read once the weights are on their way (`fetch`).
    static_assert(offsetof(GemvEpiArgs, gain) + sizeof(void*) == 64, "what the kernel needs first sits in the first 64 bytes");
    const void* Wa = p.g.W;
    const void* ha = p.g.h;
    bf16_t* y = static_cast<bf16_t*>(p.g.out);
    int n = p.g.n, cols = p.g.cols;
    unsigned head = p.head;
    int n_epi = p.n_epi;
    const void* xa = p.x;
    const void* ga = p.gain;
    asm volatile("" : "+s"(Wa), "+s"(ha), "+s"(y), "+s"(n), "+s"(cols), "+s"(head), "+s"(n_epi), "+s"(xa), "+s"(ga));
    const void* a0[P];
    const void* a1[P];
    bf16_t* outs[P];
    unsigned ms[P], metas[P], inds[P];
    float eps = 0.f;
    static_assert(P == 3, "the argument batch in fetch names every phase");
    const void PG_CONSTANT* const ka = (const void PG_CONSTANT*)__builtin_amdgcn_kernarg_segment_ptr();   // a readable address for a load whose result is not used
    using SlotPtr = const void* const PG_CONSTANT*;
    auto slot_addr = [&](const void* q, bool is_slot) -> SlotPtr { return is_slot ? (SlotPtr)(uintptr_t)q : (SlotPtr)ka; };
    // with a prologue the GEMV's input is computed from x and the gain; p.g.h is where workgroup 0 stores it
    if (head & (1u | (PRO ? kEpiXSlot | kEpiGainSlot : 2u))) {      // some operand is a pointer-table slot: all in one batch, without branches
        const bool sw = head & 1u, sh = head & (PRO ? kEpiXSlot : 2u), sg = PRO && (head & kEpiGainSlot);
        SlotPtr aw = slot_addr(Wa, sw), ah = slot_addr(PRO ? xa : ha, sh), ag = slot_addr(ga, sg);
        const void* tw = *aw;
        const void* th = *ah;
        const void* tg = PRO ? *ag : nullptr;
        asm volatile("" : "+s"(tw), "+s"(th), "+s"(tg));
        if (sw) Wa = tw;
        if (sh) { if (PRO) xa = th; else ha = th; }
        if (sg) ga = tg;
    }
    const bf16_t* W = static_cast<const bf16_t*>(Wa);
    const bf16_t* h = static_cast<const bf16_t*>(PRO ? xa : ha);
    const bf16_t* gain = PRO ? static_cast<const bf16_t*>(ga) : nullptr;
    bf16_t* hstore = (PRO && (head & kEpiStoreH) && blockIdx.x == 0) ? static_cast<bf16_t*>(const_cast<void*>(ha)) : nullptr;
    __shared__ v4u hs[RB * U * 64];
    __shared__ f32x4 part[4];
    const int tid = threadIdx.x, lane = tid & 63;
    const int j0 = (blockIdx.x * (kBlock / 64) + __builtin_amdgcn_readfirstlane(tid >> 6)) * R;   // uniform: the weight rows' addresses stay in scalar registers
    unsigned ld0[P], ld1[P];
    bool mine = false;
    unsigned idx = 0;
    bool decoder = false;       // the tail is GELU of the GEMV's result, then one or two adds with an operand from memory
    // The epilogue's operands: asked for once the weights are on their way (pointer-table slots first, with
    // scalar loads, all at once).  Always the same number of loads -- an operand that comes from a register
    // slot is fetched from the GEMV's own output buffer instead and ignored -- so that every wait on the
    // weights knows exactly how many younger loads are outstanding.
    auto fetch = [&] {
        {   // the rest of the arguments, through the kernel-argument segment's address made opaque: otherwise the
            // compiler moves these loads (invariant memory) to the top of the kernel, in front of the weight loads
            const GemvEpiArgs PG_CONSTANT* kp = (const GemvEpiArgs PG_CONSTANT*)ka;
            asm volatile("" : "+s"(kp));
            eps = kp->eps;
#pragma unroll
            for (int i = 0; i < P; i++) {
                a0[i] = kp->ph[i].in0; a1[i] = kp->ph[i].in1; outs[i] = static_cast<bf16_t*>(kp->ph[i].out);
                ms[i] = kp->ph[i].m; metas[i] = kp->ph[i].meta; inds[i] = kp->ph[i].ind;
            }
            asm volatile("" : "+s"(eps),
                              "+s"(a0[0]), "+s"(a1[0]), "+s"(outs[0]), "+s"(ms[0]), "+s"(metas[0]), "+s"(inds[0]),
                              "+s"(a0[1]), "+s"(a1[1]), "+s"(outs[1]), "+s"(ms[1]), "+s"(metas[1]), "+s"(inds[1]),
                              "+s"(a0[2]), "+s"(a1[2]), "+s"(outs[2]), "+s"(ms[2]), "+s"(metas[2]), "+s"(inds[2]));
        }
        const int e = sums_index<R * RB>(lane);
        mine = lane < sums_lanes(R * RB) && e < R * RB && j0 + e % R < n;
        idx = mine ? (unsigned)(e / R) * (unsigned)n + (unsigned)(j0 + e % R) : 0u;
        const unsigned total = (unsigned)RB * (unsigned)n;
        bool f0[P], f1[P], s0[P], s1[P];
        unsigned any = 0;
#pragma unroll
        for (int i = 0; i < P; i++) {
            const unsigned mt = metas[i];
            f0[i] = ((mt >> 8) & 0xffu) == kMergeFromMemory;
            f1[i] = (mt & 0xffu) != kGelu && ((mt >> 16) & 0xffu) == kMergeFromMemory;
            s0[i] = f0[i] && (inds[i] & 1u);
            s1[i] = f1[i] && (inds[i] & 2u);
            any |= (f0[i] ? inds[i] & 1u : 0u) | (f1[i] ? inds[i] & 2u : 0u);
        }
        any = __builtin_amdgcn_readfirstlane(any);
        asm volatile("" : "+s"(any));       // keeps what follows behind the weight loads
        {   // the decoder block's tail, recognised here (scalar arithmetic under the weights' latency) so that the
            // tail itself runs it straight through, without the operand and slot selection of the general form
            auto add_of = [](unsigned mt, unsigned q) {
                const unsigned a = (mt >> 8) & 0xffu, b = (mt >> 16) & 0xffu;
                return (mt & 0xffu) == (unsigned)kAdd && ((a == q && b == kMergeFromMemory) || (a == kMergeFromMemory && b == q));
            };
            const unsigned hq = (head >> 8) & 0xffu, d0 = metas[0] >> 24, d1 = metas[1] >> 24;
            decoder = (n_epi == 2 || n_epi == 3) && (metas[0] & 0xffu) == (unsigned)kGelu && ((metas[0] >> 8) & 0xffu) == hq &&
                      add_of(metas[1], d0) && (n_epi == 2 || add_of(metas[2], d1));
        }
        if (any) {
            SlotPtr at0[P], at1[P];
            const void* t0[P];
            const void* t1[P];
#pragma unroll
            for (int i = 0; i < P; i++) { at0[i] = slot_addr(a0[i], s0[i]); at1[i] = slot_addr(a1[i], s1[i]); }
#pragma unroll
            for (int i = 0; i < P; i++) { t0[i] = *at0[i]; t1[i] = *at1[i]; }
            asm volatile("" : "+s"(t0[0]), "+s"(t1[0]), "+s"(t0[1]), "+s"(t1[1]), "+s"(t0[2]), "+s"(t1[2]));
#pragma unroll
            for (int i = 0; i < P; i++) {
                if (s0[i]) a0[i] = t0[i];
                if (s1[i]) a1[i] = t1[i];
            }
        }
        const bf16_t* q0[P];
        const bf16_t* q1[P];
        unsigned mm[P];
        bool plain = true;      // no operand has a broadcast period: the usual case, one branch for all
#pragma unroll
        for (int i = 0; i < P; i++) {
            q0[i] = f0[i] ? static_cast<const bf16_t*>(a0[i]) : y;
            q1[i] = f1[i] ? static_cast<const bf16_t*>(a1[i]) : y;
            mm[i] = f1[i] ? ms[i] : total;
            plain = plain && mm[i] == total;
        }
        if (__builtin_expect(plain, 1)) {
#pragma unroll
            for (int i = 0; i < P; i++) {
                ld0[i] = load_raw_global_at(q0[i], idx);
                ld1[i] = load_raw_global_at(q1[i], idx);
            }
        } else {
#pragma unroll
            for (int i = 0; i < P; i++) {
                ld0[i] = load_raw_global_at(q0[i], idx);
                ld1[i] = load_raw_global_at(q1[i], idx % mm[i]);
            }
        }
    };
    float sums[R * RB];
    gemv_rows_sums<R, RB, U, EXACT, PRO>(W, h, n, cols, j0, lane, tid, hs, fetch, sums, gain, eps, hstore, part);
    float v;
    if constexpr (R * RB == 1) v = wave_sum(sums[0]);
    else v = wave_sums<R * RB>(sums, lane);
    unsigned bits = f32_to_bf16(v);
    // The epilogue's operands have been on their way since before the weights were used; claim them all now,
    // before the first store of the tail.  Loads and stores complete in one queue, in order, so a wait for
    // an operand placed after a store would wait for that store to be acknowledged as well.
    __builtin_amdgcn_s_waitcnt(0x0F70);      // vmcnt(0)
    if (mine && (head & kEpiHeadStore)) *(unsigned short PG_GLOBAL*)(uintptr_t)(y + idx) = (unsigned short)bits;
    float slot[kMergeSlots];
#pragma unroll
    for (int q = 0; q < kMergeSlots; q++) slot[q] = 0.f;
    {
        const unsigned dst = (head >> 8) & 0xffu;
#pragma unroll
        for (int q = 0; q < kMergeSlots; q++)
            if (dst == (unsigned)q) slot[q] = from_raw<bf16_t>(bits);
    }
    if (__builtin_expect(decoder, 1)) {
        // the same kernels with the same arithmetic and roundings, operands known: GELU of the GEMV's rounded result,
        // then each add takes the value before it and its operand from memory, in the order its descriptor names
        const bool st = mine;
        float val = ew_apply<kGelu, false>(from_raw<bf16_t>(bits), 0.f);
        bits = f32_to_bf16(val);
        if (st && (inds[0] & kEpiStore)) *(unsigned short PG_GLOBAL*)(uintptr_t)(outs[0] + idx) = (unsigned short)bits;
        val = from_raw<bf16_t>(bits);
        {
            const bool mem_first = ((metas[1] >> 8) & 0xffu) == kMergeFromMemory;
            const float fa = mem_first ? from_raw<bf16_t>(ld0[1]) : val, fb = mem_first ? val : from_raw<bf16_t>(ld1[1]);
            bits = f32_to_bf16(ew_apply<kAdd, false>(fa, fb));
            if (st && (inds[1] & kEpiStore)) *(unsigned short PG_GLOBAL*)(uintptr_t)(outs[1] + idx) = (unsigned short)bits;
            val = from_raw<bf16_t>(bits);
        }
        if (n_epi == 3) {
            const bool mem_first = ((metas[2] >> 8) & 0xffu) == kMergeFromMemory;
            const float fa = mem_first ? from_raw<bf16_t>(ld0[2]) : val, fb = mem_first ? val : from_raw<bf16_t>(ld1[2]);
            bits = f32_to_bf16(ew_apply<kAdd, false>(fa, fb));
            if (st && (inds[2] & kEpiStore)) *(unsigned short PG_GLOBAL*)(uintptr_t)(outs[2] + idx) = (unsigned short)bits;
        }
        return;
    }
    // Unrolled, with the one big choice (GELU or not) as the only branch inside a phase: a taken branch costs
    // this one-wave-per-SIMD tail more than a dozen arithmetic instructions.
#pragma unroll
    for (int i = 0; i < P; i++) {
        if (i >= n_epi) break;
        const unsigned mt = metas[i], ind = inds[i];
        const unsigned op = mt & 0xffu, src0 = (mt >> 8) & 0xffu, src1 = (mt >> 16) & 0xffu, dst = mt >> 24;
        float fa = from_raw<bf16_t>(ld0[i]), fb = from_raw<bf16_t>(ld1[i]);
#pragma unroll
        for (int q = 0; q < kMergeSlots; q++) {
            if (src0 == (unsigned)q) fa = slot[q];
            if (src1 == (unsigned)q) fb = slot[q];
        }
        float fo;
        if (op == kGelu) {
            fo = ew_apply<kGelu, false>(fa, 0.f);
        } else {
            const float sum = ew_apply<kAdd, false>(fa, fb), prod = ew_apply<kMul, false>(fa, fb);
            fo = op == kAdd ? sum : prod;
        }
        bits = f32_to_bf16(fo);
        if (mine && (ind & kEpiStore)) *(unsigned short PG_GLOBAL*)(uintptr_t)(outs[i] + idx) = (unsigned short)bits;
#pragma unroll
        for (int q = 0; q < kMergeSlots; q++)
            if (dst == (unsigned)q) slot[q] = from_raw<bf16_t>(bits);
    }
}

// ---- host side: pick the instantiation and the launch shape from the kernel's shape alone ----------
template <typename T, int R, int RS>
const void* gemv_by_ind(int ind) {
    switch (ind) {
    case 0: return PG_FN(k_gemv<T, 0, R, RS>);
    case 1: return PG_FN(k_gemv<T, 1, R, RS>);
    case 2: return PG_FN(k_gemv<T, 2, R, RS>);
    case 3: return PG_FN(k_gemv<T, 3, R, RS>);
    default: return nullptr;
    }
}
template <typename T, int R, int RB, int RS>
const void* gemvb_by_ind(int ind) {
    switch (ind) {
    case 0: return PG_FN(k_gemv_batched<T, 0, R, RB, RS>);
    case 1: return PG_FN(k_gemv_batched<T, 1, R, RB, RS>);
    case 2: return PG_FN(k_gemv_batched<T, 2, R, RB, RS>);
    case 3: return PG_FN(k_gemv_batched<T, 3, R, RB, RS>);
    default: return nullptr;
    }
}

template <typename T, int RB>
const void* gemv_shared_by_ind(int ind) {
    switch (ind) {
    case 0: return PG_FN(k_gemv_shared<T, 0, 2, RB>);
    case 1: return PG_FN(k_gemv_shared<T, 1, 2, RB>);
    case 2: return PG_FN(k_gemv_shared<T, 2, 2, RB>);
    case 3: return PG_FN(k_gemv_shared<T, 3, 2, RB>);
    default: return nullptr;
    }
}

template <typename T, int RS>
bool plan_gemv_rs(int ind, int rows, int n, int cols, Launch* out) {
    out->block = dim3(kBlock);
    const bool one_chunk = RS == 0 && cols == 64 * kGemvChunk * (16 / (int)sizeof(T));   // the forms that share h through LDS
    if (rows == 1 && n >= 1024) {
        // two weight rows per wave once there are enough rows to fill the chip with half the waves
        out->fn = one_chunk ? gemv_shared_by_ind<T, 1>(ind) : gemv_by_ind<T, 2, RS>(ind);
        out->grid = dim3(blocks_for(n, (kBlock / 64) * 2));
    } else if (rows == 1) {
        out->fn = gemv_by_ind<T, 1, RS>(ind);
        out->grid = dim3(blocks_for(n, kBlock / 64));
    } else if (n >= 1024) {
        if (one_chunk && rows <= 4) out->fn = rows == 2 ? gemv_shared_by_ind<T, 2>(ind) : rows == 3 ? gemv_shared_by_ind<T, 3>(ind) : gemv_shared_by_ind<T, 4>(ind);
        else out->fn = rows == 2 ? gemvb_by_ind<T, 2, 2, RS>(ind) : gemvb_by_ind<T, 2, 4, RS>(ind);
        out->grid = dim3(blocks_for(n, (kBlock / 64) * 2));
    } else {
        out->fn = rows == 2 ? gemvb_by_ind<T, 1, 2, RS>(ind) : gemvb_by_ind<T, 1, 4, RS>(ind);
        out->grid = dim3(blocks_for(n, kBlock / 64));
    }
    return out->fn != nullptr;
}

template <bool FULL, bool SINGLE>
const void* gemm_by_ind(int ind) {
    switch (ind) {
    case 0: return PG_FN(k_gemm_mfma_bf16<0, FULL, SINGLE>);
    case 1: return PG_FN(k_gemm_mfma_bf16<1, FULL, SINGLE>);
    case 2: return PG_FN(k_gemm_mfma_bf16<2, FULL, SINGLE>);
    case 3: return PG_FN(k_gemm_mfma_bf16<3, FULL, SINGLE>);
    default: return nullptr;
    }
}

template <bool FULL, int NRH>
const void* gemm_narrow_by_ind(int ind) {
    switch (ind) {
    case 0: return PG_FN(k_gemm_mfma_bf16_narrow<0, FULL, NRH>);
    case 1: return PG_FN(k_gemm_mfma_bf16_narrow<1, FULL, NRH>);
    case 2: return PG_FN(k_gemm_mfma_bf16_narrow<2, FULL, NRH>);
    case 3: return PG_FN(k_gemm_mfma_bf16_narrow<3, FULL, NRH>);
    default: return nullptr;
    }
}

// k_gemv_rows: up to 4 rows of h, rows of 8 to 8192 columns (all of a wave's loads are in registers at once);
// two weight rows per wave once half the waves fill the chip, and only then rows beyond 2048 columns.
constexpr int kRowsTwoFrom = 1024;
bool rows_served(long long rows, long long n, long long cols) {
    return rows >= 1 && rows <= 4 && n >= 1 && cols >= 8 && cols <= (n >= kRowsTwoFrom ? 8192 : 2048);
}
template <bool PRO, int RB>
const void* rows_kernel_rb(int n, int cols) {
    const int u = (cols + 511) / 512;
    if (n < kRowsTwoFrom) {
        switch (u) {
        case 1: return PG_FN(k_gemv_rows<1, RB, 1, false, PRO>);
        case 2: return PG_FN(k_gemv_rows<1, RB, 2, false, PRO>);
        case 3: return PG_FN(k_gemv_rows<1, RB, 3, false, PRO>);
        default: return PG_FN(k_gemv_rows<1, RB, 4, false, PRO>);
        }
    }
    switch (cols) {
    case 1024: return PG_FN(k_gemv_rows<2, RB, 2, true, PRO>);
    case 2048: return PG_FN(k_gemv_rows<2, RB, 4, true, PRO>);
    case 4096: return PG_FN(k_gemv_rows<2, RB, 8, true, PRO>);
    case 8192: return PG_FN(k_gemv_rows<2, RB, 16, true, PRO>);
    default: break;
    }
    if (u <= 3) return PG_FN(k_gemv_rows<2, RB, 3, false, PRO>);
    if (u <= 4) return PG_FN(k_gemv_rows<2, RB, 4, false, PRO>);
    if (u <= 8) return PG_FN(k_gemv_rows<2, RB, 8, false, PRO>);
    if (u <= 12) return PG_FN(k_gemv_rows<2, RB, 12, false, PRO>);
    return PG_FN(k_gemv_rows<2, RB, 16, false, PRO>);
}
template <bool PRO>
const void* rows_kernel(int rows, int n, int cols) {
    switch (rows) {
    case 1: return rows_kernel_rb<PRO, 1>(n, cols);
    case 2: return rows_kernel_rb<PRO, 2>(n, cols);
    case 3: return rows_kernel_rb<PRO, 3>(n, cols);
    default: return rows_kernel_rb<PRO, 4>(n, cols);
    }
}

template <typename T>
bool plan_gemv_t(int ind, int rows, int n, int cols, Launch* out) {
    constexpr int NV = 16 / (int)sizeof(T);
    if constexpr (sizeof(T) == 2) {
        // Three and four rows go to the form that shares h through LDS (at 2048 x 2048, us per launch at 2 / 3 / 4 rows: 3.3 / 3.5 /
        // 3.7; vector with h per wave 3.8 / 4.4 / 4.5; matrix-core form with 8 columns per workgroup 3.9 / 4.0 / 4.0).
        if ((rows == 3 || rows == 4) && rows_served(rows, n, cols) && !(n >= 1024 && cols == 64 * kGemvChunk * NV)) {
            out->fn = rows_kernel<false>(rows, n, cols);
            out->arg_bytes = sizeof(GemvEpiArgs);
            out->block = dim3(kBlock);
            out->grid = dim3(blocks_for(n, (kBlock / 64) * (n >= kRowsTwoFrom ? 2 : 1)));
            return true;
        }
        // A dense contraction: matrix cores from 5 rows on.
        const bool narrow_ok = rows <= 16 && cols <= 32 * 4 * kMmSteps && n >= 16;
        if (cols % 8 == 0 && rows > 4) {
            out->block = dim3(kBlock);
            // row groups of 16-row tiles: enough workgroups to fill the chip twice over at most
            const int ntiles = (rows + 15) / 16;
            out->gemm_row_groups = (unsigned)(ntiles < kMmMaxRowGroups ? ntiles : kMmMaxRowGroups);
            out->grid = dim3(blocks_for(n, 16) * out->gemm_row_groups);
            constexpr int kSuper = 32 * 4 * kMmSteps;   // columns one pass of the 4 waves covers
            if (cols == kSuper && rows >= kMmWideRows && n >= 32) {
                out->grid = dim3(blocks_for(n, 32) * out->gemm_row_groups);
                switch (ind) {
                case 0: out->fn = PG_FN(k_gemm_mfma_bf16_wide<0>); break;
                case 1: out->fn = PG_FN(k_gemm_mfma_bf16_wide<1>); break;
                case 2: out->fn = PG_FN(k_gemm_mfma_bf16_wide<2>); break;
                case 3: out->fn = PG_FN(k_gemm_mfma_bf16_wide<3>); break;
                default: out->fn = nullptr;
                }
            } else if (narrow_ok) {
                out->grid = dim3(blocks_for(n, 8));
                out->fn = cols == kSuper ? (rows <= 8 ? gemm_narrow_by_ind<true, 8>(ind) : gemm_narrow_by_ind<true, 16>(ind))
                                         : (rows <= 8 ? gemm_narrow_by_ind<false, 8>(ind) : gemm_narrow_by_ind<false, 16>(ind));
            } else if (cols == kSuper) out->fn = gemm_by_ind<true, true>(ind);
            else if (cols < kSuper) out->fn = gemm_by_ind<false, true>(ind);
            else if (cols % kSuper == 0) out->fn = gemm_by_ind<true, false>(ind);
            else out->fn = gemm_by_ind<false, false>(ind);
            return out->fn != nullptr;
        }
    }
    if (cols % (64 * kGemvChunk * NV) == 0) return plan_gemv_rs<T, 0>(ind, rows, n, cols, out);
    if (cols % NV == 0) return plan_gemv_rs<T, 1>(ind, rows, n, cols, out);
    return plan_gemv_rs<T, 2>(ind, rows, n, cols, out);
}

}  // namespace

bool plan_gemv(int dtype, int ind, int rows, int n, int cols, Launch* out) {
    if (dtype == kF32) return plan_gemv_t<float>(ind, rows, n, cols, out);
    if (dtype == kBF16) return plan_gemv_t<bf16_t>(ind, rows, n, cols, out);
    return false;
}

bool merge_head(int op, int dtype, const Shape& s, long long* n_out) {
    if (op != kGemv || dtype != kBF16 || s.rows < 1) return false;
    if (s.rows <= 4) {
        if (!rows_served(s.rows, s.n, s.cols)) return false;
    } else {
        // the matrix-core forms plan_gemv picks for rows of 2048 columns: narrow (up to 16 rows), 16 columns per
        // workgroup, wide (from kMmWideRows rows)
        if (s.cols != 64 * kGemvChunk * 8 || s.n < 32) return false;
    }
    if (s.rows * s.n > (1ll << 31)) return false;          // element indices are kept in 32 bits
    *n_out = s.rows * s.n;
    return true;
}

static_assert(kPrologueMaxRows < kMmWideRows, "a prologue exists only where a workgroup owns one tile of rows");
const void* gemv_epilogue_kernel(const Shape& s, bool with_prologue) {
    const int rows = (int)s.rows;
    if (rows <= 4) return with_prologue ? rows_kernel<true>(rows, (int)s.n, (int)s.cols) : rows_kernel<false>(rows, (int)s.n, (int)s.cols);
    if (with_prologue) {
        if (rows <= 8) return PG_FN(k_gemm_mfma_epilogue<0, true>);
        if (rows <= 16) return PG_FN(k_gemm_mfma_epilogue<1, true>);
        if (rows <= kPrologueMaxRows) return PG_FN(k_gemm_mfma_epilogue<2, true>);
        return nullptr;
    }
    if (rows <= 8) return PG_FN(k_gemm_mfma_epilogue<0>);
    if (rows <= 16) return PG_FN(k_gemm_mfma_epilogue<1>);
    if (rows < kMmWideRows) return PG_FN(k_gemm_mfma_epilogue<2>);
    return PG_FN(k_gemm_mfma_epilogue<3>);
}

}  // namespace pgk
