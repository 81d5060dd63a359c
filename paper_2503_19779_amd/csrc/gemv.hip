// gemv.hip -- y = h W^T for gfx950 (wave64): the vector-unit forms (one to four rows of h, and every fp32
// shape), the matrix-core forms (five rows and more), and the forms that carry an RMSNorm in front and
// elementwise kernels behind in the same dispatch (kernels.h, "merged dispatches").
//
// Built with -ffp-contract=off: fused multiply-adds appear only where written.
#include "device.h"

#include <type_traits>

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

// Workgroups go to the 8 XCDs in turn, each with an L2 of its own.  The index of the work that workgroup b of `total` takes,
// such that an XCD takes a contiguous stretch of it.
__device__ __forceinline__ unsigned xcd_stretch(unsigned b, unsigned total) {
    const unsigned x = b & 7u, q = total >> 3, r = total & 7u;
    return x * q + (x < r ? x : r) + (b >> 3);
}

// ---- five rows of h and more: the matrix cores ----------------------------------------------------------
// bf16, v_mfma_f32_16x16x32_bf16 with fp32 accumulation.  A GEMV's output has the same bits whichever launch of it
// computes it (eager, merged, with a prologue): K is cut into blocks of 64 and these are dealt out to eight parts in turn; a part's blocks are added up in
// order, two K-steps of 32 each, then parts i and i + 4, then those four sums in order.  Eight waves take a part each, four two each, side by side.  (Four parts err more: rows of W that
// cancel to zero, 128 rows of h, 2048 x 2048: rms of the outputs, which should be 0, 5.3e-6 where eight give 3.9e-6.)
// (Fragments -- A: lane l holds row l & 15, B: column l & 15;
// the eight consecutive k's of chunk l >> 4 of a step; accumulators: lane l holds column l & 15, rows 4 * (l >> 4) .. + 3.)
// Elements beyond a row's end are zeros on both sides: zeroing the weight side alone would turn an Inf or NaN of h
// into NaN in every output (0 * Inf).  Rows beyond the batch and columns beyond n repeat the last one and are never
// stored.
//   - k_gemm_rows: up to 16 rows of up to 2048 columns, one tile of 8 or 16 rows of h per workgroup, all loads in flight at once; the form that can carry
//     the RMSNorm in front, then up to 32 rows in tiles of 4, 8 or 16;
//   - k_gemm_whole: with kernels that ride behind, from 17 rows on, up to 2048 columns, where its grid is one workgroup per CU;
//   - k_gemm_cols: 17 to 80 rows of up to 2048 columns, and any more rows with up to 16 outputs each, alone or where k_gemm_whole's grid is larger;
//   - k_gemm_tile: everything else, K streamed through a ring in LDS.
template <class Part>
__device__ __forceinline__ float parts_sum(Part part) { return (((part(0) + part(4)) + (part(1) + part(5))) + (part(2) + part(6))) + (part(3) + part(7)); }
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));

// 16 bytes at any element boundary, `off` bytes behind a uniform address
template <bool NT>
__device__ __forceinline__ void load_at(const bf16_t* base /* uniform */, unsigned off, unsigned* w) {
    const v4u_any PG_GLOBAL* q = (const v4u_any PG_GLOBAL*)((const char PG_GLOBAL*)(uintptr_t)base + off);
    v4u t;
    if constexpr (NT) t = __builtin_nontemporal_load(q);
    else t = *q;
    w[0] = t.x; w[1] = t.y; w[2] = t.z; w[3] = t.w;
}
template <bool NT>
__device__ __forceinline__ void load_any(const bf16_t* base /* uniform */, unsigned elem, unsigned* w) {
    const v4u_any PG_GLOBAL* q = (const v4u_any PG_GLOBAL*)((const bf16_t PG_GLOBAL*)(uintptr_t)base + elem);
    v4u t;
    if constexpr (NT) t = __builtin_nontemporal_load(q);
    else t = *q;
    w[0] = t.x; w[1] = t.y; w[2] = t.z; w[3] = t.w;
}
// Rows of any number of columns (eight at least) in 16-byte vectors: a vector that reaches past the row's end is
// fetched from the row's last eight elements instead (no load leaves the row, whatever its alignment) and shifted
// into place, zeros behind.  Vector v of a row of `cols` elements: where it is fetched ...
template <bool EXACT>
__device__ __forceinline__ unsigned span_at(int cols, int v) {
    if constexpr (EXACT) return (unsigned)v * 8u;
    const int at = v * 8;
    return (unsigned)(at < cols - 8 ? at : cols - 8);
}
// ... and what becomes of it: elements past the row's end are zeros.  The one vector of a row that the end cuts was fetched the same number
// of elements before its place in every row, so the shift has nothing to decide per lane and only the wave that holds it takes the branch;
// vectors beyond the end are zeroed by selects.
__device__ __forceinline__ void span_shift(unsigned s /* elements, up to 7 */, unsigned* w) {
    if (s & 1u) { w[0] = (w[0] >> 16) | (w[1] << 16); w[1] = (w[1] >> 16) | (w[2] << 16); w[2] = (w[2] >> 16) | (w[3] << 16); w[3] >>= 16; }
    if (s & 2u) { w[0] = w[1]; w[1] = w[2]; w[2] = w[3]; w[3] = 0u; }
    if (s & 4u) { w[0] = w[2]; w[1] = w[3]; w[2] = w[3] = 0u; }
}
template <bool EXACT>
__device__ __forceinline__ void span_fix(int cols, int v, unsigned* w) {
    if constexpr (!EXACT) {
        const int over = v * 8 + 8 - cols;               // the fetched vector lies `over` elements before its place
        if (const unsigned s = 8u - ((unsigned)cols & 7u); s != 8u)
            if (over == (int)s) span_shift(s, w);        // the one that the row's end cuts: s is the same in every lane that gets here
#pragma unroll
        for (int i = 0; i < 4; i++) w[i] = over >= 8 ? 0u : w[i];
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

// What becomes of a finished tile: a lane is given NE consecutive columns of one row -- begin(r, j, ok), put(e, v) for
// each of its sums, end().
// The kernels that follow the GEMV in the chain, element for element, ride along (kernels.h,
// GemvEpiArgs): prepare() reads their table out of the kernel arguments and resolves pointer-table slots --
// the bodies call it once their weight loads are on their way, so that nothing but
// the first 64 bytes of the arguments stands between the start of the kernel and those loads; begin() asks
// for the operands, so that they arrive while the tile is staged and multiplied and the partial sums are
// exchanged; end() plays the kernels on the lane's outputs, rounding to bf16 after each as the stand-alone
// kernels do, with the GELU as the only branch.
// What the table says is worked out on the host (GemvEpiArgs::head: the decoder block's tail, slots, periods): in a
// kernel of one wave per SIMD every scalar instruction counts, and recognising the tail here cost 0.1 - 0.15 us per
// dispatch.  begin() always issues the same loads -- an operand that comes from a register slot is fetched from the
// GEMV's own output buffer instead and ignored -- so that every wait on the rows and weights knows how
// many younger loads are outstanding.
// EPI = false: nothing rides behind the GEMV, and the stage reads no table, fetches nothing and stores what it is given.
// ANY: two columns a lane where one would do (k_gemm_tile's smallest tile): a straight tail in any layout, as one column has it.
template <int NE, bool EPI, bool ANY = false>
struct MmEpilogue {
    static constexpr int P = kEpiMaxPhases;
    bf16_t* y;
    int rows, n;
    unsigned head;
    int n_epi;
    const void PG_CONSTANT* ka;   // the kernel-argument segment (a GemvEpiArgs)
    float eps = 0.f;              // the prologue's, read with the table
    const bf16_t* q0[P];          // operand addresses, pointer-table slots resolved
    const bf16_t* q1[P];
    bf16_t* outs[P];
    unsigned ms[P], metas[P], inds[P];
    // NE even: four (two) columns at a time are aligned 8-byte (4-byte) words of every operand and output
    static constexpr int VW = NE % 4 == 0 ? 4 : 2;
    bool vec = false;
    // per call
    unsigned idx[NE];
    bool ok[NE];
    unsigned ld0[P][NE], ld1[P][NE];
    float v[NE];
    __device__ __forceinline__ void prepare() {
        if constexpr (!EPI) {
            if constexpr (NE % 2 == 0) vec = n % VW == 0 && aligned_to(y, 2 * VW);
            return;
        }
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
        if (head & kEpiAnySlot) {            // some operand is a pointer-table slot: all in one batch, without branches
            auto slot_addr = [&](const void* q, unsigned is_slot) -> SlotPtr { return is_slot ? (SlotPtr)(uintptr_t)q : (SlotPtr)ka; };
            SlotPtr at0[P], at1[P];
            const void* t0[P];
            const void* t1[P];
#pragma unroll
            for (int i = 0; i < P; i++) { at0[i] = slot_addr(a0[i], inds[i] & 1u); at1[i] = slot_addr(a1[i], inds[i] & 2u); }
#pragma unroll
            for (int i = 0; i < P; i++) { t0[i] = *at0[i]; t1[i] = *at1[i]; }
            asm volatile("" : "+s"(t0[0]), "+s"(t1[0]), "+s"(t0[1]), "+s"(t1[1]), "+s"(t0[2]), "+s"(t1[2]));
#pragma unroll
            for (int i = 0; i < P; i++) {
                if (inds[i] & 1u) a0[i] = t0[i];
                if (inds[i] & 2u) a1[i] = t1[i];
            }
        }
        uintptr_t low = (uintptr_t)y;
#pragma unroll
        for (int i = 0; i < P; i++) {
            q0[i] = static_cast<const bf16_t*>(a0[i]);
            q1[i] = static_cast<const bf16_t*>(a1[i]);
            if (i < n_epi) low |= (uintptr_t)q0[i] | (uintptr_t)q1[i] | (uintptr_t)outs[i];
        }
        if constexpr (NE % 2 == 0) vec = (head & kEpiPlain) && n % VW == 0 && (low & (2u * VW - 1)) == 0;
    }
    __device__ __forceinline__ void index(int r, int j, bool col_ok) {
#pragma unroll
        for (int e = 0; e < NE; e++) {
            ok[e] = col_ok && r < rows && j + e < n;
            idx[e] = ok[e] ? (unsigned)r * (unsigned)n + (unsigned)(j + e) : 0u;
        }
    }
    // the decoder block's tail with a layout that lets it be played straight through
    __device__ __forceinline__ bool straight() const { return (head & kEpiDecoder) && (NE == 1 || ANY ? (head & kEpiPlain) != 0 : vec); }
    // what any other tail reads
    __device__ __forceinline__ void fetch_any() {
        if (head & kEpiPlain) {                // one branch for all: no division where no operand has a period
#pragma unroll
            for (int i = 0; i < P; i++)
#pragma unroll
                for (int e = 0; e < NE; e++) {
                    ld0[i][e] = load_raw_global_at(q0[i], idx[e]);
                    ld1[i][e] = load_raw_global_at(q1[i], idx[e]);
                }
        } else {
#pragma unroll
            for (int i = 0; i < P; i++) {
                const unsigned m = ms[i];
#pragma unroll
                for (int e = 0; e < NE; e++) {
                    ld0[i][e] = load_raw_global_at(q0[i], idx[e]);
                    ld1[i][e] = load_raw_global_at(q1[i], idx[e] % m);
                }
            }
        }
    }
    __device__ __forceinline__ void begin(int r, int j, bool col_ok) {
        index(r, j, col_ok);
        if constexpr (!EPI) return;
        static_assert(!EPI || NE == 1, "several columns a lane: early and late");
        if (__builtin_expect((head & kEpiDecoder) && (head & kEpiPlain), 1)) {             // two operands, in in1 (see kernels.h)
            ld1[1][0] = load_raw_global_at(q1[1], idx[0]);
            ld1[2][0] = load_raw_global_at(q1[2], idx[0]);
        } else {
            fetch_any();
        }
    }
    // NE even, beside loads that go to LDS directly: while such loads are outstanding the compiler waits for all of them wherever it
    // meets a register that some load may write, on any path.  So the straight tail's operands go to LDS directly as well, a word of two columns per
    // lane and piece (ANY: or a word for each column, where n is odd or an operand lies at an odd element; kTailBytes of LDS per wave), and other tails
    // fetch theirs when the sums are there.
    static constexpr int kWords = ANY ? NE : NE / 2, kTailBytes = 2 * (kWords ? kWords : 1) * 256;
    static __device__ __forceinline__ int word_at(int i, int e) { return ((i - 1) * kWords + (ANY ? e : e / 2)) * 256; }
    template <bool PAIR>
    __device__ __forceinline__ void operand_to_lds(int i, int e, char* to /* uniform */) {
        const void PG_GLOBAL* const at = (const void PG_GLOBAL*)((const unsigned short PG_GLOBAL*)(uintptr_t)q1[i] + idx[e]);
        auto* const lds = (__attribute__((address_space(3))) void*)to;
        if constexpr (PAIR) __builtin_amdgcn_global_load_lds(at, lds, 4, 0, 0);
        else __builtin_amdgcn_global_load_lds(at, lds, 2, 0, 0);
    }
    __device__ __forceinline__ void early(int r, int j, bool col_ok, char* to /* uniform */) {
        index(r, j, col_ok);
        if (!straight()) return;
        if (__builtin_expect(!ANY || vec, 1)) {
#pragma unroll
            for (int i = 1; i < P; i++)
#pragma unroll
                for (int e = 0; e < NE; e += 2) operand_to_lds<true>(i, e, to + word_at(i, e));
        } else {
#pragma unroll
            for (int i = 1; i < P; i++)
#pragma unroll
                for (int e = 0; e < NE; e++) operand_to_lds<false>(i, e, to + word_at(i, e));
        }
    }
    // Beside loads into registers only: two columns' words stay as they come in until late_words(); taking them apart at once would wait for them and
    // for every load before them.  Other tails fetch theirs late here too, so that every wait on the rows and weights knows what is outstanding.
    __device__ __forceinline__ void early_words(int r, int j, bool col_ok) {
        index(r, j, col_ok);
        if (__builtin_expect(straight(), 1))
#pragma unroll
            for (int i = 1; i < P; i++) {
                if constexpr (NE == 1) ld1[i][0] = load_raw_global_at(q1[i], idx[0]);
                else
#pragma unroll
                    for (int e = 0; e < NE; e += 2) ld1[i][e / 2] = *(const unsigned PG_GLOBAL*)((const unsigned short PG_GLOBAL*)(uintptr_t)q1[i] + idx[e]);
            }
    }
    __device__ __forceinline__ void late_words() {
        if (__builtin_expect(straight(), 1)) {
            if constexpr (NE > 1)
#pragma unroll
                for (int i = 1; i < P; i++)
#pragma unroll
                    for (int e = NE - 2; e >= 0; e -= 2) {
                        const unsigned t = ld1[i][e / 2];
                        ld1[i][e] = t & 0xffffu; ld1[i][e + 1] = t >> 16;
                    }
        } else {
            fetch_any();
        }
    }
    __device__ __forceinline__ void late(const char* from, int lane) {
        if (__builtin_expect(straight(), 1)) {
            __builtin_amdgcn_s_waitcnt(0x0F70);            // vmcnt(0)
            auto word = [&](int i, int e) { return reinterpret_cast<const unsigned*>(from + word_at(i, e))[lane]; };
            if (__builtin_expect(!ANY || vec, 1)) {
#pragma unroll
                for (int i = 1; i < P; i++)
#pragma unroll
                    for (int e = 0; e < NE; e += 2) { const unsigned t = word(i, e); ld1[i][e] = t & 0xffffu; ld1[i][e + 1] = t >> 16; }
            } else {
#pragma unroll
                for (int i = 1; i < P; i++)
#pragma unroll
                    for (int e = 0; e < NE; e++) ld1[i][e] = word(i, e);      // zero-extended by the load
            }
        } else {
            fetch_any();
        }
    }
    __device__ __forceinline__ void store(bf16_t* o, const unsigned* b) {
        if constexpr (NE % 2 == 0) {
            if (__builtin_expect(vec, 1)) {
#pragma unroll
                for (int e = 0; e < NE; e += VW) {
                    unsigned short PG_GLOBAL* at = (unsigned short PG_GLOBAL*)(uintptr_t)o + idx[e];
                    if constexpr (VW == 4) { if (ok[e]) *(v2u PG_GLOBAL*)at = v2u{b[e] | (b[e + 1] << 16), b[e + 2] | (b[e + 3] << 16)}; }
                    else { if (ok[e]) *(unsigned PG_GLOBAL*)at = b[e] | (b[e + 1] << 16); }
                }
                return;
            }
        }
#pragma unroll
        for (int e = 0; e < NE; e++)
            if (ok[e]) *(unsigned short PG_GLOBAL*)(uintptr_t)(o + idx[e]) = (unsigned short)b[e];
    }
    __device__ __forceinline__ void put(int e, float sum) { v[e] = sum; }
    __device__ __forceinline__ void end() {
        unsigned bits[NE];
        if constexpr (!EPI) {
#pragma unroll
            for (int e = 0; e < NE; e++) bits[e] = f32_to_bf16(v[e]);
            store(y, bits);
            return;
        }
        float slot[kMergeSlots][NE];
        // Claim every operand before the first store: loads and stores complete in one queue, in order, so a wait for
        // an operand placed after a store would wait for that store to be acknowledged as well.
        __builtin_amdgcn_s_waitcnt(0x0F70);      // vmcnt(0)
#pragma unroll
        for (int e = 0; e < NE; e++) bits[e] = f32_to_bf16(v[e]);
        if (head & kEpiHeadStore) store(y, bits);
        if (__builtin_expect(straight(), 1)) {
            // the same kernels with the same arithmetic and roundings, operands known: GELU of the GEMV's rounded result,
            // then each add takes the value before it and its operand from memory, in the order its descriptor names
#pragma unroll
            for (int e = 0; e < NE; e++) bits[e] = f32_to_bf16(ew_apply<kGelu, false>(from_raw<bf16_t>(bits[e]), 0.f));
            if (inds[0] & kEpiStore) store(outs[0], bits);
#pragma unroll
            for (int i = 1; i < P; i++) {
                if (i >= n_epi) break;
                const bool mem_first = inds[i] & kEpiMemFirst;
#pragma unroll
                for (int e = 0; e < NE; e++) {
                    const float val = from_raw<bf16_t>(bits[e]), mem = from_raw<bf16_t>(ld1[i][e]);
                    bits[e] = f32_to_bf16(ew_apply<kAdd, false>(mem_first ? mem : val, mem_first ? val : mem));
                }
                if (inds[i] & kEpiStore) store(outs[i], bits);
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
            const unsigned op = mt & 0xffu, dst = mt >> 24;
            // (a tail whose memory operand the host moved to in1 but whose layout keeps it off the straight path above)
            const bool moved = (head & kEpiDecoder) && (ind & kEpiMemFirst);
            const unsigned src0 = (mt >> 8) & 0xffu, src1 = (mt >> 16) & 0xffu;
            float fa[NE], fb[NE], fo[NE];
#pragma unroll
            for (int e = 0; e < NE; e++) {
                fa[e] = from_raw<bf16_t>(moved ? ld1[i][e] : ld0[i][e]);
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
#pragma unroll
                for (int q = 0; q < kMergeSlots; q++)
                    if (dst == (unsigned)q) slot[q][e] = from_raw<bf16_t>(bits[e]);
            }
            if (ind & kEpiStore) store(outs[i], bits);
        }
    }
};

// A matrix-core result may not be read by an LDS write until the instruction has drained (up to
// 19 wait states for the longest forms).  The compiler inserts those itself inside a block, but
// it was seen to omit them when the last multiply of a K loop and this write sit in different
// blocks (loop exit): the write then stored a stale accumulator.  32 idle cycles, tied to `acc`
// so that they stay between the two, make it independent of that.
__device__ __forceinline__ void mm_drained(f32x4& acc) { asm volatile("s_nop 15\n\ts_nop 15" : "+v"(acc)); }

__device__ __forceinline__ void mm_drained(f32x4& a, f32x4& b) { asm volatile("s_nop 15\n\ts_nop 15" : "+v"(a), "+v"(b)); }

// What rides in a GEMV's dispatch: nothing, elementwise kernels behind it, or those and the RMSNorm in front.
enum Ride { kAlone, kEpilogue, kPrologue };

// What the two families read first: the first 64 bytes of the arguments hold everything that is needed before the
// loads of h and the weights can go out, and only those are waited for here, in one batch of scalar loads; the
// epilogue's table and eps are read once the weights are on their way (MmEpilogue::prepare).  PRO: h is computed from x and
// the gain; p.g.h is where the normalised rows are stored.
struct MmHead {
    const bf16_t* W;
    const bf16_t* h;          // PRO: x
    const bf16_t* gain;
    bf16_t* hstore;           // PRO: where the normalised rows go, or null
    bf16_t* y;
    int rows, n, cols, row_groups, n_epi;
    unsigned head;
    const void PG_CONSTANT* ka;
};
template <Ride RIDE> using RideArgs = std::conditional_t<RIDE == kAlone, GemvAloneArgs, GemvEpiArgs>;
template <Ride RIDE>
__device__ __forceinline__ MmHead mm_head(const RideArgs<RIDE>& p) {
    constexpr bool PRO = RIDE == kPrologue;
    static_assert(offsetof(GemvAloneArgs, head) == offsetof(GemvEpiArgs, head) && offsetof(GemvEpiArgs, gain) + sizeof(void*) == 64, "what the kernel needs first sits in the first 64 bytes");
    const void* Wa = p.g.W;
    const void* ha = p.g.h;
    bf16_t* y = static_cast<bf16_t*>(p.g.out);
    int rows = p.g.rows, n = p.g.n, cols = p.g.cols, row_groups = p.g.row_groups;
    unsigned head = p.head;
    int n_epi = 0;
    const void* xa = nullptr;
    const void* ga = nullptr;
    if constexpr (RIDE == kAlone) {
        asm volatile("" : "+s"(Wa), "+s"(ha), "+s"(y), "+s"(rows), "+s"(n), "+s"(cols), "+s"(row_groups), "+s"(head));
    } else {
        n_epi = p.n_epi;
        xa = p.x;
        ga = p.gain;
        asm volatile("" : "+s"(Wa), "+s"(ha), "+s"(y), "+s"(rows), "+s"(n), "+s"(cols), "+s"(row_groups), "+s"(head), "+s"(n_epi), "+s"(xa), "+s"(ga));
    }
    const void PG_CONSTANT* const ka = (const void PG_CONSTANT*)__builtin_amdgcn_kernarg_segment_ptr();   // a readable address for a load whose result is not used
    using SlotPtr = const void* const PG_CONSTANT*;
    auto slot_addr = [&](const void* q, bool is_slot) -> SlotPtr { return is_slot ? (SlotPtr)(uintptr_t)q : (SlotPtr)ka; };
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
    MmHead m;
    m.W = static_cast<const bf16_t*>(Wa);
    m.h = static_cast<const bf16_t*>(PRO ? xa : ha);
    m.gain = PRO ? static_cast<const bf16_t*>(ga) : nullptr;
    m.hstore = (PRO && (head & kEpiStoreH)) ? static_cast<bf16_t*>(const_cast<void*>(ha)) : nullptr;
    m.y = y; m.rows = rows; m.n = n; m.cols = cols; m.row_groups = row_groups; m.n_epi = n_epi; m.head = head; m.ka = ka;
    return m;
}

// ---- k_gemm_rows ------------------------------------------------------------------------------------------
// One tile of NR (4, 8 or 16) rows of h and NC (8 or 16) output columns per workgroup, rows of up to 128 * KS columns
// (KS K-steps per wave).  Few rows are bound by the latency of one dispatch, by the stream of weights (loads alone of 96 KB per workgroup take
// 3.4 us of the 5.6 that 16 rows of 2048 columns take), and with the RMSNorm in front by its instructions, four cycles each:
//   - 8 columns per workgroup make 2048 columns 256 workgroups, so that every CU pulls weights; half of each multiply
//     is idle, which costs nothing here.  Rows to normalise are cut into tiles so that the grid just fills the chip (prologue_tile): every
//     workgroup normalises its tile anew;
//   - a fragment read straight from global memory would touch 16 rows x 64 bytes per instruction, at 2048 columns all 4 KB
//     apart: half cache lines, one cache channel (measured: 0.3 - 1.1 us slower per launch).  Instead each wave loads
//     its own K-slices of the rows, contiguous bytes of one row (KS = 16) or two (KS = 8) per instruction, and transposes them through its
//     private slice of LDS into fragment order: slot (lane of the load) holds 16 rows x 16 bytes, padded to 272 bytes so
//     that 16 consecutive lanes hit all banks;
//   - the rows of h (from L2) are asked for before the weights (from HBM): loads return in order, so h is normalised
//     and staged while the weights are still on their way; then the same LDS slice takes the weights.
//   - the weights come by non-temporal loads, although the tiles of rows, up to eight, all read them.  us per sub-block of decode chains by plain / non-temporal
//     loads, in brackets the megabytes of weights: one tile of rows, 8 of 2048 columns [126] 5.34 / 4.70, [400] 5.07 / 4.30; two, 32 of 2048 6.77 / 6.46, 6.51 / 6.09;
//     four, 16 of 1024 3.51 / 3.12, 3.58 / 3.07, 32 of 1024 [40] 4.15 / 3.77; eight, 32 of 512 [105] 3.02 / 2.68.  Behind only where rows of more than 1024
//     columns share cache lines, and not always: 16 of 1928 [126] 6.15 / 6.35, [400] 5.76 / 6.05, 8 of 2041 6.63 / 6.34, 6.34 / 5.96.
// TAIL: the row does not have exactly 128 * KS columns; vectors at any element boundary.
// Decode chains of 120 sub-blocks, us per iteration: 32 rows of 1024 columns 1406 -> 613 (one dispatch per sub-block, where only
// 2048 columns had that; half the K-steps); 8 / 16 / 32 rows of 2048 columns 651 / 787 / 915 -> 627 / 771 / 862 (the epilogue's
// table worked out on the host, two operand loads instead of six, workgroups in XCD order).  Tiles of rows, one barrier in the RMSNorm, row
// addresses in scalar registers, us per sub-block before / after: 16 rows of 1024 columns 4.06 / 3.33, 32 4.36 / 3.67, 8 3.48 / 3.18, 16 of 520
// 4.42 / 3.67, 16 of 2048 5.81 / 5.39, 32 6.64 / 6.46.  Eight waves of half the columns each: no faster, the instructions count (16 of 2048 5.63
// where four waves took 5.58, 32 of 1024 4.00 where they took 3.83).
constexpr int kMmSlotBytes = 272;   // 16 rows x 16 B + 16 B of padding

// k offset of the 16-byte chunk that lane `l` (of 4 * KS) of wave `wave` loads from a row; the same chunk is fragment
// step l >> 2, k-chunk l & 3 of that wave.
__device__ __forceinline__ int mm_k0(int wave, int l) { return ((l >> 3) * 8 + wave * 2 + ((l >> 2) & 1)) * 32 + (l & 3) * 8; }

// NR rows of a row-major matrix from row r0 (inside it), this wave's K-slices; rows beyond the matrix repeat its last row.  (Everything in front of
// the last weight load delays the whole kernel, and so does a branch about loads, behind which the compiler waits for more of them than it has to.)
template <int KS, bool TAIL, int NR, bool NT>
__device__ __forceinline__ void mm_load_rows(const bf16_t* m, int rows, int cols, int r0, int wave, int lane, unsigned (*g)[4]) {
    constexpr int L = 4 * KS, RPI = 64 / L;             // lanes per row, rows per instruction
    const int sub = lane / L;
    const unsigned koff = span_at<!TAIL>(cols, mm_k0(wave, lane % L) >> 3);
    const bf16_t* row = m + (size_t)r0 * cols;
    const unsigned last = (unsigned)(rows - 1 - r0);
#pragma unroll
    for (int q = 0; q < NR / RPI; q++) {
        if constexpr (RPI == 1) {
            const bf16_t* at = row + (size_t)((unsigned)q < last ? (unsigned)q : last) * (unsigned)cols;
            asm("" : "+s"(at));                          // stays a scalar address
            load_at<NT>(at, koff * 2u, g[q]);
        } else {
            const unsigned R = (unsigned)(q * RPI + sub) < last ? (unsigned)(q * RPI + sub) : last;
            load_at<NT>(row, (R * (unsigned)cols + koff) * 2u, g[q]);
        }
    }
}
template <int KS, bool TAIL, int NR>
__device__ __forceinline__ void mm_fix_rows(int cols, int wave, int lane, unsigned (*g)[4]) {
    if constexpr (TAIL) {
        // (as span_fix, but a lane's vectors lie in the same place of every row: decided once for all of them.  Decided vector by vector, with a
        // shift by a lane's own count, 16 rows of 1536 columns took 8.8 us a dispatch where 2048 columns took 5.8; now 7.1.)
        const int over = mm_k0(wave, lane % (4 * KS)) + 8 - cols;
        if (const unsigned s = 8u - ((unsigned)cols & 7u); s != 8u)
            if (over == (int)s)
#pragma unroll
                for (int q = 0; q < NR * KS / 16; q++) span_shift(s, g[q]);
#pragma unroll
        for (int q = 0; q < NR * KS / 16; q++)
#pragma unroll
            for (int i = 0; i < 4; i++) g[q][i] = over >= 8 ? 0u : g[q][i];
    }
}

// LDS operations of one wave execute in order: these writes cannot overtake the reads before them
template <int KS, int NR>
__device__ __forceinline__ void mm_stage(char* lds /* this wave's */, int lane, const unsigned (*g)[4]) {
    constexpr int L = 4 * KS, RPI = 64 / L;
#pragma unroll
    for (int q = 0; q < NR / RPI; q++)
        *reinterpret_cast<v4u*>(lds + (lane % L) * kMmSlotBytes + (q * RPI + lane / L) * 16) = v4u{g[q][0], g[q][1], g[q][2], g[q][3]};
}
// fragment (step i, k-chunk lane >> 4, row or column lane & 15) of what is staged in `lds`
template <int KS>
__device__ __forceinline__ void mm_read_frags(const char* lds, int lane, v4u* f) {
#pragma unroll
    for (int i = 0; i < KS; i++)
        f[i] = *reinterpret_cast<const v4u*>(lds + (i * 4 + (lane >> 4)) * kMmSlotBytes + (lane & 15) * 16);
}

// RMSNorm of the rows just loaded.  A lane holds 16-byte chunk c of some of the rows, eight neighbouring lanes the eight chunks of
// a K-block.  The stand-alone kernel's sums must be reproduced bit for bit: per chunk the fused sum of squares in element order
// (any lane can do that); then the stand-alone kernel's reduction, which is a tree of fixed shape over the chunk sums in chunk order
// (absent chunks are zeros) -- wave_sum adds neighbours, then pairs of pairs, of quads, of eights (a floating-point add does not
// care which operand is which), then the four sixteens in order, and the four wave sums in order.  Here eight lanes add up a
// K-block's chunks, the sums of the blocks go to LDS, and behind the one barrier every wave finishes all rows by itself: lane 4 r + w wave
// sum w of row r, its quad the row's scale, which the lanes that hold the row fetch from it; every lane scales its own chunks: (x * scale) *
// gain, one rounding.  `sq`: NR * (2 * KS + 4) floats.  hstore: this workgroup also stores the rows.
template <int KS, bool TAIL, int NR>
__device__ __forceinline__ void mm_rmsnorm_rows(unsigned (*g)[4], const unsigned* wg /* the lane's chunk of the gain */, float eps, bf16_t* hstore,
                                                int rows, int cols, int wave, int lane, float* sq) {
    constexpr int L = 4 * KS, RPI = 64 / L, Q = NR / RPI;
    constexpr int NB = 2 * KS, WS = NB / 8, kRow = NB + 4;      // K-blocks and wave sums of a row; a row of `sq`, padded
    static_assert(NB % 8 == 0 && NR <= 16, "eight blocks to a wave sum, a quad per row");
    const int sub = lane / L;
    const int k0 = mm_k0(wave, lane % L);
    float fx[Q][8];
#pragma unroll
    for (int q = 0; q < Q; q++) {
        Vec<bf16_t, 16>::unpack(g[q], fx[q]);
        float acc = 0.f;
#pragma unroll
        for (int e = 0; e < 8; e++) acc = __builtin_fmaf(fx[q][e], fx[q][e], acc);
        acc = dpp_add<0xB1>(acc);
        acc = dpp_add<0x4E>(acc);
        acc = dpp_add<0x141>(acc);
        sq[(q * RPI + sub) * kRow + (k0 >> 6)] = acc;            // the same bits from all eight lanes: no branch per row
    }
    lds_barrier();
    float scale;
    {
        const int r = (lane >> 2) < NR ? lane >> 2 : NR - 1, w = (lane & 3) < WS ? lane & 3 : 0;
        const f32x4* b = reinterpret_cast<const f32x4*>(sq + r * kRow + w * 8);
        const f32x4 b0 = b[0], b1 = b[1];
        const float wsum = (((b0.x + b0.y) + (b0.z + b0.w)) + (b1.x + b1.y)) + (b1.z + b1.w);
        float total = dpp_take<0x00>(wsum);                                // quad_perm: lane 0 of the quad in all four ...
        if constexpr (WS > 1) total += dpp_take<0x55>(wsum);               // ... lane 1, 2, 3
        if constexpr (WS > 2) { total += dpp_take<0xAA>(wsum); total += dpp_take<0xFF>(wsum); }
        scale = 1.0f / sqrtf(total / (float)cols + eps);
    }
    float fg[8];
    Vec<bf16_t, 16>::unpack(wg, fg);
#pragma unroll
    for (int q = 0; q < Q; q++) {
        float fo[8];
        const float sc = RPI == 1 ? __int_as_float(__builtin_amdgcn_readlane(__float_as_int(scale), q * 4))
                                  : __int_as_float(__builtin_amdgcn_ds_bpermute((q * RPI + sub) * 16, __float_as_int(scale)));
#pragma unroll
        for (int e = 0; e < 8; e++) fo[e] = (fx[q][e] * sc) * fg[e];
        Vec<bf16_t, 16>::pack(fo, g[q]);
    }
    if (hstore) {
#pragma unroll
        for (int q = 0; q < Q; q++) {
            const int r = q * RPI + sub;
            if (r < rows) {
                if constexpr (TAIL) span_store(hstore + (size_t)r * cols, cols, k0 >> 3, g[q]);
                else store_vec_global(hstore + (size_t)r * cols + k0, g[q]);
            }
        }
    }
}

// The grid is (column blocks) x (tiles of rows), the tiles of one column block next to each other, so that they share an XCD's
// L2.  The workgroups of column block 0 store the normalised rows.
template <int KS, bool TAIL, int NR, int NC, Ride RIDE>
__global__ __launch_bounds__(kBlock, (RIDE == kPrologue && KS > 8) ? 1 : 2) void k_gemm_rows(RideArgs<RIDE> p) {
    constexpr bool PRO = RIDE == kPrologue;
    const MmHead m = mm_head<RIDE>(p);
    constexpr int kWaveLds = 4 * KS * kMmSlotBytes;
    __shared__ __attribute__((aligned(16))) char stage[4 * kWaveLds];
    __shared__ float red[4 * 4 * 64];
    __shared__ __attribute__((aligned(16))) float sq[PRO ? NR * (2 * KS + 4) : 4];
    MmEpilogue<1, RIDE != kAlone> emit;
    emit.y = m.y; emit.rows = m.rows; emit.n = m.n; emit.head = m.head; emit.n_epi = m.n_epi; emit.ka = m.ka;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned ncb = (unsigned)(m.n + NC - 1) / NC;
    // (without the RMSNorm one tile holds all rows; read from the arguments instead: 8 rows of 2048 columns alone 3.97 where this takes 3.93, 16 of 777 with a tail 3.45 / 3.39)
    const unsigned ntiles = PRO ? (unsigned)m.row_groups & 0xffu : 1u, inv = (unsigned)m.row_groups >> 8;      // 65536 / ntiles (plan_gemm)
    // one tile of rows and a grid of several rounds: columns dealt out in turn stream better (us per launch, 5 rows of 2048 columns, 16384
    // outputs 17.6 -> 15.9, 1024 columns, 32768 outputs 16.2 -> 13.9); otherwise a stretch per XCD (below 1024 workgroups 0.1 - 0.3 us
    // faster at every size, and tiles of rows share their columns)
    const unsigned at = ntiles == 1 && ncb > 1024 ? blockIdx.x : xcd_stretch(blockIdx.x, ncb * ntiles);
    const int cb = (int)(ntiles == 1 ? at : (at * inv) >> 16), tile = (int)(at - (unsigned)cb * ntiles);
    const int cols = TAIL ? m.cols : 128 * KS;
    const int j0 = cb * NC, r0 = tile * NR;
    if (r0 >= m.rows) return;                            // whole workgroup: nothing waits on it
    char* lds = stage + wave * kWaveLds;
    unsigned g[NR * KS / 16][4], gw[NC * KS / 16][4];
    v4u a[KS], b[KS];
    mm_load_rows<KS, TAIL, NR, false>(m.h, m.rows, cols, r0, wave, lane, g);      // PRO: the rows to normalise
    unsigned wg[4] = {0u, 0u, 0u, 0u};
    if constexpr (PRO) load_any<false>(m.gain, span_at<!TAIL>(cols, mm_k0(wave, lane % (4 * KS)) >> 3), wg);   // before the weights: loads come back in order
    __builtin_amdgcn_sched_barrier(0);
    mm_load_rows<KS, TAIL, NC, true>(m.W, m.n, cols, j0, wave, lane, gw);
    emit.prepare();                                      // the epilogue's table right behind the weight loads
    // output stage: wave w finishes row w of the four that an accumulator lane holds
    auto emit_begin = [&] { emit.begin(r0 + (lane >> 4) * 4 + wave, j0 + (lane & 15), (lane & 15) < NC && (lane >> 4) * 4 < NR); };
    if constexpr (NC == 8 || NR < 16) emit_begin();
    mm_fix_rows<KS, TAIL, NR>(cols, wave, lane, g);
    if constexpr (PRO) {
        span_fix<!TAIL>(cols, mm_k0(wave, lane % (4 * KS)) >> 3, wg);
        bf16_t* hs = (m.hstore && cb == 0) ? m.hstore + (size_t)r0 * cols : nullptr;
        mm_rmsnorm_rows<KS, TAIL, NR>(g, wg, emit.eps, hs, m.rows - r0, cols, wave, lane, sq);
    }
    mm_stage<KS, NR>(lds, lane, g);
    mm_read_frags<KS>(lds, lane, a);
    mm_fix_rows<KS, TAIL, NC>(cols, wave, lane, gw);
    mm_stage<KS, NC>(lds, lane, gw);
    mm_read_frags<KS>(lds, lane, b);
    __builtin_amdgcn_sched_barrier(0);   // all fragment reads before the first multiply, not one LDS latency per pair
    if constexpr (NC != 8 && NR == 16) emit_begin();
    f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};         // the wave's two eighths of K, whose blocks take turns
#pragma unroll
    for (int i = 0; i < KS; i++)
        acc[i / 2 % 2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[i]), __builtin_bit_cast(bf16x8, b[i]), acc[i / 2 % 2], 0, 0, 0);
    mm_drained(acc[0], acc[1]);
    const f32x4 both = acc[0] + acc[1];
    float* dst = red + ((size_t)wave * 64 + lane) * 4;
    dst[0] = both.x; dst[1] = both.y; dst[2] = both.z; dst[3] = both.w;
    __syncthreads();
    const float p0 = red[((size_t)0 * 64 + lane) * 4 + wave], p1 = red[((size_t)1 * 64 + lane) * 4 + wave];
    const float p2 = red[((size_t)2 * 64 + lane) * 4 + wave], p3 = red[((size_t)3 * 64 + lane) * 4 + wave];
    emit.put(0, ((p0 + p1) + p2) + p3);
    emit.end();
}

// ---- k_gemm_cols ------------------------------------------------------------------------------------------
// The same staging for more rows: 16 output columns per workgroup, whose weight fragments stay in registers while its
// tiles of 16 rows of h pass by, the next tile's rows in flight across the multiplies of this one.  Two workgroups per CU.
// WNT, here and in k_gemm_tile: the weights by non-temporal loads (plan_gemm).
template <int KS, bool TAIL, bool WNT, Ride RIDE>
__global__ __launch_bounds__(kBlock, 2) void k_gemm_cols(RideArgs<RIDE> p) {
    const MmHead m = mm_head<RIDE>(p);
    constexpr int kWaveLds = 4 * KS * kMmSlotBytes, kRedRow = 20;
    __shared__ __attribute__((aligned(16))) char stage[4 * kWaveLds];
    __shared__ float red[4][16 * kRedRow];
    MmEpilogue<1, RIDE != kAlone> emit;
    emit.y = m.y; emit.rows = m.rows; emit.n = m.n; emit.head = m.head; emit.n_epi = m.n_epi; emit.ka = m.ka;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ncb = (m.n + 15) / 16;
    const int at = (int)xcd_stretch(blockIdx.x, (unsigned)(ncb * m.row_groups)), cb = at / m.row_groups;
    // Five tiles make row groups of two, two, one and none: the workgroups that follow each other onto a CU (32 later in an
    // XCD's stretch) are not to be of the same group, or some CUs work out four tiles and some none (80 rows of 2048 columns
    // 8.1 -> 7.2 us per launch)
    const int rg = (at + cb * m.row_groups / 32 * 2) % m.row_groups;
    const int ntiles = (m.rows + 15) / 16, per = (ntiles + m.row_groups - 1) / m.row_groups;
    const int t0 = rg * per, t1 = (t0 + per < ntiles) ? t0 + per : ntiles;
    if (t0 >= t1) return;                                // whole workgroup: nothing waits on it
    const int cols = TAIL ? m.cols : 128 * KS;
    const int j0 = cb * 16;
    char* lds = stage + wave * kWaveLds;
    unsigned g[KS][4], gw[KS][4];
    v4u a[KS], b[KS];
    mm_load_rows<KS, TAIL, 16, false>(m.h, m.rows, cols, t0 * 16, wave, lane, g);
    mm_load_rows<KS, TAIL, 16, WNT>(m.W, m.n, cols, j0, wave, lane, gw);
    emit.prepare();                                      // the epilogue's table right behind the weight loads
    mm_fix_rows<KS, TAIL, 16>(cols, wave, lane, g);
    mm_stage<KS, 16>(lds, lane, g);
    mm_read_frags<KS>(lds, lane, a);
    if (t1 - t0 > 1) mm_load_rows<KS, TAIL, 16, false>(m.h, m.rows, cols, (t0 + 1) * 16, wave, lane, g);
    mm_fix_rows<KS, TAIL, 16>(cols, wave, lane, gw);
    mm_stage<KS, 16>(lds, lane, gw);
    mm_read_frags<KS>(lds, lane, b);
    const int er = tid >> 4, ec = tid & 15;              // output stage: a lane finishes one column of one row
#pragma unroll 1
    for (int t = t0;;) {
        __builtin_amdgcn_sched_barrier(0);   // all fragment reads before the first multiply, not one LDS latency per pair
        emit.begin(t * 16 + er, j0 + ec, true);
        f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};     // the wave's two eighths of K, whose blocks take turns
#pragma unroll
        for (int i = 0; i < KS; i++)
            acc[i / 2 % 2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[i]), __builtin_bit_cast(bf16x8, b[i]), acc[i / 2 % 2], 0, 0, 0);
        mm_drained(acc[0], acc[1]);
        float* dst = red[wave] + (lane >> 4) * 4 * kRedRow + (lane & 15);
        dst[0] = acc[0].x + acc[1].x; dst[kRedRow] = acc[0].y + acc[1].y; dst[2 * kRedRow] = acc[0].z + acc[1].z; dst[3 * kRedRow] = acc[0].w + acc[1].w;
        lds_barrier();
        const int q = er * kRedRow + ec;
        emit.put(0, ((red[0][q] + red[1][q]) + red[2][q]) + red[3][q]);
        emit.end();
        if (++t >= t1) break;
        lds_barrier();                       // the sums are read: `red` is free again
        mm_fix_rows<KS, TAIL, 16>(cols, wave, lane, g);
        mm_stage<KS, 16>(lds, lane, g);
        if (t + 1 < t1) mm_load_rows<KS, TAIL, 16, false>(m.h, m.rows, cols, (t + 1) * 16, wave, lane, g);
        mm_read_frags<KS>(lds, lane, a);
    }
}

// ---- k_gemm_tile --------------------------------------------------------------------------------------------
// RT x CT tiles of 16 rows x 16 columns per workgroup, any number of columns of h and W.  Each wave streams its own
// K-blocks (64 columns of all the workgroup's rows of h and W, (RT + CT) * 2 KB) through a ring of S blocks in its own part
// of LDS, loaded from global memory into LDS directly: no registers are held by loads in flight (S blocks per wave, so
// latency is covered without a second workgroup), no wave waits for another until the partial sums meet.  A load
// instruction covers whole 128-byte lines of eight rows; lane l's line position is swapped with its row (chunk c of
// row r sits at c ^ (r & 7)), so that the fragment reads of eight consecutive lanes touch all banks once.
// What bounds it is what a CU takes in through its cache ((RT + CT) * 32 bytes * cols per RT * CT * 256 outputs), hence larger
// tiles where there are enough of them (plan_gemm); a CU holds no more than its 32 KB cache's worth of lines in flight.
// K is cut into blocks of 64 and dealt out to eight parts in turn.  Eight waves, one part
// each, so that one wave's fragment reads and multiplies hide behind another's (with four waves a round of one block
// cost them 0.3 us in turn); stand-alone launches keep workgroups of four waves (two parts a wave, whose blocks take turns
// in one stream): the same bits.
// The epilogue's operands come into LDS as well (MmEpilogue::early): as loads into registers they made the compiler wait for the first block, for
// each operand and for the second block in turn before the loop.  us per RMSNorm and GEMV without / with: 128 rows of 2048 columns 10.62 / 10.34, of 1024 7.42 /
// 7.00, 16 of 3072 10.44 / 10.15, 8 of 4096 12.09 / 11.61, 81 of 520 6.85 / 6.57; two workgroups of 16 x 16 to a CU hide such waits from each
// other, 20 of 2304 9.63 / 9.79, and keep the loads into registers.  So does the 16 x 16 tile where no 16-byte load reaches the rows (columns no multiple of 8): its
// rows and weights come through registers then, and beside those the operands' way over LDS gains little and costs up to 6 % (us per GEMV, GELU and two
// adds through LDS / registers: 33 rows of 2100 columns, 555 outputs 6.05 / 5.71, 6 of 2500, 2000 outputs 7.11 / 6.72, 24 of 2049, 2000 outputs 7.06 / 7.20).
// An odd number of outputs or an operand at an odd element, 16 rows of 3072 columns, 3001 outputs: 7.4, fetched when the sums are there 7.7, one column
// a lane with loads into registers 7.6; 8 of 4096, 33 outputs 4.7, 4.95, 4.7.
// Decode chains, us per iteration, before and after: 128 rows of 2048 columns, 120 sub-blocks 1529 -> 1330; 100 x 2000 (100
// sub-blocks) 1290 -> 850, 128 x 1024 1282 -> 793 (there also one dispatch instead of three around the GEMV); one GEMV alone, us
// per launch: 128 rows by 4096 x 4096 34.0 -> 17.4, by 2048 x 2048 8.1 -> 7.8 (the 16- and 32-column forms it replaces re-read W
// for every group of tiles).
// Rows that 16-byte loads cannot reach (cols no multiple of 8, a misaligned external) go through registers instead,
// one block ahead.
template <int N>
__device__ __forceinline__ void vm_wait() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
// 16 bytes per lane from global memory into LDS, lane l's at `to` + 16 l
template <bool NT>
__device__ __forceinline__ void load_to_lds(const bf16_t* base /* uniform */, unsigned elem, char* to /* uniform */) {
    __builtin_amdgcn_global_load_lds((const void PG_GLOBAL*)((const bf16_t PG_GLOBAL*)(uintptr_t)base + elem), (__attribute__((address_space(3))) void*)to, 16, 0, NT ? 2 : 0);
}
// The fragments of one K-block, both steps, of F tiles 2 KB apart: read and waited for in one piece (left to the compiler,
// reads of LDS that direct loads may be filling wait for all of those first)
template <int F>
__device__ __forceinline__ void ring_frags(unsigned at0, unsigned at1, v4u (&f)[2 * F]) {
    static_assert(F == 2 || F == 4 || F == 6, "tiles per block");
    if constexpr (F == 2)
        asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %4 offset:2048\n\tds_read_b128 %2, %5\n\tds_read_b128 %3, %5 offset:2048\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3]) : "v"(at0), "v"(at1) : "memory");
    else if constexpr (F == 4)
        asm volatile("ds_read_b128 %0, %8\n\tds_read_b128 %1, %8 offset:2048\n\tds_read_b128 %2, %8 offset:4096\n\tds_read_b128 %3, %8 offset:6144\n\t"
                     "ds_read_b128 %4, %9\n\tds_read_b128 %5, %9 offset:2048\n\tds_read_b128 %6, %9 offset:4096\n\tds_read_b128 %7, %9 offset:6144\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3]), "=&v"(f[4]), "=&v"(f[5]), "=&v"(f[6]), "=&v"(f[7])
                     : "v"(at0), "v"(at1) : "memory");
    else
        asm volatile("ds_read_b128 %0, %12\n\tds_read_b128 %1, %12 offset:2048\n\tds_read_b128 %2, %12 offset:4096\n\tds_read_b128 %3, %12 offset:6144\n\t"
                     "ds_read_b128 %4, %12 offset:8192\n\tds_read_b128 %5, %12 offset:10240\n\t"
                     "ds_read_b128 %6, %13\n\tds_read_b128 %7, %13 offset:2048\n\tds_read_b128 %8, %13 offset:4096\n\tds_read_b128 %9, %13 offset:6144\n\t"
                     "ds_read_b128 %10, %13 offset:8192\n\tds_read_b128 %11, %13 offset:10240\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3]), "=&v"(f[4]), "=&v"(f[5]), "=&v"(f[6]), "=&v"(f[7]), "=&v"(f[8]), "=&v"(f[9]),
                       "=&v"(f[10]), "=&v"(f[11])
                     : "v"(at0), "v"(at1) : "memory");
}

// ASIDE: the operands of a straight tail come into LDS beside the ring (MmEpilogue::early).
__device__ __forceinline__ int wave_index() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }
template <int RT, int CT, int S, int NW, bool WNT, bool ASIDE = true>
__global__ __launch_bounds__(NW * 64, RT * CT == 1 ? NW / 2 : NW / 4) void k_gemm_tile(RideArgs<NW == 8 ? kEpilogue : kAlone> p) {
    constexpr int F = RT + CT, NL = 2 * F, kBlockLds = F * 2048, kWaveLds = S * kBlockLds;
    constexpr int PK = 8 / NW;                           // eighths of K per wave
    constexpr int kRedRow = 16 * CT + 4;                 // floats of a row of partial sums, padded: rows 4 apart fall into other banks
    constexpr int kRed = 16 * RT * kRedRow;              // floats of one eighth's partial sums
    constexpr int kEach = RT * CT * 4 / NW, NE = kEach >= 2 ? kEach : NW == 8 && ASIDE ? 2 : 1, kPerRow = 16 * CT / NE;  // outputs per lane (consecutive columns), lanes per row of the tile
    static_assert(PK * kRed * 4 <= kWaveLds, "a wave's partial sums fit its ring");
    static_assert(S == 1 || S == 2, "the waits below name the blocks in flight");
    constexpr Ride RIDE = NW == 8 ? kEpilogue : kAlone;  // four waves: a stand-alone launch
    const MmHead m = mm_head<RIDE>(p);
    using Emit = MmEpilogue<NE, RIDE != kAlone, ASIDE && (kEach < NE)>;
    constexpr int kTails = RIDE != kAlone && ASIDE ? Emit::kTailBytes : 0;
    __shared__ __attribute__((aligned(128))) char ring[NW * (kWaveLds + kTails)];
    char* const tail = ring + NW * kWaveLds + wave_index() * kTails;
    Emit emit;
    emit.y = m.y; emit.rows = m.rows; emit.n = m.n; emit.head = m.head; emit.n_epi = m.n_epi; emit.ka = m.ka;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rows = m.rows, n = m.n, cols = m.cols;
    const int ncb = (n + 16 * CT - 1) / (16 * CT);
    const int at = (int)xcd_stretch(blockIdx.x, (unsigned)(ncb * m.row_groups)), cb = at / m.row_groups, rg = at % m.row_groups;
    const int r0 = rg * 16 * RT, j0 = cb * 16 * CT;
    const int nkb = (cols + 63) / 64;
    char* mine = ring + wave * kWaveLds;
    const int r8 = lane >> 3;                            // row within the eight of a load instruction
    const bool direct = cols % 8 == 0 && aligned_to(m.W, 16) && aligned_to(m.h, 16);
    const int chunk = direct ? (lane & 7) ^ r8 : lane & 7;             // 16-byte chunk of the K-block this lane loads
    const int rem = cols & 63;                           // columns of the last K-block, if it is a partial one
    // where a lane finds its fragments: row (or column) lane & 15 of a tile, chunk lane >> 4 of each step
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)mine;
    const unsigned f0 = lds0 + (lane & 15) * 128 + (((lane >> 4) ^ (lane & 7)) * 16), f1 = lds0 + (lane & 15) * 128 + (((4 + (lane >> 4)) ^ (lane & 7)) * 16);
    const bf16_t* wb = m.W + (size_t)j0 * cols;
    const int er = tid / kPerRow, ec = (tid % kPerRow) * NE;           // output stage: a lane finishes NE consecutive columns of one row
    const bf16_t* hb = m.h + (size_t)r0 * cols;
    unsigned row_at[NL];                             // element offset of the row each load instruction takes here
#pragma unroll
    for (int q = 0; q < NL; q++) {
        const int r = (q < 2 * RT ? q : q - 2 * RT) * 8 + r8, last = (q < 2 * RT ? rows - r0 : n - j0) - 1;
        row_at[q] = (unsigned)(r < last ? r : last) * (unsigned)cols;
    }
    f32x4 acc[PK][RT][CT];
#pragma unroll
    for (int pk = 0; pk < PK; pk++)
#pragma unroll
        for (int i = 0; i < RT; i++)
#pragma unroll
            for (int j = 0; j < CT; j++) acc[pk][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // the epilogue's table behind the first block's loads: asked for behind all of them it came 1.1 us later
    auto operands_begin = [&] {
        if constexpr (RIDE == kAlone) emit.index(r0 + er, j0 + ec, er < 16 * RT);
        else if constexpr (ASIDE) emit.early(r0 + er, j0 + ec, er < 16 * RT, tail);
        else emit.begin(r0 + er, j0 + ec, er < 16 * RT);
    };
    // this wave's K-blocks: wave, wave + NW, ...; number b of them belongs to its eighth b % PK
    const int nb = (nkb - wave + NW - 1) / NW;
    auto multiply = [&](f32x4 (&sum)[RT][CT], v4u (&f)[2 * F]) {
#pragma unroll
        for (int s = 0; s < 2; s++)
#pragma unroll
            for (int i = 0; i < RT; i++)
#pragma unroll
                for (int j = 0; j < CT; j++)
                    sum[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f[s * F + i]), __builtin_bit_cast(bf16x8, f[s * F + RT + j]), sum[i][j], 0, 0, 0);
    };
    if (__builtin_expect(direct, 1)) {
        auto issue = [&](int b, int slot) {
            const int k = (wave + NW * b) * 64 + chunk * 8;
            const unsigned ke = k < cols ? (unsigned)k : 0u;           // a chunk past the end is read from column 0 and zeroed later
            char* const to = mine + slot * kBlockLds;
#pragma unroll
            for (int q = 0; q < 2 * RT; q++) load_to_lds<false>(hb, row_at[q] + ke, to + q * 1024);
#pragma unroll
            for (int q = 2 * RT; q < NL; q++) load_to_lds<WNT>(wb, row_at[q] + ke, to + q * 1024);
        };
        if (nb > 0) issue(0, 0);
        emit.prepare();
        operands_begin();
        if (S == 2 && nb > 1) issue(1, 1);
        int slot = 0;
#pragma unroll 1
        for (int b0 = 0; b0 < nb; b0 += PK) {
#pragma unroll
            for (int pk = 0; pk < PK; pk++) {
                const int b = b0 + pk;
                if (PK > 1 && b >= nb) break;
                // loads complete in order: block b is in once at most the younger block's loads are outstanding (other loads
                // among them only make the wait stricter)
                if (S == 2 && b + 1 < nb) vm_wait<NL>();
                else vm_wait<0>();
                v4u f[2 * F];
                ring_frags<F>(f0 + slot * kBlockLds, f1 + slot * kBlockLds, f);
                if (b + S < nb) issue(b + S, slot);                    // the slot has been read
                if (rem && wave + NW * b == nkb - 1) {
#pragma unroll
                    for (int s = 0; s < 2; s++)
                        if ((s * 4 + (lane >> 4)) * 8 >= rem)
#pragma unroll
                            for (int i = 0; i < F; i++) f[s * F + i] = v4u{0u, 0u, 0u, 0u};
                }
                multiply(acc[pk], f);
                slot = slot + 1 == S ? 0 : slot + 1;
            }
        }
    } else {
        unsigned g[NL][4];
        auto fetch = [&](int b) {
            const unsigned ke = span_at<false>(cols, (wave + NW * b) * 8 + chunk);
#pragma unroll
            for (int q = 0; q < NL; q++) load_any<false>(q < 2 * RT ? hb : wb, row_at[q] + ke, g[q]);
        };
        if (nb > 0) fetch(0);
        emit.prepare();
        // operands on their way to LDS are waited for with the first block's rows and weights, which come into registers here: in the smallest tile
        // they follow the second block's
        constexpr bool kBehind = RIDE != kAlone && ASIDE && RT * CT == 1;
        if (!kBehind || nb == 0) operands_begin();
#pragma unroll 1
        for (int b0 = 0; b0 < nb; b0 += PK) {
#pragma unroll
            for (int pk = 0; pk < PK; pk++) {
                const int b = b0 + pk;
                if (PK > 1 && b >= nb) break;
#pragma unroll
                for (int q = 0; q < NL; q++) {
                    span_fix<false>(cols, (wave + NW * b) * 8 + chunk, g[q]);
                    *reinterpret_cast<v4u*>(mine + (q * 8 + r8) * 128 + ((chunk ^ r8) * 16)) = v4u{g[q][0], g[q][1], g[q][2], g[q][3]};
                }
                if (b + 1 < nb) fetch(b + 1);
                if (kBehind && b == 0) operands_begin();
                v4u f[2 * F];
                ring_frags<F>(f0, f1, f);                              // behind the writes above: one wave's LDS operations execute in order
                multiply(acc[pk], f);
            }
        }
    }
#pragma unroll
    for (int pk = 0; pk < PK; pk++)
#pragma unroll
        for (int i = 0; i < RT; i++)
#pragma unroll
            for (int j = 0; j < CT; j++) {
                mm_drained(acc[pk][i][j]);
                float* dst = reinterpret_cast<float*>(mine) + pk * kRed + (i * 16 + (lane >> 4) * 4) * kRedRow + j * 16 + (lane & 15);
                const f32x4 v = acc[pk][i][j];
                dst[0] = v.x; dst[kRedRow] = v.y; dst[2 * kRedRow] = v.z; dst[3 * kRedRow] = v.w;
            }
    if constexpr (RIDE != kAlone && ASIDE) emit.late(tail, lane);
    lds_barrier();
    if (er < 16 * RT) {
#pragma unroll
        for (int e = 0; e < NE; e++) {
            auto part = [&](int w) { return reinterpret_cast<const float*>(ring + (w % NW) * kWaveLds)[(w / NW) * kRed + er * kRedRow + ec + e]; };
            emit.put(e, parts_sum(part));
        }
        emit.end();
    }
}

// ---- k_gemm_whole --------------------------------------------------------------------------------------------
// k_gemm_tile's tiles for rows of up to 512 * KB columns where the grid is one workgroup per CU: eight waves, an eighth of K each (KB blocks of 64 columns),
// all of whose loads are asked for at once, into registers, vectors at any element boundary; block by block they pass through the wave's own part of
// LDS into fragment order (chunk c of row r at c ^ (r & 7), two buffers, so that a block is written while the one before is multiplied).
// What bounds it is what a CU takes in: 256 KB at 128 rows of 2048 columns, 5.0 us for the loads alone with their node (a row's lines in two loads of 64
// bytes, straight into fragment order, 9.4).  h first, then the weights: in alternation the loads alone take 5.9.
// Registers and not direct loads into LDS: behind those the compiler waits for everything outstanding wherever it needs a register that was loaded.
// us per RMSNorm and GEMV, k_gemm_cols or k_gemm_tile / this: 64 rows of 2048 columns 9.33 / 8.43, 80 of 2048 11.3 / 9.5, 64 of 1536 9.55 / 7.25, 40 of 1500 10.7 / 8.7, 72 of
// 1501 16.0 / 10.3, 64 of 520 6.34 / 5.63, 128 of 400 6.34 / 5.42, 100 of 1001 10.2 / 8.7, 128 of 1024 7.08 / 6.60, 64 of 1024 6.11 / 6.13.
// TAIL: the row's end cuts a block.
// The fragments of one K-block, both steps, of F tiles 2 KB apart
template <int F>
__device__ __forceinline__ void block_frags(unsigned at0, unsigned at1, v4u (&f)[2 * F]) {
#pragma unroll
    for (int t = 0; t < F; t++) f[t] = *(const v4u __attribute__((address_space(3)))*)(uintptr_t)(at0 + t * 2048);
#pragma unroll
    for (int t = 0; t < F; t++) f[F + t] = *(const v4u __attribute__((address_space(3)))*)(uintptr_t)(at1 + t * 2048);
}
template <int RT, int CT, int KB, bool TAIL, bool WNT>
__global__ __launch_bounds__(512, 2) void k_gemm_whole(GemvEpiArgs p) {
    constexpr int NW = 8, HL = 2 * RT, WL = 2 * CT, F = RT + CT;      // load instructions per K-block; tiles
    constexpr int kWave = (KB > 1 ? 2 : 1) * F * 2048, kRedRow = 16 * CT + 4, kRed = 16 * RT * kRedRow;
    constexpr int NE = RT * CT == 4 ? 2 : 1, kPerRow = 16 * CT / NE;      // outputs per lane (consecutive columns), lanes per row of the tile
    static_assert(kRed * 4 <= kWave, "a wave's partial sums fit where its blocks were");
    const MmHead m = mm_head<kEpilogue>(p);
    __shared__ __attribute__((aligned(128))) char lds[NW * kWave];
    MmEpilogue<NE, true> emit;
    emit.y = m.y; emit.rows = m.rows; emit.n = m.n; emit.head = m.head; emit.n_epi = m.n_epi; emit.ka = m.ka;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rows = m.rows, n = m.n, cols = m.cols;
    const unsigned ncb = (unsigned)(n + 16 * CT - 1) / (16 * CT), groups = (unsigned)m.row_groups;
    const unsigned at = xcd_stretch(blockIdx.x, ncb * groups);
    // at / groups: of at most 256 workgroups (plan_gemm), so half of one is far more than the reciprocal errs
    const unsigned cb = (unsigned)__builtin_amdgcn_readfirstlane((int)(((float)at + 0.5f) * __builtin_amdgcn_rcpf((float)groups))), rg = at - cb * groups;
    const int r0 = (int)rg * 16 * RT, j0 = (int)cb * 16 * CT;
    const int nkb = (cols + 63) / 64, r8 = lane >> 3;
    const bf16_t* wb = m.W + (size_t)j0 * cols;
    const bf16_t* hb = m.h + (size_t)r0 * cols;
    unsigned hrow[HL], wrow[WL], koff[KB];               // byte offsets: the rows of each instruction, this lane's chunk of each block
#pragma unroll
    for (int q = 0; q < WL; q++) { const unsigned r = (unsigned)(q * 8 + r8), last = (unsigned)(n - j0 - 1); wrow[q] = (r < last ? r : last) * (unsigned)cols * 2u; }
#pragma unroll
    for (int q = 0; q < HL; q++) { const unsigned r = (unsigned)(q * 8 + r8), last = (unsigned)(rows - r0 - 1); hrow[q] = (r < last ? r : last) * (unsigned)cols * 2u; }
    auto vec = [&](int b) { return (wave + NW * b) * 8 + (lane & 7); };
#pragma unroll
    for (int b = 0; b < KB; b++) {                       // only a wave's last block can reach past the row's end, or lie behind it: then the row's first chunk, not multiplied
        if (b < KB - 1) koff[b] = (unsigned)vec(b) * 16u;
        else koff[b] = wave + NW * b < nkb ? span_at<!TAIL>(cols, vec(b)) * 2u : 0u;
    }
    unsigned gw[KB][WL][4], gh[KB][HL][4];
#pragma unroll
    for (int b = 0; b < KB; b++) {
#pragma unroll
        for (int q = 0; q < HL; q++) load_at<false>(hb, hrow[q] + koff[b], gh[b][q]);
        if (b == (KB > 1 ? 1 : 0)) {
            __builtin_amdgcn_sched_barrier(0);
            emit.prepare();
            emit.early_words(r0 + tid / kPerRow, j0 + (tid % kPerRow) * NE, tid / kPerRow < 16 * RT);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int b = 0; b < KB; b++)
#pragma unroll
        for (int q = 0; q < WL; q++) load_at<WNT>(wb, wrow[q] + koff[b], gw[b][q]);
    __builtin_amdgcn_sched_barrier(0);
    char* const mine = lds + wave * kWave;
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)mine;
    const unsigned f0 = lds0 + (lane & 15) * 128 + (((lane >> 4) ^ (lane & 7)) * 16), f1 = lds0 + (lane & 15) * 128 + (((4 + (lane >> 4)) ^ (lane & 7)) * 16);
    char* const to = mine + r8 * 128 + (((lane & 7) ^ r8) * 16);      // chunk c of row r sits at c ^ (r & 7)
    f32x4 acc[RT][CT];
#pragma unroll
    for (int i = 0; i < RT; i++)
#pragma unroll
        for (int j = 0; j < CT; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto stage = [&](int b) {
        char* const at = to + (b & 1) * (F * 2048);
#pragma unroll
        for (int q = 0; q < HL; q++) {
            if (TAIL && b == KB - 1) span_fix<false>(cols, vec(b), gh[b][q]);
            *reinterpret_cast<v4u*>(at + q * 1024) = v4u{gh[b][q][0], gh[b][q][1], gh[b][q][2], gh[b][q][3]};
        }
#pragma unroll
        for (int q = 0; q < WL; q++) {
            if (TAIL && b == KB - 1) span_fix<false>(cols, vec(b), gw[b][q]);
            *reinterpret_cast<v4u*>(at + (RT * 2 + q) * 1024) = v4u{gw[b][q][0], gw[b][q][1], gw[b][q][2], gw[b][q][3]};
        }
    };
    stage(0);
#pragma unroll
    for (int b = 0; b < KB; b++) {
        v4u f[2 * F];
        block_frags<F>(f0 + (b & 1) * (F * 2048), f1 + (b & 1) * (F * 2048), f);
        if (b + 1 < KB) stage(b + 1);
        if (b < KB - 1 || wave + NW * b < nkb) {
#pragma unroll
            for (int s = 0; s < 2; s++)
#pragma unroll
                for (int i = 0; i < RT; i++)
#pragma unroll
                    for (int j = 0; j < CT; j++)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f[s * F + i]), __builtin_bit_cast(bf16x8, f[s * F + RT + j]), acc[i][j], 0, 0, 0);
        }
    }
#pragma unroll
    for (int i = 0; i < RT; i++)
#pragma unroll
        for (int j = 0; j < CT; j++) {
            mm_drained(acc[i][j]);
            float* dst = reinterpret_cast<float*>(mine) + (i * 16 + (lane >> 4) * 4) * kRedRow + j * 16 + (lane & 15);
            const f32x4 v = acc[i][j];
            dst[0] = v.x; dst[kRedRow] = v.y; dst[2 * kRedRow] = v.z; dst[3 * kRedRow] = v.w;
        }
    emit.late_words();
    lds_barrier();
    const int er = tid / kPerRow, ec = (tid % kPerRow) * NE;
    if (er < 16 * RT) {
#pragma unroll
        for (int e = 0; e < NE; e++) {
            emit.put(e, parts_sum([&](int w) { return reinterpret_cast<const float*>(lds + w * kWave)[er * kRedRow + ec + e]; }));
        }
        emit.end();
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
template <int R, int RB, int U, bool EXACT, bool PRO, class Hook>
__device__ __forceinline__ void gemv_rows_sums(const bf16_t* W, const bf16_t* h, int n, int cols, int j0 /* uniform */, int lane, int tid, v4u* hs /* [RB][U * 64] */,
                                               Hook after_issue, float (&sums)[R * RB],
                                               const bf16_t* gain, const float& eps, bf16_t* hstore, f32x4* part /* [4]: four wave sums per row */) {
    constexpr int KC = (U + 3) / 4;                      // vectors per lane of the workgroup
    if constexpr (EXACT) cols = 512 * U;
    // 512-column pieces of a row that every row this form serves has whole (rows_kernel_rb): no end to look for in them
    constexpr int WHOLE = EXACT ? U : U <= 4 ? U - 1 : U - 4;
    auto at = [&](int v, bool whole) { return whole ? span_at<true>(cols, v) : span_at<false>(cols, v); };
    auto fix = [&](int v, bool whole, unsigned* w) { if (!whole) span_fix<false>(cols, v, w); };
    auto whole_u = [](int u) { return u < WHOLE; };                     // ... vectors u * 64 + lane of a weight row
    auto whole_c = [](int c) { return (c + 1) * 4 <= WHOLE; };          // ... vectors c * 256 + tid of a row of h
    // vector c of lane tid exists for every lane unless U is no multiple of four: then the last waves have none of the last
    auto mine = [&](int c) { return U % 4 == 0 || c < KC - 1 || tid < 64 * (U % 4); };
    unsigned hv[RB][KC][4], wg[KC][4], ww[R][U][4];
#pragma unroll
    for (int rr = 0; rr < RB; rr++)
#pragma unroll
        for (int c = 0; c < KC; c++) load_any<false>(h + (size_t)rr * cols, mine(c) ? at(c * kBlock + tid, whole_c(c)) : 0u, hv[rr][c]);
    if constexpr (PRO)
#pragma unroll
        for (int c = 0; c < KC; c++) load_any<false>(gain, mine(c) ? at(c * kBlock + tid, whole_c(c)) : 0u, wg[c]);
    __builtin_amdgcn_sched_barrier(0);   // h first: loads come back in the order they were issued
#pragma unroll
    for (int r = 0; r < R; r++) {
        const bf16_t* wrow = W + (size_t)((j0 + r < n) ? j0 + r : n - 1) * cols;   // a ragged last group re-reads the last row
#pragma unroll
        for (int u = 0; u < U; u++) load_any<true>(wrow, at(u * 64 + lane, whole_u(u)), ww[r][u]);
    }
    __builtin_amdgcn_sched_barrier(0);
    after_issue();
#pragma unroll
    for (int rr = 0; rr < RB; rr++)
#pragma unroll
        for (int c = 0; c < KC; c++) {
            fix(c * kBlock + tid, whole_c(c), hv[rr][c]);
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
                if (rr == 0) fix(c * kBlock + tid, whole_c(c), wg[c]);
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
            fix(u * 64 + lane, whole_u(u), ww[r][u]);
#pragma unroll
            for (int rr = 0; rr < RB; rr++) sums[rr * R + r] = dot_acc<bf16_t>(ww[r][u], wh[rr], sums[rr * R + r]);
        }
    }
}

// GEMV with an elementwise epilogue: one lane of each wave per output e (row e / R of h, column j0 + e % R) plays it
// through the kernels that follow (see kernels.h; none of them: the plain GEMV).
template <int R, int RB, int U, bool EXACT, Ride RIDE>
__global__ __launch_bounds__(kBlock) void k_gemv_rows(RideArgs<RIDE> p) {
    constexpr bool PRO = RIDE == kPrologue;
    const MmHead m = mm_head<RIDE>(p);
    const int n = m.n;
    // up to 2048 columns an XCD takes a contiguous stretch of the outputs (decode chain, 2048 columns, 1 row 430 -> 406 us, 4 rows
    // 482 -> 472; 1024 columns, 1 row 347 -> 326), at 2048 columns only while that is one workgroup per CU: eight distant streams of
    // long rows are slower than one (1 row, 8192 outputs 9.2 against 7.9 us, 4 rows 9.8 against 9.1; below 1537 columns the
    // stretch is the faster one up to 32768 outputs); longer rows the same (4096 columns, 4 rows 289 against 304)
    const unsigned bid = U < 4 || (U == 4 && n <= 1024 * R) ? xcd_stretch(blockIdx.x, (unsigned)(n + 4 * R - 1) / (4 * R)) : blockIdx.x;
    bf16_t* hstore = bid == 0 ? m.hstore : nullptr;
    __shared__ v4u hs[RB * U * 64];
    __shared__ f32x4 part[4];
    const int tid = threadIdx.x, lane = tid & 63;
    const int j0 = (bid * (kBlock / 64) + __builtin_amdgcn_readfirstlane(tid >> 6)) * R;   // uniform: the weight rows' addresses stay in scalar registers
    MmEpilogue<1, RIDE != kAlone> emit;
    emit.y = m.y; emit.rows = RB; emit.n = n; emit.head = m.head; emit.n_epi = m.n_epi; emit.ka = m.ka;
    float sums[R * RB];
    gemv_rows_sums<R, RB, U, EXACT, PRO>(m.W, m.h, n, m.cols, j0, lane, tid, hs, [&] {
        emit.prepare();
        const int e = sums_index<R * RB>(lane);
        emit.begin(e / R, j0 + e % R, lane < sums_lanes(R * RB) && e < R * RB);
    }, sums, m.gain, emit.eps, hstore, part);
    if constexpr (R * RB == 1) emit.put(0, wave_sum(sums[0]));
    else emit.put(0, wave_sums<R * RB>(sums, lane));
    emit.end();
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

constexpr int kMmWideRows = 81;     // rows from which the 32 x 32 tile is used (see plan_gemm)

// k_gemv_rows: up to 4 rows of h, rows of 8 to 8192 columns (all of a wave's loads are in registers at once);
// two weight rows per wave once half the waves fill the chip, and only then rows beyond 2048 columns.
constexpr int kRowsTwoFrom = 1024;
bool rows_served(long long rows, long long n, long long cols) {
    return rows >= 1 && rows <= 4 && n >= 1 && cols >= 8 && cols <= (n >= kRowsTwoFrom ? 8192 : 2048) && rows * n <= (1ll << 31);
}
template <Ride RIDE, int RB>
const void* rows_kernel_rb(int n, int cols) {
    const int u = (cols + 511) / 512;
    if (n < kRowsTwoFrom) {
        switch (u) {
        case 1: return PG_FN(k_gemv_rows<1, RB, 1, false, RIDE>);
        case 2: return PG_FN(k_gemv_rows<1, RB, 2, false, RIDE>);
        case 3: return PG_FN(k_gemv_rows<1, RB, 3, false, RIDE>);
        default: return PG_FN(k_gemv_rows<1, RB, 4, false, RIDE>);
        }
    }
    switch (cols) {
    case 1024: return PG_FN(k_gemv_rows<2, RB, 2, true, RIDE>);
    case 2048: return PG_FN(k_gemv_rows<2, RB, 4, true, RIDE>);
    case 4096: return PG_FN(k_gemv_rows<2, RB, 8, true, RIDE>);
    case 8192: return PG_FN(k_gemv_rows<2, RB, 16, true, RIDE>);
    default: break;
    }
    // up to 2048 columns a form per 512, so that only a row's last piece has an end to look for (decode chains of 60 sub-blocks against one
    // form for up to 1536 columns, us per iteration: 1 row of 1400 columns 198 -> 182, 4 rows 255 -> 243, 3 rows of 1500 242 -> 238; 30 times RMSNorm,
    // GEMV and GELU, 2048 outputs: 1 / 4 rows of 256 columns 88 / 110 -> 78 / 94, of 512 88 / 110 -> 78 / 94, of 1000 88 / 111 -> 82 / 97)
    if (u <= 1) return PG_FN(k_gemv_rows<2, RB, 1, false, RIDE>);
    if (u <= 2) return PG_FN(k_gemv_rows<2, RB, 2, false, RIDE>);
    if (u <= 3) return PG_FN(k_gemv_rows<2, RB, 3, false, RIDE>);
    if (u <= 4) return PG_FN(k_gemv_rows<2, RB, 4, false, RIDE>);
    if (u <= 8) return PG_FN(k_gemv_rows<2, RB, 8, false, RIDE>);
    if (u <= 12) return PG_FN(k_gemv_rows<2, RB, 12, false, RIDE>);
    return PG_FN(k_gemv_rows<2, RB, 16, false, RIDE>);
}
template <Ride RIDE>
const void* rows_kernel(int rows, int n, int cols) {
    switch (rows) {
    case 1: return rows_kernel_rb<RIDE, 1>(n, cols);
    case 2: return rows_kernel_rb<RIDE, 2>(n, cols);
    case 3: return rows_kernel_rb<RIDE, 3>(n, cols);
    default: return rows_kernel_rb<RIDE, 4>(n, cols);
    }
}

// Matrix cores: from 5 rows on, any number of outputs per row (us per launch on the matrix cores / the vector units: 128 rows
// of 2048 columns, 8 outputs 6.8 / 31; 64 of 4096, 12 outputs 6.6 / 25.8), rows of h of any length that element offsets
// within a tile of 64 rows reach (32 bits, as are the outputs' indices).
bool mm_served(long long rows, long long n, long long cols) { return rows > 4 && cols >= 8 && cols <= (1ll << 26) && rows * n <= (1ll << 32); }

template <int KS, bool TAIL, Ride RIDE>
const void* gemm_rows_kernel(int nr, int nc) {
    if constexpr (RIDE == kPrologue) {
        if (nr == 16) return PG_FN(k_gemm_rows<KS, TAIL, 16, 16, RIDE>);
        if (nr == 8) return nc == 8 ? PG_FN(k_gemm_rows<KS, TAIL, 8, 8, RIDE>) : PG_FN(k_gemm_rows<KS, TAIL, 8, 16, RIDE>);
        return nc == 8 ? PG_FN(k_gemm_rows<KS, TAIL, 4, 8, RIDE>) : PG_FN(k_gemm_rows<KS, TAIL, 4, 16, RIDE>);
    } else {
        return nr == 8 ? PG_FN(k_gemm_rows<KS, TAIL, 8, 8, RIDE>) : PG_FN(k_gemm_rows<KS, TAIL, 16, 8, RIDE>);
    }
}
template <Ride RIDE>
const void* gemm_rows_form(int nr, int nc, int cols) {
    if (cols <= 512) return cols == 512 ? gemm_rows_kernel<4, false, RIDE>(nr, nc) : gemm_rows_kernel<4, true, RIDE>(nr, nc);
    if (cols <= 1024) return cols == 1024 ? gemm_rows_kernel<8, false, RIDE>(nr, nc) : gemm_rows_kernel<8, true, RIDE>(nr, nc);
    return cols == 2048 ? gemm_rows_kernel<16, false, RIDE>(nr, nc) : gemm_rows_kernel<16, true, RIDE>(nr, nc);
}
template <Ride RIDE, bool WNT>
const void* gemm_cols_form(int cols) {
    if (cols <= 1024) return cols == 1024 ? PG_FN(k_gemm_cols<8, false, true, RIDE>) : PG_FN(k_gemm_cols<8, true, true, RIDE>);
    return cols == 2048 ? PG_FN(k_gemm_cols<16, false, WNT, RIDE>) : PG_FN(k_gemm_cols<16, true, WNT, RIDE>);
}
template <int RT, int CT, bool TAIL, bool WNT>
const void* whole_kernel_nt(int cols) {
    const int kb = (cols + 511) / 512;
    if constexpr (TAIL && WNT) {              // (up to 1024 columns and kMmWideRows - 1 rows, where 2 x 1 tiles are never the cheapest)
        if constexpr (RT > CT) return nullptr;
        else return kb > 2 ? nullptr : kb == 1 ? PG_FN(k_gemm_whole<RT, CT, 1, true, true>) : PG_FN(k_gemm_whole<RT, CT, 2, true, true>);
    } else {
        return kb == 1 ? PG_FN(k_gemm_whole<RT, CT, 1, TAIL, WNT>) : kb == 2 ? PG_FN(k_gemm_whole<RT, CT, 2, TAIL, WNT>) : kb == 3 ? PG_FN(k_gemm_whole<RT, CT, 3, TAIL, WNT>) : PG_FN(k_gemm_whole<RT, CT, 4, TAIL, WNT>);
    }
}
template <int RT, int CT>
const void* whole_kernel(int cols, bool nt) {
    if (cols % 64) return nt ? whole_kernel_nt<RT, CT, true, true>(cols) : whole_kernel_nt<RT, CT, true, false>(cols);
    return nt ? whole_kernel_nt<RT, CT, false, true>(cols) : whole_kernel_nt<RT, CT, false, false>(cols);
}
// The cheapest tile whose grid is one workgroup per CU.  us per RMSNorm and GEMV, rows x outputs in tiles of 16: 64 rows of 2048 columns 1 x 2 8.36, 2 x 1 8.55, 1 x 1
// (512 workgroups) 8.98, 2 x 2 9.58; 48 of 2048 8.18, 8.10, 8.85, 9.32; 128 of 1024 6.47, 6.59, 6.74, 7.11; 64 of 520 1 x 1 5.73, 2 x 1 6.22, 1 x 2 6.28.
// 2 x 2 against k_gemm_tile's, from kMmWideRows rows: beyond the cache and without shared cache lines 128 of 2048 9.93 / 10.39, 96 of 1536 8.53 / 8.98, 96 of 1152
// 7.06 / 8.11 (plan_gemm), otherwise not: 100 of 2000 11.05 / 10.21, 128 of 1504 8.73 / 8.46, 128 of 2048 within the cache 9.78 / 9.58.
// Weights by plain / non-temporal loads, us per RMSNorm and GEMV with its tail, megabytes of weights in the chain in brackets: up to 1024 columns and 80 rows
// without shared cache lines 64 rows of 1024 [126] 5.5 / 5.15, [400] 5.2 / 5.1, 64 of 512 [105] 5.1 / 4.8, 33 of 1024, 4096 outputs [50] 8.65 / 8.35; with them 64 of 1000
// [127] 5.75 / 5.70, [400] 6.15 / 5.69, 40 of 1001 [126] 6.43 / 6.62, [400] 7.00 / 6.65; longer rows 64 of 2048 [200] 7.5 / 8.1, 40 of 1928 [400] 9.4 / 9.8, 40 of 1500 [400]
// 9.1 / 9.1, [200] 8.0 / 9.15.
bool plan_whole(int rows, int n, int cols, Launch* out) {
    static const int by_cost[4][2] = {{1, 1}, {1, 2}, {2, 1}, {2, 2}};
    for (const auto& t : by_cost) {
        if (t[0] * t[1] == 4 && rows >= kMmWideRows) break;
        const unsigned groups = blocks_for(rows, 16 * t[0]);
        if ((long long)blocks_for(n, 16 * t[1]) * groups > 256) continue;
        auto kernel = [&](bool nt) {
            return t[0] == 1 ? (t[1] == 1 ? whole_kernel<1, 1>(cols, nt) : whole_kernel<1, 2>(cols, nt)) : t[1] == 1 ? whole_kernel<2, 1>(cols, nt) : whole_kernel<2, 2>(cols, nt);
        };
        const bool lines = cols % 64 == 0;               // no two rows share a cache line
        if (rows < kMmWideRows && cols <= 1024) {
            out->fn = kernel(lines);
            if (!lines) out->fn_beyond_cache = kernel(true);
        } else {
            out->fn = kernel(false);
            if (lines && (rows < kMmWideRows || n >= 256)) out->fn_beyond_cache = kernel(true);
        }
        out->block = dim3(512);
        out->gemm_row_groups = groups;
        out->grid = dim3(blocks_for(n, 16 * t[1]) * groups);
        return true;
    }
    return false;
}
// The tile of a workgroup that normalises its own rows: the cheapest whose grid is still one workgroup per CU.  A row costs its bytes and its
// normalising, an output its bytes.  Decode chains, us per sub-block, rows x outputs of the tile, in brackets the workgroups (measured with a branch per row in
// the sums of squares; without it all of them are 0.1 - 0.3 faster):
//   16 rows of 2048 columns  8 x 16 [256] 5.58, 16 x 8 [256] 5.96, 8 x 8 [512] 6.90    8 of 2048  8 x 8 [256] 4.78, 4 x 16 [256] 4.97, 4 x 8 [512] 5.93
//   32 of 2048  16 x 16 [256] 6.83, 8 x 16 [512] 7.76       32 of 1024  8 x 16 [256] 3.83, 16 x 8 [256] 4.25, 16 x 16 [128] 4.40, 4 x 16 [512] 4.52
//   16 of 1024  4 x 16 [256] 3.43, 8 x 8 [256] 3.63, 8 x 16 [128] 3.78, 16 x 8 [128] 4.18    8 of 1024  4 x 8 [256] 3.31, 4 x 16 [128] 3.38, 8 x 8 [128] 3.54
//   16 of 520  4 x 16 [132] 3.86, 8 x 8 [130] 3.94, 4 x 8 [260] 4.11    32 of 400  4 x 16 [200] 3.27, 8 x 8 [200] 3.39, 4 x 8 [400] 3.64
// 4096 outputs, against one tile of 8 or 16 rows by 8 outputs [512] with the RMSNorm that went with it: 8 rows of 1024 columns 8 x 16 3.71 / 4.71, 16 of 1024
// 16 x 16 4.17 / 5.50, 16 of 2048 6.74 / 8.29.
// Where none fits (more than 4096 outputs up to 16 rows, which merge_prologue admits up to 8 rows, 2048 above): 8 x 8 up to 8 rows, 16 x 16 above.
void prologue_tile(int rows, int n, int cols, int* nr, int* nc) {
    static const int by_cost[2][5][2] = {{{4, 8}, {4, 16}, {8, 8}, {8, 16}, {16, 16}}, {{4, 8}, {8, 8}, {4, 16}, {8, 16}, {16, 16}}};
    for (const auto& t : by_cost[cols > 1024])
        if ((long long)blocks_for(n, t[1]) * blocks_for(rows, t[0]) <= 256) {
            *nr = t[0];
            *nc = t[1];
            return;
        }
    *nr = rows <= 8 ? 8 : 16;
    *nc = *nr;
}
void plan_gemm(int rows, int n, int cols, Ride ride, Launch* out) {
    const bool merged = ride != kAlone;
    const int ntiles = (rows + 15) / 16;
    out->arg_bytes = merged ? sizeof(GemvEpiArgs) : sizeof(GemvAloneArgs);
    out->block = dim3(kBlock);
    out->gemm_row_groups = (unsigned)ntiles;
    out->fn_beyond_cache = nullptr;
    if (ride == kPrologue || (rows <= 16 && cols <= 2048)) {
        int nr = rows <= 8 ? 8 : 16, nc = 8;
        if (ride == kPrologue) prologue_tile(rows, n, cols, &nr, &nc);
        const unsigned tiles = blocks_for(rows, nr);
        out->fn = ride == kPrologue ? gemm_rows_form<kPrologue>(nr, nc, cols) : merged ? gemm_rows_form<kEpilogue>(nr, nc, cols) : gemm_rows_form<kAlone>(nr, nc, cols);
        out->gemm_row_groups = tiles | ((65535u + tiles) / tiles) << 8;
        out->grid = dim3(blocks_for(n, nc) * tiles);
        return;
    }
    if (ride == kEpilogue && cols <= 2048 && plan_whole(rows, n, cols, out)) return;
    // us per launch alone, k_gemm_cols / k_gemm_tile's tiles: 17 rows of 2048 columns 4.70 / 5.69, 64 6.16 / 6.89, 64 of 1024 3.16 / 4.04; 80 of 2048 7.53 / 7.30, 40 of
    // 1500 7.37 / 6.61.  With a tail and more outputs than k_gemm_whole takes: 33 of 1024, 8200 outputs 9.0 / 12.2, 64 of 1024, 8192 outputs 10.9 / 8.4, 64 of 2048 20.0 / 13.3:
    // there, and for long ragged rows, the line is not the best one.
    // A 32-column tile of up to 16 outputs per row would be half empty; with so few workgroups, one tile of rows each.
    if (cols <= 2048 && (rows < kMmWideRows || n <= 16)) {
        out->gemm_row_groups = (unsigned)(ntiles < 4 || n <= 16 ? ntiles : 4);
        // Several workgroups read the same weights, side by side.  us per launch alone without / with non-temporal loads, in brackets the megabytes of weights in
        // the chain: 64 rows of 1024 columns [126] 3.26 / 3.29, [400] 3.42 / 3.16, of 1001 4.40 / 4.64, 4.63 / 4.56; of 2048 6.05 / 6.53, 6.43 / 6.15, 40 of
        // 1600 5.99 / 6.25, 6.26 / 6.07, 40 of 1088 4.49 / 4.47, 4.59 / 4.38; longer rows that share cache lines [400] 40 of 1300 5.86 / 6.08, 1500 7.32 / 8.00,
        // 1928 6.97 / 7.71.
        out->grid = dim3(blocks_for(n, 16) * out->gemm_row_groups);
        out->fn = merged ? gemm_cols_form<kEpilogue, false>(cols) : gemm_cols_form<kAlone, false>(cols);
        if (cols % 64 == 0) out->fn_beyond_cache = merged ? gemm_cols_form<kEpilogue, true>(cols) : gemm_cols_form<kAlone, true>(cols);
        return;
    }
    // The largest tile that still gives every CU a workgroup: 64 x 32 in 256 (RMSNorm, GEMV, GELU, GEMV and add on 128 rows of 2048
    // columns, 8192 outputs 44 us a layer, with 32 x 32 tiles 53); 32 x 32 from kMmWideRows rows, or where tiles of 16 x 16 would be
    // more than two workgroups per CU (us per launch, 32 x 32 / 16 x 16: 64 rows of 4096 columns, 2048 outputs, 512 tiles 12.6 /
    // 11.0, 2304 outputs, 576 tiles 12.9 / 14.8; 33 rows, 2304 outputs, 432 tiles 11.0 / 10.1; 70 rows, 2048 outputs, 640 tiles 10.8 / 14.0).
    const long long wide = blocks_for(n, 32), narrow = blocks_for(n, 16), two = (ntiles + 1) / 2, four = (ntiles + 3) / 4;
    if (merged) out->block = dim3(512);
    if (ntiles > 2 && wide * four >= 256) {
        out->fn = merged ? PG_FN(k_gemm_tile<4, 2, 1, 8, false>) : PG_FN(k_gemm_tile<4, 2, 2, 4, false>);
        out->gemm_row_groups = (unsigned)four;
        out->grid = dim3((unsigned)(wide * four));
    } else if (rows >= kMmWideRows || (ntiles > 1 && narrow * ntiles > 512)) {
        out->fn = merged ? PG_FN(k_gemm_tile<2, 2, 2, 8, false>) : PG_FN(k_gemm_tile<2, 2, 2, 4, false>);
        out->gemm_row_groups = (unsigned)two;
        out->grid = dim3((unsigned)wide * out->gemm_row_groups);
        // Where all workgroups that share their weights run side by side, one per CU, no two rows share a cache line, and there are enough outputs.  us per
        // launch alone without / with non-temporal loads, in brackets the megabytes of weights in the chain: 128 rows of 1024 columns [200] 4.72 / 5.35, [400] 5.73 / 5.35,
        // of 1536 5.58 / 6.72, 6.90 / 6.63, of 2048 6.37 / 7.71, 7.93 / 7.61, 64 of 2304 6.85 / 8.77, 8.82 / 8.56; rows that share cache lines [400] 100 of 2000 8.0 / 9.8;
        // larger grids [400] 100 of 3000 16.1 / 23.1, 81 of 4096 15.1 / 15.2; few outputs, 128 of 8192, 64 outputs [200] 14.0 / 20.7, 256 [400] 18.8 / 17.6.
        // With a tail, up to 2048 columns, k_gemm_whole's non-temporal form takes that place: 128 of 2048 [400] 7.38 / 6.68, [200] 6.04 / 6.81, of 1536 6.34 / 5.72.
        if (out->grid.x <= 256 && cols % 64 == 0 && n >= 256) out->fn_beyond_cache = merged ? (cols <= 2048 ? whole_kernel<2, 2>(cols, true) : PG_FN(k_gemm_tile<2, 2, 2, 8, true>)) : PG_FN(k_gemm_tile<2, 2, 2, 4, true>);
    } else {
        // (more than one workgroup per CU, rows that 16-byte loads cannot reach: see k_gemm_tile)
        out->fn = merged ? (narrow * ntiles <= 256 && cols % 8 == 0 ? PG_FN(k_gemm_tile<1, 1, 2, 8, false>) : PG_FN(k_gemm_tile<1, 1, 2, 8, false, false>)) : PG_FN(k_gemm_tile<1, 1, 2, 4, false>);
        out->grid = dim3((unsigned)(narrow * ntiles));
    }
}

template <typename T>
bool plan_gemv_t(int ind, int rows, int n, int cols, Launch* out) {
    constexpr int NV = 16 / (int)sizeof(T);
    if constexpr (sizeof(T) == 2) {
        // Three and four rows go to the form that shares h through LDS (at 2048 x 2048, us per launch at 2 / 3 / 4 rows: 3.3 / 3.5 /
        // 3.7; vector with h per wave 3.8 / 4.4 / 4.5; matrix-core form with 8 columns per workgroup 3.9 / 4.0 / 4.0).  Its sums err
        // less than the matrix cores' (rows of W that cancel to zero, 4 rows of 2048 columns: rms of the outputs 2.8e-6 against
        // 5.1e-6), and products among the subnormal fp32 numbers are kept on both.
        // Four rows of more than 4096 columns that leave whole vectors of k_gemv_rows' form empty (forms of 6144 and 8192 columns) stay
        // with the vector form that takes a row in pieces (4 rows of 5000 columns 16.7 against 16.1, of 7000 29.3 against 27.6; of
        // 6000 columns 11.2 against 12.3, of 4500, whose last vector that form reads element by element, 16.4 against 18.0).
        const bool pieces = rows == 4 && cols > 4096 && cols % NV == 0 && (cols + 511) / 512 % 4 != 0;
        if ((rows == 3 || rows == 4) && rows_served(rows, n, cols) && !pieces && !(n >= 1024 && cols == 64 * kGemvChunk * NV)) {
            out->fn = rows_kernel<kAlone>(rows, n, cols);
            out->arg_bytes = sizeof(GemvAloneArgs);
            out->block = dim3(kBlock);
            out->grid = dim3(blocks_for(n, (kBlock / 64) * (n >= kRowsTwoFrom ? 2 : 1)));
            return true;
        }
        if (mm_served(rows, n, cols)) {      // a dense contraction: matrix cores from 5 rows on
            plan_gemm(rows, n, cols, kAlone, out);
            return true;
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
    // (the epilogue counts all its elements in 32 bits)
    if (s.rows <= 4 ? !rows_served(s.rows, s.n, s.cols) : !mm_served(s.rows, s.n, s.cols) || s.rows * s.n > (1ll << 31)) return false;
    *n_out = s.rows * s.n;
    return true;
}

// Every workgroup normalises its rows anew, which is free while the grid fills the chip once or twice and the more rows the
// dearer beyond; the separate RMSNorm costs a node.  The lines count workgroups of 8 outputs from 5 rows on, whatever the tile that prologue_tile picks.  us with the
// RMSNorm in front / on its own, on both sides of each line:
//   3 and 4 rows   (RMSNorm, GEMV and GELU) 1024 workgroups: 4 rows of 1024 columns 5.8 / 7.0; 4096: 15.3 / 15.0
//                  longer than 4096 columns, 256 workgroups: 4 of 8192 10.5 / 11.4; 512: 19.5 / 17.2
//   5 to 8 rows    (from here on GELU and two adds) 8192 outputs: 8 of 1024 6.46 / 7.33, 8 of 2048 10.8 / 11.2; 8200: 6.67 / 7.43, 11.3 / 11.3
//   9 to 16 rows   4096: 16 of 1024 4.19 / 5.86, 16 of 2048 6.81 / 8.04; 4104: 6.16 / 6.37, 9.95 / 9.03
//   17 to 32 rows  4096: 32 of 1024 5.67 / 6.36; 6000: 7.30 / 7.41; 8192: 8.78 / 7.99; 8200: 9.44 / 9.74; above 1024 columns, 2048: 32 of 2048 6.18 / 6.65; 3000:
//                  8.89 / 8.30; 4096: 9.06 / 8.56; 4104: 11.3 / 9.5 (on its own: k_gemm_whole, which was not there when these two lines were drawn, at 8192 and 4096)
// One and two rows: 4096 workgroups of 2048 columns 23.4 / 25.2.
bool merge_prologue(const Shape& s) {
    if (s.rows <= 2) return true;
    const long long blocks = s.rows <= 4 ? blocks_for(s.n, s.n >= kRowsTwoFrom ? 8 : 4) : s.rows <= 16 ? blocks_for(s.n, 8) : 2 * (long long)blocks_for(s.n, 16);
    if (s.rows <= 4 && s.cols > 4096) return blocks <= 256;
    if (s.rows > 4 && (s.rows > kPrologueMaxRows || s.cols > 2048)) return false;
    return blocks <= (s.rows <= 8 || (s.rows > 16 && s.cols <= 1024) ? 1024 : 512);
}

void plan_gemv_epilogue(const Shape& s, bool with_prologue, Launch* out) {
    const int rows = (int)s.rows, n = (int)s.n, cols = (int)s.cols;
    out->mod_fn = nullptr;
    out->gemm_row_groups = 0;
    out->fn_beyond_cache = nullptr;
    if (rows > 4) { plan_gemm(rows, n, cols, with_prologue ? kPrologue : kEpilogue, out); return; }
    out->fn = with_prologue ? rows_kernel<kPrologue>(rows, n, cols) : rows_kernel<kEpilogue>(rows, n, cols);
    out->arg_bytes = sizeof(GemvEpiArgs);
    out->block = dim3(kBlock);
    out->grid = dim3(blocks_for(n, (kBlock / 64) * (n >= kRowsTwoFrom ? 2 : 1)));
}

}  // namespace pgk
