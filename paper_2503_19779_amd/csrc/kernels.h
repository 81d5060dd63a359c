// kernels.h -- argument blocks and launch descriptions shared by the device code (kernels.hip)
// and the chain runtime (chain.hip).  gfx950 only.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pgk {

enum Op : int { kAdd = 0, kMul = 1, kGelu = 2, kRmsNorm = 3, kGemv = 4, kScaleBiasRelu = 5 };
enum DType : int { kF32 = 0, kBF16 = 1 };

// One argument block per kernel, passed by value as the kernel's single parameter.  An operand
// whose bit is set in the kernel's IND template mask holds the address of a pointer-table slot
// instead of the tensor's address: the kernel loads the tensor pointer from it before anything
// else (the dereference prologue of Parameter Indirection, paper Sec. 4 "Kernel generation").
struct EwArgs {          // ADD / MUL / GELU
    void* out;
    const void* a;
    const void* b;
    long long n;
    long long m;
};
struct RmsArgs {
    void* out;
    const void* x;
    const void* g;
    int rows;
    int cols;
    float eps;
};
struct GemvArgs {
    void* out;
    const void* W;
    const void* h;
    int rows;
    int n;
    int cols;
    int row_groups;      // matrix-core form only: the grid is (column blocks) x (row groups); from Launch
};
struct SbrArgs {
    void* out;
    const void* x;
    const void* s;
    const void* b;
    long long n;
    unsigned inner;
    unsigned channels;
};

// Batched multi-tensor copy: the destination side is static and lives in device memory, the
// source pointers change every replay and travel in the argument block.
constexpr int kCopyMaxSrc = 448;           // 448 * 8 B + header < 4 KB of kernel arguments
constexpr unsigned kCopyChunkBytes = 8192;   // bytes of one tensor handled by one workgroup: 256 lanes x 2 x 16 B
struct CopyTensor { void* dst; unsigned long long bytes; };
struct CopyChunk { unsigned tensor; unsigned len; unsigned long long off; };
struct CopyArgs {
    const CopyChunk* chunks;     // [dev] chunk list, offset to this launch's first chunk
    const CopyTensor* tensors;   // [dev] per-tensor destination and size
    int src_base;                // tensor index of src[0]
    int n_chunks;
    const void* src[kCopyMaxSrc];
};

// Pointer-table writer: the pointers ride in the argument block, one wave stores them.
constexpr int kTableMaxPtrs = 480;
struct TableArgs {
    const void** table;          // [dev]
    int base;
    int n;
    const void* ptr[kTableMaxPtrs];
};

// ---- merged dispatches --------------------------------------------------------------------------------
// A captured graph need not spend one dispatch per kernel.  A run of consecutive kernels of a chain that
// all work element for element on the same n elements -- add / mul / GELU, and RMSNorm over rows of
// exactly 256 x 16 bytes -- goes out as ONE dispatch.  The tensor is cut into units of 256 lanes x 16
// bytes (lane t owns vector t of a unit; an RMSNorm row is one unit), one workgroup per unit.  The lane
// runs the kernels one after the other, each with its stand-alone arithmetic and its one rounding to
// the storage type, stores its output if something reads it from memory later (chain.hip, drop_dead_stores), and hands the stored bits on to
// the next kernel in registers when that kernel reads the same buffer element for element -- so the run costs one trip
// to memory, not one per kernel.  Operands that no kernel of the run produces are fetched up front.
constexpr int kMergeShortPhases = 4;      // kernels per merged dispatch
constexpr int kMergeMaxPhases = 8;        // ... of bf16 kernels over kMergeLongFrom to kMergeLongTo elements
// Below, runs stay at four kernels (64 kernels on 4096 elements 52 us, on 16384 in runs of eight 48; longer runs of smaller
// tensors were not measured); above, memory bounds the run and the wider kernel has fewer waves in flight (64 kernels played by k_merged, us in runs of eight / four: 2^20
// elements 77 / 88, 2^21 108 / 113, 3 * 10^6 149 / 142, 2^23 335 / 306, 2^25 1171 / 994).
constexpr long long kMergeLongFrom = 16384, kMergeLongTo = 1ll << 21;
constexpr int kMergeSlots = 3;            // outputs a lane keeps in registers for later kernels of the run
constexpr unsigned kMergeFromMemory = 255;

struct MergePhase {
    void* out;
    const void* in0;        // ADD / MUL / GELU: a; RMSNORM: x
    const void* in1;        // ADD / MUL: b; RMSNORM: gain
    unsigned m;             // ADD / MUL: period of b
    float eps;              // RMSNORM
    // op | src0 << 8 | src1 << 16 | dst << 24: the kernel (kAdd, kMul, kGelu, kRmsNorm), the register slot
    // each operand is taken from (or kMergeFromMemory), the slot that keeps the output
    unsigned meta;
    unsigned ind;           // bit 0 / 1: in0 / in1 hold the address of a pointer-table slot
};
struct MergedArgs {
    unsigned n;             // elements every kernel of the run produces
    int n_phase;
    MergePhase ph[kMergeMaxPhases];   // entries from n_phase on: meta says "operands from slots", nothing is fetched
};

// A run of those kernels in which each takes the result of the one before (the first: memory) and a second operand, if it has
// one, from memory, no RMSNorm among them: the argument block of a chain.
struct ChainPhase {
    const void* in1;        // the second operand; GELU, and entries from n_phase on: the first kernel's first operand, fetched and ignored
    void* out;
};
constexpr unsigned kChainPeriods = 1u << 31;        // ChainArgs::slots: some second operand has a period
struct ChainArgs {
    const void* in0;        // the first kernel's first operand
    unsigned n;
    unsigned slots;         // bit i: ph[i].in1 is a pointer-table slot; bit kMergeMaxPhases: in0 is
    unsigned ops;           // 4 bits per kernel: op | store << 3; entries from n_phase on: kChainEnd
    int reserved;
    ChainPhase ph[kMergeMaxPhases];
    unsigned m[kMergeMaxPhases];      // periods of the second operands (n: element for element)
};
constexpr unsigned kChainEnd = 7;

// The same idea for a GEMV followed by element-for-element kernels over its outputs (GELU of the result,
// the residual add, an input add): they ride in the GEMV's dispatch as an epilogue.  After the wave's
// reduction every lane holds the finished sums; lane e of a wave takes output e (row e >> 1 of h, column
// j0 + (e & 1)), rounds it to the storage type as the GEMV's own store would, and runs the following
// kernels on that one element, operands fetched while the weights were in flight.  No workgroup needs
// another's results, so nothing has to be waited for.
constexpr int kEpiMaxPhases = 3;
constexpr unsigned kEpiStore = 1u << 8;   // MergePhase::ind: this kernel's output is stored (something reads it from memory, or it is the buffer's last version)
// And the RMSNorm in front of the GEMV can ride along as a prologue: every workgroup of the GEMV needs the
// whole normalised vector anyway, so each one normalises the rows itself (the stand-alone kernel's
// arithmetic, lane t holding vector t of a row -- exactly where the GEMV wants h in LDS) while its
// weights are on their way, and workgroup 0 stores the result where the RMSNorm kernel would have.
// A kernel of the epilogue may update the normalised stream in place (the residual add does); the
// runtime then lets it write a shadow copy of that buffer instead, so that no workgroup can read an
// element another one has already replaced (chain.hip: versions).
constexpr unsigned kEpiHeadStore = 1u << 16;    // GemvEpiArgs::head: store the GEMV's result
constexpr unsigned kEpiXSlot = 1u << 18, kEpiGainSlot = 1u << 19;   // x / gain are pointer-table slots
constexpr unsigned kEpiStoreH = 1u << 20;       // workgroup 0 stores the normalised rows to g.h
// Worked out on the host, once (chain.hip, seal_epilogue).  In the table every operand has an address that can be read: one that comes
// from a register slot, or does not exist, names the GEMV's output buffer, with the period rows * n.
constexpr unsigned kEpiDecoder = 1u << 21;      // the kernels are GELU of the GEMV's result, then up to two adds with an operand from memory, which is in1
constexpr unsigned kEpiMemFirst = 1u << 9;      // MergePhase::ind: that operand is the add's first
constexpr unsigned kEpiAnySlot = 1u << 22;      // some operand of the epilogue is a pointer-table slot
constexpr unsigned kEpiPlain = 1u << 23;        // no operand of the epilogue has a broadcast period
// A GEMV that nothing rides with takes this much of it (a launch from the host pays for every byte of the block:
// 200 against 48 bytes cost 0.2 - 0.4 us per launch of an eager loop).
struct GemvAloneArgs {
    GemvArgs g;
    unsigned head;          // bit 0 / 1: W / h are pointer-table slots; kEpiHeadStore
    int reserved;
};
struct GemvEpiArgs {
    GemvArgs g;             // with a prologue g.h is where the normalised rows are stored, not read
    unsigned head;          // bit 0 / 1: W / h are pointer-table slots; bits 8-15: slot that keeps the GEMV's result; bits 16-23 above
    int n_epi;
    const void* x;          // prologue: [rows, cols] to normalise
    const void* gain;       // prologue: [cols]
    float eps;
    int reserved;
    MergePhase ph[kEpiMaxPhases];   // m: period of in1 (rows * n = element for element)
};

// A run of consecutive per-channel scale + bias + ReLU kernels over one tensor (each reads what the one before it
// wrote, element for element; same length, same channels): one dispatch that reads x once and keeps the elements in
// registers from kernel to kernel.  Outputs that are overwritten before anything reads them from memory are not stored.
constexpr int kSbrRunMax = 16;              // kernels per run
constexpr int kSbrRunMaxChannels = 128;     // one lane per scale and per bias of a kernel when the run's tables are loaded
struct SbrRunPhase {
    void* out;
    const void* s;          // entries from n_phase on: kernel 0's, fetched and ignored
    const void* b;
};
struct SbrRunArgs {
    const void* x;
    unsigned n;
    unsigned inner;
    unsigned channels;
    unsigned x_slot;        // x holds the address of a pointer-table slot
    int n_phase;
    unsigned stores;        // bit i: kernel i's output is stored
    unsigned slots;         // bit i / 16 + i: kernel i's scale / bias is a pointer-table slot
    unsigned reserved;
    SbrRunPhase ph[kSbrRunMax];
};

// A run of bf16 add / mul / GELU kernels, each over a tensor of its own length from memory, whose second operand (add, mul) is the
// head of what the kernel before wrote, repeated with a short period: one dispatch.  The head of the run's last output
// is also set aside for the run behind it, which cannot read it from the buffer while other workgroups overwrite that.
constexpr int kCarryRunMax = 8;             // kernels per run
constexpr int kCarryMax = 512;              // elements of a carry (two per lane of a workgroup); a power of two from 8 on
struct CarryPhase {
    void* out;
    const void* in0;
    unsigned n;
    // elements of the output that later kernels, of this run or behind it, overwrite before anything reads them from memory: not stored.  Kernels
    // of the run write multiples of 8, so what two of them store never overlaps.  A kernel behind the run may write any number and cut a
    // vector: that one is stored whole, and overwritten by a later dispatch.
    unsigned cover;
    unsigned op;
    unsigned ind;           // bit 0: in0 is a pointer-table slot
    unsigned from;          // the first kernel whose head this kernel's carry depends on: the last GELU before it, or kernel 0
    unsigned reserved;
};
struct CarryRunArgs {
    const void* carry_in;   // the first kernel's second operand, or null
    void* carry_out;        // where the last kernel's head is set aside, or null
    unsigned m;             // the period
    unsigned flags;         // bit 0: carry_in is a pointer-table slot
    int n_phase;
    unsigned reserved;
    unsigned unit0[kCarryRunMax];   // the workgroup that takes kernel i's first unit; entries from n_phase on: no workgroup's index
    CarryPhase ph[kCarryRunMax];
};

struct Launch {
    const void* fn = nullptr;        // host-side kernel handle
    hipFunction_t mod_fn = nullptr;  // the same kernel as a module function, resolved on first launch
    unsigned arg_bytes = 0;          // size of the kernel's argument block
    dim3 grid{1, 1, 1};
    dim3 block{1, 1, 1};
    unsigned gemm_row_groups = 0;    // GEMV on the matrix cores: goes into GemvArgs::row_groups (0 = other kernels); k_gemm_rows: tiles of rows | (65536 / tiles, rounded up) << 8
    const void* fn_beyond_cache = nullptr;      // ... and the kernel that takes its weights by non-temporal loads, where the chain settles that (settle_weights)
};

// The memory-side cache: weights of a chain beyond it come from memory in every iteration, where non-temporal loads of them can be the
// faster ones; weights within it are found there again, unless they were loaded that way.
constexpr long long kCacheBytes = 256ll << 20;
inline void settle_weights(Launch* l, long long chain_weight_bytes) {
    if (l->fn_beyond_cache && chain_weight_bytes > kCacheBytes) l->fn = l->fn_beyond_cache;
}

struct Shape {
    long long n = 0, m = 0, rows = 1, cols = 0, inner = 0;
};

// Kernel instantiation and launch shape for (op, dtype, mask of indirected operands, shape).  The
// choice depends on the shape alone, never on the mask or on pointer values, so the direct and the
// indirect form of a kernel run the same schedule.  False if there is no such kernel.
bool plan(int op, int dtype, int ind_mask, const Shape& shape, Launch* out);
bool plan_gemv(int dtype, int ind_mask, int rows, int n, int cols, Launch* out);    // its part for kGemv (gemv.hip)
const void* copy_kernel();
const void* table_kernel();
// Can this kernel be part of a merged dispatch?  From op, dtype and shape alone.  On success *n_out is
// the number of elements it produces (all kernels of a run must agree on it and on the dtype).
// whole_vectors: fp32 tensors must be a whole number of 16-byte vectors (runs of one workgroup per unit; a GEMV's
// epilogue works element by element and takes any n).
bool merge_candidate(int op, int dtype, const Shape& shape, bool whole_vectors, long long* n_out);
// Runs over small fp32 tensors work one element (4 bytes) per lane instead of a 16-byte vector: such
// kernels are bound by their dispatch, not by bytes, and one element per lane is what lets the fp32 GELU
// (evaluated in fp64, about 65 instructions) ride along.  No RMSNorm in such a run (its row is a unit
// of 256 lanes x 16 bytes).
constexpr long long kMergeNarrowMax = 16384;        // elements
bool merge_narrow(int dtype, long long n);
// bf16 runs without an RMSNorm up to this many elements work on 4 bytes (two elements) per lane as well: a lane's elements
// are worked out one after the other, and such a tensor makes few waves.
constexpr long long kNarrowBf16Max = 1ll << 19;
// Chains (ChainArgs) of either type stay on 4 bytes a lane up to here (64 kernels, us per iteration with 4 / 16 bytes: bf16 700001 elements
// 47 / 68, 2^20 53 / 59, 2^21 88 / 88, 2^22 174 / 172; fp32, whose GELUs have dispatches of their own, 2^18 100 / 118, 2^20 198 / 231,
// 2^21 458 / 424).
constexpr long long kNarrowChainMax = 1ll << 20;
int merge_max_phases(int dtype, long long n);
const void* merged_kernel(int dtype, bool narrow, int phases);
const void* chain_kernel(int dtype, bool narrow, int phases);
// Can this kernel be part of a run with a carry (its operands aside)?  And the kernel for a run whose longest kernel has n elements;
// *unit: the elements a workgroup takes.
bool carry_run_candidate(int op, int dtype, long long n);
void plan_carry_run(long long n, Launch* out, unsigned* unit);
// Can this scale + bias + ReLU kernel be part of a run of such kernels?  A 16-byte vector may touch two channels at
// most, the tables of all channels fit the run's LDS, and element indices fit 32 bits.
bool sbr_run_candidate(int dtype, long long n, long long inner, long long channels);
bool plan_sbr_run(int dtype, long long n, long long inner, Launch* out);
// Is this a GEMV shape an epilogue form exists for?  bf16: up to 4 rows of h of 8 to 8192 columns (k_gemv_rows;
// beyond 2048 columns only for n >= 1024), 5 rows and more of 8 columns and more (the matrix-core forms).
// *n_out = rows * n.
bool merge_head(int op, int dtype, const Shape& shape, long long* n_out);
// ... and does it also take the RMSNorm in front?  While the grid is small enough (gemv.hip); the matrix-core forms up to 2048
// columns, and up to kPrologueMaxRows rows:
// two tiles of 16 rows, one per workgroup, fill the 256 CUs once at 2048 columns; beyond, two workgroups share a CU and each
// normalises its tile, which costs more than the dispatch it saves (decode chain at 48 rows: 1261 -> 1336 us).
constexpr int kPrologueMaxRows = 32;
bool merge_prologue(const Shape& shape);
// The epilogue form for a GEMV of such a shape.
void plan_gemv_epilogue(const Shape& shape, bool with_prologue, Launch* out);

}  // namespace pgk
