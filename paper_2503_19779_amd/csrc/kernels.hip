// kernels.hip -- the chain's device code for gfx950 (wave64) except the GEMV (gemv.hip): elementwise
// add / mul / GELU, RMSNorm, per-channel scale + bias + ReLU, the batched multi-tensor copy and the
// pointer-table writer.
//
// Every compute kernel exists in a direct form (operands are tensor addresses) and in indirect
// forms (an operand is the address of a pointer-table slot that the kernel dereferences first;
// paper, Sec. 3 "Parameter Indirection" and Sec. 4 "Kernel generation": the body is unchanged,
// only a dereference prologue is added).  All forms of a kernel are instantiations of one body
// with one launch shape, so every replay mode computes bit-identical results.
//
// The chain's kernels are short (a few microseconds), so their cost is latency, not throughput:
// each shape class gets its own small instantiation (picked on the host from the shape alone, never
// from a pointer value), all loads are issued before the first use, and work is spread over lanes
// rather than looped inside one.  A misaligned external tensor changes only how a 16-byte vector is
// fetched (element loads instead of one vector load), never which lane adds what in which order, so
// results do not depend on alignment either.
//
// The translation unit is built with -ffp-contract=off: fused multiply-adds appear only where
// written.
#include "device.h"

namespace pgk {
namespace {

// ---- elementwise ----------------------------------------------------------------------------
// Each lane owns U vectors of VB bytes, 256 lanes apart; one block also does the n % NV trailing
// elements.  `o` may alias `a` (in place): a lane reads what it later overwrites.  AL: a (and b,
// when it is read by vectors) are VB-aligned.
// `bid`: the index of the block of 256 lanes this call plays (blockIdx.x in the stand-alone kernel).
template <typename T, int OP, int VB, int U, typename IdxT, bool AL>
__device__ __forceinline__ void ew_body(const T* a, const T* b, T* o, IdxT n, IdxT m, bool b_vec, unsigned bid) {
    using V = Vec<T, VB>;
    constexpr int NV = V::NV, NW = V::NW;
    constexpr bool kBinary = (OP != kGelu);
    constexpr bool kWide = sizeof(T) == 4;
    const IdxT nvec = n / NV;
    const IdxT base = (IdxT)bid * (kBlock * U) + threadIdx.x;
    unsigned wa[U][NW], wb[U][NW], rb[U][NV];
#pragma unroll
    for (int u = 0; u < U; u++) {
        const IdxT v = base + (IdxT)u * kBlock;
        if (v < nvec) {
            load_vec<T, VB, AL>(a + v * NV, wa[u]);
            if constexpr (kBinary) {
                const IdxT i0 = v * NV;
                if (b_vec) {
                    load_vec<T, VB, AL>(b + ((m == n) ? i0 : i0 % m), wb[u]);
                } else {
#pragma unroll
                    for (int e = 0; e < NV; e++) rb[u][e] = load_raw(b + (i0 + e) % m);
                }
            }
        }
    }
#pragma unroll
    for (int u = 0; u < U; u++) {
        const IdxT v = base + (IdxT)u * kBlock;
        if (v < nvec) {
            float fa[NV], fb[NV], fo[NV];
            unsigned wo[NW];
            V::unpack(wa[u], fa);
            if constexpr (kBinary) {
                if (b_vec) V::unpack(wb[u], fb);
                else
#pragma unroll
                    for (int e = 0; e < NV; e++) fb[e] = from_raw<T>(rb[u][e]);
            }
#pragma unroll
            for (int e = 0; e < NV; e++) fo[e] = ew_apply<OP, kWide>(fa[e], kBinary ? fb[e] : 0.f);
            V::pack(fo, wo);
            store_vec<VB>(o + v * NV, wo);
        }
    }
    if constexpr (NV > 1) {
        if (bid == nvec / (kBlock * U)) {   // the block that would own vector index nvec
            const IdxT i = nvec * NV + threadIdx.x;
            if (threadIdx.x < NV && i < n) {
                const float fb1 = kBinary ? load_elem(b + (i % m)) : 0.f;
                store_elem(o + i, ew_apply<OP, kWide>(load_elem(a + i), fb1));
            }
        }
    }
}

template <typename T, int OP, int IND, int VB, int U, typename IdxT>
__global__ __launch_bounds__(kBlock) void k_elementwise(EwArgs p) {
    constexpr bool kBinary = (OP != kGelu);
    constexpr int NV = Vec<T, VB>::NV;
    const T* a = static_cast<const T*>(resolve<(IND & 1) != 0>(p.a));
    const T* b = kBinary ? static_cast<const T*>(resolve<(IND & 2) != 0>(p.b)) : nullptr;
    T* o = static_cast<T*>(p.out);
    const IdxT n = (IdxT)p.n, m = (IdxT)p.m;
    const bool b_vec = kBinary && (m % NV) == 0;      // then a vector of b never wraps around the period
    const bool al = aligned_to(a, VB) && (!b_vec || aligned_to(b, VB));
    if (__builtin_expect(al, 1)) ew_body<T, OP, VB, U, IdxT, true>(a, b, o, n, m, b_vec, blockIdx.x);
    else ew_body<T, OP, VB, U, IdxT, false>(a, b, o, n, m, b_vec, blockIdx.x);
}

// ---- per-channel scale + bias + ReLU on [N, C, inner] ---------------------------------------
__device__ __forceinline__ float sbr_apply(float x, float s, float b) {
    const float v = __builtin_fmaf(x, s, b);
    return v > 0.f ? v : 0.f;
}

// VEC: inner is a multiple of the 16-byte vector, so a vector never straddles two channels.
template <typename T, bool VEC, int U, typename IdxT, bool AL>
__device__ __forceinline__ void sbr_body(const T* x, const T* s, const T* b, T* o, IdxT n, unsigned inner, unsigned channels) {
    using V = Vec<T, 16>;
    constexpr int NV = VEC ? V::NV : 1;
    const IdxT nvec = n / NV;      // n is a multiple of inner, hence of NV
    const IdxT base = (IdxT)blockIdx.x * (kBlock * U) + threadIdx.x;
    unsigned wx[U][4], rs[U], rbv[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
        const IdxT v = base + (IdxT)u * kBlock;
        if (v < nvec) {
            if constexpr (VEC) load_vec<T, 16, AL>(x + v * NV, wx[u]);
            else wx[u][0] = load_raw(x + v);
            const unsigned c = (unsigned)(((v * NV) / inner) % channels);
            rs[u] = load_raw(s + c);
            rbv[u] = load_raw(b + c);
        }
    }
#pragma unroll
    for (int u = 0; u < U; u++) {
        const IdxT v = base + (IdxT)u * kBlock;
        if (v < nvec) {
            const float fs = from_raw<T>(rs[u]), fb = from_raw<T>(rbv[u]);
            if constexpr (VEC) {
                float fx[V::NV], fo[V::NV];
                unsigned wo[V::NW];
                V::unpack(wx[u], fx);
#pragma unroll
                for (int e = 0; e < V::NV; e++) fo[e] = sbr_apply(fx[e], fs, fb);
                V::pack(fo, wo);
                store_vec<16>(o + v * NV, wo);
            } else {
                store_elem(o + v, sbr_apply(from_raw<T>(wx[u][0]), fs, fb));
            }
        }
    }
}

template <typename T, int IND, bool VEC, int U, typename IdxT>
__global__ __launch_bounds__(kBlock) void k_scale_bias_relu(SbrArgs p) {
    const T* x = static_cast<const T*>(resolve<(IND & 1) != 0>(p.x));
    const T* s = static_cast<const T*>(resolve<(IND & 2) != 0>(p.s));
    const T* b = static_cast<const T*>(resolve<(IND & 4) != 0>(p.b));
    T* o = static_cast<T*>(p.out);
    if (!VEC || aligned_to(x, 16)) sbr_body<T, VEC, U, IdxT, true>(x, s, b, o, (IdxT)p.n, p.inner, p.channels);
    else sbr_body<T, VEC, U, IdxT, false>(x, s, b, o, (IdxT)p.n, p.inner, p.channels);
}

// A run of such kernels in one dispatch (kernels.h, SbrRunArgs).  What bounds it is memory: kernel by kernel every one
// reads and writes the whole tensor; here x comes in once, the elements stay in registers, and what goes out is what is read
// later.  The scales and biases of all kernels and channels are laid out in LDS first, LDS[kernel][channel] = scale,
// [channels + channel] = bias, one load per lane and kernel: the pointers in batches of eight kernels, all values in flight together, in
// front of x (asked for kernel by kernel, a pointer, its value and a wait at a time, they took longer than x: ten of them about 10 us).  A
// wave has one stretch of the tensor, which mostly lies in one channel or two: two scales and biases per kernel for the whole
// wave, and no division per vector.  Same fused multiply-add, same rounding per kernel.
// WHOLE: inner is a multiple of the 16-byte vector.  Otherwise a vector may straddle two channels (inner >= NV, so
// never three) and the last vector of the tensor may be a partial one.  Vectors are fetched at any element boundary.
// us per iteration, values asked for one by one / together / together and by stretches: 40 fp32 kernels over [32, 64, 112, 112] in four segments
// 192 / 148 / 146 (6.3 TB/s: one read and one write per segment, two in the last), 20 over [32, 64, 111, 111] in two 122 / 95 / 81, 24 over
// [16, 33, 77, 101] in three 44 / 33 / 27.  Two vectors per lane: with four 147, 83, 27, with eight 150, 87, 29.  Non-temporal loads of x lose, 158:
// the memory-side cache holds much of what the segment before wrote; non-temporal stores change nothing.
template <typename T, bool WHOLE, int U>
__global__ __launch_bounds__(kBlock) void k_sbr_run(SbrRunArgs p) {
    using V = Vec<T, 16>;
    constexpr int NV = V::NV;
    constexpr int kHalf = kSbrRunMax / 2, kTab = 2 * kSbrRunMaxChannels;
    __shared__ float tab[kSbrRunMax * kTab];
    using SlotPtr = const void* const PG_CONSTANT*;
    const void PG_CONSTANT* const ka = (const void PG_CONSTANT*)__builtin_amdgcn_kernarg_segment_ptr();      // a readable address for a load whose result is not used
    const unsigned tid = threadIdx.x;
    const unsigned n = p.n, inner = p.inner, C = p.channels, slots = p.slots, stores = p.stores;
    const int np = p.n_phase;
    const T* x = static_cast<const T*>(resolve_rt(p.x, p.x_slot));
    // lane t < 2 C: the scale (t < C) or bias of channel t % C, eight kernels' pointers at a time, then their values, without a wait between them
    const bool is_b = tid >= C && tid < 2 * C;
    const unsigned c = tid < C ? tid : is_b ? tid - C : 0u;
    unsigned raw[kSbrRunMax];
    auto ask = [&](auto half) {
        constexpr int at = decltype(half)::value * kHalf;
        const void* sp[kHalf];
        const void* bp[kHalf];
#pragma unroll
        for (int i = 0; i < kHalf; i++) { sp[i] = p.ph[at + i].s; bp[i] = p.ph[at + i].b; }
        static_assert(kHalf == 8, "the batches name every kernel");
        asm volatile("" : "+s"(sp[0]), "+s"(sp[1]), "+s"(sp[2]), "+s"(sp[3]), "+s"(sp[4]), "+s"(sp[5]), "+s"(sp[6]), "+s"(sp[7]),
                          "+s"(bp[0]), "+s"(bp[1]), "+s"(bp[2]), "+s"(bp[3]), "+s"(bp[4]), "+s"(bp[5]), "+s"(bp[6]), "+s"(bp[7]));
        if (slots) {
            auto through = [&](const void* (&q)[kHalf], unsigned mask) {
                const void* t[kHalf];
#pragma unroll
                for (int i = 0; i < kHalf; i++) t[i] = *(((mask >> i) & 1u) ? (SlotPtr)(uintptr_t)q[i] : (SlotPtr)ka);
                asm volatile("" : "+s"(t[0]), "+s"(t[1]), "+s"(t[2]), "+s"(t[3]), "+s"(t[4]), "+s"(t[5]), "+s"(t[6]), "+s"(t[7]));
#pragma unroll
                for (int i = 0; i < kHalf; i++) if ((mask >> i) & 1u) q[i] = t[i];
            };
            through(sp, slots >> at);
            through(bp, slots >> (16 + at));
        }
#pragma unroll
        for (int i = 0; i < kHalf; i++) raw[at + i] = load_raw_global(static_cast<const T*>(is_b ? bp[i] : sp[i]) + c);
    };
    ask(std::integral_constant<int, 0>{});
    if (np > kHalf) ask(std::integral_constant<int, 1>{});
    const unsigned nfull = n / NV, left = n - nfull * NV;         // nfull >= 1: inner is a vector at least
    // a wave's vectors are one stretch of U * 64
    const unsigned wave0 = blockIdx.x * (unsigned)(kBlock * U) + (unsigned)__builtin_amdgcn_readfirstlane(tid >> 6) * (unsigned)(64 * U), v0 = wave0 + (tid & 63);
    unsigned w[U][4];
#pragma unroll
    for (int u = 0; u < U; u++) {
        const unsigned v = v0 + (unsigned)u * 64;
        const v4u t = *(const v4u_any PG_GLOBAL*)(uintptr_t)(x + (size_t)(v < nfull ? v : nfull - 1) * NV);
        w[u][0] = t.x; w[u][1] = t.y; w[u][2] = t.z; w[u][3] = t.w;
    }
    __builtin_amdgcn_sched_barrier(0);
    if (tid < 2 * C) {                   // the values are in before x is: loads come back in order
#pragma unroll
        for (int i = 0; i < kHalf; i++) tab[i * kTab + tid] = from_raw<T>(raw[i]);
        if (np > kHalf)
#pragma unroll
            for (int i = kHalf; i < kSbrRunMax; i++) tab[i * kTab + tid] = from_raw<T>(raw[i]);
    }
    lds_barrier();
    if constexpr (!WHOLE) {
        if (left && wave0 <= nfull && nfull < wave0 + 64 * U) {          // the tensor's last, partial vector
#pragma unroll
            for (int u = 0; u < U; u++)
                if (v0 + (unsigned)u * 64 == nfull) {
#pragma unroll
                    for (int k = 0; k < 4; k++) w[u][k] = 0u;
#pragma unroll
                    for (int e = 0; e < NV - 1; e++)
                        if ((unsigned)e < left) {
                            const unsigned r = load_raw_global(x + (size_t)nfull * NV + e);
                            if constexpr (sizeof(T) == 4) w[u][e] = r;
                            else w[u][e / 2] |= r << (16 * (e & 1));
                        }
                }
        }
    }
    // the stretch's first and last element
    const unsigned ea = wave0 * NV < n ? wave0 * NV : n - 1, ez = n - ea > (unsigned)(64 * U * NV) ? ea + (unsigned)(64 * U * NV) - 1 : n - 1;
    const unsigned qa = ea / inner, ca = qa % C, edge = (qa + 1) * inner;             // its first channel, and where that ends (n is a multiple of inner)
    // the kernels, one after the other; `apply` has the scales and biases of each
    auto play = [&](auto&& apply) {
#pragma unroll 1
        for (int i = 0; i < np; i++) {
            apply(tab + i * kTab);
            if ((stores >> i) & 1u) {
                T* const o = static_cast<T*>(p.ph[i].out);
#pragma unroll
                for (int u = 0; u < U; u++) {
                    const unsigned v = v0 + (unsigned)u * 64;
                    if (v < nfull) {
                        store_vec_global(o + (size_t)v0 * NV + u * 64 * NV, w[u]);
                    } else if (!WHOLE && v == nfull) {
#pragma unroll
                        for (int e = 0; e < NV - 1; e++)
                            if ((unsigned)e < left) {
                                if constexpr (sizeof(T) == 4) *(unsigned PG_GLOBAL*)(uintptr_t)(o + (size_t)nfull * NV + e) = w[u][e];
                                else *(unsigned short PG_GLOBAL*)(uintptr_t)(o + (size_t)nfull * NV + e) = (unsigned short)(w[u][e / 2] >> (16 * (e & 1)));
                            }
                    }
                }
            }
        }
    };
    if (ez < edge) {                     // one channel
        play([&](const float* t) {
            const float s0 = t[ca], b0 = t[C + ca];
#pragma unroll
            for (int u = 0; u < U; u++) {
                float f[NV];
                V::unpack(w[u], f);
#pragma unroll
                for (int e = 0; e < NV; e++) f[e] = sbr_apply(f[e], s0, b0);
                V::pack(f, w[u]);
            }
        });
    } else if (ez - edge < inner) {      // two
        const unsigned cz = ca + 1 == C ? 0u : ca + 1;
        int first[U];                    // elements of a vector in the first one: from NV on all of them, up to 0 none
#pragma unroll
        for (int u = 0; u < U; u++) first[u] = (int)(edge - (v0 + (unsigned)u * 64) * NV);
        play([&](const float* t) {
            const float s0 = t[ca], b0 = t[C + ca], s1 = t[cz], b1 = t[C + cz];
#pragma unroll
            for (int u = 0; u < U; u++) {
                float f[NV];
                V::unpack(w[u], f);
#pragma unroll
                for (int e = 0; e < NV; e++) {
                    const bool here = first[u] > (WHOLE ? 0 : e);
                    f[e] = sbr_apply(f[e], here ? s0 : s1, here ? b0 : b1);
                }
                V::pack(f, w[u]);
            }
        });
    } else {
        unsigned c0[U], c1[U], k0[U];       // channel of a vector's first elements, of the others, and how many are the first
#pragma unroll
        for (int u = 0; u < U; u++) {
            const unsigned i0 = (v0 + (unsigned)u * 64) * NV, q = i0 / inner;
            c0[u] = q % C;
            if constexpr (!WHOLE) {
                k0[u] = inner - (i0 - q * inner);
                c1[u] = c0[u] + 1 == C ? 0u : c0[u] + 1;
            }
        }
        play([&](const float* t) {
#pragma unroll
            for (int u = 0; u < U; u++) {
                float f[NV];
                V::unpack(w[u], f);
                const float s0 = t[c0[u]], b0 = t[C + c0[u]];
                if constexpr (WHOLE) {
#pragma unroll
                    for (int e = 0; e < NV; e++) f[e] = sbr_apply(f[e], s0, b0);
                } else {
                    const float s1 = t[c1[u]], b1 = t[C + c1[u]];
#pragma unroll
                    for (int e = 0; e < NV; e++) {
                        const bool here = (unsigned)e < k0[u];
                        f[e] = sbr_apply(f[e], here ? s0 : s1, here ? b0 : b1);
                    }
                }
                V::pack(f, w[u]);
            }
        });
    }
}

// ---- RMSNorm: one workgroup per row ------------------------------------------------------------
// Each thread keeps its VPT vectors of x and of the gain in registers (all fetched up front), sums
// squares with fused multiply-adds, a wave64 shuffle reduction follows, the four wave sums are
// staged through LDS and added in a fixed order by every thread.  VPT = 0 is the long-row form: it
// loops and reads x a second time.
template <typename T, bool RAGGED>
__device__ __forceinline__ void rms_store(T* o, int cols, int nfull, int v, bool al_o, const float* fo) {
    constexpr int NV = Vec<T, 16>::NV;
    if (v < nfull && (al_o || !RAGGED)) {
        unsigned w[4];
        Vec<T, 16>::pack(fo, w);
        store_vec<16>(o + (size_t)v * NV, w);
    } else if constexpr (RAGGED) {
        const int left = cols - v * NV;
#pragma unroll
        for (int e = 0; e < NV; e++)
            if (e < left) store_elem(o + (size_t)v * NV + e, fo[e]);
    }
}

template <typename T, int VPT, bool RAGGED, bool AL>
__device__ __forceinline__ void rms_body(const T* x, const T* g, T* o, int cols, float eps, bool al_o, float* part) {
    constexpr int NV = Vec<T, 16>::NV;
    const int tid = threadIdx.x;
    const int nfull = cols / NV;
    float acc = 0.f;
    if constexpr (VPT > 0) {
        unsigned wx[VPT][4], wg[VPT][4];
        float fx[VPT][NV], fg[VPT][NV];
        if (!RAGGED || nfull > 0) {
#pragma unroll
            for (int u = 0; u < VPT; u++) {
                row_vec_issue<T, AL>(x, nfull, tid + u * kBlock, wx[u]);
                row_vec_issue<T, AL>(g, nfull, tid + u * kBlock, wg[u]);
            }
        }
#pragma unroll
        for (int u = 0; u < VPT; u++) {
            row_vec_finish<T, RAGGED>(x, cols, nfull, tid + u * kBlock, wx[u], fx[u]);
#pragma unroll
            for (int e = 0; e < NV; e++) acc = __builtin_fmaf(fx[u][e], fx[u][e], acc);
        }
        acc = wave_sum(acc);
        if ((tid & 63) == 0) part[tid >> 6] = acc;
        __syncthreads();
        const float total = ((part[0] + part[1]) + part[2]) + part[3];
        const float scale = 1.0f / sqrtf(total / (float)cols + eps);
#pragma unroll
        for (int u = 0; u < VPT; u++) {
            float fo[NV];
            row_vec_finish<T, RAGGED>(g, cols, nfull, tid + u * kBlock, wg[u], fg[u]);
#pragma unroll
            for (int e = 0; e < NV; e++) fo[e] = (fx[u][e] * scale) * fg[u][e];
            rms_store<T, RAGGED>(o, cols, nfull, tid + u * kBlock, al_o, fo);
        }
    } else {
        const int nvec = (cols + NV - 1) / NV;
        for (int v = tid; v < nvec; v += kBlock) {
            unsigned w[4];
            float f[NV];
            if (!RAGGED || nfull > 0) row_vec_issue<T, AL>(x, nfull, v, w);
            row_vec_finish<T, RAGGED>(x, cols, nfull, v, w, f);
#pragma unroll
            for (int e = 0; e < NV; e++) acc = __builtin_fmaf(f[e], f[e], acc);
        }
        acc = wave_sum(acc);
        if ((tid & 63) == 0) part[tid >> 6] = acc;
        __syncthreads();
        const float total = ((part[0] + part[1]) + part[2]) + part[3];
        const float scale = 1.0f / sqrtf(total / (float)cols + eps);
        for (int v = tid; v < nvec; v += kBlock) {
            unsigned w[4], w2[4];
            float f[NV], fgv[NV], fo[NV];
            if (!RAGGED || nfull > 0) {
                row_vec_issue<T, AL>(x, nfull, v, w);
                row_vec_issue<T, AL>(g, nfull, v, w2);
            }
            row_vec_finish<T, RAGGED>(x, cols, nfull, v, w, f);
            row_vec_finish<T, RAGGED>(g, cols, nfull, v, w2, fgv);
#pragma unroll
            for (int e = 0; e < NV; e++) fo[e] = (f[e] * scale) * fgv[e];
            rms_store<T, RAGGED>(o, cols, nfull, v, al_o, fo);
        }
    }
}

// one row by one workgroup of 256 lanes; x0 / o0: the first row
template <typename T, int VPT, bool RAGGED>
__device__ __forceinline__ void rms_row(const T* x0, const T* g, T* o0, int cols, float eps, size_t row, float* part) {
    const T* x = x0 + row * cols;
    T* o = o0 + row * cols;
    // rows of an aligned buffer stay aligned when cols is a multiple of the vector; else check this row
    const bool al = aligned_to(x, 16) && aligned_to(g, 16);
    const bool al_o = aligned_to(o, 16);
    if (__builtin_expect(al, 1)) rms_body<T, VPT, RAGGED, true>(x, g, o, cols, eps, al_o, part);
    else rms_body<T, VPT, RAGGED, false>(x, g, o, cols, eps, al_o, part);
}

template <typename T, int IND, int VPT, bool RAGGED>
__global__ __launch_bounds__(kBlock) void k_rmsnorm(RmsArgs p) {
    const T* x = static_cast<const T*>(resolve<(IND & 1) != 0>(p.x));
    const T* g = static_cast<const T*>(resolve<(IND & 2) != 0>(p.g));
    __shared__ float part[kBlock / 64];
    rms_row<T, VPT, RAGGED>(x, g, static_cast<T*>(p.out), p.cols, p.eps, blockIdx.x, part);
}

// ---- merged dispatches ------------------------------------------------------------------------------
// Same arithmetic as the stand-alone kernels, element for element: ew_apply for add / mul / GELU;
// RMSNorm as rms_body does it for a row of exactly one vector per lane (fused multiply-add sum of
// squares in element order, wave_sum, the four wave sums added in a fixed order through LDS,
// 1 / sqrt(mean + eps), (x * scale) * gain); one rounding to the storage type per kernel (pack), and
// what a later kernel of the run is handed in registers is exactly the stored bits.
// One workgroup per unit, straight-line: all operand fetches of the run first (unrolled: their registers
// need static indices; a lane beyond the tensor re-reads the last vector and never stores, so there is
// no per-lane branch and all fetches are in flight together), then ONE copy of the arithmetic in a loop
// over the kernels that picks its operands out of the fetched vectors and the register slots with
// conditional moves (one copy of the GELU and of the RMSNorm reduction for up to four kernels; an
// unrolled form with every operand choice resolved at run time by branches was slower: a taken branch
// costs a one-wave-per-SIMD kernel about as much as a dozen arithmetic instructions).
// bf16 tensors of any length: the workgroup that owns the last, partial vector fetches element by element.

template <typename T, int VB, int P, bool TAIL>
__device__ __forceinline__ void merged_body(const MergedArgs& p, const T* const* in0, const T* const* in1, float* part) {
    using V = Vec<T, VB>;
    constexpr int NV = V::NV, NW = VB / 4;
    const unsigned n = p.n, nvec = n / NV, left = n - nvec * NV;      // left: elements of a last, partial vector
    // TAIL: the workgroup that owns the partial vector fetches element by element (none past the end)
    auto fetch = [](const T* q, unsigned room /* elements from q to the end of the tensor */, unsigned* w) {
        if constexpr (VB == 4 && !TAIL) {
            w[0] = *(const u32_any PG_GLOBAL*)(uintptr_t)q;
        } else if constexpr (!TAIL) {
            const v4u t = *(const v4u_any PG_GLOBAL*)(uintptr_t)q;
            w[0] = t.x; w[1] = t.y; w[2] = t.z; w[3] = t.w;
        } else {
#pragma unroll
            for (int k = 0; k < NW; k++) w[k] = 0u;
#pragma unroll
            for (int e = 0; e < NV; e++) {
                const unsigned r = load_raw_global(q + ((unsigned)e < room ? (unsigned)e : room - 1));
                if constexpr (sizeof(T) == 4) w[e] = r;
                else w[e / 2] |= r << (16 * (e & 1));
            }
        }
    };
    constexpr bool kWide = sizeof(T) == 4;
    const unsigned tid = threadIdx.x;
    // the run's table, once, in scalar registers (read inside the loop below it would be indexed memory)
    T* outs[P];
    unsigned metas[P], inds[P];
    float epss[P];
#pragma unroll
    for (int i = 0; i < P; i++) {
        outs[i] = static_cast<T*>(p.ph[i].out);
        metas[i] = p.ph[i].meta;
        inds[i] = p.ph[i].ind;
        epss[i] = p.ph[i].eps;
    }
    const unsigned v = blockIdx.x * kBlock + tid;
    const bool act = v < nvec || (TAIL && v == nvec);
    const unsigned i0 = (act ? v : nvec - (nvec ? 1u : 0u)) * NV;
    const unsigned mine = TAIL && v == nvec ? left : (unsigned)NV;     // elements this lane owns
    auto put = [&](T* out, const unsigned* w) {
        if (!TAIL || mine == (unsigned)NV) {
            if constexpr (VB == 4) *(unsigned PG_GLOBAL*)(uintptr_t)(out + i0) = w[0];
            else store_vec_global(out + i0, w);
        } else {
#pragma unroll
            for (int e = 0; e < NV - 1; e++)
                if ((unsigned)e < mine) {
                    if constexpr (sizeof(T) == 4) *(unsigned PG_GLOBAL*)(uintptr_t)(out + i0 + e) = w[e];
                    else *(unsigned short PG_GLOBAL*)(uintptr_t)(out + i0 + e) = (unsigned short)(w[e / 2] >> (16 * (e & 1)));
                }
        }
    };
    unsigned ld0[P][NW], ld1[P][NW];
#pragma unroll
    for (int i = 0; i < P; i++) {
        const unsigned mt = metas[i], op = mt & 0xffu;
        if (((mt >> 8) & 0xffu) == kMergeFromMemory) {
            fetch(in0[i] + i0, n - i0, ld0[i]);
        } else {
#pragma unroll
            for (int k = 0; k < NW; k++) ld0[i][k] = 0u;
        }
        if (op != kGelu && ((mt >> 16) & 0xffu) == kMergeFromMemory) {
            const unsigned m = p.ph[i].m;
            if (op == kRmsNorm || m == n || m % NV == 0) {
                // RMSNorm: a row is one unit, lane t holds vector t of the gain; add / mul: a vector of b never wraps around the period
                const unsigned at = op == kRmsNorm ? tid * NV : (m == n ? i0 : i0 % m);
                fetch(in1[i] + at, m == n && op != kRmsNorm ? n - i0 : (unsigned)NV, ld1[i]);
            } else {
#pragma unroll
                for (int k = 0; k < NW; k++) ld1[i][k] = 0u;
#pragma unroll
                for (int e = 0; e < NV; e++) {                     // the raw bits, element by element
                    const unsigned r = load_raw_global(in1[i] + (i0 + e) % m);
                    if constexpr (sizeof(T) == 4) ld1[i][e] = r;
                    else ld1[i][e / 2] |= r << (16 * (e & 1));
                }
            }
        } else {
#pragma unroll
            for (int k = 0; k < NW; k++) ld1[i][k] = 0u;
        }
    }
    unsigned slot[kMergeSlots][NW];
#pragma unroll
    for (int q = 0; q < kMergeSlots; q++)
#pragma unroll
        for (int k = 0; k < NW; k++) slot[q][k] = 0u;
    const int n_phase = p.n_phase;
    // All fetches have been asked for together; wait for them here, once.  Left to the compiler, the wait
    // sits at the head of the loop below and then also waits, every time round, for the store of the
    // kernel before (loads and stores of a wave share one counter): a microsecond per kernel.
    __builtin_amdgcn_s_waitcnt(0x0F70);      // vmcnt(0)
#pragma unroll 1
    for (int i = 0; i < n_phase; i++) {
        // this kernel's entry of the table and its fetched operands: uniform selects, no indexing
        T* out = outs[0];
        unsigned mt = metas[0];
        unsigned ind = inds[0];
        float eps = epss[0];
        unsigned wa[NW], wb[NW], wo[NW];
#pragma unroll
        for (int k = 0; k < NW; k++) { wa[k] = ld0[0][k]; wb[k] = ld1[0][k]; }
#pragma unroll
        for (int j = 1; j < P; j++)
            if (i == j) {
                out = outs[j]; mt = metas[j]; ind = inds[j]; eps = epss[j];
#pragma unroll
                for (int k = 0; k < NW; k++) { wa[k] = ld0[j][k]; wb[k] = ld1[j][k]; }
            }
        const unsigned op = mt & 0xffu, src0 = (mt >> 8) & 0xffu, src1 = (mt >> 16) & 0xffu, dst = mt >> 24;
#pragma unroll
        for (int q = 0; q < kMergeSlots; q++) {
            if (src0 == (unsigned)q)
#pragma unroll
                for (int k = 0; k < NW; k++) wa[k] = slot[q][k];
            if (src1 == (unsigned)q)
#pragma unroll
                for (int k = 0; k < NW; k++) wb[k] = slot[q][k];
        }
        float fa[NV], fb[NV], fo[NV];
        V::unpack(wa, fa);
        V::unpack(wb, fb);
        if (VB == 16 && op == kRmsNorm) {      // a row is one unit of 256 lanes x 16 bytes: never in the narrow form
            float acc = 0.f;
#pragma unroll
            for (int e = 0; e < NV; e++) acc = __builtin_fmaf(fa[e], fa[e], acc);
            acc = wave_sum(acc);
            if ((tid & 63) == 0) part[tid >> 6] = acc;
            lds_barrier();
            const float total = ((part[0] + part[1]) + part[2]) + part[3];
            lds_barrier();                                         // `part` is free for a later RMSNorm of the run
            const float scale = 1.0f / sqrtf(total / (float)(kBlock * NV) + eps);
#pragma unroll
            for (int e = 0; e < NV; e++) fo[e] = (fa[e] * scale) * fb[e];
        } else if (op == kAdd) {
#pragma unroll
            for (int e = 0; e < NV; e++) fo[e] = ew_apply<kAdd, kWide>(fa[e], fb[e]);
        } else if (op == kMul) {
#pragma unroll
            for (int e = 0; e < NV; e++) fo[e] = ew_apply<kMul, kWide>(fa[e], fb[e]);
        } else {
            if constexpr (!kWide || VB == 4) {                     // fp32 GELU (evaluated in fp64): one element per lane only
#pragma unroll
                for (int e = 0; e < NV; e++) fo[e] = ew_apply<kGelu, kWide>(fa[e], 0.f);
            } else {
#pragma unroll
                for (int e = 0; e < NV; e++) fo[e] = fa[e];
            }
        }
        V::pack(fo, wo);
        if (act && (ind & kEpiStore)) put(out, wo);      // else it is overwritten before anything reads it from memory
#pragma unroll
        for (int q = 0; q < kMergeSlots; q++)
            if (dst == (unsigned)q)
#pragma unroll
                for (int k = 0; k < NW; k++) slot[q][k] = wo[k];
    }
}

template <typename T, int VB, int P>
__global__ __launch_bounds__(kBlock) void k_merged(MergedArgs p) {
    __shared__ float part[kBlock / 64];
    // operand addresses, once, before any store of this kernel: pointer-table slots are read with scalar loads
    const T* in0[P];
    const T* in1[P];
#pragma unroll
    for (int i = 0; i < P; i++) {
        in0[i] = in1[i] = nullptr;
        const unsigned mt = p.ph[i].meta;
        if (((mt >> 8) & 0xffu) == kMergeFromMemory) {
            in0[i] = static_cast<const T*>(resolve_rt(p.ph[i].in0, p.ph[i].ind & 1));
        }
        if ((mt & 0xffu) != kGelu && ((mt >> 16) & 0xffu) == kMergeFromMemory) {
            in1[i] = static_cast<const T*>(resolve_rt(p.ph[i].in1, p.ph[i].ind & 2));
        }
    }
    constexpr unsigned NV = Vec<T, VB>::NV;
    const bool tail = NV > 1 && p.n % NV != 0 && blockIdx.x == p.n / NV / kBlock;
    if (__builtin_expect(!tail, 1)) merged_body<T, VB, P, false>(p, in0, in1, part);
    else if constexpr (NV > 1) merged_body<T, VB, P, true>(p, in0, in1, part);
}

// A run that is a chain (kernels.h, ChainArgs).  At these sizes it is bound by its dispatch and by what a lane does in sequence: the trip
// for the arguments, the one for the operands, the kernels one after the other, the store.  So the arguments come in one batch, every
// operand is asked for without a branch (a GELU, which has none, fetches the first operand once more), and the choice between the
// GELU and add / mul is all there is to decide per kernel.  Against the same run played by k_merged, whose table has a branch per operand
// (64 kernels, us per iteration): 4096 fp32 elements 54 -> 43, 100003 bf16 elements 52 -> 31 (154 with a dispatch per kernel), 2^23
// 326 -> 304.
template <typename T, int VB, int P, bool TAIL>
__device__ __forceinline__ void chain_body(const T* in0, const T* const* in1, const unsigned* ms, unsigned n, bool periods, unsigned ops, T* const* outs) {
    using V = Vec<T, VB>;
    constexpr int NV = V::NV, NW = VB / 4;
    constexpr bool kWide = sizeof(T) == 4;
    const unsigned v = blockIdx.x * kBlock + threadIdx.x, nvec = n / NV, left = n - nvec * NV;     // left: elements of a last, partial vector
    const unsigned mine = v < nvec ? (unsigned)NV : (TAIL && v == nvec) ? left : 0u;               // elements this lane owns
    const unsigned i0 = (mine ? v : nvec - (nvec ? 1u : 0u)) * NV;
    // NV elements of q from element `at` on, `room` of which there are; TAIL: one by one, none past the end
    auto fetch = [](const T* q, unsigned at, unsigned room, unsigned* w) {
        if constexpr (!TAIL) {
            if constexpr (VB == 4) {
                w[0] = *(const u32_any PG_GLOBAL*)((const T PG_GLOBAL*)(uintptr_t)q + at);
            } else {
                const v4u t = *(const v4u_any PG_GLOBAL*)((const T PG_GLOBAL*)(uintptr_t)q + at);
                w[0] = t.x; w[1] = t.y; w[2] = t.z; w[3] = t.w;
            }
        } else {
#pragma unroll
            for (int k = 0; k < NW; k++) w[k] = 0u;
#pragma unroll
            for (int e = 0; e < NV; e++) {
                const unsigned r = load_raw_global_at(q, at + ((unsigned)e < room ? (unsigned)e : room - 1));
                if constexpr (sizeof(T) == 4) w[e] = r;
                else w[e / 2] |= r << (16 * (e & 1));
            }
        }
    };
    unsigned w[NW], ld[P][NW];
    fetch(in0, i0, n - i0, w);
    if (__builtin_expect(!periods, 1)) {
#pragma unroll
        for (int i = 0; i < P; i++) fetch(in1[i], i0, n - i0, ld[i]);
    } else {
#pragma unroll
        for (int i = 0; i < P; i++) {
            const unsigned m = ms[i];
            if (m == n) {
                fetch(in1[i], i0, n - i0, ld[i]);
            } else if (m % NV == 0) {                              // a vector never wraps around the period
                fetch(in1[i], i0 % m, NV, ld[i]);
            } else {
#pragma unroll
                for (int k = 0; k < NW; k++) ld[i][k] = 0u;
#pragma unroll
                for (int e = 0; e < NV; e++) {
                    const unsigned r = load_raw_global_at(in1[i], (i0 + e) % m);
                    if constexpr (sizeof(T) == 4) ld[i][e] = r;
                    else ld[i][e / 2] |= r << (16 * (e & 1));
                }
            }
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);      // vmcnt(0): all operands here, once; a wait behind a store would wait for the store as well
#pragma unroll
    for (int i = 0; i < P; i++) {
        const unsigned op = (ops >> (4 * i)) & 7u;
        if (op == kChainEnd) break;
        float fa[NV], fb[NV], fo[NV];
        V::unpack(w, fa);
        V::unpack(ld[i], fb);
        if (op == (unsigned)kGelu) {
            if constexpr (!kWide || VB == 4) {
#pragma unroll
                for (int e = 0; e < NV; e++) fo[e] = ew_apply<kGelu, kWide>(fa[e], 0.f);
            } else {
#pragma unroll
                for (int e = 0; e < NV; e++) fo[e] = fa[e];      // never planned: the fp32 GELU rides only one element per lane
            }
        } else {
#pragma unroll
            for (int e = 0; e < NV; e++) {
                const float sum = ew_apply<kAdd, kWide>(fa[e], fb[e]), prod = ew_apply<kMul, kWide>(fa[e], fb[e]);
                fo[e] = op == (unsigned)kAdd ? sum : prod;
            }
        }
        V::pack(fo, w);
        if ((ops >> (4 * i)) & 8u) {                               // else it is overwritten before anything reads it from memory
            if (mine == (unsigned)NV) {
                if constexpr (VB == 4) ((unsigned PG_GLOBAL*)(uintptr_t)outs[i])[v] = w[0];
                else ((v4u PG_GLOBAL*)(uintptr_t)outs[i])[v] = v4u{w[0], w[1], w[2], w[3]};
            } else if constexpr (TAIL) {
#pragma unroll
                for (int e = 0; e < NV - 1; e++)
                    if ((unsigned)e < mine) {
                        if constexpr (sizeof(T) == 4) ((unsigned PG_GLOBAL*)(uintptr_t)outs[i])[i0 + e] = w[e];
                        else ((unsigned short PG_GLOBAL*)(uintptr_t)outs[i])[i0 + e] = (unsigned short)(w[e / 2] >> (16 * (e & 1)));
                    }
            }
        }
    }
}

template <typename T, int VB, int P>
__global__ __launch_bounds__(kBlock) void k_chain(ChainArgs p) {
    using SlotPtr = const void* const PG_CONSTANT*;
    const void PG_CONSTANT* const ka = (const void PG_CONSTANT*)__builtin_amdgcn_kernarg_segment_ptr();      // a readable address for a load whose result is not used
    const void* a0 = p.in0;
    const unsigned n = p.n, slots = p.slots, ops = p.ops;
    const void* a1[P];
    T* outs[P];
    unsigned ms[P];
#pragma unroll
    for (int i = 0; i < P; i++) { a1[i] = p.ph[i].in1; outs[i] = static_cast<T*>(p.ph[i].out); ms[i] = p.m[i]; }
#pragma unroll
    for (int i = 0; i < P; i += 4)
        asm volatile("" : "+s"(a0), "+s"(a1[i]), "+s"(a1[i + 1]), "+s"(a1[i + 2]), "+s"(a1[i + 3]), "+s"(outs[i]), "+s"(outs[i + 1]), "+s"(outs[i + 2]), "+s"(outs[i + 3]),
                          "+s"(ms[i]), "+s"(ms[i + 1]), "+s"(ms[i + 2]), "+s"(ms[i + 3]));
    if (slots & ~kChainPeriods) {            // some operand is a pointer-table slot: all in one batch, without branches
        const void* t1[P];
        SlotPtr at0 = ((slots >> kMergeMaxPhases) & 1u) ? (SlotPtr)(uintptr_t)a0 : (SlotPtr)ka;
        const void* t0 = *at0;
#pragma unroll
        for (int i = 0; i < P; i++) t1[i] = *(((slots >> i) & 1u) ? (SlotPtr)(uintptr_t)a1[i] : (SlotPtr)ka);
#pragma unroll
        for (int i = 0; i < P; i += 4) asm volatile("" : "+s"(t0), "+s"(t1[i]), "+s"(t1[i + 1]), "+s"(t1[i + 2]), "+s"(t1[i + 3]));
        if ((slots >> kMergeMaxPhases) & 1u) a0 = t0;
#pragma unroll
        for (int i = 0; i < P; i++) if ((slots >> i) & 1u) a1[i] = t1[i];
    }
    const T* in1[P];
#pragma unroll
    for (int i = 0; i < P; i++) in1[i] = static_cast<const T*>(a1[i]);
    constexpr unsigned NV = Vec<T, VB>::NV;
    const bool tail = NV > 1 && n % NV != 0 && blockIdx.x == n / NV / kBlock;
    if (__builtin_expect(!tail, 1)) chain_body<T, VB, P, false>(static_cast<const T*>(a0), in1, ms, n, slots & kChainPeriods, ops, outs);
    else if constexpr (NV > 1) chain_body<T, VB, P, true>(static_cast<const T*>(a0), in1, ms, n, slots & kChainPeriods, ops, outs);
}

// ---- runs of kernels that hand on a short carry ---------------------------------------------------------------
// kernels.h, CarryRunArgs.  What bounds the kernels one by one is their dispatch (3 us a kernel, of which 1.5 the graph's
// node), since all that makes one wait for the next is the head of its output, m <= 512 elements.  Here a workgroup plays
// one unit of one kernel (a vector of VB bytes per lane) and works the heads it needs out for itself, two elements a lane, from
// the last GELU before its kernel on: a GELU takes no carry, so nothing before it matters.  No workgroup needs another's results, and
// the units of all kernels of the run are in flight side by side.  Where two kernels write the same place only the later one
// stores (cover), so the order the units run in does not matter.  Same arithmetic, one rounding per kernel.
// What bounds it: a run of short tensors the trip for the arguments, the pointers, the elements (2.8 us with the node); of long ones
// the same and then memory, 14 MB in and 1 MB out on the mean of 32 runs in 7.5 us.  Non-temporal loads and stores: nothing is read twice, and what is left dirty in L2
// would be written back at the end of the dispatch.  256 tensors of 1 KB to 16 MB through the pointer table, us per iteration:
// with a workgroup that played all eight kernels on its stretch of elements, one after the other, 443 (its low units, which every
// kernel has, were the critical path); a unit of one kernel 294; non-temporal 264; without the stores that nothing reads 240.  96 tensors up to 1 MB 79 -> 46.
__device__ __forceinline__ float carry_apply(unsigned op, float a, float b) {
    if (op == (unsigned)kGelu) return ew_apply<kGelu, false>(a, 0.f);
    const float sum = ew_apply<kAdd, false>(a, b), prod = ew_apply<kMul, false>(a, b);
    return op == (unsigned)kAdd ? sum : prod;
}
template <int VB>
__global__ __launch_bounds__(kBlock) void k_carry_run(CarryRunArgs p) {
    using V = Vec<bf16_t, VB>;
    constexpr int NV = V::NV, NW = V::NW;
    constexpr int P = kCarryRunMax;
    __shared__ __attribute__((aligned(16))) unsigned carry[kCarryMax / 2];      // what this workgroup's kernel takes
    using SlotPtr = const void* const PG_CONSTANT*;
    const CarryRunArgs PG_CONSTANT* const ka = (const CarryRunArgs PG_CONSTANT*)__builtin_amdgcn_kernarg_segment_ptr();
    const unsigned tid = threadIdx.x, m = p.m;
    int k = 0;                                             // this workgroup's kernel
#pragma unroll
    for (int j = 1; j < P; j++) k += blockIdx.x >= p.unit0[j] ? 1 : 0;
    auto operand = [&](int j) {
        const void* q = ka->ph[j].in0;
        if (ka->ph[j].ind & 1u) q = *(SlotPtr)(uintptr_t)q;
        return static_cast<const bf16_t*>(q);
    };
    auto head_of = [&](const bf16_t* q) { return load_raw_global(q + 2 * tid) | (load_raw_global(q + 2 * tid + 1) << 16); };
    const unsigned op = ka->ph[k].op, nvec = ka->ph[k].n / NV;
    const unsigned v = (blockIdx.x - ka->unit0[k]) * (unsigned)kBlock + tid;
    const bf16_t PG_GLOBAL* const in = (const bf16_t PG_GLOBAL*)(uintptr_t)operand(k);
    const int from = op == (unsigned)kGelu ? k : (int)ka->ph[k].from;
    // the heads first: loads come back in order
    const bool chain = 2 * tid < m;
    unsigned hd[P - 1], c = 0u;
#pragma unroll
    for (int t = 0; t < P - 1; t++) {
        if (from + t >= k) break;
        const bf16_t* q = operand(from + t);
        hd[t] = chain ? head_of(q) : 0u;                   // a kernel whose head is handed on has m elements at least
    }
    if (op != (unsigned)kGelu && from == 0 && p.carry_in && chain)
        c = head_of(static_cast<const bf16_t*>((p.flags & 1u) ? *(SlotPtr)(uintptr_t)p.carry_in : p.carry_in));
    unsigned w[NW];
    const size_t at = (size_t)(v < nvec ? v : nvec - 1) * NV;
    if constexpr (VB == 16) {
        const v4u t = __builtin_nontemporal_load((const v4u_any PG_GLOBAL*)(in + at));
        w[0] = t.x; w[1] = t.y; w[2] = t.z; w[3] = t.w;
    } else {
        w[0] = *(const u32_any PG_GLOBAL*)(in + at);
    }
    float fa[NV], fo[NV];
    if (op == (unsigned)kGelu) {
        V::unpack(w, fa);
#pragma unroll
        for (int e = 0; e < NV; e++) fo[e] = ew_apply<kGelu, false>(fa[e], 0.f);
    } else {
#pragma unroll
        for (int t = 0; t < P - 1; t++) {
            if (from + t >= k) break;
            const unsigned o = ka->ph[from + t].op;
            c = pack2_bf16(carry_apply(o, __uint_as_float(hd[t] << 16), __uint_as_float(c << 16)),
                           carry_apply(o, __uint_as_float(hd[t] & 0xffff0000u), __uint_as_float(c & 0xffff0000u)));
        }
        if (chain) carry[tid] = c;
        lds_barrier();
        const unsigned cv = (tid % (m / NV)) * NW;         // this lane's vector of the carry: a unit is a whole number of periods
        unsigned wb[NW];
        float fb[NV];
#pragma unroll
        for (int i = 0; i < NW; i++) wb[i] = carry[cv + i];
        V::unpack(w, fa);
        V::unpack(wb, fb);
#pragma unroll
        for (int e = 0; e < NV; e++) {
            const float sum = ew_apply<kAdd, false>(fa[e], fb[e]), prod = ew_apply<kMul, false>(fa[e], fb[e]);
            fo[e] = op == (unsigned)kAdd ? sum : prod;
        }
    }
    unsigned wo[NW];
    V::pack(fo, wo);
    auto put = [&](void* q) {
        if constexpr (VB == 16) __builtin_nontemporal_store(v4u{wo[0], wo[1], wo[2], wo[3]}, (v4u PG_GLOBAL*)(uintptr_t)q + v);
        else *((unsigned PG_GLOBAL*)(uintptr_t)q + v) = wo[0];
    };
    // below `cover` the output is overwritten before anything reads it from memory; rounded down to a vector (kernels.h)
    if (v < nvec && v >= ka->ph[k].cover / NV) put(ka->ph[k].out);
    if (k == p.n_phase - 1 && p.carry_out && v * NV < m) put(p.carry_out);
}

// ---- batched multi-tensor copy -----------------------------------------------------------------
// One workgroup per chunk (<= kCopyChunkBytes of one tensor): every lane issues its two 128-bit
// non-temporal loads, then its two stores, and the workgroup is done -- measured on the log-uniform
// size mix, many short-lived workgroups with two vectors in flight per lane beat fewer, longer ones
// (6.2 against 5.2 TB/s).  Destinations are placeholders the library laid out itself (256-byte
// aligned, chunk offsets multiples of the chunk size), so only the source alignment varies: sources
// that are not 16-byte aligned fall back to 4-byte or 2-byte moves.
constexpr int kCopyUnroll = 2;
static_assert(kCopyChunkBytes == kBlock * kCopyUnroll * 16, "one pass of the workgroup covers one chunk");

__global__ __launch_bounds__(kBlock) void k_copy(CopyArgs p) {
    const CopyChunk c = p.chunks[blockIdx.x];
    const CopyTensor t = p.tensors[c.tensor];
    const char* __restrict__ src = static_cast<const char*>(p.src[c.tensor - p.src_base]) + c.off;
    char* __restrict__ dst = static_cast<char*>(t.dst) + c.off;
    const unsigned len = c.len;
    const unsigned tid = threadIdx.x;
    if ((reinterpret_cast<uintptr_t>(src) & 15u) == 0) {
        const v4u* s16 = reinterpret_cast<const v4u*>(src);
        v4u* d16 = reinterpret_cast<v4u*>(dst);
        const unsigned nvec = len >> 4;
        for (unsigned v0 = 0; v0 < nvec; v0 += kBlock * kCopyUnroll) {
            v4u r[kCopyUnroll];
#pragma unroll
            for (int u = 0; u < kCopyUnroll; u++) {
                const unsigned v = v0 + u * kBlock + tid;
                if (v < nvec) r[u] = __builtin_nontemporal_load(s16 + v);
            }
#pragma unroll
            for (int u = 0; u < kCopyUnroll; u++) {
                const unsigned v = v0 + u * kBlock + tid;
                if (v < nvec) __builtin_nontemporal_store(r[u], d16 + v);
            }
        }
        const unsigned i = (nvec << 4) + tid;
        if (i < len) dst[i] = src[i];
    } else if ((reinterpret_cast<uintptr_t>(src) & 3u) == 0) {
        const unsigned* s4 = reinterpret_cast<const unsigned*>(src);
        unsigned* d4 = reinterpret_cast<unsigned*>(dst);
        const unsigned nw = len >> 2;
        for (unsigned v = tid; v < nw; v += kBlock) d4[v] = s4[v];
        const unsigned i = (nw << 2) + tid;
        if (i < len) dst[i] = src[i];
    } else {
        // tensors are aligned to their element size, so a source that is not 4-byte aligned holds
        // 2-byte elements and has an even length
        const unsigned short* s2 = reinterpret_cast<const unsigned short*>(src);
        unsigned short* d2 = reinterpret_cast<unsigned short*>(dst);
        const unsigned nh = len >> 1;
        for (unsigned v = tid; v < nh; v += kBlock) d2[v] = s2[v];
    }
}

// ---- pointer-table writer ------------------------------------------------------------------------
__global__ __launch_bounds__(64) void k_table_write(TableArgs p) {
    for (int i = threadIdx.x; i < p.n; i += 64) p.table[p.base + i] = p.ptr[i];
}

// ---- host side: pick the instantiation and the launch shape from the kernel's shape alone ----------
template <typename T, int OP, int VB, int U, typename IdxT>
const void* ew_by_ind(int ind) {
    switch (ind) {
    case 0: return PG_FN(k_elementwise<T, OP, 0, VB, U, IdxT>);
    case 1: return PG_FN(k_elementwise<T, OP, 1, VB, U, IdxT>);
    case 2: if constexpr (OP != kGelu) return PG_FN(k_elementwise<T, OP, 2, VB, U, IdxT>); else return nullptr;
    case 3: if constexpr (OP != kGelu) return PG_FN(k_elementwise<T, OP, 3, VB, U, IdxT>); else return nullptr;
    default: return nullptr;
    }
}

// Shape classes: (4-byte vectors, 1 per lane) for small GELUs, whose cost is the arithmetic a lane
// does in sequence; (16-byte, 1 per lane) for short tensors; (16-byte, 4 per lane) for long ones,
// with 64-bit indices beyond 2^31 elements.
template <typename T, int OP>
bool plan_ew_t(int ind, long long n, Launch* out) {
    constexpr int NV16 = 16 / (int)sizeof(T), NV4 = 4 / (int)sizeof(T);
    const long long bytes = n * (long long)sizeof(T);
    const bool narrow = OP == kGelu && n <= (1ll << 20);
    out->block = dim3(kBlock);
    if (narrow) {
        out->fn = ew_by_ind<T, OP, 4, 1, unsigned>(ind);
        out->grid = dim3(blocks_for(n, (long long)kBlock * NV4));
    } else if (bytes <= (4ll << 20)) {
        out->fn = ew_by_ind<T, OP, 16, 1, unsigned>(ind);
        out->grid = dim3(blocks_for(n, (long long)kBlock * NV16));
    } else if (n < (1ll << 31)) {
        out->fn = ew_by_ind<T, OP, 16, 4, unsigned>(ind);
        out->grid = dim3(blocks_for(n, (long long)kBlock * 4 * NV16));
    } else {
        out->fn = ew_by_ind<T, OP, 16, 4, unsigned long long>(ind);
        out->grid = dim3(blocks_for(n, (long long)kBlock * 4 * NV16));
    }
    return out->fn != nullptr;
}

template <typename T>
bool plan_ew(int op, int ind, long long n, Launch* out) {
    switch (op) {
    case kAdd: return plan_ew_t<T, kAdd>(ind, n, out);
    case kMul: return plan_ew_t<T, kMul>(ind, n, out);
    case kGelu: return plan_ew_t<T, kGelu>(ind, n, out);
    default: return false;
    }
}

template <typename T, int VPT, bool RAGGED>
const void* rms_by_ind(int ind) {
    switch (ind) {
    case 0: return PG_FN(k_rmsnorm<T, 0, VPT, RAGGED>);
    case 1: return PG_FN(k_rmsnorm<T, 1, VPT, RAGGED>);
    case 2: return PG_FN(k_rmsnorm<T, 2, VPT, RAGGED>);
    case 3: return PG_FN(k_rmsnorm<T, 3, VPT, RAGGED>);
    default: return nullptr;
    }
}

template <typename T>
bool plan_rms(int ind, int rows, int cols, Launch* out) {
    constexpr int NV = 16 / (int)sizeof(T);
    const int nvec = (cols + NV - 1) / NV;
    const bool ragged = (cols % NV) != 0;
    if (nvec <= kBlock) out->fn = ragged ? rms_by_ind<T, 1, true>(ind) : rms_by_ind<T, 1, false>(ind);
    else if (nvec <= 4 * kBlock) out->fn = ragged ? rms_by_ind<T, 4, true>(ind) : rms_by_ind<T, 4, false>(ind);
    else out->fn = ragged ? rms_by_ind<T, 0, true>(ind) : rms_by_ind<T, 0, false>(ind);
    out->grid = dim3((unsigned)rows);
    out->block = dim3(kBlock);
    return out->fn != nullptr;
}

template <typename T, bool VEC, int U, typename IdxT>
const void* sbr_by_ind(int ind) {
    switch (ind) {
    case 0: return PG_FN(k_scale_bias_relu<T, 0, VEC, U, IdxT>);
    case 1: return PG_FN(k_scale_bias_relu<T, 1, VEC, U, IdxT>);
    case 2: return PG_FN(k_scale_bias_relu<T, 2, VEC, U, IdxT>);
    case 3: return PG_FN(k_scale_bias_relu<T, 3, VEC, U, IdxT>);
    case 4: return PG_FN(k_scale_bias_relu<T, 4, VEC, U, IdxT>);
    case 5: return PG_FN(k_scale_bias_relu<T, 5, VEC, U, IdxT>);
    case 6: return PG_FN(k_scale_bias_relu<T, 6, VEC, U, IdxT>);
    case 7: return PG_FN(k_scale_bias_relu<T, 7, VEC, U, IdxT>);
    default: return nullptr;
    }
}

template <typename T>
bool plan_sbr(int ind, long long n, long long inner, Launch* out) {
    constexpr int NV = 16 / (int)sizeof(T);
    const bool vec = (inner % NV) == 0;
    const long long units = vec ? n / NV : n;
    out->block = dim3(kBlock);
    if (n >= (1ll << 31)) {
        out->fn = vec ? sbr_by_ind<T, true, 4, unsigned long long>(ind) : sbr_by_ind<T, false, 4, unsigned long long>(ind);
        out->grid = dim3(blocks_for(units, kBlock * 4));
    } else if (units <= 16384) {
        out->fn = vec ? sbr_by_ind<T, true, 1, unsigned>(ind) : sbr_by_ind<T, false, 1, unsigned>(ind);
        out->grid = dim3(blocks_for(units, kBlock));
    } else {
        out->fn = vec ? sbr_by_ind<T, true, 4, unsigned>(ind) : sbr_by_ind<T, false, 4, unsigned>(ind);
        out->grid = dim3(blocks_for(units, kBlock * 4));
    }
    return out->fn != nullptr;
}

template <typename T>
bool plan_t(int op, int ind, const Shape& s, Launch* out) {
    switch (op) {
    case kAdd: case kMul: case kGelu: return plan_ew<T>(op, ind, s.n, out);
    case kRmsNorm: return plan_rms<T>(ind, (int)s.rows, (int)s.cols, out);
    case kGemv: return plan_gemv(sizeof(T) == 4 ? kF32 : kBF16, ind, (int)s.rows, (int)s.n, (int)s.cols, out);
    case kScaleBiasRelu: return plan_sbr<T>(ind, s.n, s.inner, out);
    default: return false;
    }
}

}  // namespace

bool plan(int op, int dtype, int ind_mask, const Shape& shape, Launch* out) {
    switch (op) {
    case kAdd: case kMul: case kGelu: out->arg_bytes = sizeof(EwArgs); break;
    case kRmsNorm: out->arg_bytes = sizeof(RmsArgs); break;
    case kGemv: out->arg_bytes = sizeof(GemvArgs); break;
    case kScaleBiasRelu: out->arg_bytes = sizeof(SbrArgs); break;
    default: return false;
    }
    out->mod_fn = nullptr;
    out->gemm_row_groups = 0;
    out->fn_beyond_cache = nullptr;
    if (dtype == kF32) return plan_t<float>(op, ind_mask, shape, out);
    if (dtype == kBF16) return plan_t<bf16_t>(op, ind_mask, shape, out);
    return false;
}
bool merge_candidate(int op, int dtype, const Shape& s, bool whole_vectors, long long* n_out) {
    if (dtype != kF32 && dtype != kBF16) return false;
    const int nv = dtype == kF32 ? 4 : 8;
    long long n = 0;
    if (op == kAdd || op == kMul || op == kGelu) {
        if (s.m <= 0) return false;
        n = s.n;
        // fp32 GELU is evaluated in fp64: mergeable only where the run works one element per lane (small tensors)
        if (op == kGelu && dtype == kF32 && !merge_narrow(dtype, n)) return false;
    } else if (op == kRmsNorm) {
        if (s.cols != (long long)kBlock * nv) return false;   // a row must be exactly one unit
        n = s.rows * s.cols;
    } else {
        return false;
    }
    // fp32 tensors of a ragged length beyond the narrow form's keep a dispatch per kernel
    if (n <= 0 || (whole_vectors && dtype == kF32 && !merge_narrow(dtype, n) && n % nv != 0) || n > (1ll << 31)) return false;
    *n_out = n;
    return true;
}

bool merge_narrow(int dtype, long long n) { return dtype == kF32 && n > 0 && n <= kMergeNarrowMax; }

int merge_max_phases(int dtype, long long n) { return dtype == kBF16 && n >= kMergeLongFrom && n <= kMergeLongTo ? kMergeMaxPhases : kMergeShortPhases; }

const void* merged_kernel(int dtype, bool narrow, int phases) {
    if (dtype == kF32) return narrow ? PG_FN(k_merged<float, 4, kMergeShortPhases>) : PG_FN(k_merged<float, 16, kMergeShortPhases>);
    if (dtype != kBF16) return nullptr;
    if (narrow) return phases <= kMergeShortPhases ? PG_FN(k_merged<bf16_t, 4, kMergeShortPhases>) : PG_FN(k_merged<bf16_t, 4, kMergeMaxPhases>);
    return phases <= kMergeShortPhases ? PG_FN(k_merged<bf16_t, 16, kMergeShortPhases>) : PG_FN(k_merged<bf16_t, 16, kMergeMaxPhases>);
}

const void* chain_kernel(int dtype, bool narrow, int phases) {
    const bool few = phases <= kMergeShortPhases;
    if (dtype == kF32) return narrow ? PG_FN(k_chain<float, 4, kMergeShortPhases>) : PG_FN(k_chain<float, 16, kMergeShortPhases>);
    if (dtype != kBF16) return nullptr;
    if (narrow) return few ? PG_FN(k_chain<bf16_t, 4, kMergeShortPhases>) : PG_FN(k_chain<bf16_t, 4, kMergeMaxPhases>);
    return few ? PG_FN(k_chain<bf16_t, 16, kMergeShortPhases>) : PG_FN(k_chain<bf16_t, 16, kMergeMaxPhases>);
}

bool carry_run_candidate(int op, int dtype, long long n) {
    return (op == kAdd || op == kMul || op == kGelu) && dtype == kBF16 && n > 0 && n % 8 == 0 && n < (1ll << 31);
}
// 4 bytes a lane up to the line of the element-for-element runs (200 tensors up to 2^18.5 elements: 77 us; with 16 bytes a lane above 2^16
// elements 91, above 2^13 97).
void plan_carry_run(long long n, Launch* out, unsigned* unit) {
    const bool narrow = n <= kNarrowBf16Max;
    out->arg_bytes = sizeof(CarryRunArgs);
    out->block = dim3(kBlock);
    out->fn = narrow ? PG_FN(k_carry_run<4>) : PG_FN(k_carry_run<16>);
    *unit = kBlock * (narrow ? 2u : 8u);
}

// One vector per lane until that makes four workgroups per CU, two per lane from there on.
constexpr long long kSbrRunSmall = 4ll * 256 * kBlock;
bool sbr_run_candidate(int dtype, long long n, long long inner, long long channels) {
    const int nv = dtype == kF32 ? 4 : 8;
    return (dtype == kF32 || dtype == kBF16) && n > 0 && n < (1ll << 31) && inner >= nv && channels >= 1 && channels <= kSbrRunMaxChannels;
}
template <typename T>
static void plan_sbr_run_t(long long n, long long inner, Launch* out) {
    constexpr int NV = 16 / (int)sizeof(T);
    const bool whole = inner % NV == 0;
    const long long nvec = (n + NV - 1) / NV;
    if (nvec <= kSbrRunSmall) {
        out->fn = whole ? PG_FN(k_sbr_run<T, true, 1>) : PG_FN(k_sbr_run<T, false, 1>);
        out->grid = dim3(blocks_for(nvec, kBlock));
    } else {
        out->fn = whole ? PG_FN(k_sbr_run<T, true, 2>) : PG_FN(k_sbr_run<T, false, 2>);
        out->grid = dim3(blocks_for(nvec, kBlock * 2));
    }
}
bool plan_sbr_run(int dtype, long long n, long long inner, Launch* out) {
    out->arg_bytes = sizeof(SbrRunArgs);
    out->block = dim3(kBlock);
    if (dtype == kF32) plan_sbr_run_t<float>(n, inner, out);
    else if (dtype == kBF16) plan_sbr_run_t<bf16_t>(n, inner, out);
    else return false;
    return true;
}

const void* copy_kernel() { return reinterpret_cast<const void*>(&k_copy); }
const void* table_kernel() { return reinterpret_cast<const void*>(&k_table_write); }

}  // namespace pgk
