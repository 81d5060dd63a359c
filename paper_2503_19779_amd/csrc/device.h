// device.h -- device-side helpers shared by the kernel files: storage formats, vector loads and stores,
// the wave64 reduction, the elementwise operations.  gfx950 only.
#pragma once

#include "kernels.h"

#include <cstddef>

namespace pgk {
namespace {

constexpr int kBlock = 256;   // threads per workgroup = 4 waves of 64

#define PG_GLOBAL __attribute__((address_space(1)))
#define PG_CONSTANT __attribute__((address_space(4)))

// ---- operand resolution -------------------------------------------------------------------
template <bool IND>
__device__ __forceinline__ const void* resolve(const void* p) {
    if constexpr (IND) {
        // uniform address: one scalar load.  What a slot holds is a tensor in global memory; saying so lets the
        // compiler use global loads where it would otherwise fall back to generic ones (which also count as LDS operations)
        return (const void*)(const void PG_GLOBAL*)*reinterpret_cast<const uintptr_t*>(p);
    } else {
        return p;
    }
}

__device__ __forceinline__ bool aligned_to(const void* p, unsigned bytes) {
    return (reinterpret_cast<uintptr_t>(p) & (bytes - 1u)) == 0;
}

// ---- storage formats ------------------------------------------------------------------------
// Two fp32 values to a packed pair of bf16: round to nearest, ties to even, NaN stays a quiet NaN.
// One gfx950 conversion instruction instead of a dozen integer ones: these kernels are latency
// bound, every instruction on the path from the last load to the store counts.
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned pack2_bf16(float lo, float hi) {
    v2f x;
    x.x = lo;
    x.y = hi;
    return __builtin_bit_cast(unsigned, __builtin_convertvector(x, v2bf));
}
__device__ __forceinline__ unsigned f32_to_bf16(float f) { return pack2_bf16(f, 0.f) & 0xffffu; }

typedef unsigned short bf16_t;

// A "vector" is VB bytes (16 or 4) = NV elements, carried in NW 32-bit words.
template <typename T, int VB> struct Vec;
template <int VB> struct Vec<float, VB> {
    static constexpr int NV = VB / 4, NW = VB / 4;
    static __device__ __forceinline__ void unpack(const unsigned* w, float* f) {
#pragma unroll
        for (int i = 0; i < NV; i++) f[i] = __uint_as_float(w[i]);
    }
    static __device__ __forceinline__ void pack(const float* f, unsigned* w) {
#pragma unroll
        for (int i = 0; i < NV; i++) w[i] = __float_as_uint(f[i]);
    }
};
template <int VB> struct Vec<bf16_t, VB> {
    static constexpr int NV = VB / 2, NW = VB / 4;
    static __device__ __forceinline__ void unpack(const unsigned* w, float* f) {
#pragma unroll
        for (int i = 0; i < NW; i++) {
            f[2 * i] = __uint_as_float(w[i] << 16);
            f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
        }
    }
    static __device__ __forceinline__ void pack(const float* f, unsigned* w) {
#pragma unroll
        for (int i = 0; i < NW; i++) w[i] = pack2_bf16(f[2 * i], f[2 * i + 1]);
    }
};

__device__ __forceinline__ unsigned load_raw(const float* p) { return *reinterpret_cast<const unsigned*>(p); }
__device__ __forceinline__ unsigned load_raw(const bf16_t* p) { return *p; }
template <typename T> __device__ __forceinline__ float from_raw(unsigned r) {
    return __uint_as_float(sizeof(T) == 4 ? r : r << 16);
}
__device__ __forceinline__ float load_elem(const float* p) { return *p; }
__device__ __forceinline__ float load_elem(const bf16_t* p) { return __uint_as_float((unsigned)*p << 16); }
__device__ __forceinline__ void store_elem(float* p, float v) { *p = v; }
__device__ __forceinline__ void store_elem(bf16_t* p, float v) { *p = (bf16_t)f32_to_bf16(v); }

typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Fetch one vector of VB bytes as words.  AL: the address is VB-aligned; otherwise the same bytes
// arrive through element-sized loads (a tensor is always element aligned).  Loads only: nothing here
// consumes the data, so a caller can issue many of these before the first wait.
template <typename T, int VB, bool AL, bool NT = false>
__device__ __forceinline__ void load_vec(const T* p, unsigned* w) {
    constexpr int NW = VB / 4;
    if constexpr (AL) {
        if constexpr (VB == 16) {
            v4u t;
            if constexpr (NT) t = __builtin_nontemporal_load(reinterpret_cast<const v4u*>(p));
            else t = *reinterpret_cast<const v4u*>(p);
            w[0] = t.x; w[1] = t.y; w[2] = t.z; w[3] = t.w;
        } else {
            w[0] = *reinterpret_cast<const unsigned*>(p);
        }
    } else if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int i = 0; i < NW; i++) w[i] = reinterpret_cast<const unsigned*>(p)[i];
    } else {
#pragma unroll
        for (int i = 0; i < NW; i++)
            w[i] = (unsigned)reinterpret_cast<const unsigned short*>(p)[2 * i] |
                   ((unsigned)reinterpret_cast<const unsigned short*>(p)[2 * i + 1] << 16);
    }
}

// Through a pointer that says "global memory" outright.  A tensor address that reached the
// kernel through a pointer-table slot or a run-time choice is a generic pointer to the compiler; generic
// loads are slower and are counted as LDS operations as well, so a wait for LDS would wait for them too.
template <typename T>
__device__ __forceinline__ unsigned load_raw_global(const T* p) {
    if constexpr (sizeof(T) == 4) return *(const unsigned PG_GLOBAL*)(uintptr_t)p;
    else return *(const unsigned short PG_GLOBAL*)(uintptr_t)p;
}
// Element i of a tensor whose address is the same in every lane: the address stays in scalar registers and
// the load takes the lane's offset beside it, with no vector arithmetic on 64-bit addresses.
template <typename T>
__device__ __forceinline__ unsigned load_raw_global_at(const T* base, unsigned i) {
    if constexpr (sizeof(T) == 4) return ((const unsigned PG_GLOBAL*)(uintptr_t)base)[i];
    else return ((const unsigned short PG_GLOBAL*)(uintptr_t)base)[i];
}
__device__ __forceinline__ void store_vec_global(void* p, const unsigned* w) {
    v4u t;
    t.x = w[0]; t.y = w[1]; t.z = w[2]; t.w = w[3];
    *(v4u PG_GLOBAL*)(uintptr_t)p = t;
}
// 16 bytes at any element boundary: one load or store instruction all the same
typedef v4u v4u_any __attribute__((aligned(2)));
typedef unsigned u32_any __attribute__((aligned(2)));      // and 4
// A pointer-table slot, or the tensor address itself: decided at run time (the merged kernels; the
// stand-alone ones decide at compile time, resolve<IND>).  The slot is read as constant memory -- nothing
// writes the table while a graph runs -- which makes it a scalar load that no vector-memory wait covers.
__device__ __forceinline__ const void* resolve_rt(const void* p, unsigned is_slot) {
    return is_slot ? *(const void* const PG_CONSTANT*)(uintptr_t)p : p;
}

// Rows of `cols` elements in 16-byte vectors: nfull = cols / NV full vectors, then (RAGGED shapes
// only) one partial vector.  Fetching is split in two so that all loads of a kernel can be in flight
// together: row_vec_issue loads vector min(v, nfull-1) -- always inside the row, no branch -- and
// row_vec_finish unpacks it, zeroes it if v lies beyond the full vectors, and reads the partial
// vector's elements one by one.
template <typename T, bool AL, bool NT = false>
__device__ __forceinline__ void row_vec_issue(const T* row, int nfull, int v, unsigned* w) {
    constexpr int NV = Vec<T, 16>::NV;
    const int vc = v < nfull ? v : nfull - 1;
    load_vec<T, 16, AL, NT>(row + (size_t)vc * NV, w);
}
// Words of vector v after the fact: zero beyond the full vectors, and (RAGGED) the partial vector
// read element by element.
template <typename T, bool RAGGED>
__device__ __forceinline__ void row_vec_fix(const T* row, int cols, int nfull, int v, unsigned* w) {
    constexpr int NV = Vec<T, 16>::NV;
    if (v >= nfull) {
#pragma unroll
        for (int i = 0; i < 4; i++) w[i] = 0u;
        if constexpr (RAGGED) {
            if (v == nfull) {
                const int left = cols - nfull * NV;
#pragma unroll
                for (int i = 0; i < NV; i++) {
                    if (i < left) {
                        const unsigned r = load_raw(row + (size_t)nfull * NV + i);
                        if constexpr (sizeof(T) == 4) w[i] = r;
                        else w[i / 2] |= r << (16 * (i & 1));
                    }
                }
            }
        }
    }
}
template <typename T, bool RAGGED>
__device__ __forceinline__ void row_vec_finish(const T* row, int cols, int nfull, int v, unsigned* w, float* f) {
    row_vec_fix<T, RAGGED>(row, cols, nfull, v, w);
    Vec<T, 16>::unpack(w, f);
}

// acc += sum of the products of two vectors' elements, in element order.  bf16: one packed
// two-element dot product (fp32 accumulate) per word; fp32: one fused multiply-add per element.
template <typename T>
__device__ __forceinline__ float dot_acc(const unsigned* a, const unsigned* b, float acc) {
    if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int i = 0; i < 4; i++) acc = __builtin_fmaf(__uint_as_float(a[i]), __uint_as_float(b[i]), acc);
    } else {
#pragma unroll
        for (int i = 0; i < 4; i++)
            acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(v2bf, a[i]), __builtin_bit_cast(v2bf, b[i]), acc, false);
    }
    return acc;
}

template <int VB>
__device__ __forceinline__ void store_vec(void* p, const unsigned* w) {
    if constexpr (VB == 16) {
        v4u t;
        t.x = w[0]; t.y = w[1]; t.z = w[2]; t.w = w[3];
        *reinterpret_cast<v4u*>(p) = t;
    } else {
        *reinterpret_cast<unsigned*>(p) = w[0];
    }
}

// ---- wave64 reduction -----------------------------------------------------------------------
// Butterfly over the 16 lanes of a DPP row, then the four row sums are read out and added in a
// fixed order.  Every lane performs the same additions on the same values, so all lanes hold the
// same bits.  Needs all 64 lanes active.
template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
    int t = __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false);
    return v + __int_as_float(t);
}
__device__ __forceinline__ float wave_sum(float v) {
    v = dpp_add<0xB1>(v);    // quad_perm [1,0,3,2]: lane ^ 1
    v = dpp_add<0x4E>(v);    // quad_perm [2,3,0,1]: lane ^ 2
    v = dpp_add<0x141>(v);   // row_half_mirror: the other quad of each 8
    v = dpp_add<0x140>(v);   // row_mirror: the other half of each 16
    float r0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0));
    float r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 16));
    float r2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 32));
    float r3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 48));
    return ((r0 + r1) + r2) + r3;
}

// N sums at once, each the same additions in the same shape as wave_sum (the same bits).  The first two steps of
// the butterfly hand over one value for every value kept, so that the later steps carry one value per lane instead
// of N: about 17 instructions for four sums where four wave_sums take 44.  Lane l returns the sum sums_index<N>(l);
// the mirrored steps reach lanes whose index bits are flipped, hence the flip in every other quad.
template <int N>
__device__ __forceinline__ int sums_index(int lane) {
    const int i4 = (lane ^ ((lane & 4) ? 3 : 0)) & 3;
    return N == 1 ? 0 : N == 2 ? (i4 & 1) : N <= 4 ? i4 : i4 + (lane & 4);
}
constexpr int sums_lanes(int n) { return n == 1 ? 1 : n == 2 ? 2 : n <= 4 ? 4 : 8; }   // lanes 0 .. that - 1 hold every sum once
template <int CTRL>
__device__ __forceinline__ float dpp_take(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float sum_rows(float v) {       // ((row 0 + row 1) + row 2) + row 3 of the four DPP rows, in every lane
    const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    const auto a = __builtin_amdgcn_permlane16_swap(h[0], h[0], false, false), b = __builtin_amdgcn_permlane16_swap(h[1], h[1], false, false);
    return ((__uint_as_float(a[0]) + __uint_as_float(a[1])) + __uint_as_float(b[0])) + __uint_as_float(b[1]);
}
template <int N>
__device__ __forceinline__ float wave_sums(const float* s, int lane) {
    static_assert(N >= 2 && N <= 8, "two to eight sums");
    const bool odd = sums_index<2>(lane) != 0, high = (sums_index<4>(lane) & 2) != 0;
    auto four = [&](float s0, float s1, float s2, float s3, bool two_only) {
        const float r01 = (odd ? s1 : s0) + dpp_take<0xB1>(odd ? s0 : s1);
        float v;
        if (two_only) {
            v = r01 + dpp_take<0x4E>(r01);
        } else {
            const float r23 = (odd ? s3 : s2) + dpp_take<0xB1>(odd ? s2 : s3);
            v = (high ? r23 : r01) + dpp_take<0x4E>(high ? r01 : r23);
        }
        v += dpp_take<0x141>(v);
        v += dpp_take<0x140>(v);
        return sum_rows(v);
    };
    const float lo = four(s[0], s[1], N > 2 ? s[N > 2 ? 2 : 0] : 0.f, N > 3 ? s[N > 3 ? 3 : 0] : 0.f, N == 2);
    if constexpr (N <= 4) {
        return lo;
    } else {
        const float hi = four(s[4], N > 5 ? s[N > 5 ? 5 : 0] : 0.f, N > 6 ? s[N > 6 ? 6 : 0] : 0.f, N > 7 ? s[N > 7 ? 7 : 0] : 0.f, false);
        return (lane & 4) ? hi : lo;
    }
}

// Workgroup barrier for an exchange through LDS only: waits for this wave's LDS operations, not for its
// outstanding global stores (which __syncthreads would, at about a microsecond apiece).
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// ---- elementwise ----------------------------------------------------------------------------
// GELU(a) = a * Phi(a) with Phi(a) = erfc(-a / sqrt 2) / 2 (keeps relative accuracy in the left
// tail).  For fp32 tensors it is evaluated in fp64 and rounded once (gelu_f32 below): an fp32 erfc is a few ulp off,
// and a chain of multiplies and cancelling adds amplifies that beyond 1e-5.  For bf16 tensors fp32
// is far more than the 8 stored bits need, and the library erfcf (a few hundred instructions over
// several branches, which a wave of mixed values all takes) made large GELU kernels ALU-bound at a
// quarter of the HBM rate; gelu_bf16 below is branch-free and about 40 instructions.
//
// erfc(z), z >= 0, as (1 - u) * exp(-z^2 + u * Q(u)) with u = z / (2 + z) in [0, 1): the exponent's
// second term is log(erfc(z) exp(z^2) (1 + z/2)), smooth in u and zero at u = 0, so that erfc(0) = 1
// comes out exactly and tiny inputs give a/2 exactly.  Q: degree 9, a Chebyshev fit on z <= 9.7
// (beyond, a * Phi(a) is below the smallest normal number), max error 8e-9 in the exponent.  z^2 is
// taken with its rounding error (one fma), the exponential as 2^k * exp2(r) with |r| <= 0.51 after a
// two-constant reduction, so the relative error stays near 2e-7 into the tail.  Checked against the
// fp64 definition on every finite bf16 input: the bf16 result is the correctly rounded one for all
// of them (the closest any exact value comes to a rounding boundary is 8e-7, at a = -0.336).
__device__ __forceinline__ float gelu_bf16(float a) {
    const float x = a * -0.70710678118654752440f;
    const float z = __builtin_fminf(__builtin_fabsf(x), 14.0f);      // erfc(14) = 0 in fp32; keeps z * z finite (and a NaN out of the exponent)
    const float u = z * __builtin_amdgcn_rcpf(2.0f + z);
    const float t = 1.0f - u;
    float p = -0.153892517f;
    p = __builtin_fmaf(p, u, 0.49560681f);
    p = __builtin_fmaf(p, u, -0.509543419f);
    p = __builtin_fmaf(p, u, 0.182105958f);
    p = __builtin_fmaf(p, u, -0.144903973f);
    p = __builtin_fmaf(p, u, 0.072065711f);
    p = __builtin_fmaf(p, u, 0.19142893f);
    p = __builtin_fmaf(p, u, 0.161542267f);
    p = __builtin_fmaf(p, u, -0.303239733f);
    p = __builtin_fmaf(p, u, -1.25675833f);
    p = p * u;
    const float s = z * z, e = __builtin_fmaf(z, z, -s);               // z^2 = s + e exactly
    constexpr float kLog2e = 1.4426950408889634f, kLn2Hi = 0.693145751953125f, kLn2Lo = 1.42860682030941723212e-6f;
    const float kf = __builtin_rintf((p - s) * kLog2e);
    float r = __builtin_fmaf(kf, -kLn2Hi, -s);
    r = r + p;
    r = r - e;
    r = __builtin_fmaf(kf, -kLn2Lo, r);
    const float v = __builtin_ldexpf(t * __builtin_amdgcn_exp2f(r * kLog2e), (int)kf);
    const float erfc_x = x < 0.f ? 2.0f - v : v;
    return (0.5f * a) * erfc_x;      // a NaN comes back through this product; -inf * 0 = NaN as in the definition
}

// The same form in fp64 for fp32 tensors, with what the rounding of z would cost taken out: z^2 = a^2 / 2 is exact (a has 24 bits), 1 - u
// keeps its rounding error, exp(r) enters as exp(r) - 1.  Q of degree 22 in the centred variable s = 2 u / u(10.4) - 1 (a
// Chebyshev fit on z <= 10.4, beyond which the result rounds to zero whatever Q is), its even and odd terms in two chains;
// exp(r) - 1 on |r| <= 0.352 by a fit of degree 11.  The fp64 result is within 7.1e-16 of a * Phi(a), relative, for every a > -14.3
// (1.5e-16 in the mean below -6, 2.7e-16 at most above -0.1); the formula with the library's erfc at a rounded z, several branches that a
// wave of mixed values takes one after the other, is within 5.5e-16 about zero and 3.2e-14 towards -14.3.  Of the 580 million
// fp32 inputs of 5e-10 <= |a| < 14.5 one result is not the correctly rounded one (two with that formula).  About 65 instructions,
// no branch.
__device__ __forceinline__ float gelu_f32(float a) {
    const double d = (double)a;
    const double z = __builtin_fmin(__builtin_fabs(d) * 0.70710678118654752440, 10.4);
    const double w = 2.0 + z, w_lo = z - (w - 2.0);                    // 2 + z = w + w_lo exactly
    double y = __builtin_amdgcn_rcp(w);
    y = __builtin_fma(__builtin_fma(-w, y, 1.0), y, y);
    y = __builtin_fma(__builtin_fma(-w, y, 1.0), y, y);
    const double t = 2.0 * y, t_lo = y * __builtin_fma(-w_lo, t, __builtin_fma(-w, t, 2.0));      // 1 - u = t + t_lo
    const double u = z * y, s = __builtin_fma(u, 2.3846153846153846, -1.0), s2 = s * s;
    double pe = 6.096496283622283e-10;
    pe = __builtin_fma(pe, s2, -4.3704153493283935e-09);
    pe = __builtin_fma(pe, s2, -1.41491445058183e-09);
    pe = __builtin_fma(pe, s2, 1.9394376933458417e-07);
    pe = __builtin_fma(pe, s2, -1.4974665463589925e-06);
    pe = __builtin_fma(pe, s2, 6.261681705770192e-06);
    pe = __builtin_fma(pe, s2, -1.0497636139937293e-05);
    pe = __builtin_fma(pe, s2, -7.345319204153287e-05);
    pe = __builtin_fma(pe, s2, 0.0009401958958586842);
    pe = __builtin_fma(pe, s2, -0.007581680008508557);
    pe = __builtin_fma(pe, s2, 0.06684199270480724);
    pe = __builtin_fma(pe, s2, -1.3408074426393273);
    double po = 1.3835186521888504e-09;
    po = __builtin_fma(po, s2, -1.8127755043420434e-08);
    po = __builtin_fma(po, s2, 1.0624132699881106e-07);
    po = __builtin_fma(po, s2, -2.5500292430170833e-07);
    po = __builtin_fma(po, s2, -1.095015580580727e-06);
    po = __builtin_fma(po, s2, 1.542531630549678e-05);
    po = __builtin_fma(po, s2, -9.697377010041972e-05);
    po = __builtin_fma(po, s2, 0.00044017709978370716);
    po = __builtin_fma(po, s2, -0.0015871845088182162);
    po = __builtin_fma(po, s2, 0.004735528189346559);
    po = __builtin_fma(po, s2, -0.02743330950618046);
    const double p = __builtin_fma(po, s, pe) * u;
    const double q = __builtin_fmin(0.5 * d * d, 1100.0);              // z^2, exact: a has 24 bits
    constexpr double kLog2e = 1.4426950408889634, kLn2Hi = 0x1.62e42fefa0000p-1, kLn2Lo = 1.6465949582897082e-12;
    const double kf = __builtin_rint((p - q) * kLog2e);
    double r = __builtin_fma(kf, -kLn2Hi, -q);
    r = r + p;
    r = __builtin_fma(kf, -kLn2Lo, r);
    double ex = 2.5096918075802424e-08;
    ex = __builtin_fma(ex, r, 2.761557975513923e-07);
    ex = __builtin_fma(ex, r, 2.7557277571635357e-06);
    ex = __builtin_fma(ex, r, 2.480153314383674e-05);
    ex = __builtin_fma(ex, r, 0.0001984126985560737);
    ex = __builtin_fma(ex, r, 0.0013888888907531355);
    ex = __builtin_fma(ex, r, 0.008333333333332001);
    ex = __builtin_fma(ex, r, 0.041666666666649345);
    ex = __builtin_fma(ex, r, 0.16666666666666666);
    ex = __builtin_fma(ex, r, 0.5);
    const double em1 = __builtin_fma(r * r, ex, r);                    // exp(r) - 1
    const double v = __builtin_ldexp(t + __builtin_fma(t, em1, t_lo), (int)kf);
    return (float)((0.5 * d) * (d > 0.0 ? 2.0 - v : v));
}

template <int OP, bool WIDE>
__device__ __forceinline__ float ew_apply(float a, float b) {
    if constexpr (OP == kAdd) {
        return a + b;
    } else if constexpr (OP == kMul) {
        return a * b;
    } else if constexpr (WIDE) {
        return gelu_f32(a);
    } else {
        return gelu_bf16(a);
    }
}

// ---- host side ------------------------------------------------------------------------------
#define PG_FN(...) reinterpret_cast<const void*>(&__VA_ARGS__)

inline unsigned blocks_for(long long n, long long per_block) {
    const long long g = (n + per_block - 1) / per_block;
    return (unsigned)(g < 1 ? 1 : g);
}

}  // namespace
}  // namespace pgk
