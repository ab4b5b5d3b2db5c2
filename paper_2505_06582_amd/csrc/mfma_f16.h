// Shared by the matrix-core spectrum accumulation and its adjoint: fp16 pairs that carry an FP32
// number, operands of v_mfma_f32_16x16x32_f16, and the polynomial of the covariance's cross term
// over a 16 x 16 sub-tile of frequencies.
#pragma once

#include "gws_internal.h"

namespace gws {

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef float float2_t __attribute__((ext_vector_type(2)));

constexpr float MM_P = 56.25f;           // 7.5^2: t = u v / MM_P spans [-1, 1]
// classes of |a|: 3, 4 and 5 coefficients, 5 with c2 carried to both fp16 parts (class 6), 6 (class 7)
constexpr float MM_A3 = 0.0175f, MM_A4 = 0.08f, MM_A5 = 0.12f, MM_A6 = 0.2f, MM_A7 = 0.35f;

static __device__ __forceinline__ double frac_m(double v) { return v - floor(v); }

// D_c(nu) = k_z - 1/lambda without cancellation (the grid has no evanescent frequency).
static __device__ __forceinline__ double dprop_m(double nu2, double il) { return -nu2 / (il + sqrt(il * il - nu2)); }

// Loads through the global address space (pointers that come out of memory are otherwise flat, which
// also waits on LDS).
#define GWS_GLOBAL_AS __attribute__((address_space(1)))
static __device__ __forceinline__ float4_t load4(const void *p) { return *(const GWS_GLOBAL_AS float4_t *)(uintptr_t)p; }
static __device__ __forceinline__ float2_t load2(const void *p) { return *(const GWS_GLOBAL_AS float2_t *)(uintptr_t)p; }
// The same value, opaque to the optimiser: what is computed from it is formed where it is used
// instead of being held in registers (or spilt) across the matrix passes.
static __device__ __forceinline__ int here_v(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// A uniform value in a scalar register; the number of set bits of m below the lane.
static __device__ __forceinline__ float uniform_f(float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); }
static __device__ __forceinline__ int rank_below(uint64_t m)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
}

static __device__ __forceinline__ half2_t to_half2(float a, float b)
{
    return __builtin_convertvector((float2_t){a, b}, half2_t);
}
static __device__ __forceinline__ uint32_t bits(half2_t h) { return __builtin_bit_cast(uint32_t, h); }
// x - h for a pair: the part the second fp16 number carries (exact in FP32).  The -1 is opaque
// to the optimiser so that each is one v_fma_mix_f32 instead of a conversion and a subtraction.
static __device__ __forceinline__ float2_t rest(float re, float im, half2_t h)
{
    float m1 = -1.0f;
    asm("" : "+s"(m1));
    return (float2_t){fmaf((float)h.x, m1, re), fmaf((float)h.y, m1, im)};
}
static __device__ __forceinline__ uint32_t half_pair(float a, float b) { return bits(to_half2(a, b)); }
struct Frag {
    uint32_t r[4];
};
// The A operands of both parts of a complex product in six registers: (-Yi, Yr, Yi), two
// Gaussians to a register; the real part reads (Yr, Yi), the imaginary part (-Yi, Yr).
struct Frag6 {
    uint32_t r[6];
    __device__ __forceinline__ Frag re() const { return Frag{{r[2], r[3], r[4], r[5]}}; }
    __device__ __forceinline__ Frag im() const { return Frag{{r[0], r[1], r[2], r[3]}}; }
};
// Four complex factors as fp16 high and low parts, (r01, r23, i01, i23).
static __device__ __forceinline__ void split4(const float (&re)[4], const float (&im)[4], uint32_t *h, uint32_t *l)
{
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const half2_t hr = to_half2(re[2 * i], re[2 * i + 1]), hi = to_half2(im[2 * i], im[2 * i + 1]);
        const float2_t lr = rest(re[2 * i], re[2 * i + 1], hr), li = rest(im[2 * i], im[2 * i + 1], hi);
        h[i] = bits(hr);
        h[i + 2] = bits(hi);
        l[i] = half_pair(lr.x, lr.y);
        l[i + 2] = half_pair(li.x, li.y);
    }
}
// Half x (0: low, 1: high) of a packed pair in FP32.
static __device__ __forceinline__ float part(uint32_t p, int x)
{
    const half2_t h = __builtin_bit_cast(half2_t, p);
    return x ? (float)h.y : (float)h.x;
}
static __device__ __forceinline__ float4_t mfma16(const Frag &a, const Frag &b, float4_t c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, a), __builtin_bit_cast(half8_t, b), c, 0, 0, 0);
}
static __device__ __forceinline__ uint32_t pk_mul(uint32_t a, uint32_t b)
{
    return bits(__builtin_bit_cast(half2_t, a) * __builtin_bit_cast(half2_t, b));
}

// a of a Gaussian's cross term: beta2 in exp2 units per index^2 of the sub-tile's 7.5 x 7.5.
constexpr float MM_A_OF_BETA2 = (float)(0.6931471805599453 * 56.25);

// Class of |a| (limits above), 0 beyond the last.
static __device__ __forceinline__ int cross_class(float aa)
{
    return aa <= MM_A3 ? 3 : aa <= MM_A4 ? 4 : aa <= MM_A5 ? 5 : aa <= MM_A6 ? 6 : aa <= MM_A7 ? 7 : 0;
}

// Coefficients k0 ... k4 of exp(-a t), |t| <= 1, for a class: Taylor, with the next two orders
// projected onto the lower ones by least squares over the sub-tile's points.  Class 7 has
// k5 = 0.8 k4^2 / k3 besides (4 / 5 of k4's ratio to k3).
static __device__ __forceinline__ void cross_poly(float a, int cls, float &k0, float &k1, float &k2, float &k3, float &k4)
{
    const float a2 = a * a, a3 = a2 * a, a4 = a2 * a2;
    k0 = 1.0f;
    k1 = -a;
    k2 = 0.5f * a2;
    k3 = k4 = 0.0f;
    if (cls == 3) {
        k1 -= a3 * (0.45758f / 6.0f);
        k0 += a4 * (-0.03819f / 24.0f);
        k2 += a4 * (0.7252f / 24.0f);
    } else if (cls == 4) {
        const float a5 = a4 * a;
        k0 += a4 * (-0.03819f / 24.0f);
        k1 -= a5 * (-0.17743f / 120.0f);
        k2 += a4 * (0.7252f / 24.0f);
        k3 = -a3 * (1.0f / 6.0f) - a5 * (1.02948f / 120.0f);
    } else {
        // orders 5 and 6 projected, or 6 and 7 where order 5 has its own coefficient
        const float a6 = a3 * a3, ao = cls == 7 ? a6 * a * (1.0f / 5040.0f) : a4 * a * (1.0f / 120.0f);
        k0 += a6 * (0.01017f / 720.0f);
        k1 -= ao * (cls == 7 ? 0.0593f : -0.17743f);
        k2 += a6 * (-0.37059f / 720.0f);
        k3 = -a3 * (1.0f / 6.0f) - ao * (cls == 7 ? -0.65565f : 1.02948f);
        k4 = a4 * (1.0f / 24.0f) + a6 * (1.29584f / 720.0f);
    }
}

}  // namespace gws
