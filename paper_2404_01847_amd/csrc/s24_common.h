// Shared host/device helpers of the s24 library (argument checks, launch
// plumbing, bf16 / binary16 conversions, the activation arithmetic).  gfx950 only.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "s24.h"

#define S24_REQUIRE(cond, code) \
    do {                        \
        if (!(cond)) return (code); \
    } while (0)

static inline bool s24_aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }
static inline bool s24_valid_dtype(int dt) { return dt == S24_F32 || dt == S24_BF16 || dt == S24_F16; }
static inline bool s24_valid_gate(int g) { return g == S24_GATE_SILU || g == S24_GATE_GELU_ERF; }
static inline bool s24_valid_layout(int l) { return l == S24_ROW_MAJOR || l == S24_COL_MAJOR; }
static inline size_t s24_elem_size(int dt) { return dt == S24_F32 ? 4 : 2; }

// Compute units of the current device, read once (256 on MI355X; that figure also stands in where no device
// answers, so that the host-side checks behave the same without a GPU).
inline int s24_cu_count()
{
    static const int n = [] {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
            return v;
        return 256;
    }();
    return n;
}

// Two 64-bit words of a kernel's arguments: two addresses, an address and two numbers, or four numbers.  What a wave needs first has to be in
// scalar registers when it starts (build.py, PRELOAD_ARGUMENTS), which a structure's members are not; but the launch pays on the host for
// each argument (3.57 us with thirteen of them, 2.86 with one structure), so they travel in vectors, and what is needed last in one
// structure.  Two sliced products through ctypes: 9.5 -> 8.1 us of host time, 8.05 as two structures that were not preloaded.
typedef uint64_t s24_words __attribute__((ext_vector_type(2)));
inline s24_words s24_pack(const void *a, const void *b) { return s24_words{reinterpret_cast<uintptr_t>(a), reinterpret_cast<uintptr_t>(b)}; }
inline s24_words s24_pack(const void *a, int lo, int hi) { return s24_words{reinterpret_cast<uintptr_t>(a), (uint64_t)(uint32_t)hi << 32 | (uint32_t)lo}; }
inline s24_words s24_pack(int a, int b, int c, int d) { return s24_words{(uint64_t)(uint32_t)b << 32 | (uint32_t)a, (uint64_t)(uint32_t)d << 32 | (uint32_t)c}; }
template <typename P> __device__ __forceinline__ P *s24_global(uint64_t word) { return (P *)(__attribute__((address_space(1))) P *)word; }
__device__ __forceinline__ int s24_low(uint64_t word) { return (int)(uint32_t)word; }
__device__ __forceinline__ int s24_high(uint64_t word) { return (int)(uint32_t)(word >> 32); }

// Call after a kernel launch: turns a refused launch into S24_ERR_LAUNCH.
static inline int s24_launch_status() { return hipGetLastError() == hipSuccess ? S24_OK : S24_ERR_LAUNCH; }

__device__ __forceinline__ float s24_bf16_to_f32(uint32_t bits16) { return __uint_as_float(bits16 << 16); }

// Two fp32 values -> two bf16 in one dword (lo in bits 0..15), round to nearest even: gfx950's packed conversion,
// one instruction where the integer form (add the rounding bias, shift, merge) takes seven.  Written as the
// instruction itself so that every kernel rounds the same fp32 value to the same bits.
__device__ __forceinline__ uint32_t s24_pack_bf16x2(float lo, float hi)
{
    uint32_t d = 0;
#if defined(__HIP_DEVICE_COMPILE__)
    asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(d) : "v"(lo), "v"(hi));
#endif
    return d;
}

// fp32 -> bf16 bits, round to nearest even.
__device__ __forceinline__ uint32_t s24_f32_to_bf16(float f) { return s24_pack_bf16x2(f, f) & 0xFFFFu; }

// Sixteen bytes past the caches (non-temporal): for what a layer's step does not read again soon, namely Z and [G|U] (kept for
// the backward pass) and the weight gradients (kept for the optimizer), and for the last read of Z and [G|U].  Plain stores
// stay in the 256 MB Infinity Cache as modified lines, which push out H and dZ before the next product reads them and then cost that
// product a write to memory for each line it misses: 128 MB read after 256 MB of plain stores came in at 2.9 TB/s, after non-temporal
// ones at 6.2.  Plain stores and loads in their place and as it is, alternating on one card: a layer of 16384 x 1280 x 5120 1002 -> 965 us a
// step; 3001 x 2048 x 5504, gated, 555 -> 522; 4160 x 1600 x 6400 with pruned gradients 455 -> 430; 16384 x 4096 x 11008, gated, 8224 -> 8179, which is noise.
typedef unsigned int s24_u32x4 __attribute__((ext_vector_type(4)));
template <typename V> __device__ __forceinline__ void s24_store_stream(void *p, V v)
{
    static_assert(sizeof(V) == 16, "sixteen bytes");
    __builtin_nontemporal_store(__builtin_bit_cast(s24_u32x4, v), static_cast<s24_u32x4 *>(p));
}
__device__ __forceinline__ uint4 s24_load_stream(const void *p)
{
    return __builtin_bit_cast(uint4, __builtin_nontemporal_load(static_cast<const s24_u32x4 *>(p)));
}

// 1 / d rounded to nearest for 2^-100 <= d <= 2^100: the hardware's estimate and one Newton step on its exact residual.  Each of these
// d is compared with the division by the tests, through s24_probe_reciprocal.
__device__ __forceinline__ float s24_reciprocal(float d)
{
    const float y = __builtin_amdgcn_rcpf(d);
    return __fmaf_rn(__fmaf_rn(-d, y, 1.0f), y, y);
}

// Storage types of the kernels: uint16_t holds bf16 bits, s24_half is IEEE binary16, float is itself.
// s24_num<T> converts between 16-bit storage and the fp32 the arithmetic runs in: one value from its 16 bits,
// the low / high half of a dword, and back (round to nearest even; binary16 overflows to infinity).
typedef _Float16 s24_half;
template <typename T> struct s24_num;
template <> struct s24_num<uint16_t> {
    static __device__ __forceinline__ float widen(uint32_t bits16) { return __uint_as_float(bits16 << 16); }
    static __device__ __forceinline__ float lo(uint32_t d) { return __uint_as_float(d << 16); }
    static __device__ __forceinline__ float hi(uint32_t d) { return __uint_as_float(d & 0xFFFF0000u); }
    static __device__ __forceinline__ uint32_t narrow(float f) { return s24_f32_to_bf16(f); }
    static __device__ __forceinline__ uint32_t pack2(float a, float b) { return s24_pack_bf16x2(a, b); }
};
template <> struct s24_num<s24_half> {
    static __device__ __forceinline__ float widen(uint32_t bits16)
    {
        return (float)__builtin_bit_cast(_Float16, (uint16_t)bits16);
    }
    static __device__ __forceinline__ float lo(uint32_t d) { return widen(d & 0xFFFFu); }
    static __device__ __forceinline__ float hi(uint32_t d) { return widen(d >> 16); }
    // The conversion is pinned to the one instruction that rounds an fp32 value to binary16.  Written as a C++
    // cast the compiler merges it with the multiplication before it into a mixed-precision instruction in some
    // kernels and not in others, and the two do not always agree in the last bit; with the instruction fixed,
    // every kernel that forms the same fp32 value stores the same bits.
    static __device__ __forceinline__ uint32_t narrow(float f)
    {
        uint32_t h = 0;
#if defined(__HIP_DEVICE_COMPILE__)
        asm("v_cvt_f16_f32 %0, %1" : "=v"(h) : "v"(f));
#endif
        return h & 0xFFFFu;
    }
    static __device__ __forceinline__ uint32_t pack2(float a, float b) { return narrow(a) | (narrow(b) << 16); }
};

// silu(g) * u in fp32, shared by the stand-alone SwiGLU kernel and the GEMM epilogue that applies it
// 1 / (1 + 2^(-x log2 e)) with the hardware exponential and reciprocal (about 2 ulp in fp32, far inside what the
// bf16 or fp32 outputs of the activation kernels need; saturates to 0 and 1 for large |x|)
__device__ __forceinline__ float s24_sigmoid(float x)
{
    return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504088896341f * x));
}
__device__ __forceinline__ float s24_silu_mul(float g, float u) { return g * s24_sigmoid(g) * u; }

// backward of h = silu(g) * u for an incoming dh: dg = dh u s (1 + g (1 - s)), du = dh silu(g), s = sigmoid(g)
__device__ __forceinline__ void s24_swiglu_grad(float dh, float g, float u, float &dg, float &du)
{
    const float s = s24_sigmoid(g);
    const float gs = g * s;
    dg = dh * u * (s + gs * (1.0f - s));
    du = dh * gs;
}

// Normal CDF Phi(x) and e = exp(-x^2/2), for GELU(x) = x Phi(x) (the erf form: Phi(x) = (1 + erf(x / sqrt 2)) / 2) and
// its slope Phi(x) + x e / sqrt(2 pi).  The lower tail is Phi(-s) = e * Q(t), t = 1 / (1 + 0.375 s), with Q(t) = t * (a
// degree-8 polynomial) fitted to the exact function (tests/fit_normal_cdf.py derives the constants, and
// tests/test_gelu_constants.py checks the ones below against math.erf on the CPU): one hardware exp2, one hardware
// reciprocal and nine fused multiply-adds, no branch, shared by the value and the slope.  In fp32: |error| < 4e-7 for
// Phi and GELU', < 4e-7 max(1, |x|) for GELU, and the lower tail keeps a relative accuracy of a few 1e-6 because the
// exponential is a factor, not a term.  The library routines (erff plus expf, both with range
// reduction and two code paths that a wave walks one after the other) cost about three times as much, which
// matters where this runs in a GEMM epilogue with nothing to hide behind.
__device__ __forceinline__ void s24_normal(float x, float &cdf, float &e)
{
    const float t = __builtin_amdgcn_rcpf(fmaf(0.375f, fabsf(x), 1.0f));
    float q = -3.291070461e-02f;
    q = fmaf(q, t, 1.368783563e-01f);
    q = fmaf(q, t, -1.865182221e-01f);
    q = fmaf(q, t, 5.062932521e-02f);
    q = fmaf(q, t, 1.562976278e-02f);
    q = fmaf(q, t, 8.863758296e-02f);
    q = fmaf(q, t, 1.284458190e-01f);
    q = fmaf(q, t, 1.496045738e-01f);
    q = fmaf(q, t, 1.496033818e-01f);
    e = __builtin_amdgcn_exp2f(-0.72134752f * x * x);
    const float tail = e * (q * t);
    cdf = x < 0.0f ? tail : 1.0f - tail;
}
// shared by the ungated activation kernels, the gated stand-alone kernels and the GEMM epilogues
__device__ __forceinline__ float s24_gelu(float x)
{
    float cdf, e;
    s24_normal(x, cdf, e);
    return x * cdf;
}
__device__ __forceinline__ float s24_gelu_slope(float x)
{
    float cdf, e;
    s24_normal(x, cdf, e);
    return fmaf(x, e * 0.3989422804f, cdf);
}

// Ungated activation and its slope, chosen at compile time (the same arithmetic as the stand-alone kernels)
template <int ACT> __device__ __forceinline__ float s24_act_value(float z)
{
    if (ACT == S24_ACT_RELU) return z > 0.0f ? z : 0.0f;
    return s24_gelu(z);
}
template <int ACT> __device__ __forceinline__ float s24_act_slope(float z)
{
    if (ACT == S24_ACT_RELU) return z > 0.0f ? 1.0f : 0.0f;
    return s24_gelu_slope(z);
}

// Gated activation h = act(g) * u with act chosen at compile time (GATE: 0 = SiLU, 1 = GELU), and its backward
template <int GATE> __device__ __forceinline__ float s24_glu(float g, float u)
{
    if (GATE == S24_GATE_SILU) return s24_silu_mul(g, u);
    return s24_gelu(g) * u;
}
template <int GATE> __device__ __forceinline__ void s24_glu_grad(float dh, float g, float u, float &dg, float &du)
{
    if (GATE == S24_GATE_SILU) {
        s24_swiglu_grad(dh, g, u, dg, du);
    } else {
        float cdf, e;
        s24_normal(g, cdf, e);
        dg = dh * u * fmaf(g, e * 0.3989422804f, cdf);
        du = dh * (g * cdf);
    }
}
