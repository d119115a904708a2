// fp32 GEMMs on the matrix cores: v_mfma_f32_32x32x2_f32 (one lane holds A row l%32 and B column l%32 at k = l/32;
// accumulator i is row 8*(i/4) + 4*(l/32) + i%4 of column l%32).  There is no fp32 sparse instruction: the compressed
// operand is expanded to its four columns per group in registers, zeros included (and see kept_sum).
//
// What bounds them is latency, not arithmetic: the fp32 layers are small (512 x 256 x 1024 has 0.27 GFLOP per product,
// 1.7 us of the unit's 157 TFLOP/s), so the whole product has to be spread over every SIMD of the chip at once.  Each
// wave therefore owns one 32T x 32T output tile and one SLICE of the contraction axis (KS slices per workgroup, 32 to 64
// of k each where the grid is small), loads its fragments from global memory straight into registers (a fragment is
// used by one wave of the workgroup only: LDS staging would buy nothing), and the slices are summed in LDS in a
// fixed order.  A lane takes its k values as runs of eight of one row (two 16-byte loads), the same runs for both
// operands; which k an instruction multiplies is free as long as both sides agree.
#include <type_traits>

#include "s24_gemm_f32.h"

namespace {

typedef __attribute__((ext_vector_type(16))) float f32x16;

__device__ __forceinline__ f32x16 mma(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

// Two kept values and their nibble (i0 | i1 << 2) -> the four values of the group
__device__ __forceinline__ void expand(float v0, float v1, uint32_t nib, float (&e)[4])
{
    const uint32_t i0 = nib & 3u, i1 = nib >> 2;
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) e[i] = i0 == i ? v0 : (i1 == i ? v1 : 0.0f);
}

// The sum over the kept elements alone: row m of the compressed operand against x[k * stride].  A pruned element is
// multiplied as a zero above, which makes NaN of an infinity or a NaN beside it; an output that is NaN is therefore taken
// again from here, so that, as on the 16-bit sparse instruction, what is pruned never reaches a result.
__device__ __forceinline__ float kept_sum(const float *Av, const uint16_t *Am, int64_t M, int64_t m, int K, const float *x, int64_t stride)
{
    float sum = 0.0f;
#pragma unroll 1
    for (int gr = 0; gr < K / 4; ++gr, x += 4 * stride) {
        const int64_t cr = (int64_t)(gr >> 4) * M + m;
        const float2 v = *reinterpret_cast<const float2 *>(Av + cr * 32 + 2 * (gr & 15));
        const uint32_t nib = ((uint32_t)Am[cr * 4 + ((gr & 15) >> 2)] >> (4 * (gr & 3))) & 0xFu;
        sum = fmaf(v.x, x[(nib & 3u) * stride], sum);
        sum = fmaf(v.y, x[(nib >> 2) * stride], sum);
    }
    return sum;
}

// Sum of one float4 over the KS slices' copies of a tile, in slice order.  Slice s is parked at s * slice floats.
template <int KS> __device__ __forceinline__ float4 slice_sum(const float *p, int slice)
{
    float4 v = *reinterpret_cast<const float4 *>(p);
#pragma unroll
    for (int s = 1; s < KS; ++s) {
        const float4 o = *reinterpret_cast<const float4 *>(p + s * slice);
        v.x += o.x; v.y += o.y; v.z += o.z; v.w += o.w;
    }
    return v;
}

// ------------------------------------------------------------------ NT
// SPARSE: A compressed.  EPI / ACT: epilogue.  GLU needs T = 2: a tile takes 32 gate rows and the 32 up rows of the same
// features, F of either (else F = M).  s_red: lds_floats(T, KS) of LDS.
constexpr int lds_floats(int T, int KS) { return KS * 32 * T * (32 * T + 4); }
template <bool SPARSE, bool ACCUM, int EPI, int ACT, int T, int KS>
__device__ __forceinline__ void f32_nt_tile(float *s_red, int tile, const float *B, const float *Av, const uint16_t *Am, int N, int K, int M, int F,
                                            int tiles_m, float *Out, float *H, const float *bias)
{
    static_assert(EPI != S24_F32_GLU || T == 2, "the gated tile pairs two row blocks");
    constexpr int TW = 32 * T, PITCH = TW + 4, SLICE = TW * PITCH, THREADS = 64 * KS;
    const int tid = threadIdx.x, lane = tid & 63;
    const int ks = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5, l = lane & 31;
    const int tm = tile % tiles_m, tn = tile / tiles_m;
    constexpr int FM = EPI == S24_F32_GLU ? 32 : TW;   // features of the (gated) output per tile
    const int m0 = tm * FM, n0 = tn * TW;

    f32x16 acc[T][T];
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j) acc[i][j] = f32x16{};
    // rows of this lane (clamped at the edge; such rows are never stored)
    int arow[T];
    const float *b[T];
#pragma unroll
    for (int i = 0; i < T; ++i) {
        arow[i] = EPI == S24_F32_GLU ? i * F + min(m0 + l, F - 1) : min(m0 + 32 * i + l, M - 1);
        b[i] = B + (int64_t)min(n0 + 32 * i + l, N - 1) * K;
    }
    // units of 16 of k: lane half h takes k 8h .. 8h+7 of a unit
    const int units = K / 16, u0 = s24_slice_begin(units, ks, KS), u1 = s24_slice_begin(units, ks + 1, KS);
    struct Frag { float4 a[T][2]; float4 b[T][2]; uint32_t nib[T]; };
    auto load = [&](int u, Frag &f) {
        const int k = 16 * u + 8 * h;
#pragma unroll
        for (int i = 0; i < T; ++i) {
            if constexpr (SPARSE) {   // four kept values of the run's two groups, and their byte of the index words
                const int64_t cr = (int64_t)(u >> 2) * M + arow[i];
                f.a[i][0] = *reinterpret_cast<const float4 *>(Av + cr * 32 + 8 * (u & 3) + 4 * h);
                f.nib[i] = (uint32_t)Am[cr * 4 + (u & 3)] >> (8 * h);
            } else {
                const float *a = Av + (int64_t)arow[i] * K + k;
                f.a[i][0] = *reinterpret_cast<const float4 *>(a);
                f.a[i][1] = *reinterpret_cast<const float4 *>(a + 4);
            }
            f.b[i][0] = *reinterpret_cast<const float4 *>(b[i] + k);
            f.b[i][1] = *reinterpret_cast<const float4 *>(b[i] + k + 4);
        }
    };
    auto multiply = [&](const Frag &f) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {   // the run's two groups of four
            float e[T][4], x[T][4];
#pragma unroll
            for (int i = 0; i < T; ++i) {
                if constexpr (SPARSE) {
                    const float4 v = f.a[i][0];
                    expand(q ? v.z : v.x, q ? v.w : v.y, (f.nib[i] >> (4 * q)) & 0xFu, e[i]);
                } else {
                    const float4 v = f.a[i][q];
                    e[i][0] = v.x; e[i][1] = v.y; e[i][2] = v.z; e[i][3] = v.w;
                }
                const float4 w = f.b[i][q];
                x[i][0] = w.x; x[i][1] = w.y; x[i][2] = w.z; x[i][3] = w.w;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int i = 0; i < T; ++i)
#pragma unroll
                    for (int j = 0; j < T; ++j) acc[i][j] = mma(e[i][k], x[j][k], acc[i][j]);
        }
    };
    Frag f0, f1;
    if (u0 < u1) load(u0, f0);
    int u = u0;
    for (; u + 1 < u1; u += 2) {   // the next unit's loads go out before the current one is multiplied
        load(u + 1, f1);
        multiply(f0);
        load(min(u + 2, u1 - 1), f0);
        multiply(f1);
    }
    if (u < u1) multiply(f0);
    float *part = s_red + ks * SLICE;
#pragma unroll
    for (int j = 0; j < T; ++j)
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<float4 *>(part + (32 * j + l) * PITCH + 32 * i + 8 * q + 4 * h) =
                    make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
    __syncthreads();
    constexpr int QUADS = FM / 4, ITEMS = TW * QUADS;   // four features of one token per item
#pragma unroll 1
    for (int it = tid; it < ITEMS; it += THREADS) {
        const int q = it % QUADS, row = it / QUADS, m = m0 + 4 * q, n = n0 + row;
        if (n >= N || m >= (EPI == S24_F32_GLU ? F : M)) continue;   // M, F multiples of 16
        const float *p = s_red + row * PITCH + 4 * q;
        auto finish = [&](const float *src, int feature) {
            float4 v = slice_sum<KS>(src, SLICE);
            if constexpr (SPARSE) {
                const float *x = B + (int64_t)n * K;
                if (v.x != v.x) v.x = kept_sum(Av, Am, M, feature, K, x, 1);
                if (v.y != v.y) v.y = kept_sum(Av, Am, M, feature + 1, K, x, 1);
                if (v.z != v.z) v.z = kept_sum(Av, Am, M, feature + 2, K, x, 1);
                if (v.w != v.w) v.w = kept_sum(Av, Am, M, feature + 3, K, x, 1);
            }
            if (bias != nullptr) {
                const float2 b0 = *reinterpret_cast<const float2 *>(bias + feature), b1 = *reinterpret_cast<const float2 *>(bias + feature + 2);
                v.x += b0.x; v.y += b0.y; v.z += b1.x; v.w += b1.y;
            }
            float4 *o = reinterpret_cast<float4 *>(Out + (int64_t)n * M + feature);
            if (ACCUM) {
                const float4 old = *o;
                v.x += old.x; v.y += old.y; v.z += old.z; v.w += old.w;
            }
            *o = v;
            return v;
        };
        if constexpr (EPI == S24_F32_GLU) {
            const float4 z = finish(p, m), u = finish(p + 32, F + m);
            *reinterpret_cast<float4 *>(H + (int64_t)n * F + m) =
                make_float4(s24_glu<ACT>(z.x, u.x), s24_glu<ACT>(z.y, u.y), s24_glu<ACT>(z.z, u.z), s24_glu<ACT>(z.w, u.w));
        } else {
            const float4 z = finish(p, m);
            if constexpr (EPI == S24_F32_ACT) {
                *reinterpret_cast<float4 *>(H + (int64_t)n * M + m) = make_float4(s24_act_value<ACT>(z.x), s24_act_value<ACT>(z.y), s24_act_value<ACT>(z.z), s24_act_value<ACT>(z.w));
            }
        }
    }
}

// first: B, Av; second: Am, N, K; third: M, F, tiles of features, nothing
struct NtEnds { float *Out, *H; const float *bias; };
template <bool SPARSE, bool ACCUM, int EPI, int ACT, int T, int KS>
__global__ __launch_bounds__(64 * KS) void f32_nt_kernel(const s24_words first, const s24_words second, const s24_words third, const NtEnds e)
{
    __shared__ __attribute__((aligned(16))) float s_red[lds_floats(T, KS)];
    f32_nt_tile<SPARSE, ACCUM, EPI, ACT, T, KS>(s_red, (int)blockIdx.x, s24_global<const float>(first.x), s24_global<const float>(first.y), s24_global<const uint16_t>(second.x),
                                                s24_low(second.y), s24_high(second.y), s24_low(third.x), s24_high(third.x), s24_low(third.y), e.Out, e.H, e.bias);
}

// ------------------------------------------------------------------ TN (weight gradients)
// Both operands are token-major: a lane reads T consecutive columns of one token (the columns of tile block i are
// T*(l%32) + i), lane half h takes every second token.
struct TnWindow {
    const float *A, *X, *Wt;
    const uint16_t *Am, *mask;
    float *dW;
    int T, M, N, tiles_m, first;   // first: the problem's first tile in the grid
    float lambda;
};
constexpr int kMaxTn = 4;
// Up to this many tokens the sum is one chain: split into slices of a pair or less it is rounded more often (distance from
// fp64 against the chain's: 3 tokens 1.10, 5: 1.07, 7: 1.02, 8: 0.94, 16: 0.87).  A launch of such problems alone has one
// wave per tile (5 tokens, 768 x 3072: 6.4 us with eight waves, 4.7 with one).
constexpr int kWholeTokens = 7;
struct TnArgs {
    TnWindow w[kMaxTn];
};

template <int T> struct Run { float v[T]; };

// D: batches of eight token pairs in flight (see s24_f32_tn)
template <bool SPARSE, bool ACCUM, int T, int KS, int D>
__device__ __forceinline__ void f32_tn_tile(float *s_red, int tile, const TnArgs &args)
{
    constexpr int TW = 32 * T, PITCH = TW + 4, SLICE = TW * PITCH, THREADS = 64 * KS;
    const int tid = threadIdx.x, lane = tid & 63;
    const int ks = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5, l = lane & 31;
    int which = 0;
#pragma unroll
    for (int i = 1; i < kMaxTn; ++i)
        if (tile >= args.w[i].first) which = i;
    const TnWindow &g = args.w[which];
    const int t = tile - g.first;
    const int m0 = (t % g.tiles_m) * TW, n0 = (t / g.tiles_m) * TW;
    const int M = g.M, N = g.N;
    f32x16 acc[T][T];
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j) acc[i][j] = f32x16{};
    // columns of this lane, clamped at the edge (M and N are multiples of 16: a run of T is all in or all out)
    const int mc = min(m0 + T * l, M - T), nc = min(n0 + T * l, N - T);
    if constexpr (SPARSE) {
        // A compressed along the tokens: a lane reads one group (two kept values, one nibble) of its T rows and expands it;
        // lane half h takes every second group of four tokens
        const int groups = g.T / 4, half = groups / 2, p0 = s24_slice_begin(half, ks, KS), p1 = s24_slice_begin(half, ks + 1, KS);   // T is a multiple of 64
        for (int p = p0; p < p1; ++p) {
            const int gr = 2 * p + h;
            float e[T][4];
            Run<T> x[4];
#pragma unroll
            for (int i = 0; i < T; ++i) {
                const int64_t cr = (int64_t)(gr >> 4) * M + mc + i;
                const float2 v = *reinterpret_cast<const float2 *>(g.A + cr * 32 + 2 * (gr & 15));
                expand(v.x, v.y, ((uint32_t)g.Am[cr * 4 + ((gr & 15) >> 2)] >> (4 * (gr & 3))) & 0xFu, e[i]);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) x[k] = *reinterpret_cast<const Run<T> *>(g.X + (int64_t)(4 * gr + k) * N + nc);
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int i = 0; i < T; ++i)
#pragma unroll
                    for (int j = 0; j < T; ++j) acc[i][j] = mma(e[i][k], x[k].v[j], acc[i][j]);
        }
    } else {
        constexpr int U = 8;   // token pairs loaded together
        const int pairs = s24_token_pairs(g.T);
        const bool whole = g.T <= kWholeTokens;   // the first slice takes all
        const int p0 = whole ? (ks == 0 ? 0 : pairs) : s24_slice_begin(pairs, ks, KS), p1 = whole ? pairs : s24_slice_begin(pairs, ks + 1, KS);
        const float *a = g.A + mc, *x = g.X + nc;
        struct Batch { Run<T> a[U], x[U]; };
        auto load = [&](Batch &f, int p) {   // the U whole pairs from p on
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t tok = 2 * (p + u) + h;
                f.a[u] = *reinterpret_cast<const Run<T> *>(a + tok * M);
                f.x[u] = *reinterpret_cast<const Run<T> *>(x + tok * N);
            }
        };
        auto pair = [&](const Run<T> &av, const Run<T> &xv) {
#pragma unroll
            for (int i = 0; i < T; ++i)
#pragma unroll
                for (int j = 0; j < T; ++j) acc[i][j] = mma(av.v[i], xv.v[j], acc[i][j]);
        };
        auto multiply = [&](const Batch &f) {
#pragma unroll
            for (int u = 0; u < U; ++u) pair(f.a[u], f.x[u]);
        };
        int p = p0;
        if constexpr (D == 1) {
            Batch f;
            for (; p + U <= p1 && p + U <= g.T / 2; p += U) {
                load(f, p);
                multiply(f);
            }
        } else {
            const int batches = max(min(p1, g.T / 2) - p0, 0) / U;
            Batch f[D];
#pragma unroll
            for (int d = 0; d < D; ++d)
                if (d < batches) load(f[d], p0 + U * d);
            int b = 0;
            for (; b + 2 * D <= batches; b += D) {
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    multiply(f[d]);
                    load(f[d], p0 + U * (b + D + d));
                }
            }
#pragma unroll
            for (int d = 0; d < D; ++d)
                if (b + d < batches) {
                    multiply(f[d]);
                    if (b + D + d < batches) load(f[d], p0 + U * (b + D + d));
                }
#pragma unroll
            for (int d = 0; d < D; ++d)
                if (b + D + d < batches) multiply(f[d]);
            p = p0 + U * batches;
        }
        for (; p < p1; ++p) {   // rest of the slice; the token past an odd count contributes zero
            const int tok = 2 * p + h;
            const int64_t tc = min(tok, g.T - 1);
            Run<T> av1 = *reinterpret_cast<const Run<T> *>(a + tc * M), xv1 = *reinterpret_cast<const Run<T> *>(x + tc * N);
#pragma unroll
            for (int i = 0; i < T; ++i)   // both operands: zero times an infinity of the repeated last token would be NaN
                if (tok >= g.T) av1.v[i] = xv1.v[i] = 0.0f;
            pair(av1, xv1);
        }
    }
    // park: matrix row r of block i is output row T*r + i, column c of block j output column T*c + j
    float *part = s_red + ks * SLICE;
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int r = 8 * (e / 4) + 4 * h + (e & 3);
            Run<T> o;
#pragma unroll
            for (int j = 0; j < T; ++j) o.v[j] = acc[i][j][e];
            *reinterpret_cast<Run<T> *>(part + (T * r + i) * PITCH + T * l) = o;
        }
    __syncthreads();
    constexpr int QUADS = TW / 4, ITEMS = TW * QUADS;
#pragma unroll 1
    for (int it = tid; it < ITEMS; it += THREADS) {
        const int q = it % QUADS, row = it / QUADS, m = m0 + row, n = n0 + 4 * q;
        if (m >= M || n >= N) continue;
        float4 v = slice_sum<KS>(s_red + row * PITCH + 4 * q, SLICE);
        if constexpr (SPARSE) {
            if (v.x != v.x) v.x = kept_sum(g.A, g.Am, M, m, g.T, g.X + n, N);
            if (v.y != v.y) v.y = kept_sum(g.A, g.Am, M, m, g.T, g.X + n + 1, N);
            if (v.z != v.z) v.z = kept_sum(g.A, g.Am, M, m, g.T, g.X + n + 2, N);
            if (v.w != v.w) v.w = kept_sum(g.A, g.Am, M, m, g.T, g.X + n + 3, N);
        }
        float4 *o = reinterpret_cast<float4 *>(g.dW + (int64_t)m * N + n);
        if (ACCUM) {
            const float4 old = *o;
            v.x = old.x + v.x; v.y = old.y + v.y; v.z = old.z + v.z; v.w = old.w + v.w;
        }
        if (g.Wt != nullptr) {   // masked decay: the one fused multiply-add of the stand-alone kernel
            const float4 w = *reinterpret_cast<const float4 *>(g.Wt + (int64_t)m * N + n);
            const uint32_t keep = (uint32_t)g.mask[(int64_t)(m >> 2) * (N >> 2) + (n >> 2)] >> (4 * (m & 3));
            if (!(keep & 1u)) v.x = fmaf(g.lambda, w.x, v.x);
            if (!(keep & 2u)) v.y = fmaf(g.lambda, w.y, v.y);
            if (!(keep & 4u)) v.z = fmaf(g.lambda, w.z, v.z);
            if (!(keep & 8u)) v.w = fmaf(g.lambda, w.w, v.w);
        }
        *o = v;
    }
}

template <bool SPARSE, bool ACCUM, int T, int KS, int D>
__global__ __launch_bounds__(64 * KS) void f32_tn_kernel(const TnArgs args)
{
    __shared__ __attribute__((aligned(16))) float s_red[lds_floats(T, KS)];
    f32_tn_tile<SPARSE, ACCUM, T, KS, D>(s_red, (int)blockIdx.x, args);
}

// An input gradient in eight slices and weight gradients that do not depend on it in one launch: neither fills the chip, and each is a
// launch and a few trips to memory that the other one can hide.  The input gradient's tiles walk the longer sums and go first.
// 512 tokens, 256 x 1024 (10.2 and 12.5 us under the tracer): 54.6 -> 47.2 us a step.
// first: B, Av; second: Am, tiles of the input gradient, N; third: K, M, its tiles of features, nothing
template <int D>
__global__ __launch_bounds__(512) void f32_nt_tn_kernel(const s24_words first, const s24_words second, const s24_words third, float *Out, const TnArgs args)
{
    __shared__ __attribute__((aligned(16))) float s_red[lds_floats(1, 8)];
    const int nt_tiles = s24_low(second.y), M = s24_high(third.x);
    if ((int)blockIdx.x < nt_tiles)
        f32_nt_tile<true, false, S24_F32_PLAIN, 0, 1, 8>(s_red, (int)blockIdx.x, s24_global<const float>(first.x), s24_global<const float>(first.y), s24_global<const uint16_t>(second.x),
                                                         s24_high(second.y), s24_low(third.x), M, M, s24_low(third.y), Out, nullptr, nullptr);
    else f32_tn_tile<false, false, 1, 8, D>(s_red, (int)blockIdx.x - nt_tiles, args);
}

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

template <bool SPARSE, bool ACCUM, int EPI, int ACT, int T, int KS>
int launch_nt(const S24F32Nt &g, hipStream_t st)
{
    const int64_t F = EPI == S24_F32_GLU ? g.M / 2 : g.M;
    const int64_t tiles_m = ceil_div(F, EPI == S24_F32_GLU ? 32 : 32 * T), tiles = tiles_m * ceil_div(g.N, 32 * T);
    S24_REQUIRE(tiles < (1ll << 31), S24_ERR_SHAPE);
    hipLaunchKernelGGL((f32_nt_kernel<SPARSE, ACCUM, EPI, ACT, T, KS>), dim3((unsigned)tiles), dim3(64 * KS), 0, st, s24_pack(g.B, g.Av), s24_pack(g.Am, (int)g.N, (int)g.K),
                       s24_pack((int)g.M, (int)F, (int)tiles_m, 0), (NtEnds{g.Out, g.H, g.bias}));
    return s24_launch_status();
}

// Tile and slices by the size of the product (the slices decide the order of the sum, so the rule looks at the whole
// product only: a fused epilogue gives the bits of the plain product).  Measured in us (N x K x M: 8 slices of a 32-tile
// / 4 slices of a 32-tile / 4 slices of a 64-tile; one thread per output before):
//   512 x 256 x 1024: 7.3 / 6.5 / 10.0 (109)      512 x 1024 x 256: 9.2 / 10.1 / 26.3 (114)
//   333 x 1792 x 448: 13.4 / 15.3 / 45.4 (281)    1024 x 768 x 3072: 66 / 61 / 53 (2480)     2048 x 1024 x 4096: 228 / 199 / 168 (8608)
// The 64-tile reads half the operand bytes per product, which only counts once its own grid fills the chip.
inline bool nt_deep(int64_t N, int64_t K, int64_t M) { return K >= 512 && ceil_div(M, 32) * ceil_div(N, 32) <= s24_cu_count(); }   // few tiles, long sums: 8 slices
template <bool SPARSE, bool ACCUM, int EPI, int ACT> int choose_nt(const S24F32Nt &g, hipStream_t st)
{
    const bool deep = nt_deep(g.N, g.K, g.M);
    if constexpr (EPI == S24_F32_GLU) {
        if (deep) return launch_nt<SPARSE, ACCUM, EPI, ACT, 2, 8>(g, st);
        return launch_nt<SPARSE, ACCUM, EPI, ACT, 2, 4>(g, st);
    } else {
        if (deep) return launch_nt<SPARSE, ACCUM, EPI, ACT, 1, 8>(g, st);
        if (ceil_div(g.M, 64) * ceil_div(g.N, 64) < 2 * s24_cu_count()) return launch_nt<SPARSE, ACCUM, EPI, ACT, 1, 4>(g, st);
        return launch_nt<SPARSE, ACCUM, EPI, ACT, 2, 4>(g, st);
    }
}

template <bool SPARSE, int T, int KS, int D = 1> int launch_tn(TnArgs &a, int64_t tiles, bool accum, hipStream_t st)
{
    const dim3 grid((unsigned)tiles), block(64 * KS);
    if (accum) hipLaunchKernelGGL((f32_tn_kernel<SPARSE, true, T, KS, D>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((f32_tn_kernel<SPARSE, false, T, KS, D>), grid, block, 0, st, a);
    return s24_launch_status();
}
}  // namespace

int s24_f32_nt(const S24F32Nt &g, hipStream_t st)
{
    if (g.Am == nullptr) return choose_nt<false, false, S24_F32_PLAIN, 0>(g, st);   // dense comparison GEMM
    if (g.accum) return choose_nt<true, true, S24_F32_PLAIN, 0>(g, st);
    if (g.epilogue == S24_F32_ACT)
        return g.act == S24_ACT_RELU ? choose_nt<true, false, S24_F32_ACT, S24_ACT_RELU>(g, st) : choose_nt<true, false, S24_F32_ACT, S24_ACT_GELU_ERF>(g, st);
    if (g.epilogue == S24_F32_GLU)
        return g.act == S24_GATE_SILU ? choose_nt<true, false, S24_F32_GLU, S24_GATE_SILU>(g, st) : choose_nt<true, false, S24_F32_GLU, S24_GATE_GELU_ERF>(g, st);
    return choose_nt<true, false, S24_F32_PLAIN, 0>(g, st);
}

// 32-tiles until the 64-tile's own grid is three workgroups per compute unit: 512 tokens, 1024 x 256 out: 8.1 against 15.1 us
// (58 with one thread per output); 1024 tokens, 3072 x 768: 78 against 84 (1282); 2048 tokens, 4096 x 1024: 248 against 214.
// Batches in flight (one, two, four; us): below 128 tokens a slice has none of a whole batch and the code for more only costs (64 tokens, 1024 x
// 256: 3.72, 3.83, 3.91).  With up to one workgroup of 32-tiles per compute unit a wave's trips to memory are what takes the time:
// four (512, 1024 x 256: 7.43, 6.84, 6.65; 2048: 35.0, 17.7, 19.1).  Up to two, four batches' registers still leave room for both, and up to 512 tokens
// they are the fastest (512, 896 x 512: 11.1, 11.4, 10.7); past that the waves' turns are what takes the time while the operands stay in an XCD's 4 MB of L2
// (1000, 768 x 512: 18.7, 19.6, 20.7), and two are the fastest once they do not (1200: 25.6, 22.3, 25.2; 2048: 43.3, 32.1, 36.9).  Beyond
// two workgroups the waves that more registers would displace hide more (1000, 1024 x 1024: 32.3, 37.5, 40.8).  The 64-tile has its two
// waves per SIMD anyway and takes two (64, 4096 x 1024: 16.9, 17.1; 512: 67.1, 52.6).
namespace {
struct TnPlan {
    TnArgs a;
    int T, D;        // tile of 32 T; batches in flight
    int64_t tiles;
    bool whole;      // one wave per tile
};
TnPlan plan_tn(const S24F32TnProblem *pr, int count)
{
    int64_t tiles[2] = {0, 0}, tokens = 0, bytes = 0;   // tokens: of the longest problem; bytes: of all operands
    TnPlan plan{};
    for (int T = 1; T <= 2; ++T)
        for (int i = 0; i < count; ++i) tiles[T - 1] += ceil_div(pr[i].M, 32 * T) * ceil_div(pr[i].N, 32 * T);
    const int64_t cus = s24_cu_count();
    const int T = plan.T = tiles[1] < 3 * cus ? 1 : 2;
    plan.whole = true;
    for (int i = 0; i < kMaxTn; ++i) {
        if (i < count) {
            plan.whole = plan.whole && pr[i].T <= kWholeTokens;
            tokens = std::max(tokens, pr[i].T);
            bytes += pr[i].T * (pr[i].M + pr[i].N) * (int64_t)sizeof(float);
            const int64_t tm = ceil_div(pr[i].M, 32 * T);
            plan.a.w[i] = TnWindow{pr[i].A, pr[i].X, pr[i].Wt, pr[i].Am, pr[i].mask, pr[i].dW, (int)pr[i].T, (int)pr[i].M, (int)pr[i].N, (int)tm, (int)plan.tiles, pr[i].lambda};
            plan.tiles += tm * ceil_div(pr[i].N, 32 * T);
        } else {
            plan.a.w[i] = plan.a.w[count - 1];
            plan.a.w[i].first = 0x7FFFFFFF;   // no tile of the grid
        }
    }
    if (T == 2) plan.D = tokens < 128 ? 1 : 2;
    else if (tokens < 128 || plan.tiles > 2 * cus) plan.D = 1;
    else if (plan.tiles <= cus || tokens <= 512) plan.D = 4;
    else plan.D = bytes < 11 << 19 ? 1 : 2;
    return plan;
}
}  // namespace

int s24_f32_tn(const S24F32TnProblem *pr, int count, bool accum, hipStream_t st)
{
    TnPlan p = plan_tn(pr, count);
    S24_REQUIRE(p.tiles < (1ll << 31), S24_ERR_SHAPE);
    if (pr[0].Am != nullptr) return p.T == 1 ? launch_tn<true, 1, 8>(p.a, p.tiles, accum, st) : launch_tn<true, 2, 8>(p.a, p.tiles, accum, st);
    if (p.whole) return p.T == 1 ? launch_tn<false, 1, 1>(p.a, p.tiles, accum, st) : launch_tn<false, 2, 1>(p.a, p.tiles, accum, st);
    if (p.T == 2) return p.D == 1 ? launch_tn<false, 2, 8>(p.a, p.tiles, accum, st) : launch_tn<false, 2, 8, 2>(p.a, p.tiles, accum, st);
    if (p.D == 1) return launch_tn<false, 1, 8>(p.a, p.tiles, accum, st);
    return p.D == 2 ? launch_tn<false, 1, 8, 2>(p.a, p.tiles, accum, st) : launch_tn<false, 1, 8, 4>(p.a, p.tiles, accum, st);
}

// Together where the input gradient has a tile for at most every compute unit and the weight gradients take the 32-tile in eight slices
bool s24_f32_nt_tn(const S24F32Nt &g, const S24F32TnProblem *pr, int count, hipStream_t st, int &status)
{
    if (!nt_deep(g.N, g.K, g.M)) return false;
    const TnPlan p = plan_tn(pr, count);
    if (p.whole || p.T != 1 || p.tiles >= 1ll << 30) return false;
    const int64_t tiles_m = ceil_div(g.M, 32), tiles = tiles_m * ceil_div(g.N, 32);
    auto launch = [&](auto d) {
        hipLaunchKernelGGL((f32_nt_tn_kernel<decltype(d)::value>), dim3((unsigned)(tiles + p.tiles)), dim3(512), 0, st, s24_pack(g.B, g.Av), s24_pack(g.Am, (int)tiles, (int)g.N),
                           s24_pack((int)g.K, (int)g.M, (int)tiles_m, 0), g.Out, p.a);
    };
    if (p.D == 1) launch(std::integral_constant<int, 1>());
    else if (p.D == 2) launch(std::integral_constant<int, 2>());
    else launch(std::integral_constant<int, 4>());
    status = s24_launch_status();
    return true;
}
