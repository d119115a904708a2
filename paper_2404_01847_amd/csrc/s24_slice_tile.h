// A tile of a sparse NT product in slices of its contraction, as s24_gemm_slice.hip describes them.
//
// Operands of the instruction: lane l holds, of A row l%16, the eight kept values of k in [16*(l/16), 16*(l/16)+16) with
// their 2-bit positions in the low half of the index register; of B column l%16, element j is k = 32*(j/8) + 8*(l/16) + j%8;
// accumulator i is row 4*(l/16) + i of column l%16.  In the chunk-major storage (vals[K/64][M][32], meta[K/64][M][4]) 16
// rows of a chunk are 1024 contiguous bytes, lane by lane in this order, and a lane's index word is the uint16 behind
// them: a fragment is one 16-byte load, with no LDS in between.
#pragma once
#include "s24_gemm_slice.h"
#include "s24_lds.h"

namespace s24_slice {

using namespace s24_lds;

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) __bf16 bf16x16;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(16))) _Float16 f16x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
struct Two { uint4 a, b; };

template <typename T> __device__ __forceinline__ f32x4 mma(uint4 a, Two b, f32x4 c, uint32_t idx);
template <> __device__ __forceinline__ f32x4 mma<uint16_t>(uint4 a, Two b, f32x4 c, uint32_t idx)
{
    return __builtin_amdgcn_smfmac_f32_16x16x64_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x16, b), c, (int)idx, 0, 0);
}
template <> __device__ __forceinline__ f32x4 mma<s24_half>(uint4 a, Two b, f32x4 c, uint32_t idx)
{
    return __builtin_amdgcn_smfmac_f32_16x16x64_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x16, b), c, (int)idx, 0, 0);
}

// Slices per workgroup.  One number for all shapes: among the products that come here an output's bits depend on K alone, so
// that a product with and without a fused epilogue agrees to the last bit.  Which products come here depends on their tokens
// and features too (slices_if_faster there), and the tiles of s24_gemm.hip sum in another order: a token alone and the same token
// among thousands, or a stacked weight and its halves, may differ in the last bits.
constexpr int KS = 8;

// A workgroup owns 16*TM features x 16*TN tokens; wave s of its KS waves takes the 64-chunks s, s + KS, ... of the
// contraction, D of them in flight, and the slices are summed in LDS in wave order, so the result does not depend on
// scheduling.  GLU: the tile's row blocks are 8*TM gate rows and the 8*TM up rows of the same features (F of either).
// Tokens go through LDS, in a ring that belongs to the wave alone (no barrier): eight lanes copy the 128 bytes that a token has in a chunk,
// and the fragments come from there.  A wave waits for its own copies by their number: OPS operations to a chunk, in the order of `load`.
// s0 .. s3: stage_bytes(TN) of LDS each, of the last two only where TN = 1.  (One array per ring stage: the compiler then knows which stage
// a copy writes and does not make reads of the other ones wait for it.)
constexpr int stage_bytes(int TN) { return KS * 2048 * TN; }
template <typename T, bool ACCUM, int EPI, int ACT, int TM, int TN, bool STREAM>
__device__ __forceinline__ void slice_tile(lds_byte *s0, lds_byte *s1, lds_byte *s2, lds_byte *s3, int block, const uint16_t *__restrict__ B,
                                           const uint16_t *__restrict__ Av, const uint16_t *__restrict__ Am, int N, int K, int M, int F, int tiles_n, int tiles,
                                           uint16_t *Out, uint16_t *H, const uint16_t *Z, const uint16_t *bias)
{
    static_assert(EPI != S24_SLICE_GLU || TM % 2 == 0, "the gated tile pairs row blocks");
    constexpr int THREADS = 64 * KS, D = TN == 1 ? 4 : 2;
    constexpr int TWM = 16 * TM, TWN = 16 * TN;
    constexpr int FM = EPI == S24_SLICE_GLU ? TWM / 2 : TWM;   // features of the (gated) output per tile
    constexpr int WAVE = 2048 * TN;   // bytes of a wave's part of a stage
    const int tid = threadIdx.x, lane = tid & 63;
    const int ks = __builtin_amdgcn_readfirstlane(tid >> 6);
    // workgroups are dealt round-robin to the eight XCDs: each takes one contiguous eighth of the tile list, the token
    // tiles of one feature tile next to each other, so that they read its weights through one L2
    const int per_xcd = (tiles + 7) / 8, t = (block & 7) * per_xcd + (block >> 3);
    if (t >= tiles) return;
    const int tm = t / tiles_n, tn = t - tm * tiles_n;
    const int m0 = tm * FM, n0 = tn * TWN;
    const int l = lane & 15, q = lane >> 4;

    // byte offsets of this lane from wave-uniform bases (rows clamped at the edge; such rows are never stored)
    uint32_t oa[TM], ob[2 * TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int row = EPI == S24_SLICE_GLU ? (i < TM / 2 ? 0 : F) + min(m0 + 16 * (i % (TM / 2 > 0 ? TM / 2 : 1)) + l, F - 1)
                                             : min(m0 + 16 * i + l, M - 1);
        oa[i] = (uint32_t)row * 64u + 16u * q;
    }
#pragma unroll
    for (int j = 0; j < 2 * TN; ++j) {   // copy j: eight tokens, slot c of row r holds piece c ^ (r/2 % 8)
        const int row = 8 * j + (lane >> 3);
        ob[j] = (uint32_t)(min(n0 + row, N - 1) - n0) * (uint32_t)K * 2u + 16u * ((lane & 7) ^ ((row >> 1) & 7));
    }
    const char *baseB = reinterpret_cast<const char *>(B + (int64_t)n0 * K);
    const char *baseV = reinterpret_cast<const char *>(Av), *baseM = reinterpret_cast<const char *>(Am);

    struct Frag { uint4 a[TM]; uint32_t ix[TM]; };
    auto stage = [&](int d) { return (d == 0 ? s0 : d == 1 ? s1 : d == 2 ? s2 : s3) + ks * WAVE; };
    auto load = [&](Frag &f, int d, int c) {
        const char *pv = baseV + (int64_t)c * M * 64, *pm = baseM + (int64_t)c * M * 8, *pb = baseB + (int64_t)c * 128;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 2 * TN; ++j) buffer_to_lds<16>(buffer_of(pb), (lds_ptr)(stage(d) + 1024 * j), ob[j]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < TM; ++i) f.a[i] = buffer_load_16<STREAM>(buffer_of(pv), oa[i]);
#pragma unroll
        for (int i = 0; i < TM; ++i) f.ix[i] = buffer_load_2(buffer_of(pm), oa[i] >> 3, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{};
    // `behind`: chunks that are certain to have been requested after this one.  Its own values and index words need no wait here: they are in registers.
    constexpr int OPS = 2 * TN + 2 * TM;
    auto multiply = [&](const Frag &f, int d, int behind) {
        if (behind == 0) wait_copies<2 * TM>();
        else if (behind == 1) wait_copies<OPS + 2 * TM>();
        else if (behind == 2) wait_copies<2 * OPS + 2 * TM>();
        else wait_copies<3 * OPS + 2 * TM>();
        Two b[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            b[j].a = lds_load(stage(d) + b_slot(16 * j + l, q));
            b[j].b = lds_load(stage(d) + b_slot(16 * j + l, 4 + q));
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = mma<T>(f.a[i], b[j], acc[i][j], f.ix[i]);
    };
    const int nk = K / 64, steps = ks < nk ? (nk - ks + KS - 1) / KS : 0;
    // (Two ways through, so that on the longer one it is known how many copies are in flight behind the one to wait for.)
    Frag f[D];
    int i = 0;
    if (steps >= D) {
#pragma unroll
        for (int d = 0; d < D; ++d) load(f[d], d, ks + KS * d);
        for (; i + 2 * D <= steps; i += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                multiply(f[d], d, D - 1);
                load(f[d], d, ks + KS * (i + D + d));
            }
        }
#pragma unroll
        for (int d = 0; d < D; ++d) {
            multiply(f[d], d, D - 1 - d);
            if (d < D - 1 && i + D + d < steps) load(f[d], d, ks + KS * (i + D + d));
        }
        i += D;
    } else {
#pragma unroll
        for (int d = 0; d < D - 1; ++d)
            if (d < steps) load(f[d], d, ks + KS * d);
    }
#pragma unroll
    for (int d = 0; d < D - 1; ++d)
        if (i + d < steps) multiply(f[d], d, 0);

    // A wave parks its sums in the first two stages of its own ring, rows of 64 TM bytes (a token), quad c of row r at slot c ^ (its swizzle)
    constexpr int ROW = 64 * TM, RPS = WAVE / ROW;   // tokens that a wave's part of a stage holds
    static_assert(2 * RPS >= TWN, "the tile must fit two stages");
    auto parked = [&](int row, int quad) {   // of the first wave
        const int s = TM == 4 ? row & 15 : TM == 2 ? (row >> 1) & 7 : (row >> 2) & 3;
        return (row < RPS ? s0 : s1) + (row % RPS) * ROW + ((quad ^ s) << 4);
    };
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int k = 0; k < TM; ++k)
            lds_store(parked(16 * j + l, 4 * k + q) + ks * WAVE, acc[k][j]);

    // four features of one token per item; what the epilogue reads from memory is fetched ahead of the barrier
    using Num = s24_num<T>;
    constexpr int QUADS = FM / 4, ITEMS = TWN * QUADS, PER = (ITEMS + THREADS - 1) / THREADS;
    const int limit = EPI == S24_SLICE_GLU ? F : M;
    uint2 old[PER], b0[PER], b1[PER];
    bool live[PER];
    int64_t at[PER];
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const int it = tid + p * THREADS, m = m0 + 4 * (it % QUADS), n = n0 + it / QUADS;
        live[p] = it < ITEMS && n < N && m < limit;   // M and F are multiples of 16
        at[p] = (int64_t)n * M + m;
        old[p] = b0[p] = b1[p] = make_uint2(0, 0);
        if (live[p]) {
            if (ACCUM) old[p] = *reinterpret_cast<const uint2 *>(Out + at[p]);
            if (EPI == S24_SLICE_ACT_BWD) old[p] = *reinterpret_cast<const uint2 *>(Z + at[p]);
            if (!ACCUM && EPI != S24_SLICE_ACT_BWD && bias != nullptr) {
                b0[p] = *reinterpret_cast<const uint2 *>(bias + m);
                if (EPI == S24_SLICE_GLU) b1[p] = *reinterpret_cast<const uint2 *>(bias + F + m);
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        if (!live[p]) continue;
        const int it = tid + p * THREADS;
        const int row = it / QUADS, quad = it % QUADS;
        // sum of the slices, plus two packed addends (bias, or the old output); without them the bits of the sum stay
        auto total = [&](const lds_byte *s, uint2 add, bool has) {
            float4 v = __builtin_bit_cast(float4, lds_load(s));
#pragma unroll
            for (int k = 1; k < KS; ++k) {
                const float4 o = __builtin_bit_cast(float4, lds_load(s + k * WAVE));
                v.x += o.x; v.y += o.y; v.z += o.z; v.w += o.w;
            }
            if (has) { v.x += Num::lo(add.x); v.y += Num::hi(add.x); v.z += Num::lo(add.y); v.w += Num::hi(add.y); }
            return v;
        };
        auto packed = [&](float4 v) { return make_uint2(Num::pack2(v.x, v.y), Num::pack2(v.z, v.w)); };
        const bool biased = !ACCUM && EPI != S24_SLICE_ACT_BWD && bias != nullptr;
        const uint2 z = packed(total(parked(row, quad), ACCUM ? old[p] : b0[p], ACCUM || biased));
        uint16_t *out = Out + at[p];
        if constexpr (EPI == S24_SLICE_ACT_BWD) {
            *reinterpret_cast<uint2 *>(out) =
                make_uint2(Num::pack2(Num::lo(z.x) * s24_act_slope<ACT>(Num::lo(old[p].x)), Num::hi(z.x) * s24_act_slope<ACT>(Num::hi(old[p].x))),
                           Num::pack2(Num::lo(z.y) * s24_act_slope<ACT>(Num::lo(old[p].y)), Num::hi(z.y) * s24_act_slope<ACT>(Num::hi(old[p].y))));
        } else {
            *reinterpret_cast<uint2 *>(out) = z;
            if constexpr (EPI == S24_SLICE_ACT)
                *reinterpret_cast<uint2 *>(H + at[p]) =
                    make_uint2(Num::pack2(s24_act_value<ACT>(Num::lo(z.x)), s24_act_value<ACT>(Num::hi(z.x))),
                               Num::pack2(s24_act_value<ACT>(Num::lo(z.y)), s24_act_value<ACT>(Num::hi(z.y))));
            if constexpr (EPI == S24_SLICE_GLU) {
                const uint2 u = packed(total(parked(row, quad + QUADS), b1[p], biased));
                *reinterpret_cast<uint2 *>(out + F) = u;
                const int64_t n = n0 + it / QUADS, m = m0 + 4 * (it % QUADS);
                *reinterpret_cast<uint2 *>(H + n * F + m) =
                    make_uint2(Num::pack2(s24_glu<ACT>(Num::lo(z.x), Num::lo(u.x)), s24_glu<ACT>(Num::hi(z.x), Num::hi(u.x))),
                               Num::pack2(s24_glu<ACT>(Num::lo(z.y), Num::lo(u.y)), s24_glu<ACT>(Num::hi(z.y), Num::hi(u.y))));
            }
        }
    }
}
}  // namespace s24_slice
