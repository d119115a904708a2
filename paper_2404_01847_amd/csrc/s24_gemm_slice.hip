// Sparse NT products of few tokens or few features, bf16 and binary16: out[n][m] = sum_k B[n][k] A[m][k] with A compressed
// along k, on v_smfmac_f32_16x16x64_{bf16,f16}.
//
// With one 128 x 128 tile per workgroup, 16 tokens x 4096 features are 32 workgroups that walk K = 11008 in 172 steps of 0.28 us each
// on an eighth of the chip.  Here a tile is 16 x 16 to 64 x 64, eight waves of a workgroup split its contraction, each on its own
// with no barrier, and the slices are summed in LDS.
// What bounds them, where it is not the weights' way from memory, is the first-level cache: it takes a 16-byte load four lanes at a time and spends a
// cycle on each 128-byte line that these touch.  A fragment of the values, read as the instruction wants it, is 32 cycles (16 rows of 64
// bytes, two to a line); one of tokens, 16 rows of K elements each, would be 128, and is 32 copied to LDS row by row.  With the tokens read
// straight into registers: 256 x 768, K = 3072 9.1 us, now 7.0; 256 x 3072, K = 768 with activation 8.5 and 5.8; 16 x 4096, K = 11008, weights out
// of the caches 18.3 and 13.3, 16 x 22016 (gated), K = 4096 26.8 and 21.0 (23.6 of it by the tokens' way, the rest by reading weights that nobody
// else reads past the caches: 101 MB at 5.2 TB/s).  The values through LDS as well are 16 cycles, but then fewer are in flight: 16 x 4096,
// K = 11008 14.0 -> 15.5.  64 x 64 tiles are for up to one of them per compute unit: 1024 x 1024, K = 4096 19.9 us in tiles of
// s24_gemm.hip, 14.4 here; 512 x 2048, K = 2048 11.1 and 7.9.
//
// Operands of the instruction: lane l holds, of A row l%16, the eight kept values of k in [16*(l/16), 16*(l/16)+16) with
// their 2-bit positions in the low half of the index register; of B column l%16, element j is k = 32*(j/8) + 8*(l/16) + j%8;
// accumulator i is row 4*(l/16) + i of column l%16.  In the chunk-major storage (vals[K/64][M][32], meta[K/64][M][4]) 16
// rows of a chunk are 1024 contiguous bytes, lane by lane in this order, and a lane's index word is the uint16 behind
// them: a fragment is one 16-byte load, with no LDS in between.
#include "s24_gemm_slice.h"
#include "s24_lds.h"

namespace {

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
// and features too (slice_pays there), and the tiles of s24_gemm.hip sum in another order: a token alone and the same token
// among thousands, or a stacked weight and its halves, may differ in the last bits.
constexpr int KS = 8;

// A workgroup owns 16*TM features x 16*TN tokens; wave s of its KS waves takes the 64-chunks s, s + KS, ... of the
// contraction, D of them in flight, and the slices are summed in LDS in wave order, so the result does not depend on
// scheduling.  GLU: the tile's row blocks are 8*TM gate rows and the 8*TM up rows of the same features (F of either).
// The arguments are one by one and in the order in which they are needed: see FLAGS in build.py.
// Tokens go through LDS, in a ring that belongs to the wave alone (no barrier): eight lanes copy the 128 bytes that a token has in a chunk,
// and the fragments come from there.
template <typename T, bool ACCUM, int EPI, int ACT, int TM, int TN, bool STREAM>
__global__ __launch_bounds__(64 * KS, TN == 4 ? 2 : 4) void spmm_slice_kernel(const uint16_t *__restrict__ B, const uint16_t *__restrict__ Av, const uint16_t *__restrict__ Am,
                                                                int N, int K, int M, int F, int tiles_n, int tiles, uint16_t *Out, uint16_t *H,
                                                                const uint16_t *Z, const uint16_t *bias)
{
    static_assert(EPI != S24_SLICE_GLU || TM % 2 == 0, "the gated tile pairs row blocks");
    constexpr int THREADS = 64 * KS, D = TN == 1 ? 4 : 2;
    constexpr int TWM = 16 * TM, TWN = 16 * TN;
    constexpr int FM = EPI == S24_SLICE_GLU ? TWM / 2 : TWM;   // features of the (gated) output per tile
    // One array per ring stage: the compiler then knows which stage a copy writes and does not make reads of the other ones wait for it.
    constexpr int WAVE = 2048 * TN, STAGE = KS * WAVE;         // bytes of a wave's part of a stage
    __shared__ __attribute__((aligned(16))) unsigned char s0[STAGE];
    __shared__ __attribute__((aligned(16))) unsigned char s1[STAGE];
    __shared__ __attribute__((aligned(16))) unsigned char s2[D > 2 ? STAGE : 16];
    __shared__ __attribute__((aligned(16))) unsigned char s3[D > 2 ? STAGE : 16];
    const int tid = threadIdx.x, lane = tid & 63;
    const int ks = __builtin_amdgcn_readfirstlane(tid >> 6);
    // workgroups are dealt round-robin to the eight XCDs: each takes one contiguous eighth of the tile list, the token
    // tiles of one feature tile next to each other, so that they read its weights through one L2
    const int per_xcd = (tiles + 7) / 8, t = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
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
    auto multiply = [&](const Frag &f, int d) {
        Two b[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            b[j].a = *reinterpret_cast<const uint4 *>(stage(d) + b_slot(16 * j + l, q));
            b[j].b = *reinterpret_cast<const uint4 *>(stage(d) + b_slot(16 * j + l, 4 + q));
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = mma<T>(f.a[i], b[j], acc[i][j], f.ix[i]);
    };
    const int nk = K / 64, steps = ks < nk ? (nk - ks + KS - 1) / KS : 0;
    // (Two ways through, so that on the longer one the compiler knows how many copies are in flight behind the one it waits for.)
    Frag f[D];
    int i = 0;
    if (steps >= D) {
#pragma unroll
        for (int d = 0; d < D; ++d) load(f[d], d, ks + KS * d);
        for (; i + 2 * D <= steps; i += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                multiply(f[d], d);
                load(f[d], d, ks + KS * (i + D + d));
            }
        }
#pragma unroll
        for (int d = 0; d < D; ++d) {
            multiply(f[d], d);
            if (i + D + d < steps) load(f[d], d, ks + KS * (i + D + d));
        }
        i += D;
    } else {
#pragma unroll
        for (int d = 0; d < D - 1; ++d)
            if (d < steps) load(f[d], d, ks + KS * d);
    }
#pragma unroll
    for (int d = 0; d < D - 1; ++d)
        if (i + d < steps) multiply(f[d], d);

    // A wave parks its sums in the first two stages of its own ring, rows of 64 TM bytes (a token), quad c of row r at slot c ^ (its swizzle)
    constexpr int ROW = 64 * TM, RPS = WAVE / ROW;   // tokens that a wave's part of a stage holds
    static_assert(2 * RPS >= TWN, "the tile must fit two stages");
    auto parked = [&](int row, int quad) {   // of the first wave
        const int s = TM == 4 ? row & 15 : TM == 2 ? (row >> 1) & 7 : (row >> 2) & 3;
        return reinterpret_cast<float *>((row < RPS ? s0 : s1) + (row % RPS) * ROW + ((quad ^ s) << 4));
    };
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int k = 0; k < TM; ++k)
            *reinterpret_cast<float4 *>(parked(16 * j + l, 4 * k + q) + ks * (WAVE / 4)) = make_float4(acc[k][j][0], acc[k][j][1], acc[k][j][2], acc[k][j][3]);

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
        auto total = [&](const float *s, uint2 add, bool has) {
            float4 v = *reinterpret_cast<const float4 *>(s);
#pragma unroll
            for (int k = 1; k < KS; ++k) {
                const float4 o = *reinterpret_cast<const float4 *>(s + k * (WAVE / 4));
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

template <typename T, bool ACCUM, int EPI, int ACT, int TM, int TN>
void launch(const S24SliceNt &g, hipStream_t st)
{
    constexpr int FM = EPI == S24_SLICE_GLU ? 8 * TM : 16 * TM;
    const int64_t F = g.M / 2, feats = EPI == S24_SLICE_GLU ? F : g.M;
    const int tiles_m = (int)((feats + FM - 1) / FM), tiles_n = (int)((g.N + 16 * TN - 1) / (16 * TN)), tiles = tiles_m * tiles_n;
    const dim3 grid(((tiles + 7) / 8) * 8), block(64 * KS);
#define S24_LAUNCH_SLICE(STREAM)                                                                                                            \
    hipLaunchKernelGGL((spmm_slice_kernel<T, ACCUM, EPI, ACT, TM, TN, STREAM>), grid, block, 0, st, g.B, g.Av, g.Am, (int)g.N, (int)g.K, (int)g.M, \
                       (int)F, tiles_n, tiles, g.Out, g.H, g.Z, g.bias)
    if constexpr (TN == 1) {
        if (tiles_n == 1) {   // every weight is read once
            S24_LAUNCH_SLICE(true);
            return;
        }
    }
    S24_LAUNCH_SLICE(false);
#undef S24_LAUNCH_SLICE
}

template <typename T, int TM, int TN> int launch_epilogue(const S24SliceNt &g, hipStream_t st)
{
    if (g.epilogue == S24_SLICE_PLAIN) {
        if (g.accum) launch<T, true, S24_SLICE_PLAIN, 0, TM, TN>(g, st);
        else launch<T, false, S24_SLICE_PLAIN, 0, TM, TN>(g, st);
    } else if (g.epilogue == S24_SLICE_GLU) {
        constexpr int TG = TM < 2 ? 2 : TM;
        if (g.act == S24_GATE_SILU) launch<T, false, S24_SLICE_GLU, S24_GATE_SILU, TG, TN>(g, st);
        else launch<T, false, S24_SLICE_GLU, S24_GATE_GELU_ERF, TG, TN>(g, st);
    } else if (g.epilogue == S24_SLICE_ACT) {
        if (g.act == S24_ACT_RELU) launch<T, false, S24_SLICE_ACT, S24_ACT_RELU, TM, TN>(g, st);
        else launch<T, false, S24_SLICE_ACT, S24_ACT_GELU_ERF, TM, TN>(g, st);
    } else {
        if (g.act == S24_ACT_RELU) launch<T, false, S24_SLICE_ACT_BWD, S24_ACT_RELU, TM, TN>(g, st);
        else launch<T, false, S24_SLICE_ACT_BWD, S24_ACT_GELU_ERF, TM, TN>(g, st);
    }
    return s24_launch_status();
}

// Tile of a product by its cost in us: a launch, and per round of workgroups over the compute units a filling and draining and so
// much for each 64 of k (fitted to 380 products, 1-2048 tokens, K = 256-32000, 256-56000 features; half of them within 7 %).
// Two workgroups to a compute unit count as two rounds: they share its first-level cache, which is what bounds them.
struct Plan { int tm, tn; double launch, round, chunk, us; };
Plan plan(int64_t N, int64_t K, int64_t M)
{
    constexpr Plan tiles[5] = {{1, 1, 2.2, 0.25, 0.037, 0}, {2, 1, 2.2, 0.25, 0.060, 0}, {4, 1, 2.3, 0.25, 0.105, 0}, {4, 2, 2.1, 0.48, 0.122, 0}, {4, 4, 1.6, 1.2, 0.170, 0}};
    const int64_t cus = s24_cu_count();
    Plan best{};
    for (Plan t : tiles) {
        if (N <= 16 * (t.tn / 2)) continue;   // half of the tile or more would be empty
        const int64_t n = ((M + 16 * t.tm - 1) / (16 * t.tm)) * ((N + 16 * t.tn - 1) / (16 * t.tn)), rounds = (n + cus - 1) / cus;
        t.us = t.launch + (double)rounds * (t.round + t.chunk * (double)(K / 64));
        if (best.tm == 0 || t.us < best.us) best = t;
    }
    return best;
}

}  // namespace

double s24_slice_us(int64_t N, int64_t K, int64_t M) { return plan(N, K, M).us; }

int s24_slice_nt(const S24SliceNt &g, int dt, hipStream_t st)
{
    const Plan p = plan(g.N, g.K, g.M);
    auto with = [&](auto t) {
        using T = decltype(t);
        if (p.tm == 1) return launch_epilogue<T, 1, 1>(g, st);
        if (p.tm == 2) return launch_epilogue<T, 2, 1>(g, st);
        if (p.tn == 1) return launch_epilogue<T, 4, 1>(g, st);
        if (p.tn == 2) return launch_epilogue<T, 4, 2>(g, st);
        return launch_epilogue<T, 4, 4>(g, st);
    };
    return dt == S24_BF16 ? with(uint16_t{}) : with(s24_half{});
}
