// The last input gradient of a layer (sparse NT, in slices) and its weight gradients (dense TN) in one launch, bf16 and binary16.
#include <type_traits>

#include "s24_gemm_joint.h"
#include "s24_slice_tile.h"

namespace {

using namespace s24_lds;
using namespace s24_dw;

// A 128 x 128 tile of a weight gradient of few tokens, by eight waves of 32 (rows of dW) x 64: same tokens to an instruction and same order
// of the sums as in dense_tn_tile (s24_gemm.hip), so the same bits.  With 256 tokens the products are a third of the time and the rest is the way in and out, which more waves with less
// to do each get over sooner; W and the mask are requested before anything else.  s0 .. s3: SHORT_STAGE bytes of LDS each.
constexpr int SHORT_STAGE = 2 * 32 * 256, SHORT_THREADS = 512;
__device__ __forceinline__ f32x4 mfma16(uint16_t, bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f32x4 mfma16(s24_half, bf16x8 a, bf16x8 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}
template <typename ET, bool DECAY>
__device__ __forceinline__ void short_tn_tile(lds_byte *s0, lds_byte *s1, lds_byte *s2, lds_byte *s3, int block, const DwBatch &batch)
{
    constexpr int ROW = 256, OPERAND = 32 * ROW;   // bytes of a token's row in a tile, of an operand in a stage
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave & 3, wn = wave >> 2;
    const int slot = block >> 3;
    int which = 0;
#pragma unroll
    for (int i = 1; i < kMaxBatch; ++i)
        if (slot >= batch.first_slot[i]) which = i;
    const DwWindow &win = batch.w[which];
    const int per_xcd = batch.first_slot[which + 1] - batch.first_slot[which];
    const int t = (block & 7) * per_xcd + (slot - batch.first_slot[which]);
    if (t >= win.tiles_m * win.tiles_n) return;
    const int T = win.T, M = win.M, N = win.N, ldy = win.ldy, ldx = win.ldx, ldw = win.ldw;
    const float lambda = win.lambda;
    constexpr int GROUP = 8;
    const int group_sz = GROUP * win.tiles_m, grp = t / group_sz, in_grp = t - grp * group_sz;
    const int gw = min(GROUP, win.tiles_n - grp * GROUP);
    const int m0 = (in_grp / gw) * 128, n0 = (grp * GROUP + in_grp % gw) * 128;
    const int nk = (T + 31) / 32;

    // The wave's output: row 4 j + lane / 16 of pass j, columns 4 (lane % 16) .. +3.  M is a multiple of 16 and the wave's rows start at a
    // multiple of 32: the four rows of a pass are all inside or all outside; passes and columns past the edge re-read the last ones inside.
    const int mw = m0 + 32 * wm, nw = n0 + 64 * wn;
    uint2 wv[DECAY ? 8 : 1];
    uint32_t keep[DECAY ? 8 : 1];
    if constexpr (DECAY) {
        const int first = min(mw, M - 16), last = ((M - first) >> 2) - 1, nc = min(nw + 4 * (lane & 15), N - 4);
        const rsrc_t wbuf = buffer_of(win.Wt + (int64_t)first * ldw), mbuf = buffer_of(win.mask + (int64_t)(first >> 2) * (ldw >> 2));
        const uint32_t voff_w = ((uint32_t)(lane >> 4) * (uint32_t)ldw + (uint32_t)nc) * 2u, voff_m = (uint32_t)(nc >> 2) * 2u;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t jc = (uint32_t)min(j, last);
            wv[j] = buffer_load_8(wbuf, voff_w, jc * 8u * (uint32_t)ldw);
            keep[j] = buffer_load_2(mbuf, voff_m, jc * 2u * (uint32_t)(ldw >> 2));
        }
    }
    // copies: wave w takes rows 4w .. 4w + 3 of either tile, 16 lanes to a row
    const int crow = 4 * wave + (lane >> 4), cc = (lane & 15) ^ tr_swizzle<ROW>(crow);
    const uint32_t va = (uint32_t)(min(crow, T - 1) * ldy + m0 + 8 * min(cc, (min(M - m0, 128) >> 3) - 1)) * 2u;
    const uint32_t vb = (uint32_t)(min(crow, T - 1) * ldx + n0 + 8 * min(cc, (min(N - n0, 128) >> 3) - 1)) * 2u;
    auto issue = [&](lds_byte *st, int kc) {   // past the last chunk the last one again, into a stage that nobody will read
        const int64_t row = max(min(kc * 32, T - 32), 0);
        buffer_to_lds<16>(buffer_of(win.dY + row * ldy), (lds_ptr)(st + wave * 1024), va);
        buffer_to_lds<16>(buffer_of(win.X + row * ldx), (lds_ptr)(st + OPERAND + wave * 1024), vb);
        __builtin_amdgcn_sched_barrier(0);
    };
    const int gi = lane & 15, G = lane >> 4, frow = 8 * G + (gi >> 2), fcol = 4 * (gi & 3);
    int offA[2], offB[4];
#pragma unroll
    for (int i = 0; i < 2; ++i) offA[i] = tr_off<ROW>(frow, 32 * wm + 16 * i + fcol);
#pragma unroll
    for (int j = 0; j < 4; ++j) offB[j] = OPERAND + tr_off<ROW>(frow, 64 * wn + 16 * j + fcol);
    auto fragment = [&](const lds_byte *p) {
        return join(__builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16)(p)), __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16)(p + 4 * ROW)));
    };
    f32x4 acc[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{};
    __builtin_amdgcn_sched_barrier(0);
    issue(s0, 0);
    issue(s1, 1);
    issue(s2, 2);
    // rows of the last chunk that must not contribute: those that the last whole step covered, or those past T
    auto clear_tail = [&](lds_byte *cur) {
        const int live = T - 32 * (nk - 1), row = T < 32 ? live : 0;
        for (int at = 16 * tid; at < (32 - live) * ROW; at += 16 * SHORT_THREADS) {
            lds_store(cur + row * ROW + at, make_uint4(0, 0, 0, 0));
            lds_store(cur + OPERAND + row * ROW + at, make_uint4(0, 0, 0, 0));
        }
    };
    auto multiply = [&](const lds_byte *cur) {
        bf16x8 fa[2], fb[4];
#pragma unroll
        for (int i = 0; i < 2; ++i) fa[i] = fragment(cur + offA[i]);
#pragma unroll
        for (int j = 0; j < 4; ++j) fb[j] = fragment(cur + offB[j]);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = mfma16(ET{}, fb[j], fa[i], acc[i][j]);
    };
    auto chunk = [&](lds_byte *cur, lds_byte *refill, int kc) {
        wait_and_barrier<4>();   // chunk kc has landed for everybody, and everybody is done with the one before
        issue(refill, kc + 3);
        multiply(cur);
    };
    const int whole = T / 32;
    int kc = 0;
#pragma unroll 1
    for (; kc + 4 <= whole; kc += 4) {
        chunk(s0, s3, kc);
        chunk(s1, s0, kc + 1);
        chunk(s2, s1, kc + 2);
        chunk(s3, s2, kc + 3);
    }
    if (kc < whole) chunk(s0, s3, kc);
    if (kc + 1 < whole) chunk(s1, s0, kc + 1);
    if (kc + 2 < whole) chunk(s2, s1, kc + 2);
    if (whole < nk) {
        lds_byte *cur = whole - kc == 0 ? s0 : whole - kc == 1 ? s1 : whole - kc == 2 ? s2 : s3;
        wait_and_barrier<0>();
        clear_tail(cur);
        __syncthreads();
        multiply(cur);
    }
    wait_and_barrier<0>();   // the last copies have landed and nobody reads the ring any more: half a stage takes a wave's sums
    lds_byte *est = ((wave >> 1) == 0 ? s0 : (wave >> 1) == 1 ? s1 : (wave >> 1) == 2 ? s2 : s3) + (wave & 1) * OPERAND;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) lds_store(est + (16 * i + gi) * ROW + (((4 * j + G) ^ gi) << 4), acc[i][j]);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int row = 4 * j + (lane >> 4), m = mw + row, n = nw + 4 * (lane & 15);
        float4 o = __builtin_bit_cast(float4, lds_load(est + row * ROW + (((lane & 15) ^ (row & 15)) << 4)));
        if (m >= M || n >= N) continue;   // N is a multiple of 16: the four columns are all in or all out
        if constexpr (DECAY) {
            const uint32_t kp = keep[j] >> (4 * (lane >> 4));   // row of the 4 x 4 block: the pass starts at a multiple of four
            if (!(kp & 1u)) o.x = fmaf(lambda, s24_num<ET>::lo(wv[j].x), o.x);
            if (!(kp & 2u)) o.y = fmaf(lambda, s24_num<ET>::hi(wv[j].x), o.y);
            if (!(kp & 4u)) o.z = fmaf(lambda, s24_num<ET>::lo(wv[j].y), o.z);
            if (!(kp & 8u)) o.w = fmaf(lambda, s24_num<ET>::hi(wv[j].y), o.w);
        }
        s24_store_stream(win.dW + (int64_t)m * ldw + n, o);
    }
}

// An input gradient in slices (s24_slice_tile.h) and weight gradients of few tokens that do not depend on it in one launch: neither fills the chip,
// and two workgroups share a compute unit, so that one is on its way to memory while the other one multiplies.  The input gradient's
// workgroups (`dx_blocks`, a multiple of eight) walk the longer sums and go first.  256 tokens x 768 x 3072 (7.8 and 12.2 us under the tracer): 42.6 -> 36.9 us a step.
// first: B, Av; second: Am, dx_blocks, N; third: K, M, tiles of tokens, all tiles of the input gradient
template <typename T, bool DECAY, int TM>
__global__ __launch_bounds__(512, 4) void dx_dw_kernel(const s24_words first, const s24_words second, const s24_words third, uint16_t *Out, const DwBatch batch)
{
    static_assert(s24_slice::stage_bytes(1) == SHORT_STAGE && 64 * s24_slice::KS == SHORT_THREADS, "one ring for either");
    __shared__ __attribute__((aligned(16))) unsigned char s0[SHORT_STAGE];
    __shared__ __attribute__((aligned(16))) unsigned char s1[SHORT_STAGE];
    __shared__ __attribute__((aligned(16))) unsigned char s2[SHORT_STAGE];
    __shared__ __attribute__((aligned(16))) unsigned char s3[SHORT_STAGE];
    lds_byte *const l0 = (lds_byte *)s0, *const l1 = (lds_byte *)s1, *const l2 = (lds_byte *)s2, *const l3 = (lds_byte *)s3;
    const int dx_blocks = s24_low(second.y), M = s24_high(third.x);
    if ((int)blockIdx.x < dx_blocks)
        s24_slice::slice_tile<T, false, S24_SLICE_PLAIN, 0, TM, 1, false>(l0, l1, l2, l3, (int)blockIdx.x, s24_global<const uint16_t>(first.x), s24_global<const uint16_t>(first.y),
                                                                          s24_global<const uint16_t>(second.x), s24_high(second.y), s24_low(third.x), M, M, s24_low(third.y),
                                                                          s24_high(third.y), Out, nullptr, nullptr, nullptr);
    else short_tn_tile<T, DECAY>(l0, l1, l2, l3, (int)blockIdx.x - dx_blocks, batch);
}

}  // namespace

void s24_dx_dw(const S24SliceNt &g, int tm, const DwBatch &batch, bool decay, int dt, hipStream_t st)
{
    const int tiles_n = (int)((g.N + 15) / 16), tiles = (int)((g.M + 16 * tm - 1) / (16 * tm)) * tiles_n, dx_blocks = (tiles + 7) / 8 * 8;
    const dim3 grid(dx_blocks + 8 * batch.first_slot[kMaxBatch]), block(SHORT_THREADS);
    auto launch = [&](auto t, auto dec, auto blocks) {
        hipLaunchKernelGGL((dx_dw_kernel<decltype(t), decltype(dec)::value, decltype(blocks)::value>), grid, block, 0, st, s24_pack(g.B, g.Av), s24_pack(g.Am, dx_blocks, (int)g.N),
                           s24_pack((int)g.K, (int)g.M, tiles_n, tiles), g.Out, batch);
    };
    auto with = [&](auto t, auto dec) {
        if (tm == 1) launch(t, dec, std::integral_constant<int, 1>());
        else if (tm == 2) launch(t, dec, std::integral_constant<int, 2>());
        else launch(t, dec, std::integral_constant<int, 4>());
    };
    if (dt == S24_BF16) {
        if (decay) with(uint16_t{}, std::true_type());
        else with(uint16_t{}, std::false_type());
    } else {
        if (decay) with(s24_half{}, std::true_type());
        else with(s24_half{}, std::false_type());
    }
}
