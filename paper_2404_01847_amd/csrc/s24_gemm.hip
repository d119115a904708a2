// GEMMs of the 2:4-sparse FFN step on gfx950 matrix cores, for bf16 and IEEE binary16 operands alike (fp32
// accumulation; the element type only selects the instruction and the epilogue conversions).
//
//   sparse NT  out[n][m] = sum_k B[n][k] * A[m][k], A 2:4-compressed along k
//              (Eq. 2 with A = W, Eq. 3 with A = W^T): v_smfmac_f32_16x16x64_{bf16,f16},
//              with the activation forward / backward (Sec. 5.2) and the bias as optional epilogues
//   sparse TN  dW = S_z(dY^T) X (Eq. 4): the same instruction, the dense operand read through transposing LDS reads
//   dense  NT  Y = X W^T (Eq. 1, first GEMM; the comparison kernel): v_mfma_f32_16x16x32_{bf16,f16}
//   dense  TN  dW = dY^T X (Eq. 1, third GEMM): v_mfma_f32_16x16x32_{bf16,f16}, both operands copied as they lie in memory,
//              k-contiguous fragments by ds_read_b64_tr_b16; masked decay (Eq. 10) as an optional epilogue
// fp32 data takes the kernels of s24_gemm_f32.hip, sparse NT products of few tokens or features those of s24_gemm_slice.hip.
//
// Register layout of the sparse instruction (one 16x16 tile, 64 of k): lane l holds for A row l%16 the eight kept values of
// k in [16*(l/16), 16*(l/16)+16) in order, with their 2-bit positions in bits [2j+1:2j] of the index register half chosen by
// ABID; for B column l%16, element j holds k = 32*(j/8) + 8*(l/16) + j%8; accumulator i holds row 4*(l/16)+i of column l%16.
// One metadata word (a uint16 per 16 of k) is exactly one lane's index half, and the chunk-major storage of the compressed
// operand (vals[K/64][M][32], meta[K/64][M][4]) makes the 64-byte value run and the
// four index words of one row and chunk contiguous, rows back to back.
#include <algorithm>
#include <type_traits>

#include "s24_dw.h"
#include "s24_gemm_f32.h"
#include "s24_gemm_joint.h"
#include "s24_gemm_slice.h"
#include "s24_lds.h"
#include "s24_overlap.h"

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) __bf16 bf16x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(16))) _Float16 f16x16;

// The 16-bit kernels move operands as raw bits (fragments are typed bf16x8 / bf16x16 whatever they hold); the
// element type T (uint16_t = bf16 bits, s24_half = IEEE binary16) only selects the matrix instruction and the
// conversions of the epilogues.
// c += a b on v_mfma_f32_16x16x32, the accumulator in place.  Written as an instruction because the compiler's own form does
// not tie its result to its accumulator operand: with all 256 accumulation registers in use (the 128 x 128 wave tile) it
// shuffled accumulators between register files, a move per instruction.  The compiler does not pad hazards around it, so
// the distances are kept here: fragments come from LDS reads; what vector instructions compute for it (the cleared
// accumulators, the packed index words) is done when mma_operands passes, two wait states ahead of the next instruction;
// and nobody reads an accumulator until mma_drain has passed, which waits for the matrix unit.  Both name the registers as
// operands, so that no computation of them moves past.  Copies that the register allocator may add are beyond that: a host
// test follows the built library's instructions.
#if defined(__HIP_DEVICE_COMPILE__)
#define S24_MFMA_16X16X32(TYPE, a, b, c) \
    asm volatile("v_mfma_f32_16x16x32_" TYPE " %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b))
#define S24_SMFMAC_16X16X64(TYPE, HALF, a, b, c, idx) \
    asm volatile("v_smfmac_f32_16x16x64_" TYPE " %0, %1, %2, %3 abid:" HALF : "+v"(c) : "v"(a), "v"(b), "v"(idx))
#define S24_TIE(CLASS, x) asm volatile("" : CLASS(x))
#define S24_MMA_WAIT(N) asm volatile(N ::: "memory")
#else
#define S24_MFMA_16X16X32(TYPE, a, b, c) (void)(a), (void)(b), (void)(c)
#define S24_SMFMAC_16X16X64(TYPE, HALF, a, b, c, idx) (void)(a), (void)(b), (void)(c), (void)(idx)
#define S24_TIE(CLASS, x) (void)(x)
#define S24_MMA_WAIT(N) (void)0
#endif
// the register class of the accumulators: "a" for the dense instruction, "v" for the sparse one
enum MmaRegs { ACC_AGPR, ACC_VGPR };
template <MmaRegs REGS, int R, int C> __device__ __forceinline__ void mma_tie(f32x4 (&acc)[R][C])
{
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
        for (int j = 0; j < C; ++j) {
            if constexpr (REGS == ACC_AGPR) S24_TIE("+a", acc[i][j]);
            else S24_TIE("+v", acc[i][j]);
        }
}
template <int FIRST, int COUNT, int N> __device__ __forceinline__ void mma_tie(uint32_t (&idx)[N])
{
#pragma unroll
    for (int i = FIRST; i < FIRST + COUNT; ++i) S24_TIE("+v", idx[i]);
}
// The ties above come before the two wait states and, being volatile as the instructions are, these before any of those.
__device__ __forceinline__ void mma_operands() { S24_MMA_WAIT("s_nop 1"); }
template <MmaRegs REGS, int R, int C> __device__ __forceinline__ void mma_drain(f32x4 (&acc)[R][C])
{
    S24_MMA_WAIT("s_nop 15\n\ts_nop 15");
    mma_tie<REGS>(acc);
}
template <typename T> struct Mma;
template <> struct Mma<uint16_t> {
    static __device__ __forceinline__ void dense16(bf16x8 a, bf16x8 b, f32x4 &c) { S24_MFMA_16X16X32("bf16", a, b, c); }
    template <int ABID> static __device__ __forceinline__ void sparse16(bf16x8 a, bf16x16 b, f32x4 &c, uint32_t idx)
    {
        if constexpr (ABID == 0) S24_SMFMAC_16X16X64("bf16", "0", a, b, c, idx);
        else S24_SMFMAC_16X16X64("bf16", "1", a, b, c, idx);
    }
};
template <> struct Mma<s24_half> {
    static __device__ __forceinline__ void dense16(bf16x8 a, bf16x8 b, f32x4 &c) { S24_MFMA_16X16X32("f16", a, b, c); }
    template <int ABID> static __device__ __forceinline__ void sparse16(bf16x8 a, bf16x16 b, f32x4 &c, uint32_t idx)
    {
        if constexpr (ABID == 0) S24_SMFMAC_16X16X64("f16", "0", a, b, c, idx);
        else S24_SMFMAC_16X16X64("f16", "1", a, b, c, idx);
    }
};

constexpr int kThreads = 256;

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }
__device__ __forceinline__ bf16x16 as_bf16x16(uint4 lo, uint4 hi)
{
    struct { uint4 a, b; } t{lo, hi};
    return __builtin_bit_cast(bf16x16, t);
}

// ------------------------------------------------------------------ sparse NT
// Large tile: workgroup tile 256 (m) x 256 (n) x 64 (k), eight waves as 2 (m) x 4 (n), each
// wave 128 x 64 = 8 x 4 accumulator blocks of 16 x 16.  Both operands are copied from
// global memory straight into LDS (no register staging) through a ring of
// three 50 KB stages; the one barrier of a chunk sits between its two halves, where the matrix unit
// still has the second half's operands in registers, and the copies of chunk kc+3 go out from that barrier to the next
// (see the main loop).  LDS layouts: dense operand rows of 128 bytes with the
// 16-byte chunk c of row r at slot c ^ ((r>>1) & 7); compressed operand
// rows of 64 bytes with chunk c at slot c ^ (-(r>>2) & 3).  A full-rate 128-bit LDS read needs distinct 16-byte slots modulo
// 256 bytes in each group of 16 lanes it takes at a time, which are lanes 0-3, 12-15 and 20-27 (and 4-11, 16-19, 28-31) of
// each half wave: rows 0-3 and 12-15 of one k quarter beside rows 4-11 of the next.  Both layouts give that, and for 16
// consecutive rows of one quarter (c ^ (r>>2) alone does not: 260 conflict cycles per chunk of 1600).
// The 16-wide sparse instruction alone holds 1.81 GHz where the 32-wide one holds 1.62 (3.65 against 3.31 PFLOP/s
// dense-equivalent on random operands, in one job).  What bounds the kernel is the path of the copies together with that clock:
// 8192 x 8192 x 28672 1719 -> 1656 us, with M and K exchanged 1626 -> 1566, 16384 x 5120, K = 1280 122 -> 114 (short runs on a
// card not yet warm; the second product launched on end takes 1.85-1.92 ms at 1.36-1.41 GHz, on zero operands 1.34 at 2.3).
namespace big {
constexpr int BM = 256, BN = 256, THREADS = 512;   // the large tile
using namespace s24_lds;

// Clock probe (instrumentation, off unless a buffer is registered): workgroup 0 of a large-tile kernel
// reports how many core-clock cycles and how many ticks of the fixed 100 MHz reference passed between its
// first and its last instruction.  Their ratio is the core clock the chip sustained under this kernel.
struct ClockStamp { unsigned long long cycles, ticks; };
__device__ __forceinline__ ClockStamp clock_now()
{
    return {__builtin_readcyclecounter(), __builtin_amdgcn_s_memrealtime()};
}
__device__ __forceinline__ void clock_report(unsigned long long *probe, const ClockStamp &t0)
{
    if (probe != nullptr && blockIdx.x == 0 && threadIdx.x == 0) {
        const ClockStamp t1 = clock_now();
        probe[0] = t1.cycles - t0.cycles;
        probe[1] = t1.ticks - t0.ticks;
    }
}

// Output of one wave's 64 (n) x 32 MI (m) accumulator tile as bf16.  The wave parks the tile in LDS as
// 64 rows of 64 MI bytes and streams it out 16 bytes per lane, LPR lanes covering one row
// segment of the output.  Inside a row the 8-byte unit u is stored at u ^ stage_swizzle(row), an even number, so the
// accumulator writes of 32 lanes (16 rows, two neighbouring units) fall on distinct banks and a 16-byte piece stays whole.
// `estage` is EWAVE bytes of LDS private to the wave and no longer used for anything else.
// MI = 4: 128 features, rows of 256 bytes; 2: 64 features, rows of 128 bytes, two to a round of the banks.
constexpr int EWAVE = 64 * 256;
template <int MI> __device__ __forceinline__ int stage_swizzle(int nl) { return MI == 4 ? 2 * (nl & 15) : 2 * ((nl >> 1) & 7); }
template <typename T, int MI>
__device__ __forceinline__ void stage_tile(const f32x4 (&acc)[2 * MI][4], unsigned char *estage, int lane)
{
    constexpr int RB = 64 * MI;
#pragma unroll
    for (int ni = 0; ni < 4; ++ni)
#pragma unroll
        for (int mi = 0; mi < 2 * MI; ++mi) {
            const int nl = 16 * ni + (lane & 15), u = 4 * mi + (lane >> 4);
            *reinterpret_cast<uint2 *>(estage + nl * RB + ((u ^ stage_swizzle<MI>(nl)) << 3)) =
                make_uint2(s24_num<T>::pack2(acc[mi][ni][0], acc[mi][ni][1]), s24_num<T>::pack2(acc[mi][ni][2], acc[mi][ni][3]));
        }
}
// Z = X W^T + d (Sec. 5.2 step 2): adds the bias of output feature m to the wave's 32 MI (m) x 64 (n) accumulator
// tile before it is rounded.  `bias` points at the entry of the tile's first feature; features at or past `limit`
// (edge tiles; never stored) read the last four valid entries instead.
template <typename T, int MI>
__device__ __forceinline__ void add_bias(f32x4 (&acc)[2 * MI][4], const uint16_t *__restrict__ bias, int limit, int lane)
{
#pragma unroll
    for (int mi = 0; mi < 2 * MI; ++mi) {
        const int m = min(16 * mi + 4 * (lane >> 4), limit - 4);
        const uint2 b = *reinterpret_cast<const uint2 *>(bias + m);
        const float b4[4] = {s24_num<T>::lo(b.x), s24_num<T>::hi(b.x), s24_num<T>::lo(b.y), s24_num<T>::hi(b.y)};
#pragma unroll
        for (int ni = 0; ni < 4; ++ni)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[mi][ni][e] += b4[e];
        // four loads in flight at a time: all at once would not fit beside the accumulators
        if (mi % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
}
// 16-byte chunk c (eight bf16, columns 8c .. 8c+7) of row nl of a staged tile
template <int MI = 4> __device__ __forceinline__ uint4 staged_chunk(const unsigned char *estage, int nl, int c)
{
    return *reinterpret_cast<const uint4 *>(estage + nl * (64 * MI) + (((2 * c) ^ stage_swizzle<MI>(nl)) << 3));
}
template <typename T, int MI>
__device__ __forceinline__ void staged_store(const f32x4 (&acc)[2 * MI][4], unsigned char *estage, uint16_t *__restrict__ Out,
                                             int N, int M, int n_base, int m_base, int lane)
{
    stage_tile<T, MI>(acc, estage, lane);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0(0));   // the wave reads back only what it wrote itself
    asm volatile("" ::: "memory");
    constexpr int LPR = 4 * MI;   // lanes per row of the tile (16-byte pieces)
#pragma unroll 4
    for (int j = 0; j < LPR; ++j) {
        const int nl = (64 / LPR) * j + lane / LPR, c = lane % LPR;
        const int n = n_base + nl, m = m_base + 8 * c;
        if (n >= N || m >= M) continue;   // M is a multiple of 16 (and of 8): a chunk is all in or all out
        *reinterpret_cast<uint4 *>(Out + (int64_t)n * M + m) = staged_chunk<MI>(estage, nl, c);
    }
}

// GELU, or its slope, of bf16 values from a table in LDS.  A bf16 value between 2^-EXP and 16 is one of 128 per octave and sign, so a
// workgroup computes each of them once (9 to 20 per lane) instead of 128 or 64 tile elements per lane at 26 to 29 issue slots
// each, two of the instructions on the quarter-rate unit: on a tile of 20 chunks that arithmetic was a third of the time.  An element then
// costs four packed 16-bit instructions and an LDS read, and has the bits that the function gives it.  Zeros (padded tokens) and finite
// values from 16 on (a feature that is an outlier) send the wave's eight at a time through a longer lookup with the function's limits.
// Infinities, NaNs and the smallest values send them to the function: one in 1e4 normally distributed values of
// the usual spread.  Not for binary16, whose octaves have 1024 values.  16384 tokens, K = 1280, 5120 features, alternating on one card,
// the function alone and now: forward 168 -> 144 us, backward 185 -> 161 (with ReLU, another card, 134 and 139); 4160, 1600, 6400: 69 -> 62 and
// 74 -> 67; in the 128 x 128 tile, whose lanes have half as many elements to a table, 8192, 768, 3072: 48 -> 44 and 47 -> 45.
// Every other token zero: 157 -> 145 and 187 -> 169, 66 -> 63 and 74 -> 70, 44.8 -> 45.7 and 46.4 -> 47.3; the last half of them: 158 -> 140 and
// 185 -> 161, 67 -> 61 and 74 -> 69, 45.1 -> 43.7 and 45.8 -> 46.1; one feature in 128 past 16: 171 -> 161 and 187 -> 170, 71 -> 68 and 74 -> 71, 49.5 -> 48.4
// and 47.4 -> 47.7 (with the function for those, 177 and 189, 73 and 78, 52 and 48).
template <int ACT_MODE, int ACT> struct ActTable {
    typedef std::conditional_t<ACT_MODE == 1, uint16_t, float> entry;   // H as it is stored; the slope is multiplied before it is rounded
    static constexpr int EXP = ACT_MODE == 1 ? 16 : 14, FIRST = (127 - EXP) << 7, COUNT = (EXP + 4) << 7;   // of either sign
    static constexpr int BYTES = 2 * COUNT * (int)sizeof(entry);
    typedef std::conditional_t<ACT_MODE == 1, uint32_t, float2> pair;   // of two neighbours
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

    static __device__ __forceinline__ entry value(float z)
    {
        if constexpr (ACT_MODE == 1) return (uint16_t)s24_f32_to_bf16(s24_act_value<ACT>(z));
        else return s24_act_slope<ACT>(z);
    }
    // by the whole workgroup; readable after a barrier
    template <int THREADS> static __device__ __forceinline__ void build(entry *tab, int tid)
    {
        static_assert(COUNT % 128 == 0, "whole waves");
        for (int i = tid; i < COUNT; i += THREADS) {   // both signs together: they share most of the arithmetic
            const float z = s24_num<uint16_t>::widen(FIRST + i);
            tab[i] = value(z);
            tab[COUNT + i] = value(-z);
        }
    }
    static __device__ __forceinline__ pair join(entry lo, entry hi)
    {
        if constexpr (ACT_MODE == 1) return lo | ((uint32_t)hi << 16);
        else return make_float2(lo, hi);
    }
    // of the eight values in z
    static __device__ __forceinline__ void lookup(const entry *tab, const uint32_t (&z)[4], pair (&out)[4])
    {
        constexpr unsigned short ABS = 0x7FFF, INF = 0x7F80, N = COUNT;
        u16x2 at[4], far = {0, 0};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const u16x2 b = __builtin_bit_cast(u16x2, z[k]), from_first = (b & ABS) - (unsigned short)FIRST;
            far = __builtin_elementwise_max(far, from_first);
            at[k] = (b >> (unsigned short)15) * N + from_first;
        }
        if (!__any(far.x >= COUNT || far.y >= COUNT)) {
#pragma unroll
            for (int k = 0; k < 4; ++k) out[k] = join(tab[at[k].x], tab[at[k].y]);
            return;
        }
        u16x2 most = {0, 0}, least = {0xFFFF, 0xFFFF};   // of the magnitudes, and of those that are not zero, less one
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const u16x2 mag = __builtin_bit_cast(u16x2, z[k]) & ABS;
            most = __builtin_elementwise_max(most, mag);
            least = __builtin_elementwise_min(least, mag - (unsigned short)1);
        }
        if (__any(most.x >= INF || most.y >= INF || least.x < FIRST - 1 || least.y < FIRST - 1)) {
#pragma unroll
            for (int k = 0; k < 4; ++k) out[k] = join(value(s24_num<uint16_t>::lo(z[k])), value(s24_num<uint16_t>::hi(z[k])));
            return;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {   // from 16 on the entry of the largest value below it, which is the limit of either sign but of H itself
            const u16x2 b = __builtin_bit_cast(u16x2, z[k]), from_first = (b & ABS) - (unsigned short)FIRST, last = {N - 1, N - 1};
            const u16x2 a = (b >> (unsigned short)15) * N + __builtin_elementwise_min(from_first, last);
            const entry lo = tab[a.x], hi = tab[a.y];
            if constexpr (ACT_MODE == 1) {   // beyond the table H is z where that is positive or zero, and else minus zero
                const u16x2 past = __builtin_elementwise_min(__builtin_elementwise_sub_sat(from_first, last), (u16x2){1, 1}) * (unsigned short)0xFFFF;
                const uint32_t mask = __builtin_bit_cast(uint32_t, past), h = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(b, (u16x2){0x8000, 0x8000}));
                out[k] = (h & mask) | (join(lo, hi) & ~mask);
            } else {
                out[k] = make_float2((z[k] & 0x7FFFu) == 0 ? value(0.0f) : lo, (z[k] & 0x7FFF0000u) == 0 ? value(0.0f) : hi);
            }
        }
    }
};

constexpr int spmm_stage(int MI, int WN) { return 64 * WN * 128 + 64 * MI * (64 + 8); }   // tokens, values, index words of a chunk

// ACT_MODE 1 (forward of an ungated layer): the rounded tile Z is written to Out and H = act(Z) beside it, as the
// stand-alone activation kernel would form it from the stored Z.  ACT_MODE 2 (input gradient of the second
// projection): the rounded tile of dH is not written but multiplied by act'(Z), Z read from `GU`, into Out = dZ.
// SWIGLU (forward of a gated layer, Sec. 5.2): the compressed operand holds the gate rows [0, F) and the up rows
// [F, 2F) of one stacked weight (M = 2F).  A workgroup tile then takes 128 gate features and the 128 up features
// of the same indices, its epilogue pairs them and writes G and U (the halves of Out, row stride M) and
// H = act(G) * U (row stride F, act = SiLU or GELU by GATE), G and U rounded to the storage type before H is formed,
// as the stand-alone kernel sees them.  A bias d[2F] (Sec. 5.2 step 2), if given, is added before that rounding.
// GATE_BWD (input gradient of the down projection of a gated layer): the tile of dH = dY (M.*W_down) is not
// written; its rounding to the storage type goes straight into the backward of the activation, dG = dH U act'(G),
// dU = dH act(G), with G and U read from, and dG and dU written to, the halves of [N][2M] buffers.
// T is the storage type of every 16-bit buffer (bf16 bits or binary16).
// BIAS compiles the bias add into the plain forward kernel (the gated forward tests the pointer at run time; the
// plain kernel without a bias keeps its register budget, which the extra loads would push into scratch).
// The tile of workgroup `block`; s0 .. s2: spmm_stage(MI, WN) bytes of LDS each.  (One array per ring stage, and this in line: the compiler then knows which
// stage a direct-to-LDS copy writes and does not make reads of the other stages wait for it.)
template <typename T, bool ACCUM, bool SWIGLU, bool GATE_BWD, int GATE, bool BIAS, int ACT_MODE, int ACT, int MI, int WN>
__device__ __forceinline__ void spmm_nt_tile(unsigned char *s0, unsigned char *s1, unsigned char *s2, unsigned block, const uint16_t *__restrict__ B,
                                             const uint16_t *__restrict__ Av, const uint16_t *__restrict__ Am, uint16_t *__restrict__ Out, int N, int K,
                                             int M, int tiles_m, int tiles_n, unsigned long long *probe, uint16_t *__restrict__ H, int F,
                                             const uint16_t *__restrict__ GU, const uint16_t *__restrict__ bias)
{
    static_assert(!(ACCUM && (SWIGLU || GATE_BWD)) && !(SWIGLU && GATE_BWD), "the gated epilogues overwrite");
    static_assert(ACT_MODE == 0 || !(ACCUM || SWIGLU || GATE_BWD), "one epilogue at a time");
    // MI = accumulator blocks per wave along m, WN = waves along n (two along m).  MI 4, WN 4: the 256 x 256 tile of eight
    // waves (128 x 64 each).  MI 2, WN 2: a 128 x 128 tile of four waves (64 x 64 each) on 25 KB stages, two workgroups
    // per compute unit; every epilogue but the gated ones.  MI 4, WN 2: a 256 (m) x 128 (n) tile of four waves (128 x 64
    // each) on 34 KB stages.  The two smaller ones are for outputs with too few large tiles to fill the chip.  What
    // bounds them is LDS: a chunk of the small tile is 25 KB written and 50 KB read, 600 cycles at 128 bytes each, of
    // which the matrix cores need 256; the medium one has 34 + 68 KB for twice the work.
    static_assert((MI == 4 && (WN == 4 || WN == 2)) || (MI == 2 && WN == 2 && !SWIGLU && !GATE_BWD), "the small tile has no gated epilogue");
    constexpr int BM = 64 * MI, BN = 64 * WN, WM = 32 * MI;   // workgroup tile, wave tile along m
    constexpr int NA = 2 * MI / WN, NX = MI / WN, NC = 4 + NA + NX;   // copies per lane and chunk: values, index words, all
    constexpr int B_STAGE = BN * 128, A_STAGE = BM * 64, M_STAGE = BM * 8, STAGE = B_STAGE + A_STAGE + M_STAGE;
    const ClockStamp t_start = clock_now();
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform, kept in a scalar register
    const int wm = wave & 1, wn = wave >> 1;
    // Workgroups are dealt round-robin to the eight XCDs; give each XCD one contiguous
    // slab of the tile grid and walk it in groups of eight n-tiles so that the
    // workgroups resident on one XCD share operand rows in its L2.
    const int total = tiles_m * tiles_n, per_xcd = (total + 7) / 8;
    const int t = (int)(block & 7) * per_xcd + (int)(block >> 3);
    if (t >= total) return;
    constexpr int GROUP = 4;   // 4 token tiles x 8 feature tiles resident per XCD: least unique bytes per round
    const int group_sz = GROUP * tiles_m, grp = t / group_sz, in_grp = t - grp * group_sz;
    const int gw = min(GROUP, tiles_n - grp * GROUP);
    const int tm = in_grp / gw, tn = grp * GROUP + in_grp % gw;
    const int m0 = SWIGLU ? tm * 128 : tm * BM, n0 = tn * BN;   // SWIGLU: m0 = first feature of the tile
    const int nk = K / 64;
    // row of the compressed operand behind tile row i (clamped at the edge; such rows are never stored)
    auto a_row = [&](int i) {
        if (SWIGLU) return (i < 128 ? 0 : F) + min(m0 + (i & 127), F - 1);
        return min(m0 + i, M - 1);
    };

    // Sources of the direct-to-LDS copies: a wave-uniform base per operand (advanced by one chunk per stage, in
    // scalar registers: the base of a buffer descriptor) plus a fixed 32-bit byte offset per lane, so that seven
    // copies cost seven address registers and no vector arithmetic
    const char *baseB = reinterpret_cast<const char *>(B + (int64_t)n0 * K);
    const char *baseV = reinterpret_cast<const char *>(Av), *baseM = reinterpret_cast<const char *>(Am);
    uint32_t ob[4], oa[NA], om[NX];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = 32 * wave + 8 * i + (lane >> 3);
        const int c = (lane & 7) ^ ((row >> 1) & 7);
        ob[i] = ((uint32_t)(min(n0 + row, N - 1) - n0) * (uint32_t)K + 8u * c) * 2u;   // a tile's rows span < 4 GB (host check)
    }
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int row = 16 * NA * wave + 16 * i + (lane >> 2);
        const int c = (lane & 3) ^ a_swizzle(row);
        oa[i] = ((uint32_t)a_row(row) * 32u + 8u * c) * 2u;
    }
    // index words: 4-byte direct-to-LDS copies (copy i: row 32 * (NX * wave + i) + lane/2, dword lane%2)
#pragma unroll
    for (int i = 0; i < NX; ++i) om[i] = ((uint32_t)a_row(32 * (NX * wave + i) + (lane >> 1)) * 4u + 2u * (lane & 1)) * 2u;
    // Copy c of a chunk's NC per lane: four of the dense operand, NA of the values, NX of the index words.  Every chunk
    // issues all of them, so the wait counts below are constants; past the last chunk the last one is read again into a
    // stage nobody will read.  pb, pv, pm: the operands at the chunk.
    const char *pb = baseB, *pv = baseV, *pm = baseM;
    auto issue = [&](unsigned char *st, int c) {
        if (c < 4) buffer_to_lds<16>(buffer_of(pb), (lds_ptr)(st + (32 * wave + 8 * c) * 128), ob[c]);
        else if (c < 4 + NA) buffer_to_lds<16>(buffer_of(pv), (lds_ptr)(st + B_STAGE + 16 * (NA * wave + c - 4) * 64), oa[c - 4]);
        else buffer_to_lds<4>(buffer_of(pm), (lds_ptr)(st + B_STAGE + A_STAGE + 256 * (NX * wave + c - 4 - NA)), om[c - 4 - NA]);
    };
    // Copy c of the chunk after next but one goes out beside the copy_slot(c)-th matrix instruction from the start of phase B
    // (see the main loop), EARLY of them in that phase and the rest in phase A of the next chunk: spread over all of a
    // chunk's 8 MI instructions, not its second half, the copies queue less (28672 features, K = 8192: 1627 -> 1575 us, and
    // with the waves in phase B preferred, whose copies are the next to be waited for, 1566; twice as dense instead: 1740).
    constexpr auto copy_slot = [](int c) { return c * 8 * MI / NC; };
    constexpr int EARLY = (NC + 1) / 2;
    const int64_t step_v = (int64_t)M * 64, step_m = (int64_t)M * 8;
    auto advance = [&](int kc) {   // to chunk kc, or not past the last one
        if (kc < nk) { pb += 128; pv += step_v; pm += step_m; }
    };
    auto issue_all = [&](unsigned char *st, int kc) {
        if (kc > 0) advance(kc);
#pragma unroll
        for (int c = 0; c < NC; ++c) issue(st, c);
    };

    f32x4 acc[2 * MI][4];
#pragma unroll
    for (int mi = 0; mi < 2 * MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < 4; ++ni) acc[mi][ni] = f32x4{};

    // Fragments of a stage: tokens 16 ni .. of the wave, whole 64-chunk (two LDS reads); features 16 mi .. (one read)
    const int l16 = lane & 15, g = lane >> 4;
    auto load_b = [&](const unsigned char *st, int ni, int h) {
        return *reinterpret_cast<const uint4 *>(st + 2048 * ni + b_slot(64 * wn + l16, 4 * h + g));
    };
    auto load_a = [&](const unsigned char *st, int mi) {
        return as_bf16x8(*reinterpret_cast<const uint4 *>(st + B_STAGE + 1024 * mi + a_slot(WM * wm + l16, g)));
    };
    // the index words of feature blocks 2i and 2i + 1: a lane reads a dword of each (32 of k, two words) and packs its half of both
    const uint32_t half_sel = (g & 1) ? 0x07060302u : 0x05040100u;
    auto load_index = [&](const unsigned char *st, int i) {
        const unsigned char *p = st + B_STAGE + A_STAGE + 256 * i + (WM * wm + l16) * 8 + 4 * (g >> 1);
        return make_uint2(*reinterpret_cast<const uint32_t *>(p), *reinterpret_cast<const uint32_t *>(p + 128));
    };
    auto pack_index = [&](uint2 d) { return __builtin_amdgcn_perm(d.y, d.x, half_sel); };

    // The activation's table, where it serves: H's fits beside the ring of the two larger tiles and is computed under the first copies,
    // the other ones lie in the part of the drained ring that parks no tile.
    typedef ActTable<ACT_MODE, ACT> Table;
    constexpr bool TABLE = ACT_MODE != 0 && ACT == S24_ACT_GELU_ERF && std::is_same_v<T, uint16_t>;
    constexpr bool EARLY_TABLE = TABLE && ACT_MODE == 1 && MI == 4;
    constexpr int PARKED = MI == 4 && WN == 4 ? 2 * EWAVE : 0;   // in s2
    static_assert(!TABLE || EARLY_TABLE || PARKED + Table::BYTES <= STAGE, "the table must fit");
    typename Table::entry *table = reinterpret_cast<typename Table::entry *>(s2 + PARKED);
    if constexpr (EARLY_TABLE) {
        __shared__ typename Table::entry s_table[2 * Table::COUNT];
        table = s_table;
    }

    // keep the program order of these groups: the constant wait counts rely on it
    issue_all(s0, 0);
    __builtin_amdgcn_sched_barrier(0);
    issue_all(s1, 1);
    __builtin_amdgcn_sched_barrier(0);
    advance(2);
#pragma unroll
    for (int c = 0; c < EARLY; ++c) issue(s2, c);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (EARLY_TABLE) Table::template build<128 * WN>(table, tid);
    wait_and_barrier<NC + EARLY>();   // chunk 0 has landed for everybody
    uint4 fb[4][2];      // token fragments of the chunk about to be multiplied, first-half feature fragments and index words
    bf16x8 fa0[MI];
    uint32_t ix[MI];     // of feature blocks 2i and 2i + 1; the first half of them on entry to a chunk
#pragma unroll
    for (int i = 0; i < MI / 2; ++i) ix[i] = pack_index(load_index(s0, i));
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) fa0[mi] = load_a(s0, mi);
#pragma unroll
    for (int ni = 0; ni < 4; ++ni)
#pragma unroll
        for (int h = 0; h < 2; ++h) fb[ni][h] = load_b(s0, ni, h);
    mma_tie<0, MI / 2>(ix);
    mma_tie<ACC_VGPR>(acc);
    mma_operands();

    // One chunk, software-pipelined across the workgroup barrier.  On entry the token fragments of chunk kc and the first
    // half of its feature fragments are in registers.  Phase A: their 4 MI matrix instructions, with the LDS reads of the
    // second half's features between them.  Then the one barrier of the chunk: every wave has read all it needs of chunk
    // kc's stage, and chunk kc+1 (copied two chunks ago) has landed for everybody.  Phase B: the second half's
    // matrix instructions, whose operands are already in registers -- so the matrix unit has work while
    // the fragments of chunk kc+1 come in from LDS, the token fragments each into the registers of the one that has just had its
    // last use, and the copies of chunk kc+3 begin to go out into the stage chunk kc just vacated (one at a time, see copy_slot;
    // the others in phase A of the next chunk).  A barrier at the
    // top of the chunk instead, with nothing in registers, exposed the LDS latency of twelve reads per wave once per chunk.
    auto chunk = [&](unsigned char *cur, const unsigned char *nxt, unsigned char *prv, int kc) {
        bf16x8 fa1[MI];
        uint2 raw[MI / 2];
        auto multiply = [&](const bf16x8 (&a)[MI], int first, int i) {   // the i-th matrix instruction of a phase
            const int ni = i / MI, j = i % MI, b = (ni & 1) ? MI - 1 - j : j, mi = first + b;
            if (mi & 1) Mma<T>::template sparse16<1>(a[b], as_bf16x16(fb[ni][0], fb[ni][1]), acc[mi][ni], ix[mi / 2]);
            else Mma<T>::template sparse16<0>(a[b], as_bf16x16(fb[ni][0], fb[ni][1]), acc[mi][ni], ix[mi / 2]);
            __builtin_amdgcn_sched_barrier(0);
        };
#pragma unroll
        for (int i = 0; i < 4 * MI; ++i) {
            multiply(fa0, 0, i);
            if (i < MI) fa1[i] = load_a(cur, MI + i);
            if (i >= MI && i < MI + MI / 2) raw[i - MI] = load_index(cur, MI / 2 + i - MI);
#pragma unroll
            for (int c = EARLY; c < NC; ++c)
                if (copy_slot(c) - 4 * MI == i) issue(prv, c);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = 0; i < MI / 2; ++i) ix[MI / 2 + i] = pack_index(raw[i]);
        mma_tie<MI / 2, MI / 2>(ix);   // the wait and the barrier below are the wait states
        advance(kc + 3);
        // all but the NC most recent copies (chunk kc+2) are complete: this lane's part of chunk kc+1 is in LDS,
        // and its own LDS reads of chunk kc are done
        wait_and_barrier<NC>();
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int i = 0; i < 4 * MI; ++i) {
            multiply(fa1, MI, i);
            if (i < MI) fa0[i] = load_a(nxt, i);
            if (i >= MI / 2 && i < MI) raw[i - MI / 2] = load_index(nxt, i - MI / 2);
            if (i % MI == (i + 1 < 4 * MI ? 0 : MI - 1) && i >= MI) {   // a token block is done: its successor's two reads
                const int ni = i + 1 < 4 * MI ? i / MI - 1 : 3;
                if (i + 1 == 4 * MI) __builtin_amdgcn_sched_barrier(0);
                fb[ni][0] = load_b(nxt, ni, 0);
                fb[ni][1] = load_b(nxt, ni, 1);
            }
#pragma unroll
            for (int c = 0; c < EARLY; ++c)
                if (copy_slot(c) == i) issue(cur, c);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = 0; i < MI / 2; ++i) ix[i] = pack_index(raw[i]);
        mma_tie<0, MI / 2>(ix);
        mma_operands();
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_sched_barrier(0);
    };
    // past the last chunk the prefetched fragments come from a stage that holds a re-read of the last chunk (or
    // is being refilled with one); they are never multiplied
    int kc = 0;
    for (; kc + 3 <= nk; kc += 3) {
        chunk(s0, s1, s2, kc);
        chunk(s1, s2, s0, kc + 1);
        chunk(s2, s0, s1, kc + 2);
    }
    if (kc < nk) chunk(s0, s1, s2, kc);
    if (kc + 1 < nk) chunk(s1, s2, s0, kc + 1);
    mma_drain<ACC_VGPR>(acc);
    // drain the copies still in flight, then reuse the ring as a staging area for the output tile
    wait_and_barrier<0>();
    clock_report(probe, t_start);
    if constexpr (ACCUM) {
        // beta = 1: add the old output in fp32 straight from the accumulators (a single rounding)
#pragma unroll
        for (int ni = 0; ni < 4; ++ni) {
            const int n = n0 + 64 * wn + 16 * ni + l16;
            if (n >= N) continue;
#pragma unroll
            for (int mi = 0; mi < 2 * MI; ++mi) {
                const int m = m0 + WM * wm + 16 * mi + 4 * g;
                if (m >= M) continue;
                uint2 *dst = reinterpret_cast<uint2 *>(Out + (int64_t)n * M + m);
                const uint2 old = *dst;
                *dst = make_uint2(s24_num<T>::pack2(acc[mi][ni][0] + s24_num<T>::lo(old.x), acc[mi][ni][1] + s24_num<T>::hi(old.x)),
                                  s24_num<T>::pack2(acc[mi][ni][2] + s24_num<T>::lo(old.y), acc[mi][ni][3] + s24_num<T>::hi(old.y)));
            }
        }
        return;
    }
    // a wave's parking area for its output tile (64 rows of 64 MI bytes) in the drained ring
    static_assert((WN == 4 ? 3 : 2) * (EWAVE * MI / 4) <= STAGE, "wave tiles must fit the ring stages");
    auto region = [&](int w) {
        if constexpr (MI == 4 && WN == 2) return (w < 2 ? s0 : s1) + (w & 1) * EWAVE;
        else if constexpr (MI == 4) return (w < 3 ? s0 : (w < 6 ? s1 : s2)) + (w % 3) * EWAVE;
        else return (w < 2 ? s0 : s1) + (w & 1) * (EWAVE / 2);
    };
    if constexpr (SWIGLU) {
        if (bias != nullptr) add_bias<T, MI>(acc, bias + (wm ? F : 0) + m0, F - m0, lane);   // wave-uniform
    } else if constexpr (BIAS) {
        add_bias<T, MI>(acc, bias + m0 + WM * wm, M - (m0 + WM * wm), lane);   // launched only with a bias
    }
    if constexpr (GATE_BWD) {
        unsigned char *est = region(wave);
        stage_tile<T, 4>(acc, est, lane);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0(0));   // the wave reads back only what it wrote itself
        asm volatile("" ::: "memory");
        const int n_base = n0 + 64 * wn, m_base = m0 + 128 * wm;
        // the accumulators are dead now: all 32 loads of G and U go out before anything is computed
        const int c = lane & 15, m = min(m_base + 8 * c, M - 8);
        uint4 g[16], u[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int64_t o = (int64_t)min(n_base + 4 * j + (lane >> 4), N - 1) * 2 * M + m;
            g[j] = s24_load_stream(GU + o);
            u[j] = s24_load_stream(GU + o + M);
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int nl = 4 * j + (lane >> 4), n = n_base + nl;
            const uint4 dh = staged_chunk(est, nl, c);
            const uint32_t dw[4] = {dh.x, dh.y, dh.z, dh.w}, gw[4] = {g[j].x, g[j].y, g[j].z, g[j].w};
            const uint32_t uw[4] = {u[j].x, u[j].y, u[j].z, u[j].w};
            uint32_t dgw[4], duw[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                float dg0, du0, dg1, du1;
                s24_glu_grad<GATE>(s24_num<T>::lo(dw[k]), s24_num<T>::lo(gw[k]), s24_num<T>::lo(uw[k]), dg0, du0);
                s24_glu_grad<GATE>(s24_num<T>::hi(dw[k]), s24_num<T>::hi(gw[k]), s24_num<T>::hi(uw[k]), dg1, du1);
                dgw[k] = s24_num<T>::pack2(dg0, dg1);
                duw[k] = s24_num<T>::pack2(du0, du1);
            }
            if (n < N && m_base + 8 * c < M) {   // M is a multiple of 16: a chunk is all in or all out
                const int64_t o = (int64_t)n * 2 * M + m;
                *reinterpret_cast<uint4 *>(Out + o) = make_uint4(dgw[0], dgw[1], dgw[2], dgw[3]);
                *reinterpret_cast<uint4 *>(Out + o + M) = make_uint4(duw[0], duw[1], duw[2], duw[3]);
            }
        }
    } else if constexpr (ACT_MODE == 2) {
        unsigned char *est = region(wave);
        stage_tile<T, MI>(acc, est, lane);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0(0));   // the wave reads back only what it wrote itself
        asm volatile("" ::: "memory");
        constexpr int LPR = 4 * MI, RPP = 64 / LPR;   // lanes per tile row (16-byte pieces), rows per pass
        const int n_base = n0 + 64 * wn, m_base = m0 + WM * wm;
        const int c = lane % LPR, m = min(m_base + 8 * c, M - 8);
        uint4 z[LPR];   // the accumulators are dead: all loads of Z go out before anything is computed
#pragma unroll
        for (int j = 0; j < LPR; ++j)
            z[j] = s24_load_stream(GU + (int64_t)min(n_base + RPP * j + lane / LPR, N - 1) * M + m);
        if constexpr (TABLE) {   // under the loads of Z
            Table::template build<128 * WN>(table, tid);
            wait_and_barrier<63>();
        }
#pragma unroll
        for (int j = 0; j < LPR; ++j) {
            const int nl = RPP * j + lane / LPR, n = n_base + nl;
            const uint4 dh = staged_chunk<MI>(est, nl, c);
            const uint32_t dw[4] = {dh.x, dh.y, dh.z, dh.w}, zw[4] = {z[j].x, z[j].y, z[j].z, z[j].w};
            uint32_t o[4];
            float2 slope[4];
            if constexpr (TABLE) {
                Table::lookup(table, zw, slope);
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k) slope[k] = make_float2(s24_act_slope<ACT>(s24_num<T>::lo(zw[k])), s24_act_slope<ACT>(s24_num<T>::hi(zw[k])));
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) o[k] = s24_num<T>::pack2(s24_num<T>::lo(dw[k]) * slope[k].x, s24_num<T>::hi(dw[k]) * slope[k].y);
            if (n < N && m_base + 8 * c < M)   // M is a multiple of 16: a chunk is all in or all out
                *reinterpret_cast<uint4 *>(Out + (int64_t)n * M + m) = make_uint4(o[0], o[1], o[2], o[3]);
        }
    } else if constexpr (ACT_MODE == 1) {
        unsigned char *est = region(wave);
        stage_tile<T, MI>(acc, est, lane);
        if constexpr (TABLE && !EARLY_TABLE) {
            Table::template build<128 * WN>(table, tid);
            wait_and_barrier<0>();
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0(0));
        asm volatile("" ::: "memory");
        constexpr int LPR = 4 * MI, RPP = 64 / LPR;
        const int n_base = n0 + 64 * wn, m_base = m0 + WM * wm;
#pragma unroll 4
        for (int j = 0; j < LPR; ++j) {
            const int nl = RPP * j + lane / LPR, c = lane % LPR;
            const int n = n_base + nl, m = m_base + 8 * c;
            if (n >= N || m >= M) continue;
            const uint4 zc = staged_chunk<MI>(est, nl, c);
            const uint32_t zw[4] = {zc.x, zc.y, zc.z, zc.w};
            uint32_t h[4];
            if constexpr (TABLE) {
                Table::lookup(table, zw, h);
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    h[k] = s24_num<T>::pack2(s24_act_value<ACT>(s24_num<T>::lo(zw[k])), s24_act_value<ACT>(s24_num<T>::hi(zw[k])));
            }
            s24_store_stream(Out + (int64_t)n * M + m, zc);
            *reinterpret_cast<uint4 *>(H + (int64_t)n * M + m) = make_uint4(h[0], h[1], h[2], h[3]);
        }
    } else if constexpr (!SWIGLU) {
        staged_store<T, MI>(acc, region(wave), Out, N, M, n0 + 64 * wn, m0 + WM * wm, lane);
    } else {
        // waves (0, wn) and (1, wn) hold the gate and the up tile of the same 64 tokens x 128 features: both park
        // their bf16 tiles, then each takes 32 of the 64 token rows and writes G, U and H in 16-byte pieces
        stage_tile<T, 4>(acc, region(wave), lane);
        wait_and_barrier<0>();
        const unsigned char *sg = region(2 * wn), *su = region(2 * wn + 1);
#pragma unroll 2
        for (int j = 0; j < 8; ++j) {
            const int idx = j * 64 + lane, nl = 32 * wm + (idx >> 4), c = idx & 15;
            const int n = n0 + 64 * wn + nl, f = m0 + 8 * c;
            if (n >= N || f >= F) continue;   // F is a multiple of 8: a chunk is all in or all out
            const uint4 g = staged_chunk(sg, nl, c), u = staged_chunk(su, nl, c);
            const uint32_t gw[4] = {g.x, g.y, g.z, g.w}, uw[4] = {u.x, u.y, u.z, u.w};
            uint32_t hw[4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                hw[k] = s24_num<T>::pack2(s24_glu<GATE>(s24_num<T>::lo(gw[k]), s24_num<T>::lo(uw[k])),
                                          s24_glu<GATE>(s24_num<T>::hi(gw[k]), s24_num<T>::hi(uw[k])));
            s24_store_stream(Out + (int64_t)n * M + f, g);
            s24_store_stream(Out + (int64_t)n * M + F + f, u);
            *reinterpret_cast<uint4 *>(H + (int64_t)n * F + f) = make_uint4(hw[0], hw[1], hw[2], hw[3]);
        }
    }
}

template <typename T, bool ACCUM, bool SWIGLU = false, bool GATE_BWD = false, int GATE = S24_GATE_SILU, bool BIAS = false,
          int ACT_MODE = 0, int ACT = S24_ACT_RELU, int MI = 4, int WN = MI>
__global__ __launch_bounds__(128 * WN) void spmm_nt_big_kernel(const uint16_t *__restrict__ B,
                                                              const uint16_t *__restrict__ Av,
                                                              const uint16_t *__restrict__ Am,
                                                              uint16_t *__restrict__ Out, int N, int K, int M,
                                                              int tiles_m, int tiles_n, unsigned long long *probe,
                                                              uint16_t *__restrict__ H = nullptr, int F = 0,
                                                              const uint16_t *__restrict__ GU = nullptr,
                                                              const uint16_t *__restrict__ bias = nullptr)
{
    constexpr int RING = spmm_stage(MI, WN);
    __shared__ __attribute__((aligned(16))) unsigned char s0[RING];
    __shared__ __attribute__((aligned(16))) unsigned char s1[RING];
    __shared__ __attribute__((aligned(16))) unsigned char s2[RING];
    spmm_nt_tile<T, ACCUM, SWIGLU, GATE_BWD, GATE, BIAS, ACT_MODE, ACT, MI, WN>(s0, s1, s2, blockIdx.x, B, Av, Am, Out, N, K, M, tiles_m, tiles_n, probe, H, F, GU, bias);
}
}  // namespace big

// ------------------------------------------------------------------ dense NT
// The dense GEMM in the same tiling family as the sparse kernel: both operands copied straight into LDS.
namespace bignt {
// Dense NT GEMM, 256 x 256 tiles, eight waves of 128 x 64: the comparison kernel beside the sparse one, on the
// same schedule.  32 of k per ring stage (two 16 KB operand tiles, 64-byte rows), four stages, three chunks in
// flight; a chunk is two halves of the wave's feature blocks, the first running from registers while the
// second's fragments come in, the one barrier of the chunk between them, and after it the next chunk's
// fragments and the copies of chunk kc+4 dealt out between the second half's matrix instructions.
// 8192 tokens x 28672 features, K = 8192: 2975 -> 2808 us with the 16-wide instruction (1.29 -> 1.37 PFLOP/s), 16384 x 5120,
// K = 1280: 197 -> 187; 8192 x 1024, K = 4096 (medium tiles): 70 -> 67.
// MI and WN as in the sparse kernel: 256 x 256 tiles of eight waves, and for outputs with too few of them 256 (m) x 128 (n)
// and, two workgroups per compute unit, 128 x 128 tiles of four waves.
using big::a_slot;
using big::a_swizzle;
using big::glb_ptr;
using big::lds_ptr;
using big::wait_vm_lgkm0;

template <typename T, int MI, int WN>
__global__ __launch_bounds__(128 * WN) void dense_nt_big_kernel(const uint16_t *__restrict__ X,
                                                               const uint16_t *__restrict__ W, uint16_t *__restrict__ Y,
                                                               int N, int K, int M, int tiles_m, int tiles_n, unsigned long long *probe)
{
    constexpr int BM = 64 * MI, BN = 64 * WN, WM = 32 * MI, OPERAND = BN * 64, STAGE = OPERAND + BM * 64;
    constexpr int NW = 2 * MI / WN, NC = 2 + NW;   // copies per lane and chunk: of the weights, all
    const big::ClockStamp t_start = big::clock_now();
    __shared__ __attribute__((aligned(16))) unsigned char s0[STAGE];
    __shared__ __attribute__((aligned(16))) unsigned char s1[STAGE];
    __shared__ __attribute__((aligned(16))) unsigned char s2[STAGE];
    __shared__ __attribute__((aligned(16))) unsigned char s3[STAGE];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    const int total = tiles_m * tiles_n, per_xcd = (total + 7) / 8;
    const int t = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (t >= total) return;
    constexpr int GROUP = 8;
    const int group_sz = GROUP * tiles_m, grp = t / group_sz, in_grp = t - grp * group_sz;
    const int gw = min(GROUP, tiles_n - grp * GROUP);
    const int tm = in_grp / gw, tn = grp * GROUP + in_grp % gw;
    const int m0 = tm * BM, n0 = tn * BN;
    const int nk = K / 32;

    // copies: two of X and NW of the weights per lane and chunk; copy i of a wave's N fills rows 16 (N wave + i) .. +15
    // (four 16-byte slots each); slot c of row r holds source chunk c ^ ((r >> 2) & 3).  Wave-uniform bases (one per operand,
    // advanced by 64 bytes per chunk) and fixed 32-bit lane offsets: 256 rows of K elements span < 4 GB (host check).
    const char *baseX = reinterpret_cast<const char *>(X + (int64_t)n0 * K), *baseW = reinterpret_cast<const char *>(W + (int64_t)m0 * K);
    uint32_t ox[2], ow[NW];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = 16 * (2 * wave + i) + (lane >> 2);
        const int c = (lane & 3) ^ a_swizzle(row);
        ox[i] = ((uint32_t)(min(n0 + row, N - 1) - n0) * (uint32_t)K + 8u * c) * 2u;
    }
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        const int row = 16 * (NW * wave + i) + (lane >> 2);
        const int c = (lane & 3) ^ a_swizzle(row);
        ow[i] = ((uint32_t)(min(m0 + row, M - 1) - m0) * (uint32_t)K + 8u * c) * 2u;
    }
    // copies over both phases of the main loop, as in the sparse kernel
    constexpr auto copy_slot = [](int c) { return c * 8 * MI / NC; };
    constexpr int EARLY = (NC + 1) / 2;
    // copy c of a chunk's NC per lane; every chunk issues all of them, past the last one it re-reads that into a stage nobody reads
    const char *px = baseX, *pw = baseW;
    auto issue = [&](unsigned char *st, int c) {
        if (c < 2) big::buffer_to_lds<16>(big::buffer_of(px), (lds_ptr)(st + 16 * (2 * wave + c) * 64), ox[c]);
        else big::buffer_to_lds<16>(big::buffer_of(pw), (lds_ptr)(st + OPERAND + 16 * (NW * wave + c - 2) * 64), ow[c - 2]);
    };
    auto advance = [&](int kc) {   // to chunk kc, or not past the last one
        if (kc < nk) { px += 64; pw += 64; }
    };
    auto issue_all = [&](unsigned char *st, int kc) {
        if (kc > 0) advance(kc);
#pragma unroll
        for (int c = 0; c < NC; ++c) issue(st, c);
    };
    f32x4 acc[2 * MI][4];
#pragma unroll
    for (int mi = 0; mi < 2 * MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < 4; ++ni) acc[mi][ni] = f32x4{};
    // fragments of a stage: 16 rows x 32 of k, lane group g = lane / 16 takes source chunk g
    const int l16 = lane & 15, g = lane >> 4;
    auto load_b = [&](const unsigned char *st, int ni) {
        return as_bf16x8(*reinterpret_cast<const uint4 *>(st + 1024 * ni + a_slot(64 * wn + l16, g)));
    };
    auto load_a = [&](const unsigned char *st, int mi) {
        return as_bf16x8(*reinterpret_cast<const uint4 *>(st + OPERAND + 1024 * mi + a_slot(WM * wm + l16, g)));
    };
    // keep the program order of these groups: the constant wait counts rely on it
    issue_all(s0, 0);
    __builtin_amdgcn_sched_barrier(0);
    issue_all(s1, 1);
    __builtin_amdgcn_sched_barrier(0);
    issue_all(s2, 2);
    __builtin_amdgcn_sched_barrier(0);
    advance(3);
#pragma unroll
    for (int c = 0; c < EARLY; ++c) issue(s3, c);
    __builtin_amdgcn_sched_barrier(0);
    big::wait_and_barrier<2 * NC + EARLY>();   // chunk 0 has landed for everybody
    bf16x8 fb[4], fa0[MI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) fa0[mi] = load_a(s0, mi);
#pragma unroll
    for (int ni = 0; ni < 4; ++ni) fb[ni] = load_b(s0, ni);
    mma_tie<ACC_AGPR>(acc);
    mma_operands();
    auto chunk = [&](unsigned char *cur, const unsigned char *nxt, unsigned char *prv, int kc) {
        bf16x8 fa1[MI];
        auto multiply = [&](const bf16x8 (&a)[MI], int first, int i) {   // the i-th matrix instruction of a phase
            const int ni = i / MI, j = i % MI, b = (ni & 1) ? MI - 1 - j : j;
            Mma<T>::dense16(a[b], fb[ni], acc[first + b][ni]);
            __builtin_amdgcn_sched_barrier(0);
        };
#pragma unroll
        for (int i = 0; i < 4 * MI; ++i) {
            multiply(fa0, 0, i);
            if (i < MI) fa1[i] = load_a(cur, MI + i);
#pragma unroll
            for (int c = EARLY; c < NC; ++c)
                if (copy_slot(c) - 4 * MI == i) issue(prv, c);
            __builtin_amdgcn_sched_barrier(0);
        }
        advance(kc + 4);
        // all but the copies of chunks kc+2 and kc+3 are complete: this lane's part of chunk kc+1 is
        // in LDS, and its own reads of chunk kc are done
        big::wait_and_barrier<2 * NC>();
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int i = 0; i < 4 * MI; ++i) {
            multiply(fa1, MI, i);
            if (i < MI) fa0[i] = load_a(nxt, i);
            if (i >= MI && i % MI == 0) fb[i / MI - 1] = load_b(nxt, i / MI - 1);   // each after its last use
            if (i + 1 == 4 * MI) fb[3] = load_b(nxt, 3);
#pragma unroll
            for (int c = 0; c < EARLY; ++c)
                if (copy_slot(c) == i) issue(cur, c);
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(0);
    };
    // past the last chunk the prefetched fragments come from a stage that holds a re-read of the last chunk (or is
    // being refilled with one); they are never multiplied
    int kc = 0;
    for (; kc + 4 <= nk; kc += 4) {
        chunk(s0, s1, s3, kc);
        chunk(s1, s2, s0, kc + 1);
        chunk(s2, s3, s1, kc + 2);
        chunk(s3, s0, s2, kc + 3);
    }
    if (kc < nk) chunk(s0, s1, s3, kc);
    if (kc + 1 < nk) chunk(s1, s2, s0, kc + 1);
    if (kc + 2 < nk) chunk(s2, s3, s1, kc + 2);
    mma_drain<ACC_AGPR>(acc);
    big::wait_and_barrier<0>();   // last (redundant) copies drained, nobody reads the ring any more: reuse it
    big::clock_report(probe, t_start);
    constexpr int PER = WN / 2;   // waves that park their output tile in one ring stage
    static_assert(PER * (big::EWAVE * MI / 4) <= STAGE, "wave tiles must fit the ring stages");
    const int home = wave / PER;
    unsigned char *est = (home == 0 ? s0 : (home == 1 ? s1 : (home == 2 ? s2 : s3))) + (wave % PER) * big::EWAVE;
    big::staged_store<T, MI>(acc, est, Y, N, M, n0 + 64 * wn, m0 + WM * wm, lane);
}
}  // namespace bignt

// ------------------------------------------------------------------ dense TN (dW), large tile
// dW[m][n] = sum_t dY[t][m] X[t][n] with 256 x 256 workgroup tiles.  Both operands are token-major, so a
// tile chunk (32 tokens x 256 columns) is copied into LDS as it lies in memory, rows of 512 bytes, and the
// matrix-core fragments (8 consecutive t per lane) are gathered with the transposing LDS read.
// ds_read_b64_tr_b16: in a group of 16 lanes, lane i points at row i/4, columns 4*(i%4)..+3 of a
// 4 (t) x 16 (columns) patch and receives, for column i, the four consecutive t (measured on the device
// with an index-filled tile); two such reads give one lane its eight k values.
// LDS swizzle: 16-byte chunk c of token row t sits at slot c ^ (4 (t&3)) ^ (2 (t>>3 & 1)), which keeps the eight 32-byte row
// segments (rows 0-3 and 8-11 of 16 columns) touched by 32 lanes in one cycle on distinct banks.
// Four waves, one per SIMD, each a 128 x 128 tile of 8 x 8 accumulator blocks (256 accumulator registers):
// against eight waves of 128 x 64 this reads a third less LDS per matrix instruction, which matters
// because the chip sheds clock under the combined matrix + LDS + copy load.
// 16 x 16 blocks and not 32 x 32: the clock the chip holds under matrix load was the bound, and the 16-wide instruction moves
// half as many accumulator bits per FLOP: alone, on random operands, it runs at 2.05-2.10 PFLOP/s (2.02 GHz) where the 32-wide
// one gets 1.81 (1.79 GHz); binary16 1.91 against 1.66.  Here: 8192 tokens, 8192 x 28672: 1.32 -> 1.42 PFLOP/s (2921 -> 2711 us, clock
// 1.47 -> 1.64 GHz); 16384 tokens, 1280 x 5120: 188 -> 172 us.  What is left is mostly not the clock: on zero operands, at
// 2.3 GHz, that gradient takes 2.45-2.47 ms, 6-8 % less than on random ones at 1.7 GHz in the same run and no less than with the
// 32-wide instruction.  That wall, 1.56 PFLOP/s, is the supply of operands; which part of it has not been measured.
// The token axis moves through a ring of four 32 KB stages.  A chunk is waited for one iteration before it is used, so the
// fragments of chunk kc+1 are fetched during the matrix instructions of chunk kc and the barrier finds the matrix unit
// busy; the copies of chunk kc+3 are dealt out between the matrix instructions rather than issued in one burst.
namespace dmatn {
using namespace s24_lds;
using namespace s24_dw;
constexpr int THREADS = 256;
// WTM x WTN: wave tile in units of 32: 4 x 4 -> 256 x 256 workgroup tiles; 4 x 2, 3 x 2 and 2 x 2 -> 256 x 128, 192 x 128 and
// 128 x 128 tiles for outputs with too few large tiles to fill the chip.  BT = tokens per ring stage: 32 for the large tile (128 KB
// of LDS); for the small tile 32 (64 KB, two workgroups per CU) when there are more tiles than CUs, else 64 (a
// small tile has a quarter of the matrix work per token, so the barrier is paid half as often).
template <int WTM_, int WTN_, int BT_> struct Cfg {
    static constexpr int WTM = WTM_, WTN = WTN_, BM = 64 * WTM, BN = 64 * WTN, BT = BT_;
    static constexpr int ROWA = BM * 2, ROWX = BN * 2;                              // bytes of a token's row in the dY / X tile
    static constexpr int OPERAND = BT * ROWA, STAGE = OPERAND + BT * ROWX;
    static constexpr int NIA = BT * ROWA / 4096, NIX = BT * ROWX / 4096, NI = NIA + NIX;   // copies per wave and chunk
};
// DECAY: the masked decay term is added in the epilogue: dW[m][n] += lambda * Wt[m][n] where bit
// 4*(m%4) + n%4 of mask[m/4][n/4] is clear, with the same single fused multiply-add the stand-alone
// decay kernel applies to the stored gradient, so both routes give the same bits.
// `block`, s0 .. s3 (C::STAGE bytes each): as in big::spmm_nt_tile
template <typename ET, typename C, bool ACCUM, bool DECAY>
__device__ __forceinline__ void dense_tn_tile(unsigned char *s0, unsigned char *s1, unsigned char *s2, unsigned char *s3, unsigned block, const DwBatch &batch,
                                              unsigned long long *probe)
{
    constexpr int WTM = C::WTM, WTN = C::WTN, BM = C::BM, BN = C::BN, BT = C::BT, ROWA = C::ROWA, ROWX = C::ROWX;
    constexpr int OPERAND = C::OPERAND, STAGE = C::STAGE, NIA = C::NIA, NIX = C::NIX, NI = C::NI;
    constexpr int KS = BT / 32, CPS = NI / KS;   // 32-token steps per chunk, copies issued per step
    static_assert(CPS * KS == NI, "every step issues the same number of copies");
    constexpr int MB = 2 * WTM, NB = 2 * WTN;     // 16 x 16 accumulator blocks of a wave
    const big::ClockStamp t_start = big::clock_now();
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    const int slot = (int)(block >> 3);
    int which = 0;   // wave-uniform: the problem this workgroup's tile belongs to
#pragma unroll
    for (int i = 1; i < kMaxBatch; ++i)
        if (slot >= batch.first_slot[i]) which = i;
    const DwWindow &win = batch.w[which];
    const int per_xcd = batch.first_slot[which + 1] - batch.first_slot[which];
    const int t = (int)(block & 7) * per_xcd + (slot - batch.first_slot[which]);
    if (t >= win.tiles_m * win.tiles_n) return;
    const uint16_t *__restrict__ dY = win.dY, *__restrict__ X = win.X, *__restrict__ Wt = win.Wt, *__restrict__ mask = win.mask;
    float *__restrict__ dW = win.dW;
    const int T = win.T, M = win.M, N = win.N, ldy = win.ldy, ldx = win.ldx, ldw = win.ldw;
    const int tiles_m = win.tiles_m, tiles_n = win.tiles_n;
    const float lambda = win.lambda;
    constexpr int GROUP = 8;
    const int group_sz = GROUP * tiles_m, grp = t / group_sz, in_grp = t - grp * group_sz;
    const int gw = min(GROUP, tiles_n - grp * GROUP);
    const int tm = in_grp / gw, tn = grp * GROUP + in_grp % gw;
    const int m0 = tm * BM, n0 = tn * BN;
    const int nk = (T + BT - 1) / BT;

    // Copies: instruction g of an operand fills the 16-byte slots 64g .. 64g+63 of its stage region, slot ->
    // (row = slot / slots per row, chunk = the rest); the source chunk is chunk ^ tr_swizzle(row).  Columns past the
    // matrix edge are clamped to its last 16-byte chunk.  A lane's byte offsets from the first token row of its copies
    // are fixed for the whole kernel; only the (wave-uniform) row base moves, so a copy costs no vector
    // arithmetic.  The tokens of a 32-token step are contiguous rows, and always 32 of them: the step that would reach past
    // the last token starts at T - 32 and overlaps its predecessor (clear_tail drops the overlap), and so does one that would
    // lie past it altogether; with fewer than 32 tokens in all, rows past T - 1 re-read row T - 1.  Which tokens one matrix
    // instruction sums therefore does not depend on the tile or its BT, nor do the bits of the result.  (A stage of two steps
    // that started at T - 64 as a whole gave other bits than two stages of one for T % 64 of 33 to 63.)
    const int part = wave * KS / 4;   // the step of a stage whose rows this wave copies
    static_assert(KS <= 2 && BT / 4 <= 32, "a wave copies rows of one step");
    uint32_t voffA[NIA], voffB[NIX];
    const int lastA = (min(M - m0, BM) >> 3) - 1, lastB = (min(N - n0, BN) >> 3) - 1;
#pragma unroll
    for (int j = 0; j < NIA; ++j) {
        constexpr int CPR = ROWA / 16;
        const int slot = (wave * NIA + j) * 64 + lane, row = min(slot / CPR - 32 * part, T - 1), c = (slot % CPR) ^ tr_swizzle<ROWA>(slot / CPR);
        voffA[j] = (uint32_t)(row * ldy + m0 + 8 * min(c, lastA)) * 2u;
    }
#pragma unroll
    for (int j = 0; j < NIX; ++j) {
        constexpr int CPR = ROWX / 16;
        const int slot = (wave * NIX + j) * 64 + lane, row = min(slot / CPR - 32 * part, T - 1), c = (slot % CPR) ^ tr_swizzle<ROWX>(slot / CPR);
        voffB[j] = (uint32_t)(row * ldx + n0 + 8 * min(c, lastB)) * 2u;
    }
    auto first_row = [&](int kc) { return max(min(kc * BT + 32 * part, T - 32), 0); };   // of this wave's copies
    const char *baseA = reinterpret_cast<const char *>(dY), *baseB = reinterpret_cast<const char *>(X);
    // Copy c of a chunk's list (the dY tile's NIA, then the X tile's NIX), rowsA and rowsB its first token row.
    // The copies are buffer loads into LDS: a descriptor (scalar registers) whose base is the first of those token
    // rows, and the lane's fixed 32-bit offset; nothing of a copy's address is computed on the vector unit.
    auto issue = [&](unsigned char *st, const char *rowsA, const char *rowsB, int c) {
        if (c < NIA) big::buffer_to_lds<16>(big::buffer_of(rowsA), (lds_ptr)(st + (wave * NIA + c) * 1024), voffA[c]);
        else big::buffer_to_lds<16>(big::buffer_of(rowsB), (lds_ptr)(st + OPERAND + (wave * NIX + c - NIA) * 1024), voffB[c - NIA]);
    };
    auto issue_all = [&](unsigned char *st, int kc) {
        const char *ra = baseA + (int64_t)first_row(kc) * ldy * 2, *rb = baseB + (int64_t)first_row(kc) * ldx * 2;
#pragma unroll
        for (int c = 0; c < NI; ++c) issue(st, ra, rb, c);
    };
    f32x4 acc[MB][NB];
#pragma unroll
    for (int mi = 0; mi < MB; ++mi)
#pragma unroll
        for (int ni = 0; ni < NB; ++ni) acc[mi][ni] = f32x4{};

    // fragment addressing of this lane: group G = lane/16 takes tokens 8G .. 8G+7 of a step, 16 columns per block
    const int gi = lane & 15, G = lane >> 4;
    const int frow = 8 * G + (gi >> 2), fcol = 4 * (gi & 3);
    // Byte offsets of a lane's fragments from a stage, and the same plus two stages for the upper two, whose distance does
    // not fit an instruction's offset field (kept in registers of their own: added on the spot, they were 16 vector
    // instructions per chunk).
    constexpr int FAR = 2 * STAGE;
    int offA[2][MB], offB[2][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i) offA[0][i] = tr_off<ROWA>(frow, 32 * WTM * wm + 16 * i + fcol);
#pragma unroll
    for (int i = 0; i < NB; ++i) offB[0][i] = OPERAND + tr_off<ROWX>(frow, 32 * WTN * wn + 16 * i + fcol);
#pragma unroll
    for (int i = 0; i < MB; ++i) {
        offA[1][i] = offA[0][i] + FAR;
        asm volatile("" : "+v"(offA[1][i]));
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        offB[1][i] = offB[0][i] + FAR;
        asm volatile("" : "+v"(offB[1][i]));
    }
    // Half h (tokens 8G + 4h ..) of fragment i of step ks.  S: number of the stage `st`
    auto load_a = [&](const unsigned char *st, auto S, int ks, int i, int h) {
        return tr_half((S < 2 ? st + offA[0][i] : st - FAR + offA[1][i]) + (32 * ks + 4 * h) * ROWA);
    };
    auto load_b = [&](const unsigned char *st, auto S, int ks, int i, int h) {
        return tr_half((S < 2 ? st + offB[0][i] : st - FAR + offB[1][i]) + (32 * ks + 4 * h) * ROWX);
    };
    // The last chunk of a token count that is not a multiple of BT holds rows that must not contribute: of each step the
    // leading ones that its predecessor already covered, or, when there are fewer than 32 tokens in all, the trailing
    // ones past T.  They are cleared in both tiles: in one alone, an infinity in the other would make a NaN.
    auto clear_tail = [&](unsigned char *st, int kc) {
        auto clear = [&](unsigned char *rows, int bytes) {
            for (int at = 16 * tid; at < bytes; at += 16 * THREADS) *reinterpret_cast<uint4 *>(rows + at) = make_uint4(0, 0, 0, 0);
        };
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int live = max(min(T - kc * BT - 32 * ks, 32), 0), row = 32 * ks + (T < 32 ? live : 0);
            clear(st + row * ROWA, (32 - live) * ROWA);
            clear(st + OPERAND + row * ROWX, (32 - live) * ROWX);
        }
        __syncthreads();
    };
    const bool partial = (T % BT) != 0;

    // prologue: chunks 0..2 in flight, chunk 0 landed, its first fragments in registers
    issue_all(s0, 0);
    __builtin_amdgcn_sched_barrier(0);
    issue_all(s1, 1);
    __builtin_amdgcn_sched_barrier(0);
    issue_all(s2, 2);
    __builtin_amdgcn_sched_barrier(0);
    big::wait_and_barrier<2 * NI>();
    if (partial && nk == 1) clear_tail(s0, 0);
    // Fragments: of X those of the current and of the next 32-token step; of dY one set, each replaced by the next step's
    // as soon as its row of accumulators is done (the last one at the start of that step).
    const std::integral_constant<int, 0> c0;
    const std::integral_constant<int, 1> c1;
    const std::integral_constant<int, 2> c2;
    const std::integral_constant<int, 3> c3;
    bf16x8 fa[MB], fb[2][NB];
#pragma unroll
    for (int ni = 0; ni < NB; ++ni) fb[0][ni] = join(load_b(s0, c0, 0, ni, 0), load_b(s0, c0, 0, ni, 1));
#pragma unroll
    for (int mi = 0; mi < MB - 1; ++mi) fa[mi] = join(load_a(s0, c0, 0, mi, 0), load_a(s0, c0, 0, mi, 1));
    mma_tie<ACC_AGPR>(acc);
    mma_operands();
    const char *rowsA = baseA + (int64_t)first_row(3) * ldy * 2, *rowsB = baseB + (int64_t)first_row(3) * ldx * 2;   // of the next chunk to copy

    // One step: rows of NB matrix instructions.  A wave is alone on its SIMD and issues an instruction every four cycles, a
    // matrix instruction lasts sixteen: whatever else goes out between two of them beyond three instructions leaves the matrix
    // unit idle (a wait state before each cost 6 % of the kernel).  So the rest is dealt out evenly: beside row mi the
    // LDS reads of one dY fragment and its share of the NB X fragments', one read per matrix instruction, one copy, and a part of
    // the address of the next chunk's rows.  The X fragment is the instruction's row operand: a lane's four accumulators
    // are then four consecutive columns of one row of dW.  Neighbouring instructions share a fragment, at the turns
    // of the serpentine the other one: the operand bits that toggle cost clock.
    // `cs` / `ns`: numbers of the stages cur / nxt; `which`: the X fragment set of this step.
    auto step = [&](const unsigned char *cur, auto cs, int ks, const unsigned char *nxt, auto ns, int ksn, unsigned char *refill, int copy0, int next_row,
                    auto which) {
        constexpr int P = decltype(which)::value;
        static_assert((2 * NB + MB - 1) / MB + 2 <= NB && CPS <= MB, "one read per matrix instruction, one copy per row");
        int64_t nextA = 0, nextB = 0;
        v4i16 lo{}, loA{};
#pragma unroll
        for (int mi = 0; mi < MB; ++mi) {
            const int x0 = 2 * NB * mi / MB, RB = 2 * NB * (mi + 1) / MB - x0, R = RB + 2;   // reads of X beside this row, all reads
#pragma unroll
            for (int nj = 0; nj < NB; ++nj) {
                const int ni = (mi & 1) ? NB - 1 - nj : nj;
                Mma<ET>::dense16(fb[P][ni], fa[mi], acc[mi][ni]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    if (r * NB / R != nj) continue;
                    if (r < RB) {
                        const int i = x0 + r;
                        if (i % 2 == 0) lo = load_b(nxt, ns, ksn, i / 2, 0);
                        else fb[1 - P][i / 2] = join(lo, load_b(nxt, ns, ksn, i / 2, 1));
                    } else if (mi == 0) {
                        if (r == RB) loA = load_a(cur, cs, ks, MB - 1, 0);
                        else fa[MB - 1] = join(loA, load_a(cur, cs, ks, MB - 1, 1));
                    } else {
                        if (r == RB) loA = load_a(nxt, ns, ksn, mi - 1, 0);
                        else fa[mi - 1] = join(loA, load_a(nxt, ns, ksn, mi - 1, 1));
                    }
                }
                if (nj == NB - 1 && mi < CPS) issue(refill, rowsA, rowsB, copy0 + mi);
                if (next_row >= 0 && nj == 1) {   // the address of the next chunk's rows, a product or a sum at a time
                    if (mi == MB - 4) { nextA = (int64_t)next_row * ldy * 2; asm volatile("" : "+s"(nextA)); }
                    if (mi == MB - 3) { nextB = (int64_t)next_row * ldx * 2; asm volatile("" : "+s"(nextB)); }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (next_row >= 0) { rowsA = baseA + nextA; rowsB = baseB + nextB; }
    };
    // Iteration kc: all but the NI most recent copies (chunk kc+2) are complete, so chunk kc+1 is in LDS for
    // every wave after the barrier, and nobody reads the stage of chunk kc-1 any more: it takes chunk kc+3.  (The last read
    // of that stage fed the last row of iteration kc-1; the reads still in flight here are of chunk kc and need no wait.)
    // Past the last chunk the fragments fetched ahead come from a stage nobody uses and are dropped.
    auto chunk = [&](const unsigned char *cur, auto cs, unsigned char *nxt, auto ns, unsigned char *refill, int kc, bool tail) {
        big::wait_and_barrier<NI, false>();
        if (tail && partial && kc + 2 == nk) clear_tail(nxt, kc + 1);
        const int next_row = first_row(kc + 4);
        if constexpr (KS == 1) {
            step(cur, cs, 0, nxt, ns, 0, refill, 0, next_row, std::integral_constant<int, decltype(cs)::value & 1>());
        } else {
            step(cur, cs, 0, cur, cs, 1, refill, 0, -1, c0);
            step(cur, cs, 1, nxt, ns, 0, refill, CPS, next_row, c1);
        }
    };
    int kc = 0;
    for (; kc + 6 <= nk; kc += 4) {   // the chunk that needs its overlap cleared is never `nxt` in here
        chunk(s0, c0, s1, c1, s3, kc, false);
        chunk(s1, c1, s2, c2, s0, kc + 1, false);
        chunk(s2, c2, s3, c3, s1, kc + 2, false);
        chunk(s3, c3, s0, c0, s2, kc + 3, false);
    }
    for (; kc < nk; kc += 4) {
        chunk(s0, c0, s1, c1, s3, kc, true);
        if (kc + 1 >= nk) break;
        chunk(s1, c1, s2, c2, s0, kc + 1, true);
        if (kc + 2 >= nk) break;
        chunk(s2, c2, s3, c3, s1, kc + 2, true);
        if (kc + 3 >= nk) break;
        chunk(s3, c3, s0, c0, s2, kc + 3, true);
    }
    // Epilogue through LDS, so that global memory sees 16-byte accesses along rows: each wave parks a slice of its tile
    // at a time (32*RB rows x 64 columns of fp32, 256-byte rows) in its own ring stage, then lane l of pass j
    // owns row (64j + l) / 16, columns 4 * (l % 16) .. +3: one LDS read, one 16-byte store, and for the
    // optional terms one 16-byte load of the old gradient, one 8-byte load of W and one mask word.
    // The W and mask loads of a whole slice are issued in one go, well before they are needed: those of
    // the first slice ahead of the wait that drains the ring, those of the second before it is parked in LDS.
    // Loaded pass by pass where they are used, their latency was exposed eight times per tile with only four
    // waves on the compute unit to hide it (c5: 0.45 ms per step).
    // They are buffer loads: pass j reads four rows further down than pass j - 1, which is a wave-uniform step (a
    // scalar register), so the 64 loads of a slice share two address registers.  M is a multiple of 16 and a wave's
    // rows start at a multiple of 32: the four rows of a pass are all inside the matrix or all outside, and passes
    // past the edge re-read the last pass inside (a wave with no row inside re-reads the tile's first rows).
    constexpr int RB = WTM * 8192 <= STAGE ? WTM : WTM / 2, NR = WTM / RB;   // row blocks per slice, slices down a wave's tile
    static_assert(RB * 8192 <= STAGE && RB * NR == WTM, "a wave's slice fits one stage");
    constexpr int NP = 8 * RB;   // passes per slice
    uint2 wv[DECAY ? NP : 1];
    uint32_t keep[DECAY ? NP : 1];
    const int wave_rows = min(M - m0 - 32 * WTM * wm, 32 * WTM);   // rows of this wave's sub-tile inside the matrix
    const int wave_row0 = wave_rows > 0 ? 32 * WTM * wm : 0, last_pass = wave_rows > 0 ? (wave_rows >> 2) - 1 : 0;
    auto decay_loads = [&](int h2, int r2) {
        if constexpr (DECAY) {
            const int nc = min(n0 + 32 * WTN * wn + 64 * h2 + 4 * (lane & 15), N - 4);
            const big::rsrc_t wbuf = big::buffer_of(Wt + (int64_t)(m0 + wave_row0) * ldw);
            const big::rsrc_t mbuf = big::buffer_of(mask + (int64_t)((m0 + wave_row0) >> 2) * (ldw >> 2));
            const uint32_t voff_w = ((uint32_t)(lane >> 4) * (uint32_t)ldw + (uint32_t)nc) * 2u, voff_m = (uint32_t)(nc >> 2) * 2u;
            const uint32_t shift = 4 * (lane >> 4);   // row of the 4 x 4 block: the tile starts at a multiple of four
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                const uint32_t jc = (uint32_t)min(NP * r2 + j, last_pass);
                wv[j] = big::buffer_load_8(wbuf, voff_w, jc * 8u * (uint32_t)ldw);
                keep[j] = big::buffer_load_2(mbuf, voff_m, jc * 2u * (uint32_t)(ldw >> 2)) >> shift;
            }
        }
    };
    mma_drain<ACC_AGPR>(acc);
    decay_loads(0, 0);
    big::wait_and_barrier<0>();   // last (redundant) copies drained, nobody reads the ring any more: reuse it
    big::clock_report(probe, t_start);
    unsigned char *est = wave == 0 ? s0 : (wave == 1 ? s1 : (wave == 2 ? s2 : s3));
#pragma unroll
    for (int slice = 0; slice < NR * (WTN / 2); ++slice) {
        const int h2 = slice / NR, r2 = slice % NR;
        if (slice > 0) decay_loads(h2, r2);
#pragma unroll
        for (int nj = 0; nj < 4; ++nj)
#pragma unroll
            for (int mi = 0; mi < 2 * RB; ++mi) {   // 16-byte piece c of row r sits at slot c ^ (r & 15)
                const int row = 16 * mi + (lane & 15), c4 = 4 * nj + (lane >> 4);
                *reinterpret_cast<f32x4 *>(est + row * 256 + ((c4 ^ (row & 15)) << 4)) = acc[2 * RB * r2 + mi][4 * h2 + nj];
            }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(big::wait_vm_lgkm0(63));   // LDS only: the wave reads back only what it wrote itself
        asm volatile("" ::: "memory");
        const int ms = m0 + 32 * WTM * wm + 32 * RB * r2, ns = n0 + 32 * WTN * wn + 64 * h2;   // the slice's first row and column
        constexpr int BATCH = 8;
#pragma unroll
        for (int j0 = 0; j0 < NP; j0 += BATCH) {
            float4 v[BATCH], old[BATCH];
            bool live[BATCH];
#pragma unroll
            for (int b = 0; b < BATCH; ++b) {
                const int idx = (j0 + b) * 64 + lane, row = idx >> 4, c4 = idx & 15;
                const int m = ms + row, n = ns + 4 * c4;
                live[b] = m < M && n < N;   // N is a multiple of 16: the four columns are all in or all out
                const int mc = min(m, M - 1), nc = min(n, N - 4);
                v[b] = *reinterpret_cast<const float4 *>(est + row * 256 + ((c4 ^ (row & 15)) << 4));
                if (ACCUM) old[b] = *reinterpret_cast<const float4 *>(dW + (int64_t)mc * ldw + nc);
            }
#pragma unroll
            for (int b = 0; b < BATCH; ++b) {
                const int idx = (j0 + b) * 64 + lane, row = idx >> 4, c4 = idx & 15;
                const int m = ms + row, n = ns + 4 * c4;
                float4 o = v[b];
                if (ACCUM) { o.x = old[b].x + o.x; o.y = old[b].y + o.y; o.z = old[b].z + o.z; o.w = old[b].w + o.w; }
                if constexpr (DECAY) {
                    const uint2 w2 = wv[j0 + b];
                    const uint32_t kp = keep[j0 + b];
                    if (!(kp & 1u)) o.x = fmaf(lambda, s24_num<ET>::lo(w2.x), o.x);
                    if (!(kp & 2u)) o.y = fmaf(lambda, s24_num<ET>::hi(w2.x), o.y);
                    if (!(kp & 4u)) o.z = fmaf(lambda, s24_num<ET>::lo(w2.y), o.z);
                    if (!(kp & 8u)) o.w = fmaf(lambda, s24_num<ET>::hi(w2.y), o.w);
                }
                if (live[b]) s24_store_stream(dW + (int64_t)m * ldw + n, o);
            }
            __builtin_amdgcn_sched_barrier(0);   // one batch at a time: hoisting the next batches' reads costs registers
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(big::wait_vm_lgkm0(63));   // LDS reads done before the other half overwrites
        asm volatile("" ::: "memory");
    }
}

template <typename ET, typename C, bool ACCUM, bool DECAY>
__global__ __launch_bounds__(THREADS) void dense_tn_dma_kernel(const DwBatch batch, unsigned long long *probe)
{
    __shared__ __attribute__((aligned(16))) unsigned char s0[C::STAGE];
    __shared__ __attribute__((aligned(16))) unsigned char s1[C::STAGE];
    __shared__ __attribute__((aligned(16))) unsigned char s2[C::STAGE];
    __shared__ __attribute__((aligned(16))) unsigned char s3[C::STAGE];
    dense_tn_tile<ET, C, ACCUM, DECAY>(s0, s1, s2, s3, blockIdx.x, batch, probe);
}
}  // namespace dmatn

// ------------------------------------------------------------------ weight gradients and an input gradient in one launch
// Neither needs the other's result, and a grid that is a bad fraction of a round over the compute units leaves the chip part empty
// to its end: here the input gradient's tiles (256 features x 128 tokens) follow the weight gradients' in the list, so that the compute units which these
// leave idle, or leave early, take them.  Only as many run beside the others as there is room for: the whole grids side by side on two
// streams share the L2s and the way into LDS all the time, and took longer than one after the other.
// Input gradient and weight gradients apart and together: 8192 tokens, 768 x 3072 105 -> 90 us; 16384, 1280 x 5120 478 -> 447; 3001, 2048 x 11008 (and
// the down weight) 257 -> 237; 3083, 576 x 4608 60 -> 43; 4096, 768 x 3072 62 -> 52.
template <typename ET, bool DECAY, typename C>
__global__ __launch_bounds__(256) void dw_dx_kernel(const uint16_t *__restrict__ B, const uint16_t *__restrict__ Av, const uint16_t *__restrict__ Am,
                                                    uint16_t *__restrict__ Out, int N, int K, int M, int dw_blocks, int tiles_m, int tiles_n,
                                                    const dmatn::DwBatch batch, unsigned long long *probe)
{
    constexpr int DX = big::spmm_stage(4, 2), RING = DX > C::STAGE ? DX : C::STAGE;
    static_assert(3 * RING + C::STAGE <= 160 * 1024 && dmatn::THREADS == 256, "one ring for either");
    __shared__ __attribute__((aligned(16))) unsigned char s0[RING];
    __shared__ __attribute__((aligned(16))) unsigned char s1[RING];
    __shared__ __attribute__((aligned(16))) unsigned char s2[RING];
    __shared__ __attribute__((aligned(16))) unsigned char s3[C::STAGE];
    if ((int)blockIdx.x < dw_blocks)   // a multiple of eight
        dmatn::dense_tn_tile<ET, C, false, DECAY>(s0, s1, s2, s3, blockIdx.x, batch, probe);
    else
        big::spmm_nt_tile<ET, false, false, false, S24_GATE_SILU, false, 0, S24_ACT_RELU, 4, 2>(s0, s1, s2, blockIdx.x - (unsigned)dw_blocks, B, Av, Am, Out, N, K, M, tiles_m,
                                                                                              tiles_n, nullptr, nullptr, 0, nullptr, nullptr);
}

// ------------------------------------------------------------------ sparse TN (weight gradient from a pruned dY)
// dW[m][n] = sum_t A[m][t] X[t][n] with A = S_z(dY^T) compressed along the tokens (Eq. 4).  The compressed
// operand takes the sparse NT kernel's path (chunk-major values and index words copied into the same LDS
// layout, one 128-bit read per fragment), the token-major X tile takes the dense TN kernel's (rows of 512 bytes
// copied as they lie, fragments gathered with the transposing LDS read).  A lane's dense fragment of a 64-token chunk is two
// 8-token runs 32 tokens apart: four transposing reads.
// MI and WN as in the sparse NT kernel: 256 x 256 tiles of eight waves, 256 (m) x 128 (n) and 128 x 128 ones of four; ring of
// three stages, fp32 output through LDS.
// On the 16-wide instruction, schedule of the NT kernel: 8192 tokens, 8192 x 28672 2044 -> 2014 us, 16384 tokens, 5120 x 1280
// 121 -> 115, 4160 tokens, 1600 x 6400 54.1 -> 53.3; smaller ones unchanged.
namespace sptn {
using big::a_slot;
using big::a_swizzle;
using big::glb_ptr;
using big::lds_ptr;

template <typename ET, bool ACCUM, bool DECAY, int MI, int WN>
__global__ __launch_bounds__(128 * WN) void spmm_tn_big_kernel(const uint16_t *__restrict__ Av,
                                                              const uint16_t *__restrict__ Am,
                                                              const uint16_t *__restrict__ X, float *__restrict__ dW,
                                                              int T, int M, int N, int tiles_m, int tiles_n,
                                                              unsigned long long *probe, const uint16_t *__restrict__ Wt,
                                                              const uint16_t *__restrict__ mask, float lambda)
{
    constexpr int BM = 64 * MI, BN = 64 * WN, WM = 32 * MI, ROWB = BN * 2, CPR = ROWB / 16;
    constexpr int B_STAGE = 64 * ROWB, A_STAGE = BM * 64, M_STAGE = BM * 8, STAGE = B_STAGE + A_STAGE + M_STAGE;
    constexpr int NA = 2 * MI / WN, NX = MI / WN, NC = 4 + NA + NX;   // copies per lane and chunk: values, index words, all
    const big::ClockStamp t_start = big::clock_now();
    __shared__ __attribute__((aligned(16))) unsigned char s0[STAGE];
    __shared__ __attribute__((aligned(16))) unsigned char s1[STAGE];
    __shared__ __attribute__((aligned(16))) unsigned char s2[STAGE];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    const int total = tiles_m * tiles_n, per_xcd = (total + 7) / 8;
    const int t = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (t >= total) return;
    constexpr int GROUP = 8;
    const int group_sz = GROUP * tiles_m, grp = t / group_sz, in_grp = t - grp * group_sz;
    const int gw = min(GROUP, tiles_n - grp * GROUP);
    const int tm = in_grp / gw, tn = grp * GROUP + in_grp % gw;
    const int m0 = tm * BM, n0 = tn * BN;
    const int nk = T / 64;

    // Copies per lane and chunk: four of the X tile, NA of the values, NX index dwords;
    // buffer loads into LDS with a wave-uniform base per operand and chunk and a fixed 32-bit byte offset per lane
    // (64 token rows of X and one chunk of the compressed operand span less than 4 GB: host check).
    const char *baseX = reinterpret_cast<const char *>(X), *baseV = reinterpret_cast<const char *>(Av);
    const char *baseM = reinterpret_cast<const char *>(Am);
    uint32_t ob[4], oa[NA], om[NX];
    const int lastB = (min(N - n0, BN) >> 3) - 1;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int slot = (wave * 4 + j) * 64 + lane, row = slot / CPR, c = (slot % CPR) ^ dmatn::tr_swizzle<16 * CPR>(row);
        ob[j] = ((uint32_t)row * (uint32_t)N + (uint32_t)(n0 + 8 * min(c, lastB))) * 2u;
    }
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int row = 16 * (NA * wave + i) + (lane >> 2);
        const int c = (lane & 3) ^ a_swizzle(row);
        oa[i] = ((uint32_t)min(m0 + row, M - 1) * 32u + 8u * c) * 2u;
    }
#pragma unroll
    for (int i = 0; i < NX; ++i) om[i] = ((uint32_t)min(m0 + 32 * (NX * wave + i) + (lane >> 1), M - 1) * 4u + 2u * (lane & 1)) * 2u;
    // Copy c of a chunk's NC per lane, spread over both phases of the main loop as in the sparse NT kernel; every chunk issues all
    // of them, past the last one it re-reads that into a stage nobody will read, so that the wait counts below are constants
    constexpr auto copy_slot = [](int c) { return c * 8 * MI / NC; };
    constexpr int EARLY = (NC + 1) / 2;
    const char *px = baseX, *pv = baseV, *pm = baseM;
    auto issue = [&](unsigned char *st, int c) {
        if (c < 4) big::buffer_to_lds<16>(big::buffer_of(px), (lds_ptr)(st + (wave * 4 + c) * 1024), ob[c]);
        else if (c < 4 + NA) big::buffer_to_lds<16>(big::buffer_of(pv), (lds_ptr)(st + B_STAGE + 16 * (NA * wave + c - 4) * 64), oa[c - 4]);
        else big::buffer_to_lds<4>(big::buffer_of(pm), (lds_ptr)(st + B_STAGE + A_STAGE + 256 * (NX * wave + c - 4 - NA)), om[c - 4 - NA]);
    };
    const int64_t step_x = (int64_t)N * 128, step_v = (int64_t)M * 64, step_m = (int64_t)M * 8;
    auto advance = [&](int kc) {   // to chunk kc, or not past the last one
        if (kc < nk) { px += step_x; pv += step_v; pm += step_m; }
    };
    auto issue_all = [&](unsigned char *st, int kc) {
        if (kc > 0) advance(kc);
#pragma unroll
        for (int c = 0; c < NC; ++c) issue(st, c);
    };

    f32x4 acc[2 * MI][4];
#pragma unroll
    for (int mi = 0; mi < 2 * MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < 4; ++ni) acc[mi][ni] = f32x4{};

    // X fragment addressing: lane group g = lane / 16 takes tokens 8g .. 8g+7 and 32 + 8g .. of a chunk, 16 columns per block
    const int l16 = lane & 15, g = lane >> 4;
    int offB[4];
#pragma unroll
    for (int ni = 0; ni < 4; ++ni) offB[ni] = dmatn::tr_off<ROWB>(8 * g + (l16 >> 2), 64 * wn + 16 * ni + 4 * (l16 & 3));
    // Quarter h of X fragment ni (four tokens a lane), value fragments and index words as in the NT kernel
    auto load_b = [&](const unsigned char *st, int ni, int h) {
        return dmatn::tr_half(st + offB[ni] + (32 * (h >> 1) + 4 * (h & 1)) * ROWB);
    };
    auto load_a = [&](const unsigned char *st, int mi) {
        return as_bf16x8(*reinterpret_cast<const uint4 *>(st + B_STAGE + 1024 * mi + a_slot(WM * wm + l16, g)));
    };
    const uint32_t half_sel = (g & 1) ? 0x07060302u : 0x05040100u;
    auto load_index = [&](const unsigned char *st, int i) {
        const unsigned char *p = st + B_STAGE + A_STAGE + 256 * i + (WM * wm + l16) * 8 + 4 * (g >> 1);
        return make_uint2(*reinterpret_cast<const uint32_t *>(p), *reinterpret_cast<const uint32_t *>(p + 128));
    };
    auto pack_index = [&](uint2 d) { return __builtin_amdgcn_perm(d.y, d.x, half_sel); };

    // keep the program order of these groups: the constant wait counts rely on it
    issue_all(s0, 0);
    __builtin_amdgcn_sched_barrier(0);
    issue_all(s1, 1);
    __builtin_amdgcn_sched_barrier(0);
    advance(2);
#pragma unroll
    for (int c = 0; c < EARLY; ++c) issue(s2, c);
    __builtin_amdgcn_sched_barrier(0);
    big::wait_and_barrier<NC + EARLY>();   // chunk 0 has landed for everybody
    struct Quarters { dmatn::v4i16 q[4]; };
    Quarters fb[4];
    bf16x8 fa0[MI];
    uint32_t ix[MI];
#pragma unroll
    for (int i = 0; i < MI / 2; ++i) ix[i] = pack_index(load_index(s0, i));
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) fa0[mi] = load_a(s0, mi);
#pragma unroll
    for (int ni = 0; ni < 4; ++ni)
#pragma unroll
        for (int h = 0; h < 4; ++h) fb[ni].q[h] = load_b(s0, ni, h);
    mma_tie<0, MI / 2>(ix);
    mma_tie<ACC_VGPR>(acc);
    mma_operands();

    // One chunk, pipelined across the workgroup barrier exactly as in the NT kernel: the first half's matrix
    // instructions run from registers while the second half's value fragments come in; after the one barrier of the chunk
    // the second half's matrix instructions cover the next chunk's fragments, each X fragment's four reads into the registers
    // of the one that has just had its last use, and the first copies of chunk kc+3 into the stage just vacated.
    auto chunk = [&](unsigned char *cur, const unsigned char *nxt, unsigned char *prv, int kc) {
        bf16x8 fa1[MI];
        uint2 raw[MI / 2];
        auto multiply = [&](const bf16x8 (&a)[MI], int first, int i) {   // the i-th matrix instruction of a phase
            const int ni = i / MI, j = i % MI, b = (ni & 1) ? MI - 1 - j : j, mi = first + b;
            const bf16x16 x = __builtin_bit_cast(bf16x16, fb[ni]);
            if (mi & 1) Mma<ET>::template sparse16<1>(a[b], x, acc[mi][ni], ix[mi / 2]);
            else Mma<ET>::template sparse16<0>(a[b], x, acc[mi][ni], ix[mi / 2]);
            __builtin_amdgcn_sched_barrier(0);
        };
#pragma unroll
        for (int i = 0; i < 4 * MI; ++i) {
            multiply(fa0, 0, i);
            if (i < MI) fa1[i] = load_a(cur, MI + i);
            if (i >= MI && i < MI + MI / 2) raw[i - MI] = load_index(cur, MI / 2 + i - MI);
#pragma unroll
            for (int c = EARLY; c < NC; ++c)
                if (copy_slot(c) - 4 * MI == i) issue(prv, c);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = 0; i < MI / 2; ++i) ix[MI / 2 + i] = pack_index(raw[i]);
        mma_tie<MI / 2, MI / 2>(ix);   // the wait and the barrier below are the wait states
        advance(kc + 3);
        big::wait_and_barrier<NC>();   // this lane's part of chunk kc+1 is in LDS, its own reads of chunk kc are done
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int i = 0; i < 4 * MI; ++i) {
            multiply(fa1, MI, i);
            if (i < MI) fa0[i] = load_a(nxt, i);
            if (i >= MI / 2 && i < MI) raw[i - MI / 2] = load_index(nxt, i - MI / 2);
            if (i >= MI) {   // block i / MI - 1 is done: its successor's four reads beside the MI instructions of the next block
#pragma unroll
                for (int h = 4 / MI * (i % MI); h < 4 / MI * (i % MI + 1); ++h) fb[i / MI - 1].q[h] = load_b(nxt, i / MI - 1, h);
            }
            if (i + 1 == 4 * MI) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int h = 0; h < 4; ++h) fb[3].q[h] = load_b(nxt, 3, h);
            }
#pragma unroll
            for (int c = 0; c < EARLY; ++c)
                if (copy_slot(c) == i) issue(cur, c);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = 0; i < MI / 2; ++i) ix[i] = pack_index(raw[i]);
        mma_tie<0, MI / 2>(ix);
        mma_operands();
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_sched_barrier(0);
    };
    // past the last chunk the prefetched fragments come from a stage that holds a re-read of the last chunk (or is
    // being refilled with one); they are never multiplied
    int kc = 0;
    for (; kc + 3 <= nk; kc += 3) {
        chunk(s0, s1, s2, kc);
        chunk(s1, s2, s0, kc + 1);
        chunk(s2, s0, s1, kc + 2);
    }
    if (kc < nk) chunk(s0, s1, s2, kc);
    if (kc + 1 < nk) chunk(s1, s2, s0, kc + 1);
    mma_drain<ACC_VGPR>(acc);
    big::wait_and_barrier<0>();   // copies drained, nobody reads the ring any more: reuse it
    big::clock_report(probe, t_start);
    // fp32 output through LDS in 16-byte row segments: a wave parks RB row blocks x 64 columns at a time in its part of
    // the ring, lane l of pass j owns row (64j + l) / 16, columns 4 * (l % 16) .. +3
    constexpr int RB = MI / 2, PER = WN == 4 ? 3 : 2, REGION = RB * 8192;   // PER waves' staging areas per ring stage
    static_assert(PER * REGION <= STAGE && 2 * WN <= 3 * PER, "staging areas must fit the ring");
    unsigned char *est = (wave < PER ? s0 : (wave < 2 * PER ? s1 : s2)) + (wave % PER) * REGION;
#pragma unroll
    for (int h2 = 0; h2 < MI / RB; ++h2) {
#pragma unroll
        for (int ni = 0; ni < 4; ++ni)
#pragma unroll
            for (int mj = 0; mj < 2 * RB; ++mj)
#pragma unroll
                for (int e = 0; e < 4; ++e) {   // 16-byte piece c of row r sits at slot c ^ (r & 12)
                    const int row = 16 * mj + 4 * g + e, c4 = 4 * ni + (l16 >> 2);
                    *reinterpret_cast<float *>(est + row * 256 + ((c4 ^ (row & 12)) << 4) + (l16 & 3) * 4) = acc[2 * RB * h2 + mj][ni][e];
                }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(big::wait_vm_lgkm0(0));   // the wave reads back only what it wrote itself
        asm volatile("" ::: "memory");
        constexpr int BATCH = 8;
#pragma unroll 1
        for (int j0 = 0; j0 < 8 * RB; j0 += BATCH) {
            float4 v[BATCH], old[BATCH];
            uint2 wv[BATCH];
            uint32_t keep[BATCH];
            bool live[BATCH];
#pragma unroll
            for (int b = 0; b < BATCH; ++b) {
                const int idx = (j0 + b) * 64 + lane, row = idx >> 4, c4 = idx & 15;
                const int m = m0 + WM * wm + 32 * RB * h2 + row, n = n0 + 64 * wn + 4 * c4;
                live[b] = m < M && n < N;   // N is a multiple of 16: the four columns are all in or all out
                const int mc = min(m, M - 1), nc = min(n, N - 4);
                v[b] = *reinterpret_cast<const float4 *>(est + row * 256 + ((c4 ^ (row & 12)) << 4));
                if (ACCUM) old[b] = *reinterpret_cast<const float4 *>(dW + (int64_t)mc * N + nc);
                if (DECAY) {
                    wv[b] = *reinterpret_cast<const uint2 *>(Wt + (int64_t)mc * N + nc);
                    keep[b] = mask[(int64_t)(mc >> 2) * (N >> 2) + (nc >> 2)] >> (4 * (mc & 3));
                }
            }
#pragma unroll
            for (int b = 0; b < BATCH; ++b) {
                const int idx = (j0 + b) * 64 + lane, row = idx >> 4, c4 = idx & 15;
                const int m = m0 + WM * wm + 32 * RB * h2 + row, n = n0 + 64 * wn + 4 * c4;
                float4 o = v[b];
                if (ACCUM) { o.x = old[b].x + o.x; o.y = old[b].y + o.y; o.z = old[b].z + o.z; o.w = old[b].w + o.w; }
                if (DECAY) {
                    if (!(keep[b] & 1u)) o.x = fmaf(lambda, s24_num<ET>::lo(wv[b].x), o.x);
                    if (!(keep[b] & 2u)) o.y = fmaf(lambda, s24_num<ET>::hi(wv[b].x), o.y);
                    if (!(keep[b] & 4u)) o.z = fmaf(lambda, s24_num<ET>::lo(wv[b].y), o.z);
                    if (!(keep[b] & 8u)) o.w = fmaf(lambda, s24_num<ET>::hi(wv[b].y), o.w);
                }
                if (live[b]) s24_store_stream(dW + (int64_t)m * N + n, o);
            }
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(big::wait_vm_lgkm0(0));   // LDS reads done before the other half overwrites
        asm volatile("" ::: "memory");
    }
}
}  // namespace sptn

__global__ __launch_bounds__(kThreads) void fill_zero_kernel(float *__restrict__ p, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < n) p[i] = 0.0f;
}

inline unsigned ceil_div(int64_t a, int64_t b) { return (unsigned)((a + b - 1) / b); }

unsigned long long *g_clock_probe = nullptr;   // device buffer of two counters, or none

// dtype and sizes first; pointers are only required when the output is not empty.
int check_gemm(const void *a, const void *b, const void *c, int64_t p, int64_t q, int64_t r, int dt, int64_t out_elems)
{
    S24_REQUIRE(s24_valid_dtype(dt), S24_ERR_DTYPE);
    S24_REQUIRE(p >= 0 && q >= 0 && r >= 0, S24_ERR_SHAPE);
    S24_REQUIRE(p < (1ll << 31) && q < (1ll << 31) && r < (1ll << 31), S24_ERR_SHAPE);
    // the large-tile kernels address a tile's operand rows with 32-bit byte offsets from a per-tile base:
    // 256 rows of the contraction axis, and all rows of one 64-chunk of a compressed operand, must span < 4 GB
    S24_REQUIRE(q < (1ll << 23) && r < (1ll << 23), S24_ERR_SHAPE);
    if (out_elems == 0) return S24_OK;
    S24_REQUIRE(a && b && c, S24_ERR_NULL);
    S24_REQUIRE(s24_aligned(a, 16) && s24_aligned(b, 16) && s24_aligned(c, 16), S24_ERR_ALIGN);
    return S24_OK;
}

// Runs `...` with T bound to the storage type of a 16-bit dtype.
#define S24_WITH_16BIT_TYPE(dt, ...)      \
    do {                                  \
        if ((dt) == S24_BF16) {           \
            using T = uint16_t;           \
            __VA_ARGS__;                  \
        } else {                          \
            using T = s24_half;           \
            __VA_ARGS__;                  \
        }                                 \
    } while (0)

// Which tile a sparse NT product takes.  Costs in full rounds of the large tile at the same depth (us per 64 of k at K = 5504 to
// 11008: large 0.82 with every compute unit busy and 0.53 with few; medium 0.45 and 0.33; small 0.58 with two workgroups per
// compute unit, 0.29 with one, 0.27 with few):
//   large    256 x 256, one workgroup per compute unit: least LDS and L2 traffic per FLOP, where its tiles fill the chip
//   medium   256 x 128: between half a round and a round of them, e.g. 4160 tokens x 1600 features, K = 6400: large 65, small
//            62, medium 48 us; 3001 x 2048, K = 11008: 104, 97, 72 us
//   small    128 x 128, two per compute unit: at most one round of single ones (1024 x 2048, K = 5504: large 51, medium 34,
//            small 27 us), or a contraction so short that a tile is mostly prologue and epilogue, which two co-resident
//            workgroups overlap (8192 x 3072, K = 768 with activation: 50, 56, 49 us; 8508 x 2112, K = 384: 22, 22, 19)
// The constants are a fit to the kernels on the 32-wide instruction, over 128-16384 tokens, 256-4096 x 1024-22016 features.  On the
// present ones a round of small tiles measures 0.57, 0.59, 0.61, 0.63 and 0.69 of a large one at K = 384, 640, 1024, 2048 and 5504,
// flatter than the 0.505 to 0.82 below; with every tile timed at 128 products (128-16384 tokens, widths of 256-17000) the tile
// chosen takes 0.8 % more than the best one at the mean and 2 % at the ninetieth percentile.
// A grid of large tiles whose last round is mostly empty (320 tiles on 256 compute units) can give its last token-tile rows
// to a smaller tile: the first `slab` tokens run in whole rounds of large tiles (16384 x 1280, K = 5120: 122 -> 112 us), where
// that saves more than the second launch costs, 3 us of a round's 5 + 0.75 per 64 of k (2347 x 20032, K = 384, is not cut: 47 us in
// large tiles, 41 in small ones).
// Tokens are independent rows and these tiles sum in the same order: the choice among them does not change a bit of the
// result.  (The slices of s24_gemm_slice.hip, chosen before them, sum in another.)
struct NtTile {
    enum Kind { Large, Medium, Small } kind;
    int64_t slab;   // tokens of a first launch of its own, or 0
    int bm() const { return kind == Small ? 128 : 256; }
    int bn() const { return kind == Large ? 256 : 128; }
    int threads() const { return kind == Large ? 512 : 256; }
};
// Cost of a full round of medium and small tiles, and of a partial round (offset, slope over its fill) of each kind
struct NtCosts {
    double large0, large1, medium, medium0, medium1, small, small0, small1;
};
inline double nt_cost(NtTile::Kind kind, int64_t M, int64_t N, const NtCosts &c)
{
    const int64_t cus = s24_cu_count();
    const NtTile t{kind, 0};
    const int64_t tiles = (int64_t)ceil_div(M, t.bm()) * ceil_div(N, t.bn()), per = kind == NtTile::Small ? 2 * cus : cus;
    const double full = (double)(tiles / per), rest = (double)(tiles % per) / cus;
    if (kind == NtTile::Large) return full + (rest > 0 ? c.large0 + c.large1 * rest : 0);
    if (kind == NtTile::Medium) return c.medium * full + (rest > 0 ? c.medium0 + c.medium1 * rest : 0);
    return c.small * full + (rest == 0 ? 0 : rest <= 1 ? c.small0 + c.small1 * rest : c.small);
}
inline NtTile cheapest_tile(int64_t M, int64_t N, const NtCosts &c)
{
    const double l = nt_cost(NtTile::Large, M, N, c), m = nt_cost(NtTile::Medium, M, N, c), s = nt_cost(NtTile::Small, M, N, c);
    return {l <= m && l <= s ? NtTile::Large : m <= s ? NtTile::Medium : NtTile::Small, 0};
}
inline NtCosts sparse_costs(int64_t K) { return {0.73, 0.27, 0.69, 0.49, 0.20, K <= 640 ? 0.505 : K <= 1024 ? 0.54 : K <= 2048 ? 0.7 : 0.82, 0.37, 0.06}; }
inline double round_us(int64_t K) { return 5.0 + 0.75 * (double)(K / 64); }   // a round of large tiles
inline NtTile nt_tile(int64_t M, int64_t N, int64_t K) { return cheapest_tile(M, N, sparse_costs(K)); }
// The same for a product whose tokens may be cut in two launches
inline NtTile nt_tile_or_slab(int64_t M, int64_t N, int64_t K)
{
    NtTile t = nt_tile(M, N, K);
    const int64_t cus = s24_cu_count(), tm = ceil_div(M, 256), tiles = tm * ceil_div(N, 256);
    if (tiles <= cus || tiles % cus == 0 || tm > cus) return t;
    const int64_t rows = tiles / cus * cus / tm, slab = 256 * rows;   // whole token-tile rows within the whole rounds
    const NtCosts c = sparse_costs(K);
    const NtTile strip = cheapest_tile(M, N - slab, c);
    const double cut = nt_cost(NtTile::Large, M, slab, c) + nt_cost(strip.kind, M, N - slab, c) + 3.0 / round_us(K);
    if (cut < nt_cost(t.kind, M, N, c)) t.slab = slab;
    return t;
}
// The dense product: us per 64 of k, large 1.45 and 0.94 (full, few), medium 0.85 and 0.54, small 1.04 with two workgroups per
// compute unit, 0.44 with one.  8192 x 1024, K = 4096: large 75, medium 65, small 76 us; 500 x 4096, K = 16384: 240, 178, 119;
// 2048 x 3072, K = 768: 20, 16, 17.  0.5 % above the best tile at the mean of 128 products.  (On one set of operands, launched on end.  Out of
// the caches they add their way in: the first product in medium tiles 64 us so, 76 on eight sets in turn, 79 in a dense step.)
inline NtTile dense_tile(int64_t M, int64_t N) { return cheapest_tile(M, N, {0.53, 0.30, 0.62, 0.40, 0.20, 0.70, 0.26, 0.08}); }
// The sparse weight gradient: us per 64 tokens, large 0.83 and 0.53 (full, few), medium 0.46 and 0.35, small 0.63 with two
// workgroups per compute unit and 0.30 with one.  8192 tokens, 768 x 3072: large 77, medium 54, small 45 us; 2048, 512 x 2048: 24,
// 16, 14; 16384, 1280 x 5120: 162, 117, 215; 3008, 1472 x 4032: 37, 27, 31.  0.8 % above the best tile at the mean of 128.
inline NtTile sparse_dw_tile(int64_t M, int64_t N) { return cheapest_tile(M, N, {0.50, 0.45, 0.62, 0.36, 0.10, 0.60, 0.29, 0.08}); }
// Runs MACRO(..., MI, WN) with the wave layout of a tile
#define S24_WITH_NT_TILE(tile, MACRO, ...)                              \
    do {                                                                \
        if ((tile).kind == NtTile::Large) MACRO(__VA_ARGS__, 4, 4);     \
        else if ((tile).kind == NtTile::Medium) MACRO(__VA_ARGS__, 4, 2); \
        else MACRO(__VA_ARGS__, 2, 2);                                  \
    } while (0)

// Whether a product of N tokens and M features runs in slices (s24_gemm_slice.hip), and in which.  Up to 16 tokens, of which a tile would multiply
// seven eighths of nothing: yes (16 x 16384, K = 4096, weights out of the caches: 28 us in tiles, 13.7 in slices; x 50304: 44.5 and 43.0),
// unless the 128 x 128 tiles are nearly two per compute unit and the contraction is long, so that they too keep the memory busy
// (x 65536, K = 8192: 103 and 109; K = 2048: 40 and 29; 57344, K = 8192: 95 and 92).  With more tokens not where these tiles are more than
// one per compute unit (40 x 43008, K = 8192: 84 and 93), else where that is estimated to be the faster.  The small grids in question
// keep a tile's launch, prologue and epilogue in the open: 2.5 us beyond the share of a round, the middle of 1 without and 4 with an
// activation, since one rule for all epilogues gives them the same bits.  Weights out of the caches come in at 5 TB/s either way.  Of 380
// products (1-2048 tokens, K = 256-32000, 256-56000 features) the choice takes 1 % more than the best tile of either kind at the mean.
inline S24SlicePlan slices_if_faster(int64_t N, int64_t K, int64_t M)
{
    const int64_t cus = s24_cu_count(), small = (int64_t)ceil_div(M, 128) * ceil_div(N, 128);
    if (N <= 16) return K >= 4096 && 4 * small > 7 * cus && small <= 2 * cus ? S24SlicePlan{} : s24_slice_plan(N, K, M);
    if (small > cus) return {};
    const NtCosts c = sparse_costs(K);
    const double tiles = 2.5 + round_us(K) * std::min(nt_cost(NtTile::Large, M, N, c), std::min(nt_cost(NtTile::Medium, M, N, c), nt_cost(NtTile::Small, M, N, c)));
    const S24SlicePlan p = s24_slice_plan(N, K, M);
    return p.us <= std::max(tiles, 2.0 + 1.125 * (double)M * (double)K / 5.0e6) ? p : S24SlicePlan{};
}

// Outputs that the gated backward epilogue serves: three quarters of the compute units have a large tile
inline bool gated_bwd_fits(int64_t p, int64_t f) { return (int64_t)ceil_div(f, 256) * ceil_div(p, 256) >= 3 * s24_cu_count() / 4; }

// Whether the input gradient of p tokens and q features, contraction r, runs in slices.  One rule for s24_spmm_bwd_dx and
// s24_spmm_bwd_dx_act, whose bits agree; and neither does where s24_spmm_bwd_dx_glu takes its large tiles (possible at up to
// 16 tokens from 48897 features on), so that all three sum in one order.
inline S24SlicePlan bwd_dx_slices(int64_t p, int64_t r, int64_t q) { return gated_bwd_fits(p, q) ? S24SlicePlan{} : slices_if_faster(p, r, q); }

// Out[N][M] = beta * Out + B[N][K] . A^T (+ bias[M], only with beta = 0)
int launch_spmm(const void *B, const void *Av, const uint16_t *Am, void *Out, int64_t N, int64_t K, int64_t M, float beta,
                int dt, hipStream_t st, const void *bias, const S24SlicePlan &slices)
{
    if (N == 0 || M == 0) return S24_OK;
    const bool accum = beta != 0.0f;
    if (dt == S24_F32) {
        return s24_f32_nt({static_cast<const float *>(B), static_cast<const float *>(Av), Am, static_cast<float *>(Out), nullptr,
                           static_cast<const float *>(bias), N, K, M, accum, S24_F32_PLAIN, 0}, st);
    }
    auto *b = static_cast<const uint16_t *>(B), *av = static_cast<const uint16_t *>(Av), *d = static_cast<const uint16_t *>(bias);
    auto *o = static_cast<uint16_t *>(Out);
    S24_REQUIRE((int64_t)ceil_div(M, 128) * ceil_div(N, 128) < (1ll << 30), S24_ERR_SHAPE);
    if (slices) return s24_slice_nt({b, av, Am, o, nullptr, nullptr, d, N, K, M, accum, S24_SLICE_PLAIN, 0}, slices, dt, st);
    const NtTile tile = nt_tile_or_slab(M, N, K);
    if (tile.slab != 0) {
        const int rc = launch_spmm(B, Av, Am, Out, tile.slab, K, M, beta, dt, st, bias, {});
        if (rc != S24_OK) return rc;
        return launch_spmm(b + tile.slab * K, Av, Am, o + tile.slab * M, N - tile.slab, K, M, beta, dt, st, bias, {});
    }
    const int tiles_m = (int)ceil_div(M, tile.bm()), tiles_n = (int)ceil_div(N, tile.bn());
    const dim3 grid(((tiles_m * tiles_n + 7) / 8) * 8), block(tile.threads());
#define S24_LAUNCH_NT(ACC, BIASED, MI, WN)                                                                                             \
    hipLaunchKernelGGL((big::spmm_nt_big_kernel<T, ACC, false, false, S24_GATE_SILU, BIASED, 0, S24_ACT_RELU, MI, WN>), grid, block, 0, \
                       st, b, av, Am, o, (int)N, (int)K, (int)M, tiles_m, tiles_n, tile.kind == NtTile::Large ? g_clock_probe : nullptr, \
                       nullptr, 0, nullptr, d)
    S24_WITH_16BIT_TYPE(dt, {
        if (accum) S24_WITH_NT_TILE(tile, S24_LAUNCH_NT, true, false);
        else if (d != nullptr) S24_WITH_NT_TILE(tile, S24_LAUNCH_NT, false, true);
        else S24_WITH_NT_TILE(tile, S24_LAUNCH_NT, false, false);
    });
#undef S24_LAUNCH_NT
    return s24_launch_status();
}

}  // namespace

extern "C" int s24_spmm_fwd(const void *X, const void *vals, const uint16_t *meta, void *Y, int64_t p, int64_t q, int64_t r,
                            s24_dtype dt, void *stream)
{
    return s24_spmm_fwd_bias(X, vals, meta, nullptr, Y, p, q, r, dt, stream);
}

extern "C" int s24_spmm_fwd_bias(const void *X, const void *vals, const uint16_t *meta, const void *bias, void *Y, int64_t p,
                                 int64_t q, int64_t r, s24_dtype dt, void *stream)
{
    S24_REQUIRE(q % 64 == 0 && r % 16 == 0 && q > 0, S24_ERR_SHAPE);
    const int rc = check_gemm(X, vals, Y, p, q, r, dt, p * r);
    if (rc != S24_OK || p * r == 0) return rc;
    S24_REQUIRE(meta != nullptr, S24_ERR_NULL);
    S24_REQUIRE(s24_aligned(meta, 4) && s24_aligned(bias, 8), S24_ERR_ALIGN);
    return launch_spmm(X, vals, meta, Y, p, q, r, 0.0f, dt, static_cast<hipStream_t>(stream), bias, dt == S24_F32 ? S24SlicePlan{} : slices_if_faster(p, q, r));
}

extern "C" int s24_spmm_bwd_dx(const void *dY, const void *valsT, const uint16_t *metaT, void *dX, int64_t p, int64_t q,
                               int64_t r, float beta, s24_dtype dt, void *stream)
{
    S24_REQUIRE(r % 64 == 0 && q % 16 == 0 && r > 0, S24_ERR_SHAPE);
    S24_REQUIRE(beta == 0.0f || beta == 1.0f, S24_ERR_UNSUPPORTED);
    const int rc = check_gemm(dY, valsT, dX, p, q, r, dt, p * q);
    if (rc != S24_OK || p * q == 0) return rc;
    S24_REQUIRE(metaT != nullptr, S24_ERR_NULL);
    S24_REQUIRE(s24_aligned(metaT, 4), S24_ERR_ALIGN);
    return launch_spmm(dY, valsT, metaT, dX, p, r, q, beta, dt, static_cast<hipStream_t>(stream), nullptr, dt == S24_F32 ? S24SlicePlan{} : bwd_dx_slices(p, r, q));
}

extern "C" int s24_spmm_fwd_glu(const void *X, const void *vals, const uint16_t *meta, const void *bias, void *GU, void *H,
                                int64_t p, int64_t q, int64_t f, s24_gate gate, s24_dtype dt, void *stream)
{
    S24_REQUIRE(s24_valid_gate(gate), S24_ERR_DTYPE);
    S24_REQUIRE(q % 64 == 0 && f % 16 == 0 && q > 0, S24_ERR_SHAPE);
    const int rc = check_gemm(X, vals, GU, p, q, 2 * f, dt, p * f);
    if (rc != S24_OK || p * f == 0) return rc;
    S24_REQUIRE(meta != nullptr && H != nullptr, S24_ERR_NULL);
    S24_REQUIRE(s24_aligned(meta, 4) && s24_aligned(H, 16) && s24_aligned(bias, 8), S24_ERR_ALIGN);
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (const S24SlicePlan slices = dt == S24_F32 ? S24SlicePlan{} : slices_if_faster(p, q, 2 * f))
        return s24_slice_nt({static_cast<const uint16_t *>(X), static_cast<const uint16_t *>(vals), meta, static_cast<uint16_t *>(GU),
                             static_cast<uint16_t *>(H), nullptr, static_cast<const uint16_t *>(bias), p, q, 2 * f, false, S24_SLICE_GLU, gate}, slices, dt, st);
    NtTile tile = nt_tile(2 * f, p, q);
    // The small tile has no gated epilogue: it is taken only where it saves more than the pass over Z costs, 2.4 us per million
    // gated features (6 bytes each) less the 1 us that the fused epilogue costs itself.  10041 tokens, 19072 rows, K = 64: fused
    // 122 us, in two calls 209; 2655 x 7360, K = 448: 28 and 31; but 527 x 1312, K = 960: 12.9 and 9.2.
    if (tile.kind == NtTile::Small) {
        const NtCosts c = sparse_costs(q);
        const double l = nt_cost(NtTile::Large, 2 * f, p, c), m = nt_cost(NtTile::Medium, 2 * f, p, c);
        const double pass = (2.4e-6 * (double)p * (double)f - 1.0) / (2.0 + round_us(q));
        if (std::min(l, m) < nt_cost(NtTile::Small, 2 * f, p, c) + pass) tile.kind = l <= m ? NtTile::Large : NtTile::Medium;
    }
    if (dt != S24_F32 && tile.kind != NtTile::Small) {   // 128 gate and 128 up features per tile
        const int tiles_m = (int)ceil_div(f, 128), tiles_n = (int)ceil_div(p, tile.bn());
        const dim3 grid(((tiles_m * tiles_n + 7) / 8) * 8), block(tile.threads());
        auto *x = static_cast<const uint16_t *>(X), *av = static_cast<const uint16_t *>(vals), *d = static_cast<const uint16_t *>(bias);
        auto *gu = static_cast<uint16_t *>(GU), *h = static_cast<uint16_t *>(H);
#define S24_LAUNCH_FWD_GLU(G, WN)                                                                                                    \
    hipLaunchKernelGGL((big::spmm_nt_big_kernel<T, false, true, false, G, false, 0, S24_ACT_RELU, 4, WN>), grid, block, 0, st, x, av, meta, \
                       gu, (int)p, (int)q, (int)(2 * f), tiles_m, tiles_n, tile.kind == NtTile::Large ? g_clock_probe : nullptr, h, (int)f, \
                       nullptr, d)
        S24_WITH_16BIT_TYPE(dt, {
            if (gate == S24_GATE_SILU && tile.kind == NtTile::Large) S24_LAUNCH_FWD_GLU(S24_GATE_SILU, 4);
            else if (gate == S24_GATE_SILU) S24_LAUNCH_FWD_GLU(S24_GATE_SILU, 2);
            else if (tile.kind == NtTile::Large) S24_LAUNCH_FWD_GLU(S24_GATE_GELU_ERF, 4);
            else S24_LAUNCH_FWD_GLU(S24_GATE_GELU_ERF, 2);
        });
#undef S24_LAUNCH_FWD_GLU
        return s24_launch_status();
    }
    if (dt == S24_F32)
        return s24_f32_nt({static_cast<const float *>(X), static_cast<const float *>(vals), meta, static_cast<float *>(GU), static_cast<float *>(H),
                           static_cast<const float *>(bias), p, q, 2 * f, false, S24_F32_GLU, gate}, st);
    // shapes the fused epilogue does not cover: the GEMM into [p][2f], then the stand-alone activation on its halves
    const int rc2 = launch_spmm(X, vals, meta, GU, p, q, 2 * f, 0.0f, dt, st, bias, {});
    if (rc2 != S24_OK) return rc2;
    return s24_glu_fwd(GU, S24_ROW_MAJOR, 2 * f, H, S24_ROW_MAJOR, f, p, f, gate, dt, st);
}

extern "C" int s24_spmm_fwd_swiglu(const void *X, const void *vals, const uint16_t *meta, void *GU, void *H, int64_t p,
                                   int64_t q, int64_t f, s24_dtype dt, void *stream)
{
    return s24_spmm_fwd_glu(X, vals, meta, nullptr, GU, H, p, q, f, S24_GATE_SILU, dt, stream);
}

extern "C" int s24_spmm_bwd_dx_glu(const void *dY, const void *valsT, const uint16_t *metaT, const void *GU, void *dGU,
                                   int64_t p, int64_t f, int64_t r, s24_gate gate, s24_dtype dt, void *stream)
{
    S24_REQUIRE(s24_valid_gate(gate), S24_ERR_DTYPE);
    S24_REQUIRE(r % 64 == 0 && f % 16 == 0 && r > 0, S24_ERR_SHAPE);
    const int rc = check_gemm(dY, valsT, dGU, p, f, r, dt, p * f);
    if (rc != S24_OK || p * f == 0) return rc;
    S24_REQUIRE(metaT != nullptr && GU != nullptr, S24_ERR_NULL);
    S24_REQUIRE(s24_aligned(metaT, 4) && s24_aligned(GU, 16), S24_ERR_ALIGN);
    const int tiles_m = (int)ceil_div(f, big::BM), tiles_n = (int)ceil_div(p, big::BN);
    // only the large-tile 16-bit kernel carries this epilogue; other shapes take s24_spmm_bwd_dx + s24_glu_bwd
    S24_REQUIRE(dt != S24_F32 && gated_bwd_fits(p, f), S24_ERR_UNSUPPORTED);
    const dim3 grid(((tiles_m * tiles_n + 7) / 8) * 8), block(big::THREADS);
    hipStream_t st = static_cast<hipStream_t>(stream);
    auto *dy = static_cast<const uint16_t *>(dY), *av = static_cast<const uint16_t *>(valsT), *gu = static_cast<const uint16_t *>(GU);
    auto *o = static_cast<uint16_t *>(dGU);
#define S24_LAUNCH_BWD_GLU(G)                                                                                              \
    hipLaunchKernelGGL((big::spmm_nt_big_kernel<T, false, false, true, G>), grid, block, 0, st, dy, av, metaT, o, (int)p, \
                       (int)r, (int)f, tiles_m, tiles_n, g_clock_probe, nullptr, 0, gu, nullptr)
    S24_WITH_16BIT_TYPE(dt, {
        if (gate == S24_GATE_SILU) S24_LAUNCH_BWD_GLU(S24_GATE_SILU);
        else S24_LAUNCH_BWD_GLU(S24_GATE_GELU_ERF);
    });
#undef S24_LAUNCH_BWD_GLU
    return s24_launch_status();
}

extern "C" int s24_spmm_bwd_dx_swiglu(const void *dY, const void *valsT, const uint16_t *metaT, const void *GU, void *dGU,
                                      int64_t p, int64_t f, int64_t r, s24_dtype dt, void *stream)
{
    return s24_spmm_bwd_dx_glu(dY, valsT, metaT, GU, dGU, p, f, r, S24_GATE_SILU, dt, stream);
}

extern "C" int s24_spmm_fwd_act(const void *X, const void *vals, const uint16_t *meta, const void *bias, void *Z, void *H,
                                int64_t p, int64_t q, int64_t r, s24_act act, s24_dtype dt, void *stream)
{
    S24_REQUIRE(act == S24_ACT_RELU || act == S24_ACT_GELU_ERF, S24_ERR_DTYPE);
    S24_REQUIRE(q % 64 == 0 && r % 16 == 0 && q > 0, S24_ERR_SHAPE);
    const int rc = check_gemm(X, vals, Z, p, q, r, dt, p * r);
    if (rc != S24_OK || p * r == 0) return rc;
    S24_REQUIRE(meta != nullptr && H != nullptr, S24_ERR_NULL);
    S24_REQUIRE(s24_aligned(meta, 4) && s24_aligned(H, 16) && s24_aligned(bias, 8), S24_ERR_ALIGN);
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (dt != S24_F32) {
        if (const S24SlicePlan slices = slices_if_faster(p, q, r))
            return s24_slice_nt({static_cast<const uint16_t *>(X), static_cast<const uint16_t *>(vals), meta, static_cast<uint16_t *>(Z),
                                 static_cast<uint16_t *>(H), nullptr, static_cast<const uint16_t *>(bias), p, q, r, false, S24_SLICE_ACT, act}, slices, dt, st);
        const NtTile tile = nt_tile(r, p, q);
        const int tiles_m = (int)ceil_div(r, tile.bm()), tiles_n = (int)ceil_div(p, tile.bn());
        S24_REQUIRE((int64_t)tiles_m * tiles_n < (1ll << 30), S24_ERR_SHAPE);
        const dim3 grid(((tiles_m * tiles_n + 7) / 8) * 8), block(tile.threads());
        auto *x = static_cast<const uint16_t *>(X), *av = static_cast<const uint16_t *>(vals), *d = static_cast<const uint16_t *>(bias);
        auto *z = static_cast<uint16_t *>(Z), *h = static_cast<uint16_t *>(H);
#define S24_LAUNCH_FWD_ACT(A, BIASED, MI, WN)                                                                                           \
    hipLaunchKernelGGL((big::spmm_nt_big_kernel<T, false, false, false, S24_GATE_SILU, BIASED, 1, A, MI, WN>), grid, block, 0, st, x, av, \
                       meta, z, (int)p, (int)q, (int)r, tiles_m, tiles_n, tile.kind == NtTile::Large ? g_clock_probe : nullptr, h, 0,     \
                       nullptr, d)
        S24_WITH_16BIT_TYPE(dt, {
            if (act == S24_ACT_RELU && d != nullptr) S24_WITH_NT_TILE(tile, S24_LAUNCH_FWD_ACT, S24_ACT_RELU, true);
            else if (act == S24_ACT_RELU) S24_WITH_NT_TILE(tile, S24_LAUNCH_FWD_ACT, S24_ACT_RELU, false);
            else if (d != nullptr) S24_WITH_NT_TILE(tile, S24_LAUNCH_FWD_ACT, S24_ACT_GELU_ERF, true);
            else S24_WITH_NT_TILE(tile, S24_LAUNCH_FWD_ACT, S24_ACT_GELU_ERF, false);
        });
#undef S24_LAUNCH_FWD_ACT
        return s24_launch_status();
    }
    return s24_f32_nt({static_cast<const float *>(X), static_cast<const float *>(vals), meta, static_cast<float *>(Z), static_cast<float *>(H),
                       static_cast<const float *>(bias), p, q, r, false, S24_F32_ACT, act}, st);
}

extern "C" int s24_spmm_bwd_dx_act(const void *dY, const void *valsT, const uint16_t *metaT, const void *Z, void *dZ,
                                   int64_t p, int64_t f, int64_t r, s24_act act, s24_dtype dt, void *stream)
{
    S24_REQUIRE(act == S24_ACT_RELU || act == S24_ACT_GELU_ERF, S24_ERR_DTYPE);
    S24_REQUIRE(r % 64 == 0 && f % 16 == 0 && r > 0, S24_ERR_SHAPE);
    const int rc = check_gemm(dY, valsT, dZ, p, f, r, dt, p * f);
    if (rc != S24_OK || p * f == 0) return rc;
    S24_REQUIRE(metaT != nullptr && Z != nullptr, S24_ERR_NULL);
    S24_REQUIRE(s24_aligned(metaT, 4) && s24_aligned(Z, 16), S24_ERR_ALIGN);
    // the 16-bit kernels carry this epilogue; fp32 takes s24_spmm_bwd_dx + s24_act_bwd
    S24_REQUIRE(dt != S24_F32, S24_ERR_UNSUPPORTED);
    if (const S24SlicePlan slices = bwd_dx_slices(p, r, f))
        return s24_slice_nt({static_cast<const uint16_t *>(dY), static_cast<const uint16_t *>(valsT), metaT, static_cast<uint16_t *>(dZ), nullptr,
                             static_cast<const uint16_t *>(Z), nullptr, p, r, f, false, S24_SLICE_ACT_BWD, act}, slices, dt, static_cast<hipStream_t>(stream));
    const NtTile tile = nt_tile(f, p, r);
    const int tiles_m = (int)ceil_div(f, tile.bm()), tiles_n = (int)ceil_div(p, tile.bn());
    S24_REQUIRE((int64_t)tiles_m * tiles_n < (1ll << 30), S24_ERR_SHAPE);
    const dim3 grid(((tiles_m * tiles_n + 7) / 8) * 8), block(tile.threads());
    hipStream_t st = static_cast<hipStream_t>(stream);
    auto *dy = static_cast<const uint16_t *>(dY), *av = static_cast<const uint16_t *>(valsT), *z = static_cast<const uint16_t *>(Z);
    auto *o = static_cast<uint16_t *>(dZ);
#define S24_LAUNCH_BWD_ACT(A, MI, WN)                                                                                                  \
    hipLaunchKernelGGL((big::spmm_nt_big_kernel<T, false, false, false, S24_GATE_SILU, false, 2, A, MI, WN>), grid, block, 0, st, dy, av, \
                       metaT, o, (int)p, (int)r, (int)f, tiles_m, tiles_n, tile.kind == NtTile::Large ? g_clock_probe : nullptr, nullptr, \
                       0, z, nullptr)
    S24_WITH_16BIT_TYPE(dt, {
        if (act == S24_ACT_RELU) S24_WITH_NT_TILE(tile, S24_LAUNCH_BWD_ACT, S24_ACT_RELU);
        else S24_WITH_NT_TILE(tile, S24_LAUNCH_BWD_ACT, S24_ACT_GELU_ERF);
    });
#undef S24_LAUNCH_BWD_ACT
    return s24_launch_status();
}

extern "C" int s24_dense_gemm(const void *X, const void *W, void *Y, int64_t p, int64_t q, int64_t r, s24_dtype dt,
                              void *stream)
{
    S24_REQUIRE(q % 64 == 0 && r % 16 == 0 && q > 0, S24_ERR_SHAPE);
    const int rc = check_gemm(X, W, Y, p, q, r, dt, p * r);
    if (rc != S24_OK || p * r == 0) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (dt == S24_F32) {
        return s24_f32_nt({static_cast<const float *>(X), static_cast<const float *>(W), nullptr, static_cast<float *>(Y), nullptr, nullptr, p, q, r,
                           false, S24_F32_PLAIN, 0}, st);
    }
    auto *x = static_cast<const uint16_t *>(X), *w = static_cast<const uint16_t *>(W);
    auto *y = static_cast<uint16_t *>(Y);
    S24_REQUIRE((int64_t)ceil_div(r, 128) * ceil_div(p, 128) < (1ll << 30), S24_ERR_SHAPE);
    const NtTile tile = dense_tile(r, p);
    const int tiles_m = (int)ceil_div(r, tile.bm()), tiles_n = (int)ceil_div(p, tile.bn());
    const dim3 grid(((tiles_m * tiles_n + 7) / 8) * 8), block(tile.threads());
#define S24_LAUNCH_DENSE(MI, WN)                                                                                              \
    hipLaunchKernelGGL((bignt::dense_nt_big_kernel<T, MI, WN>), grid, block, 0, st, x, w, y, (int)p, (int)q, (int)r, tiles_m, \
                       tiles_n, tile.kind == NtTile::Large ? g_clock_probe : nullptr)
    S24_WITH_16BIT_TYPE(dt, {
        if (tile.kind == NtTile::Large) S24_LAUNCH_DENSE(4, 4);
        else if (tile.kind == NtTile::Medium) S24_LAUNCH_DENSE(4, 2);
        else S24_LAUNCH_DENSE(2, 2);
    });
#undef S24_LAUNCH_DENSE
    return s24_launch_status();
}

namespace {
// One weight gradient as the batched kernel sees it (16-bit operands; W == nullptr: no decay term)
struct DwProblem {
    const uint16_t *dY, *X;
    float *dW;
    const uint16_t *W, *mask;
    int64_t p, q, r;
    float lambda;
};
enum class DwTile { Large, Medium, Small, Medium192 };   // 256 x 256, 256 x 128, 128 x 128, 192 x 128
int64_t dw_tiles_m(DwTile t, int64_t r) { return ceil_div(r, t == DwTile::Small ? 128 : t == DwTile::Medium192 ? 192 : 256); }
int64_t dw_tiles_n(DwTile t, int64_t q) { return ceil_div(q, t == DwTile::Large ? 256 : 128); }
// The window [m_off, m_off + mm) x [n_off, n_off + nn) of a problem's output, in tiles of `tile`
dmatn::DwWindow dw_window(const DwProblem &pr, DwTile tile, int64_t m_off, int64_t mm, int64_t n_off, int64_t nn)
{
    dmatn::DwWindow w{};
    w.dY = pr.dY + m_off;
    w.X = pr.X + n_off;
    w.dW = pr.dW + m_off * pr.q + n_off;
    w.Wt = pr.W ? pr.W + m_off * pr.q + n_off : nullptr;
    w.mask = pr.W ? pr.mask + (m_off / 4) * (pr.q / 4) + n_off / 4 : nullptr;
    w.T = (int)pr.p;
    w.M = (int)mm;
    w.N = (int)nn;
    w.ldy = (int)pr.r;
    w.ldx = (int)pr.q;
    w.ldw = (int)pr.q;
    w.tiles_m = (int)dw_tiles_m(tile, mm);
    w.tiles_n = (int)dw_tiles_n(tile, nn);
    w.lambda = pr.lambda;
    return w;
}
// Tile of a grid that the large tile does not fill, by cost in us (fitted to every tile's time at 40 pairs of gradients, 128-11000
// tokens, layers of 256 x 768 to 1408 x 4608; the bits are the same).  Per 32 tokens: small tiles 0.53 with two workgroups per
// compute unit and 0.18 with one, medium ones 0.45 and 0.24 with few, large ones 0.75 and 0.43; on top of that the filling and
// draining of a tile.  The small tile reads 32 KB of LDS per 16 KB copied, the medium one 48 per 24 for twice the work: where the
// small tile needs two workgroups per compute unit and the medium one does not, that is 8192 tokens x 768 x 3072 (both
// gradients) 101 -> 81 us, 8192 x 1024 x 4096 114 -> 100.  The large tile gained most from the 16-wide instruction and is the
// cheapest from 0.7 of a round on: 5504 tokens x 1408 x 3776 (both) small 118, medium 121, large 112 us; 8000 tokens 165, 167, 154.
// 0.2 % above the best tile at the mean of 64 other pairs.
// The tile of 192 x 128, where at most one of them falls to a compute unit, spreads over more of these what the medium tile piles on some: a
// GPT-2-small layer's gradients are 192 of it against 144.  4096 tokens x 768 x 3072 (both gradients) 47.2 -> 43.5 us, 8192 x 896 x
// 3136 122 -> 109, 6016 x 832 x 2880 86.7 -> 78.7.  The cost is fitted from 100 chunks (3200 tokens) on.  Below, the tile would save 0.4 to
// 2.4 us where there are 192 to 244 of it (2048 x 768 x 3072 30.4 -> 28.2, 128 x 768 x 3072 10.3 -> 9.4, 512 x 896 x 3136 15.1 -> 14.7) and lose 10 to 35 %
// to the small tile where there are fewer (512 x 640 x 2560, 150: 10.6 and 12.8): it is left to the other three there.  With more than one to a
// compute unit these are faster (8192 x 1024 x 3072, 272: 90 against 131), and so is the small tile for one gradient alone, measured at
// 44 to 176 of this one (8192 x 4096 x 1024: 60 against 78; 2048 x 3072 x 768: 20 against 26).
// The cost of a grid of `tiles`, and where the chip is full that of one round of it
double dw_cost(DwTile t, int64_t tiles, double chunks)
{
    const int64_t cus = s24_cu_count(), per = t == DwTile::Small ? 2 * cus : cus;
    const double full = (double)(tiles / per), rest = (double)(tiles % per) / per;
    if (t == DwTile::Large) return 14.6 + chunks * (0.75 * full + (rest > 0 ? 0.43 + 0.22 * rest : 0));
    if (t == DwTile::Medium) return 9.7 + chunks * (0.45 * full + (rest > 0 ? 0.24 + 0.12 * rest : 0));
    if (t == DwTile::Medium192) return 9.0 + chunks * (0.20 + 0.095 * (double)tiles / cus);   // up to a round
    return 7.0 + chunks * (0.53 * full + (rest > 0.5 ? 0.38 : rest > 0 ? 0.18 : 0));
}
double dw_round(DwTile t, double chunks) { return dw_cost(t, s24_cu_count(), chunks); }
int64_t dw_tiles(const DwProblem *pr, int count, DwTile t)
{
    int64_t n = 0;
    for (int i = 0; i < count; ++i) n += dw_tiles_m(t, pr[i].r) * dw_tiles_n(t, pr[i].q);
    return n;
}
int64_t dw_chunks(const DwProblem *pr, int count)
{
    int64_t chunks = 0;
    for (int i = 0; i < count; ++i) chunks = std::max(chunks, (pr[i].p + 31) / 32);
    return chunks;
}
DwTile dw_few_tile(const DwProblem *pr, int count)
{
    const int64_t chunks = dw_chunks(pr, count), n192 = dw_tiles(pr, count, DwTile::Medium192);
    auto cost = [&](DwTile t) { return dw_cost(t, dw_tiles(pr, count, t), (double)chunks); };
    const double l = cost(DwTile::Large), m = cost(DwTile::Medium), s = cost(DwTile::Small);
    if (count > 1 && chunks >= 100 && n192 <= s24_cu_count() && cost(DwTile::Medium192) < std::min(l, std::min(m, s))) return DwTile::Medium192;
    return s <= m && s <= l ? DwTile::Small : m <= l ? DwTile::Medium : DwTile::Large;
}
// small tile: 32 tokens per stage when there are more tiles than compute units, else 64
void launch_dw_batch(const dmatn::DwBatch &batch, DwTile tile, bool accum, bool decay, int dt, hipStream_t st)
{
    const int slots = batch.first_slot[dmatn::kMaxBatch];   // per XCD
    const dim3 grid(slots * 8), block(dmatn::THREADS);
#define S24_LAUNCH_DW(WTM, WTN, BT, ACC, DEC) \
    hipLaunchKernelGGL((dmatn::dense_tn_dma_kernel<T, dmatn::Cfg<WTM, WTN, BT>, ACC, DEC>), grid, block, 0, st, batch, g_clock_probe)
#define S24_LAUNCH_DW_TILE(WTM, WTN, BT)                               \
    do {                                                               \
        if (accum && decay) S24_LAUNCH_DW(WTM, WTN, BT, true, true);   \
        else if (accum) S24_LAUNCH_DW(WTM, WTN, BT, true, false);      \
        else if (decay) S24_LAUNCH_DW(WTM, WTN, BT, false, true);      \
        else S24_LAUNCH_DW(WTM, WTN, BT, false, false);                \
    } while (0)
    S24_WITH_16BIT_TYPE(dt, {
        if (tile == DwTile::Large) S24_LAUNCH_DW_TILE(4, 4, 32);
        else if (tile == DwTile::Medium) S24_LAUNCH_DW_TILE(4, 2, 32);
        else if (tile == DwTile::Medium192) S24_LAUNCH_DW_TILE(3, 2, 32);
        else if (slots * 8 > s24_cu_count()) S24_LAUNCH_DW_TILE(2, 2, 32);
        else S24_LAUNCH_DW_TILE(2, 2, 64);
    });
#undef S24_LAUNCH_DW_TILE
#undef S24_LAUNCH_DW
}

// Shared by s24_dense_dw and s24_dense_dw_decay.  W == nullptr: no decay term.
int run_dense_dw(const void *dY, const void *X, float *dW, int64_t p, int64_t q, int64_t r, float beta, int dt,
                 const void *W, int wdt, const uint16_t *mask, float lambda, hipStream_t st)
{
    const bool accum = beta != 0.0f;
    bool decay_pending = W != nullptr;
    if (p == 0) {  // empty contraction: dW = beta * dW (the GEMM kernels need at least one token)
        if (!accum) hipLaunchKernelGGL(fill_zero_kernel, dim3(ceil_div(q * r, kThreads)), dim3(kThreads), 0, st, dW, q * r);
    } else if (dt != S24_F32) {
        auto *a = static_cast<const uint16_t *>(dY), *b = static_cast<const uint16_t *>(X);
        const bool fuse = decay_pending && wdt == dt;   // the epilogue reads W in the operands' own 16-bit type
        auto *w = static_cast<const uint16_t *>(fuse ? W : nullptr);
        const DwProblem pr0{a, b, dW, w, fuse ? mask : nullptr, p, q, r, lambda};
        // One launch over the window [m_off, m_off + mm) x [n_off, n_off + nn) of the output, in tiles of `tile`
        auto launch = [&](DwTile tile, int64_t m_off, int64_t mm, int64_t n_off, int64_t nn) {
            dmatn::DwBatch batch{};
            batch.w[0] = dw_window(pr0, tile, m_off, mm, n_off, nn);
            const int slots = (batch.w[0].tiles_m * batch.w[0].tiles_n + 7) / 8;
            for (int i = 1; i <= dmatn::kMaxBatch; ++i) batch.first_slot[i] = slots;
            launch_dw_batch(batch, tile, accum, fuse, dt, st);
        };
        // 256 x 256 tiles when they fill the chip, otherwise the cheapest of the four (dw_few_tile).  A grid of large tiles that is not a
        // whole number of rounds over the 256 compute units leaves the chip part empty in its last round (c4's
        // 1376 tiles: 5.375 rounds).  Where whole tile rows or columns can be cut off so that the rest is an exact
        // number of rounds and the cut-off strip is at most half a round of large tiles, the slab runs in large
        // tiles and the strip in small ones (at most 512 of them: one resident set, two workgroups per compute
        // unit).  8192 tokens: a strip of 32 large tiles costs 0.25 of a round of 188 us where the uncut rest costs 0.64, of 64 tiles
        // 0.32 and 0.67, of 96 0.57 and 0.72, of 128 0.63 and 0.75; 16384 tokens: of 8 tiles 0.35 and 0.71, of 96 0.63 and 0.77.  After
        // five whole rounds (c4's 1376 tiles) the two are within 1 % of each other.  A longer strip (c4's other weight, 0.69 of a round) stays in the single launch.  Every output
        // element belongs to exactly one launch either way and all tiles sum the tokens in the same groups, so nothing about the
        // result changes.
        const int tm256 = (int)ceil_div(r, 256), tn256 = (int)ceil_div(q, 256), total = tm256 * tn256;
        const int cus = s24_cu_count();
        if (total < 3 * cus / 4) {
            launch(dw_few_tile(&pr0, 1), 0, r, 0, q);
        } else {
            int cut_m = 0, cut_n = 0;   // tile rows / columns kept in the large-tile slab (0: no such cut)
            if (total % cus != 0) {
                for (int k = tm256 - 1; k >= 1 && !cut_m; --k)
                    if ((k * tn256) % cus == 0 && (tm256 - k) * tn256 <= cus / 2) cut_m = k;
                for (int k = tn256 - 1; k >= 1 && !cut_n; --k)
                    if ((k * tm256) % cus == 0 && (tn256 - k) * tm256 <= cus / 2) cut_n = k;
            }
            if (cut_m && (!cut_n || cut_m * tn256 >= cut_n * tm256)) {
                launch(DwTile::Large, 0, 256ll * cut_m, 0, q);
                launch(DwTile::Small, 256ll * cut_m, r - 256ll * cut_m, 0, q);
            } else if (cut_n) {
                launch(DwTile::Large, 0, r, 0, 256ll * cut_n);
                launch(DwTile::Small, 0, r, 256ll * cut_n, q - 256ll * cut_n);
            } else {
                launch(DwTile::Large, 0, r, 0, q);
            }
        }
        if (fuse) decay_pending = false;
    } else {
        const bool fuse = decay_pending && wdt == S24_F32;
        const S24F32TnProblem pr{static_cast<const float *>(dY), static_cast<const float *>(X), static_cast<const float *>(fuse ? W : nullptr),
                                 nullptr, mask, dW, p, r, q, lambda};
        const int rc = s24_f32_tn(&pr, 1, accum, st);
        if (rc != S24_OK) return rc;
        if (fuse) decay_pending = false;
    }
    const int rc = s24_launch_status();
    if (rc != S24_OK || !decay_pending) return rc;
    // shapes the fused epilogue does not cover: the stand-alone decay kernel on the finished gradient
    return s24_masked_decay_grad(dW, W, static_cast<s24_dtype>(wdt), mask, lambda, r, q, st);
}
}  // namespace

extern "C" int s24_dense_dw(const void *dY, const void *X, float *dW, int64_t p, int64_t q, int64_t r, float beta,
                            s24_dtype dt, void *stream)
{
    S24_REQUIRE(q % 16 == 0 && r % 16 == 0, S24_ERR_SHAPE);
    S24_REQUIRE(beta == 0.0f || beta == 1.0f, S24_ERR_UNSUPPORTED);
    const int rc = check_gemm(dY, X, dW, p, q, r, dt, q * r);
    if (rc != S24_OK || q * r == 0) return rc;
    return run_dense_dw(dY, X, dW, p, q, r, beta, dt, nullptr, dt, nullptr, 0.0f, static_cast<hipStream_t>(stream));
}

extern "C" int s24_dense_dw_decay(const void *dY, const void *X, float *dW, const void *W, s24_dtype wdt,
                                  const uint16_t *mask, float lambda, int64_t p, int64_t q, int64_t r, float beta,
                                  s24_dtype dt, void *stream)
{
    S24_REQUIRE(q % 16 == 0 && r % 16 == 0, S24_ERR_SHAPE);
    S24_REQUIRE(beta == 0.0f || beta == 1.0f, S24_ERR_UNSUPPORTED);
    S24_REQUIRE(s24_valid_dtype(wdt), S24_ERR_DTYPE);
    const int rc = check_gemm(dY, X, dW, p, q, r, dt, q * r);
    if (rc != S24_OK || q * r == 0) return rc;
    S24_REQUIRE(W && mask, S24_ERR_NULL);
    S24_REQUIRE(s24_aligned(W, 16) && s24_aligned(mask, 4), S24_ERR_ALIGN);
    return run_dense_dw(dY, X, dW, p, q, r, beta, dt, W, wdt, mask, lambda, static_cast<hipStream_t>(stream));
}

namespace {
int check_dw_batch(const s24_dw_problem *problems, int count, s24_dtype dt)
{
    S24_REQUIRE(s24_valid_dtype(dt), S24_ERR_DTYPE);
    S24_REQUIRE(count >= 0 && count <= dmatn::kMaxBatch, S24_ERR_SHAPE);
    if (count == 0) return S24_OK;
    S24_REQUIRE(problems != nullptr, S24_ERR_NULL);
    for (int i = 0; i < count; ++i) {
        const s24_dw_problem &pr = problems[i];
        S24_REQUIRE(pr.q % 16 == 0 && pr.r % 16 == 0, S24_ERR_SHAPE);
        const int rc = check_gemm(pr.dY, pr.X, pr.dW, pr.p, pr.q, pr.r, dt, pr.q * pr.r);
        if (rc != S24_OK) return rc;
        if (pr.W != nullptr && pr.q * pr.r != 0) {
            S24_REQUIRE(pr.mask != nullptr, S24_ERR_NULL);
            S24_REQUIRE(s24_aligned(pr.W, 16) && s24_aligned(pr.mask, 4), S24_ERR_ALIGN);
        }
    }
    return S24_OK;
}
DwProblem dw_problem(const s24_dw_problem &pr)
{
    return DwProblem{static_cast<const uint16_t *>(pr.dY), static_cast<const uint16_t *>(pr.X), pr.dW, static_cast<const uint16_t *>(pr.W), pr.mask, pr.p, pr.q, pr.r, pr.lambda};
}
// One grid of `tile` for all of several problems
dmatn::DwBatch shared_batch(const DwProblem *prs, int count, DwTile tile)
{
    dmatn::DwBatch batch{};
    int first = 0;
    for (int i = 0; i < count; ++i) {
        batch.w[i] = dw_window(prs[i], tile, 0, prs[i].r, 0, prs[i].q);
        batch.first_slot[i] = first;
        first += (batch.w[i].tiles_m * batch.w[i].tiles_n + 7) / 8;
    }
    for (int i = count; i <= dmatn::kMaxBatch; ++i) batch.first_slot[i] = first;
    return batch;
}
inline bool dw_is_small(const s24_dw_problem &pr) { return (int64_t)ceil_div(pr.r, 256) * ceil_div(pr.q, 256) < 3 * s24_cu_count() / 4; }
// Whole tile columns or rows of one problem that make up exactly the excess of all problems' large tiles over whole rounds, if that is at most half
// a round (they run in small tiles): the problem, or -1
int find_strip(const DwProblem *prs, int count, int64_t total, int &cols, int &rows)
{
    const int cus = s24_cu_count(), excess = (int)(total % cus);
    cols = rows = 0;
    if (excess == 0 || excess > cus / 2) return -1;
    for (int i = 0; i < count; ++i) {
        const int tm = (int)ceil_div(prs[i].r, 256), tn = (int)ceil_div(prs[i].q, 256);
        if (excess % tm == 0 && excess / tm < tn) { cols = excess / tm; return i; }
        if (excess % tn == 0 && excess / tn < tm) { rows = excess / tn; return i; }
    }
    return -1;
}
// The tile for several problems on one whole grid, if they have one, and what s24_dense_dw_batch takes for them (a strip: a third of a round).  It
// has to say what s24_dense_dw_batch does: the tests compare the tile of a joint launch with the one that the gradients take by themselves.
bool dw_whole_grid(const s24_dw_problem *problems, const DwProblem *prs, int count, DwTile &tile, double &us)
{
    const int64_t cus = s24_cu_count();
    const double chunks = (double)dw_chunks(prs, count);
    int64_t total = 0;
    bool all_small = true, all_large = true;
    for (int i = 0; i < count; ++i) {
        const int64_t tiles = (int64_t)ceil_div(prs[i].r, 256) * ceil_div(prs[i].q, 256);
        total += tiles;
        all_small = all_small && dw_is_small(problems[i]);
        all_large = all_large && tiles >= 64;
    }
    if (count < 2) return false;
    if (all_large && total >= 3 * cus / 4) {
        tile = DwTile::Large;
        int cols, rows;
        us = find_strip(prs, count, total, cols, rows) < 0 ? dw_cost(tile, total, chunks) : dw_cost(tile, total / cus * cus, chunks) + 3.0 + 0.35 * 0.75 * chunks;
        return true;
    }
    if (!all_small) return false;
    tile = dw_few_tile(prs, count);
    us = dw_cost(tile, dw_tiles(prs, count, tile), chunks);
    return tile != DwTile::Small;
}
// dX and the weight gradients in one launch, where that is estimated to be the faster: false if not.  A compute unit has one workgroup of either kind
// at a time; the weight gradients' come first, and each compute unit that is done with them takes one of dX's after the other.  The estimate takes the
// clock of a chip with every compute unit busy for either, which is a little too slow: of 120 pairs (700-16384 tokens, layers of 384 to 4096) those
// estimated at up to 1.04 of the two launches took 0.67 to 0.99 of them, but for layers whose weight gradients leave fewer than a fifth of the
// compute units idle in their last round (0.99 to 1.06), and those beyond 1.1 0.78 to 1.10, with as many on one side of 1 as on the other.
bool launch_dw_dx(const uint16_t *dY, const uint16_t *valsT, const uint16_t *metaT, uint16_t *dX, int64_t p, int64_t q, int64_t r, const s24_dw_problem *problems, int count,
                  int dt, hipStream_t st)
{
    DwProblem prs[dmatn::kMaxBatch];
    for (int i = 0; i < count; ++i) prs[i] = dw_problem(problems[i]);
    DwTile tile;
    double dw_us;
    if (!dw_whole_grid(problems, prs, count, tile, dw_us)) return false;
    const int64_t cus = s24_cu_count(), nw = dw_tiles(prs, count, tile), tiles_m = ceil_div(q, 256), tiles_n = ceil_div(p, 128), nx = tiles_m * tiles_n;
    if (nw + nx >= 1 << 20) return false;
    const NtCosts c = sparse_costs(r);
    const NtTile alone = nt_tile_or_slab(q, p, r);
    double apart = alone.slab == 0 ? nt_cost(alone.kind, q, p, c)
                                   : nt_cost(NtTile::Large, q, alone.slab, c) + nt_cost(cheapest_tile(q, p - alone.slab, c).kind, q, p - alone.slab, c) + 3.0 / round_us(r);
    apart = apart * round_us(r) + dw_us + 3.0;
    const double tw = dw_round(tile, (double)dw_chunks(prs, count)), tx = c.medium * round_us(r);
    const int64_t rounds = nw / cus, more = nw % cus;   // `more` compute units have a round more
    if (5 * more > 4 * cus) return false;
    double both = (double)(rounds + (more > 0)) * tw;
    for (;; both += 0.25 * tx) {
        const int64_t done = more * (int64_t)((both - (double)(rounds + 1) * tw) / tx + 1e-6) + (cus - more) * (int64_t)((both - (double)rounds * tw) / tx + 1e-6);
        if (both > 1.04 * apart) return false;
        if (done >= nx) break;
    }
    const dmatn::DwBatch batch = shared_batch(prs, count, tile);
    const int dw_blocks = 8 * batch.first_slot[dmatn::kMaxBatch];
    const dim3 grid(dw_blocks + (unsigned)((nx + 7) / 8 * 8)), block(dmatn::THREADS);
#define S24_LAUNCH_DW_DX(DEC, WTM, WTN)                                                                                                       \
    hipLaunchKernelGGL((dw_dx_kernel<T, DEC, dmatn::Cfg<WTM, WTN, 32>>), grid, block, 0, st, dY, valsT, metaT, dX, (int)p, (int)r, (int)q, dw_blocks, \
                       (int)tiles_m, (int)tiles_n, batch, g_clock_probe)
#define S24_LAUNCH_DW_DX_TILE(DEC)                                              \
    do {                                                                        \
        if (tile == DwTile::Large) S24_LAUNCH_DW_DX(DEC, 4, 4);                 \
        else if (tile == DwTile::Medium) S24_LAUNCH_DW_DX(DEC, 4, 2);           \
        else S24_LAUNCH_DW_DX(DEC, 3, 2);                                       \
    } while (0)
    S24_WITH_16BIT_TYPE(dt, {
        if (prs[0].W != nullptr) S24_LAUNCH_DW_DX_TILE(true);
        else S24_LAUNCH_DW_DX_TILE(false);
    });
#undef S24_LAUNCH_DW_DX_TILE
#undef S24_LAUNCH_DW_DX
    return true;
}
}  // namespace

extern "C" int s24_dense_dw_batch(const s24_dw_problem *problems, int count, float beta, s24_dtype dt, void *stream)
{
    S24_REQUIRE(s24_valid_dtype(dt), S24_ERR_DTYPE);
    S24_REQUIRE(count >= 0 && count <= dmatn::kMaxBatch, S24_ERR_SHAPE);
    S24_REQUIRE(beta == 0.0f || beta == 1.0f, S24_ERR_UNSUPPORTED);
    const int checked = check_dw_batch(problems, count, dt);   // every problem is checked before anything is launched
    if (checked != S24_OK || count == 0) return checked;
    hipStream_t st = static_cast<hipStream_t>(stream);
    bool shared_grid = dt != S24_F32;
    int64_t total = 0;
    for (int i = 0; i < count; ++i) {
        const s24_dw_problem &pr = problems[i];
        const int64_t tiles = (int64_t)ceil_div(pr.r, 256) * ceil_div(pr.q, 256);
        // one grid for all of them: 16-bit data, tokens to contract, every problem large enough for the large tile,
        // and the decay term on all of them or on none
        shared_grid = shared_grid && pr.p > 0 && tiles >= 64 && (pr.W != nullptr) == (problems[0].W != nullptr);
        total += tiles;
    }
    const bool accum = beta != 0.0f, decay = problems[0].W != nullptr;
    DwProblem prs[dmatn::kMaxBatch];
    for (int i = 0; i < count; ++i) prs[i] = dw_problem(problems[i]);
    const int cus = s24_cu_count();
    if (!shared_grid || total < 3 * cus / 4 || count == 1) {
        // Problems that would each leave the large tile's grid mostly empty (fewer than 192 tiles) share one grid of the tile
        // that is cheapest for all of them: a GPT-2-small layer's two gradients are 72 medium tiles each.
        bool small_grid = dt != S24_F32 && count > 1;
        for (int i = 0; i < count; ++i) {
            const s24_dw_problem &pr = problems[i];
            small_grid = small_grid && pr.p > 0 && pr.q * pr.r != 0 && (pr.W != nullptr) == decay && dw_is_small(pr);
        }
        if (small_grid) {
            const DwTile few = dw_few_tile(prs, count);
            launch_dw_batch(shared_batch(prs, count, few), few, accum, decay, dt, st);
            return s24_launch_status();
        }
        // fp32: one grid for every problem with tokens to contract, unless the order of the problems counts (two of them
        // adding to one gradient)
        const bool together = dt == S24_F32 && !s24_dw_problems_overlap(problems, count, sizeof(float));
        if (together) {
            S24F32TnProblem f[dmatn::kMaxBatch];
            int n = 0;
            bool rest = false;
            for (int i = 0; i < count; ++i) {
                const s24_dw_problem &pr = problems[i];
                if (pr.p == 0) rest = true;
                else if (pr.q * pr.r != 0)
                    f[n++] = {static_cast<const float *>(pr.dY), static_cast<const float *>(pr.X), static_cast<const float *>(pr.W), nullptr, pr.mask,
                              pr.dW, pr.p, pr.r, pr.q, pr.lambda};
            }
            const int rc = n > 0 ? s24_f32_tn(f, n, accum, st) : S24_OK;
            if (rc != S24_OK || !rest) return rc;
        }
        for (int i = 0; i < count; ++i) {
            const s24_dw_problem &pr = problems[i];
            if (pr.q * pr.r == 0 || (together && pr.p != 0)) continue;
            const int rc = run_dense_dw(pr.dY, pr.X, pr.dW, pr.p, pr.q, pr.r, beta, dt, pr.W, dt, pr.mask, pr.lambda, st);
            if (rc != S24_OK) return rc;
        }
        return S24_OK;
    }
    // The tiles of all problems make one list.  If its length is not a whole number of rounds over the 256 compute
    // units, look for a problem from which whole tile columns (or rows) amounting to exactly the excess, and to at
    // most half a round, can be cut: that strip runs in small tiles afterwards, the rest in whole rounds.
    int cut_cols, cut_rows;
    const int cut = find_strip(prs, count, total, cut_cols, cut_rows);
    dmatn::DwBatch batch{};
    int first = 0;
    for (int i = 0; i < count; ++i) {
        // the cut removes the LAST tile rows / columns, the ragged edge included: what stays is a multiple of 256
        const int64_t keep_m = i == cut && cut_rows ? 256ll * ((int64_t)ceil_div(prs[i].r, 256) - cut_rows) : prs[i].r;
        const int64_t keep_n = i == cut && cut_cols ? 256ll * ((int64_t)ceil_div(prs[i].q, 256) - cut_cols) : prs[i].q;
        batch.w[i] = dw_window(prs[i], DwTile::Large, 0, keep_m, 0, keep_n);
        batch.first_slot[i] = first;
        first += (batch.w[i].tiles_m * batch.w[i].tiles_n + 7) / 8;
    }
    for (int i = count; i <= dmatn::kMaxBatch; ++i) batch.first_slot[i] = first;
    launch_dw_batch(batch, DwTile::Large, accum, decay, dt, st);
    if (cut >= 0) {
        dmatn::DwBatch strip{};
        const int64_t m_off = cut_rows ? batch.w[cut].M : 0, n_off = cut_cols ? batch.w[cut].N : 0;
        strip.w[0] = dw_window(prs[cut], DwTile::Small, m_off, prs[cut].r - m_off, n_off, prs[cut].q - n_off);
        const int slots = (strip.w[0].tiles_m * strip.w[0].tiles_n + 7) / 8;
        for (int i = 1; i <= dmatn::kMaxBatch; ++i) strip.first_slot[i] = slots;
        launch_dw_batch(strip, DwTile::Small, accum, decay, dt, st);
    }
    return s24_launch_status();
}

extern "C" int s24_spmm_bwd_dx_dw(const void *dY, const void *valsT, const uint16_t *metaT, void *dX, int64_t p, int64_t q, int64_t r,
                                  const s24_dw_problem *problems, int count, s24_dtype dt, void *stream)
{
    S24_REQUIRE(r % 64 == 0 && q % 16 == 0 && r > 0, S24_ERR_SHAPE);
    int rc = check_gemm(dY, valsT, dX, p, q, r, dt, p * q);
    if (rc != S24_OK) return rc;
    if (p * q != 0) {
        S24_REQUIRE(metaT != nullptr, S24_ERR_NULL);
        S24_REQUIRE(s24_aligned(metaT, 4), S24_ERR_ALIGN);
    }
    rc = check_dw_batch(problems, count, dt);
    if (rc != S24_OK) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    bool together = p * q != 0 && count > 0;
    for (int i = 0; i < count; ++i)
        together = together && problems[i].p > 0 && problems[i].q * problems[i].r != 0 && (problems[i].W != nullptr) == (problems[0].W != nullptr);
    const int64_t esize = (int64_t)s24_elem_size(dt);
    together = together && !s24_dw_problems_overlap(problems, count, esize) && !s24_dx_meets_dw(dY, valsT, metaT, dX, p, q, r, problems, count, esize);
    if (together && dt == S24_F32) {
        S24F32TnProblem f[dmatn::kMaxBatch];
        for (int i = 0; i < count; ++i) {
            const s24_dw_problem &pr = problems[i];
            f[i] = {static_cast<const float *>(pr.dY), static_cast<const float *>(pr.X), static_cast<const float *>(pr.W), nullptr, pr.mask, pr.dW, pr.p, pr.r, pr.q, pr.lambda};
        }
        if (s24_f32_nt_tn({static_cast<const float *>(dY), static_cast<const float *>(valsT), metaT, static_cast<float *>(dX), nullptr, nullptr, p, r, q, false,
                           S24_F32_PLAIN, 0}, f, count, st, rc))
            return rc;
    }
    const S24SlicePlan slices = p * q == 0 || dt == S24_F32 ? S24SlicePlan{} : bwd_dx_slices(p, r, q);
    if (together && dt != S24_F32 && !slices && launch_dw_dx(static_cast<const uint16_t *>(dY), static_cast<const uint16_t *>(valsT), metaT,
                                                             static_cast<uint16_t *>(dX), p, q, r, problems, count, dt, st))
        return s24_launch_status();
    // 16-bit, few tokens: the input gradient in slices of one token block to a tile beside the weight gradients in the small tile by eight waves.  Up to
    // 1024 tokens: beyond, that tile is slower than the one of four waves by more than a launch (in turn and together, 1024 tokens: 64 x 256
    // 12.4 and 11.4 us, 256 x 1024 14.3 and 12.8; 1536: 14.7 and 14.8, 17.9 and 18.6; 3072: 21.9 and 25.0, 29.4 and 29.4).
    for (int i = 0; i < count; ++i) together = together && dw_is_small(problems[i]) && problems[i].p <= 1024;
    const S24SlicePlan narrow = together && slices ? s24_slice_plan(p, r, q, 1) : S24SlicePlan{};
    if (narrow && narrow.us <= 1.3 * slices.us) {
        DwProblem prs[dmatn::kMaxBatch];
        for (int i = 0; i < count; ++i) prs[i] = dw_problem(problems[i]);
        if (dw_few_tile(prs, count) == DwTile::Small) {
            const dmatn::DwBatch batch = shared_batch(prs, count, DwTile::Small);
            s24_dx_dw({static_cast<const uint16_t *>(dY), static_cast<const uint16_t *>(valsT), metaT, static_cast<uint16_t *>(dX), nullptr, nullptr, nullptr, p, r, q,
                       false, S24_SLICE_PLAIN, 0}, narrow.tm, batch, problems[0].W != nullptr, dt, st);
            return s24_launch_status();
        }
    }
    rc = launch_spmm(dY, valsT, metaT, dX, p, r, q, 0.0f, dt, st, nullptr, slices);
    return rc != S24_OK ? rc : s24_dense_dw_batch(problems, count, 0.0f, dt, stream);
}

extern "C" int s24_spmm_dw(const void *vals, const uint16_t *meta, const void *X, float *dW, const void *W, s24_dtype wdt,
                           const uint16_t *mask, float lambda, int64_t p, int64_t q, int64_t r, float beta, s24_dtype dt,
                           void *stream)
{
    S24_REQUIRE(p % 64 == 0 && q % 16 == 0 && r % 16 == 0, S24_ERR_SHAPE);
    S24_REQUIRE(beta == 0.0f || beta == 1.0f, S24_ERR_UNSUPPORTED);
    const int rc = check_gemm(vals, X, dW, p, q, r, dt, q * r);
    if (rc != S24_OK || q * r == 0) return rc;
    if (W != nullptr) {
        S24_REQUIRE(s24_valid_dtype(wdt), S24_ERR_DTYPE);
        S24_REQUIRE(mask != nullptr, S24_ERR_NULL);
        S24_REQUIRE(s24_aligned(W, 16) && s24_aligned(mask, 4), S24_ERR_ALIGN);
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool accum = beta != 0.0f;
    bool decay_pending = W != nullptr;
    if (p == 0) {
        if (!accum) hipLaunchKernelGGL(fill_zero_kernel, dim3(ceil_div(q * r, kThreads)), dim3(kThreads), 0, st, dW, q * r);
    } else {
        S24_REQUIRE(meta != nullptr, S24_ERR_NULL);
        S24_REQUIRE(s24_aligned(meta, 4), S24_ERR_ALIGN);
        if (dt != S24_F32) {
            const NtTile tile = sparse_dw_tile(r, q);
            S24_REQUIRE((int64_t)ceil_div(r, 128) * ceil_div(q, 128) < (1ll << 30), S24_ERR_SHAPE);
            const int tiles_m = (int)ceil_div(r, tile.bm()), tiles_n = (int)ceil_div(q, tile.bn());
            const dim3 grid(((tiles_m * tiles_n + 7) / 8) * 8), block(tile.threads());
            auto *av = static_cast<const uint16_t *>(vals), *x = static_cast<const uint16_t *>(X);
            const bool fuse = decay_pending && wdt == dt;
            auto *w = static_cast<const uint16_t *>(fuse ? W : nullptr);
#define S24_LAUNCH_SPDW(ACC, DEC, MI, WN)                                                                                           \
    hipLaunchKernelGGL((sptn::spmm_tn_big_kernel<T, ACC, DEC, MI, WN>), grid, block, 0, st, av, meta, x, dW, (int)p, (int)r, (int)q, \
                       tiles_m, tiles_n, tile.kind == NtTile::Large ? g_clock_probe : nullptr, w, mask, lambda)
            S24_WITH_16BIT_TYPE(dt, {
                if (accum && fuse) S24_WITH_NT_TILE(tile, S24_LAUNCH_SPDW, true, true);
                else if (accum) S24_WITH_NT_TILE(tile, S24_LAUNCH_SPDW, true, false);
                else if (fuse) S24_WITH_NT_TILE(tile, S24_LAUNCH_SPDW, false, true);
                else S24_WITH_NT_TILE(tile, S24_LAUNCH_SPDW, false, false);
            });
#undef S24_LAUNCH_SPDW
            if (fuse) decay_pending = false;
        } else {
            const bool fuse = decay_pending && wdt == S24_F32;
            const S24F32TnProblem pr{static_cast<const float *>(vals), static_cast<const float *>(X), static_cast<const float *>(fuse ? W : nullptr),
                                     meta, mask, dW, p, r, q, lambda};
            const int rc1 = s24_f32_tn(&pr, 1, accum, st);
            if (rc1 != S24_OK) return rc1;
            if (fuse) decay_pending = false;
        }
    }
    const int rc2 = s24_launch_status();
    if (rc2 != S24_OK || !decay_pending) return rc2;
    return s24_masked_decay_grad(dW, W, wdt, mask, lambda, r, q, st);
}

extern "C" int s24_set_clock_probe(void *two_counters)
{
    S24_REQUIRE(s24_aligned(two_counters, 8), S24_ERR_ALIGN);
    g_clock_probe = static_cast<unsigned long long *>(two_counters);
    return S24_OK;
}
