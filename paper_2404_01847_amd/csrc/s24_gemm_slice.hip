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
#include "s24_slice_tile.h"

namespace {

using s24_slice::KS;

// first: B, Av; second: Am, N, K; third: M, F, tiles of tokens, all tiles
struct SliceEnds { uint16_t *Out, *H; const uint16_t *Z, *bias; };
template <typename T, bool ACCUM, int EPI, int ACT, int TM, int TN, bool STREAM>
__global__ __launch_bounds__(64 * KS, TN == 4 ? 2 : 4) void spmm_slice_kernel(const s24_words first, const s24_words second, const s24_words third, const SliceEnds e)
{
    constexpr int STAGE = s24_slice::stage_bytes(TN);
    __shared__ __attribute__((aligned(16))) unsigned char s0[STAGE];
    __shared__ __attribute__((aligned(16))) unsigned char s1[STAGE];
    __shared__ __attribute__((aligned(16))) unsigned char s2[TN == 1 ? STAGE : 16];
    __shared__ __attribute__((aligned(16))) unsigned char s3[TN == 1 ? STAGE : 16];
    s24_slice::slice_tile<T, ACCUM, EPI, ACT, TM, TN, STREAM>((s24_lds::lds_byte *)s0, (s24_lds::lds_byte *)s1, (s24_lds::lds_byte *)s2, (s24_lds::lds_byte *)s3, (int)blockIdx.x,
                                                              s24_global<const uint16_t>(first.x), s24_global<const uint16_t>(first.y), s24_global<const uint16_t>(second.x),
                                                              s24_low(second.y), s24_high(second.y), s24_low(third.x), s24_high(third.x), s24_low(third.y), s24_high(third.y),
                                                              e.Out, e.H, e.Z, e.bias);
}

template <typename T, bool ACCUM, int EPI, int ACT, int TM, int TN>
void launch(const S24SliceNt &g, hipStream_t st)
{
    constexpr int FM = EPI == S24_SLICE_GLU ? 8 * TM : 16 * TM;
    const int64_t F = g.M / 2, feats = EPI == S24_SLICE_GLU ? F : g.M;
    const int tiles_m = (int)((feats + FM - 1) / FM), tiles_n = (int)((g.N + 16 * TN - 1) / (16 * TN)), tiles = tiles_m * tiles_n;
    const dim3 grid(((tiles + 7) / 8) * 8), block(64 * KS);
#define S24_LAUNCH_SLICE(STREAM)                                                                                                            \
    hipLaunchKernelGGL((spmm_slice_kernel<T, ACCUM, EPI, ACT, TM, TN, STREAM>), grid, block, 0, st, s24_pack(g.B, g.Av), s24_pack(g.Am, (int)g.N, (int)g.K), \
                       s24_pack((int)g.M, (int)F, tiles_n, tiles), (SliceEnds{g.Out, g.H, g.Z, g.bias}))
    // Weights that nobody else reads (one token tile) go past the caches from 48 MB on.  Smaller ones of a layer stay in the 256 MB Infinity Cache from
    // one pass to the next: one token through 2048 x 8192 (19 MB each), three layers in turn, 12.8 us past the caches and 11.1 through them;
    // 3584 x 9600 (39) 19.3 and 15.8.  Larger ones mostly do not (16 tokens, 4544 x 12288, 63 MB each, 30.9 and 32.1; one layer of 8192 x 28672
    // 136 and 150), and a first pass over them has to push others out: 3072 x 16384 (57) 40 and 47.  Both are equal at 54 MB.  The lowest tile
    // has too few bytes in flight for the longer way: one token, 101 MB of 22016 -> 4096 18.5 and 15.7, where they were pushed out 19.6 and 19.7.
    if constexpr (TN == 1 && TM > 1) {
        if (tiles_n == 1 && g.M * g.K / 8 * 9 >= 48ll << 20) {   // values and index words are 9/8 byte per place
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

}  // namespace

// Tile of a product by its cost in us: a launch, and per round of workgroups over the compute units a filling and draining and so
// much for each 64 of k (fitted to 380 products, 1-2048 tokens, K = 256-32000, 256-56000 features; half of them within 7 %).
// Two workgroups to a compute unit count as two rounds: they share its first-level cache, which is what bounds them.
S24SlicePlan s24_slice_plan(int64_t N, int64_t K, int64_t M, int max_tn)
{
    struct Tile { int tm, tn; double launch, round, chunk; };
    constexpr Tile tiles[5] = {{1, 1, 2.2, 0.25, 0.037}, {2, 1, 2.2, 0.25, 0.060}, {4, 1, 2.3, 0.25, 0.105}, {4, 2, 2.1, 0.48, 0.122}, {4, 4, 1.6, 1.2, 0.170}};
    const int64_t cus = s24_cu_count();
    S24SlicePlan best{};
    for (const Tile &t : tiles) {
        if (t.tn > max_tn || N <= 16 * (t.tn / 2)) continue;   // half of the tile or more would be empty
        const int64_t n = ((M + 16 * t.tm - 1) / (16 * t.tm)) * ((N + 16 * t.tn - 1) / (16 * t.tn)), rounds = (n + cus - 1) / cus;
        const double us = t.launch + (double)rounds * (t.round + t.chunk * (double)(K / 64));
        if (!best || us < best.us) best = {t.tm, t.tn, us};
    }
    return best;
}

int s24_slice_nt(const S24SliceNt &g, const S24SlicePlan &p, int dt, hipStream_t st)
{
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
