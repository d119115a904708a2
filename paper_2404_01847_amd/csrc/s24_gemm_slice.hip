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

// The arguments are one by one and in the order in which they are needed: see FLAGS in build.py.
template <typename T, bool ACCUM, int EPI, int ACT, int TM, int TN, bool STREAM>
__global__ __launch_bounds__(64 * KS, TN == 4 ? 2 : 4) void spmm_slice_kernel(const uint16_t *__restrict__ B, const uint16_t *__restrict__ Av,
                                                                             const uint16_t *__restrict__ Am, int N, int K, int M, int F, int tiles_n, int tiles,
                                                                             uint16_t *Out, uint16_t *H, const uint16_t *Z, const uint16_t *bias)
{
    constexpr int STAGE = s24_slice::stage_bytes(TN);
    __shared__ __attribute__((aligned(16))) unsigned char s0[STAGE];
    __shared__ __attribute__((aligned(16))) unsigned char s1[STAGE];
    __shared__ __attribute__((aligned(16))) unsigned char s2[TN == 1 ? STAGE : 16];
    __shared__ __attribute__((aligned(16))) unsigned char s3[TN == 1 ? STAGE : 16];
    s24_slice::slice_tile<T, ACCUM, EPI, ACT, TM, TN, STREAM>((s24_lds::lds_byte *)s0, (s24_lds::lds_byte *)s1, (s24_lds::lds_byte *)s2, (s24_lds::lds_byte *)s3, (int)blockIdx.x, B, Av, Am, N, K, M, F, tiles_n, tiles, Out, H, Z, bias);
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
Plan plan(int64_t N, int64_t K, int64_t M, int max_tn = 4)
{
    constexpr Plan tiles[5] = {{1, 1, 2.2, 0.25, 0.037, 0}, {2, 1, 2.2, 0.25, 0.060, 0}, {4, 1, 2.3, 0.25, 0.105, 0}, {4, 2, 2.1, 0.48, 0.122, 0}, {4, 4, 1.6, 1.2, 0.170, 0}};
    const int64_t cus = s24_cu_count();
    Plan best{};
    for (Plan t : tiles) {
        if (t.tn > max_tn || N <= 16 * (t.tn / 2)) continue;   // half of the tile or more would be empty
        const int64_t n = ((M + 16 * t.tm - 1) / (16 * t.tm)) * ((N + 16 * t.tn - 1) / (16 * t.tn)), rounds = (n + cus - 1) / cus;
        t.us = t.launch + (double)rounds * (t.round + t.chunk * (double)(K / 64));
        if (best.tm == 0 || t.us < best.us) best = t;
    }
    return best;
}

}  // namespace

double s24_slice_us(int64_t N, int64_t K, int64_t M) { return plan(N, K, M).us; }

bool s24_slice_narrow_tile(int64_t N, int64_t K, int64_t M, int &tm)
{
    const Plan p = plan(N, K, M, 1);
    tm = p.tm;
    return p.us <= 1.3 * plan(N, K, M).us;
}

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
