// Transposable 2:4 mask search and prune/compress (Sec. 5.1 and Sec. 5 item 1).
//
// One lane owns one aligned 4x4 block at a time.  A workgroup of 256 lanes
// takes a tile of 32 x 32 blocks (128 x 128 weights, four blocks per lane), or
// of 32 x 16 or 16 x 16 for matrices with few of them (launch_sized).  The compressed operands are stored chunk-major (64 of the
// contraction axis per chunk, all rows of a chunk together), so a tile covers
// one or two chunks of each orientation and the column-wise operand, after an
// LDS transpose, leaves in runs of 4 or 8 KB.
//
// Scoring.  A legal block is a choice of one of six column pairs per row
// whose columns each get picked twice.  Rows 0-1 and rows 2-3 are scored
// separately ("top" and "bottom" halves) and matched through the column-count
// vector of the top half, which leaves 19 classes:
//   6  where both top rows use the same pair (bottom rows both use its
//      complement): four column sums of the halves;
//   1  where the top rows use complementary pairs (so do the bottom rows):
//      one whole row plus the two largest per-column gains of the other row;
//   12 where the top rows share exactly one column x and miss one column w:
//      column sum x (top) + column sum w (bottom) + the better crossing of the
//      two remaining columns in each half, which only depends on that pair.
// That is about 100 additions and 45 maxima per block instead of 90 x 7
// additions, and yields the same maximum because every legal block falls in
// exactly one class and each class maximum is taken over exactly its blocks.
//
// Exactness and tie-break.  Scores are held in fp64.  Let 2^(E+1) bound the
// largest magnitude of the block and eps = 2^(E-47).  If every nonzero
// magnitude is a multiple of 2048*eps, all partial sums are integers times
// eps below 2^52*eps, hence exact.  Each cell (i,j) is first increased by
// beta_j * 6^(3-i) * eps with beta = (0,2,3,4): the total added to a pattern
// is below 2048*eps, cannot reorder different true scores, and orders equal
// scores exactly like the pattern ids (smaller id = larger bonus).  The bonus
// is read back from the low 11 bits of (best + 2^52*eps) and indexes a table
// that returns the block mask and id.  Blocks whose magnitudes span more
// binades than that window take a slow path that scores all 90 patterns in
// 320-bit fixed point.
#include <algorithm>
#include <cstddef>
#include <type_traits>

#include "s24_common.h"

namespace {

// Column pairs in row-string order ("0011" < "0101" < ... < "1100"): pair k
// keeps columns kC1[k] < kC2[k]; the complementary pair is 5 - k.
__host__ __device__ constexpr int pair_c1(int k) { return k == 0 ? 2 : (k <= 2 ? 1 : 0); }
__host__ __device__ constexpr int pair_c2(int k) { return (k == 0 || k == 1 || k == 3) ? 3 : ((k == 2 || k == 4) ? 2 : 1); }
__host__ __device__ constexpr unsigned pair_bits(int k) { return (1u << pair_c1(k)) | (1u << pair_c2(k)); }
__host__ __device__ constexpr int pair_of(int a, int b)
{
    const int lo = a < b ? a : b, hi = a < b ? b : a;
    for (int k = 0; k < 6; ++k)
        if (pair_c1(k) == lo && pair_c2(k) == hi) return k;
    return -1;
}

constexpr int kRowMult[4] = {216, 36, 6, 1};
constexpr int kColBonus[4] = {0, 2, 3, 4};
constexpr int kBonusBase = 2 * (216 + 36 + 6 + 1);  // every row contributes at least 2

// Pattern by bonus: entries past the largest legal index, 5*216 + 5*36 = 1260, stand for every illegal one (mask and id 0).
constexpr int kLutEntries = 1264;
struct MaskLut {
    uint16_t mask[kLutEntries];
    uint8_t id[kLutEntries];
};

// Index: sum_i 6^(3-i) * (5 - k_i) for row pair indices k_i.  Walking
// (k0,k1,k2,k3) in ascending order visits the legal blocks in id order.
constexpr MaskLut make_lut()
{
    MaskLut t{};
    int n = 0;
    for (int a = 0; a < 6; ++a)
        for (int b = 0; b < 6; ++b)
            for (int c = 0; c < 6; ++c)
                for (int d = 0; d < 6; ++d) {
                    const unsigned rows[4] = {pair_bits(a), pair_bits(b), pair_bits(c), pair_bits(d)};
                    bool ok = true;
                    for (int j = 0; j < 4; ++j) {
                        int s = 0;
                        for (int i = 0; i < 4; ++i) s += (rows[i] >> j) & 1u;
                        if (s != 2) ok = false;
                    }
                    if (!ok) continue;
                    const int x = 216 * (5 - a) + 36 * (5 - b) + 6 * (5 - c) + (5 - d);
                    t.mask[x] = (uint16_t)(rows[0] | rows[1] << 4 | rows[2] << 8 | rows[3] << 12);
                    t.id[x] = (uint8_t)n;
                    ++n;
                }
    return t;
}

struct PatList {
    uint16_t mask[S24_NUM_PATTERNS];
};
constexpr PatList make_patlist()
{
    PatList p{};
    const MaskLut t = make_lut();
    for (int x = 0; x < kLutEntries; ++x)
        if (t.mask[x] != 0) p.mask[t.id[x]] = t.mask[x];
    return p;
}
__device__ const PatList g_patterns = make_patlist();

// What the compressor needs for a bf16 block, precomputed per pattern id (48 bytes each).
// A selector is a v_perm_b32 byte selector that picks two of the four 16-bit values held in a
// register pair {hi : lo} (positions 2,3 : positions 0,1) and packs them into one dword.
struct CompressEntry {
    uint32_t rowsel[4];   // row i: its two kept columns out of {cols 2,3 : cols 0,1}
    uint32_t colsel[4];   // column j: its two kept rows out of {rows 2,3 : rows 0,1}
    uint32_t rowmeta_lo;  // metadata nibbles of rows 0 and 1 at bits 0 and 16
    uint32_t rowmeta_hi;  // rows 2 and 3
    uint32_t colmeta;     // nibbles of columns 0..3 at bits 0, 4, 8, 12
    uint32_t pad;
};
struct CompressLut {
    CompressEntry e[S24_NUM_PATTERNS];
};
constexpr uint32_t perm_selector(int p0, int p1)
{
    return (uint32_t)(2 * p0) | ((uint32_t)(2 * p0 + 1) << 8) | ((uint32_t)(2 * p1) << 16) | ((uint32_t)(2 * p1 + 1) << 24);
}
constexpr CompressLut make_compress_lut()
{
    CompressLut t{};
    const PatList pl = make_patlist();
    for (int id = 0; id < S24_NUM_PATTERNS; ++id) {
        const unsigned m = pl.mask[id];
        uint32_t rowmeta[4] = {0, 0, 0, 0};
        for (int i = 0; i < 4; ++i) {
            int kept[2] = {0, 0}, n = 0;
            for (int j = 0; j < 4; ++j)
                if ((m >> (4 * i + j)) & 1u) kept[n++] = j;
            t.e[id].rowsel[i] = perm_selector(kept[0], kept[1]);
            rowmeta[i] = (uint32_t)(kept[0] | (kept[1] << 2));
        }
        t.e[id].rowmeta_lo = rowmeta[0] | (rowmeta[1] << 16);
        t.e[id].rowmeta_hi = rowmeta[2] | (rowmeta[3] << 16);
        for (int j = 0; j < 4; ++j) {
            int kept[2] = {0, 0}, n = 0;
            for (int i = 0; i < 4; ++i)
                if ((m >> (4 * i + j)) & 1u) kept[n++] = i;
            t.e[id].colsel[j] = perm_selector(kept[0], kept[1]);
            t.e[id].colmeta |= (uint32_t)(kept[0] | (kept[1] << 2)) << (4 * j);
        }
    }
    return t;
}
// All tables in one piece, so that a workgroup stages what it needs with one or two 16-byte loads per lane (1296 two-byte and 1296
// one-byte entries one by one were twelve loads and as many LDS writes per lane, ahead of everything else).
struct alignas(16) MaskTables {
    MaskLut lut;
    CompressLut clut;
};
static_assert(sizeof(MaskLut) % 16 == 0 && offsetof(MaskLut, id) % 16 == 0 && sizeof(CompressLut) % 16 == 0, "whole vectors");
__device__ const MaskTables g_tables = {make_lut(), make_compress_lut()};

// Pattern id of a given block mask through the bonus-indexed table: row nibble -> pair index k
// (0 for anything illegal), then the same mixed-radix index the search produces.
__device__ __forceinline__ unsigned lut_index_of_mask(unsigned m)
{
    unsigned x = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const unsigned m4 = (m >> (4 * i)) & 0xFu;
        // k for m4 = 3,5,6 in the low word (4 bits each), for m4 = 9,10,12 in the high word
        const unsigned tbl = (m4 & 8u) ? 0x00000130u : 0x02405000u;
        const unsigned k = (tbl >> (4 * (m4 & 7u))) & 7u;
        x = x * 6u + (5u - k);
    }
    return x;
}

// ---------------------------------------------------------------------------
// Slow path: exact scores of all 90 patterns in fixed point.  A magnitude given
// as an fp32 bit pattern is sig * 2^(shift-149) with sig < 2^24; a score is kept
// as ten limbs of 32 payload bits (units of 2^-149), enough for eight fp32
// magnitudes of any exponent.  First maximum in id order wins.
// ---------------------------------------------------------------------------
struct Mag16 { uint32_t v[16]; };
struct Fixed320 { uint32_t limb[10]; };

// Deliberately loop-based with locally indexed arrays: this path is rare, and
// keeping it small keeps the register budget of the common path.
__device__ __forceinline__ Fixed320 fixed_score(const Mag16 &mag, unsigned pattern)
{
    uint64_t acc[10];
#pragma unroll 1
    for (int L = 0; L < 10; ++L) acc[L] = 0;
#pragma unroll 1
    for (int t = 0; t < 16; ++t) {
        if (!((pattern >> t) & 1u)) continue;
        const uint32_t e = mag.v[t] >> 23, sig = (mag.v[t] & 0x7FFFFFu) | (e ? 0x800000u : 0u), shift = (e ? e : 1u) - 1u;
        const uint64_t v = (uint64_t)sig << (shift & 31u);
        acc[shift >> 5] += (uint32_t)v;
        acc[(shift >> 5) + 1] += (uint32_t)(v >> 32);   // the limb is at most 7, so the next one at most 8
    }
    Fixed320 s;
    uint64_t carry = 0;
#pragma unroll 1
    for (int L = 0; L < 10; ++L) {
        const uint64_t x = acc[L] + carry;
        s.limb[L] = (uint32_t)x;
        carry = x >> 32;
    }
    return s;
}
// a > b: 1, a < b: -1, equal: 0 (lexicographic from the top limb)
__device__ __forceinline__ int fixed_compare(const Fixed320 &a, const Fixed320 &b)
{
    int r = 0;
#pragma unroll 1
    for (int L = 9; L >= 0; --L)
        if (r == 0 && a.limb[L] != b.limb[L]) r = a.limb[L] > b.limb[L] ? 1 : -1;
    return r;
}
__device__ __noinline__ unsigned slow_best_pattern(Mag16 mag)
{
    Fixed320 best{};
    unsigned best_id = 0;
#pragma unroll 1
    for (unsigned k = 0; k < S24_NUM_PATTERNS; ++k) {
        const Fixed320 s = fixed_score(mag, g_patterns.mask[k]);
        if (fixed_compare(s, best) > 0) {
            best = s;
            best_id = k;
        }
    }
    return (unsigned)g_patterns.mask[best_id] | (best_id << 16);
}
// The same for one block scored by the whole wave (`mag` uniform, all 64 lanes active): one or two patterns per lane, then a
// butterfly.  A large fp32 matrix has a block or two this wide, and one lane's walk over 90 patterns held the launch up by 70 us.
__device__ __noinline__ unsigned wave_slow_best_pattern(Mag16 mag)
{
    unsigned id = threadIdx.x & 63;
    Fixed320 best = fixed_score(mag, g_patterns.mask[id]);
    if (id + 64u < S24_NUM_PATTERNS) {
        const Fixed320 s = fixed_score(mag, g_patterns.mask[id + 64u]);
        if (fixed_compare(s, best) > 0) {
            best = s;
            id += 64u;
        }
    }
#pragma unroll 1
    for (int off = 32; off > 0; off >>= 1) {
        Fixed320 o;
#pragma unroll 1
        for (int L = 0; L < 10; ++L) o.limb[L] = (uint32_t)__shfl_xor((int)best.limb[L], off, 64);
        const unsigned oid = (unsigned)__shfl_xor((int)id, off, 64);
        const int c = fixed_compare(o, best);
        if (c > 0 || (c == 0 && oid < id)) {
            best = o;
            id = oid;
        }
    }
    return (unsigned)g_patterns.mask[id] | (id << 16);
}

// ---------------------------------------------------------------------------
// Middle path: the 90 sums in fp64, first maximum in id order.  Exact as long as every sum of
// eight magnitudes fits fp64's 53 bits, i.e. the block spans at most 26 binades of fp32 data (42 of bf16
// data); used for blocks too wide for the fast path's window, which also has to hold the tie-break bits.
// Two forms.  16-bit weights hardly ever need it (their window is 26 to 29 binades): one lane walks the patterns in a call
// that costs the common path no registers.
// ---------------------------------------------------------------------------
__device__ __noinline__ unsigned mid_best_pattern(Mag16 mag)
{
    double a[16];
#pragma unroll
    for (int t = 0; t < 16; ++t) a[t] = (double)__uint_as_float(mag.v[t]);
    double best = -1.0;
    unsigned best_id = 0;
#pragma unroll 1
    for (unsigned k = 0; k < S24_NUM_PATTERNS; ++k) {
        const unsigned pm = g_patterns.mask[k];
        double sum = 0.0;
#pragma unroll
        for (int t = 0; t < 16; ++t) sum += ((pm >> t) & 1u) ? a[t] : 0.0;
        if (sum > best) {
            best = sum;
            best_id = k;
        }
    }
    return (unsigned)g_patterns.mask[best_id] | (best_id << 16);
}
// fp32 weights (window 13 binades) need it for one block in 300, so nearly every wave has some: there the wave scores one
// lane's block together, one or two patterns per lane, and agrees on the winner by a butterfly, about 150 instructions
// where the one-lane walk takes 4300 with the other 63 lanes waiting.  fp32 search, 1024 x 256: 71 -> 5 us; 22016 x 4096:
// 439 -> 78; search and compress 79 -> 8 and 633 -> 263.  (In the 16-bit kernels its registers cost 5 to 10 %.)
// All 64 lanes must be active; every lane returns the answer for the block of lane `src`.
struct WavePatterns {
    unsigned id, other_id, pm, pm2;   // of this lane
    __device__ __forceinline__ WavePatterns()
    {
        id = threadIdx.x & 63;
        other_id = min(id + 64u, (unsigned)S24_NUM_PATTERNS - 1u);   // lanes 26..63 repeat the last pattern
        pm = g_patterns.mask[id], pm2 = g_patterns.mask[other_id];
    }
    __device__ __forceinline__ void add(int t, double a, double &best, double &second) const
    {
        best += ((pm >> t) & 1u) ? a : 0.0;
        second += ((pm2 >> t) & 1u) ? a : 0.0;
    }
    __device__ __forceinline__ unsigned first_of_best(double best, double second) const
    {
        unsigned win = id;
        best = __builtin_fmax(best, -1.0);   // a pattern whose sum is NaN never wins, as in the one-lane walk
        if (second > best) {
            best = second;
            win = other_id;
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const double o = __shfl_xor(best, off, 64);
            const unsigned oid = (unsigned)__shfl_xor((int)win, off, 64);
            if (o > best || (o == best && oid < win)) {
                best = o;
                win = oid;
            }
        }
        return (unsigned)g_patterns.mask[win] | (win << 16);
    }
};
__device__ __forceinline__ unsigned wave_mid_best_pattern(const uint32_t (&mag)[16], int src)
{
    const WavePatterns patterns;
    double best = 0.0, second = 0.0;
#pragma unroll
    for (int t = 0; t < 16; ++t) patterns.add(t, (double)__uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)mag[t], src)), best, second);
    return patterns.first_of_best(best, second);
}

// The blocks of the lanes that set `mid` or `slow`, one after the other by the whole wave.  All 64 lanes must be active; a lane that
// set neither gets 0.
__device__ __forceinline__ unsigned wave_wide_blocks(const uint32_t (&mag)[16], bool mid, bool slow)
{
    unsigned rare = 0;
    for (unsigned long long todo = __ballot(mid); todo != 0; todo &= todo - 1) {
        const int src = (int)__builtin_ctzll(todo);
        const unsigned res = wave_mid_best_pattern(mag, src);
        if ((int)(threadIdx.x & 63) == src) rare = res;
    }
    for (unsigned long long todo = __ballot(slow); todo != 0; todo &= todo - 1) {
        const int src = (int)__builtin_ctzll(todo);
        Mag16 m16;
#pragma unroll
        for (int t = 0; t < 16; ++t) m16.v[t] = (uint32_t)__builtin_amdgcn_readlane((int)mag[t], src);
        const unsigned res = wave_slow_best_pattern(m16);
        if ((int)(threadIdx.x & 63) == src) rare = res;
    }
    return rare;
}

// Exponents of the block's largest and of its smallest magnitude other than zero (255 if there is none)
__device__ __forceinline__ void exponents(const uint32_t (&mag)[16], uint32_t &emax, uint32_t &emin)
{
    uint32_t mx = 0, mn = 0xFFFFFFFFu;
#pragma unroll
    for (int t = 0; t < 16; ++t) {
        mx = max(mx, mag[t]);
        mn = min(mn, mag[t] - 1u);  // zero wraps to the top and never wins
    }
    emax = max(mx >> 23, 1u);
    emin = (mn == 0xFFFFFFFFu) ? 255u : max(mn >> 23, 1u);
}

// ---------------------------------------------------------------------------
// Fast path.  mag[4*i+j] = |w_ij| as fp32 bit patterns.  Returns mask | id<<16.
// WINDOW = binades below the block maximum within which every element is a
// multiple of 2048*eps (29 for bf16 data, 13 for fp32 data).  What becomes of wider blocks: each lane walks through its own; the
// wave takes them together (all 64 lanes must call); or the caller has their answer, in `given`.
// ---------------------------------------------------------------------------
enum class Wide { Lane, Wave, Given };
template <int WINDOW, int WIDE, Wide HOW>
__device__ __forceinline__ unsigned best_pattern(const uint32_t (&mag)[16], const uint16_t *lut_mask, const uint8_t *lut_id, unsigned given = 0)
{
    uint32_t emax, emin;
    exponents(mag, emax, emin);
    const bool wide = emin + WINDOW < emax;
    if (HOW == Wide::Given && wide) return given;
    unsigned rare = 0;
    if constexpr (HOW == Wide::Wave) {
        rare = wave_wide_blocks(mag, wide && emin + WIDE >= emax, emin + WIDE < emax);
    } else if (HOW == Wide::Lane && wide) {
        Mag16 m16;
#pragma unroll
        for (int t = 0; t < 16; ++t) m16.v[t] = mag[t];
        return (emin + WIDE >= emax) ? mid_best_pattern(m16) : slow_best_pattern(m16);
    }

    const double eps = __hiloint2double((int)((emax + 849u) << 20), 0);       // 2^(E-47), E = emax-127
    const double big = __hiloint2double((int)((emax + 849u + 52u) << 20), 0);  // 2^52 * eps
    double a[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const double v = (double)__uint_as_float(mag[4 * i + j]);
            a[i][j] = (j == 0) ? v : __builtin_fma((double)(kColBonus[j] * kRowMult[i]), eps, v);
        }
    // column sums of the top (rows 0,1) and bottom (rows 2,3) halves
    double dt[4], db[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        dt[j] = a[0][j] + a[1][j];
        db[j] = a[2][j] + a[3][j];
    }
    // (i) both top rows keep the pair {c1,c2}, both bottom rows its complement
    double best = 0.0;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const double tot = (dt[pair_c1(k)] + dt[pair_c2(k)]) + (db[pair_c1(5 - k)] + db[pair_c2(5 - k)]);
        best = (k == 0) ? tot : __builtin_fmax(best, tot);
    }
    // (ii) complementary pairs in each half: all of row 1 plus the two largest gains of swapping a
    // column to row 0 (and the same for rows 3 and 2)
    {
        auto half = [](const double (&r0)[4], const double (&r1)[4]) {
            const double d0 = r0[0] - r1[0], d1 = r0[1] - r1[1], d2 = r0[2] - r1[2], d3 = r0[3] - r1[3];
            const double m1 = __builtin_fmax(d0, d1), n1 = __builtin_fmin(d0, d1);
            const double m2 = __builtin_fmax(d2, d3), n2 = __builtin_fmin(d2, d3);
            const double hi = __builtin_fmax(m1, m2), lo = __builtin_fmin(m1, m2);
            const double second = __builtin_fmax(lo, __builtin_fmax(n1, n2));
            return ((r1[0] + r1[1]) + (r1[2] + r1[3])) + (hi + second);
        };
        best = __builtin_fmax(best, half(a[0], a[1]) + half(a[2], a[3]));
    }
    // (iii) top rows share column x and keep one each of {y,z}; bottom rows share w and keep the
    // other of {y,z}: dt[x] + db[w] + best crossing of {y,z} in the top + in the bottom
    double cross[6];   // indexed by the pair {y,z}
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const int y = pair_c1(k), z = pair_c2(k);
        cross[k] = __builtin_fmax(a[0][y] + a[1][z], a[0][z] + a[1][y]) +
                   __builtin_fmax(a[2][y] + a[3][z], a[2][z] + a[3][y]);
    }
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            if (w == x) continue;
            int y = -1, z = -1;
            for (int c = 0; c < 4; ++c)
                if (c != x && c != w) (y < 0 ? y : z) = c;
            best = __builtin_fmax(best, (dt[x] + db[w]) + cross[pair_of(y, z)]);
        }
    const unsigned bonus = (unsigned)__double2loint(best + big) & 0x7FFu;
    const unsigned x = min(bonus - (unsigned)kBonusBase, kLutEntries - 1u);   // (a wide block's index is clamped and unused)
    return HOW == Wide::Wave && wide ? rare : (unsigned)lut_mask[x] | ((unsigned)lut_id[x] << 16);
}

// ---------------------------------------------------------------------------
// Integer fast path (bf16 data).  The same class decomposition and the same tie-break bonus as above, in
// 32-bit integers, which the vector unit adds and compares at twice the rate of fp64: with E the exponent of the
// block's largest magnitude, every magnitude times 2^(155-E) is an integer below 2^29 whose lowest set bit is at
// or above bit 11 as long as it lies within ten binades of the largest (8 significand bits + 10 + 11 = 29), so a
// sum of eight stays below 2^32 and the low 11 bits are free for the bonus.  The product with a power of two and the
// conversion to an integer are exact.  Returns kHardBlock for a block that does not fit (an element more than ten
// binades down, a zero or subnormal element, a block maximum below 2^-99): those take the fp64 path above.
// ---------------------------------------------------------------------------
constexpr unsigned kHardBlock = 0xFFFFFFFFu;

__device__ __forceinline__ unsigned int_best_pattern(const uint32_t (&mag)[16], const uint16_t *lut_mask, const uint8_t *lut_id)
{
    uint32_t mx = mag[0], mn = mag[0];
#pragma unroll
    for (int t = 1; t < 16; ++t) {
        mx = max(mx, mag[t]);
        mn = min(mn, mag[t]);
    }
    const uint32_t E = mx >> 23, emin = mn >> 23;
    if (emin == 0u || emin + 10u < E || E < 28u) return kHardBlock;
    const float scale = __uint_as_float((282u - E) << 23);   // 2^(155-E)
    // r = the scaled magnitudes; the tie-break bonus of a cell, B(i, j), never gets an instruction of its own: every
    // sum below that takes a cell in adds the cell's bonus as part of a compile-time constant (a three-operand add),
    // and every candidate total contains each of its eight cells exactly once.
    uint32_t r[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) r[i][j] = (uint32_t)(__uint_as_float(mag[4 * i + j]) * scale);
    auto B = [](int i, int j) { return (uint32_t)(kColBonus[j] * kRowMult[i]); };
    uint32_t dt[4], db[4];   // both top rows / both bottom rows keep column j
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        dt[j] = r[0][j] + r[1][j] + (B(0, j) + B(1, j));
        db[j] = r[2][j] + r[3][j] + (B(2, j) + B(3, j));
    }
    uint32_t st[4][4], sb[4][4];   // row 0 keeps column p and row 1 column q (p != q); rows 2 and 3 likewise
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (p == q) continue;
            st[p][q] = r[0][p] + r[1][q] + (B(0, p) + B(1, q));
            sb[p][q] = r[2][p] + r[3][q] + (B(2, p) + B(3, q));
        }
    // (i) both top rows keep the pair {c1,c2}, both bottom rows its complement
    uint32_t best = 0;
#pragma unroll
    for (int k = 0; k < 6; ++k)
        best = max(best, (dt[pair_c1(k)] + dt[pair_c2(k)]) + (db[pair_c1(5 - k)] + db[pair_c2(5 - k)]));
    // (ii) complementary pairs in each half: row 0 (row 2) keeps {y,z}, row 1 (row 3) the other two columns {w,x}
    {
        uint32_t top = 0, bot = 0;
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const int y = pair_c1(k), z = pair_c2(k), w = pair_c1(5 - k), x = pair_c2(5 - k);
            top = max(top, st[y][w] + st[z][x]);
            bot = max(bot, sb[y][w] + sb[z][x]);
        }
        best = max(best, top + bot);
    }
    // (iii) top rows share column x, bottom rows share column w, the two remaining columns cross in each half
    uint32_t cross[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const int y = pair_c1(k), z = pair_c2(k);
        cross[k] = max(st[y][z], st[z][y]) + max(sb[y][z], sb[z][y]);
    }
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            if (w == x) continue;
            int y = -1, z = -1;
            for (int c = 0; c < 4; ++c)
                if (c != x && c != w) (y < 0 ? y : z) = c;
            best = max(best, dt[x] + db[w] + cross[pair_of(y, z)]);
        }
    const unsigned xi = min((best & 0x7FFu) - (unsigned)kBonusBase, kLutEntries - 1u);
    return (unsigned)lut_mask[xi] | ((unsigned)lut_id[xi] << 16);
}

// ---------------------------------------------------------------------------
// Per-dtype access to one block row (four consecutive weights).
// ---------------------------------------------------------------------------
template <typename T> struct RowOps;

template <> struct RowOps<uint16_t> {  // bf16
    using Row = uint2;     // four bf16
    using Pair = uint32_t; // two bf16
    static constexpr int kWindow = 29, kWide = 42;
    static __device__ __forceinline__ Row load(const uint16_t *p) { return *reinterpret_cast<const uint2 *>(p); }
    static __device__ __forceinline__ uint32_t bits(const Row &r, int j)
    {
        const uint64_t v = ((uint64_t)r.y << 32) | r.x;
        return (uint32_t)(v >> (16 * j)) & 0xFFFFu;
    }
    static __device__ __forceinline__ uint32_t mag(const Row &r, int j)  // compile-time j
    {
        const uint32_t d = (j < 2) ? r.x : r.y;
        return (j & 1) ? (d & 0x7FFF0000u) : ((d << 16) & 0x7FFF0000u);
    }
    static __device__ __forceinline__ Pair pair(uint32_t lo, uint32_t hi) { return lo | (hi << 16); }
};

// IEEE binary16: the same 16-bit moves as bf16; a magnitude widens to fp32 exactly (binary16 subnormals are fp32
// normals).  An element with fp32 exponent e is a multiple of 2^(e-10), so the fast path's window is 26 binades,
// and eight of them sum exactly in fp64 over 39 binades, which is all binary16 has: no block needs the slow path.
template <> struct RowOps<s24_half> {
    using Row = uint2;
    using Pair = uint32_t;
    static constexpr int kWindow = 26, kWide = 39;
    static __device__ __forceinline__ Row load(const s24_half *p) { return *reinterpret_cast<const uint2 *>(p); }
    static __device__ __forceinline__ uint32_t bits(const Row &r, int j) { return RowOps<uint16_t>::bits(r, j); }
    static __device__ __forceinline__ uint32_t mag(const Row &r, int j)  // compile-time j
    {
        const uint32_t d = (j < 2) ? r.x : r.y;
        return __float_as_uint(s24_num<s24_half>::widen(((j & 1) ? (d >> 16) : d) & 0x7FFFu));
    }
    static __device__ __forceinline__ Pair pair(uint32_t lo, uint32_t hi) { return lo | (hi << 16); }
};

template <> struct RowOps<float> {
    using Row = uint4;
    using Pair = uint2;
    static constexpr int kWindow = 13, kWide = 26;
    static __device__ __forceinline__ Row load(const float *p) { return *reinterpret_cast<const uint4 *>(p); }
    static __device__ __forceinline__ uint32_t bits(const Row &r, int j)
    {
        return j == 0 ? r.x : (j == 1 ? r.y : (j == 2 ? r.z : r.w));
    }
    static __device__ __forceinline__ uint32_t mag(const Row &r, int j) { return bits(r, j) & 0x7FFFFFFFu; }
    static __device__ __forceinline__ Pair pair(uint32_t lo, uint32_t hi) { return make_uint2(lo, hi); }
};

// The blocks of the lanes that set `wide` (p: the lane's block), all 64 lanes active.  Few to a wave are scored by the wave together and
// many by a lane each: in fp64 either costs as much at about 28, in fixed point (400 us, 29 a block) at 14.  In a call, from memory and
// with a loop over rows, so that the common path keeps the registers of seven waves per SIMD.  bf16 search, one block in a hundred 40 binades
// wide: 5120 x 1280 110 us (1460 with each lane's walk in the loop, 609 with the integer path's queue), 3072 x 768 92 (974, 698); without
// such blocks 6.79 and 4.74 (6.78 and 4.66; 7.38 and 4.70 with all of this inlined after the scores, for six waves).
template <typename T> __device__ __noinline__ unsigned wide_blocks(const T *p, int64_t ldw, bool wide)
{
    using Ops = RowOps<T>;
    auto load = [ldw](const T *at) {
        Mag16 mag;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const typename Ops::Row row = Ops::load(at + i * ldw);
#pragma unroll
            for (int j = 0; j < 4; ++j) mag.v[4 * i + j] = Ops::mag(row, j);
        }
        return mag;
    };
    auto of_lane = [p](int src) {
        const uint64_t at = (uint64_t)p;
        return reinterpret_cast<const T *>((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)at, src) |
                                           (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(at >> 32), src) << 32);
    };
    unsigned res = 0;
    uint32_t emax = 0, emin = 0;
    if (wide) exponents(load(p).v, emax, emin);
    const bool slow = emin + Ops::kWide < emax, mid = wide && !slow;
    unsigned long long mids = __ballot(mid), slows = __ballot(slow);
    if (__popcll(mids) > 28) {
        if (mid) res = mid_best_pattern(load(p));
        mids = 0;
    }
    if (__popcll(slows) > 14) {
        if (slow) res = slow_best_pattern(load(p));
        slows = 0;
    }
    for (; slows != 0; slows &= slows - 1) {
        const int src = (int)__builtin_ctzll(slows);
        const unsigned r = wave_slow_best_pattern(load(of_lane(src)));
        if ((int)(threadIdx.x & 63) == src) res = r;
    }
    for (; mids != 0; mids &= mids - 1) {   // a row at a time, which takes few registers
        const int src = (int)__builtin_ctzll(mids);
        const T *at = of_lane(src);
        const WavePatterns patterns;
        double best = 0.0, second = 0.0;
#pragma unroll 1
        for (int i = 0; i < 4; ++i) {
            const typename Ops::Row row = Ops::load(at + i * ldw);
#pragma unroll
            for (int j = 0; j < 4; ++j) patterns.add(4 * i + j, (double)__uint_as_float(Ops::mag(row, j)), best, second);
        }
        const unsigned r = patterns.first_of_best(best, second);
        if ((int)(threadIdx.x & 63) == src) res = r;
    }
    return res;
}

// A workgroup's tile is TBW blocks wide and 256 / TBW * S blocks tall, S blocks per lane.
//   32 x 32 (S = 4): the lookup tables are staged once per 1024 blocks and the next block's rows are requested while the
//   current one is scored: the better shape for the largest matrices.
//   16 x 16 (S = 1): four times as many workgroups of a quarter of the length; 32 x 16 (S = 2) between the two.
// A launch covers up to kMaxWeights weights: tiles first_tile[i] .. first_tile[i+1]-1 belong to weight i (unused entries repeat the
// total).  A launch for a weight of a million parameters is mostly its start, one workgroup's way through and its drain.  Both weights of a
// layer, searched and compressed, in a launch each and (with the tables staged as above) in one: 1024 x 256 fp32 17.3 -> 9.2 us,
// 3072 x 768 bf16 16.2 -> 10.4, 5120 x 1280 27.9 -> 20.5; with given masks 3072 x 768 11.9 -> 7.9, 5504 x 2048 (two and one) 39.4 -> 34.
constexpr int kMaxWeights = 4;
struct MaskWeight {
    const void *W;
    int64_t ldw;
    int br, bq;             // blocks
    const uint16_t *mask_in;
    uint16_t *mask_out;
    uint8_t *index_out;
    void *vals;
    uint16_t *meta;
    void *valsT;
    uint16_t *metaT;
};
struct MaskBatch {
    MaskWeight w[kMaxWeights];
    int first_tile[kMaxWeights + 1];
    int begin;              // first tile of this launch
};

// bf16, searched alone in the small tile: see wide_blocks
template <typename T, bool SEARCH, bool COMPRESS, int S> constexpr bool kBf16Small = SEARCH && !COMPRESS && sizeof(T) == 2 && RowOps<T>::kWindow == 29 && S == 1;

template <typename T, bool SEARCH, bool COMPRESS, int TBW, int S>
__global__ __launch_bounds__(256, (kBf16Small<T, SEARCH, COMPRESS, S> ? 7 : 1)) void mask_compress_kernel(const MaskBatch batch)
{
    using Ops = RowOps<T>;
    using Row = typename Ops::Row;
    using Pair = typename Ops::Pair;
    constexpr int LR = 256 / TBW, TBH = LR * S, PITCH = TBH + 1;   // rows of lanes, tile height, LDS pitch of the transposed pairs
    static_assert(!COMPRESS || TBH % 16 == 0, "a tile holds whole chunks of the column-wise operand");
    constexpr bool FAST = COMPRESS && sizeof(T) == 2;   // bf16: table-driven compressor
    // bf16 search on its own in the large tile: integer scoring, the blocks it cannot take queued for the fp64 path.  The queue is a
    // second trip through the workgroup: in the smaller tiles, whose launches wait for one workgroup, fp64 scoring inside the loop is the faster
    // (5120 x 1280: 8.8 -> 6.7 us).  (In the fused search + compress kernel the four blocks' rows held in registers across the queue cost
    // more than the cheaper scoring saves: measured 4-8 % slower, so it keeps the fp64 scoring too.)
    constexpr bool DEFER = SEARCH && !COMPRESS && sizeof(T) == 2 && RowOps<T>::kWindow == 29 && S == 4;
    constexpr bool BF16_SMALL = kBf16Small<T, SEARCH, COMPRESS, S>;
    __shared__ int s_nhard;
    __shared__ uint16_t s_hard[DEFER ? 256 * S : 1];
    __shared__ uint32_t s_fix[DEFER ? 256 * S : 1];
    // the part of the tables that this instance uses: masks for a search, ids, compressor entries
    constexpr int TAB_FIRST = SEARCH ? 0 : offsetof(MaskLut, id) / 16, TAB_LAST = (FAST ? sizeof(MaskTables) : sizeof(MaskLut)) / 16;
    constexpr int TAB = SEARCH || FAST ? TAB_LAST - TAB_FIRST : 0, TAB_PER_LANE = (TAB + 255) / 256;
    __shared__ uint4 s_tables[TAB ? TAB : 1];
    const uint16_t *s_lut_mask = reinterpret_cast<const uint16_t *>(s_tables);
    const uint8_t *s_lut_id = reinterpret_cast<const uint8_t *>(s_tables + (SEARCH ? offsetof(MaskLut, id) / 16 : 0));
    const uint4 *s_clut = s_tables + (sizeof(MaskLut) / 16 - TAB_FIRST);
    __shared__ Pair s_valsT[COMPRESS ? 4 * TBW * PITCH : 1];
    __shared__ uint8_t s_nibT[COMPRESS ? 4 * TBW * PITCH : 1];

    const int tid = threadIdx.x;
    uint4 table[TAB_PER_LANE ? TAB_PER_LANE : 1];   // requested ahead of the weights: it is in the L2 and there first
#pragma unroll
    for (int k = 0; k < TAB_PER_LANE; ++k) table[k] = reinterpret_cast<const uint4 *>(&g_tables)[TAB_FIRST + min(tid + 256 * k, TAB - 1)];
    const int batch_tile = batch.begin + (int)blockIdx.x;
    int which = 0;   // wave-uniform
#pragma unroll
    for (int i = 1; i < kMaxWeights; ++i)
        if (batch_tile >= batch.first_tile[i]) which = i;
    const MaskWeight &weight = batch.w[which];
    const T *__restrict__ W = static_cast<const T *>(weight.W);
    const int64_t ldw = weight.ldw;
    const int br = weight.br, bq = weight.bq;
    const uint16_t *__restrict__ mask_in = weight.mask_in;
    uint16_t *__restrict__ mask_out = weight.mask_out;
    uint8_t *__restrict__ index_out = weight.index_out;
    T *__restrict__ vals = static_cast<T *>(weight.vals), *__restrict__ valsT = static_cast<T *>(weight.valsT);
    uint16_t *__restrict__ meta = weight.meta, *__restrict__ metaT = weight.metaT;
    const unsigned tile = (unsigned)(batch_tile - batch.first_tile[which]), tiles_q = (unsigned)(bq + TBW - 1) / TBW;
    const int bj0 = (int)(tile % tiles_q) * TBW, bi0 = (int)(tile / tiles_q) * TBH;
    const int lbj = tid % TBW;
    const int bj = bj0 + lbj;
    const int64_t R = 4 * (int64_t)br, Q = 4 * (int64_t)bq;  // rows of vals / of valsT

    // first weight row of this lane's first block; block s of the lane lies LR s block rows further down
    const T *wrow = W + (int64_t)(4 * (bi0 + tid / TBW)) * ldw + 4 * bj;
    auto fetch = [&](Row (&dst)[4], const T *p, bool ok) {
        if (ok) {
#pragma unroll
            for (int i = 0; i < 4; ++i) dst[i] = Ops::load(p + i * ldw);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) dst[i] = Row{};
        }
    };
    auto magnitudes = [&](const Row (&rows)[4], uint32_t (&mag)[16]) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) mag[4 * i + j] = Ops::mag(rows[i], j);
    };
    // Index words along q.  nib_lo, nib_hi: a block's nibbles of rows 0 and 1, and of 2 and 3, 16 bits apart.  Four lanes' nibbles
    // form a word, the four words of a chunk's 16 lanes a row's eight bytes, and the block row's four rows are contiguous: the
    // first of the 16 lanes gathers all of it and stores 32 bytes (2-byte stores from every fourth lane were four of them).
    auto store_meta = [&](uint32_t nib_lo, uint32_t nib_hi, int bi, bool valid) {
        auto from = [](uint32_t v, auto lanes) {   // of the lane so many further up in the group of 16 (row_shl)
            return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x100 + decltype(lanes)::value, 0xF, 0xF, true);
        };
        const std::integral_constant<int, 1> l1;
        const std::integral_constant<int, 2> l2;
        const std::integral_constant<int, 4> l4;
        const std::integral_constant<int, 8> l8;
        nib_lo |= from(nib_lo, l1) << 4;
        nib_hi |= from(nib_hi, l1) << 4;
        nib_lo |= from(nib_lo, l2) << 8;
        nib_hi |= from(nib_hi, l2) << 8;
        const uint32_t next_lo = from(nib_lo, l4), next_hi = from(nib_hi, l4);
        uint32_t row[4][2];   // words 0 and 1 of rows 0 .. 3
        row[0][0] = __builtin_amdgcn_perm(next_lo, nib_lo, 0x05040100u);
        row[1][0] = __builtin_amdgcn_perm(next_lo, nib_lo, 0x07060302u);
        row[2][0] = __builtin_amdgcn_perm(next_hi, nib_hi, 0x05040100u);
        row[3][0] = __builtin_amdgcn_perm(next_hi, nib_hi, 0x07060302u);
#pragma unroll
        for (int i = 0; i < 4; ++i) row[i][1] = from(row[i][0], l8);   // words 2 and 3
        if (valid && (lbj & 15) == 0) {   // br and bq are multiples of 16: the 16 lanes are all inside the matrix or all outside
            typedef uint32_t two_rows __attribute__((ext_vector_type(4), aligned(8)));
            two_rows *dst = reinterpret_cast<two_rows *>(meta + ((int64_t)(bj >> 4) * R + 4 * bi) * 4);
            dst[0] = two_rows{row[0][0], row[0][1], row[1][0], row[1][1]};
            dst[1] = two_rows{row[2][0], row[2][1], row[3][0], row[3][1]};
        }
    };
    // What follows the search for block s of this lane (rows in registers, mask m and pattern id known):
    // the mask and id stores and, when compressing, both compressed orientations.
    auto emit = [&](const Row (&rows)[4], unsigned m, unsigned id, int s) {
        const int lbi = tid / TBW + LR * s;
        const int bi = bi0 + lbi;
        const bool valid = (bi < br) && (bj < bq);
        if constexpr (SEARCH) {
            if (valid) {
                if (mask_out) mask_out[(int64_t)bi * bq + bj] = (uint16_t)m;
                if (index_out) index_out[(int64_t)bi * bq + bj] = (uint8_t)id;
            }
        }
        if constexpr (FAST) {
            if constexpr (!SEARCH) id = s_lut_id[min(lut_index_of_mask(m), kLutEntries - 1u)];
            const uint4 rsel = s_clut[3 * id], csel = s_clut[3 * id + 1], mt = s_clut[3 * id + 2];
            const uint32_t rs[4] = {rsel.x, rsel.y, rsel.z, rsel.w}, cs[4] = {csel.x, csel.y, csel.z, csel.w};
            // along q: one dword (two kept bf16) per block row.  The four lanes of a quad (four neighbouring blocks
            // of one block row) transpose their 4 x 4 dwords among themselves, two exchanges with the lane one away and
            // two with the lane two away, so that lane k of the quad ends up with row k of all four blocks: 16
            // contiguous bytes of that row's run, one store instead of four 4-byte ones.  (br and bq are multiples
            // of 16: a quad is all inside the matrix or all outside.)
            uint32_t pr[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) pr[i] = __builtin_amdgcn_perm(rows[i].y, rows[i].x, rs[i]);
            {
                const bool odd = lbj & 1, upper = lbj & 2;
#pragma unroll
                for (int i = 0; i < 4; i += 2) {   // with lane ^ 1: an even lane hands over row i+1, an odd one row i
                    const uint32_t got = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(odd ? pr[i] : pr[i + 1]), 0xB1, 0xF, 0xF, false);
                    if (odd) pr[i] = got;
                    else pr[i + 1] = got;
                }
#pragma unroll
                for (int j = 0; j < 2; ++j) {      // with lane ^ 2: a lower lane hands over entry j+2, an upper one entry j
                    const uint32_t got = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(upper ? pr[j] : pr[j + 2]), 0x4E, 0xF, 0xF, false);
                    if (upper) pr[j] = got;
                    else pr[j + 2] = got;
                }
            }
            if (valid)
                *reinterpret_cast<uint4 *>(reinterpret_cast<uint32_t *>(vals) + ((int64_t)(bj >> 4) * R + 4 * bi + (lbj & 3)) * 16 + (bj & 12)) =
                    make_uint4(pr[0], pr[1], pr[2], pr[3]);
            uint32_t nib_lo = mt.x, nib_hi = mt.y;
            store_meta(nib_lo, nib_hi, bi, valid);
            // along r: gather each column from the four rows, pick its two kept rows, park in LDS
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t half = (j & 1) ? 0x07060302u : 0x05040100u;
                const uint32_t r0 = (j < 2) ? rows[0].x : rows[0].y, r1 = (j < 2) ? rows[1].x : rows[1].y;
                const uint32_t r2 = (j < 2) ? rows[2].x : rows[2].y, r3 = (j < 2) ? rows[3].x : rows[3].y;
                const uint32_t col_lo = __builtin_amdgcn_perm(r1, r0, half);  // rows 0,1 of column j
                const uint32_t col_hi = __builtin_amdgcn_perm(r3, r2, half);  // rows 2,3
                const int a = (j * TBW + lbj) * PITCH + lbi;
                s_valsT[a] = __builtin_amdgcn_perm(col_hi, col_lo, cs[j]);
                s_nibT[a] = (uint8_t)((mt.z >> (4 * j)) & 0xFu);
            }
        } else if constexpr (COMPRESS) {
            // along q: two kept weights and one nibble per block row
            uint32_t nib_lo = 0, nib_hi = 0;  // nibbles of rows (0,1) and (2,3), 16 bits apart
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const unsigned m4 = (m >> (4 * i)) & 0xFu;
                const int i0 = (__ffs((int)m4) - 1) & 3;
                const int i1 = (31 - __clz((int)(m4 | 1u))) & 3;
                const Pair pr = Ops::pair(Ops::bits(rows[i], i0), Ops::bits(rows[i], i1));
                // chunk bj/16 of row 4bi+i, pair bj%16 of its 16 pairs
                if (valid) reinterpret_cast<Pair *>(vals)[((int64_t)(bj >> 4) * R + 4 * bi + i) * 16 + (bj & 15)] = pr;
                const uint32_t nib = (uint32_t)(i0 | (i1 << 2));
                if (i < 2) nib_lo |= nib << (16 * i);
                else nib_hi |= nib << (16 * (i - 2));
            }
            store_meta(nib_lo, nib_hi, bi, valid);
            // along r: kept rows of each column go through LDS to be written transposed
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const unsigned c = m >> j;
                const unsigned cm = (c & 1u) | ((c >> 3) & 2u) | ((c >> 6) & 4u) | ((c >> 9) & 8u);
                const int i0 = (__ffs((int)cm) - 1) & 3;
                const int i1 = (31 - __clz((int)(cm | 1u))) & 3;
                uint32_t e[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) e[i] = Ops::bits(rows[i], j);
                const uint32_t v0 = i0 == 0 ? e[0] : (i0 == 1 ? e[1] : (i0 == 2 ? e[2] : e[3]));
                const uint32_t v1 = i1 == 0 ? e[0] : (i1 == 1 ? e[1] : (i1 == 2 ? e[2] : e[3]));
                const int a = (j * TBW + lbj) * PITCH + lbi;
                s_valsT[a] = Ops::pair(v0, v1);
                s_nibT[a] = (uint8_t)(i0 | (i1 << 2));
            }
        }
    };

    auto stage_tables = [&]() {
        if (DEFER && tid == 0) s_nhard = 0;
        if constexpr (TAB > 0) {
#pragma unroll
            for (int k = 0; k < TAB_PER_LANE; ++k)
                if (tid + 256 * k < TAB) s_tables[tid + 256 * k] = table[k];
            __syncthreads();
        }
    };

    if constexpr (DEFER) {
        // bf16 search: all S blocks of the lane are scored by the integer fast path first; the few blocks it
        // cannot take (about one in forty for normally distributed weights) are queued in LDS and scored afterwards
        // by the fp64 path, one per lane, so that a rare block costs one lane's time instead of stalling its whole
        // wave in a divergent branch.
        Row blk[S][4];
        unsigned res[S];
#pragma unroll
        for (int s = 0; s < S; ++s) fetch(blk[s], wrow + (int64_t)(4 * LR * s) * ldw, (bi0 + tid / TBW + LR * s < br) && (bj < bq));
        stage_tables();
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const bool valid = (bi0 + tid / TBW + LR * s < br) && (bj < bq);
            uint32_t mag[16];
            magnitudes(blk[s], mag);
            res[s] = valid ? int_best_pattern(mag, s_lut_mask, s_lut_id) : 0x33CCu;   // off the edge: pattern 0, never stored
            if (res[s] == kHardBlock) s_hard[atomicAdd(&s_nhard, 1)] = (uint16_t)(256 * s + tid);
        }
        __syncthreads();
        const int nhard = s_nhard;
        for (int e = tid; e < nhard; e += 256) {
            const int code = s_hard[e], hs = code >> 8, owner = code & 255;
            const T *p = W + (int64_t)(4 * (bi0 + owner / TBW + LR * hs)) * ldw + 4 * (bj0 + owner % TBW);
            Row rows[4];
            fetch(rows, p, true);
            uint32_t mag[16];
            magnitudes(rows, mag);
            s_fix[code] = best_pattern<Ops::kWindow, Ops::kWide, Wide::Lane>(mag, s_lut_mask, s_lut_id);
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const unsigned r = res[s] == kHardBlock ? s_fix[256 * s + tid] : res[s];
            emit(blk[s], r & 0xFFFFu, r >> 16, s);
        }
    } else {
        // The rows of the next block are requested before the current one is scored.
        Row nxt[4];
        unsigned m_nxt = 0x33CCu;
        const uint16_t *mrow = mask_in + (int64_t)(bi0 + tid / TBW) * bq + bj;
        auto request = [&](int bi) {
            const bool ok = (bi < br) && (bj < bq);
            fetch(nxt, wrow, ok);
            if constexpr (!SEARCH) m_nxt = ok ? *mrow : 0x33CCu;
        };
        request(bi0 + tid / TBW);
        stage_tables();
#pragma unroll 1
        for (int s = 0; s < S; ++s) {
            const int bi = bi0 + tid / TBW + LR * s;
            Row rows[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) rows[i] = nxt[i];
            unsigned m = m_nxt, id = 0;
            if (s + 1 < S) {
                wrow += 4 * LR * ldw;
                mrow += (int64_t)LR * bq;
                request(bi + LR);
            }
            if constexpr (SEARCH) {
                uint32_t mag[16];
                magnitudes(rows, mag);
                unsigned rare = 0;
                if constexpr (BF16_SMALL) {
                    uint32_t emax, emin;
                    exponents(mag, emax, emin);
                    const bool wide = emin + Ops::kWindow < emax;
                    if (__any(wide)) rare = wide_blocks<T>(wrow, ldw, wide);
                }
                constexpr Wide HOW = sizeof(T) == 4 ? Wide::Wave : BF16_SMALL ? Wide::Given : Wide::Lane;
                const unsigned res = best_pattern<Ops::kWindow, Ops::kWide, HOW>(mag, s_lut_mask, s_lut_id, rare);
                m = res & 0xFFFFu;
                id = res >> 16;
            }
            emit(rows, m, id, s);
        }
    }
    if constexpr (COMPRESS) {
        __syncthreads();
        // valsT: TBH / 16 chunks (16 pairs each) of the tile's 4 TBW columns of W.  One item = four consecutive pairs of
        // one column; consecutive lanes take consecutive items of a column, then the next column, so a
        // chunk of the tile leaves as one contiguous run.
        Pair *outT = reinterpret_cast<Pair *>(valsT);
#pragma unroll
        for (int it = 0; it < S; ++it) {
            const int idx = tid + 256 * it;                    // TBW * TBH items
            const int quad = idx & 3, col = (idx >> 2) % (4 * TBW), half = idx / (16 * TBW);   // col = 4*lbj + j
            const int j = col & 3, lb = col >> 2;
            const int lbi = 16 * half + 4 * quad, bi = bi0 + lbi;
            if (bj0 + lb < bq && bi < br) {   // br is a multiple of 16: a quad is all in or all out
                const Pair *src = &s_valsT[(j * TBW + lb) * PITCH + lbi];
                Pair *dst = outT + ((int64_t)(bi >> 4) * Q + 4 * (bj0 + lb) + j) * 16 + (bi & 15);
                if constexpr (sizeof(Pair) == 4) {
                    *reinterpret_cast<uint4 *>(dst) = make_uint4(src[0], src[1], src[2], src[3]);
                } else {
                    uint4 *two = reinterpret_cast<uint4 *>(dst);
                    two[0] = make_uint4(src[0].x, src[0].y, src[1].x, src[1].y);
                    two[1] = make_uint4(src[2].x, src[2].y, src[3].x, src[3].y);
                }
            }
        }
        // metaT: per column and chunk four words; one thread packs the 16 nibbles of one (column, chunk)
        if (tid < 4 * TBW * (TBH / 16)) {
            const int col = tid % (4 * TBW), half = tid / (4 * TBW);
            const int j = col & 3, lb = col >> 2;
            if (bj0 + lb < bq && bi0 + 16 * half < br) {
                const uint8_t *n = &s_nibT[(j * TBW + lb) * PITCH + 16 * half];
                uint32_t w01 = 0, w23 = 0;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    w01 |= (uint32_t)n[e] << (4 * e);
                    w23 |= (uint32_t)n[8 + e] << (4 * e);
                }
                const int kc = (bi0 >> 4) + half;   // chunk index along r
                *reinterpret_cast<uint2 *>(metaT + ((int64_t)kc * Q + 4 * (bj0 + lb) + j) * 4) = make_uint2(w01, w23);
            }
        }
    }
}

template <typename T, bool SEARCH, bool COMPRESS, int TBW, int S>
int launch_tiles(MaskBatch &batch, int count, hipStream_t st)
{
    constexpr int TBH = 256 / TBW * S;
    constexpr int64_t LAUNCH = 1 << 23;   // a launch holds less than 2^32 work items (of more it silently runs the remainder)
    int64_t tiles = 0;
    for (int i = 0; i <= kMaxWeights; ++i) {
        batch.first_tile[i] = (int)tiles;
        if (i < count) tiles += (int64_t)((batch.w[i].bq + TBW - 1) / TBW) * ((batch.w[i].br + TBH - 1) / TBH);
        S24_REQUIRE(tiles <= INT32_MAX - LAUNCH, S24_ERR_SHAPE);   // more weights than any memory holds
    }
    for (int64_t begin = 0; begin < tiles; begin += LAUNCH) {
        batch.begin = (int)begin;
        hipLaunchKernelGGL((mask_compress_kernel<T, SEARCH, COMPRESS, TBW, S>), dim3((unsigned)std::min(tiles - begin, LAUNCH)), dim3(256), 0, st,
                           batch);
    }
    return s24_launch_status();
}
// Which tile, by the number of 32 x 32 tiles of all weights together, in compute units (256 of them); measured in us, 32 x 32 / 32 x 16 /
// 16 x 16 blocks.  The small tile has the shortest way through a workgroup, which is what a launch of few tiles waits for:
//   bf16 search            100 tiles: 6.5 / 4.4 / 3.9    400: 9.0 / 7.9 / 6.7    1376: 17.7 / 18.9 / 16.8    2752: 36.0 / 39.3 / 38.0
//   fp16, fp32 search      400: 9.3 / 8.3 / 7.0, 14.0 / 12.1 / 11.2    2752: 34.5 / 35.4 / 33.5, 48.1 / 47.4 / 44.8
//   bf16 search, compress  288: 12.4 / 11.0 / 10.4    800: 20.9 / 20.4 / 20.5    1300: 28.3 / 29.0 / 28.7    5504: 93 / 103 / 103
//   fp32 search, compress  32: 20.1 / 12.8 / 9.2    512: 32.1 / 32.4 / 30.0    2048: 95.9 / 97.3 / 90.5
//   bf16 given mask        288: 10.0 / 8.9 / 7.9    800: 17.4 / 16.4 / 16.2    1376: 26.4 / 23.7 / 23.9    8192: 115 / 114 / 122
//   fp32 given mask        128: 16.3 / 11.1 / 9.2    288: 22.0 / 17.6 / 18.7    512: 28.8 / 25.8 / 29.2    2048: 95.2 / 99.9 / 97.6
template <typename T, bool SEARCH, bool COMPRESS> int launch_sized(MaskBatch &batch, int count, hipStream_t st)
{
    constexpr bool HALF = sizeof(T) == 2;
    int64_t tiles = 0;
    for (int i = 0; i < count; ++i) tiles += (int64_t)((batch.w[i].bq + 31) / 32) * ((batch.w[i].br + 31) / 32);
    const int64_t cus = s24_cu_count();
    if constexpr (SEARCH && (HALF ? !COMPRESS && RowOps<T>::kWindow != 29 : true)) {
        return launch_tiles<T, SEARCH, COMPRESS, 16, 1>(batch, count, st);
    } else {
        if (tiles < (!COMPRESS ? 8 : HALF ? 4 : 1) * cus) return launch_tiles<T, SEARCH, COMPRESS, 16, 1>(batch, count, st);
        if constexpr (!SEARCH)
            if (HALF || tiles < 4 * cus) return launch_tiles<T, SEARCH, COMPRESS, 32, 2>(batch, count, st);
        if constexpr (SEARCH || !HALF) return launch_tiles<T, SEARCH, COMPRESS, 32, 4>(batch, count, st);
    }
}

// `count` weights of one dtype; the masks of all of them are searched, or those of all of them are given
int launch(MaskBatch &batch, int count, s24_dtype dt, bool compress, hipStream_t st)
{
    const bool search = batch.w[0].mask_in == nullptr;
    auto run = [&](auto t) {
        using T = decltype(t);
        if (!compress) return launch_sized<T, true, false>(batch, count, st);
        return search ? launch_sized<T, true, true>(batch, count, st) : launch_sized<T, false, true>(batch, count, st);
    };
    return dt == S24_BF16 ? run(uint16_t{}) : dt == S24_F16 ? run(s24_half{}) : run(float{});
}

// ------------------------------------------------------------------ monitors
// Flip count: || m_new - m_old ||_1 over all mask cells.  Eight blocks per 16-byte load of each mask, up to four loads per
// thread in flight; wave sums by cross-lane adds, one 64-bit atomic per workgroup.
__global__ __launch_bounds__(256) void clear_counter_kernel(unsigned long long *counter) { *counter = 0ull; }

__global__ __launch_bounds__(256) void mask_flips_kernel(const uint16_t *__restrict__ mask_new,
                                                         const uint16_t *__restrict__ mask_old, int64_t nblocks,
                                                         uint32_t *__restrict__ block_flips,
                                                         unsigned long long *__restrict__ total)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x, whole = nblocks / 8;   // vectors of eight masks
    unsigned count = 0;
    auto add = [&](int64_t v, const uint4 &a, const uint4 &b) {
        const uint32_t x[4] = {a.x ^ b.x, a.y ^ b.y, a.z ^ b.z, a.w ^ b.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            count += __builtin_popcount(x[k]);
            if (block_flips) {
                block_flips[8 * v + 2 * k] += __builtin_popcount(x[k] & 0xFFFFu);
                block_flips[8 * v + 2 * k + 1] += __builtin_popcount(x[k] >> 16);
            }
        }
    };
    const uint4 *vn = reinterpret_cast<const uint4 *>(mask_new), *vo = reinterpret_cast<const uint4 *>(mask_old);
    int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; v + 3 * stride < whole; v += 4 * stride) {
        uint4 a[4], b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            a[u] = vn[v + u * stride];
            b[u] = vo[v + u * stride];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) add(v + u * stride, a[u], b[u]);
    }
    for (; v < whole; v += stride) add(v, vn[v], vo[v]);
    if (blockIdx.x == 0 && threadIdx.x == 0)
        for (int64_t b = 8 * whole; b < nblocks; ++b) {
            const unsigned c = __builtin_popcount((unsigned)(mask_new[b] ^ mask_old[b]));
            count += c;
            if (block_flips) block_flips[b] += c;
        }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) count += __shfl_down(count, off, 64);
    // one atomic per workgroup: thousands of them on one address would cost more than the scan itself
    __shared__ unsigned s_part[4];
    if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = count;
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned long long sum = (unsigned long long)s_part[0] + s_part[1] + s_part[2] + s_part[3];
        if (sum != 0) atomicAdd(total, sum);
    }
}

// L1-norm gap: one block per lane.  The 90 kept norms fall into the classes of the search (see the top of this file), and
// inside a class a norm is a sum of independent choices, so the two largest of a class follow from the two largest of each
// choice: 6 totals; best and second best of 6 top and 6 bottom halves (36 patterns); for each of the 12 pairs (column shared
// by the top rows, column shared by the bottom rows) two crossings in either half (48).  About 260 fp64 operations where
// the 90 sums one by one took 4300 with their selects (bf16 5120 x 1280: 80 -> 9 us).  Sums are exact in any order as
// long as the block spans at most WIDE binades; a wider block takes the 90 sums one by one in index order, which is
// what fixes its rounding, and so does one with an infinity or a NaN, which minima and maxima would drop.
struct Top2 {
    double first, second;
    __device__ __forceinline__ void merge(double f, double s)   // f >= s
    {
        second = __builtin_fmax(__builtin_fmax(second, s), __builtin_fmin(first, f));
        first = __builtin_fmax(first, f);
    }
    __device__ __forceinline__ void add(double v)
    {
        second = __builtin_fmax(second, __builtin_fmin(first, v));
        first = __builtin_fmax(first, v);
    }
};
template <typename T> __device__ __forceinline__ double block_gap(const T *__restrict__ W, int64_t ldw, int bi, int bj)
{
    using Ops = RowOps<T>;
    uint32_t mag[16];
    uint32_t mx = 0, mn = 0xFFFFFFFFu;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const typename Ops::Row row = Ops::load(W + (int64_t)(4 * bi + i) * ldw + 4 * bj);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t m = Ops::mag(row, j);
            mag[4 * i + j] = m;
            mx = max(mx, m);
            mn = min(mn, m - 1u);   // zero wraps to the top and never wins
        }
    }
    double a[4][4];
#pragma unroll
    for (int t = 0; t < 16; ++t) a[t / 4][t % 4] = (double)__uint_as_float(mag[t]);
    const uint32_t emax = max(mx >> 23, 1u), emin = mn == 0xFFFFFFFFu ? 255u : max(mn >> 23, 1u);
    double first = 0.0, second = 0.0;
    if (emin + Ops::kWide < emax || emax == 255u) {
#pragma unroll 1
        for (int k = 0; k < S24_NUM_PATTERNS; ++k) {
            const unsigned m = g_patterns.mask[k];
            double sum = 0.0;
#pragma unroll
            for (int t = 0; t < 16; ++t) sum += ((m >> t) & 1u) ? a[t / 4][t % 4] : 0.0;
            if (k == 0) {
                first = sum;
            } else if (sum > first) {
                second = first;
                first = sum;
            } else if (k == 1 || sum > second) {
                second = sum;
            }
        }
    } else {
        double st[4][4], sb[4][4];   // row 0 keeps column p and row 1 column q; rows 2 and 3 likewise
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                st[p][q] = a[0][p] + a[1][q];
                sb[p][q] = a[2][p] + a[3][q];
            }
        Top2 best{0.0, 0.0};         // norms are not negative, and there are more than two of them
#pragma unroll
        for (int k = 0; k < 6; ++k)
            best.add((st[pair_c1(k)][pair_c1(k)] + st[pair_c2(k)][pair_c2(k)]) + (sb[pair_c1(5 - k)][pair_c1(5 - k)] + sb[pair_c2(5 - k)][pair_c2(5 - k)]));
        Top2 top{0.0, 0.0}, bot{0.0, 0.0};
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const int y = pair_c1(k), z = pair_c2(k), w = pair_c1(5 - k), x = pair_c2(5 - k);
            top.add(st[y][w] + st[z][x]);
            bot.add(sb[y][w] + sb[z][x]);
        }
        best.merge(top.first + bot.first, __builtin_fmax(top.first + bot.second, top.second + bot.first));
        Top2 cross[6];
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const int y = pair_c1(k), z = pair_c2(k);
            const double th = __builtin_fmax(st[y][z], st[z][y]), tl = __builtin_fmin(st[y][z], st[z][y]);
            const double bh = __builtin_fmax(sb[y][z], sb[z][y]), bl = __builtin_fmin(sb[y][z], sb[z][y]);
            cross[k] = Top2{th + bh, __builtin_fmax(th + bl, tl + bh)};
        }
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                if (w == x) continue;
                int y = -1, z = -1;
                for (int c = 0; c < 4; ++c)
                    if (c != x && c != w) (y < 0 ? y : z) = c;
                const double shared = st[x][x] + sb[w][w];
                const Top2 &c = cross[pair_of(y, z)];
                best.merge(shared + c.first, shared + c.second);
            }
        first = best.first;
        second = best.second;
    }
    return first - second;
}
// A workgroup's tile is 2^wide block columns (up to a wave's 64, fewer for a narrower matrix) x 256 / 2^wide block rows.
template <typename T, bool NARROW>
__global__ __launch_bounds__(256) void l1_gap_kernel(const T *__restrict__ W, int64_t ldw, int br, int bq, int narrow,
                                                     double *__restrict__ gap)
{
    const int wide = NARROW ? narrow : 6;
    const unsigned tiles_q = ((unsigned)bq + (1u << wide) - 1u) >> wide, tile = blockIdx.x;
    const int bj = (int)(((tile % tiles_q) << wide) + (threadIdx.x & ((1u << wide) - 1u)));
    const int bi = (int)((tile / tiles_q) * (256u >> wide) + (threadIdx.x >> wide));
    if (bi >= br || bj >= bq) return;
    gap[(int64_t)bi * bq + bj] = block_gap(W, ldw, bi, bj);
}

// Shape and dtype are checked first; an empty matrix (r or q zero) is accepted
// whatever the pointers are, since nothing will be read or written.
int check_weight(const void *W, int dt, int64_t r, int64_t q, int64_t ldw, int64_t gran)
{
    S24_REQUIRE(s24_valid_dtype(dt), S24_ERR_DTYPE);
    S24_REQUIRE(r >= 0 && q >= 0 && r % gran == 0 && q % gran == 0 && ldw >= q, S24_ERR_SHAPE);
    S24_REQUIRE(r / 4 < (1ll << 30) && q / 4 < (1ll << 30), S24_ERR_SHAPE);
    if (r == 0 || q == 0) return S24_OK;
    S24_REQUIRE(W != nullptr, S24_ERR_NULL);
    const size_t row_bytes = dt == S24_F32 ? 16 : 8;  // one block row is loaded as a single vector
    S24_REQUIRE(s24_aligned(W, row_bytes) && (ldw * s24_elem_size(dt)) % row_bytes == 0, S24_ERR_ALIGN);
    return S24_OK;
}

}  // namespace

extern "C" int s24_transposable_mask(const void *W, s24_dtype dt, int64_t r, int64_t q, int64_t ldw, uint16_t *mask,
                                     uint8_t *index, void *stream)
{
    const int rc = check_weight(W, dt, r, q, ldw, 4);
    if (rc != S24_OK || r == 0 || q == 0) return rc;
    S24_REQUIRE(mask != nullptr, S24_ERR_NULL);
    MaskBatch batch{};
    batch.w[0] = MaskWeight{W, ldw, (int)(r / 4), (int)(q / 4), nullptr, mask, index, nullptr, nullptr, nullptr, nullptr};
    return launch(batch, 1, dt, false, static_cast<hipStream_t>(stream));
}

extern "C" int s24_compress(const void *W, s24_dtype dt, int64_t r, int64_t q, int64_t ldw, const uint16_t *mask,
                            void *vals, uint16_t *meta, void *valsT, uint16_t *metaT, uint16_t *mask_out, void *stream)
{
    const s24_compress_problem problem{W, mask, vals, meta, valsT, metaT, mask_out, r, q, ldw};
    return s24_compress_batch(&problem, 1, dt, stream);
}

extern "C" int s24_compress_batch(const s24_compress_problem *problems, int count, s24_dtype dt, void *stream)
{
    S24_REQUIRE(s24_valid_dtype(dt), S24_ERR_DTYPE);
    S24_REQUIRE(count >= 0 && count <= kMaxWeights, S24_ERR_SHAPE);
    if (count == 0) return S24_OK;
    S24_REQUIRE(problems != nullptr, S24_ERR_NULL);
    MaskBatch batch{};
    int used = 0;
    for (int i = 0; i < count; ++i) {   // every weight is checked before anything is launched
        const s24_compress_problem &pr = problems[i];
        const int rc = check_weight(pr.W, dt, pr.r, pr.q, pr.ldw, 64);
        if (rc != S24_OK) return rc;
        if (pr.r == 0 || pr.q == 0) continue;
        S24_REQUIRE(pr.vals && pr.meta && pr.valsT && pr.metaT, S24_ERR_NULL);
        // the kernel stores 16 bytes of values and 8 bytes of index words at a time (and the GEMMs that consume the
        // operands copy them in 16-byte pieces)
        S24_REQUIRE(s24_aligned(pr.vals, 16) && s24_aligned(pr.valsT, 16) && s24_aligned(pr.meta, 8) && s24_aligned(pr.metaT, 8) &&
                        s24_aligned(pr.mask, 2) && s24_aligned(pr.mask_out, 2),
                    S24_ERR_ALIGN);
        // a given mask is not written back
        batch.w[used] = MaskWeight{pr.W, pr.ldw, (int)(pr.r / 4), (int)(pr.q / 4), pr.mask, pr.mask ? nullptr : pr.mask_out, nullptr,
                                   pr.vals, pr.meta, pr.valsT, pr.metaT};
        S24_REQUIRE((batch.w[used].mask_in == nullptr) == (batch.w[0].mask_in == nullptr), S24_ERR_UNSUPPORTED);
        ++used;
    }
    return used ? launch(batch, used, dt, true, static_cast<hipStream_t>(stream)) : S24_OK;
}

extern "C" int s24_mask_flips(const uint16_t *mask_new, const uint16_t *mask_old, int64_t nblocks, uint32_t *block_flips,
                              uint64_t *flips, void *stream)
{
    S24_REQUIRE(nblocks >= 0, S24_ERR_SHAPE);
    S24_REQUIRE(flips != nullptr, S24_ERR_NULL);
    S24_REQUIRE(s24_aligned(flips, 8), S24_ERR_ALIGN);
    if (nblocks > 0) {
        S24_REQUIRE(mask_new && mask_old, S24_ERR_NULL);
        S24_REQUIRE(s24_aligned(mask_new, 16) && s24_aligned(mask_old, 16) && s24_aligned(block_flips, 4), S24_ERR_ALIGN);
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    auto *total = reinterpret_cast<unsigned long long *>(flips);
    hipLaunchKernelGGL(clear_counter_kernel, dim3(1), dim3(1), 0, st, total);
    if (nblocks > 0) {
        const int64_t vecs = (nblocks + 7) / 8;
        // One vector per lane up to a quarter of a workgroup per compute unit, beyond that four, in at most a workgroup per
        // compute unit: the atomics on the one counter take 17 ns each, one after the other (one vector per lane and up to 1024
        // workgroups: 409600 blocks 6.1 -> 4.6 us, 2.8 M 17.0 -> 8.4, 14.7 M 22.9 -> 14.8; four vectors per lane from the
        // first: 12288 blocks 4.0 -> 4.4).  With per-block counts a vector is eight counters read and written: one per lane up
        // to a workgroup per compute unit (12288 blocks: 4.6 against 5.9 with four), two from 4 M blocks on (14.7 M: 43 us
        // against 52 with one workgroup and 48 with four per compute unit; 2.8 M: 13.5 with one, 14.3 with two).
        const int64_t cus = s24_cu_count(), full = (vecs + 255) / 256;
        const unsigned grid = (unsigned)(block_flips != nullptr ? std::min(full, vecs < 2048 * cus ? cus : 2 * cus)
                                         : full <= cus / 4      ? full
                                                                : std::min((vecs + 1023) / 1024, cus));
        hipLaunchKernelGGL(mask_flips_kernel, dim3(grid), dim3(256), 0, st, mask_new, mask_old, nblocks, block_flips, total);
    }
    return s24_launch_status();
}

extern "C" int s24_l1_norm_gap(const void *W, s24_dtype dt, int64_t r, int64_t q, int64_t ldw, double *gap, void *stream)
{
    const int rc = check_weight(W, dt, r, q, ldw, 4);
    if (rc != S24_OK || r == 0 || q == 0) return rc;
    S24_REQUIRE(gap != nullptr, S24_ERR_NULL);
    S24_REQUIRE(s24_aligned(gap, 8), S24_ERR_ALIGN);
    const int br = (int)(r / 4), bq = (int)(q / 4);
    int wide = 0;
    while (wide < 6 && (1 << wide) < bq) ++wide;
    hipStream_t st = static_cast<hipStream_t>(stream);
    // A launch takes as many rows of tiles as make at most 2^23 workgroups: it holds less than 2^32 work items (of more it
    // silently runs the remainder).
    const int64_t height = 256 >> wide, tiles_q = ((int64_t)bq + (1 << wide) - 1) >> wide, step = height * std::max<int64_t>(1, (1 << 23) / tiles_q);
    for (int64_t b0 = 0; b0 < br; b0 += step) {
        const int rows = (int)std::min<int64_t>(br - b0, step);
        const dim3 grid((unsigned)(tiles_q * ((rows + height - 1) / height))), block(256);
        auto launch_gap = [&](auto t) {
            using T = decltype(t);
            const T *w = static_cast<const T *>(W) + 4 * b0 * ldw;
            if (wide < 6) hipLaunchKernelGGL((l1_gap_kernel<T, true>), grid, block, 0, st, w, ldw, rows, bq, wide, gap + b0 * bq);
            else hipLaunchKernelGGL((l1_gap_kernel<T, false>), grid, block, 0, st, w, ldw, rows, bq, wide, gap + b0 * bq);
        };
        if (dt == S24_BF16) launch_gap(uint16_t{});
        else if (dt == S24_F16) launch_gap(s24_half{});
        else launch_gap(float{});
    }
    return s24_launch_status();
}
