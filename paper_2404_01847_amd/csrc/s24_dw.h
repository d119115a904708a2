// What the kernels of the 16-bit weight gradients share: the problems of a launch, and the layout in which an operand lies in LDS.
#pragma once
#include "s24_lds.h"

namespace s24_dw {
// One launch covers up to four weight gradients (DwBatch): their tiles share one grid, so that the compute units
// left idle by the last, partial round of one problem take tiles of the next.  The operands of a problem may be
// windows of larger matrices: M and N are the extents of the window's output, ldy, ldx and ldw the row strides
// (elements) of dY, of X and of dW / Wt (the mask's row stride is ldw / 4; a window starts at a multiple of four
// rows and columns).
struct DwWindow {
    const uint16_t *dY, *X, *Wt, *mask;
    float *dW;
    int T, M, N, ldy, ldx, ldw, tiles_m, tiles_n;
    float lambda;
};
constexpr int kMaxBatch = 4;
// Workgroups are dealt round-robin to the eight XCDs.  Each XCD takes, of every problem in turn, one contiguous
// eighth of its tile list: first_slot[i] .. first_slot[i+1]-1 are the positions in an XCD's own list that belong to
// problem i (unused entries repeat the total), so every problem is spread over all XCDs exactly as a launch of its
// own would spread it, and the workgroups resident on one XCD share operand rows in its L2.
struct DwBatch {
    DwWindow w[kMaxBatch];
    int first_slot[kMaxBatch + 1];
};

typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16 *lds_v4i16;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

// 16-byte slot of chunk c of token row t: c ^ tr_swizzle(t).  Rows of 384 bytes lie half a round of the banks apart, so the lowest bit of
// the row needs no part in it, and their 24 slots take an exchange within eight only.
template <int ROWB> __device__ __forceinline__ int tr_swizzle(int row)
{
    static_assert(ROWB % 256 == 0 || ROWB % 256 == 128, "rows of whole or half rounds of the banks");
    return (ROWB % 256 == 0 ? (row & 3) << 2 : (row & 2) << 1) ^ ((row >> 2) & 2);
}
template <int ROWB>
__device__ __forceinline__ int tr_off(int row, int col)
{
    return row * ROWB + (((col >> 3) ^ tr_swizzle<ROWB>(row)) << 4) + ((col & 7) << 1);
}
__device__ __forceinline__ v4i16 tr_half(const unsigned char *p) { return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16)(p)); }
__device__ __forceinline__ bf16x8 join(v4i16 lo, v4i16 hi)
{
    struct { v4i16 a, b; } t{lo, hi};
    return __builtin_bit_cast(bf16x8, t);
}
}  // namespace s24_dw
