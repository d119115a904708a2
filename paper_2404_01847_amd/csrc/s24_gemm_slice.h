// Sparse NT products whose output is too small to fill the chip (s24_gemm_slice.hip), called by the GEMM entry points
// after their checks.  bf16 and binary16 operands.
#pragma once
#include "s24_common.h"

enum S24SliceEpilogue { S24_SLICE_PLAIN, S24_SLICE_ACT, S24_SLICE_GLU, S24_SLICE_ACT_BWD };

// Out[N][M] = beta * Out + B[N][K] . A^T (+ bias[M]); A compressed along K (vals [K/64][M][32], meta [K/64][M][4]).
// ACT: H[N][M] = act(Out) beside it.  GLU: A stacks gate and up rows (M = 2F), H[N][F] = act(gate) * up.
// ACT_BWD: Out = (rounded product) * act'(Z), Z [N][M].  `act` is the s24_act or the s24_gate.
struct S24SliceNt {
    const uint16_t *B, *Av, *Am;
    uint16_t *Out, *H;
    const uint16_t *Z, *bias;
    int64_t N, K, M;
    bool accum;
    S24SliceEpilogue epilogue;
    int act;
};
// Tile of a product, 16 tm features x 16 tn tokens, and what it takes in us while its operands are in the caches; tm = 0: not in slices
struct S24SlicePlan {
    int tm, tn;
    double us;
    explicit operator bool() const { return tm != 0; }
};
S24SlicePlan s24_slice_plan(int64_t N, int64_t K, int64_t M, int max_tn = 4);
int s24_slice_nt(const S24SliceNt &g, const S24SlicePlan &p, int dt, hipStream_t st);
