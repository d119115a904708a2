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
double s24_slice_us(int64_t N, int64_t K, int64_t M);   // what it takes while its operands are in the caches
// Row blocks of the best tile with one token block, if it costs no more than 1.3 of the best of all
bool s24_slice_narrow_tile(int64_t N, int64_t K, int64_t M, int &tm);
int s24_slice_nt(const S24SliceNt &g, int dt, hipStream_t st);
