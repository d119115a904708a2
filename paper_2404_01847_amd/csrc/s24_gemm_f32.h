// fp32 matrix products of the library (s24_gemm_f32.hip), called by the GEMM entry points after their checks.
#pragma once
#include "s24_common.h"
#include "s24_split.h"

enum S24F32Epilogue { S24_F32_PLAIN, S24_F32_ACT, S24_F32_GLU };

// Out[N][M] = beta * Out + B[N][K] . A^T (+ bias[M]); A compressed along K (Am != NULL: vals [K/64][M][32], meta) or
// dense [M][K] (Am == NULL).  ACT: H[N][M] = act(Out) beside it.  GLU: A stacks gate and up rows (M = 2F), H[N][F] =
// act(gate) * up.  `act` is the s24_act or the s24_gate.
struct S24F32Nt {
    const float *B, *Av;
    const uint16_t *Am;
    float *Out, *H;
    const float *bias;
    int64_t N, K, M;
    bool accum;
    S24F32Epilogue epilogue;
    int act;
};
int s24_f32_nt(const S24F32Nt &g, hipStream_t st);

// dW[M][N] = beta * dW + A^T X over T tokens (+ lambda * Wt where the mask prunes, Wt != NULL), for up to four problems
// in one grid.  A is dense dY [T][M] (Am == NULL) or compressed along the tokens (vals [T/64][M][32], meta).
struct S24F32TnProblem {
    const float *A, *X, *Wt;
    const uint16_t *Am, *mask;
    float *dW;
    int64_t T, M, N;
    float lambda;
};
int s24_f32_tn(const S24F32TnProblem *pr, int count, bool accum, hipStream_t st);

// Input gradient (sparse, overwritten, no epilogue) and weight gradients (dense dY, overwritten) in one launch, where that pays: false if it does
// not, and nothing was launched.  None of them may read or write what another one writes.
bool s24_f32_nt_tn(const S24F32Nt &g, const S24F32TnProblem *pr, int count, hipStream_t st, int &status);
