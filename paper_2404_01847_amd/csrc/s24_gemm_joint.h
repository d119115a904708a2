// An input gradient and weight gradients in one launch (s24_gemm_joint.hip), called by the GEMM entry points after their checks.
#pragma once
#include "s24_dw.h"
#include "s24_gemm_slice.h"

// g (plain, overwritten) in slices of 16 tm features x 16 tokens, beside the gradients of `batch` (windows in tiles of 128 x 128, overwritten).
void s24_dx_dw(const S24SliceNt &g, int tm, const s24_dw::DwBatch &batch, bool decay, int dt, hipStream_t st);
