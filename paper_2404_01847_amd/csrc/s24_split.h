// How a contraction is dealt out among the waves of a workgroup.  Plain C++ without HIP, so that the arithmetic can be
// checked on the CPU at sizes that no test could allocate.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#define S24_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define S24_HOST_DEVICE inline
#endif

// Pairs of tokens, the last one alone where the count is odd (tokens + 1 may not fit an int)
S24_HOST_DEVICE int s24_token_pairs(int tokens) { return tokens / 2 + tokens % 2; }

// First of the n units that slice s of `slices` takes (slice s ends where slice s + 1 begins).  The product takes 64 bits:
// eight slices of 2^28 units are past an int.
S24_HOST_DEVICE int s24_slice_begin(int n, int s, int slices) { return (int)((int64_t)n * s / slices); }
