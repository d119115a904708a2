// Which weight gradients may share a grid.  Plain C++ without HIP, so that it can be checked on the CPU.
#pragma once
#include <stdint.h>

#include "s24.h"

// True if the gradient of one problem overlaps a buffer of another (its gradient, operands, weight or mask), so that the
// result depends on the order of the two.  esize: bytes of an operand's element.
inline bool s24_dw_problems_overlap(const s24_dw_problem *problems, int count, int64_t esize)
{
    for (int i = 0; i < count; ++i) {
        const s24_dw_problem &w = problems[i];
        const uintptr_t begin = reinterpret_cast<uintptr_t>(w.dW), end = begin + (uintptr_t)(w.r * w.q) * 4;
        if (begin == end) continue;
        for (int j = 0; j < count; ++j) {
            const s24_dw_problem &o = problems[j];
            const int64_t cells = o.r * o.q;
            if (j == i || cells == 0) continue;   // nothing of an empty output's problem is read
            auto meets = [&](const void *p, int64_t bytes) {
                const uintptr_t a = reinterpret_cast<uintptr_t>(p);
                return bytes > 0 && a < end && begin < a + (uintptr_t)bytes;
            };
            if (meets(o.dW, cells * 4) || meets(o.dY, o.p * o.r * esize) || meets(o.X, o.p * o.q * esize)) return true;
            if (o.W != nullptr && (meets(o.W, cells * esize) || meets(o.mask, cells / 16 * 2))) return true;
        }
    }
    return false;
}

// True if the input gradient dX [p][q] = dY [p][r] (M.*W) (W compressed: valsT, metaT) and some of the problems cannot run at once: one
// writes what the other reads or writes.
inline bool s24_dx_meets_dw(const void *dY, const void *valsT, const void *metaT, const void *dX, int64_t p, int64_t q, int64_t r, const s24_dw_problem *problems,
                            int count, int64_t esize)
{
    auto meet = [](const void *a, int64_t na, const void *b, int64_t nb) {
        const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
        return a != nullptr && b != nullptr && na > 0 && nb > 0 && x < y + (uintptr_t)nb && y < x + (uintptr_t)na;
    };
    const int64_t dx = p * q * esize;
    for (int i = 0; i < count; ++i) {
        const s24_dw_problem &o = problems[i];
        const int64_t cells = o.r * o.q;
        if (cells == 0) continue;
        if (meet(dX, dx, o.dW, cells * 4) || meet(dX, dx, o.dY, o.p * o.r * esize) || meet(dX, dx, o.X, o.p * o.q * esize)) return true;
        if (o.W != nullptr && (meet(dX, dx, o.W, cells * esize) || meet(dX, dx, o.mask, cells / 16 * 2))) return true;
        if (meet(o.dW, cells * 4, dY, p * r * esize) || meet(o.dW, cells * 4, valsT, r * q / 2 * esize) || meet(o.dW, cells * 4, metaT, r * q / 8)) return true;
    }
    return false;
}
