"""The sliced products copy their tokens into LDS and read them without a barrier: a wave waits for its own copies by their number.  Here the
tile runs on the CPU, a lane at a time, on a memory whose copies land only when a wait of the kernel's own says so: each read has to find the
chunk that is due.  (On the device the compiler adds waits of its own; which ones, depends on how it sees the ways through the kernel meet.)"""
import ctypes as C
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"

RUNTIME = """
#pragma once
#include <math.h>
#include <stddef.h>
#include <stdint.h>
#include <algorithm>
using std::max; using std::min;
#define __device__
#define __host__
#define __global__
#define __forceinline__ inline
struct float2 { float x, y; }; struct float4 { float x, y, z, w; };
struct uint2 { unsigned x, y; }; struct alignas(16) uint4 { unsigned x, y, z, w; };
inline uint2 make_uint2(unsigned x, unsigned y) { return {x, y}; }
inline uint4 make_uint4(unsigned x, unsigned y, unsigned z, unsigned w) { return {x, y, z, w}; }
inline float __uint_as_float(uint32_t u) { return __builtin_bit_cast(float, u); }
inline float __fmaf_rn(float a, float b, float c) { return fmaf(a, b, c); }
typedef void *hipStream_t;
enum { hipSuccess, hipDeviceAttributeMultiprocessorCount };
inline int hipGetDevice(int *) { return 1; }
inline int hipDeviceGetAttribute(int *, int, int) { return 1; }
inline int hipGetLastError() { return 0; }
extern struct Thread { unsigned x; } threadIdx;
inline void __syncthreads() {}
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define __builtin_amdgcn_exp2f(x) exp2f(x)
#define __builtin_amdgcn_sched_barrier(x) ((void)0)
#define __builtin_amdgcn_s_barrier() ((void)0)
#define __builtin_amdgcn_s_waitcnt(x) ((void)0)
#define __builtin_amdgcn_readfirstlane(x) (x)
inline int products = 0;
template <typename A, typename B, typename V> V product(A, B, V c) { ++products; return c; }
#define __builtin_amdgcn_smfmac_f32_16x16x64_bf16(a, b, c, i, x, y) product(a, b, c)
#define __builtin_amdgcn_smfmac_f32_16x16x64_f16(a, b, c, i, x, y) product(a, b, c)
"""

HARNESS = """
#include <deque>
#include <map>
#include <vector>
#include "s24_gemm_slice.h"
#include "s24_lds.h"
using namespace s24_lds;
Thread threadIdx;
static const char *tokens;
struct Op { uintptr_t lds; int chunk; };   // chunk < 0: a load into registers
static std::deque<Op> flight;
static std::map<uintptr_t, int> landed;
static std::vector<int> seen;
static int early, parked;
template <int BYTES> void copy(rsrc_t from, lds_ptr to, uint32_t) { flight.push_back({(uintptr_t)to, (int)(((const char *)from - tokens) / 128)}); }
template <bool STREAM> uint4 load16(rsrc_t, uint32_t) { flight.push_back({0, -1}); return {}; }
inline uint32_t load2(rsrc_t, uint32_t, uint32_t) { flight.push_back({0, -1}); return 0; }
template <int VM> void wait()
{
    for (; flight.size() > VM; flight.pop_front())
        if (flight.front().chunk >= 0) landed[flight.front().lds] = flight.front().chunk;
}
inline uint4 read(const lds_byte *p)
{
    if (parked) return {};
    const uintptr_t at = (uintptr_t)p;
    auto it = landed.upper_bound(at);
    int chunk = -1;
    if (it != landed.begin() && at < (--it)->first + 1024) chunk = it->second;
    for (const Op &o : flight) early += o.chunk >= 0 && o.lds <= at && at < o.lds + 1024;
    seen.push_back(chunk);
    return {};
}
template <typename V> void write(lds_byte *, V) { for (const Op &o : flight) early += o.chunk >= 0; parked = 1; }
#define buffer_to_lds copy
#define buffer_load_16 load16
#define buffer_load_2 load2
#define wait_copies wait
#define lds_load read
#define lds_store write
#include "s24_slice_tile.h"
template <typename T, int TM, int TN> int run(int chunks, int wave, int lane)
{
    const int N = 16 * TN, M = 16 * TM, K = 64 * chunks;
    std::vector<uint16_t> out(N * M);
    std::vector<unsigned char> lds(4 * s24_slice::stage_bytes(4) + 1024);
    lds_byte *s = (lds_byte *)(((uintptr_t)lds.data() + 1023) & ~(uintptr_t)1023);
    constexpr int STAGE = s24_slice::stage_bytes(TN);
    static uint16_t dummy;
    tokens = (const char *)&dummy;
    flight.clear(); landed.clear(); seen.clear();
    early = parked = products = 0;
    threadIdx.x = 64 * wave + lane;
    s24_slice::slice_tile<T, false, S24_SLICE_PLAIN, 0, TM, TN, false>(s, s + STAGE, s + 2 * STAGE, s + 3 * STAGE, 0, &dummy, &dummy, &dummy, N, K, M, M, 1, 1, out.data(), nullptr, nullptr, nullptr);
    std::vector<int> want;
    int steps = 0;
    for (int c = wave; c < chunks; c += s24_slice::KS, ++steps) want.insert(want.end(), 2 * TN, c);
    return early != 0 ? 1 : seen != want ? 2 : products != steps * TM * TN ? 3 : !parked ? 4 : 0;
}
extern "C" int run_slice(int half, int tm, int tn, int chunks, int wave, int lane)
{
    auto with = [&](auto t) {
        using T = decltype(t);
        if (tn == 1) return tm == 1 ? run<T, 1, 1>(chunks, wave, lane) : tm == 2 ? run<T, 2, 1>(chunks, wave, lane) : run<T, 4, 1>(chunks, wave, lane);
        return tn == 2 ? run<T, 4, 2>(chunks, wave, lane) : run<T, 4, 4>(chunks, wave, lane);
    };
    return half ? with(s24_half{}) : with(uint16_t{});
}
"""


@pytest.fixture(scope="module")
def tile(tmp_path_factory):
    if not os.path.exists(CLANG):
        assert not os.path.exists("/opt/rocm/bin/hipcc"), "a compiler without its clang++: the waits go unchecked"
        pytest.skip("no clang++")
    d = tmp_path_factory.mktemp("slice")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(RUNTIME)
    (d / "tile.cpp").write_text(HARNESS)
    so = str(d / "tile.so")
    subprocess.run([CLANG, "-O1", "-std=c++17", "-shared", "-fPIC", "-w", "-I", str(d), "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2404_01847_amd", "csrc"), str(d / "tile.cpp"), "-o", so], check=True)
    return C.CDLL(so)


@pytest.mark.parametrize("half", [0, 1])
@pytest.mark.parametrize("tm, tn", [(1, 1), (2, 1), (4, 1), (4, 2), (4, 4)])
def test_every_read_of_a_slice_follows_the_wait_for_its_copy(tile, half, tm, tn):
    # no chunk to a wave up to thirteen: the short way, the long one from as many chunks as there are stages, and each of its remainders
    bad = {(n, w): r for n in (*range(1, 100), 104) for w in range(8) if (r := tile.run_slice(half, tm, tn, n, w, (7 * n) % 64))}
    assert not bad, "1: read or parked over before it landed, 2: another chunk, 3: not all multiplied, 4: never parked"
