// Copies from global memory straight into LDS and the layouts that the sparse products' operands take there.
#pragma once
#include "s24_common.h"

namespace s24_lds {
typedef __attribute__((address_space(3))) void *lds_ptr;
typedef const __attribute__((address_space(1))) void *glb_ptr;
// LDS handed to a device function: with the address space in its type the compiler keeps 32-bit addresses and LDS instructions
typedef __attribute__((address_space(3))) unsigned char lds_byte;
typedef __attribute__((address_space(3))) s24_u32x4 lds_u32x4;
__device__ __forceinline__ uint4 lds_load(const lds_byte *p) { return __builtin_bit_cast(uint4, *(const lds_u32x4 *)p); }
template <typename V> __device__ __forceinline__ void lds_store(lds_byte *p, V v)
{
    static_assert(sizeof(V) == 16, "sixteen bytes");
    *(lds_u32x4 *)p = __builtin_bit_cast(s24_u32x4, v);
}

__device__ __forceinline__ int b_slot(int row, int c) { return row * 128 + ((c ^ ((row >> 1) & 7)) << 4); }
__device__ __forceinline__ int a_swizzle(int row) { return -(row >> 2) & 3; }
__device__ __forceinline__ int a_slot(int row, int c) { return row * 64 + ((c ^ a_swizzle(row)) << 4); }

// Buffer descriptor for direct-to-LDS copies: base address in scalar registers, raw (unstructured) addressing, no
// bounds clamp that the kernels rely on (every offset they form is inside the operand and below 4 GB, which the host
// checks; the descriptor declares the full 4 GB of records).
// (The host pass of the compiler does not know these builtins: it sees empty bodies.)
#if defined(__HIP_DEVICE_COMPILE__)
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t buffer_of(const void *base)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, 0xFFFFFFFFu, 0x27000);
}
// BYTES (16 or 4) per lane from byte offset `voff` of the buffer to lds + 64 * BYTES * (lane's index in the wave)
template <int BYTES> __device__ __forceinline__ void buffer_to_lds(rsrc_t buf, lds_ptr lds, uint32_t voff)
{
    static_assert(BYTES == 16 || BYTES == 4, "copy width");
    if constexpr (BYTES == 16) __builtin_amdgcn_raw_ptr_buffer_load_lds(buf, lds, 16, voff, 0, 0, 0);
    else __builtin_amdgcn_raw_ptr_buffer_load_lds(buf, lds, 4, voff, 0, 0, 0);
}
// 8 bytes / 2 bytes into registers from byte offset voff (per lane) + soff (wave-uniform, a scalar register): a load
// whose address costs one vector register however many of them a wave issues in a row
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint2 buffer_load_8(rsrc_t buf, uint32_t voff, uint32_t soff)
{
    const u32x2_t v = __builtin_amdgcn_raw_buffer_load_b64(buf, (int)voff, (int)soff, 0);
    return make_uint2(v.x, v.y);
}
__device__ __forceinline__ uint32_t buffer_load_2(rsrc_t buf, uint32_t voff, uint32_t soff)
{
    return __builtin_amdgcn_raw_buffer_load_b16(buf, (int)voff, (int)soff, 0);
}
// 16 bytes; STREAM: past the caches (non-temporal)
template <bool STREAM> __device__ __forceinline__ uint4 buffer_load_16(rsrc_t buf, uint32_t voff)
{
    return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(buf, (int)voff, 0, STREAM ? 2 : 0));
}
#else
typedef const void *rsrc_t;
__device__ __forceinline__ rsrc_t buffer_of(const void *base) { return base; }
template <int BYTES> __device__ __forceinline__ void buffer_to_lds(rsrc_t, lds_ptr, uint32_t) {}
__device__ __forceinline__ uint2 buffer_load_8(rsrc_t, uint32_t, uint32_t) { return make_uint2(0, 0); }
__device__ __forceinline__ uint32_t buffer_load_2(rsrc_t, uint32_t, uint32_t) { return 0; }
template <bool STREAM> __device__ __forceinline__ uint4 buffer_load_16(rsrc_t, uint32_t) { return make_uint4(0, 0, 0, 0); }
#endif

// s_waitcnt immediate: vmcnt(n), lgkmcnt(0), expcnt unconstrained
__host__ __device__ constexpr int wait_vm_lgkm0(int n) { return (n & 15) | (7 << 4) | ((n >> 4) << 14); }

// Until at most VM of the wave's vector-memory operations are in flight: ahead of reads of what older ones copied into LDS.  (Left to
// itself the compiler waits for the copies that it believes to alias a read.  Where two ways through a kernel meet, it knows those of one way
// only and waits too little: never rely on it.)
template <int VM> __device__ __forceinline__ void wait_copies()
{
    static_assert(VM < 64, "the counter's range");
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0(VM) | 15 << 8);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
}

// Workgroup barrier that leaves up to VM vector-memory operations (direct-to-LDS copies of later
// chunks) in flight.  The raw wait and barrier instructions carry no memory semantics for the
// compiler, so they are fenced on both sides against reordering of LDS accesses, in the
// optimiser (empty asm with a memory clobber) and in the instruction scheduler.
// LDS_READS: whether the wave's own LDS reads have to be back as well.
template <int VM, bool LDS_READS = true>
__device__ __forceinline__ void wait_and_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0(VM) | (LDS_READS ? 0 : 15 << 8));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
}
}  // namespace s24_lds
