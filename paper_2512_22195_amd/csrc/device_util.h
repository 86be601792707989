// Small device helpers shared by every kernel file: bf16 rounding, loads through the global
// address space, agent-scope accesses and the arrival counter built on them.
#pragma once

#include "matkv_internal.h"

namespace matkv {
namespace dev {

typedef unsigned int u32x2v __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4v __attribute__((ext_vector_type(4)));

// fp32 -> bf16, round to nearest even on the bit pattern; NaN stays NaN
__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// Two floats to two bf16, as f32_to_bf16_rne rounds them (the hardware conversion).
__device__ __forceinline__ uint32_t pack_bf16(float x, float y) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x, y}, bf16x2));
}

// 16-byte load through the global address space (a pointer rebuilt from an integer would
// otherwise be treated as generic and loaded with the slower flat instructions).
__device__ __forceinline__ uint4 ldg16(const void* p) {
    typedef const __attribute__((address_space(1))) u32x4v* gptr;
    const u32x4v r = *(gptr)(uintptr_t)p;
    return make_uint4(r.x, r.y, r.z, r.w);
}

// 8-byte load through the global address space.
__device__ __forceinline__ uint2 ldg8(const void* p) {
    typedef const __attribute__((address_space(1))) u32x2v* gptr;
    const u32x2v r = *(gptr)(uintptr_t)p;
    return make_uint2(r.x, r.y);
}

// ---- global memory straight into LDS ------------------------------------------------------------
// One instruction moves 16 bytes per lane from sbase + voff (voff: per-lane byte offset) to LDS
// bytes lds + 16 * lane (lds: byte address, the same in every lane).  No register holds the data,
// so what is in flight is bounded by LDS alone, and the copy counts like a load: in order, on
// vmcnt.  The compiler does not see these copies: dma_wait<N>() - all but the wave's N youngest
// copies have landed - and a barrier stand between a copy and the reads of its bytes by any wave,
// and a barrier between those reads and the next copy onto the same bytes.
__device__ __forceinline__ void dma16(const void* sbase, uint32_t voff, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds), "v"(voff), "s"(sbase) : "memory", "m0");
}
template <int N>
__device__ __forceinline__ void dma_wait() {
    static_assert(N >= 0 && N <= 63, "vmcnt has six bits");
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}
// Byte address of an LDS object, as dma16 takes it (the object counts as written from here on).
__device__ __forceinline__ uint32_t lds_address(void* p) {
    typedef __attribute__((address_space(3))) char* lptr;
    return (uint32_t)(uintptr_t)(lptr)p;
}

// Agent-scope relaxed accesses: coherent across the chip's L2 slices without cache flushes.
__device__ __forceinline__ void st_agent2(float* p, float x, float y) {
    const uint64_t v = (uint64_t)__float_as_uint(x) | ((uint64_t)__float_as_uint(y) << 32);
    __hip_atomic_store(reinterpret_cast<uint64_t*>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 ld_agent2(const float* p) {
    const uint64_t r = __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return make_float2(__uint_as_float((uint32_t)r), __uint_as_float((uint32_t)(r >> 32)));
}
// 16 bytes the same way, `off` bytes behind a wave-uniform address (no such atomic load exists; the cache policy is that of the one above).
__device__ __forceinline__ float4 ld_agent4(const float* base, uint32_t off) {
    typedef float f32x4v __attribute__((ext_vector_type(4)));
    constexpr int kSc1 = 16;
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, 0xffffffffu, 0x00027000);
    const f32x4v v = __builtin_bit_cast(f32x4v, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, kSc1));
    return make_float4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ void st_agent4(void* base, uint32_t off, const uint4& v) {
    constexpr int kSc1 = 16;
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(base, 0, 0xffffffffu, 0x00027000);
    __builtin_amdgcn_raw_buffer_store_b128(u32x4v{v.x, v.y, v.z, v.w}, r, off, 0, kSc1);
}
// 16 bytes `off` bytes behind a wave-uniform address.  NT: not kept in the last-level cache (memory that is not read again before
// it would have been displaced there), and as a buffer load, which a large cache's walk is 0.5 % faster with; the ordinary
// load is 2 to 6 % faster where a step is short (8B shape, one user of 1000 tokens: eight layers 583 -> 569 us per pass of eight
// steps, 32 layers 10.7 -> 10.1 us per layer step).
template <bool NT>
__device__ __forceinline__ uint4 ld16_at(const void* base, uint32_t off) {
    if (!NT) return ldg16(reinterpret_cast<const char*>(base) + off);
    constexpr int kNt = 2;
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, 0xffffffffu, 0x00027000);
    const u32x4v v = __builtin_bit_cast(u32x4v, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, kNt));
    return make_uint4(v.x, v.y, v.z, v.w);
}

// One workgroup's arrival at a counter: every thread has waited for its own agent-scope stores,
// the barrier orders them before thread 0's ticket.  Returns true in every thread of the
// workgroup that arrived last of `expected`.
__device__ __forceinline__ bool arrive_at(int32_t* counter, int expected, int* sm_last) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
        const int prev = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *sm_last = (prev == expected - 1);
    }
    __syncthreads();
    return *sm_last != 0;
}
// The same for a wave: its own agent-scope stores are acknowledged before its ticket is drawn.  True in the wave that
// arrived last of `expected`, which also makes the counter ready for the next launch.
__device__ __forceinline__ bool wave_arrives_last(int32_t* counter, int expected) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_s_waitcnt(0);
    int prev = 0;
    if ((threadIdx.x & 63) == 0) prev = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (__builtin_amdgcn_readfirstlane(prev) != expected - 1) return false;
    if ((threadIdx.x & 63) == 0) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    return true;
}
// (by the workgroup that arrived last: ready for the next launch)
__device__ __forceinline__ void reset_counter_at(int32_t* counter) {
    if (threadIdx.x == 0) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace dev
}  // namespace matkv
