// Direct global -> LDS loads, explicit waits, and the operand types of the matrix cores.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace a3po {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t dma_u32x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void *lds_ptr_t;

// 16 bytes per lane from g to l + 16 * lane (l is the same for the whole wavefront)
__device__ __forceinline__ void dma16(const char *g, char *l)
{
    __builtin_amdgcn_global_load_lds(reinterpret_cast<const dma_u32x4_t *>(g), (lds_ptr_t)l, 16, 0, 0);
}

// The same through a buffer descriptor (off: byte offset per lane; at: one for the whole wavefront).  The compiler takes
// the global form for an access that may return out of order with ordinary loads and then waits for everything in
// flight, vmcnt(0), before the first use of a register that an ordinary load fills; the buffer form has no such effect.
// Reads at or beyond `bytes` return zeros.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t dma_buffer(const void *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t buffer, uint32_t off, uint32_t at, char *l)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(buffer, (lds_ptr_t)l, 16, (int)off, (int)at, 0, 0);
}

// Accesses to LDS beside a ring that direct loads fill (staging tiles, partial results).  The __restrict__ parameter puts each
// into an alias scope of its own; without one the compiler takes that LDS for a part of the ring and waits for the direct
// loads in flight.  (Such accesses keep their order among themselves: neither is said to be free of the other's scope.)
template <typename T>
__device__ __forceinline__ void lds_put(void *__restrict__ p, T v) { *reinterpret_cast<T *>(p) = v; }
template <typename T>
__device__ __forceinline__ T lds_get(const void *__restrict__ p) { return *reinterpret_cast<const T *>(p); }

// s_waitcnt with the given vector-memory and LDS counts (the export count is left alone)
__device__ __forceinline__ constexpr int waitcnt_imm(int vmcnt, int lgkmcnt)
{
    return 0x0070 | (vmcnt & 15) | ((vmcnt >> 4) << 14) | ((lgkmcnt & 15) << 8);
}
constexpr int kNoVmWait = 63, kNoLgkmWait = 15;

}  // namespace a3po
