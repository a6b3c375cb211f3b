// Loads from global memory straight into LDS, shared by the kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pctree {

// 16 bytes per lane from global memory straight into LDS (lane l's bytes at
// lds_dst + 16 l), counted in vmcnt like any vector-memory load.  Issued as
// inline assembly: the compiler does not see the LDS write, so it does not
// make later LDS reads wait for every load in flight (it cannot tell the
// buffers apart); the kernels order them themselves with a vmcnt wait and,
// between waves, a barrier.  M0 holds the LDS base; nothing else in the kernels
// that use it keeps a value in M0 across it.  A load into LDS needs one wait
// state after a scalar write of M0, which the compiler places around its own
// instructions only: the s_nop (without it the load may use the M0 before).
__device__ __forceinline__ uint32_t lds_base(const void* lds_dst) {
  return __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)lds_dst);
}
__device__ __forceinline__ void load_lds16(const void* src, const void* lds_dst) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src),
               "s"(lds_base(lds_dst))
               : "memory", "m0");
}
// The same with a uniform base and the lane's byte offset.
__device__ __forceinline__ void load_lds16(const void* base, uint32_t off, const void* lds_dst) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %2" ::"v"(off),
               "s"(lds_base(lds_dst)), "s"(base)
               : "memory", "m0");
}

}  // namespace pctree
