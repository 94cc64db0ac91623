// Direct loads from memory to LDS (no registers in between).
#pragma once

#include "bmm_internal.h"

namespace bmm {

// 16 bytes per lane from base + voff to LDS at lds + 16 * lane (base and lds uniform).
// The compiler does not see them: the caller waits for vmcnt before anyone
// reads them.  m0, which they change, is an output, so the compiler knows that they do.
// Global addresses need
// 8-byte alignment only, which rows of odd pitch have.
__device__ __forceinline__ void load_lds16(const void* base, uint32_t voff, uint32_t lds) {
  uint32_t m0;
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3"
               : "={m0}"(m0)
               : "s"(lds), "v"(voff), "s"(base)
               : "memory");
}

__device__ __forceinline__ void load_lds16(const void* addr, uint32_t lds) {
  uint32_t m0;
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, off"
               : "={m0}"(m0)
               : "s"(lds), "v"(addr)
               : "memory");
}

}  // namespace bmm
