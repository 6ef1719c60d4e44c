// Buffer loads whose destination is LDS: operands do not pass through registers on their way in.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hydra {

typedef __attribute__((ext_vector_type(4))) unsigned int rsrc_u32x4;

// 128-bit buffer descriptor (base, stride 0, size in bytes, raw dword format) for bytes [first, total) of a matrix;
// reads beyond it return zero
__device__ __forceinline__ rsrc_u32x4 rsrc_words(const void* base, long first, long total) {
  long rem = total - first;
  rem = rem < 0 ? 0 : (rem > 0x7fffffffL ? 0x7fffffffL : rem);
  const uint64_t p = (uint64_t)(uintptr_t)base + (uint64_t)(rem > 0 ? first : 0);
  rsrc_u32x4 r;
  r.x = __builtin_amdgcn_readfirstlane((unsigned)p);
  r.y = __builtin_amdgcn_readfirstlane((unsigned)(p >> 32) & 0xffffu);
  r.z = __builtin_amdgcn_readfirstlane((unsigned)rem);
  r.w = 0x00020000u;
  return r;
}
// A descriptor whose words a vector instruction (readfirstlane) may have written just before: a load may read them five wait states later on
// gfx9, which the compiler counts for its own loads, not for those in the asm blocks below.  Where the words are worked out by the scalar
// unit, or long before, nothing is to be waited for (in the attention kernels these states cost 0.5 to 0.8 %); a test looks at every such
// load of the built library.
__device__ __forceinline__ rsrc_u32x4 rsrc_settled(rsrc_u32x4 r) {
  asm("s_nop 4" : "+s"(r));
  return r;
}
// One wave-wide load of 16 bytes per lane from a buffer into LDS: lane l's bytes land at lds_addr + 16 l (lds_addr is
// a byte address inside the workgroup's LDS, uniform over the wave).  The compiler does not see the LDS write:
// callers order it against LDS reads with an explicit vmcnt wait and a barrier.  A load into LDS must not issue right behind the write
// of its M0: one wait state stands between them on gfx9, which the compiler puts in for its own loads but not inside an asm block.
__device__ __forceinline__ void load_to_lds_b128(rsrc_u32x4 rs, unsigned lds_addr, unsigned voff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds_addr), "v"(voff), "s"(rs) : "m0");
}
// The same with 4 bytes per lane: lane l's at lds_addr + 4 l
__device__ __forceinline__ void load_to_lds_b32(rsrc_u32x4 rs, unsigned lds_addr, unsigned voff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds" ::"s"(lds_addr), "v"(voff), "s"(rs) : "m0");
}

}  // namespace hydra
