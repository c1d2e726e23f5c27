// Direct global-to-LDS loads, issued and waited for by hand.
// The compiler cannot tell which LDS reads depend on which of these loads and
// would wait for all of them before every read; written as assembly (they
// have no output register) they stay in flight across several K slices, and
// wait_barrier() states how many may.  Loads return in order, and the
// compiler's own waits count only its own loads, so they wait longer, never
// shorter, than they need.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dsp {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Buffer resource over [base, base + bytes), wave-uniform.
__device__ __forceinline__ u32x4 dma_rsrc(const void* base, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(base);
  u32x4 r;
  r[0] = __builtin_amdgcn_readfirstlane((uint32_t)a);
  r[1] = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
  r[2] = __builtin_amdgcn_readfirstlane(bytes);
  r[3] = 0x00020000u;
  // the readfirstlanes are vector instructions: a memory instruction may read
  // the scalar registers they write 5 wait states later, which the compiler does
  // not see to for assembly
  asm volatile("s_nop 4" : "+s"(r));
  return r;
}
// the same resource `add` bytes further (wave-uniform: scalar arithmetic)
__device__ __forceinline__ u32x4 dma_advance(u32x4 r, uint64_t add) {
  const uint64_t a = (((uint64_t)r[1] << 32) | r[0]) + add;
  r[0] = (uint32_t)a;
  r[1] = (uint32_t)(a >> 32);
  return r;
}
// 16 bytes per lane from rsrc + voff + soff to LDS address `at` + 16 lane
// (`at`, soff: wave-uniform).  m0 holds `at`; nothing else in these kernels uses
// it (it is a reserved register, which a clobber list may not name).
__device__ __forceinline__ void dma_b128(u32x4 rsrc, uint32_t voff, uint32_t soff, uint32_t at) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               :
               : "s"(at), "v"(voff), "s"(rsrc), "s"(soff)
               : "memory");
}
// at most N of this wave's loads in flight, all its LDS reads returned, then
// the work-group's barrier
template <int N>
__device__ __forceinline__ void wait_barrier() {
  static_assert(N < 64, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(N) : "memory");
}

}  // namespace
}  // namespace dsp
