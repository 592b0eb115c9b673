// Pieces shared by the kernels that stream weights or cache entries through an LDS ring (gemm_wide.hip, gemm_proj.hip,
// attn_mfma.hip).
#pragma once
#include "common.hpp"

namespace sx {

constexpr int kProducers = 2;       // waves of a workgroup that only bring weights in

typedef __attribute__((address_space(3))) void* lds_ptr_t;

// s_waitcnt immediate that waits for vmcnt <= n only (gfx9 encoding: vmcnt in bits 3:0 and 15:14, expcnt 6:4 and
// lgkmcnt 11:8 left at their maxima)
constexpr int vmcnt_imm(int n) { return 0x0F70 | (n & 15) | (((n >> 4) & 3) << 14); }

// Direct global -> LDS load, 16 bytes per lane: lane l's bytes land at lds_base + 16 l (lds_base
// wave-uniform).  Written as an instruction rather than through the builtin so that the compiler does not put a full
// vector-memory wait in front of every later LDS read; the kernels pace these loads themselves with s_waitcnt vmcnt and a
// barrier.  "nt": the stream is read once.  m0 is written here and used by nothing else in these kernels.
__device__ __forceinline__ void load_to_lds16(const void* src, const void* lds_base) {
  const uint32_t l = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_ptr_t)lds_base));
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off nt" ::"s"(l), "v"(src) : "memory");
}

// The same with a wave-uniform base and a 32-bit byte offset per lane: the address arithmetic of a request is then
// scalar.  (A 64-bit address per lane is some 30 vector instructions; 16 of them per 32 KB take a producer wave as
// long as the memory takes to deliver them.)
__device__ __forceinline__ void load_to_lds16(const char* base, uint32_t off, const void* lds_base) {
  const uint32_t l = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_ptr_t)lds_base));
  const uint64_t b64 = reinterpret_cast<uint64_t>(base);   // uniform by construction: pin it to scalar registers
  const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(static_cast<uint32_t>(b64))));
  const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(static_cast<uint32_t>(b64 >> 32))));
  const uint64_t sb = static_cast<uint64_t>(lo) | (static_cast<uint64_t>(hi) << 32);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(l), "v"(off), "s"(sb) : "memory");
}

}  // namespace sx
