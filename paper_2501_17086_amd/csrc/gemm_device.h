// Device helpers shared by the matrix-core GEMM kernels: direct global -> LDS copies, counted waits, vector types and
// the activations of the forward epilogues.
#pragma once
#include "gelu.h"
#include "hbp_common.h"
#include <atomic>

namespace hbp {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef short short8v __attribute__((ext_vector_type(8)));
typedef float float16v __attribute__((ext_vector_type(16)));

__device__ uint4 g_zero_chunks[64];  // source of chunks past the end of the contraction (zero-initialised)

// 16 bytes per lane, global -> LDS at lds_base + lane * 16.  lds_base is
// wave-uniform.  The compiler does not see this write to LDS: callers order it
// against LDS reads with a counted wait + a workgroup barrier.
__device__ __forceinline__ void dma16(const void* gptr, unsigned lds_base) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off\n"
               :: "v"(gptr), "s"(lds_base) : "memory");
}
// the same with a wave-uniform 64-bit base and a 32-bit unsigned byte offset per lane
__device__ __forceinline__ void dma16_s(unsigned off, const void* sbase_in, unsigned lds_base) {
  // (the base is uniform by construction; say so where the register allocator has moved it to vector registers)
  const unsigned long long b = reinterpret_cast<unsigned long long>(sbase_in);
  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)b);
  const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(b >> 32));
  const unsigned long long u = (unsigned long long)lo | ((unsigned long long)hi << 32);
  const void* sbase = reinterpret_cast<const void*>(u);
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1\n"
               :: "v"(off), "s"(sbase), "s"(lds_base) : "memory");
}
// at most N vector-memory operations outstanding (N <= 63), and no LDS operation
template <int N>
__device__ __forceinline__ void wait_vm_lds() {
  __builtin_amdgcn_s_waitcnt(0x0070 | (N & 15) | ((N >> 4) << 14));
}
template <int N>
__device__ __forceinline__ void wait_vm() {
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// GELU and its derivative, on v_exp_f32 and v_rcp_f32
__device__ __forceinline__ void gelu_both(float a, float& z, float& dz) {
  gelu_pair(a, z, dz, [](float x) { return __builtin_amdgcn_exp2f(x); }, [](float x) { return __builtin_amdgcn_rcpf(x); });
}

// Raises a kernel's dynamic shared-memory limit once per device (one flag array per kernel instantiation; setting
// the attribute twice from two threads is harmless, so a relaxed flag is enough).
constexpr int MAX_DEVICES = 64;
inline hipError_t raise_lds_limit(const void* kern, int bytes, std::atomic<bool> (&done)[MAX_DEVICES]) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
  if (done[dev].load(std::memory_order_acquire)) return hipSuccess;
  e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e != hipSuccess) return e;
  done[dev].store(true, std::memory_order_release);
  return hipSuccess;
}

}  // namespace
}  // namespace hbp
