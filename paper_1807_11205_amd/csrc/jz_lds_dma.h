// Building blocks of the kernels that bring their operands in with LDS-direct loads (jz_igemm_dma.h, jz_conv_f32.hip): the
// loads themselves, hand-placed waits, and compile-time loops.  Included inside a kernel file's anonymous namespace.
#pragma once

#define JZ_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))

// The host pass of hipcc parses these bodies too and has no AMDGPU register constraints, hence the guards.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
#endif
}
// Wait until at most KEEP LDS reads are outstanding ...
template <int KEEP>
__device__ __forceinline__ void lds_wait() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(KEEP));
#endif
}
// ... and tie an operand to that point: volatile asm statements keep their order, and an MFMA that consumes the
// "output" of this empty statement cannot be scheduled above it (hence not above the wait either).
template <class V>
__device__ __forceinline__ void lds_pin(V& v) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(v));
#endif
}

typedef __attribute__((address_space(3))) unsigned char lds_byte;
// one LDS-direct load: 64 lanes x 16 bytes from `rsrc` at per-lane byte offset `voff` to LDS at dst + lane * 16
__device__ __forceinline__ void jz_dma16(__amdgpu_buffer_rsrc_t rsrc, lds_byte* dst, unsigned voff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, dst, 16, (int)voff, 0, 0, 0);
}

// compile-time loop: f(std::integral_constant<int, I>{}) for I = B .. E-1 (immediates of inline assembly and the
// slot arithmetic of the schedule need constant expressions)
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}
// nothing may be moved across this point by the instruction scheduler
__device__ __forceinline__ void sched_fence() {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_sched_barrier(0);
#endif
}
// one LDS-direct load with the wave-uniform part of the offset in a scalar register
__device__ __forceinline__ void jz_dma16s(__amdgpu_buffer_rsrc_t rsrc, lds_byte* dst, unsigned voff, unsigned soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, dst, 16, (int)voff, (int)soff, 0, 0);
}

__device__ __forceinline__ unsigned xcd_remap(unsigned bid, unsigned nb) {
  // consecutive workgroup ids land on different XCDs (each with its own L2); give every XCD one
  // contiguous run of tiles instead so that neighbouring tiles share their operand rows in L2
  const unsigned X = 8;
  unsigned q = nb / X, rem = nb % X, xcd = bid % X, local = bid / X;
  return xcd * q + (xcd < rem ? xcd : rem) + local;
}
