// Device helpers shared by the FP64 MFMA kernels.
#pragma once
#include "internal.h"

typedef double d4 __attribute__((ext_vector_type(4)));
// last operand of the FP64 MFMA builtin: on CDNA3/CDNA4 its bits are the
// DGEMM negate modifiers of the A, B and C operands; 1 negates A
constexpr int kNegA = 1;

// complex value with the sign bit of its imaginary part xor-ed with sgn
// (0 or 0x80000000): the conjugate, or the value itself, without arithmetic
__device__ __forceinline__ cplx flip_im(cplx v, unsigned sgn) {
  v.y = __hiloint2double(__double2hiint(v.y) ^ (int)sgn, __double2loint(v.y));
  return v;
}
// element offset of batch bz (one or two batch indices)
__device__ __forceinline__ i64 boff(const GemmArgs& g, i64 bz, i64 s1, i64 s2) {
  if (g.nb2 <= 1) return bz * s1;
  return (bz / g.nb2) * s1 + (bz % g.nb2) * s2;
}
// 16 bytes per lane from global memory straight into LDS (the wave's 64
// elements land as one contiguous KiB)
__device__ __forceinline__ void dma16(const cplx* src, cplx* lds) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                   (__attribute__((address_space(3))) void*)lds, 16, 0, 0);
}
