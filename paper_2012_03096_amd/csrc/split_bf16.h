// fp32 operands written exactly as sums of three bf16 terms, for products on the bf16 matrix cores (the arithmetic and
// its error bound: conv_split_kernel.h).
#pragma once
#include <hip/hip_runtime.h>

namespace pbkd {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
typedef unsigned uintx2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

// two floats -> their nearest bf16, packed (low half = a)
__device__ __forceinline__ unsigned pack_bf16_rn(float a, float b) {
  const floatx2 v = {a, b};
  return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}

// 16 bytes per lane from a buffer straight into LDS: lane l lands 16 l bytes behind `lds`, which must be the same for
// the whole wave; soff likewise.  Completion counts as a vector-memory load's.
__device__ __forceinline__ void load16_to_lds(__amdgpu_buffer_rsrc_t r, char *lds, unsigned voff, unsigned soff) {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)lds, 16, voff, soff, 0, 0);
#endif
}

// x0, x1 -> their three pieces, packed: p[k] holds piece k of both (low half = x0's)
__device__ __forceinline__ void split3_bf16(float x0, float x1, unsigned (&p)[3]) {
  p[0] = pack_bf16_rn(x0, x1);
  const float r0 = x0 - __builtin_bit_cast(float, p[0] << 16);
  const float r1 = x1 - __builtin_bit_cast(float, p[0] & 0xffff0000u);
  p[1] = pack_bf16_rn(r0, r1);
  const float s0 = r0 - __builtin_bit_cast(float, p[1] << 16);
  const float s1 = r1 - __builtin_bit_cast(float, p[1] & 0xffff0000u);
  p[2] = pack_bf16_rn(s0, s1);
}

// the same with the first two pieces cut off instead of rounded: each piece the next eight bits of the number
__device__ __forceinline__ void split3_bf16_cut(float x0, float x1, unsigned (&p)[3]) {
  auto cut = [](float f) { return __builtin_bit_cast(float, __builtin_bit_cast(unsigned, f) & 0xffff0000u); };
  auto pair = [](float a, float b) { return __builtin_amdgcn_perm(__builtin_bit_cast(unsigned, b), __builtin_bit_cast(unsigned, a), 0x07060302u); };
  p[0] = pair(x0, x1);
  const float r0 = x0 - cut(x0), r1 = x1 - cut(x1);
  p[1] = pair(r0, r1);
  p[2] = pair(r0 - cut(r0), r1 - cut(r1));
}

}  // namespace pbkd
