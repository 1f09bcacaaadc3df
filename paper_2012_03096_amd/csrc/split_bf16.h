// fp32 operands written exactly as sums of three bf16 terms, for products on the bf16 matrix cores (the arithmetic and
// its error bound: conv_split_kernel.h).
#pragma once
#include <hip/hip_runtime.h>

namespace pbkd {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
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

// x0, x1 -> their two fp16 pieces, packed: x = p0 + p1 to within 2^-22 |x| (2^-24 rms) or half an fp16 subnormal step,
// 2^-25, whichever is larger; |x| < 65520
__device__ __forceinline__ void split2_f16(float x0, float x1, unsigned (&p)[2]) {
  const f16x2 h = __builtin_convertvector((floatx2){x0, x1}, f16x2);
  p[0] = __builtin_bit_cast(unsigned, h);
#if defined(__HIP_DEVICE_COMPILE__)
  // x - h is exact in fp32, so the fused step that takes h as it is and rounds the difference to fp16 is the same as four
  // (back to fp32 and subtract, twice) and a conversion; the compiler does not form it
  unsigned l;
  asm("v_fma_mixlo_f16 %0, -%1, 1.0, %2 op_sel_hi:[1,0,0]" : "=v"(l) : "v"(p[0]), "v"(x0));
  asm("v_fma_mixhi_f16 %0, -%1, 1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "+v"(l) : "v"(p[0]), "v"(x1));
  p[1] = l;
#endif
}

}  // namespace pbkd
