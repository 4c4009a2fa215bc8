// Operands of v_mfma_f32_16x16x32_bf16 from the blob's packed slices: the 2-bit field of a weight OR-ed into the mantissa
// of a bf16 power of two.  Shared by the kernels that multiply slice by slice in bf16.
#pragma once

#include "mbq_common.h"

namespace mbq {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

namespace bf {

__device__ inline floatx4 mfma(const uint4& a, const uint4& b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b),
                                                 c, 0, 0, 0);
}

template <int R>
__device__ inline uint32_t rotr(uint32_t w) {
  if constexpr (R == 0) return w;
  return __builtin_amdgcn_alignbit(w, w, R);
}

// bf16 pairs of 2^5, 2^3, 2^1, 2^-1
constexpr uint32_t kPow5 = 0x42004200u, kPow3 = 0x41004100u, kPow1 = 0x40004000u, kPowM1 = 0x3F003F00u;

// Unpack constants kept in registers.  (t & mask) | bias is one v_and_or_b32 only when neither
// operand is a literal (a VOP3 instruction cannot carry one on gfx9), so the three field masks live
// in scalar registers and the four bf16-pair biases 2^5, 2^3, 2^1, 2^-1 in vector registers; both are
// made opaque to constant folding once, at kernel entry.
struct UnpackConsts {
  uint32_t mask[3];  // 0x00030003 << 0, 2, 4
  uint32_t bias[4];
};

__device__ inline UnpackConsts make_unpack_consts() {
  UnpackConsts c;
  c.mask[0] = 0x00030003u; c.mask[1] = 0x000C000Cu; c.mask[2] = 0x00300030u;
  c.bias[0] = kPow5; c.bias[1] = kPow3; c.bias[2] = kPow1; c.bias[3] = kPowM1;
#pragma unroll
  for (int i = 0; i < 3; ++i) asm volatile("" : "+s"(c.mask[i]));
#pragma unroll
  for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(c.bias[i]));
  return c;
}

// B operands (a-step, b-step) of the two k-steps held by one dword of slice E.
// The unrotated field of (step, slot s = 2j + h) sits at bit 16h + 4j + 2 step; slice E is
// stored rotated left by 2 - 2E.  Slice 0 is consumed one field position up (no rotation
// for j = 0); its bias exponents are lowered accordingly.  Operand values:
//   slice 0: 32 + c, 8 + c          slice 1: 32 + c/4, 8 + c/4
//   slice 2: 8 + c/16, 2 + c/16     slice 3: 2 + c/64, 0.5 + c/64
template <int E>
__device__ inline void unpack_dword(uint32_t w, const UnpackConsts& uc, uint4& Ba, uint4& Bb) {
  constexpr int rho = (2 - 2 * E) & 31;
  constexpr int a0 = (E == 0) ? 2 : 0;
  const uint32_t ma = uc.mask[(E == 0) ? 1 : 0];
  const uint32_t mb = uc.mask[(E == 0) ? 2 : 1];
  const uint32_t ba = uc.bias[(E <= 1) ? 0 : (E == 2 ? 1 : 2)];
  const uint32_t bb = uc.bias[(E <= 1) ? 1 : (E == 2 ? 2 : 3)];
  const uint32_t t0 = rotr<(0 + rho - a0) & 31>(w);
  const uint32_t t1 = rotr<(4 + rho - a0) & 31>(w);
  const uint32_t t2 = rotr<(8 + rho - a0) & 31>(w);
  const uint32_t t3 = rotr<(12 + rho - a0) & 31>(w);
  Ba.x = (t0 & ma) | ba; Bb.x = (t0 & mb) | bb;
  Ba.y = (t1 & ma) | ba; Bb.y = (t1 & mb) | bb;
  Ba.z = (t2 & ma) | ba; Bb.z = (t2 & mb) | bb;
  Ba.w = (t3 & ma) | ba; Bb.w = (t3 & mb) | bb;
}

}  // namespace bf
}  // namespace mbq
