// The per-token activation quantiser (paper App. E.4), step by step in fp32, shared by its own launch and by the router
// launch of a stage that carries it along.  Include only where contraction is off (-ffp-contract=off): every step is one
// fp32 operation, and the codes must not depend on how the compiler fuses them.
#pragma once

#include "mbq_common.h"

namespace mbq {

struct ActArgs {
  const uint16_t* X;
  const float* shift;  // null with scale: no transform
  const float* scale;
  uint16_t* Xint;
  float* row_scale;
  uint16_t* Xr;
  int abits;
};

namespace act {

__device__ __forceinline__ float bf16_value(uint32_t bits16) { return __uint_as_float(bits16 << 16); }
// round to nearest even; finite inputs
__device__ __forceinline__ uint32_t bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return u >> 16;
}
__device__ __forceinline__ uint4 pack8(const float v[8]) {
  uint4 o;
  o.x = bf16_bits(v[0]) | (bf16_bits(v[1]) << 16);
  o.y = bf16_bits(v[2]) | (bf16_bits(v[3]) << 16);
  o.z = bf16_bits(v[4]) | (bf16_bits(v[5]) << 16);
  o.w = bf16_bits(v[6]) | (bf16_bits(v[7]) << 16);
  return o;
}
__device__ __forceinline__ void params8(const float* __restrict__ p, int j, float v[8]) {
  const float4 a = reinterpret_cast<const float4*>(p)[2 * j], b = reinterpret_cast<const float4*>(p)[2 * j + 1];
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
  v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
// transformed values of columns 8 j .. 8 j + 7
__device__ __forceinline__ void transformed8(const uint4* __restrict__ x8, int j, const float* __restrict__ shift,
                                             const float* __restrict__ scale, float t[8]) {
#pragma clang fp contract(off)
  const uint4 v = x8[j];
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    t[2 * h] = bf16_value(w[h] & 0xFFFFu);
    t[2 * h + 1] = bf16_value(w[h] >> 16);
  }
  if (scale) {
    float d[8], s[8];
    params8(shift, j, d);
    params8(scale, j, s);
#pragma unroll
    for (int h = 0; h < 8; ++h) t[h] = (t[h] - d[h]) / s[h];
  }
}
struct Code {
  float scale, zp, top;
};
// the row's quantiser from each thread's extremes (zero included); every thread of the workgroup calls it
template <int kThreads>
__device__ __forceinline__ Code row_code(float lo, float hi, int abits, int tid) {
#pragma clang fp contract(off)
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    lo = fminf(lo, __shfl_xor(lo, off));
    hi = fmaxf(hi, __shfl_xor(hi, off));
  }
  constexpr int kWavefronts = kThreads / 64;
  __shared__ float s_lo[kWavefronts], s_hi[kWavefronts];
  if ((tid & 63) == 0) {
    s_lo[tid >> 6] = lo;
    s_hi[tid >> 6] = hi;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kWavefronts; ++w) {
    lo = fminf(lo, s_lo[w]);
    hi = fmaxf(hi, s_hi[w]);
  }
  Code c;
  c.top = (float)((1 << abits) - 1);
  const float rng = fmaxf(hi - lo, 0x1p-100f);
  c.scale = rng / c.top;
  c.zp = fminf(fmaxf(rintf((-lo) / c.scale), 0.f), c.top);
  return c;
}
// q - zp: integers of at most abits bits and a sign, exact in bf16
__device__ __forceinline__ void whole8(const float t[8], const Code& c, float xi[8]) {
#pragma clang fp contract(off)
#pragma unroll
  for (int h = 0; h < 8; ++h) {
    const float q = fminf(fmaxf(rintf(t[h] / c.scale) + c.zp, 0.f), c.top);
    xi[h] = q - c.zp;
  }
}
// the router's input of the same columns, in the original space, rounded to bf16
__device__ __forceinline__ uint4 rebuilt8(const float xi[8], const Code& c, int j, const float* __restrict__ shift,
                                          const float* __restrict__ scale) {
#pragma clang fp contract(off)
  float r[8];
#pragma unroll
  for (int h = 0; h < 8; ++h) r[h] = xi[h] * c.scale;
  if (scale) {
    float d[8], s[8];
    params8(shift, j, d);
    params8(scale, j, s);
#pragma unroll
    for (int h = 0; h < 8; ++h) r[h] = r[h] * s[h] + d[h];
  }
  return pack8(r);
}

constexpr int kHeldThreads = 512, kHeldChunks = 4;  // a row of up to 16384 columns in the registers of 512 threads
constexpr int64_t kHeldColumns = 8 * kHeldThreads * kHeldChunks;

}  // namespace act
}  // namespace mbq
