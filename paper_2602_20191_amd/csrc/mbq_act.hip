// Activation-quantised variant of the layer (paper App. E.4; `abits` of App. C.1): per-token quantiser of the
// transformed activations X~ = (X - delta) / s, the integers q - zp as the main path's bf16 operand, the router's
// input rebuilt in the original space (X_r = X~ s + delta), and the row scaling that finishes the main path.
//
// This translation unit is compiled with -ffp-contract=off: every step of the quantiser is one fp32 operation
// (the codes must not depend on how the compiler fuses them).
#include "mbq_act_quant.h"

namespace mbq {

// One workgroup per token.  Pass 1 finds the row's extremes (zero included), pass 2 writes the codes.  kHold > 0: the
// row fits in kHold chunks of eight values per thread and the transformed values of pass 1 stay in registers;
// kHold = 0: pass 2 re-reads the row (it is in cache) and computes the transformed values again with the same two
// operations.
template <int kThreads, int kHold>
__global__ __launch_bounds__(kThreads) void act_quant_kernel(const uint16_t* __restrict__ X, int64_t K, int abits,
                                                        const float* __restrict__ let_shift,
                                                        const float* __restrict__ let_scale,
                                                        uint16_t* __restrict__ Xint, float* __restrict__ row_scale,
                                                        uint16_t* __restrict__ Xr) {
  const int64_t row = blockIdx.x;
  const int tid = threadIdx.x;
  const uint4* x8 = reinterpret_cast<const uint4*>(X + row * K);  // eight bf16 values per load
  const int n8 = (int)(K >> 3);
  float lo = 0.f, hi = 0.f;
  auto widen = [&](const float t[8]) {
#pragma unroll
    for (int h = 0; h < 8; ++h) {
      lo = fminf(lo, t[h]);
      hi = fmaxf(hi, t[h]);
    }
  };
  float held[kHold > 0 ? kHold : 1][8];
  if constexpr (kHold > 0) {
#pragma unroll
    for (int c = 0; c < kHold; ++c) {
      const int j = tid + c * kThreads;
      if (j < n8) {
        act::transformed8(x8, j, let_shift, let_scale, held[c]);
        widen(held[c]);
      }
    }
  } else {
    for (int j = tid; j < n8; j += kThreads) {
      float t[8];
      act::transformed8(x8, j, let_shift, let_scale, t);
      widen(t);
    }
  }
  const act::Code code = act::row_code<kThreads>(lo, hi, abits, tid);
  if (tid == 0) row_scale[row] = code.scale;

  uint4* out8 = reinterpret_cast<uint4*>(Xint + row * K);
  uint4* xr8 = Xr ? reinterpret_cast<uint4*>(Xr + row * K) : nullptr;
  auto write_chunk = [&](int j, const float t[8]) {
    float xi[8];
    act::whole8(t, code, xi);
    out8[j] = act::pack8(xi);
    if (xr8) xr8[j] = act::rebuilt8(xi, code, j, let_shift, let_scale);
  };
  if constexpr (kHold > 0) {
#pragma unroll
    for (int c = 0; c < kHold; ++c) {
      const int j = tid + c * kThreads;
      if (j < n8) write_chunk(j, held[c]);
    }
  } else {
    for (int j = tid; j < n8; j += kThreads) {
      float t[8];
      act::transformed8(x8, j, let_shift, let_scale, t);
      write_chunk(j, t);
    }
  }
}

// Y[i][n] = Y[i][n] * row_scale[i] (+ bias[n]): one multiplication and one addition, in place.
__global__ __launch_bounds__(256) void scale_rows_kernel(float* __restrict__ Y, int64_t total, int64_t N,
                                                         const float* __restrict__ row_scale,
                                                         const float* __restrict__ bias) {
#pragma clang fp contract(off)
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= total) return;
  const int64_t i = idx / N, n = idx - i * N;
  float y = Y[idx] * row_scale[i];
  if (bias) y = y + bias[n];
  Y[idx] = y;
}

struct ScaleList {
  float* Y[MBQ_MAX_GROUP];
  const float* bias[MBQ_MAX_GROUP];
  long long total[MBQ_MAX_GROUP];  // T * N
  int N[MBQ_MAX_GROUP];
};
__global__ __launch_bounds__(256) void scale_rows_group_kernel(const ScaleList list,
                                                               const float* __restrict__ row_scale) {
#pragma clang fp contract(off)
  const int j = blockIdx.y;
  float* __restrict__ Y = list.Y[j];
  const float* __restrict__ bias = list.bias[j];
  const long long total = list.total[j];
  const int N = list.N[j];
  for (long long idx = (long long)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (long long)gridDim.x * 256) {
    const long long i = idx / N;
    float y = Y[idx] * row_scale[i];
    if (bias) y = y + bias[idx - i * N];
    Y[idx] = y;
  }
}

mbq_status launch_scale_rows_group(int n, float* const* Y, int64_t T, const int64_t* N, const float* row_scale,
                                   const float* const* bias, hipStream_t stream) {
  ScaleList list = {};
  long long most = 0;
  for (int j = 0; j < n; ++j) {
    list.Y[j] = Y[j];
    list.bias[j] = bias ? bias[j] : nullptr;
    list.total[j] = (long long)T * N[j];
    list.N[j] = (int)N[j];
    if (list.total[j] > most) most = list.total[j];
  }
  long long blocks = (most + 255) / 256;
  if (blocks > 65536) blocks = 65536;  // the kernel strides
  hipLaunchKernelGGL(scale_rows_group_kernel, dim3((unsigned)blocks, (unsigned)n), dim3(256), 0, stream, list,
                     row_scale);
  return hip_status(hipGetLastError(), "scale_rows_group_kernel launch");
}

mbq_status launch_act_quant(const uint16_t* X, int64_t T, int64_t K, int abits, const float* let_shift,
                            const float* let_scale, uint16_t* Xint, float* row_scale, uint16_t* Xr,
                            hipStream_t stream) {
  // up to 16384 columns a row is held in registers by 512 threads (four chunks of eight values each)
  if (K <= act::kHeldColumns)
    hipLaunchKernelGGL((act_quant_kernel<act::kHeldThreads, act::kHeldChunks>), dim3((unsigned)T), dim3(act::kHeldThreads), 0, stream, X, K, abits, let_shift,
                       let_scale, Xint, row_scale, Xr);
  else
    hipLaunchKernelGGL((act_quant_kernel<256, 0>), dim3((unsigned)T), dim3(256), 0, stream, X, K, abits, let_shift,
                       let_scale, Xint, row_scale, Xr);
  return hip_status(hipGetLastError(), "act_quant_kernel launch");
}

// The router launch of a stage can quantise the activations itself: rows that its workgroups hold in registers, and
// nothing written by the launch where other workgroups still read.  (With a launch of its own the quantiser is done with
// its inputs before anything else is written, so a caller may lay outputs over them.)
bool act_carried(const ActArgs& aq, int64_t T, int64_t K, const Span* others, int n_others) {
  if (K > act::kHeldColumns) return false;
  const size_t row_bytes = (size_t)(T * K) * sizeof(uint16_t), let_bytes = aq.scale ? (size_t)K * sizeof(float) : 0;
  const Span in[3] = {{aq.X, row_bytes}, {aq.shift, let_bytes}, {aq.scale, let_bytes}};
  auto apart = [&](const Span& o) {
    for (const Span& i : in) {
      const uintptr_t a = (uintptr_t)i.p, b = (uintptr_t)o.p;
      if (i.bytes != 0 && a < b + o.bytes && b < a + i.bytes) return false;
    }
    return true;
  };
  if (!apart({aq.Xint, row_bytes}) || !apart({aq.Xr, row_bytes}) || !apart({aq.row_scale, (size_t)T * sizeof(float)}))
    return false;
  for (int i = 0; i < n_others; ++i)
    if (!apart(others[i])) return false;
  return true;
}

mbq_status launch_scale_rows(float* Y, int64_t T, int64_t N, const float* row_scale, const float* bias,
                             hipStream_t stream) {
  const int64_t total = T * N;
  hipLaunchKernelGGL(scale_rows_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream, Y, total, N,
                     row_scale, bias);
  return hip_status(hipGetLastError(), "scale_rows_kernel launch");
}

}  // namespace mbq
