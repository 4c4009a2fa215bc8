// Internal definitions shared by the translation units of libmbq.so.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mbq.h"

namespace mbq {

constexpr int kGroup = 128;    // input features per quantisation group (paper App. C.1)
constexpr int kSlices = 4;     // E, number of 2-bit slices (paper Sec. 4.1 default)
constexpr int kTileN = 16;     // rows of one code tile
constexpr int kTileK = 256;    // columns of one code tile
constexpr int kTileWords = 256;  // uint32 words of one code tile of one slice (64 lanes x 4)
constexpr int kMaxDecodeTokens = 64;
constexpr int kMaxKSplit = 8;

// Geometry of the packed blob of an N x K matrix.
struct Shape {
  int64_t N, K;
  int NT;               // row tiles, ceil(N / 16)
  int KB;               // column tiles, ceil(K / 256)
  int G;                // real groups per row, K / group
  size_t slice_words;   // uint32 words of one slice = NT * KB * 256
  size_t meta_offset;   // byte offset of the {s0, z0} section
  size_t bytes;         // total blob bytes
  int group;            // columns per quantisation group: 128, or 64 / 32 (configurations; slow kernels only)
  int gshift;           // log2(group)
};

// false (and error set) if invalid
bool make_shape(int64_t N, int64_t K, Shape* out, int group = kGroup);
void set_error(const char* fmt, ...);
mbq_status hip_status(hipError_t e, const char* what);
int knob(int index);  // the calling thread's snapshot of the hooks, taken by the outermost ApiScope
// Every entry point that dispatches opens one; the outermost on a thread snapshots the test/experiment hooks, so
// all decisions of one call (also of the calls it makes in turn) see the same values.
// Compute units of the CURRENT device (asked once per device; 256 if the query fails).  Launch shapes are sized
// by it, so a process that drives several devices gets each device's own figure.
int device_compute_units();

struct ApiScope {
  ApiScope();
  ~ApiScope();
};

// ---- blob addressing (device + host) -------------------------------------------
// Word index, inside one slice, of the dword holding weight (n, k).
__host__ __device__ inline size_t code_word(int NT, int KB, int64_t n, int64_t k) {
  const int r = (int)(k & 255);
  const int d = r >> 6;
  const int kq = (r & 31) >> 3;
  const int lane = 16 * kq + (int)(n & 15);
  return ((size_t)(n >> 4) * KB + (size_t)(k >> 8)) * kTileWords + (size_t)lane * 4 + d;
}
// Bit position of the 2-bit field of weight column k in slice e's (rotated) dword.
__host__ __device__ inline int code_bit(int e, int64_t k) {
  const int r = (int)(k & 255);
  const int step = (r & 63) >> 5;
  const int s = r & 7;
  return (16 * (s & 1) + 4 * (s >> 1) + 2 * step + 2 - 2 * e) & 31;
}
// Index of the float2 {s0, z0} of (row n, group g) inside the meta section; per_tile = groups per 256 columns.
__host__ __device__ inline size_t meta_index(int KB, int64_t n, int g, int per_tile = 2) {
  return ((size_t)(n >> 4) * (per_tile * KB) + g) * kTileN + (size_t)(n & 15);
}

// Output arrays that the activation-preparation launch clears for a linear kernel that adds into
// them (all null: nothing to clear).
struct ZeroList {
  float* p[MBQ_MAX_GROUP];
  long long n[MBQ_MAX_GROUP];  // floats
};

// How a router's outputs map onto the blob's eight-bit code (Sec. 4.1 with other slice widths, App. C.1): the router
// has P outputs (one per slice of the configuration) and output q stands for the first bits[q] bits of the code.
// digits[q] = base-4 digits that precision touches, minus one (what the tokens are sorted and bucketed by, and what the
// weight loaders go by).  A precision array holds value[q]: digits[q] when every bits[q] is even (the linear kernels'
// native precision), bits[q] - 1 otherwise (a token may then stop at the high bit of its last digit; only the kernels
// that say so understand that); shift = 0 / 1 turns a stored value back into digits.
// Default: four outputs of 2, 4, 6, 8 bits.
struct RouteView {
  int P;
  int bits[MBQ_N_PRECISIONS];
  int digits[MBQ_N_PRECISIONS];
  int value[MBQ_N_PRECISIONS];
  int shift;
  int group;  // columns per quantisation group (the routers do not care; the blob's metadata section does)
};
constexpr RouteView kDefaultView = {MBQ_N_PRECISIONS, {2, 4, 6, 8}, {0, 1, 2, 3}, {0, 1, 2, 3}, 0, kGroup};

// ---- kernels' host launchers (each enqueues on `stream`, returns a status) ------
mbq_status launch_encode(const float* W, const Shape& sh, void* blob, const float* ext_scale, const float* ext_zero,
                         hipStream_t stream);
// groups of 64 or 32 columns (sh.group): same code section, a metadata section of 256 / group pairs per tile row
mbq_status launch_encode_small_group(const float* W, const Shape& sh, void* blob, hipStream_t stream);
mbq_status launch_unpack(const void* blob, const Shape& sh, uint8_t* codes, float* scale, float* zero,
                         hipStream_t stream);
mbq_status launch_dequant(const void* blob, const Shape& sh, int p, float* What, hipStream_t stream);
mbq_status launch_dequant_bits(const void* blob, const Shape& sh, int bits, float* What, hipStream_t stream);
mbq_status launch_unpack_view(const void* blob, const Shape& sh, const RouteView& view, uint8_t* codes, float* scale,
                              float* zero, hipStream_t stream);
mbq_status launch_route(const uint16_t* X, int64_t T, int64_t K, const float* Wr, const float* br,
                        int32_t* prec, int32_t* perm, int32_t* offsets, double* logits, void* ws,
                        hipStream_t stream, const RouteView& view = kDefaultView);
mbq_status launch_route_group(const uint16_t* X, int64_t T, int64_t K, int n, const float* const* Wr,
                              const float* const* br, int32_t* const* prec, int32_t* const* perm,
                              int32_t* const* offsets, double* const* logits, void* ws, hipStream_t stream,
                              void* prep, int prep_blocks, const ZeroList* zl, bool defer_bucket,
                              const RouteView& view = kDefaultView, const uint16_t* Xprep = nullptr,
                              const struct ActArgs* aq = nullptr, void* sums = nullptr,
                              const struct PrefillPrep* pf = nullptr);
// aq: the launch also quantises the activations (act_carried); only where the call defers its sort
// sums: the launch also leaves there what launch_mid_sums would, of X or, with aq, of the integers; only where the call
// defers its sort
// pf: the launch also does the work of the prefill kernel's pre-kernel; only where route_defers_sort(T) is false
struct Span {  // a range of device memory
  const void* p;
  size_t bytes;
};
// others: what the launch writes besides the quantiser's results
bool act_carried(const struct ActArgs& aq, int64_t T, int64_t K, const Span* others, int n_others);
bool route_can_carry_prep(int64_t T);
bool route_defers_sort(int64_t T);
mbq_status launch_route_mlp(const uint16_t* X, int64_t T, int64_t K, const float* W1, const float* b1, int H,
                            const float* W2, const float* b2, double delta, int32_t* prec, int32_t* perm,
                            int32_t* offsets, double* scores, void* ws, hipStream_t stream);
int route_mlp_max_hidden();
size_t route_mlp_workspace_bytes(int64_t T, int H);
mbq_status launch_threshold_quantile(const double* scores, int64_t T, long long k, double* delta_out,
                                     hipStream_t stream);
mbq_status launch_linear_simple(const uint16_t* X, int64_t T, const void* blob, const Shape& sh,
                                const int32_t* prec, float* Y, hipStream_t stream, bool bit_view = false);
mbq_status launch_linear_decode(const uint16_t* X, int64_t T, const void* blob, const Shape& sh,
                                const int32_t* perm, const int32_t* offsets, float* Y, void* ws,
                                hipStream_t stream);
mbq_status launch_linear_prefill(const uint16_t* X, int64_t T, const void* blob, const Shape& sh,
                                 const int32_t* perm, const int32_t* offsets, float* Y, void* ws,
                                 hipStream_t stream);
// the same for up to MBQ_MAX_GROUP matrices over one X (one K), each with its own routing, in one launch
// the work of the pre-kernel of a call, for another launch to do (false: none can); `prepared`: one has done it
bool prefill_prep_of(const uint16_t* X, int64_t T, int n, const Shape* shapes, float* const* Y, void* ws,
                     struct PrefillPrep* prep);
mbq_status launch_linear_prefill_group(const uint16_t* X, int64_t T, int n, const void* const* blobs, const Shape* shapes,
                                       const int32_t* const* perm, const int32_t* const* offsets, float* const* Y,
                                       void* ws, hipStream_t stream, bool prepared = false);
mbq_status launch_linear_decode16(const uint16_t* X, int64_t T, const void* blob, const Shape& sh,
                                  const int32_t* prec, const int32_t* perm, float* Y, hipStream_t stream);
// the same for up to MBQ_MAX_GROUP matrices over one X (one K), each with its own routing, in one launch
// Outputs that launch_linear_decode16(_group) ADDS into for this call (K split of small outputs): the caller clears
// them first, with launch_zero_outputs or through the router launch.
void decode16_zero_list(int64_t T, int n, const Shape* shapes, float* const* Y, ZeroList* zl);
mbq_status launch_zero_outputs(const ZeroList& zl, hipStream_t stream);
// sort_perm / sort_offsets (arrays of n, or null): the tokens are not sorted yet (perm is ignored); the launch sorts
// them by the precisions itself and writes the order and the bucket offsets there (T <= 128)
mbq_status launch_linear_decode16_group(const uint16_t* X, int64_t T, int n, const void* const* blobs,
                                        const Shape* shapes, const int32_t* const* prec, const int32_t* const* perm,
                                        float* const* Y, hipStream_t stream, int32_t* const* sort_perm,
                                        int32_t* const* sort_offsets);
// parts along K that a matrix of 33 .. 64 tokens takes the kernel of mbq_linear_mid.hip in, 0: it does not.  ws begins with
// what launch_mid_sums (or the router launch) left there (mid_group_sums below).
int mid_parts(int64_t T, const Shape& sh);
mbq_status launch_mid_sums(const uint16_t* X, int64_t T, int64_t K, void* sums, hipStream_t stream);
mbq_status launch_linear_mid_group(const uint16_t* X, int64_t T, int n, const void* const* blobs, const Shape* shapes,
                                   const int32_t* const* prec, const int32_t* const* perm, float* const* Y, void* ws,
                                   hipStream_t stream, int32_t* const* sort_perm, int32_t* const* sort_offsets);
bool decode_f4_supports(int64_t T, const Shape& sh);
int decode_f4_k_parts(int n, const Shape* shapes);
void decode_f4_zero_list(int64_t T, int n, const Shape* shapes, float* const* Y, ZeroList* zl);
// A 16-byte load of data that a launch reads once (packed weights in the decode kernels), with the
// non-temporal hint: the stream then does not push the activations, router parameters and outputs that
// the neighbouring launches share out of the caches.
__device__ __forceinline__ uint4 load_once(const uint4* p) {
  typedef uint32_t u32x4_nt __attribute__((ext_vector_type(4)));
  const u32x4_nt v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_nt*>(p));
  return uint4{v.x, v.y, v.z, v.w};
}
// share `part` of `parts` of the clearing, done by `nthreads` threads of which this is `tid`
__device__ inline void zero_share(const ZeroList& zl, int part, int parts, int tid, int nthreads) {
#pragma unroll
  for (int j = 0; j < MBQ_MAX_GROUP; ++j) {
    float* p = zl.p[j];
    if (p == nullptr) continue;
    const long long n = zl.n[j];
    for (long long i = (long long)part * nthreads + tid; i < n; i += (long long)parts * nthreads) p[i] = 0.f;
  }
}
// One lane's share of the sums that launch_linear_mid_group starts from, sums[group][token] = {even, odd} over a group's even
// and odd steps of 32 columns: `sum` of the eight columns from column 8 c of a token's row; the 16 lanes of an aligned
// quarter of a wavefront hold consecutive ones (a group), four of them a step.
__device__ __forceinline__ void mid_group_sums(float sum, int c, int token, int T, float* __restrict__ sums) {
  sum += __shfl_xor(sum, 1, 64);
  sum += __shfl_xor(sum, 2, 64);
  sum += __shfl_xor(sum, 8, 64);  // steps 0 and 2, 1 and 3
  if ((c & 11) == 0) sums[2 * ((size_t)(c >> 4) * T + token) + ((c >> 2) & 1)] = sum;
}
__device__ __forceinline__ float sum8(const uint4& v) {
  const uint32_t u[4] = {v.x, v.y, v.z, v.w};
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < 4; ++j) s += __uint_as_float(u[j] << 16) + __uint_as_float(u[j] & 0xFFFF0000u);
  return s;
}
// 16 bytes per lane from base + offset straight into LDS at lds + 16 * lane.  Written in assembly because the compiler
// takes every LDS read for a possible reader of such a load and would wait for all of them ahead of the first read of
// a group; the kernel waits itself, once per group.  (The instruction has no register result; M0, which holds the LDS
// address, is put back.)
__device__ __forceinline__ void dma_16(uint32_t lds, uint32_t offset, const void* base) {
  uint32_t m0;
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3\n\ts_mov_b32 m0, %0"
               : "=&s"(m0)
               : "s"(lds), "v"(offset), "s"(base)
               : "memory");
}
// What a prefill launch starts from: the sums of X over groups, Sx[token][group], and cleared arrays (zl: outputs, zs: arrays
// of the workspace).  A workgroup does rows row0 .. row0 + rows - 1 and its share of the clearing.
struct PrefillPrep {
  const uint16_t* X;
  float* Sx;
  ZeroList zl, zs;
};
__device__ inline void prefill_clear(const ZeroList& zl, int64_t at, int64_t step) {
  typedef float f32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
  for (int j = 0; j < MBQ_MAX_GROUP; ++j) {
    float* p = zl.p[j];
    if (p == nullptr) continue;
    const int64_t n = zl.n[j], n4 = (reinterpret_cast<uintptr_t>(p) & 15) == 0 ? n >> 2 : 0;
    for (int64_t i = at; i < n4; i += step) reinterpret_cast<f32x4*>(p)[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int64_t i = 4 * n4 + at; i < n; i += step) p[i] = 0.f;
  }
}
// the sums of one row by 256 threads, t = 0 .. 255; copy: where the row goes besides (null: nowhere)
__device__ inline void prefill_row_sums(const uint4* src, int64_t K, int t, float* sums, uint4* copy) {
  const int chunks = (int)(K >> 3);  // a multiple of 16: groups of 16 lanes are whole
  for (int c = t; c < chunks; c += 256) {
    const uint4 v = src[c];
    if (copy) copy[c] = v;
    float s = sum8(v);
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
    if ((t & 15) == 0) sums[c >> 4] = s;
  }
}
__device__ inline void prefill_prep_share(const PrefillPrep& p, int64_t T, int64_t K, int64_t row0, int rows, int threads) {
  const int64_t at = (int64_t)blockIdx.x * threads + threadIdx.x, step = (int64_t)gridDim.x * threads;
  prefill_clear(p.zl, at, step);
  prefill_clear(p.zs, at, step);
  for (int64_t r = row0 + (threadIdx.x >> 8); r < row0 + rows && r < T; r += threads >> 8)
    prefill_row_sums(reinterpret_cast<const uint4*>(p.X + r * K), K, threadIdx.x & 255, p.Sx + r * (K >> 7), nullptr);
}
// The last launch of calls whose parts of K have arrays of their own: Y += array 1, += array 2, .. in that order (nothing to
// launch if no matrix has any).  arrays: Y among them, at most kMaxKSplit; array 1 lies at `array`, the others array_floats
// apart, 16-byte aligned.
struct Fold {
  float* Y[MBQ_MAX_GROUP];
  const float* array[MBQ_MAX_GROUP];
  int64_t array_floats[MBQ_MAX_GROUP];
  int64_t n[MBQ_MAX_GROUP];  // floats of Y
  int arrays[MBQ_MAX_GROUP];
};
mbq_status launch_fold(const Fold& f, int n, hipStream_t stream);
size_t decode_f4_workspace_bytes(int64_t T, const Shape& sh);
mbq_status launch_decode_f4_prep(const uint16_t* X, int64_t T, int64_t K, int KB, void* ws, const ZeroList& zl,
                                 hipStream_t stream);
// perm/offsets (arrays of n, or null): the launch also sorts the tokens of every matrix by precision.
// row_scale: output row i is to be multiplied by row_scale[i] (and bias[j][n] added); a launch that does so sets *scaled.
mbq_status launch_linear_decode_f4(int64_t T, int n, const void* const* blobs, const Shape* shapes,
                                   const int32_t* const* prec, float* const* Y, const void* ws, hipStream_t stream,
                                   int32_t* const* perm, int32_t* const* offsets, unsigned long long* stamps = nullptr,
                                   bool bit_view = false, const float* row_scale = nullptr,
                                   const float* const* bias = nullptr, bool* scaled = nullptr);
// bit_view (the precision arrays hold bits - 1, see RouteView) is understood by the one-token-tile kernels only
bool decode_f4_takes_bit_view(int64_t T, const Shape& sh);
// timeline build of the ring kernel: workgroups it launches at most, and 8-byte slots each of them writes
int decode_f4_timeline_workgroups();
int decode_f4_timeline_slots();
// activation-quantised variant (App. E.4): per-token quantiser and the row scaling that finishes the main path
mbq_status launch_act_quant(const uint16_t* X, int64_t T, int64_t K, int abits, const float* let_shift,
                            const float* let_scale, uint16_t* Xint, float* row_scale, uint16_t* Xr,
                            hipStream_t stream);
mbq_status launch_scale_rows(float* Y, int64_t T, int64_t N, const float* row_scale, const float* bias,
                             hipStream_t stream);
// the same for the outputs of up to MBQ_MAX_GROUP projections in one launch (bias: array of n, entries may be null)
mbq_status launch_scale_rows_group(int n, float* const* Y, int64_t T, const int64_t* N, const float* row_scale,
                                   const float* const* bias, hipStream_t stream);
size_t decode_workspace_bytes(int64_t T, const Shape& sh);
size_t prefill_workspace_bytes(int64_t T, const Shape& sh);

}  // namespace mbq
