// C-ABI entry points of libmbq.so: argument checks, shape arithmetic, dispatch.
#include <stdarg.h>
#include <stdio.h>

#include <atomic>

#include "mbq_act_quant.h"
#include "mbq_bench.h"
#include "mbq_common.h"

namespace mbq {

static thread_local char g_error[512] = "";
// Test and experiment hooks (mbq_set_knob).  A call takes one snapshot of them when it enters the library and
// dispatches on that snapshot only, so a change made by another thread never splits one call's decisions.
constexpr int kKnobs = 8;
static std::atomic<int> g_knobs[kKnobs];
static thread_local int t_knobs[kKnobs] = {0, 0, 0, 0, 0, 0, 0, 0};
static thread_local int t_depth = 0;
ApiScope::ApiScope() {
  if (t_depth++ == 0)
    for (int i = 0; i < kKnobs; ++i) t_knobs[i] = g_knobs[i].load(std::memory_order_relaxed);
}
ApiScope::~ApiScope() { --t_depth; }

void set_error(const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_error, sizeof(g_error), fmt, ap);
  va_end(ap);
}

mbq_status hip_status(hipError_t e, const char* what) {
  if (e == hipSuccess) return MBQ_OK;
  set_error("%s: %s", what, hipGetErrorString(e));
  return MBQ_ERR_HIP;
}

int knob(int index) { return (index >= 0 && index < kKnobs) ? t_knobs[index] : 0; }

bool make_shape(int64_t N, int64_t K, Shape* out, int group) {
  if (N <= 0 || K <= 0) {
    set_error("N and K must be positive (N=%lld, K=%lld)", (long long)N, (long long)K);
    return false;
  }
  if (K % kGroup != 0) {
    set_error("K=%lld is not a multiple of the group size %d", (long long)K, kGroup);
    return false;
  }
  if (N > (int64_t)1 << 24 || K > (int64_t)1 << 24 || N * K > (int64_t)1 << 36) {
    set_error("shape %lld x %lld is too large", (long long)N, (long long)K);
    return false;
  }
  Shape s;
  s.N = N;
  s.K = K;
  s.NT = (int)((N + kTileN - 1) / kTileN);
  s.KB = (int)((K + kTileK - 1) / kTileK);
  s.group = group;
  s.gshift = group == 128 ? 7 : (group == 64 ? 6 : 5);
  s.G = (int)(K / group);
  s.slice_words = (size_t)s.NT * s.KB * kTileWords;
  s.meta_offset = (size_t)kSlices * s.slice_words * 4;
  s.bytes = s.meta_offset + (size_t)s.NT * ((kTileK / group) * s.KB) * kTileN * 8;
  *out = s;
  return true;
}

int device_compute_units() {
  constexpr int kDevices = 64;
  static std::atomic<int> cached[kDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kDevices) return 256;
  int n = cached[dev].load(std::memory_order_relaxed);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cached[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

static bool aligned(const void* p, size_t a) { return ((uintptr_t)p % a) == 0; }

// The slice configuration a call runs under (the *_cfg entry points set it for the duration of the call they forward
// to; everything else sees the default: four slices of two bits).
static thread_local const RouteView* t_view = &kDefaultView;
struct ViewScope {
  const RouteView* saved;
  explicit ViewScope(const RouteView* v) : saved(t_view) { t_view = v; }
  ~ViewScope() { t_view = saved; }
};
// What the activation-quantised stage call adds to the stage call it forwards to: the linear kernels multiply the
// integers, the quantiser runs inside the router launch or in a launch ahead of it, and the linear launch may scale the
// output rows itself (then `scaled` is set and no launch follows).  Null outside such a call.
struct ActStage {
  ActArgs aq;
  const float* const* bias;
  bool scaled;
};
static thread_local ActStage* t_act = nullptr;
struct ActScope {
  explicit ActScope(ActStage* a) { t_act = a; }
  ~ActScope() { t_act = nullptr; }
};
// the quantiser's own launch, where the router launch does not carry it; `aq` is left null then.  n, prec, Y, N, ws: what
// a router launch that carries it writes (n = 0: it may not)
static mbq_status act_ahead(int64_t T, int64_t K, int n, int32_t* const* prec, float* const* Y, const int64_t* N,
                            const void* ws, size_t ws_bytes, const ActArgs** aq, hipStream_t s) {
  *aq = nullptr;
  if (!t_act) return MBQ_OK;
  const ActArgs& a = t_act->aq;
  Span written[2 * MBQ_MAX_GROUP + 1];
  int spans = 0;
  for (int i = 0; i < n; ++i) {
    written[spans++] = {prec[i], (size_t)T * sizeof(int32_t)};
    written[spans++] = {Y[i], (size_t)(T * N[i]) * sizeof(float)};
  }
  written[spans++] = {ws, ws_bytes};
  if (n > 0 && act_carried(a, T, K, written, spans)) {
    *aq = &a;
    return MBQ_OK;
  }
  return launch_act_quant(a.X, T, K, a.abits, a.shift, a.scale, a.Xint, a.row_scale, a.Xr, s);
}
// cfg -> view; the configurations this library runs are those that cut the blob's eight-bit code
static bool make_view(const mbq_config* cfg, RouteView* v, const char* who) {
  if (!cfg) {
    set_error("%s: null configuration", who);
    return false;
  }
  if (cfg->n_slices < 1 || cfg->n_slices > MBQ_MAX_SLICES) {
    set_error("%s: %d slices, supported 1..%d", who, cfg->n_slices, MBQ_MAX_SLICES);
    return false;
  }
  if (cfg->group != kGroup && cfg->group != 64 && cfg->group != 32) {
    set_error("%s: group size %d, supported: %d, 64, 32", who, cfg->group, kGroup);
    return false;
  }
  int bits = 0;
  bool odd = false;
  *v = kDefaultView;
  v->P = cfg->n_slices;
  for (int e = 0; e < cfg->n_slices; ++e) {
    const int b = cfg->slice_bits[e];
    if (b < 1 || bits + b > 2 * kSlices) {
      set_error("%s: slice %d has %d bits; supported: widths of at least 1 bit that add up to at most %d bits", who, e, b,
                2 * kSlices);
      return false;
    }
    bits += b;
    v->bits[e] = bits;
    v->digits[e] = (bits + 1) / 2 - 1;
    odd = odd || (bits & 1) != 0;
  }
  for (int e = cfg->n_slices; e < MBQ_N_PRECISIONS; ++e) {
    v->bits[e] = v->bits[cfg->n_slices - 1];
    v->digits[e] = v->digits[cfg->n_slices - 1];
  }
  v->shift = odd ? 1 : 0;
  v->group = cfg->group;
  for (int e = 0; e < MBQ_N_PRECISIONS; ++e) v->value[e] = odd ? v->bits[e] - 1 : v->digits[e];
  return true;
}

// Precision arrays that count bits (see RouteView) above one token tile: the one-token-tile decode kernels, which
// understand them, run once per 16 tokens - a pass over the weights each, far from the kernels of the digit
// configurations at these token counts, and three to four orders of magnitude from the one-thread-per-output kernel
// that would run otherwise.  The chunks follow each other on the stream and share the prepared-activation area.
static mbq_status bit_view_in_chunks(const uint16_t* X, int64_t T, int n, const void* const* blobs, const Shape* sh,
                                     const int32_t* const* prec, float* const* Y, void* ws, hipStream_t s) {
  for (int64_t t0 = 0; t0 < T; t0 += 16) {
    const int64_t tc = T - t0 < 16 ? T - t0 : 16;
    const int32_t* pc[MBQ_MAX_GROUP];
    float* yc[MBQ_MAX_GROUP];
    for (int i = 0; i < n; ++i) {
      pc[i] = prec[i] + t0;
      yc[i] = Y[i] + t0 * sh[i].N;
    }
    ZeroList zl;
    decode_f4_zero_list(tc, n, sh, yc, &zl);
    mbq_status st = launch_decode_f4_prep(X + t0 * sh[0].K, tc, sh[0].K, sh[0].KB, ws, zl, s);
    if (st != MBQ_OK) return st;
    st = launch_linear_decode_f4(tc, n, blobs, sh, pc, yc, ws, s, nullptr, nullptr, nullptr, true);
    if (st != MBQ_OK) return st;
  }
  return MBQ_OK;
}

// 17..64 tokens (and one token tile when the FP4-operand kernels are switched off): the register-stationary
// kernel, except for matrices with few row tiles (see dispatch_linear)
static bool takes_stationary_kernel(int64_t T, const Shape& sh) {
  // (re-measured with the K split of the stationary kernel: up to 32 column blocks it is as fast or faster - 1536 x
  // 5120 at 17..32 tokens 13 us against 16; beyond, few row tiles favour the other kernel - 1024 x 14336 16 us against 21)
  return knob(3) != 1 && (knob(3) == 2 || sh.KB <= 32 || sh.NT >= 128 || (T > 32 && sh.NT >= 32));
}

// Above the decode limit the register-stationary kernel still beats the prefill kernel on small matrices: it walks the
// weights once per 32 sorted tokens without a pre-kernel and fills the chip with fewer columns.  Measured on cold weights,
// stationary / prefill in us per call, from the uniform mix to {70,20,8,2} %:
//   1024 x 4096: 12 / 23 at 65 tokens, 11 / 27..36 at 128, 16 / 34..44 at 256;  2048 x 4096: 19 / 26 at 65, 23 / 40..48 at 256;
//   4096 x 4096: 30 / 33 at 65, 24 / 36..45 at 128;  8192 x 4096: 50 / 46 at 65, 42 / 50..53 at 128;
//   11008 x 4096: 68 / 57..62 at 80, 54 / 58..64 at 128, as a pair 115 / 91..105 at 128;
//   14336 x 4096: 82 / 56 and 66 / 56..63;  4096 x 14336: 98 / 58 and 81 / 59..64;  28672 x 8192: 234 / 190 and 232 / 176..202.
// AUTO takes it up to 128 tokens for matrices of at most 8192 code blocks of 16 x 256 (8192 x 4096 has 8192), up to 512 for
// at most 2048, and from 161 to 256 tokens for at most 4096 blocks if there are more columns than rows:
//   2048 x 8192: 43 / 37..45 at 129, 43 / 44..52 at 160, 40 / 44..56 at 192, 43 / 48..57 at 256;
//   2048 x 5504: 42 / 32..40 at 129, 39 / 38..48 at 192, 43 / 45..53 at 256.
// With as many rows as columns a matrix alone would gain by it too (4096 x 4096 at 256 tokens 41 / 48..57, 3072 x 3072 30 /
// 40..49), but has company more often than not and has to take the same kernel there: three of 4096 x 4096 take 108..115 /
// 66..74, three of 3072 x 3072 99 / 63..67.  Tokens that are all at two bits, which only the device knows, would favour it
// everywhere below 256 tokens (4096 x 4096 at 256: 22 / 55).
constexpr int64_t kMaxStationaryTokens = 128, kMaxStationaryTokensSmall = 512;
constexpr int64_t kMinStationaryTokensNarrow = 161, kMaxStationaryTokensNarrow = 256;
constexpr int64_t kSmallMatrixBlocks = 2048, kNarrowMatrixBlocks = 4096, kMiddleMatrixBlocks = 8192;
constexpr int kAlgoStationary = 100;  // internal: what AUTO resolves to in those ranges
static int resolve_auto(int64_t T, const Shape& sh) {
  if (T <= kMaxDecodeTokens) return MBQ_ALGO_DECODE;
  const int64_t blocks = (int64_t)sh.NT * sh.KB;
  const bool stationary = T <= (blocks <= kSmallMatrixBlocks    ? kMaxStationaryTokensSmall
                                : blocks <= kMiddleMatrixBlocks ? kMaxStationaryTokens
                                                                : 0) ||
                          (blocks <= kNarrowMatrixBlocks && sh.N < sh.K && T >= kMinStationaryTokensNarrow &&
                           T <= kMaxStationaryTokensNarrow);
  return (stationary && knob(3) == 0 && takes_stationary_kernel(T, sh)) ? kAlgoStationary : MBQ_ALGO_PREFILL;
}

static bool takes_mid_kernel(int64_t T, const Shape& sh) {
  return knob(3) == 0 && mid_parts(T, sh) > 0;
}

// Matrices of a call that share a launch.
struct Sharing {
  int n = 0;
  const void* blob[MBQ_MAX_GROUP];
  Shape sh[MBQ_MAX_GROUP];
  const int32_t *prec[MBQ_MAX_GROUP], *perm[MBQ_MAX_GROUP];
  float* Y[MBQ_MAX_GROUP];
  int32_t *sort_perm[MBQ_MAX_GROUP], *sort_offsets[MBQ_MAX_GROUP];  // where a launch that sorts leaves the order

  void add(const void* b, const Shape& s, const int32_t* p, const int32_t* order, float* y, int32_t* to_perm, int32_t* to_offsets) {
    blob[n] = b;
    sh[n] = s;
    prec[n] = p;
    perm[n] = order;
    Y[n] = y;
    sort_perm[n] = to_perm;
    sort_offsets[n++] = to_offsets;
  }
  mbq_status launch_mid(const uint16_t* X, int64_t T, void* ws, hipStream_t s, bool sort) const {
    if (n == 0) return MBQ_OK;
    return launch_linear_mid_group(X, T, n, blob, sh, prec, perm, Y, ws, s, sort ? sort_perm : nullptr,
                                   sort ? sort_offsets : nullptr);
  }
  mbq_status launch_stationary(const uint16_t* X, int64_t T, hipStream_t s, bool sort) const {
    if (n == 0) return MBQ_OK;
    return launch_linear_decode16_group(X, T, n, blob, sh, prec, perm, Y, s, sort ? sort_perm : nullptr,
                                        sort ? sort_offsets : nullptr);
  }
  void zero_list(int64_t T, ZeroList* zl) const {  // of the register-stationary kernel
    *zl = ZeroList{};
    if (n > 0) decode16_zero_list(T, n, sh, Y, zl);
  }
};

// algo is DECODE (T <= 64), PREFILL, SIMPLE or kAlgoStationary here
mbq_status dispatch_linear(const uint16_t* X, int64_t T, const void* blob, const Shape& sh, const int32_t* prec,
                           const int32_t* perm, const int32_t* offsets, float* Y, void* ws, int algo,
                           hipStream_t s) {
  switch (algo) {
    case MBQ_ALGO_SIMPLE:
      return launch_linear_simple(X, T, blob, sh, prec, Y, s);
    case kAlgoStationary: {
      ZeroList zl;
      decode16_zero_list(T, 1, &sh, &Y, &zl);
      mbq_status st = launch_zero_outputs(zl, s);
      if (st != MBQ_OK) return st;
      return launch_linear_decode16(X, T, blob, sh, prec, perm, Y, s);
    }
    case MBQ_ALGO_DECODE:
      // One token tile (T <= 16): the FP4-operand kernels (activation preparation, then the
      // linear kernel).  17..64 tokens run the bf16-operand kernels, one pass per 16
      // precision-sorted tokens: the register-stationary chunked kernel, except for matrices with few
      // row tiles, where keeping every column block in flight (K split + reduction) fills the chip
      // better (measured on weights that are not in the last-level cache).
      if (knob(3) == 0 && decode_f4_supports(T, sh)) {
        ZeroList zl;
        decode_f4_zero_list(T, 1, &sh, &Y, &zl);
        mbq_status st = launch_decode_f4_prep(X, T, sh.K, sh.KB, ws, zl, s);
        if (st != MBQ_OK) return st;
        return launch_linear_decode_f4(T, 1, &blob, &sh, &prec, &Y, ws, s, nullptr, nullptr);
      }
      if (takes_mid_kernel(T, sh)) {
        mbq_status st = launch_mid_sums(X, T, sh.K, ws, s);
        if (st != MBQ_OK) return st;
        return launch_linear_mid_group(X, T, 1, &blob, &sh, &prec, &perm, &Y, ws, s, nullptr, nullptr);
      }
      if (takes_stationary_kernel(T, sh)) {
        ZeroList zl;
        decode16_zero_list(T, 1, &sh, &Y, &zl);
        mbq_status st = launch_zero_outputs(zl, s);  // nothing to do unless the launch splits K
        if (st != MBQ_OK) return st;
        return launch_linear_decode16(X, T, blob, sh, prec, perm, Y, s);
      }
      return launch_linear_decode(X, T, blob, sh, perm, offsets, Y, ws, s);
    default:
      return launch_linear_prefill(X, T, blob, sh, perm, offsets, Y, ws, s);
  }
}

// ---- scratch memory of mbq_linear_static ---------------------------------------------------------------------------
// Device memory that belongs to the library image: every GPU the library runs on holds its own copy at its own address
// until the process ends.  In host code the array's name is only a handle for hipGetSymbolAddress, never an address.
static __device__ __align__(256) unsigned char scratch[MBQ_STATIC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
static std::atomic<void*> g_scratch_ptr[kMaxDevices];

// the address of `scratch` on the current device (looked up once per device, with that device current)
static mbq_status scratch_on_current_device(void** out) {
  int dev = -1;
  mbq_status st = hip_status(hipGetDevice(&dev), "hipGetDevice");
  if (st != MBQ_OK) return st;
  if (dev < 0 || dev >= kMaxDevices) {
    set_error("mbq_linear_static: device index %d outside 0..%d", dev, kMaxDevices - 1);
    return MBQ_ERR_INVALID_ARG;
  }
  void* ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (ptr == nullptr) {
    st = hip_status(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)), "hipGetSymbolAddress(scratch)");
    if (st != MBQ_OK) return st;
    if (ptr == nullptr) {
      set_error("mbq_linear_static: hipGetSymbolAddress returned a null address");
      return MBQ_ERR_HIP;
    }
    g_scratch_ptr[dev].store(ptr, std::memory_order_release);  // (a second thread may look it up too: same value)
  }
  *out = ptr;
  return MBQ_OK;
}

}  // namespace mbq

using namespace mbq;

extern "C" {

size_t mbq_static_scratch_bytes(void) { return MBQ_STATIC_SCRATCH_BYTES; }

mbq_status mbq_linear_static(const uint16_t* X, int64_t T, const void* blob, int64_t N, int64_t K,
                             const int32_t* prec, const int32_t* perm, const int32_t* offsets, float* Y, int algo,
                             void* stream) {
  ApiScope scope;
  Shape sh;
  if (!make_shape(N, K, &sh)) return MBQ_ERR_BAD_SHAPE;
  if (T < 0 || T > (int64_t)1 << 24) {
    set_error("mbq_linear_static: bad token count %lld", (long long)T);
    return MBQ_ERR_BAD_SHAPE;
  }
  const size_t need = mbq_linear_workspace_bytes(T, N, K);
  if (need > (size_t)MBQ_STATIC_SCRATCH_BYTES) {
    set_error("mbq_linear_static: T=%lld, N=%lld, K=%lld needs %zu bytes of scratch memory, the built-in buffer holds "
              "%zu: use mbq_linear with a workspace of your own", (long long)T, (long long)N, (long long)K, need,
              (size_t)MBQ_STATIC_SCRATCH_BYTES);
    return MBQ_ERR_WORKSPACE;
  }
  if (T == 0) return mbq_linear(X, T, blob, N, K, prec, perm, offsets, Y, nullptr, 0, algo, stream);
  void* ws = nullptr;
  mbq_status st = scratch_on_current_device(&ws);
  if (st != MBQ_OK) return st;
  return mbq_linear(X, T, blob, N, K, prec, perm, offsets, Y, ws, (size_t)MBQ_STATIC_SCRATCH_BYTES, algo, stream);
}

const char* mbq_version(void) { return "mbq 0.1 (gfx950)"; }

const char* mbq_last_error(void) { return g_error; }

size_t mbq_blob_bytes(int64_t N, int64_t K) {
  Shape sh;
  return make_shape(N, K, &sh) ? sh.bytes : 0;
}

size_t mbq_route_workspace_bytes(int64_t T, int64_t K) {
  (void)T;
  (void)K;
  return 256;
}

size_t mbq_linear_workspace_bytes(int64_t T, int64_t N, int64_t K) {
  ApiScope scope;
  Shape sh;
  if (T < 0 || !make_shape(N, K, &sh)) return 0;
  size_t a = decode_workspace_bytes(T, sh);
  size_t b = prefill_workspace_bytes(T, sh);
  size_t c = decode_f4_workspace_bytes(T, sh);
  if (b > a) a = b;
  if (c > a) a = c;
  return a + 256;
}

mbq_status mbq_set_knob(int k, int value) {
  if (k < 0 || k >= kKnobs || k == 6) {
    set_error("unknown knob %d", k);
    return MBQ_ERR_INVALID_ARG;
  }
  g_knobs[k].store(value, std::memory_order_relaxed);
  return MBQ_OK;
}

mbq_status mbq_encode(const float* W, int64_t N, int64_t K, void* blob, void* stream) {
  Shape sh;
  if (!make_shape(N, K, &sh)) return MBQ_ERR_BAD_SHAPE;
  if (!W || !blob || !aligned(blob, 256) || !aligned(W, 16)) {
    set_error("mbq_encode: W must be 16-byte and blob 256-byte aligned and non-null");
    return MBQ_ERR_INVALID_ARG;
  }
  return launch_encode(W, sh, blob, nullptr, nullptr, (hipStream_t)stream);
}

mbq_status mbq_encode_with_params(const float* W, int64_t N, int64_t K, const float* scale, const float* zero,
                                  void* blob, void* stream) {
  Shape sh;
  if (!make_shape(N, K, &sh)) return MBQ_ERR_BAD_SHAPE;
  if (!W || !blob || !scale || !zero || !aligned(blob, 256) || !aligned(W, 16)) {
    set_error("mbq_encode_with_params: W must be 16-byte and blob 256-byte aligned; W, scale, zero, blob non-null");
    return MBQ_ERR_INVALID_ARG;
  }
  return launch_encode(W, sh, blob, scale, zero, (hipStream_t)stream);
}

mbq_status mbq_unpack(const void* blob, int64_t N, int64_t K, uint8_t* codes, float* scale, float* zero,
                      void* stream) {
  Shape sh;
  if (!make_shape(N, K, &sh)) return MBQ_ERR_BAD_SHAPE;
  if (!blob || !aligned(blob, 256)) {
    set_error("mbq_unpack: blob must be non-null and 256-byte aligned");
    return MBQ_ERR_INVALID_ARG;
  }
  return launch_unpack(blob, sh, codes, scale, zero, (hipStream_t)stream);
}

mbq_status mbq_dequant(const void* blob, int64_t N, int64_t K, int p, float* What, void* stream) {
  Shape sh;
  if (!make_shape(N, K, &sh)) return MBQ_ERR_BAD_SHAPE;
  if (!blob || !What || !aligned(blob, 256) || p < 0 || p >= MBQ_N_PRECISIONS) {
    set_error("mbq_dequant: null/misaligned pointer or precision index %d outside 0..3", p);
    return MBQ_ERR_INVALID_ARG;
  }
  return launch_dequant(blob, sh, p, What, (hipStream_t)stream);
}

mbq_status mbq_route(const uint16_t* X, int64_t T, int64_t K, const float* Wr, const float* br, int P,
                     int32_t* prec, int32_t* perm, int32_t* offsets, double* logits, void* ws,
                     size_t ws_bytes, void* stream) {
  ApiScope scope;
  if (P != t_view->P) {
    set_error("mbq_route: P=%d, the slice configuration has %d precisions", P, t_view->P);
    return MBQ_ERR_BAD_SHAPE;
  }
  if (T < 0 || K <= 0 || K % kGroup != 0 || T > (int64_t)1 << 24 || K > (int64_t)1 << 24) {
    set_error("mbq_route: bad sizes T=%lld K=%lld", (long long)T, (long long)K);
    return MBQ_ERR_BAD_SHAPE;
  }
  if (!offsets || (T > 0 && (!X || !Wr || !br || !prec || !perm)) || !aligned(X, 16) || !aligned(Wr, 16)) {
    set_error("mbq_route: null or misaligned pointer (X and Wr need 16-byte alignment)");
    return MBQ_ERR_INVALID_ARG;
  }
  if (ws_bytes < mbq_route_workspace_bytes(T, K) || !ws || !aligned(ws, 256)) {
    set_error("mbq_route: workspace too small or misaligned (%zu < %zu)", ws_bytes, mbq_route_workspace_bytes(T, K));
    return MBQ_ERR_WORKSPACE;
  }
  return launch_route(X, T, K, Wr, br, prec, perm, offsets, logits, ws, (hipStream_t)stream, *t_view);
}

mbq_status mbq_route_group(const uint16_t* X, int64_t T, int64_t K, int n_proj, const float* const* Wr_host,
                           const float* const* br_host, int P, int32_t* const* prec_host,
                           int32_t* const* perm_host, int32_t* const* offsets_host, void* ws, size_t ws_bytes,
                           void* stream) {
  ApiScope scope;
  if (P != t_view->P) {
    set_error("mbq_route_group: P=%d, the slice configuration has %d precisions", P, t_view->P);
    return MBQ_ERR_BAD_SHAPE;
  }
  if (n_proj < 1 || n_proj > MBQ_MAX_GROUP) {
    set_error("mbq_route_group: n_proj=%d outside 1..%d", n_proj, MBQ_MAX_GROUP);
    return MBQ_ERR_INVALID_ARG;
  }
  if (T < 0 || K <= 0 || K % kGroup != 0 || T > (int64_t)1 << 24 || K > (int64_t)1 << 24) {
    set_error("mbq_route_group: bad sizes T=%lld K=%lld", (long long)T, (long long)K);
    return MBQ_ERR_BAD_SHAPE;
  }
  if (!Wr_host || !br_host || !prec_host || !perm_host || !offsets_host || (T > 0 && (!X || !aligned(X, 16)))) {
    set_error("mbq_route_group: null pointer array or null/misaligned X");
    return MBQ_ERR_INVALID_ARG;
  }
  for (int i = 0; i < n_proj; ++i)
    if (!offsets_host[i] ||
        (T > 0 && (!Wr_host[i] || !br_host[i] || !prec_host[i] || !perm_host[i] || !aligned(Wr_host[i], 16)))) {
      set_error("mbq_route_group: null or misaligned pointer for projection %d", i);
      return MBQ_ERR_INVALID_ARG;
    }
  if (ws_bytes < mbq_route_workspace_bytes(T, K) || !ws || !aligned(ws, 256)) {
    set_error("mbq_route_group: workspace too small or misaligned (%zu < %zu)", ws_bytes,
              mbq_route_workspace_bytes(T, K));
    return MBQ_ERR_WORKSPACE;
  }
  return launch_route_group(X, T, K, n_proj, Wr_host, br_host, prec_host, perm_host, offsets_host, nullptr, ws,
                            (hipStream_t)stream, nullptr, 0, nullptr, false, *t_view);
}

size_t mbq_route_mlp_workspace_bytes(int64_t T, int64_t K, int H) {
  (void)K;
  if (T < 0 || H < 1 || H > route_mlp_max_hidden()) return 0;
  return route_mlp_workspace_bytes(T, H);
}

mbq_status mbq_route_mlp(const uint16_t* X, int64_t T, int64_t K, const float* W1, const float* b1, int H,
                         const float* W2, const float* b2, int E, double delta, int32_t* prec, int32_t* perm,
                         int32_t* offsets, double* scores, void* ws, size_t ws_bytes, void* stream) {
  if (E != MBQ_N_PRECISIONS || H < 1 || H > route_mlp_max_hidden()) {
    set_error("mbq_route_mlp: E=%d (must be %d) or hidden width %d outside 1..%d", E, MBQ_N_PRECISIONS, H,
              route_mlp_max_hidden());
    return MBQ_ERR_BAD_SHAPE;
  }
  if (T < 0 || K <= 0 || K % kGroup != 0 || T > (int64_t)1 << 24 || K > (int64_t)1 << 24) {
    set_error("mbq_route_mlp: bad sizes T=%lld K=%lld", (long long)T, (long long)K);
    return MBQ_ERR_BAD_SHAPE;
  }
  if (!offsets || (T > 0 && (!X || !W1 || !b1 || !W2 || !b2 || !prec || !perm)) || !aligned(X, 16) ||
      !aligned(W1, 16) || delta != delta) {
    set_error("mbq_route_mlp: null or misaligned pointer (X and W1 need 16-byte alignment) or delta is NaN");
    return MBQ_ERR_INVALID_ARG;
  }
  if (ws_bytes < mbq_route_mlp_workspace_bytes(T, K, H) || !ws || !aligned(ws, 256)) {
    set_error("mbq_route_mlp: workspace too small or misaligned (%zu < %zu)", ws_bytes,
              mbq_route_mlp_workspace_bytes(T, K, H));
    return MBQ_ERR_WORKSPACE;
  }
  return launch_route_mlp(X, T, K, W1, b1, H, W2, b2, delta, prec, perm, offsets, scores, ws, (hipStream_t)stream);
}

mbq_status mbq_threshold_quantile(const double* scores, int64_t T, int E, double rho, double* delta_out,
                                  void* stream) {
  if (E != MBQ_N_PRECISIONS || T < 1 || T > (int64_t)1 << 28) {
    set_error("mbq_threshold_quantile: E=%d (must be %d) or T=%lld outside 1..2^28", E, MBQ_N_PRECISIONS,
              (long long)T);
    return MBQ_ERR_BAD_SHAPE;
  }
  if (!scores || !delta_out || !(rho >= 0.0 && rho <= 1.0)) {
    set_error("mbq_threshold_quantile: null pointer or rho outside [0, 1]");
    return MBQ_ERR_INVALID_ARG;
  }
  const int64_t M = T * (E - 1);
  long long k = (long long)__builtin_floor(rho * (double)M + 0.5);
  if (k < 0) k = 0;
  if (k > M) k = M;
  return launch_threshold_quantile(scores, T, k, delta_out, (hipStream_t)stream);
}

mbq_status mbq_routed_linear_group(const uint16_t* X, int64_t T, int64_t K, int n_proj,
                                   const float* const* Wr_host, const float* const* br_host, int P,
                                   const void* const* blob_host, const int64_t* N_host, int32_t* const* prec_host,
                                   int32_t* const* perm_host, int32_t* const* offsets_host, float* const* Y_host,
                                   void* ws_route, size_t ws_route_bytes, void* ws_linear, size_t ws_linear_bytes,
                                   int algo, void* stream) {
  ApiScope scope;
  const uint16_t* XL = t_act ? t_act->aq.Xint : X;  // what the linear kernels multiply
  const ActArgs* aq = nullptr;
  if (t_view->shift != 0 || t_view->group != kGroup) {
    // A configuration with an odd cumulative width: the precision arrays count bits.  The loader-wavefront decode
    // kernels understand that (one token tile); every other shape goes through the slow
    // one-thread-per-output kernel, and so does every shape of a configuration with groups of 64 or 32 columns.
    // (T = 0: the routing call writes the empty offsets.)
    const bool bit_view = t_view->shift != 0;
    if (T == 0)  // the routing call checks its arguments and writes the empty offsets; there is nothing to multiply
      return mbq_route_group(X, T, K, n_proj, Wr_host, br_host, P, prec_host, perm_host, offsets_host, ws_route,
                             ws_route_bytes, stream);
    if (P != t_view->P || n_proj < 1 || n_proj > MBQ_MAX_GROUP || T < 0 || T > (int64_t)1 << 24 || K <= 0 ||
        K % kGroup != 0 || K > (int64_t)1 << 24) {
      set_error("mbq_routed_linear_group_cfg: bad sizes (P=%d, n_proj=%d, T=%lld, K=%lld)", P, n_proj, (long long)T,
                (long long)K);
      return MBQ_ERR_BAD_SHAPE;
    }
    if (algo < MBQ_ALGO_AUTO || algo > MBQ_ALGO_PREFILL || !N_host || !blob_host || !Y_host || !Wr_host || !br_host ||
        !prec_host || !perm_host || !offsets_host) {
      set_error("mbq_routed_linear_group_cfg: bad algo or null pointer array");
      return MBQ_ERR_INVALID_ARG;
    }
    for (int i = 0; i < n_proj; ++i)
      if (!Wr_host[i] || !aligned(Wr_host[i], 16) || !br_host[i] || !prec_host[i] || !perm_host[i] || !offsets_host[i]) {
        set_error("mbq_routed_linear_group_cfg: null or misaligned router pointer for projection %d", i);
        return MBQ_ERR_INVALID_ARG;
      }
    if (!ws_route || !aligned(ws_route, 256) || ws_route_bytes < mbq_route_workspace_bytes(T, K)) {
      set_error("mbq_routed_linear_group_cfg: route workspace too small or misaligned");
      return MBQ_ERR_WORKSPACE;
    }
    Shape sh[MBQ_MAX_GROUP];
    for (int i = 0; i < n_proj; ++i) {
      if (!make_shape(N_host[i], K, &sh[i], t_view->group)) return MBQ_ERR_BAD_SHAPE;
      if (!blob_host[i] || !aligned(blob_host[i], 256) || !Y_host[i] || !X || !aligned(X, 16)) {
        set_error("mbq_routed_linear_group_cfg: null or misaligned pointer for projection %d", i);
        return MBQ_ERR_INVALID_ARG;
      }
      if (!ws_linear || !aligned(ws_linear, 256) || ws_linear_bytes < mbq_linear_workspace_bytes(T, N_host[i], K)) {
        set_error("mbq_routed_linear_group_cfg: linear workspace too small or misaligned");
        return MBQ_ERR_WORKSPACE;
      }
    }
    if (bit_view && t_view->group == kGroup && algo != MBQ_ALGO_SIMPLE && algo != MBQ_ALGO_PREFILL && knob(3) == 0 &&
        decode_f4_takes_bit_view(T, sh[0]) && route_can_carry_prep(T)) {
      ZeroList zl;
      decode_f4_zero_list(T, n_proj, sh, Y_host, &zl);
      mbq_status st = launch_route_group(X, T, K, n_proj, Wr_host, br_host, prec_host, perm_host, offsets_host,
                                         nullptr, ws_route, (hipStream_t)stream, ws_linear, sh[0].KB, &zl, true,
                                         *t_view, XL);
      if (st != MBQ_OK) return st;
      return launch_linear_decode_f4(T, n_proj, blob_host, sh, prec_host, Y_host, ws_linear, (hipStream_t)stream,
                                     perm_host, offsets_host, nullptr, true);
    }
    mbq_status st = launch_route_group(X, T, K, n_proj, Wr_host, br_host, prec_host, perm_host, offsets_host, nullptr,
                                       ws_route, (hipStream_t)stream, nullptr, 0, nullptr, false, *t_view);
    if (st == MBQ_OK && bit_view && t_view->group == kGroup && (algo == MBQ_ALGO_AUTO || algo == MBQ_ALGO_DECODE) &&
        knob(3) == 0 && decode_f4_takes_bit_view(16, sh[0]))
      return bit_view_in_chunks(XL, T, n_proj, blob_host, sh, prec_host, Y_host, ws_linear, (hipStream_t)stream);
    for (int i = 0; st == MBQ_OK && i < n_proj; ++i)
      st = launch_linear_simple(XL, T, blob_host[i], sh[i], prec_host[i], Y_host[i], (hipStream_t)stream, bit_view);
    return st;
  }
  // the fused form: the router launch also prepares the activations of the decode kernel
  if (algo == MBQ_ALGO_AUTO || algo == MBQ_ALGO_DECODE) {
    Shape sh[MBQ_MAX_GROUP];
    bool ok = n_proj >= 1 && n_proj <= MBQ_MAX_GROUP && N_host && blob_host && Y_host && P == t_view->P &&
              T >= 1 && K > 0 && K % kGroup == 0 && X && aligned(X, 16) && Wr_host && br_host && prec_host &&
              perm_host && offsets_host && ws_route && aligned(ws_route, 256) &&
              ws_route_bytes >= mbq_route_workspace_bytes(T, K) && ws_linear && aligned(ws_linear, 256);
    for (int i = 0; ok && i < n_proj; ++i) {
      ok = N_host[i] > 0 && make_shape(N_host[i], K, &sh[i]) && blob_host[i] && aligned(blob_host[i], 256) &&
           Y_host[i] && Wr_host[i] && aligned(Wr_host[i], 16) && br_host[i] && prec_host[i] && perm_host[i] &&
           offsets_host[i] && ws_linear_bytes >= mbq_linear_workspace_bytes(T, N_host[i], K);
    }
    if (ok && knob(3) == 0 && decode_f4_supports(T, sh[0]) && route_can_carry_prep(T)) {
      ZeroList zl;
      decode_f4_zero_list(T, n_proj, sh, Y_host, &zl);
      mbq_status st = act_ahead(T, K, n_proj, prec_host, Y_host, N_host, ws_linear, ws_linear_bytes, &aq,
                                (hipStream_t)stream);
      if (st != MBQ_OK) return st;
      st = launch_route_group(X, T, K, n_proj, Wr_host, br_host, prec_host, perm_host, offsets_host, nullptr, ws_route,
                              (hipStream_t)stream, ws_linear, sh[0].KB, &zl, true, *t_view, XL, aq);
      if (st != MBQ_OK) return st;
      return launch_linear_decode_f4(T, n_proj, blob_host, sh, prec_host, Y_host, ws_linear, (hipStream_t)stream,
                                     perm_host, offsets_host, nullptr, false, t_act ? t_act->aq.row_scale : nullptr,
                                     t_act ? t_act->bias : nullptr, t_act ? &t_act->scaled : nullptr);
    }
    // up to 128 tokens with every matrix on the register-stationary kernel or, at 33 to 64, on that of wide matrices and long
    // rows: the router launch only writes the precisions (no meeting of its workgroups), clears what the former adds into and
    // leaves the sums that the latter starts from; the linear launches, one for the matrices of each kernel, sort the tokens
    // themselves.  (12288 and twice 1024 x 12288 at 64 tokens: a launch for each matrix 140 us, a launch for each kernel 110, the
    // register-stationary kernel for all three 161.)
    const int64_t defer_limit = (algo == MBQ_ALGO_AUTO) ? kMaxStationaryTokens : kMaxDecodeTokens;
    if (ok && T <= defer_limit && route_defers_sort(T)) {
      Sharing mid, stationary;
      bool all = true;
      for (int i = 0; i < n_proj; ++i) {
        Sharing* to = takes_mid_kernel(T, sh[i]) ? &mid
                      : (T <= kMaxDecodeTokens ? takes_stationary_kernel(T, sh[i]) : resolve_auto(T, sh[i]) == kAlgoStationary)
                          ? &stationary
                          : nullptr;
        all = all && to != nullptr;
        if (to) to->add(blob_host[i], sh[i], prec_host[i], perm_host[i], Y_host[i], perm_host[i], offsets_host[i]);
      }
      if (all) {
        const hipStream_t s = (hipStream_t)stream;
        ZeroList zl;
        stationary.zero_list(T, &zl);
        const bool sums = mid.n > 0;
        mbq_status st = act_ahead(T, K, n_proj, prec_host, Y_host, N_host, sums ? ws_linear : nullptr,
                                  sums ? ws_linear_bytes : 0, &aq, s);
        if (st != MBQ_OK) return st;
        const bool sums_here = sums && t_act && !aq;  // the routers read the rebuilt activations, the linear launch the integers
        st = launch_route_group(X, T, K, n_proj, Wr_host, br_host, prec_host, perm_host, offsets_host, nullptr, ws_route, s,
                                nullptr, 0, &zl, true, *t_view, nullptr, aq, sums && !sums_here ? ws_linear : nullptr);
        if (st == MBQ_OK && sums_here) st = launch_mid_sums(XL, T, K, ws_linear, s);
        if (st == MBQ_OK) st = mid.launch_mid(XL, T, ws_linear, s, true);
        if (st == MBQ_OK) st = stationary.launch_stationary(XL, T, s, true);
        return st;
      }
    }
  }
  // above 128 tokens with every matrix on the prefill kernel: the router launch also does the work of its pre-kernel
  // (on compute units that the routers leave idle; the launch of its own took 10 us twice in a 7B-shaped MLP at 2048 tokens,
  // 667 -> 653 us, 40 us twice in a 70B-shaped one at 4096, 5380 -> 5345; at 256 tokens 667 either way)
  if (algo == MBQ_ALGO_AUTO || algo == MBQ_ALGO_PREFILL) {
    Shape sh[MBQ_MAX_GROUP];
    bool ok = n_proj >= 1 && n_proj <= MBQ_MAX_GROUP && N_host && blob_host && Y_host && P == t_view->P &&
              T > kMaxDecodeTokens && T <= (int64_t)1 << 24 && !route_defers_sort(T) && K > 0 && K % kGroup == 0 &&
              K <= (int64_t)1 << 24 && X && aligned(X, 16) && XL && aligned(XL, 16) && Wr_host && br_host && prec_host &&
              perm_host && offsets_host && ws_route && aligned(ws_route, 256) &&
              ws_route_bytes >= mbq_route_workspace_bytes(T, K) && ws_linear && aligned(ws_linear, 256);
    for (int i = 0; ok && i < n_proj; ++i)
      ok = N_host[i] > 0 && make_shape(N_host[i], K, &sh[i]) && blob_host[i] && aligned(blob_host[i], 256) &&
           Y_host[i] && Wr_host[i] && aligned(Wr_host[i], 16) && br_host[i] && prec_host[i] && perm_host[i] &&
           offsets_host[i] && ws_linear_bytes >= mbq_linear_workspace_bytes(T, N_host[i], K) &&
           (algo == MBQ_ALGO_PREFILL || resolve_auto(T, sh[i]) == MBQ_ALGO_PREFILL);
    PrefillPrep prep;
    if (ok && prefill_prep_of(XL, T, n_proj, sh, Y_host, ws_linear, &prep)) {
      mbq_status st = act_ahead(T, K, 0, nullptr, nullptr, nullptr, nullptr, 0, &aq, (hipStream_t)stream);
      if (st != MBQ_OK) return st;
      st = launch_route_group(X, T, K, n_proj, Wr_host, br_host, prec_host, perm_host, offsets_host, nullptr, ws_route,
                              (hipStream_t)stream, nullptr, 0, nullptr, false, *t_view, nullptr, nullptr, nullptr, &prep);
      if (st != MBQ_OK) return st;
      return launch_linear_prefill_group(XL, T, n_proj, blob_host, sh, perm_host, offsets_host, Y_host, ws_linear,
                                         (hipStream_t)stream, true);
    }
  }
  // otherwise exactly the two calls (they check the arguments)
  mbq_status st = MBQ_OK;
  if (T > 0) st = act_ahead(T, K, 0, nullptr, nullptr, nullptr, nullptr, 0, &aq, (hipStream_t)stream);
  if (st != MBQ_OK) return st;
  st = mbq_route_group(X, T, K, n_proj, Wr_host, br_host, P, prec_host, perm_host, offsets_host,
                                  ws_route, ws_route_bytes, stream);
  if (st != MBQ_OK) return st;
  return mbq_linear_group(XL, T, K, n_proj, blob_host, N_host, prec_host, perm_host, offsets_host, Y_host, ws_linear,
                          ws_linear_bytes, algo, stream);
}

mbq_status mbq_linear(const uint16_t* X, int64_t T, const void* blob, int64_t N, int64_t K,
                      const int32_t* prec, const int32_t* perm, const int32_t* offsets, float* Y, void* ws,
                      size_t ws_bytes, int algo, void* stream) {
  ApiScope scope;
  Shape sh;
  if (!make_shape(N, K, &sh)) return MBQ_ERR_BAD_SHAPE;
  if (T < 0 || T > (int64_t)1 << 24) {
    set_error("mbq_linear: bad token count %lld", (long long)T);
    return MBQ_ERR_BAD_SHAPE;
  }
  if (algo < MBQ_ALGO_AUTO || algo > MBQ_ALGO_PREFILL) {
    set_error("mbq_linear: unknown algo %d", algo);
    return MBQ_ERR_INVALID_ARG;
  }
  if (T == 0) return MBQ_OK;
  if (!X || !blob || !prec || !perm || !offsets || !Y || !aligned(blob, 256) || !aligned(X, 16)) {
    set_error("mbq_linear: null or misaligned pointer (X 16-byte, blob 256-byte alignment)");
    return MBQ_ERR_INVALID_ARG;
  }
  if (!ws || !aligned(ws, 256) || ws_bytes < mbq_linear_workspace_bytes(T, N, K)) {
    set_error("mbq_linear: workspace too small or misaligned (%zu < %zu)", ws_bytes,
              mbq_linear_workspace_bytes(T, N, K));
    return MBQ_ERR_WORKSPACE;
  }
  if (algo == MBQ_ALGO_AUTO) algo = resolve_auto(T, sh);
  if (algo == MBQ_ALGO_DECODE && T > kMaxDecodeTokens) {
    set_error("mbq_linear: the decode kernel handles at most %d tokens (T=%lld)", kMaxDecodeTokens,
              (long long)T);
    return MBQ_ERR_BAD_SHAPE;
  }
  return dispatch_linear(X, T, blob, sh, prec, perm, offsets, Y, ws, algo, (hipStream_t)stream);
}

mbq_status mbq_linear_group(const uint16_t* X, int64_t T, int64_t K, int n_proj, const void* const* blob_host,
                            const int64_t* N_host, const int32_t* const* prec_host,
                            const int32_t* const* perm_host, const int32_t* const* offsets_host,
                            float* const* Y_host, void* ws, size_t ws_bytes, int algo, void* stream) {
  ApiScope scope;
  if (n_proj < 1 || n_proj > MBQ_MAX_GROUP) {
    set_error("mbq_linear_group: n_proj=%d outside 1..%d", n_proj, MBQ_MAX_GROUP);
    return MBQ_ERR_INVALID_ARG;
  }
  if (!blob_host || !N_host || !prec_host || !perm_host || !offsets_host || !Y_host) {
    set_error("mbq_linear_group: null pointer array");
    return MBQ_ERR_INVALID_ARG;
  }
  if (T < 0 || T > (int64_t)1 << 24) {
    set_error("mbq_linear_group: bad token count %lld", (long long)T);
    return MBQ_ERR_BAD_SHAPE;
  }
  if (algo < MBQ_ALGO_AUTO || algo > MBQ_ALGO_PREFILL) {
    set_error("mbq_linear_group: unknown algo %d", algo);
    return MBQ_ERR_INVALID_ARG;
  }
  Shape sh[MBQ_MAX_GROUP];
  size_t need = 0;
  for (int i = 0; i < n_proj; ++i) {
    if (!make_shape(N_host[i], K, &sh[i])) return MBQ_ERR_BAD_SHAPE;
    const size_t b = mbq_linear_workspace_bytes(T, N_host[i], K);
    if (b > need) need = b;
  }
  if (T == 0) return MBQ_OK;
  if (!X || !aligned(X, 16)) {
    set_error("mbq_linear_group: null or misaligned X");
    return MBQ_ERR_INVALID_ARG;
  }
  for (int i = 0; i < n_proj; ++i)
    if (!blob_host[i] || !prec_host[i] || !perm_host[i] || !offsets_host[i] || !Y_host[i] ||
        !aligned(blob_host[i], 256)) {
      set_error("mbq_linear_group: null or misaligned pointer for projection %d", i);
      return MBQ_ERR_INVALID_ARG;
    }
  if (!ws || !aligned(ws, 256) || ws_bytes < need) {
    set_error("mbq_linear_group: workspace too small or misaligned (%zu < %zu)", ws_bytes, need);
    return MBQ_ERR_WORKSPACE;
  }
  int algo_of[MBQ_MAX_GROUP];  // per matrix: AUTO may pick different kernels above the decode limit
  bool all_stationary = true;
  for (int i = 0; i < n_proj; ++i) {
    algo_of[i] = algo == MBQ_ALGO_AUTO ? resolve_auto(T, sh[i]) : algo;
    all_stationary = all_stationary && algo_of[i] == kAlgoStationary;
  }
  if (algo == MBQ_ALGO_AUTO) algo = all_stationary ? kAlgoStationary : (T <= kMaxDecodeTokens ? MBQ_ALGO_DECODE : MBQ_ALGO_PREFILL);
  if (algo == MBQ_ALGO_DECODE && T > kMaxDecodeTokens) {
    set_error("mbq_linear_group: the decode kernel handles at most %d tokens (T=%lld)", kMaxDecodeTokens,
              (long long)T);
    return MBQ_ERR_BAD_SHAPE;
  }
  hipStream_t s = (hipStream_t)stream;
  if (algo == MBQ_ALGO_DECODE && knob(3) == 0 && decode_f4_supports(T, sh[0])) {
    ZeroList zl;
    decode_f4_zero_list(T, n_proj, sh, Y_host, &zl);
    mbq_status st = launch_decode_f4_prep(X, T, K, sh[0].KB, ws, zl, s);
    if (st != MBQ_OK) return st;
    return launch_linear_decode_f4(T, n_proj, blob_host, sh, prec_host, Y_host, ws, s, nullptr, nullptr);
  }
  if (algo == MBQ_ALGO_DECODE || algo == kAlgoStationary) {
    // the matrices of the kernel of wide matrices and long rows share a launch, and those of the register-stationary kernel
    // when no other is left over
    Sharing mid, stationary;
    for (int i = 0; i < n_proj; ++i) {
      Sharing* to = algo == MBQ_ALGO_DECODE && takes_mid_kernel(T, sh[i]) ? &mid
                    : takes_stationary_kernel(T, sh[i])                   ? &stationary
                                                                          : nullptr;
      if (to) to->add(blob_host[i], sh[i], prec_host[i], perm_host[i], Y_host[i], nullptr, nullptr);
    }
    mbq_status st = MBQ_OK;
    if (mid.n > 0) {
      st = launch_mid_sums(X, T, K, ws, s);
      if (st == MBQ_OK) st = mid.launch_mid(X, T, ws, s, false);
      if (st != MBQ_OK) return st;
    }
    if (mid.n + stationary.n == n_proj) {
      ZeroList zl;
      stationary.zero_list(T, &zl);
      st = launch_zero_outputs(zl, s);
      return st == MBQ_OK ? stationary.launch_stationary(X, T, s, false) : st;
    }
    for (int i = 0; i < n_proj && mid.n > 0; ++i) {
      if (takes_mid_kernel(T, sh[i])) continue;
      st = dispatch_linear(X, T, blob_host[i], sh[i], prec_host[i], perm_host[i], offsets_host[i], Y_host[i], ws, algo_of[i], s);
      if (st != MBQ_OK) return st;
    }
    if (mid.n > 0) return MBQ_OK;
  }
  // the matrices that take the prefill kernel share a launch; the others follow one by one
  const void* pf_blob[MBQ_MAX_GROUP];
  Shape pf_shape[MBQ_MAX_GROUP];
  const int32_t* pf_perm[MBQ_MAX_GROUP];
  const int32_t* pf_offsets[MBQ_MAX_GROUP];
  float* pf_Y[MBQ_MAX_GROUP];
  int n_pf = 0;
  for (int i = 0; i < n_proj; ++i)
    if (algo_of[i] == MBQ_ALGO_PREFILL) {
      pf_blob[n_pf] = blob_host[i];
      pf_shape[n_pf] = sh[i];
      pf_perm[n_pf] = perm_host[i];
      pf_offsets[n_pf] = offsets_host[i];
      pf_Y[n_pf++] = Y_host[i];
    }
  if (n_pf > 0) {
    mbq_status st = launch_linear_prefill_group(X, T, n_pf, pf_blob, pf_shape, pf_perm, pf_offsets, pf_Y, ws, s);
    if (st != MBQ_OK) return st;
  }
  for (int i = 0; i < n_proj; ++i) {
    if (algo_of[i] == MBQ_ALGO_PREFILL) continue;
    mbq_status st =
        dispatch_linear(X, T, blob_host[i], sh[i], prec_host[i], perm_host[i], offsets_host[i], Y_host[i], ws, algo_of[i], s);
    if (st != MBQ_OK) return st;
  }
  return MBQ_OK;
}

// ---- other slice configurations (Sec. 4.1 general E and b_e; App. C.1 slice_bits_list) ---------------------------
// The blob holds the eight-bit code of every weight as four base-4 digits whatever the configuration: a
// configuration whose slices end on digit boundaries cuts the same code at other places (a 4-bit slice with the
// centred zero point 8 and scale s/16 IS two 2-bit slices with zero point 2 and scales s/4, s/16), and its first-slice
// parameters are the stored ones moved by a power of two.  So only the router (how many outputs, which digit count
// each stands for) and the checking helpers know about it.

mbq_status mbq_config_check(const mbq_config* cfg) {
  RouteView v;
  return make_view(cfg, &v, "mbq_config_check") ? MBQ_OK : MBQ_ERR_BAD_SHAPE;
}

int mbq_config_bits(const mbq_config* cfg, int p) {
  RouteView v;
  if (!make_view(cfg, &v, "mbq_config_bits") || p < 0 || p >= v.P) return -1;
  return v.bits[p];
}

int mbq_config_precision_value(const mbq_config* cfg, int p) {
  RouteView v;
  if (!make_view(cfg, &v, "mbq_config_precision_value") || p < 0 || p >= v.P) return -1;
  return v.value[p];
}

int mbq_config_counts_bits(const mbq_config* cfg) {
  RouteView v;
  if (!make_view(cfg, &v, "mbq_config_counts_bits")) return -1;
  return v.shift;
}

size_t mbq_blob_bytes_cfg(const mbq_config* cfg, int64_t N, int64_t K) {
  RouteView v;
  Shape sh;
  return make_view(cfg, &v, "mbq_blob_bytes_cfg") && make_shape(N, K, &sh, v.group) ? sh.bytes : 0;
}

mbq_status mbq_encode_cfg(const float* W, int64_t N, int64_t K, const mbq_config* cfg, void* blob, void* stream) {
  RouteView v;
  if (!make_view(cfg, &v, "mbq_encode_cfg")) return MBQ_ERR_BAD_SHAPE;
  if (v.group == kGroup) return mbq_encode(W, N, K, blob, stream);
  Shape sh;
  if (!make_shape(N, K, &sh, v.group)) return MBQ_ERR_BAD_SHAPE;
  if (!W || !blob || !aligned(blob, 256) || !aligned(W, 16)) {
    set_error("mbq_encode_cfg: W must be 16-byte and blob 256-byte aligned and non-null");
    return MBQ_ERR_INVALID_ARG;
  }
  return launch_encode_small_group(W, sh, blob, (hipStream_t)stream);
}

mbq_status mbq_unpack_cfg(const void* blob, int64_t N, int64_t K, const mbq_config* cfg, uint8_t* codes,
                          float* scale, float* zero, void* stream) {
  RouteView v;
  if (!make_view(cfg, &v, "mbq_unpack_cfg")) return MBQ_ERR_BAD_SHAPE;
  Shape sh;
  if (!make_shape(N, K, &sh, v.group)) return MBQ_ERR_BAD_SHAPE;
  if (!blob || !aligned(blob, 256)) {
    set_error("mbq_unpack_cfg: blob must be non-null and 256-byte aligned");
    return MBQ_ERR_INVALID_ARG;
  }
  return launch_unpack_view(blob, sh, v, codes, scale, zero, (hipStream_t)stream);
}

mbq_status mbq_dequant_cfg(const void* blob, int64_t N, int64_t K, const mbq_config* cfg, int p, float* What,
                           void* stream) {
  RouteView v;
  if (!make_view(cfg, &v, "mbq_dequant_cfg")) return MBQ_ERR_BAD_SHAPE;
  if (p < 0 || p >= v.P) {
    set_error("mbq_dequant_cfg: precision index %d outside 0..%d", p, v.P - 1);
    return MBQ_ERR_INVALID_ARG;
  }
  Shape sh;
  if (!make_shape(N, K, &sh, v.group)) return MBQ_ERR_BAD_SHAPE;
  if (!blob || !What || !aligned(blob, 256)) {
    set_error("mbq_dequant_cfg: null or misaligned pointer");
    return MBQ_ERR_INVALID_ARG;
  }
  return launch_dequant_bits(blob, sh, v.bits[p], What, (hipStream_t)stream);
}

mbq_status mbq_linear_cfg(const uint16_t* X, int64_t T, const void* blob, int64_t N, int64_t K,
                          const mbq_config* cfg, const int32_t* prec, const int32_t* perm, const int32_t* offsets,
                          float* Y, void* ws, size_t ws_bytes, int algo, void* stream) {
  RouteView v;
  if (!make_view(cfg, &v, "mbq_linear_cfg")) return MBQ_ERR_BAD_SHAPE;
  if (v.shift == 0 && v.group == kGroup)
    return mbq_linear(X, T, blob, N, K, prec, perm, offsets, Y, ws, ws_bytes, algo, stream);
  ApiScope scope;
  Shape sh;
  if (!make_shape(N, K, &sh, v.group)) return MBQ_ERR_BAD_SHAPE;
  if (T < 0 || T > (int64_t)1 << 24) {
    set_error("mbq_linear_cfg: bad token count %lld", (long long)T);
    return MBQ_ERR_BAD_SHAPE;
  }
  if (algo < MBQ_ALGO_AUTO || algo > MBQ_ALGO_PREFILL) {
    set_error("mbq_linear_cfg: unknown algo %d", algo);
    return MBQ_ERR_INVALID_ARG;
  }
  if (T == 0) return MBQ_OK;
  if (!X || !blob || !prec || !Y || !aligned(blob, 256) || !aligned(X, 16)) {
    set_error("mbq_linear_cfg: null or misaligned pointer (X 16-byte, blob 256-byte alignment)");
    return MBQ_ERR_INVALID_ARG;
  }
  if (!ws || !aligned(ws, 256) || ws_bytes < mbq_linear_workspace_bytes(T, N, K)) {
    set_error("mbq_linear_cfg: workspace too small or misaligned (%zu < %zu)", ws_bytes,
              mbq_linear_workspace_bytes(T, N, K));
    return MBQ_ERR_WORKSPACE;
  }
  hipStream_t s = (hipStream_t)stream;
  if (v.group == kGroup && algo != MBQ_ALGO_SIMPLE && algo != MBQ_ALGO_PREFILL && knob(3) == 0 &&
      decode_f4_takes_bit_view(T, sh)) {
    ZeroList zl;
    decode_f4_zero_list(T, 1, &sh, &Y, &zl);
    mbq_status st = launch_decode_f4_prep(X, T, sh.K, sh.KB, ws, zl, s);
    if (st != MBQ_OK) return st;
    return launch_linear_decode_f4(T, 1, &blob, &sh, &prec, &Y, ws, s, nullptr, nullptr, nullptr, true);
  }
  if (v.shift != 0 && v.group == kGroup && (algo == MBQ_ALGO_AUTO || algo == MBQ_ALGO_DECODE) && knob(3) == 0 &&
      decode_f4_takes_bit_view(16, sh))
    return bit_view_in_chunks(X, T, 1, &blob, &sh, &prec, &Y, ws, s);
  return launch_linear_simple(X, T, blob, sh, prec, Y, s, v.shift != 0);
}

mbq_status mbq_route_cfg(const uint16_t* X, int64_t T, int64_t K, const float* Wr, const float* br,
                         const mbq_config* cfg, int32_t* prec, int32_t* perm, int32_t* offsets, double* logits,
                         void* ws, size_t ws_bytes, void* stream) {
  RouteView v;
  if (!make_view(cfg, &v, "mbq_route_cfg")) return MBQ_ERR_BAD_SHAPE;
  ViewScope scope(&v);
  return mbq_route(X, T, K, Wr, br, v.P, prec, perm, offsets, logits, ws, ws_bytes, stream);
}

mbq_status mbq_route_group_cfg(const uint16_t* X, int64_t T, int64_t K, int n_proj, const float* const* Wr_host,
                               const float* const* br_host, const mbq_config* cfg, int32_t* const* prec_host,
                               int32_t* const* perm_host, int32_t* const* offsets_host, void* ws, size_t ws_bytes,
                               void* stream) {
  RouteView v;
  if (!make_view(cfg, &v, "mbq_route_group_cfg")) return MBQ_ERR_BAD_SHAPE;
  ViewScope scope(&v);
  return mbq_route_group(X, T, K, n_proj, Wr_host, br_host, v.P, prec_host, perm_host, offsets_host, ws, ws_bytes,
                         stream);
}

mbq_status mbq_routed_linear_group_cfg(const uint16_t* X, int64_t T, int64_t K, int n_proj,
                                       const float* const* Wr_host, const float* const* br_host,
                                       const mbq_config* cfg, const void* const* blob_host, const int64_t* N_host,
                                       int32_t* const* prec_host, int32_t* const* perm_host,
                                       int32_t* const* offsets_host, float* const* Y_host, void* ws_route,
                                       size_t ws_route_bytes, void* ws_linear, size_t ws_linear_bytes, int algo,
                                       void* stream) {
  RouteView v;
  if (!make_view(cfg, &v, "mbq_routed_linear_group_cfg")) return MBQ_ERR_BAD_SHAPE;
  ViewScope scope(&v);
  return mbq_routed_linear_group(X, T, K, n_proj, Wr_host, br_host, v.P, blob_host, N_host, prec_host, perm_host,
                                 offsets_host, Y_host, ws_route, ws_route_bytes, ws_linear, ws_linear_bytes, algo,
                                 stream);
}

static mbq_status check_act_quant(const uint16_t* X, int64_t T, int64_t K, int abits, const float* let_shift,
                                  const float* let_scale, const uint16_t* Xint, const float* row_scale,
                                  const uint16_t* Xr) {
  if (T < 0 || K <= 0 || K % kGroup != 0 || T > (int64_t)1 << 24 || K > (int64_t)1 << 24) {
    set_error("mbq_act_quant: bad sizes (T=%lld, K=%lld; K must be a multiple of %d)", (long long)T, (long long)K,
              kGroup);
    return MBQ_ERR_BAD_SHAPE;
  }
  if (abits < 2 || abits > 8) {
    set_error("mbq_act_quant: abits = %d, supported 2..8", abits);
    return MBQ_ERR_INVALID_ARG;
  }
  if ((let_shift == nullptr) != (let_scale == nullptr)) {
    set_error("mbq_act_quant: pass both the shift and the scale of the transform, or neither");
    return MBQ_ERR_INVALID_ARG;
  }
  if (T == 0) return MBQ_OK;
  if (!X || !Xint || !row_scale || !aligned(X, 16) || !aligned(Xint, 16) || !aligned(Xr, 16) ||
      !aligned(let_shift, 16) || !aligned(let_scale, 16)) {
    set_error("mbq_act_quant: null or misaligned pointer (16-byte alignment for X, Xint, Xr, shift and scale)");
    return MBQ_ERR_INVALID_ARG;
  }
  return MBQ_OK;
}

mbq_status mbq_act_quant(const uint16_t* X, int64_t T, int64_t K, int abits, const float* let_shift,
                         const float* let_scale, uint16_t* Xint, float* row_scale, uint16_t* Xr, void* stream) {
  const mbq_status st = check_act_quant(X, T, K, abits, let_shift, let_scale, Xint, row_scale, Xr);
  if (st != MBQ_OK || T == 0) return st;
  return launch_act_quant(X, T, K, abits, let_shift, let_scale, Xint, row_scale, Xr, (hipStream_t)stream);
}

mbq_status mbq_routed_linear_group_act(const uint16_t* X, int64_t T, int64_t K, int abits, const float* let_shift,
                                       const float* let_scale, int n_proj, const float* const* Wr_host,
                                       const float* const* br_host, int P, const void* const* blob_host,
                                       const int64_t* N_host, const float* const* bias_host,
                                       int32_t* const* prec_host, int32_t* const* perm_host,
                                       int32_t* const* offsets_host, float* const* Y_host, uint16_t* Xint,
                                       float* row_scale, uint16_t* Xr, void* ws_route, size_t ws_route_bytes,
                                       void* ws_linear, size_t ws_linear_bytes, int algo, void* stream) {
  ApiScope scope;
  if (n_proj < 1 || n_proj > MBQ_MAX_GROUP || !N_host || !Y_host) {
    set_error("mbq_routed_linear_group_act: n_proj = %d (1..%d) or a null N / Y array", n_proj, MBQ_MAX_GROUP);
    return MBQ_ERR_INVALID_ARG;
  }
  if (T > 0 && !Xr) {
    set_error("mbq_routed_linear_group_act: the buffer for the router's input is null");
    return MBQ_ERR_INVALID_ARG;
  }
  for (int i = 0; i < n_proj; ++i)
    if (N_host[i] <= 0 || N_host[i] > (int64_t)1 << 24 || (T > 0 && !Y_host[i])) {
      set_error("mbq_routed_linear_group_act: bad N or null Y for projection %d", i);
      return MBQ_ERR_INVALID_ARG;
    }
  mbq_status st = check_act_quant(X, T, K, abits, let_shift, let_scale, Xint, row_scale, Xr);
  if (st != MBQ_OK) return st;
  ActStage stage = {{X, let_shift, let_scale, Xint, row_scale, Xr, abits}, bias_host, false};
  {
    ActScope act_scope(&stage);
    st = mbq_routed_linear_group(Xr, T, K, n_proj, Wr_host, br_host, P, blob_host, N_host, prec_host, perm_host,
                                 offsets_host, Y_host, ws_route, ws_route_bytes, ws_linear, ws_linear_bytes, algo,
                                 stream);
  }
  if (st != MBQ_OK || T == 0 || stage.scaled) return st;
  return launch_scale_rows_group(n_proj, Y_host, T, N_host, row_scale, bias_host, (hipStream_t)stream);
}

mbq_status mbq_scale_rows(float* Y, int64_t T, int64_t N, const float* row_scale, const float* bias, void* stream) {
  if (T < 0 || N <= 0 || T > (int64_t)1 << 24 || N > (int64_t)1 << 24) {
    set_error("mbq_scale_rows: bad sizes (T=%lld, N=%lld)", (long long)T, (long long)N);
    return MBQ_ERR_BAD_SHAPE;
  }
  if (T == 0) return MBQ_OK;
  if (!Y || !row_scale) {
    set_error("mbq_scale_rows: null pointer");
    return MBQ_ERR_INVALID_ARG;
  }
  return launch_scale_rows(Y, T, N, row_scale, bias, (hipStream_t)stream);
}

}  // extern "C"
