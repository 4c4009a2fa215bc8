// Router scores + argmax (paper Sec. 4.2 Eq. 4, read as one linear map to four
// logits) and the token permutation by precision (Sec. 4.3, challenge 3).
#include "mbq_act_quant.h"
#include "mbq_common.h"
#include "mbq_f4_prep.h"

namespace mbq {

constexpr int kP = MBQ_N_PRECISIONS;

__device__ inline float bf16_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ inline float bf16_hi(uint32_t u) { return __uint_as_float(u & 0xFFFF0000u); }

// Stable counting sort of token ids by precision by ONE workgroup of NW wavefronts
// (Sec. 4.3, token permutation).  Counting and ranking use wavefront ballots: a lane's rank
// inside its wavefront is the population count of the ballot below its lane.
template <int NW>
__device__ inline void bucket_by_workgroup(const int32_t* prec, int64_t T,
                                           int32_t* __restrict__ perm, int32_t* __restrict__ offsets, int shift = 0) {
  __shared__ int s_wave[NW][kP];  // per-wavefront counts of the current pass
  __shared__ int s_run[kP];       // running write position of each precision
  constexpr int NT = NW * 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));

  // pass 1: totals
  int cnt[kP] = {0, 0, 0, 0};
  for (int64_t base = 0; base < T; base += NT) {
    const int64_t i = base + tid;
    const int p = (i < T) ? (prec[i] >> shift) : -1;
#pragma unroll
    for (int q = 0; q < kP; ++q) cnt[q] += __popcll(__ballot(p == q));
  }
  if (lane == 0)
#pragma unroll
    for (int q = 0; q < kP; ++q) s_wave[wave][q] = cnt[q];
  __syncthreads();
  if (tid == 0) {
    int pos = 0;
    for (int q = 0; q < kP; ++q) {
      int c = 0;
      for (int w = 0; w < NW; ++w) c += s_wave[w][q];
      s_run[q] = pos;
      offsets[q] = pos;
      pos += c;
    }
    offsets[kP] = pos;
  }
  __syncthreads();

  // pass 2: stable placement, NT tokens at a time in token order
  for (int64_t base = 0; base < T; base += NT) {
    const int64_t i = base + tid;
    const int p = (i < T) ? (prec[i] >> shift) : -1;
    int rank_in_wave = 0;
#pragma unroll
    for (int q = 0; q < kP; ++q) {
      const uint64_t b = __ballot(p == q);
      if (p == q) rank_in_wave = __popcll(b & below);
      if (lane == 0) s_wave[wave][q] = __popcll(b);
    }
    __syncthreads();
    if (p >= 0) {
      int pos = s_run[p] + rank_in_wave;
      for (int w = 0; w < wave; ++w) pos += s_wave[w][p];
      perm[pos] = (int32_t)i;
    }
    __syncthreads();
    if (tid < kP) {
      int c = 0;
      for (int w = 0; w < NW; ++w) c += s_wave[w][tid];
      s_run[tid] += c;
    }
    __syncthreads();
  }
}

// Cross-lane moves of a double through the data-parallel-primitive path of the vector ALU (no LDS
// round trip as for a general shuffle): CTRL is a DPP control word, here a permutation inside each
// group of four lanes (quad_perm) or a rotation inside each row of 16 lanes (row_ror).
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
  const long long b = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b & 0xFFFFFFFFll), CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, false);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (long long)(unsigned)lo);
}
constexpr int kDppQuadXor1 = 0xB1, kDppQuadXor2 = 0x4E;  // quad_perm [1,0,3,2], [2,3,0,1]
constexpr int kDppRowRor4 = 0x124, kDppRowRor8 = 0x128;

// Sums four per-lane values over the wavefront.  The first two exchanges halve the number of values a
// lane carries (lanes 1 apart split the four between them, then lanes 2 apart), so that seven moves of
// a double do the work of twenty-four; afterwards lane l holds the total of value wave_sum4_index(l).
__device__ __forceinline__ int wave_sum4_index(int lane) { return 2 * (lane & 1) + ((lane >> 1) & 1); }
__device__ __forceinline__ double wave_sum4(const double (&acc)[4], int lane) {
  const bool odd = (lane & 1) != 0, upper = (lane & 2) != 0;
  double keep0 = odd ? acc[2] : acc[0], keep1 = odd ? acc[3] : acc[1];
  keep0 += dpp_move<kDppQuadXor1>(odd ? acc[0] : acc[2]);
  keep1 += dpp_move<kDppQuadXor1>(odd ? acc[1] : acc[3]);
  double v = upper ? keep1 : keep0;
  v += dpp_move<kDppQuadXor2>(upper ? keep0 : keep1);
  v += dpp_move<kDppRowRor4>(v);
  v += dpp_move<kDppRowRor8>(v);
  v += __shfl_xor(v, 16, 64);
  v += __shfl_xor(v, 32, 64);
  return v;
}

constexpr int kRouteGroupMax = MBQ_MAX_GROUP;

struct RouteOut {
  const float* Wr;
  const float* br;
  int32_t* prec;
  int32_t* perm;
  int32_t* offsets;
  double* logits;
};
struct RouteGroup {
  RouteOut r[kRouteGroupMax];
  RouteView view;
};

typedef double f64x4 __attribute__((ext_vector_type(4)));

// The product of 16 token rows with 16 weight rows in fp64 on the matrix cores, by NW wavefronts that take the K axis in
// blocks of 32 columns in turn.  One v_mfma_f64_16x16x4 takes A[token i][k] from lane i + 16 k and B[k][unit j] from lane
// j + 16 k, so a lane reads 8 consecutive columns of its token's row and of its unit's row (16-byte loads) and feeds them
// to 8 MFMAs, column c of every lane quarter forming the K = 4 of MFMA c (bf16 x fp32 products are exact in fp64).
// The result lane l, register r is D[token 4 r + l / 16][unit l % 16].
// A wavefront's chain is load, eight MFMAs, load: what bounds small launches is the number of trips to memory one after
// the other, so sixteen wavefronts share a tile and two blocks are requested at a time.
template <int NW>
__device__ __forceinline__ f64x4 tile_product(const uint16_t* __restrict__ xrow, const float* __restrict__ wrow, int64_t K,
                                              int wave, int lane) {
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
  auto feed = [&](const uint4& xv, const float4& wa, const float4& wb) {
    const double x[8] = {bf16_lo(xv.x), bf16_hi(xv.x), bf16_lo(xv.y), bf16_hi(xv.y),
                         bf16_lo(xv.z), bf16_hi(xv.z), bf16_lo(xv.w), bf16_hi(xv.w)};
    const double w[8] = {wa.x, wa.y, wa.z, wa.w, wb.x, wb.y, wb.z, wb.w};
#pragma unroll
    for (int c = 0; c < 8; ++c) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x[c], w[c], acc, 0, 0, 0);
  };
  constexpr int kStep = NW * 32;
  int64_t k0 = (int64_t)wave * 32;  // (K is a multiple of 128: a block of 32 is there or not, for all lanes alike)
  const int at = (lane >> 4) * 8;
#pragma unroll 1
  for (; k0 + kStep < K; k0 += 2 * kStep) {
    const int64_t k = k0 + at;
    const uint4 xa = *reinterpret_cast<const uint4*>(xrow + k), xb = *reinterpret_cast<const uint4*>(xrow + k + kStep);
    const float4 wa0 = *reinterpret_cast<const float4*>(wrow + k), wa1 = *reinterpret_cast<const float4*>(wrow + k + 4);
    const float4 wb0 = *reinterpret_cast<const float4*>(wrow + k + kStep);
    const float4 wb1 = *reinterpret_cast<const float4*>(wrow + k + kStep + 4);
    feed(xa, wa0, wa1);
    feed(xb, wb0, wb1);
  }
  if (k0 < K) {
    const int64_t k = k0 + at;
    feed(*reinterpret_cast<const uint4*>(xrow + k), *reinterpret_cast<const float4*>(wrow + k),
         *reinterpret_cast<const float4*>(wrow + k + 4));
  }
  return acc;
}
constexpr int kTileWaves = 16;

// General router, many tokens: one workgroup scores 16 tokens for ALL routers of the call (up to four of up to four outputs
// each are the 16 weight rows of a tile), so the tokens are read once per stage.  Its time is that of one tile's fp64
// MFMAs, about 3.1 ns x K, while a compute unit has at most one tile (T <= 4096): taken above 1024 tokens.  7B-shaped
// stages at 2048 tokens 26 us on average, where a launch of vector code per router took 31; 70B-shaped ones at 4096 tokens
// 59 us instead of 132 a stage; at 256 tokens it would be 52 instead of 23.
__global__ __launch_bounds__(64 * kTileWaves) void route_kernel(const uint16_t* __restrict__ X, int64_t T, int64_t K,
                                                                const RouteGroup group, int n, const PrefillPrep pf) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t tok0 = (int64_t)blockIdx.x * 16;
  if (blockIdx.y == 1) {  // (only with pf) these workgroups run beside the tiles', which leave the memory pipes idle
    prefill_prep_share(pf, T, K, tok0, 16, 64 * kTileWaves);
    return;
  }
  const int P = group.view.P;
  __shared__ double s_part[kTileWaves][64][4];
  __shared__ double s_logit[16][16];
  {
    const int unit = lane & 15;
    const int64_t tok = (tok0 + unit < T) ? tok0 + unit : T - 1;  // valid rows either way; surplus results are dropped
    const int j = (unit >> 2) < n ? unit >> 2 : 0;
    const float* Wr = j == 0 ? group.r[0].Wr : j == 1 ? group.r[1].Wr : j == 2 ? group.r[2].Wr : group.r[3].Wr;
    const f64x4 acc = tile_product<kTileWaves>(X + tok * K, Wr + (int64_t)min(unit & 3, P - 1) * K, K, wave, lane);
#pragma unroll
    for (int r = 0; r < 4; ++r) s_part[wave][lane][r] = acc[r];
  }
  __syncthreads();
  if (tid < 256) {
    const int l = tid >> 2, r = tid & 3;  // one result of the 16 x 16 tile per thread
    double v = 0.0;
#pragma unroll
    for (int w = 0; w < kTileWaves; ++w) v += s_part[w][l][r];
    s_logit[4 * r + (l >> 4)][l & 15] = v;
  }
  __syncthreads();
  if (tid < 64) {
    const int64_t tok = tok0 + (tid & 15);
    const int j = tid >> 4;
    if (j < n && tok < T) {
      const RouteOut& out = group.r[j];
      double best = 0.0;
      int arg = 0;
#pragma unroll
      for (int q = 0; q < kP; ++q) {
        if (q < P) {
          const double s = s_logit[tid & 15][4 * j + q] + (double)out.br[q];
          if (out.logits) out.logits[tok * P + q] = s;
          if (q == 0 || s > best) {  // strict: the first maximum wins ties
            best = s;
            arg = q;
          }
        }
      }
      out.prec[tok] = group.view.value[arg];
    }
  }
}

// General router, fewer tokens: a workgroup of 256 threads scores TPW consecutive tokens for router blockIdx.y.  The K axis
// is split over the threads in chunks of 8 columns; each thread keeps 4 x TPW fp64 partial sums (bf16 x fp32 products are
// exact in fp64), reduced over the wavefront (wave_sum4) and over the four wavefronts through LDS.
template <int TPW>
__global__ __launch_bounds__(256) void route_rows_kernel(const uint16_t* __restrict__ X, int64_t T, int64_t K,
                                                         const RouteGroup group, int n, const PrefillPrep pf) {
  const int64_t tok0 = (int64_t)blockIdx.x * TPW;
  if ((int)blockIdx.y == n) {  // (only with pf)
    prefill_prep_share(pf, T, K, tok0, TPW, 256);
    return;
  }
  const RouteOut& out = group.r[blockIdx.y];
  const int P = group.view.P;
  const int tid = threadIdx.x;
  double acc[TPW][kP];
#pragma unroll
  for (int t = 0; t < TPW; ++t)
#pragma unroll
    for (int q = 0; q < kP; ++q) acc[t][q] = 0.0;

  for (int64_t k = (int64_t)tid * 8; k < K; k += 256 * 8) {
    float w[kP][8];
#pragma unroll
    for (int q = 0; q < kP; ++q) {
      const float4* src = reinterpret_cast<const float4*>(out.Wr + (int64_t)min(q, P - 1) * K + k);  // rows past P: unused
      float4 a = src[0], b = src[1];
      w[q][0] = a.x; w[q][1] = a.y; w[q][2] = a.z; w[q][3] = a.w;
      w[q][4] = b.x; w[q][5] = b.y; w[q][6] = b.z; w[q][7] = b.w;
    }
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
      if (tok0 + t < T) {
        const uint4 xv = *reinterpret_cast<const uint4*>(X + (tok0 + t) * K + k);
        const float x[8] = {bf16_lo(xv.x), bf16_hi(xv.x), bf16_lo(xv.y), bf16_hi(xv.y),
                            bf16_lo(xv.z), bf16_hi(xv.z), bf16_lo(xv.w), bf16_hi(xv.w)};
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
          for (int q = 0; q < kP; ++q) acc[t][q] = fma((double)x[j], (double)w[q][j], acc[t][q]);
      }
    }
  }
  __shared__ double red[4][TPW][kP];
  const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const double v = wave_sum4(acc[t], lane);
    if (lane < kP) red[wave][t][wave_sum4_index(lane)] = v;
  }
  __syncthreads();
  if (tid < TPW && tok0 + tid < T) {
    double best = 0.0;
    int arg = 0;
#pragma unroll
    for (int q = 0; q < kP; ++q) {
      if (q < P) {
        const double s = ((red[0][tid][q] + red[1][tid][q]) + (red[2][tid][q] + red[3][tid][q])) + (double)out.br[q];
        if (out.logits) out.logits[(tok0 + tid) * P + q] = s;
        if (q == 0 || s > best) {  // strict: the first maximum wins ties
          best = s;
          arg = q;
        }
      }
    }
    out.prec[tok0 + tid] = group.view.value[arg];
  }
}

// The stable counting sort behind a launch that wrote precisions: one workgroup per router.
struct SortGroup {
  const int32_t* prec[kRouteGroupMax];
  int32_t* perm[kRouteGroupMax];
  int32_t* offsets[kRouteGroupMax];
};
__global__ __launch_bounds__(1024) void sort_kernel(const SortGroup g, int64_t T, int shift) {
  const int j = blockIdx.x;
  bucket_by_workgroup<16>(g.prec[j], T, g.perm[j], g.offsets[j], shift);
}

// Small batches (T <= 128; the packed meeting word below up to kSmallRouteTokens), one or several routers over the same activations
// (the projections of a decoder block that share their input, Sec. 4.3, fused router launch).
// blockIdx.x = token, blockIdx.y = router.  512 threads split the K axis in chunks of 8 columns,
// two chunks in flight per thread.  Workgroups meet through ONE 64-bit atomic add per token: the
// word carries 2 bits per token and an arrival count in its top byte, so the workgroup that
// arrives last holds every token's precision in the returned value and buckets them with
// wavefront ballots, without fences or a second pass over memory.  The word is cleared ahead of the launch.
constexpr int kSmallRouteTokens = 28;
//
// The launch can carry the activation preparation of the FP4-operand decode kernel along: plane
// blockIdx.y == n_routers of the grid prepares 256-column block blockIdx.x with its first
// wavefront (prep == nullptr: no such plane).  defer_bucket: only the precisions are written; the linear
// kernel that follows sorts the tokens (it reads every precision anyway), which takes the atomic
// round trip and the sort out of this launch.
//
// kAct (K <= 16384): the activation-quantised stage in the same launch.  A workgroup holds its token's whole row, so it
// quantises the row itself (each router's workgroup again, router 0 writes the results out) and scores the rebuilt
// values from registers; the preparation plane then works a token at a time too, from integers in LDS.  Quantiser and
// router as two launches took 5.1 + 4.9 us a stage, most of it launching; together 5.6 us at K = 4096, 9 at K = 11008.
// Together with the row scaling in the linear launch: 7B-shaped block, 16 tokens, 4-bit activations 108.5 -> 103 us; 2048
// x 5120 block at 8 tokens 67 -> 55 us, 4096 x 11008 with kv / 4 at 64 tokens 196 -> 188 us.
template <bool kAct>
__global__ __launch_bounds__(512) void route_small_kernel(const uint16_t* __restrict__ X, int T, int64_t K,
                                                          RouteGroup group, int n_routers,
                                                          unsigned long long* words, char* prep, int prep_blocks,
                                                          const ZeroList zl, int defer_bucket,
                                                          const uint16_t* __restrict__ Xprep, const ActArgs aq,
                                                          float* __restrict__ sums) {
  // Xprep: the activations the linear kernel multiplies (X itself, except in the activation-quantised variant,
  // where the routers read the rebuilt activations and the linear kernel the integers)
  // sums: where router 0 also leaves the group sums that the kernel of wide matrices and long rows at 33 to 64 tokens starts
  // from (null: nowhere)
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int tok = blockIdx.x;
  const bool plane = (int)blockIdx.y == n_routers;
  if (!kAct && plane) {
    if (wave == 0) {
      if ((int)blockIdx.x < prep_blocks) f4::prep_block(Xprep, T, K, prep, (int)blockIdx.x, lane);
    } else {
      zero_share(zl, (int)blockIdx.x, (int)gridDim.x, tid - 64, 448);  // outputs a split-K linear kernel adds into
    }
    return;
  }
  if (kAct && plane) {
    zero_share(zl, (int)blockIdx.x, (int)gridDim.x, tid, 512);
    if (prep == nullptr || tok >= 16) return;
  } else if (tok >= T) {
    return;
  }
  const RouteOut& out = group.r[plane ? 0 : blockIdx.y];
  const float* __restrict__ Wr = out.Wr;
  double acc[kP] = {0.0, 0.0, 0.0, 0.0};
  auto load_w = [&](int64_t k, float4 (&w)[kP][2]) {
#pragma unroll
    for (int q = 0; q < kP; ++q) {
      const int64_t row = min(q, group.view.P - 1);  // rows past P do not exist: re-read the last one, never used
      const float4* s = reinterpret_cast<const float4*>(Wr + row * K + k);
      w[q][0] = s[0]; w[q][1] = s[1];
    }
  };
  auto add = [&](const uint4& xv, const float4 (&w)[kP][2]) {
    const float xs[8] = {bf16_lo(xv.x), bf16_hi(xv.x), bf16_lo(xv.y), bf16_hi(xv.y),
                         bf16_lo(xv.z), bf16_hi(xv.z), bf16_lo(xv.w), bf16_hi(xv.w)};
#pragma unroll
    for (int q = 0; q < kP; ++q) {
      const float ws[8] = {w[q][0].x, w[q][0].y, w[q][0].z, w[q][0].w, w[q][1].x, w[q][1].y, w[q][1].z, w[q][1].w};
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[q] = fma((double)xs[j], (double)ws[j], acc[q]);
    }
  };
  if constexpr (kAct) {
    constexpr int kChunks = act::kHeldChunks, kThreads = act::kHeldThreads;
    static_assert(kThreads == 512, "the thread count of this launch");
    __shared__ uint4 s_row[act::kHeldColumns / 8];  // integers of the row (preparation plane)
    const int n8 = (int)(K >> 3);
    const uint4* x8 = reinterpret_cast<const uint4*>(aq.X + (int64_t)min(tok, T - 1) * K);
    float held[kChunks][8], lo = 0.f, hi = 0.f;
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      const int j = tid + c * kThreads;
      if (j < n8) {
        act::transformed8(x8, j, aq.shift, aq.scale, held[c]);
#pragma unroll
        for (int h = 0; h < 8; ++h) {
          lo = fminf(lo, held[c][h]);
          hi = fmaxf(hi, held[c][h]);
        }
      }
    }
    float4 w[kP][2];
    if (!plane && tid < n8) load_w((int64_t)tid * 8, w);  // on their way while the workgroup meets
    const act::Code code = act::row_code<kThreads>(lo, hi, aq.abits, tid);
    if (plane) {
#pragma unroll
      for (int c = 0; c < kChunks; ++c) {
        const int j = tid + c * kThreads;
        if (j < n8) {
          float xi[8];
          act::whole8(held[c], code, xi);
          s_row[j] = (tok < T) ? act::pack8(xi) : uint4{0u, 0u, 0u, 0u};  // rows without a token are zeros
        }
      }
      __syncthreads();
      const int kb = tid >> 2, qa = tid & 3;
      if (kb < prep_blocks) {
        uint4 raw[2][2][2];
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
          for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int step = 0; step < 2; ++step) {
              const int col = kb * kTileK + f4::prep_column(qa, g, c, step);
              raw[g][c][step] = (col < K) ? s_row[col >> 3] : uint4{0u, 0u, 0u, 0u};
            }
        f4::prep_values<1, 2>(raw, tok, qa, prep + (size_t)kb * f4::kPrepBytesPerBlock);
      }
      return;
    }
    const bool writes = blockIdx.y == 0;
    if (writes && tid == 0) aq.row_scale[tok] = code.scale;
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      const int j = tid + c * kThreads;
      if (j < n8) {
        if (c > 0) load_w((int64_t)j * 8, w);
        float xi[8];
        act::whole8(held[c], code, xi);
        const uint4 xr = act::rebuilt8(xi, code, j, aq.shift, aq.scale);
        if (writes) {
          reinterpret_cast<uint4*>(aq.Xint + (int64_t)tok * K)[j] = act::pack8(xi);
          reinterpret_cast<uint4*>(aq.Xr + (int64_t)tok * K)[j] = xr;
          if (sums != nullptr)
            mid_group_sums(((xi[0] + xi[1]) + (xi[2] + xi[3])) + ((xi[4] + xi[5]) + (xi[6] + xi[7])), j, tok, T, sums);
        }
        add(xr, w);
      }
    }
  } else {
    const uint16_t* x = X + (int64_t)tok * K;
    for (int64_t k = (int64_t)tid * 8; k < K; k += 2 * 4096) {
      const bool two = k + 4096 < K;
      const int64_t k2 = two ? k + 4096 : k;  // a valid address either way
      const uint4 xa = *reinterpret_cast<const uint4*>(x + k);
      const uint4 xb = *reinterpret_cast<const uint4*>(x + k2);
      float4 wa[kP][2], wb[kP][2];
      load_w(k, wa);
      load_w(k2, wb);
      add(xa, wa);
      if (two) add(xb, wb);
      if (sums != nullptr && blockIdx.y == 0) {
        mid_group_sums(sum8(xa), (int)(k >> 3), tok, T, sums);
        if (two) mid_group_sums(sum8(xb), (int)(k2 >> 3), tok, T, sums);
      }
    }
  }
  __shared__ double red[8][kP];
  {
    const double v = wave_sum4(acc, lane);
    if (lane < kP) red[wave][wave_sum4_index(lane)] = v;
  }
  __syncthreads();
  if (wave != 0) return;
  // lanes 0..3 finish one logit each; every lane then sees all four
  const int P = group.view.P;
  double mine = 0.0;
  if (lane < P) {
    mine = ((red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane])) +
           ((red[4][lane] + red[5][lane]) + (red[6][lane] + red[7][lane])) + (double)out.br[lane];
    if (out.logits) out.logits[(int64_t)tok * P + lane] = mine;
  }
  double best = __shfl(mine, 0, 64);
  int arg = 0;
#pragma unroll
  for (int q = 1; q < kP; ++q) {
    const double s = __shfl(mine, q, 64);
    if (q < P && s > best) {  // strict: the first maximum wins ties
      best = s;
      arg = q;
    }
  }
  // the router's output q stands for the first bits[q] bits of the code: `value` is what the precision array holds,
  // `arg` from here on the digit count minus one that tokens are sorted by
  const RouteView& vw = group.view;
  const int value = arg == 0 ? vw.value[0] : arg == 1 ? vw.value[1] : arg == 2 ? vw.value[2] : vw.value[3];
  arg = arg == 0 ? vw.digits[0] : arg == 1 ? vw.digits[1] : arg == 2 ? vw.digits[2] : vw.digits[3];
  if (defer_bucket) {  // the consumer of the precisions sorts the tokens itself: no meeting, the workgroup is done
    if (lane == 0) out.prec[tok] = value;
    return;
  }
  if (T > kSmallRouteTokens) {
    // Too many tokens for the packed word: the word only counts arrivals; precisions travel through memory
    // (store, fence, count; the last to arrive fences and reads them back) and one wavefront sorts them.
    unsigned long long arrived = 0ull;
    if (lane == 0) {
      out.prec[tok] = value;
      __threadfence();
      arrived = atomicAdd(words + blockIdx.y, 1ull) + 1ull;
    }
    arrived = __shfl(arrived, 0, 64);
    if ((int)arrived != T) return;
    __threadfence();
    // stable counting sort of up to 128 tokens by one wavefront: lane holds tokens lane and lane + 64
    const int p = (lane < T) ? (__hip_atomic_load(out.prec + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> vw.shift) : -1;
    const int p2 = (lane + 64 < T) ? (__hip_atomic_load(out.prec + lane + 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> vw.shift) : -1;
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    int start = 0, my_pos = 0, my_pos2 = 0;
#pragma unroll
    for (int q = 0; q < kP; ++q) {
      const uint64_t b = __ballot(p == q), b2 = __ballot(p2 == q);
      if (p == q) my_pos = start + __popcll(b & below);
      if (p2 == q) my_pos2 = start + __popcll(b) + __popcll(b2 & below);
      if (lane == q) out.offsets[q] = start;
      start += __popcll(b) + __popcll(b2);
    }
    if (lane == kP) out.offsets[kP] = start;
    if (p >= 0) out.perm[my_pos] = lane;
    if (p2 >= 0) out.perm[my_pos2] = lane + 64;
    if (lane == 0) words[blockIdx.y] = 0ull;
    return;
  }
  unsigned long long all = 0ull;
  if (lane == 0) {
    out.prec[tok] = value;
    const unsigned long long inc = ((unsigned long long)arg << (2 * tok)) + (1ull << 56);
    all = atomicAdd(words + blockIdx.y, inc) + inc;
  }
  all = __shfl(all, 0, 64);
  if ((int)(all >> 56) != T) return;
  // last workgroup of this router: stable counting sort of the T tokens by precision
  const int p = (lane < T) ? (int)((all >> (2 * lane)) & 3ull) : -1;
  const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  int start = 0, my_pos = 0;
#pragma unroll
  for (int q = 0; q < kP; ++q) {
    const uint64_t b = __ballot(p == q);
    if (p == q) my_pos = start + __popcll(b & below);
    if (lane == q) out.offsets[q] = start;
    start += __popcll(b);
  }
  if (lane == kP) out.offsets[kP] = start;
  if (p >= 0) out.perm[my_pos] = lane;
  if (lane == 0) words[blockIdx.y] = 0ull;  // ready for the next call
}

// The arrival counters of a workspace (its first 256 bytes), cleared ahead of a launch that meets through them:
// a caller's workspace may hold anything, for instance what a call that was cut short left behind.
__global__ __launch_bounds__(64) void clear_counters_kernel(unsigned int* __restrict__ counters) {
  counters[threadIdx.x] = 0u;
}
static mbq_status clear_counters(void* ws, hipStream_t stream) {
  hipLaunchKernelGGL(clear_counters_kernel, dim3(1), dim3(64), 0, stream, reinterpret_cast<unsigned int*>(ws));
  return hip_status(hipGetLastError(), "clear_counters_kernel launch");
}

static mbq_status launch_sort(int n, const int32_t* const* prec, int32_t* const* perm, int32_t* const* offsets, int64_t T,
                              int shift, hipStream_t stream) {
  SortGroup g;
  for (int i = 0; i < kRouteGroupMax; ++i) {
    g.prec[i] = prec[i < n ? i : 0];
    g.perm[i] = perm[i < n ? i : 0];
    g.offsets[i] = offsets[i < n ? i : 0];
  }
  hipLaunchKernelGGL(sort_kernel, dim3((unsigned)n), dim3(1024), 0, stream, g, T, shift);
  return hip_status(hipGetLastError(), "sort_kernel launch");
}

// Workspace: the per-router words of the small-batch kernel from byte 64.
bool route_can_carry_prep(int64_t T) { return T >= 1 && T <= kSmallRouteTokens && knob(4) != 1; }
// one launch for all routers of a call: up to two tokens per lane of the sorting wavefront
static bool route_small_supports(int64_t T) { return T >= 1 && T <= 128 && knob(4) != 1; }
// the one-launch kernel can leave the token sort to the consumer of the precisions (defer_bucket below), which
// sorts up to 128 tokens
bool route_defers_sort(int64_t T) { return route_small_supports(T); }

// prep != nullptr (only when route_can_carry_prep(T)): the launch also prepares the activations
// of the FP4-operand decode kernel, prep_blocks 256-column blocks, into prep.
mbq_status launch_route_group(const uint16_t* X, int64_t T, int64_t K, int n, const float* const* Wr,
                              const float* const* br, int32_t* const* prec, int32_t* const* perm,
                              int32_t* const* offsets, double* const* logits, void* ws, hipStream_t stream,
                              void* prep, int prep_blocks, const ZeroList* zl, bool defer_bucket,
                              const RouteView& view, const uint16_t* Xprep, const ActArgs* aq, void* sums,
                              const PrefillPrep* pf) {
  if (T == 0) return launch_sort(n, prec, perm, offsets, 0, 0, stream);  // the (all-zero) offsets
  RouteGroup g;
  g.view = view;
  for (int i = 0; i < kRouteGroupMax; ++i) {
    const int j = i < n ? i : 0;
    g.r[i] = RouteOut{Wr[j], br[j], prec[j], perm[j], offsets[j], logits ? logits[j] : nullptr};
  }
  if (route_small_supports(T)) {
    if (!defer_bucket) {  // a launch that sorts meets through the counters
      mbq_status st = clear_counters(ws, stream);
      if (st != MBQ_OK) return st;
    }
    if (!route_can_carry_prep(T)) prep = nullptr;
    unsigned long long* words = reinterpret_cast<unsigned long long*>(reinterpret_cast<char*>(ws) + 64);
    bool clears = false;  // outputs to clear also without a preparation: the extra plane then only clears
    if (zl)
      for (int i = 0; i < kRouteGroupMax; ++i) clears = clears || zl->p[i] != nullptr;
    const bool plane = prep != nullptr || clears;
    if (aq) {  // (the plane prepares a token per workgroup, all 16 rows of the tile)
      const unsigned gx = (prep && T < 16) ? 16u : (unsigned)T;
      hipLaunchKernelGGL(route_small_kernel<true>, dim3(gx, (unsigned)n + (plane ? 1u : 0u)), dim3(512), 0, stream, X,
                         (int)T, K, g, n, words, reinterpret_cast<char*>(prep), prep ? prep_blocks : 0,
                         (plane && zl) ? *zl : ZeroList{}, defer_bucket ? 1 : 0, Xprep, *aq,
                         reinterpret_cast<float*>(sums));
    } else {
      const unsigned gx = (prep && prep_blocks > (int)T) ? (unsigned)prep_blocks : (unsigned)T;
      hipLaunchKernelGGL(route_small_kernel<false>, dim3(gx, (unsigned)n + (plane ? 1u : 0u)), dim3(512), 0, stream, X,
                         (int)T, K, g, n, words, reinterpret_cast<char*>(prep), prep ? prep_blocks : 0,
                         (plane && zl) ? *zl : ZeroList{}, defer_bucket ? 1 : 0, Xprep ? Xprep : X, ActArgs{},
                         reinterpret_cast<float*>(sums));
    }
    return hip_status(hipGetLastError(), "route_small_kernel launch");
  }
  const unsigned planes = pf ? 1u : 0u;  // one more plane of workgroups for the work of the prefill's pre-kernel
  const PrefillPrep prefill = pf ? *pf : PrefillPrep{};
  if (T <= 256)
    hipLaunchKernelGGL(route_rows_kernel<1>, dim3((unsigned)T, (unsigned)n + planes), dim3(256), 0, stream, X, T, K, g, n,
                       prefill);
  else if (T <= 1024)
    hipLaunchKernelGGL(route_rows_kernel<4>, dim3((unsigned)((T + 3) / 4), (unsigned)n + planes), dim3(256), 0, stream, X, T,
                       K, g, n, prefill);
  else
    hipLaunchKernelGGL(route_kernel, dim3((unsigned)((T + 15) / 16), 1u + planes), dim3(64 * kTileWaves), 0, stream, X, T, K,
                       g, n, prefill);
  mbq_status st = hip_status(hipGetLastError(), "route_kernel launch");
  if (st != MBQ_OK) return st;
  return launch_sort(n, prec, perm, offsets, T, view.shift, stream);
}

mbq_status launch_route(const uint16_t* X, int64_t T, int64_t K, const float* Wr, const float* br,
                        int32_t* prec, int32_t* perm, int32_t* offsets, double* logits, void* ws,
                        hipStream_t stream, const RouteView& view) {
  double* const lg[1] = {logits};
  return launch_route_group(X, T, K, 1, &Wr, &br, &prec, &perm, &offsets, logits ? lg : nullptr, ws, stream,
                            nullptr, 0, nullptr, false, view);
}

// ---------------------------------------------------------------------------------------------
// The paper's own router (Sec. 4.2 Eq. 4): a 2-layer MLP scores every slice, S = relu(X W1^T + b1)
// W2^T + b2 (the activation is not given in the paper; ReLU is the reading taken), and the
// run-time threshold of Sec. 4.2 turns scores into slice gates, G = 1[(S - delta) > 0].  The base
// slice is always active (shared-expert slice); a token's precision is the number of leading
// active residual slices, so that it names a prefix of slices like every other path here.
//
// Three launches.  Hidden layer: a workgroup of 256 threads produces eight hidden units of TPW consecutive
// tokens (grid = token groups x hidden chunks, so small batches still fill the chip): the K axis is
// split over the threads in chunks of 8 columns (bf16 x fp32 products are exact in fp64, accumulation
// in fp64), partial sums meet through wavefront shuffles and LDS, bias and ReLU are applied and the
// hidden vector goes to the workspace.  Scores: one thread per (token, slice) forms the score in a
// fixed order, one thread per token decides; sort_kernel buckets the tokens.
constexpr int kMlpHiddenChunk = 8;
constexpr int kMlpMaxHidden = 512;

template <int TPW>
__global__ __launch_bounds__(256) void route_mlp_hidden_kernel(const uint16_t* __restrict__ X, int64_t T, int64_t K,
                                                               const float* __restrict__ W1,
                                                               const float* __restrict__ b1, int H,
                                                               double* __restrict__ hidden) {
  constexpr int HC = kMlpHiddenChunk;
  const int64_t tok0 = (int64_t)blockIdx.x * TPW;
  const int h0 = (int)blockIdx.y * HC;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  __shared__ double s_red[4][TPW][HC];
  double acc[TPW][HC];
#pragma unroll
  for (int t = 0; t < TPW; ++t)
#pragma unroll
    for (int j = 0; j < HC; ++j) acc[t][j] = 0.0;
  for (int64_t k = (int64_t)tid * 8; k < K; k += 256 * 8) {
    double w[HC][8];
#pragma unroll
    for (int j = 0; j < HC; ++j) {
      const int h = (h0 + j < H) ? h0 + j : H - 1;  // a valid row either way; surplus units are dropped below
      const float4* src = reinterpret_cast<const float4*>(W1 + (int64_t)h * K + k);
      const float4 a = src[0], b = src[1];
      w[j][0] = a.x; w[j][1] = a.y; w[j][2] = a.z; w[j][3] = a.w;
      w[j][4] = b.x; w[j][5] = b.y; w[j][6] = b.z; w[j][7] = b.w;
    }
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
      const int64_t tok = (tok0 + t < T) ? tok0 + t : T - 1;  // a valid row either way
      const uint4 xv = *reinterpret_cast<const uint4*>(X + tok * K + k);
      const double x[8] = {bf16_lo(xv.x), bf16_hi(xv.x), bf16_lo(xv.y), bf16_hi(xv.y),
                           bf16_lo(xv.z), bf16_hi(xv.z), bf16_lo(xv.w), bf16_hi(xv.w)};
#pragma unroll
      for (int j = 0; j < HC; ++j)
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[t][j] = fma(x[c], w[j][c], acc[t][j]);
    }
  }
#pragma unroll
  for (int t = 0; t < TPW; ++t)
#pragma unroll
    for (int j = 0; j < HC; ++j) {
      double v = acc[t][j];
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) v += __shfl_down(v, off, 64);
      if (lane == 0) s_red[wave][t][j] = v;
    }
  __syncthreads();
  if (tid < TPW * HC) {
    const int t = tid / HC, j = tid % HC;
    if (h0 + j < H && tok0 + t < T) {
      const double pre = ((s_red[0][t][j] + s_red[1][t][j]) + (s_red[2][t][j] + s_red[3][t][j])) + (double)b1[h0 + j];
      hidden[(tok0 + t) * H + h0 + j] = pre > 0.0 ? pre : 0.0;
    }
  }
}

// Hidden layer of larger batches on the fp64 matrix cores (tile_product): a workgroup owns a tile of 16 tokens x 16 hidden
// units.
__global__ __launch_bounds__(64 * kTileWaves) void route_mlp_hidden_mfma_kernel(const uint16_t* __restrict__ X, int64_t T,
                                                                               int64_t K, const float* __restrict__ W1,
                                                                               const float* __restrict__ b1, int H,
                                                                               double* __restrict__ hidden) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t tok0 = (int64_t)blockIdx.x * 16;
  const int h0 = (int)blockIdx.y * 16;
  const int64_t tok = (tok0 + (lane & 15) < T) ? tok0 + (lane & 15) : T - 1;  // valid rows either way;
  const int h = (h0 + (lane & 15) < H) ? h0 + (lane & 15) : H - 1;            // surplus results are dropped
  const f64x4 acc = tile_product<kTileWaves>(X + tok * K, W1 + (int64_t)h * K, K, wave, lane);
  __shared__ double s_part[kTileWaves][64][4];
#pragma unroll
  for (int r = 0; r < 4; ++r) s_part[wave][lane][r] = acc[r];
  __syncthreads();
  if (tid < 256) {
    const int l = tid >> 2, r = tid & 3;  // one result of the 16 x 16 tile per thread
    const int64_t t = tok0 + 4 * r + (l >> 4);
    const int hu = h0 + (l & 15);
    if (t < T && hu < H) {
      double pre = 0.0;
#pragma unroll
      for (int w = 0; w < kTileWaves; ++w) pre += s_part[w][l][r];
      pre += (double)b1[hu];
      hidden[t * H + hu] = pre > 0.0 ? pre : 0.0;
    }
  }
}

// 64 tokens per workgroup: thread (token, slice) forms the score, then one thread per token decides.
__global__ __launch_bounds__(256) void route_mlp_score_kernel(const double* __restrict__ hidden, int64_t T, int H,
                                                              const float* __restrict__ W2,
                                                              const float* __restrict__ b2, double delta,
                                                              int32_t* __restrict__ prec,
                                                              double* __restrict__ scores) {
  const int tid = threadIdx.x;
  const int64_t tok = (int64_t)blockIdx.x * 64 + (tid >> 2);
  const int e = tid & 3;
  __shared__ double s_score[64][kP];
  if (tok < T) {
    const double* hrow = hidden + tok * H;
    const float* wrow = W2 + (int64_t)e * H;
    double s = 0.0;
    // (sixteen units' loads at a time: one after the other they took 12 us at H = 64)
    int j = 0;
#pragma unroll 1
    for (; j + 16 <= H; j += 16) {
      double hv[16];
      float wv[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        hv[i] = hrow[j + i];
        wv[i] = wrow[j + i];
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) s = fma(hv[i], (double)wv[i], s);
    }
    for (; j < H; ++j) s = fma(hrow[j], (double)wrow[j], s);
    s += (double)b2[e];
    s_score[tid >> 2][e] = s;
    if (scores) scores[tok * kP + e] = s;
  }
  __syncthreads();
  if (tid < 64 && (int64_t)blockIdx.x * 64 + tid < T) {
    int p = 0;
#pragma unroll
    for (int q = 1; q < kP; ++q) {
      if (p == q - 1 && (s_score[tid][q] - delta) > 0.0) p = q;  // strict: a score on the threshold is inactive
    }
    prec[(int64_t)blockIdx.x * 64 + tid] = p;
  }
}

// ws: 256 spare bytes, then the hidden layer, fp64 [T][H]
size_t route_mlp_workspace_bytes(int64_t T, int H) { return 256 + (size_t)T * (size_t)H * sizeof(double); }

mbq_status launch_route_mlp(const uint16_t* X, int64_t T, int64_t K, const float* W1, const float* b1, int H,
                            const float* W2, const float* b2, double delta, int32_t* prec, int32_t* perm,
                            int32_t* offsets, double* scores, void* ws, hipStream_t stream) {
  double* hidden = reinterpret_cast<double*>(reinterpret_cast<char*>(ws) + 256);
  if (T == 0) return launch_sort(1, &prec, &perm, &offsets, 0, 0, stream);  // the (all-zero) offsets
  const unsigned chunks = (unsigned)((H + kMlpHiddenChunk - 1) / kMlpHiddenChunk);
  if (T <= 256)
    hipLaunchKernelGGL(route_mlp_hidden_kernel<1>, dim3((unsigned)T, chunks), dim3(256), 0, stream, X, T, K, W1, b1,
                       H, hidden);
  else
    hipLaunchKernelGGL(route_mlp_hidden_mfma_kernel, dim3((unsigned)((T + 15) / 16), (unsigned)((H + 15) / 16)),
                       dim3(64 * kTileWaves), 0, stream, X, T, K, W1, b1, H, hidden);
  mbq_status st = hip_status(hipGetLastError(), "route_mlp_hidden_kernel launch");
  if (st != MBQ_OK) return st;
  hipLaunchKernelGGL(route_mlp_score_kernel, dim3((unsigned)((T + 63) / 64)), dim3(256), 0, stream, hidden, T, H, W2,
                     b2, delta, prec, scores);
  st = hip_status(hipGetLastError(), "route_mlp_score_kernel launch");
  if (st != MBQ_OK) return st;
  return launch_sort(1, &prec, &perm, &offsets, T, 0, stream);
}
int route_mlp_max_hidden() { return kMlpMaxHidden; }

// Layer-wise threshold calibration (App. C.2): the (k+1)-th largest of the T (E-1) residual-slice
// scores, found by a most-significant-bit-first radix selection on the order-preserving integer
// image of the doubles; one workgroup, 64 passes over the scores (an offline step).
__device__ inline unsigned long long ordered_key(double v) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}
__global__ __launch_bounds__(1024) void threshold_quantile_kernel(const double* __restrict__ scores, int64_t T,
                                                                   long long k, double* __restrict__ delta_out) {
  const int64_t M = T * (kP - 1);
  __shared__ unsigned long long s_cnt[16];
  __shared__ unsigned long long s_total;
  if (k >= M) {  // every residual score stays active
    if (threadIdx.x == 0) *delta_out = -__builtin_huge_val();
    return;
  }
  unsigned long long prefix = 0ull, mask = 0ull;
  long long want = k;  // rank (0 = largest) among the scores that match the prefix so far
  for (int bit = 63; bit >= 0; --bit) {
    const unsigned long long cand = prefix | (1ull << bit), cmask = mask | (1ull << bit);
    unsigned long long c = 0;
    for (int64_t i = threadIdx.x; i < M; i += 1024) {
      const double v = scores[(i / (kP - 1)) * kP + 1 + (i % (kP - 1))];
      c += ((ordered_key(v) & cmask) == cand) ? 1ull : 0ull;
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) c += __shfl_down(c, off, 64);
    if ((threadIdx.x & 63) == 0) s_cnt[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
      unsigned long long tot = 0;
      for (int w = 0; w < 16; ++w) tot += s_cnt[w];
      s_total = tot;
    }
    __syncthreads();
    const unsigned long long ones = s_total;  // scores that match the prefix and have this bit set (the larger ones)
    if ((unsigned long long)want < ones) {
      prefix = cand;
    } else {
      want -= (long long)ones;
    }
    mask = cmask;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const unsigned long long u = (prefix >> 63) ? (prefix & 0x7FFFFFFFFFFFFFFFull) : ~prefix;
    *delta_out = __longlong_as_double((long long)u);
  }
}

mbq_status launch_threshold_quantile(const double* scores, int64_t T, long long k, double* delta_out,
                                     hipStream_t stream) {
  hipLaunchKernelGGL(threshold_quantile_kernel, dim3(1), dim3(1024), 0, stream, scores, T, k, delta_out);
  return hip_status(hipGetLastError(), "threshold_quantile_kernel launch");
}

}  // namespace mbq
