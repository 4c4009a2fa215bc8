// Routed linear for 33 to 64 tokens on wide matrices and on long rows: one pass over the weights for all the tokens.
//
// Paper Sec. 4.2 Eq. 6 slice by slice, Y_i = sum_{e <= p_i} W_e^T X_i, in the bf16 operands of mbq_bf16_codes.h; tokens in
// the order of their precision (Sec. 4.3, token permutation), so slice e meets the rows from its first token on: row tiles
// below are left out, and in the one where it begins the rows below count as zeros.  Every block of packed weights is
// unpacked once, for 64 rows (the register-stationary kernel of mbq_linear_decode16.hip unpacks it once per 32).
//
// Work split: a workgroup of four wavefronts owns 64 output columns (a wavefront 16) and a part of the K axis; two
// workgroups share a compute unit.  Activations: blocks of 256 columns are copied to LDS a block ahead (32 KiB, rows in
// sorted order, one barrier a block) and read by all four wavefronts.  A wavefront that read its own from the L2 instead
// (each with a share of the K axis and partial tiles meeting in LDS) was bound by it: 16 columns take in 7.5 times the
// bytes of their weights that way, and 13 TB/s is what the L2s gave; 14336 x 4096 twice took 79 us.
// Weights: one block ahead in registers.  Offsets of the operands: the accumulators of a group start with minus what they
// will add up to (a constant of the row), so a group's result is small when it is scaled by s0 and added to the sum; the
// zero points follow as fp32 MFMAs, K = 4, every two blocks.
// Long rows are cut into up to eight parts of the K axis: part 0 stores into Y, the others into arrays of the workspace,
// which fold_kernel adds in order, so the result does not depend on which comes first.
// Wide matrices are the sum of two halves of K.  Where a call has no more workgroups than the chip has compute units (a matrix
// alone) a workgroup of eight wavefronts forms both at a time, which meet in LDS; otherwise one of four forms them in
// turn: the same bits.  (One wavefront a SIMD issues an instruction every 7 cycles, two of them every 4.6: 14336 x 4096 alone
// at 64 tokens 42 us in the register-stationary kernel, 48 with four wavefronts and no halves, 39 now; twice the matrix takes
// 1 to 3 % longer in turn than without halves.)
//
// Bound by instruction issue: a block takes 360 vector instructions (192 of them unpacking) and 92 MFMAs a wavefront at 64
// tokens of an even mix, 7500 cycles for the two wavefronts of a SIMD.  Stage calls (router included) with the
// register-stationary kernel and with this one, us: twice 14336 x 4096 at 64 tokens 73 -> 61, skewed mix 61 -> 51, at 48 tokens 72
// -> 56; 4096 x 14336 at 64 tokens 52 -> 39, 4096 x 11008 41 -> 36, at 33 tokens 41 -> 33.  Two tiles a wavefront (spills), operands of
// four steps at a time with the next slice's unpacking dealt out under the MFMAs (62.3 -> 64.3), eight wavefronts a
// workgroup (65.8) were no faster.
#include <type_traits>

#include "mbq_bf16_codes.h"

namespace mbq {

namespace mid {

using namespace bf;

constexpr int kWaves = 4;
constexpr int kMaxBlocks = 16;  // of a workgroup: their row constants wait in LDS
constexpr int kMaxParts = 8;
constexpr int kMinRows = 33, kMaxRows = 64;
static_assert(kMaxParts <= kMaxKSplit, "the workspace holds the arrays");
constexpr int kRowBytes = 2 * kGroup;  // one group of one row: 16 chunks of 16 bytes, swizzled by the row

struct Proj {
  const uint4* codes;
  size_t slice_vec;  // uint4 per slice
  const float2* meta;
  int64_t N;
  int NT;
  const int32_t* prec;
  const int32_t* perm;      // precision-sorted token order, or null: sorted here
  int32_t* sort_perm;       // with perm == null: where the order and the bucket offsets go
  int32_t* sort_offsets;
  float* Y;
  float* slot;              // T x N arrays of partial sums besides Y, slot_floats apart: part s > 0 stores into slot s - 1
  int64_t slot_floats;
  int parts;                // workgroups along K
  int half;                 // > 0: blocks of the first half of K, an even number; the halves' sums are added last
  int wg_begin;             // first workgroup of the matrix
};
struct Group {
  Proj p[MBQ_MAX_GROUP];
  int n;
};

struct Item {  // a 16 x 256 block: four slices and {s0, z0} of two groups
  uint4 w[4];
  float2 mt[2];
};

}  // namespace mid

// Wide matrices, whose K axis has two halves: SIDES = 2, eight wavefronts, four on each half, or IN_TURN, one half after the
// other.  Long rows: neither.  (An instance of its own each: 8192 x 28672 at 64 tokens of a skewed mix 93.5 us, 95.3 with IN_TURN a
// run-time branch.)
template <int RT, int SIDES, bool IN_TURN>
__global__ __launch_bounds__(64 * mid::kWaves * SIDES, 2) void mid_kernel(const uint16_t* __restrict__ X, int T, int64_t K, int KB,
                                                                          const float2* __restrict__ sums, const mid::Group g) {
  using namespace mid;
  constexpr int kRows = 16 * RT;
  constexpr int kHalf = kRows * kRowBytes;   // a group of the pass's rows
  constexpr int kStage = 2 * kHalf;          // a block
  constexpr int kBlocks = kMaxBlocks / SIDES;
  __shared__ __attribute__((aligned(1024))) char smem[SIDES * 2 * kStage + 2 * kMaxBlocks * kRows * 8];
  const int wave_of = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int side = SIDES == 1 ? 0 : wave_of / kWaves, wave = SIDES == 1 ? wave_of : wave_of % kWaves;
  float* const s_rows = reinterpret_cast<float*>(smem + SIDES * 2 * kStage);
  float* const s_c1 = s_rows + side * (4 * kBlocks * kRows);  // [group][row]: what the accumulators of a group start with
  float* const s_ss = s_c1 + 2 * kBlocks * kRows;             // [group][row]: sums of the group's activations
  Proj P = g.p[0];
#pragma unroll
  for (int j = 1; j < MBQ_MAX_GROUP; ++j)
    if (j < g.n && (int)blockIdx.x >= g.p[j].wg_begin) P = g.p[j];
  const int wg = (int)blockIdx.x - P.wg_begin;
  const int part = wg % P.parts, col_set = wg / P.parts;
  const int b0 = SIDES == 2 ? side * P.half : (int)((int64_t)part * KB / P.parts);
  const int nblk = SIDES == 2 ? (side ? KB - P.half : P.half) : (int)((int64_t)(part + 1) * KB / P.parts) - b0;
  const int lane = threadIdx.x & 63, l15 = lane & 15, kq = lane >> 4;
  const int G = (int)(K / kGroup);
  char* const stages = smem + side * (2 * kStage);
  const uint32_t lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)stages;

  // ---- rows: lane r holds row r of the precision-sorted tokens ----
  int token = -1, p = -1;
  if (P.perm != nullptr) {
    if (lane < T) {
      token = P.perm[lane];
      p = P.prec[token];
    }
  } else {
    // stable counting sort of the T <= 64 tokens by precision: a lane holds token `lane`
    const int mine = lane < T ? min(max(P.prec[lane], 0), MBQ_N_PRECISIONS - 1) : -1;
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    int start = 0, pos = 0, off = 0;
#pragma unroll
    for (int q = 0; q < MBQ_N_PRECISIONS; ++q) {
      const uint64_t with = __ballot(mine == q);
      if (mine == q) pos = start + __popcll(with & below);
      if (lane == q) off = start;
      start += __popcll(with);
    }
    if (lane == MBQ_N_PRECISIONS) off = start;
    int* const order = reinterpret_cast<int*>(s_rows) + 64 * wave_of;  // (the wavefront's own; in order within it)
    if (mine >= 0) order[pos] = lane | (mine << 8);
    const int e = lane < T ? order[lane] : -1;
    token = e < 0 ? -1 : (e & 0xFF);
    p = e < 0 ? -1 : (e >> 8);
    if (wg == 0 && wave_of == 0) {
      if (mine >= 0) P.sort_perm[pos] = lane;
      if (lane <= MBQ_N_PRECISIONS) P.sort_offsets[lane] = off;
    }
  }
  int pm = 0;              // highest precision
  int first_tile[4];       // row tile where slice e begins
  uint32_t mask[4];        // rows of that tile which it counts for
  first_tile[0] = 0;
  mask[0] = ~0u;
#pragma unroll
  for (int e = 1; e < 4; ++e) {
    const int first = __popcll(__ballot(p >= 0 && p < e));
    if (first < T) pm = e;
    first_tile[e] = first >> 4;
    mask[e] = l15 >= (first & 15) ? ~0u : 0u;
  }
  // ---- activations: an instruction moves 256 bytes of four rows (16 lanes a row); rows 16 j + 4 wave + kq.  LDS chunk l15
  // of a row holds its chunk l15 ^ (row & 15), so the 16 rows of a fragment read hit different banks.  Rows past the last:
  // token 0, never stored ----
  uint32_t x_at[RT];
#pragma unroll
  for (int j = 0; j < RT; ++j) {
    const int t = max(__shfl(token, 16 * j + 4 * wave + kq, 64), 0);
    x_at[j] = (uint32_t)t * 2u * (uint32_t)K + 16u * (uint32_t)(l15 ^ (4 * wave + kq));
  }
  auto load_x = [&](int kb, uint32_t stage) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      // (a second group that the last block may lack: the first one again, under zero scales)
      const char* src = reinterpret_cast<const char*>(X) + (size_t)min(2 * kb + h, G - 1) * kRowBytes;
#pragma unroll
      for (int j = 0; j < RT; ++j) dma_16(lds + stage + (uint32_t)(h * kHalf + (16 * j + 4 * wave) * kRowBytes), x_at[j], src);
    }
  };
  // ---- weights: this wavefront's tile (past the matrix: the last one again, not stored; a slice that no row needs: the
  // highest one needed again) ----
  const int nt = min(col_set * kWaves + wave, P.NT - 1);
  const uint32_t lane16 = 16u * (uint32_t)lane, meta_at = 8u * (uint32_t)l15;
  auto load_item = [&](int kb, Item& I) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      I.w[e] = *reinterpret_cast<const uint4*>(
          reinterpret_cast<const char*>(P.codes + (size_t)min(e, pm) * P.slice_vec + ((size_t)nt * KB + kb) * 64) + lane16);
#pragma unroll
    for (int h = 0; h < 2; ++h)
      I.mt[h] = *reinterpret_cast<const float2*>(
          reinterpret_cast<const char*>(P.meta + ((size_t)nt * (2 * KB) + 2 * kb + h) * kTileN) + meta_at);
  };
  Item A, B;
  load_x(b0, 0u);
  load_item(b0, A);

  // ---- row constants of the part's groups (wavefront w: groups w, w + 4, ..) ----
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");  // the order has been read from there
  {
    const float coefA = (p >= 3) ? 74.f : (p == 2) ? 72.f : (p == 1) ? 64.f : 32.f;  // biases of the operands of slices 0..p
    const float coefB = (p >= 3) ? 18.5f : (p == 2) ? 18.f : (p == 1) ? 16.f : 8.f;
    const float q = (p >= 3) ? 0.328125f : (p == 2) ? 0.3125f : (p == 1) ? 0.25f : 0.f;
    const float2* src = sums + max(token, 0);
    for (int gi = wave; gi < 2 * nblk; gi += kWaves) {
      const float2 s = 2 * b0 + gi < G ? src[(size_t)(2 * b0 + gi) * T] : float2{0.f, 0.f};
      const float ss = s.x + s.y;
      if (lane < kRows) {
        s_c1[gi * kRows + lane] = -(coefA * s.x + coefB * s.y + (1.5f * q - 0.5f) * ss);
        s_ss[gi * kRows + lane] = ss;
      }
    }
  }
  const UnpackConsts uc = make_unpack_consts();
  floatx4 y[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) y[rt] = floatx4{0.f, 0.f, 0.f, 0.f};
  float zero_at = 0.f;  // -s0 z0 of this lane's column: group kq of the four of two blocks

  uint32_t stage = 0u;
  int i = 0;
  auto settle = [&](Item& I) {  // the compiler's own wait for these loads is placed here
#pragma unroll
    for (int e = 0; e < 4; ++e) asm volatile("" : "+v"(I.w[e].x), "+v"(I.w[e].y), "+v"(I.w[e].z), "+v"(I.w[e].w));
#pragma unroll
    for (int h = 0; h < 2; ++h) asm volatile("" : "+v"(I.mt[h].x), "+v"(I.mt[h].y));
  };
  auto block = [&](Item& cur, Item& nxt) {
    const bool last = i + 1 == nblk;
    const int kb_next = b0 + (last ? i : i + 1);  // (the last block is requested once more: the other stage is free)
    load_x(kb_next, stage ^ (uint32_t)kStage);
    load_item(kb_next, nxt);
    __builtin_amdgcn_sched_barrier(0);
    uint4 xf[2][RT][2];
    // fragments of step s of half group d
    auto read_x = [&](int d, uint4 (&x)[RT][2]) {
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int chunk = 8 * (d & 1) + 4 * s + kq;
        const char* at = stages + stage + (d >> 1) * kHalf + l15 * kRowBytes + ((chunk ^ l15) * 16);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) x[rt][s] = *reinterpret_cast<const uint4*>(at + rt * 16 * kRowBytes);
      }
    };
    floatx4 D[RT];
    auto half_group = [&](auto d_tag) {  // 64 columns: the operands of two steps come from one dword of a slice
      constexpr int d = decltype(d_tag)::value;
      if constexpr ((d & 1) == 0) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
          D[rt] = *reinterpret_cast<const floatx4*>(s_c1 + (2 * i + (d >> 1)) * kRows + 16 * rt + 4 * kq);
      }
      if constexpr (d < 3) read_x(d + 1, xf[(d + 1) & 1]);
      const uint4(&x)[RT][2] = xf[d & 1];
      auto slice = [&](auto e_tag) {
        constexpr int E = decltype(e_tag)::value;
        uint4 Bo[2];
        unpack_dword<E>(d == 0 ? cur.w[E].x : d == 1 ? cur.w[E].y : d == 2 ? cur.w[E].z : cur.w[E].w, uc, Bo[0], Bo[1]);
        if constexpr (E == 0) {
#pragma unroll
          for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) D[rt] = mfma(x[rt][s], Bo[s], D[rt]);
        } else {
          // from the first row tile with rows of this precision; rows of it that are below count as zeros
#pragma unroll
          for (int r0 = 0; r0 < RT; ++r0) {
            // (three of the four are passed by: out of line, which the compiler does by itself but with IN_TURN's outer
            // loop; 14336 x 4096 twice at 64 tokens 60.9 -> 61.3 us with that, 62.2 in line, a skewed mix 48.9 -> 50.4, 51.0)
            if (IN_TURN ? __builtin_expect(first_tile[E] == r0, 0) : first_tile[E] == r0) {
              const uint32_t mk = mask[E];
#pragma unroll
              for (int s = 0; s < 2; ++s) {
                const uint4 xm = {x[r0][s].x & mk, x[r0][s].y & mk, x[r0][s].z & mk, x[r0][s].w & mk};
                D[r0] = mfma(xm, Bo[s], D[r0]);
#pragma unroll
                for (int rt = r0 + 1; rt < RT; ++rt) D[rt] = mfma(x[rt][s], Bo[s], D[rt]);
              }
            }
          }
        }
      };
      slice(std::integral_constant<int, 0>{});
      if (pm >= 1) slice(std::integral_constant<int, 1>{});
      if (pm >= 2) slice(std::integral_constant<int, 2>{});
      if (pm >= 3) slice(std::integral_constant<int, 3>{});
      if constexpr ((d & 1) == 1) {
        constexpr int h = d >> 1;
        const float s0 = cur.mt[h].x;
        if (kq == 2 * (i & 1) + h) zero_at = -s0 * cur.mt[h].y;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int r = 0; r < 4; ++r) y[rt][r] += s0 * D[rt][r];
      }
    };
    read_x(0, xf[0]);
    half_group(std::integral_constant<int, 0>{});
    half_group(std::integral_constant<int, 1>{});
    half_group(std::integral_constant<int, 2>{});
    half_group(std::integral_constant<int, 3>{});
    // the zero points of up to four groups: y[row][col] -= s0 z0 (sum of the group's activations), K = 4 in fp32
    if ((i & 1) == 1 || last) {
      const int of = (i & 1) && kq < 2 ? i - 1 : i;
      const float* ss = s_ss + (2 * of + (kq & 1)) * kRows + l15;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) y[rt] = __builtin_amdgcn_mfma_f32_16x16x4f32(ss[16 * rt], zero_at, y[rt], 0, 0, 0);
      zero_at = 0.f;
    }
    // this wavefront's requests have landed and its reads of the stage are done; behind the barrier everybody's are
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    settle(nxt);
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    stage ^= (uint32_t)kStage;
    ++i;
  };
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  settle(A);
  asm volatile("s_barrier" ::: "memory");
  // (the first half has an even number of blocks, so the second begins with the same registers and at the same place of a
  // pair of blocks as a side of its own would)
  floatx4 y_first[RT];
  for (int end = IN_TURN ? P.half : nblk;; end = nblk) {
#pragma unroll 1
    for (int q = i; q < end; q += 2) {
      block(A, B);
      if (q + 1 < end) block(B, A);
    }
    if (end == nblk) break;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      y_first[rt] = y[rt];
      y[rt] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
  }
  if constexpr (IN_TURN) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) y[rt] = y_first[rt] + y[rt];
  }
  if constexpr (SIDES == 2) {  // as many barriers on either side
    for (int r = nblk; r < max(P.half, KB - P.half); ++r) asm volatile("s_barrier" ::: "memory");
  }

  // ---- rows in original token order, through LDS (the stages are free): an instruction writes 256 bytes of four rows ----
  constexpr int kCols = 16 * kWaves, kLd = kCols + 4, kVec = kCols / 4;
  float* const s_out = reinterpret_cast<float*>(smem);
  static_assert(kRows * kLd * 4 <= 2 * kStage, "the tile fits the stages");
#pragma unroll
  for (int half = 0; half < SIDES; ++half) {
    if (side == half) {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float& at = s_out[(16 * rt + 4 * kq + r) * kLd + 16 * wave + l15];
          at = half == 0 ? y[rt][r] : at + y[rt][r];
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  }
  float* const out = part == 0 ? P.Y : P.slot + (part - 1) * P.slot_floats;
  const bool wide = (P.N & 3) == 0 && (reinterpret_cast<uintptr_t>(out) & 15) == 0;
#pragma unroll
  for (int u = 0; u < kRows * kVec; u += 64 * kWaves * SIDES) {
    const int row = (u + (int)threadIdx.x) / kVec, q = (u + (int)threadIdx.x) % kVec;
    const floatx4 v = *reinterpret_cast<const floatx4*>(s_out + row * kLd + 4 * q);
    const int64_t col = (int64_t)col_set * kCols + 4 * q;
    const int t = __shfl(token, row, 64);
    if (row < T && col < P.N) {
      float* at = out + (int64_t)t * P.N + col;
      if (wide) {
        *reinterpret_cast<floatx4*>(at) = v;
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (col + r < P.N) at[r] = v[r];
      }
    }
  }
}

// sums[group][token] = {even, odd}: sums of the activations of a group's even and odd blocks of 32 columns
__global__ __launch_bounds__(256) void mid_sums_kernel(const uint16_t* __restrict__ X, int T, int64_t K,
                                                       float* __restrict__ sums) {
  const int token = blockIdx.x;
  const uint4* src = reinterpret_cast<const uint4*>(X + (int64_t)token * K);
  const int chunks = (int)(K >> 3);  // a multiple of 16: groups of 16 lanes are whole
  for (int c = threadIdx.x; c < chunks; c += 256) mid_group_sums(sum8(src[c]), c, token, T, sums);
}

mbq_status launch_mid_sums(const uint16_t* X, int64_t T, int64_t K, void* sums, hipStream_t stream) {
  hipLaunchKernelGGL(mid_sums_kernel, dim3((unsigned)T), dim3(256), 0, stream, X, (int)T, K, reinterpret_cast<float*>(sums));
  return hip_status(hipGetLastError(), "mid_sums_kernel launch");
}

namespace mid {
static inline size_t sums_bytes(int64_t T, int64_t K) { return ((size_t)T * (size_t)(K / kGroup) * 8 + 255) / 256 * 256; }
static inline int64_t slot_floats(int64_t T, int64_t N) { return (T * N + 63) / 64 * 64; }
static inline int first_half(int KB) { return (KB + 1) / 4 * 2; }  // even, within one of the other half, at most half of kMaxBlocks
}  // namespace mid

// Parts of the K axis, 0: the matrix does not take this kernel.  The choice depends on T and the matrix alone, and a call for
// several matrices gives the bits of separate calls, so it is taken only where it won both ways; stage calls on cold weights
// in us (register-stationary kernel / this one), at 33, 48 and 64 tokens of an even mix (skewed mixes are within 5 % of the
// same ratio):
//   wide matrices, one part, alone (halves of K side by side) up to a workgroup a compute unit: 14336 x 4096 42 / 36, 42 / 36,
//   42 / 39; 12800 x 4096 42 / 36, 42 / 36, 42 / 38; beyond, in turn: 18432 x 4096 50 / 55, 50 / 55, 51 / 59 (not taken), 24576 x
//   4096 62 / 55, 63 / 55, 64 / 60, 32000 x 4096 78 / 58, 79 / 59, 80 / 64; twice (in turn): 14336 x 4096 71 / 57, 72 / 56, 73 / 61;
//   where the line lies, the same as ratios, alone and twice, at 33, 48, 49 and 64 tokens (the other kernel's time goes in
//   steps): 4096 columns, 13312 rows 1.16 1.17 1.05 1.09, twice 1.19 1.21 1.06 1.12, 12288 rows 0.98 1.06 0.95 0.99, twice 1.25 1.14
//   0.99 1.06 (not taken), 11264 rows 0.92 1.07 0.95 0.99 (not taken); 3584 columns, 11776 rows 1.03 1.10 0.98 1.03, twice 1.38 1.22
//   1.07 1.14, 11264 rows 0.98 1.10 0.98 1.03 (not taken); 3328 columns, 10752 rows 1.04 1.05 1.03 1.08, twice 1.46 1.48 1.05 1.11,
//   10240 rows 0.98 0.99 0.89 0.98 (not taken); 3072: 10752 rows 1.12 1.13 1.07 1.11; 2048: 10752 rows 1.13 1.16 1.06 1.11, twice 1.06
//   1.10 0.99 1.05, 10240 rows twice 1.02 1.05 0.95 1.00 (not taken); 1536: 10752 rows 1.19 1.24 1.13 1.19; 1024: 10752 rows 1.00 1.07
//   0.93 0.97, twice 1.08 1.16 0.95 0.99 (taken up to 48 tokens), 13312 rows 1.10 1.16 0.98 1.02, twice 1.18 1.26 1.03 1.06; 768: 10752
//   rows 1.02 1.06 0.95 0.98; 512: 10752 rows 1.14 1.22 1.06 1.12;
//   long rows, eight parts: 4096 x 11008 41 / 33, 41 / 33, 41 / 36; 3072 x 8320 34 / 29, 34 / 29, 34 / 30; 8192 x 28672 145 / 104,
//   145 / 103, 145 / 112; 2048 x 8192 23 / 24, 24 / 24, 24 / 25 (not taken);
//   with more rows than half the columns (q and o of an attention, where q has company) from K = 9984 on: 12288 x 12288 alone 90
//   / 74, 98 / 75, 98 / 81; with two of 1280 x 9984, of which each kernel takes its share in a launch of its own, 137 / 88, 139 /
//   89, 137 / 96; with two of 1152 x 9216 89 / 86, 90 / 87, 90 / 93 (not taken, though 9216 x 9216 alone 71 / 57, 71 / 57, 70 / 63
//   and three of them 186 / 159, 186 / 161, 236 / 178).
// What a matrix alone decides can be wrong for its company: 5120 x 13824 twice at 64 tokens 101 / 104 (61 / 55 alone), with
// 1024 x 11008 4096 x 11008 53 / 59 (42 / 36 alone).
// At 32 tokens both kernels unpack once and are as fast.
int mid_parts(int64_t T, const Shape& sh) {
  if (T < mid::kMinRows || T > mid::kMaxRows) return 0;
  const int least = (sh.KB + mid::kMaxBlocks - 1) / mid::kMaxBlocks;
  if (sh.N >= 2 * sh.K && least == 1) {
    const int alone_most = 256 * mid::kWaves, apart_least = 384 * mid::kWaves;  // code tiles
    const int from = sh.KB >= 15 ? 800 : sh.KB == 14 ? 736 : (sh.KB == 3 || sh.KB == 4) && T > 48 ? 832 : 672;
    return (sh.NT >= from && sh.NT <= alone_most) || sh.NT >= apart_least ? 1 : 0;
  }
  if (sh.KB <= (2 * sh.N <= sh.K ? 32 : 38) || sh.NT < 192 || sh.N > sh.K) return 0;
  // (the workspace of a call has room for kMaxKSplit arrays of at least T rows, decode_workspace_bytes: seven and the sums,
  // which take less than an array as 64 N > K)
  return mid::kMaxParts >= least ? mid::kMaxParts : 0;
}

mbq_status launch_linear_mid_group(const uint16_t* X, int64_t T, int n, const void* const* blobs, const Shape* shapes,
                                   const int32_t* const* prec, const int32_t* const* perm, float* const* Y,
                                   void* ws, hipStream_t stream, int32_t* const* sort_perm,
                                   int32_t* const* sort_offsets) {
  const Shape& sh = shapes[0];
  // matrices that are cut share the workspace's room one after the other
  bool cut = false;
  for (int i = 0; i < n; ++i) cut = cut || mid_parts(T, shapes[i]) > 1;
  if (cut && n > 1) {
    for (int i = 0; i < n; ++i) {
      const mbq_status st =
          launch_linear_mid_group(X, T, 1, blobs + i, shapes + i, prec + i, sort_perm ? nullptr : perm + i, Y + i, ws, stream,
                                  sort_perm ? sort_perm + i : nullptr, sort_perm ? sort_offsets + i : nullptr);
      if (st != MBQ_OK) return st;
    }
    return MBQ_OK;
  }
  mid::Group g;
  Fold fold;
  int grid = 0;
  float* slot = reinterpret_cast<float*>(reinterpret_cast<char*>(ws) + mid::sums_bytes(T, sh.K));
  for (int i = 0; i < MBQ_MAX_GROUP; ++i) {
    const int j = i < n ? i : 0;
    const Shape& s = shapes[j];
    mid::Proj& p = g.p[i];
    p.codes = reinterpret_cast<const uint4*>(blobs[j]);
    p.slice_vec = s.slice_words / 4;
    p.meta = reinterpret_cast<const float2*>(reinterpret_cast<const char*>(blobs[j]) + s.meta_offset);
    p.N = s.N;
    p.NT = s.NT;
    p.prec = prec[j];
    p.perm = sort_perm ? nullptr : perm[j];
    p.sort_perm = sort_perm ? sort_perm[j] : nullptr;
    p.sort_offsets = sort_perm ? sort_offsets[j] : nullptr;
    p.Y = Y[j];
    p.slot = slot;
    p.slot_floats = mid::slot_floats(T, s.N);
    p.parts = mid_parts(T, s);
    p.half = p.parts == 1 ? mid::first_half(s.KB) : 0;
    p.wg_begin = grid;
    fold.Y[i] = Y[j];
    fold.array[i] = slot;
    fold.array_floats[i] = p.slot_floats;
    fold.n[i] = T * s.N;
    fold.arrays[i] = i < n ? p.parts : 1;
    if (i < n) {
      grid += (s.NT + mid::kWaves - 1) / mid::kWaves * p.parts;
      slot += (p.parts - 1) * p.slot_floats;
    }
  }
  g.n = n;
  // halves of K side by side where that leaves no workgroup waiting for another (they need a compute unit each), in turn
  // where two workgroups share one: the same bits
  const bool sides = !cut && grid <= device_compute_units();
  const auto launch = [&](auto rt, auto n_sides, auto turn) {
    hipLaunchKernelGGL((mid_kernel<decltype(rt)::value, decltype(n_sides)::value, decltype(turn)::value>), dim3(grid),
                       dim3(64 * mid::kWaves * decltype(n_sides)::value), 0, stream, X, (int)T, sh.K, sh.KB,
                       reinterpret_cast<const float2*>(ws), g);
  };
  const std::integral_constant<int, 1> one{};
  const std::integral_constant<int, 2> two{};
  const std::integral_constant<int, 3> three{};
  const std::integral_constant<int, 4> four{};
  const std::true_type yes{};
  const std::false_type no{};
  if (T <= 48) sides ? launch(three, two, no) : cut ? launch(three, one, no) : launch(three, one, yes);
  else sides ? launch(four, two, no) : cut ? launch(four, one, no) : launch(four, one, yes);
  mbq_status st = hip_status(hipGetLastError(), "mid_kernel launch");
  return st == MBQ_OK ? launch_fold(fold, n, stream) : st;
}

}  // namespace mbq
