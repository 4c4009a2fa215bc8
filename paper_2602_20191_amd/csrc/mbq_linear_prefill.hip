// Prefill-side routed linear: a bf16 MFMA tiled GEMM per precision bucket.
//
// Paper Sec. 4.2 Eq. 6 in the merged-code form of App. B (truncating the merged
// integer code is the coarser quantiser): for a token of precision p,
//   Y[i][n] = sum_g (s0/64) * ( sum_{k in g} x_ik V_nk + (0.5 * 4^(3-p) - 64 z0) * Sx[i][g] )
// with V = I_p * 4^(3-p) the 8-bit code whose unused low digits are zero and Sx the group
// sums of x.  Tokens are taken in the order of their precision (Sec. 4.3, token permutation), so a
// tile of them has one precision and reads only slices 0..p.
//
// How the group scale reaches the matrix cores without a second accumulator set:
//   s0 = m * 2^t with m in [1/2, 2) chosen so that the bf16 exponent below is even.  The MFMA
//   B operand is the exact bf16 number (OFF + V) * 2^t (OFF = 256 for p <= 2, where V/2 sits in
//   the seven mantissa bits under a per-row exponent byte; OFF = 0 for p = 3), so a group's
//   products are already in units of 2^t and only the mantissa factor m is left.  The running
//   accumulator R is kept in units of the CURRENT group's m:  R <- R * (m_prev / m_cur) at a
//   group boundary (one multiply per element, ratio in (1/4, 4)), then the group's MFMAs
//   accumulate straight into R.  After the last group R * m_last / 64 is the sum in true units.
//   The zero-point / offset term  -sum_g s0 (OFF/64 - half/64 + z0) Sx[i][g]  is a rank-16 update
//   done every 16 groups with MFMAs, so it costs no vector work in the group loop.
//
// Tile: 128 tokens x 256 outputs by FOUR wavefronts (each all rows x 64 columns, 4 x 2 MFMAs of 32x32x16), two such
// workgroups on a compute unit.  What decides the shape:
//   * The packed weights never go through LDS.  The blob stores a code tile in the operand order of the 16x16x32 MFMA,
//     so a wavefront loads the codes of its own 64 columns into registers (one group ahead) and unpacks them straight
//     into the B operand.  (The 32x32x16 MFMA takes 32 columns, two code tiles, and from each the codes of two of the four
//     lane quarters, in two rounds of four steps: kq = hh and hh + 2 for the lanes' halves hh.)  LDS then carries the activations only: 64 KB per 32 columns and compute unit, half of what
//     the matrix cores' time would allow (the 256 x 256 tile of eight wavefronts that this replaces moved 132 KB
//     through LDS per 32 columns with a workgroup barrier each).
//   * One barrier per group of 128 columns.  The activations of the next group (32 KiB, loaded straight into LDS by
//     the memory pipeline) and its codes are requested at the top of a group and waited for at its end, about two
//     thousand cycles later; the two workgroups of a compute unit are not in step, so one computes while the other
//     stands at its barrier, and one's unpacking runs under the other's MFMAs.
//   * 32x32x16 and not 16x16x32: the same products in half the instructions (32.5 cycles against 2 x 17), half as many
//     column tiles, so half of a group's scales, ratios and operand registers (11008 x 4096 at 2048 tokens 189 -> 184 us at
//     2 bits, 220 -> 200 at 4, 240 -> 222 at 6, 303 -> 291 at 8 bits).
//   * Remainders of a bucket run the same loop with 1, 2 or 3 row tiles of 32 instead of 4 (a bucket's last 16..32 tokens
//     used to hold a compute unit as long as 256 tokens: four such remainders set the time below 1024 tokens).
//   * Rows are fetched through the permutation (16 lanes read 256 bytes of one token), so no sorted copy is made.
//   * A wavefront alone issues a vector instruction every 7 cycles, two share a SIMD at 4.6 for most of the unpacking's
//     (measured), and 16 cycles of MFMA hide two of them but not four: so unpacking and rescaling are dealt out under
//     the MFMAs one column tile later (`spread`), and nothing but those stands in the group loop.
//   * What a tile costs besides its groups matters at K = 4096 and where a launch is one round: its row sums come through
//     LDS, its rows leave through LDS (see load_sums and the stores): 16400 + 8000 cycles -> 7500 + 1000 a tile.
// Whole calls, before the last three and the zero-point term in bf16 pieces, and now: 11008 x 4096 at 2048 tokens,
// {50,30,15,5} % mix 248 -> 210 us (878 TFLOP/s), all tokens at 2 bits 210 -> 174 us, at 8 bits 335 -> 284 us; 28672 x 8192 at
// 4096 tokens, {70,20,8,2} % mix 1912 -> 1680 us (1145 TFLOP/s; a dense bf16 library product reaches 1383 on this card), at
// 256 tokens 304 -> 249 us; 3000 x 2176 at 777 tokens 56 -> 43 us.  Bound by the clock, which falls to 1.9 GHz and below
// under this load: at 28672 x 8192 and 2 bits leaving out the rescaling, or the unpacking, or both gains 7 %, leaving out the
// copies of the activations 8 %; codes of 4 bits, which differ in the bits that the multipliers see, take 9 % longer than
// those of 2 bits without any unpacking too.
#include "mbq_common.h"

namespace mbq {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

namespace pf {

constexpr int kBM = 128, kBN = 256;

constexpr int kRowBytes = 2 * kGroup;         // one group of one token: 16 chunks of 16 bytes, swizzled by the row
constexpr int kStageBytes = kBM * kRowBytes;  // 32 KiB, two stages
constexpr int kSumsBytes = kBM * 16 * 6;      // group sums of the tile's rows, 16 groups at a time, in three bf16 pieces
constexpr int kRowsBytes = 2 * kBM * 4;       // tokens of the rows, byte offsets of their activations
constexpr int kPadRows = 256;                 // rows of the workspace beyond those of the activations
constexpr int kMaxSplits = 8;

// A matrix of a launch.
struct Proj {
  const uint32_t* codes;
  size_t slice_words;
  const float2* meta;
  const int32_t* perm;
  const int32_t* offsets;
  float* Y;
  int64_t N;
  float* slot;         // T x N arrays of partial sums besides Y, slot_floats apart
  int64_t slot_floats;
  int NT;              // 16-row code tiles
  int cols;            // column tiles of kBN
  int splits, slots;   // parts along K, arrays that take them (Y is the first)
  int block_begin;     // index of this matrix's first workgroup
};
struct Group {
  Proj p[MBQ_MAX_GROUP];
  int n;
};

// ---- pre-kernel: Sx[token][g] = sum_{k in g} X[token][k]; arrays that the tile kernel adds into are cleared; sorted
// copy Xs[r][:] = X[perm[r]][:] where one is wanted.  A stage call has the router launch do this (PrefillPrep). -------
__global__ __launch_bounds__(256) void prefill_prep_kernel(const PrefillPrep p, int64_t K, const int32_t* __restrict__ perm,
                                                           uint16_t* __restrict__ Xs) {
  const int64_t r = blockIdx.x;
  if (!Xs) {
    prefill_prep_share(p, gridDim.x, K, r, 1, 256);
    return;
  }
  prefill_clear(p.zl, r * 256 + threadIdx.x, (int64_t)gridDim.x * 256);
  prefill_clear(p.zs, r * 256 + threadIdx.x, (int64_t)gridDim.x * 256);
  const int64_t token = perm[r];
  prefill_row_sums(reinterpret_cast<const uint4*>(p.X + token * K), K, threadIdx.x, p.Sx + token * (K >> 7),
                   reinterpret_cast<uint4*>(Xs + r * K));
}

__device__ __forceinline__ floatx16 mfma(const u32x4& a, const u32x4& b, floatx16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
__device__ __forceinline__ uint32_t rotr32(uint32_t w, int r) {  // r compile-time after inlining
  return (r & 31) == 0 ? w : __builtin_amdgcn_alignbit(w, w, r & 31);
}
__host__ __device__ constexpr uint32_t rotl_c(uint32_t m, int r) {
  return ((r & 31) == 0) ? m : ((m << (r & 31)) | (m >> (32 - (r & 31))));
}
// mantissa factor m of a group scale (see the header): exponent field forced to 126 or 127
__device__ __forceinline__ float scale_mantissa(float s0) {
  return __uint_as_float((__float_as_uint(s0) & 0x00FFFFFFu) ^ 0x3F800000u);
}
// biased bf16 exponent E (even) of (256 + V) * 2^t
__device__ __forceinline__ uint32_t scale_exponent(float s0) { return ((__float_as_uint(s0) >> 23) + 9u) & ~1u; }

// dma_16 with 4 bytes per lane and an address of its own
__device__ __forceinline__ void dma_4(uint32_t lds, const void* address) {
  uint32_t m0;
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %2, off\n\ts_mov_b32 m0, %0"
               : "=&s"(m0)
               : "s"(lds), "v"(address)
               : "memory");
}

// eight floats as sums of three bf16, each the rest rounded to nearest (8 bits, then at most 15 of 24 left, then at most 7: the
// last is exact); the second piece is at most 2^-9 of the number, the third 2^-18.  (A row sum's pieces are exact down to the
// smallest rows: sums of bf16 numbers are multiples of 2^-133, which bf16 holds.)
__device__ __forceinline__ void split_bf16(const float (&v)[8], u32x4 (&pieces)[3]) {
  typedef float floatx2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float r0 = v[2 * i], r1 = v[2 * i + 1];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const uint32_t piece = __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{r0, r1}, bf16x2));
      pieces[j][i] = piece;
      r0 -= __uint_as_float(piece << 16);
      r1 -= __uint_as_float(piece & 0xFFFF0000u);
    }
    pieces[2][i] = __builtin_amdgcn_perm(__float_as_uint(r1), __float_as_uint(r0), 0x07060302u);
  }
}

// scheduling hint: the region's MFMAs one by one, `each` vector instructions behind every one of them
template <int MFMAS>
__device__ __forceinline__ void spread(int each) {
#define MBQ_SPREAD(n)                                         \
  case n:                                                     \
    _Pragma("unroll") for (int a = 0; a < MFMAS; ++a) {       \
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);      \
      __builtin_amdgcn_sched_group_barrier(0x002, n, 0);      \
    }                                                         \
    break;
  switch (each) {
    MBQ_SPREAD(2) MBQ_SPREAD(3) MBQ_SPREAD(4) MBQ_SPREAD(5) MBQ_SPREAD(6) MBQ_SPREAD(7) MBQ_SPREAD(8) MBQ_SPREAD(9)
    MBQ_SPREAD(10) MBQ_SPREAD(11) MBQ_SPREAD(12) MBQ_SPREAD(13) MBQ_SPREAD(14) MBQ_SPREAD(16) MBQ_SPREAD(18) MBQ_SPREAD(19)
    MBQ_SPREAD(20) MBQ_SPREAD(21) MBQ_SPREAD(22) MBQ_SPREAD(23) MBQ_SPREAD(24) MBQ_SPREAD(26) MBQ_SPREAD(28) MBQ_SPREAD(30)
    default: break;
  }
#undef MBQ_SPREAD
}

// One tile: rows row0 .. row0 + rows - 1 of the sorted tokens, columns 256 ntile_n ..; groups g0 .. g0 + G - 1.
// P = precision index of the tokens, MR = 16-row tiles, an even number (16 MR >= rows; the products take them in pairs).
// gather: X is in token order and rows are fetched through perm; otherwise X is the sorted copy.
// halfway, kPieces: when and how the zero-point term is removed, see remove_in_pieces.
// out: the T x N array the tile goes to; accumulate: it is added there (two parts of K share the array).
template <int P, int MR, bool kPieces>
__device__ __forceinline__ void tile(const uint16_t* __restrict__ X, int64_t K, int KB, bool gather, const Proj& M,
                                     const float* __restrict__ Sx, int row0, int rows, int ntile_n, char* smem, int g0,
                                     int G, bool halfway, float* out, bool accumulate) {
  constexpr float kOff = (P == 3) ? 0.f : 256.f;
  constexpr float kHalf = 0.5f * (float)(1 << (2 * (3 - P)));
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l15 = lane & 15, kq = lane >> 4;
  const int l31 = lane & 31, hh = lane >> 5;
  const int32_t* __restrict__ perm = M.perm;

  // ---- A: one instruction moves a group of four rows (16 lanes a row); MR instructions a wavefront and group: rows
  // 4 wave + 16 j + kq.  LDS chunk l15 of a row holds its chunk l15 ^ (row & 15), so the 16 rows of a fragment read
  // hit different banks.  Rows past the tile repeat its last row. ----
  const uint16_t* xbase = (gather ? X : X + (int64_t)row0 * K) + (int64_t)g0 * kGroup;
  // The tokens of the rows and where their activations begin wait in LDS: the zero-point term and the stores need the
  // former, P = 3 reads the latter at every group (its unpacking leaves no registers for them).
  constexpr bool kOffLds = P == 3 && MR == 8;
  float* const s_sum = reinterpret_cast<float*>(smem + 2 * kStageBytes);
  int* const s_token = reinterpret_cast<int*>(smem + 2 * kStageBytes + kSumsBytes);
  uint32_t* const s_row = reinterpret_cast<uint32_t*>(s_token + kBM);
  if (tid < 16 * MR) {
    const int r = min(tid, rows - 1), token = perm[row0 + r];
    s_token[tid] = token;
    s_row[tid] = 2u * (uint32_t)(gather ? token : r) * (uint32_t)K;
  }
  __syncthreads();
  const uint32_t a_chunk = 16u * (uint32_t)(l15 ^ (4 * wave + kq));
  uint32_t a_off[kOffLds ? 1 : MR];
  if constexpr (!kOffLds) {
#pragma unroll
    for (int j = 0; j < MR; ++j) a_off[j] = s_row[4 * wave + 16 * j + kq] + a_chunk;
  }
  const uint32_t lds0 =
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)smem + (uint32_t)(4 * wave * kRowBytes);
  auto load_a = [&](int g, uint32_t stage) {
    const uint16_t* src = xbase + (int64_t)g * kGroup;
#pragma unroll
    for (int j = 0; j < MR; ++j)
      dma_16(lds0 + stage + (uint32_t)(j * 16 * kRowBytes), kOffLds ? s_row[4 * wave + 16 * j + kq] + a_chunk : a_off[kOffLds ? 0 : j], src);
  };
  // ---- B: this wavefront's two column tiles of 32, a pair of code tiles each; four dwords a lane, tile, slice and group ----
  const uint32_t* wptr[2];
  const float* sptr[2];
  uint32_t w_tile[2];  // words from the first of a pair's code tiles to this lane's
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    int nt = ntile_n * (kBN / kTileN) + 4 * wave + 2 * c;
    nt = nt < M.NT ? nt : 0;  // past the matrix: reads another tile, never stored
    wptr[c] = M.codes + (size_t)nt * KB * kTileWords;
    sptr[c] = reinterpret_cast<const float*>(M.meta + (size_t)nt * (2 * KB) * kTileN);
    w_tile[c] = (l31 >= 16 && nt + 1 < M.NT) ? (uint32_t)KB * kTileWords : 0u;
  }
  u32x2 w_cur[2][2][P + 1], w_nxt[2][2][P + 1];
  float s_cur[2], s_nxt[2];
  auto load_w = [&](int g, u32x2 (&w)[2][2][P + 1], float (&s)[2]) {
    const int ga = g0 + g;
    // (32-bit offsets from wave-uniform addresses: one code tile row is at most 2^26 bytes)
    const uint32_t v = (uint32_t)(ga >> 1) * kTileWords + 2u * (uint32_t)(ga & 1) + 4u * (uint32_t)(16 * hh + l15);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e <= P; ++e)
          w[c][j][e] = *reinterpret_cast<const u32x2*>(wptr[c] + e * M.slice_words + (w_tile[c] + v + 128u * (uint32_t)j));
      s[c] = sptr[c][(w_tile[c] >> 2) + (uint32_t)(2 * (ga * kTileN + l15))];
    }
  };
  // the compiler's own wait for these loads is placed here (they have landed: the explicit wait came first)
  auto settle = [&](u32x2 (&w)[2][2][P + 1], float (&s)[2]) {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e <= P; ++e) asm volatile("" : "+v"(w[c][j][e]));
      asm volatile("" : "+v"(s[c]));
    }
  };
  // per-row operand constant of the group: the replicated high exponent byte (P <= 2) or the bits of 2^t (P = 3)
  uint32_t b_x[2];
  // merged fields of the four weights with bit residue 2 r (r = step or step + 2), byte aligned; P <= 2: one bit
  // further, V / 2
  auto merge_bits = [&](int pair, int c, int j, int r) -> uint32_t {
    uint32_t bits = w_cur[c][j][0][pair] & rotl_c(0xC0C0C0C0u, 2 * r - 4);
    if constexpr (P >= 1) bits |= w_cur[c][j][1][pair] & rotl_c(0x30303030u, 2 * r - 4);
    if constexpr (P >= 2) bits |= w_cur[c][j][2][pair] & rotl_c(0x0C0C0C0Cu, 2 * r - 4);
    if constexpr (P >= 3) bits |= w_cur[c][j][3][pair] & rotl_c(0x03030303u, 2 * r - 4);
    return rotr32(bits, (2 * r - 4 + (P == 3 ? 0 : 1)) & 31);
  };
  // two bf16 of one merged word: bytes (0, 2) and (1, 3)
  auto expand_pair = [&](uint32_t w, int c, int b0) -> uint32_t {
    if constexpr (P == 3) {
      const float sc = __uint_as_float(b_x[c]);
      const float f0 = (float)((w >> (8 * b0)) & 0xFFu) * sc;
      const float f1 = (float)((w >> (8 * (b0 + 2))) & 0xFFu) * sc;
      return __builtin_amdgcn_perm(__float_as_uint(f1), __float_as_uint(f0), 0x07060302u);
    } else {
      return __builtin_amdgcn_perm(b_x[c], w, b0 ? 0x04030401u : 0x04020400u);
    }
  };
  auto unpack = [&](int step, int c) -> u32x4 {  // B operand of a step (16 columns) of the group, column tile c
    const int h = step & 3, j = step >> 2;
    const uint32_t lo = merge_bits(h >> 1, c, j, h & 1), hi = merge_bits(h >> 1, c, j, (h & 1) + 2);
    return u32x4{expand_pair(lo, c, 0), expand_pair(hi, c, 0), expand_pair(lo, c, 1), expand_pair(hi, c, 1)};
  };

  constexpr int RT = MR / 2;  // row tiles of 32
  floatx16 acc[RT][2];
#pragma unroll
  for (int a = 0; a < RT; ++a)
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[a][c][i] = 0.f;
  float m_cur[2];

  load_a(0, 0u);
  load_w(0, w_cur, s_cur);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  settle(w_cur, s_cur);
  asm volatile("s_barrier" ::: "memory");
#pragma unroll
  for (int c = 0; c < 2; ++c) m_cur[c] = scale_mantissa(s_cur[c]);

  // The zero-point / offset term of groups g .. last - 1 (at most 16), in the accumulator's units, as a rank-16 update by
  // MFMAs: lane half hh holds groups 8 hh .. 8 hh + 7 (the order of the k axis is free as long as both operands
  // share it).  Every 16 groups and not once at the end: the offset is many times the signal, and what the accumulator
  // carries sets its rounding (11008 x 4096: 1.8e-6 relative against 2.8e-6 with one update at the end, 4096 x 28672
  // 1.9e-6 against 6.4e-6).  halfway: the update comes when half of its groups are done, so that
  // the accumulator carries the offset of half as many (3000 x 2176 at 777 tokens in two parts: 0.93e-6 relative behind
  // them, 0.74e-6 half way, 0.70e-6 in four parts).  Taken for parts of at most 16 groups, which replace twice as many
  // parts where there is no room for those; long parts lose up to 7 % by it (8192 x 28672 at 256 tokens 263 -> 282 us: the
  // scales of groups to come are not in cache yet).
  // In fp32 (32x32x2, 64 cycles each) the update takes as many cycles as two groups.  kPieces: both operands as sums of
  // three bf16, exact to 24 bits, and six of their nine products (the other three are below 2^-25 of a product) in 32x32x16
  // MFMAs, two fifths of that.  The rows' sums are split once for the workgroup, in their place in LDS.  The first product
  // goes into the accumulator, the small ones come together in registers of their own and are added at once, so that the sum
  // is rounded twice at its size and not eight times: against 64 bits 1.5e-6 -> 1.4e-6 relative for 11008 x 4096 at 2
  // bits, 1.8e-6 -> 1.7e-6 for the mix (all six into the accumulator, the smallest first: 1.6e-6 and 1.9e-6), and 184 -> 175
  // us, 28672 x 8192 at 256 tokens 273 -> 250.  In fp32 it stays for parts of at most 8 groups, where that rounds less
  // (1000 x 2176 at 777 tokens 0.90e-6 against 0.93e-6), and for P = 3, whose unpacking leaves no registers for the
  // pieces (11008 x 4096 at 2048 tokens 284 us in fp32, 294 in pieces).
  // The rows' sums of 16 groups come to LDS at the beginning of these groups ([row][16], by four bytes a lane: a token's
  // sums need not be aligned) and are there at the first barrier behind.  Fetched where they are used, token by token and
  // then sum by sum, they took a dozen trips to memory one after the other: about 8 us a tile.
  const int Gtot = (int)(K / kGroup);
  auto load_sums = [&](int g) {
    const uint32_t lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)smem + 2 * kStageBytes;
    const float* src = Sx + g0 + min(g + l15, G - 1);
#pragma unroll
    for (int j = 0; j < MR; ++j)
      dma_4(lds + (uint32_t)((4 * wave + 16 * j) * 64), src + (int64_t)s_token[4 * wave + 16 * j + kq] * Gtot);
  };
  auto remove_in_fp32 = [&](int g, int last) {
    constexpr float kC = (kHalf - kOff) * (1.f / 64.f);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const float units = 64.f / m_cur[c];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        float bv[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int gg = min(g + 8 * hh + 4 * j + s, last - 1);
          const float2 mt =
              *reinterpret_cast<const float2*>(sptr[c] + ((w_tile[c] >> 2) + (uint32_t)(2 * ((g0 + gg) * kTileN + l15))));
          bv[s] = (g + 8 * hh + 4 * j + s < last) ? mt.x * (kC - mt.y) * units : 0.f;
        }
#pragma unroll
        for (int a = 0; a < RT; ++a) {
          const floatx4 av = *reinterpret_cast<const floatx4*>(s_sum + (32 * a + l31) * 16 + 8 * hh + 4 * j);
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const float v = (g + 8 * hh + 4 * j + s < last) ? av[s] : 0.f;
            acc[a][c] = __builtin_amdgcn_mfma_f32_32x32x2f32(v, bv[s], acc[a][c], 0, 0, 0);
          }
        }
      }
    }
  };
  auto remove_in_pieces = [&](int g, int last) {
    constexpr float kC = (kHalf - kOff) * (1.f / 64.f);
    const int k0 = g + 8 * hh;      // this lane's first group as an operand
    float2 mt[2][8];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int s = 0; s < 8; ++s)
        mt[c][s] = *reinterpret_cast<const float2*>(
            sptr[c] + ((w_tile[c] >> 2) + (uint32_t)(2 * ((g0 + min(k0 + s, last - 1)) * kTileN + l15))));
    u32x4* const s_piece = reinterpret_cast<u32x4*>(s_sum);  // [piece][row][16 groups]
    {
      float v[8];
      const int row = tid >> 1, half = tid & 1;
      if (tid < 32 * MR) {
        const floatx4* own = reinterpret_cast<const floatx4*>(s_sum + row * 16 + 8 * half);
#pragma unroll
        for (int s = 0; s < 8; ++s) v[s] = (g + 8 * half + s < last) ? own[s >> 2][s & 3] : 0.f;
      }
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      if (tid < 32 * MR) {
        u32x4 pieces[3];
        split_bf16(v, pieces);
#pragma unroll
        for (int i = 0; i < 3; ++i) s_piece[i * 2 * kBM + tid] = pieces[i];
      }
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }
    u32x4 b[2][3];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const float units = 64.f / m_cur[c];
      float v[8];
#pragma unroll
      for (int s = 0; s < 8; ++s) v[s] = (k0 + s < last) ? mt[c][s].x * (kC - mt[c][s].y) * units : 0.f;
      split_bf16(v, b[c]);
    }
#pragma unroll
    for (int a = 0; a < RT; ++a) {
      u32x4 x[3];
#pragma unroll
      for (int i = 0; i < 3; ++i) x[i] = s_piece[i * 2 * kBM + 2 * (32 * a + l31) + hh];
      floatx16 small[2];
#pragma unroll
      for (int i = 0; i < 16; ++i) small[0][i] = small[1][i] = 0.f;
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3 - i; ++j)
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            floatx16& sum = i + j == 0 ? acc[a][c] : small[c];
            sum = mfma(x[i], b[c][j], sum);
          }
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[a][c][i] += small[c][i];
    }
  };

  uint32_t stage = 0u;
  int q = 0;
#pragma unroll 1
  for (int first = 0; first < G + 16; first += 16) {
    const int last = min(G, first + 16);
    const int stop = first < G && halfway ? (first + last + 1) >> 1 : last;
    if (first < G) {
      // every wavefront has read the sums before these (the reads are over, not just issued: what follows overwrites them)
      if (first > 0) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      load_sums(first);
    }
#pragma unroll 1
    for (; q < stop; ++q) {
      // the next group on its way (the last group is requested once more: the other stage is free)
      const int qn = q + 1 < G ? q + 1 : q;
      load_a(qn, stage ^ (uint32_t)kStageBytes);
      load_w(qn, w_nxt, s_nxt);
      __builtin_amdgcn_sched_barrier(0);
      float ratio[2];
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const uint32_t E = scale_exponent(s_cur[c]);
        b_x[c] = (P == 3) ? ((E - 8u) << 23) : ((E >> 1) * 0x01010101u);
        const float r = m_cur[c] * __builtin_amdgcn_rcpf(scale_mantissa(s_cur[c]));
        ratio[c] = (q > 0) ? r : 1.f;
        // the factor actually in force (keeps the chain consistent): m / ratio within
        // 0.5000002 of a last place (a reciprocal off by one place and a corrected quotient: the rounded one but for 3 in 10^7)
        const float inv = __builtin_amdgcn_rcpf(ratio[c]), quot = m_cur[c] * inv;
        m_cur[c] = __builtin_fmaf(__builtin_fmaf(-quot, ratio[c], m_cur[c]), inv, quot);
      }
      // fragment of row tile a, step: row 32 a + l31, the chunk whose codes this lane unpacks for the step
      auto read_a = [&](int step, int a) -> u32x4 {
        const uint32_t at = stage + (uint32_t)l31 * kRowBytes + (uint32_t)(((4 * (step & 3) + 2 * (step >> 2) + hh) ^ l15) * 16);
        return *reinterpret_cast<const u32x4*>(smem + at + a * 32 * kRowBytes);
      };
      // HR row tiles at a time, their fragments read one part ahead; the operand of column tile c of the next step is
      // unpacked into the same registers right behind the last MFMAs that read it.  A scheduling fence per column tile
      // keeps the registers of one part alive at a time: without it the compiler hoists unpacking and spills.
      constexpr int HR = P == 3 && RT == 4 ? 1 : RT;
      constexpr int kParts = RT / HR;
      u32x4 af[2][HR], bf[2];
#pragma unroll
      for (int a = 0; a < HR; ++a) af[0][a] = read_a(0, a);
      bf[0] = unpack(0, 0);
      auto rescale = [&](int part, int c) {  // to the units of this group
#pragma unroll
        for (int a = 0; a < HR; ++a)
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[part * HR + a][c][i] *= ratio[c];
      };
      rescale(0, 0);
#pragma unroll
      for (int hp = 0; hp < 8 * kParts; ++hp) {
        const int h = hp / kParts, part = hp % kParts;
        if (hp + 1 < 8 * kParts) {
#pragma unroll
          for (int a = 0; a < HR; ++a) af[(hp + 1) & 1][a] = read_a((hp + 1) / kParts, ((hp + 1) % kParts) * HR + a);
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) {
#pragma unroll
          for (int a = 0; a < HR; ++a) acc[part * HR + a][c] = mfma(af[hp & 1][a], bf[c], acc[part * HR + a][c]);
          // under these MFMAs: the operand whose last MFMAs were issued one column tile ago, the next tiles' units
          const bool un0 = part == kParts - 1 && c == 1 && h < 7, un1 = part == 0 && c == 0;
          if (un0) bf[0] = unpack(h + 1, 0);
          if (un1) bf[1] = unpack(h, 1);
          const bool re = h == 0 && (c == 0 || part + 1 < kParts);
          if (re) rescale(c == 0 ? part : part + 1, c ^ 1);
          spread<HR>(((un0 || un1 ? 8 + 2 * P : 0) + (re ? 16 * HR : 0) + HR - 1) / HR);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      // this wavefront's requests have landed and its reads of the stage are done; behind the barrier everybody's are
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
      settle(w_nxt, s_nxt);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int e = 0; e <= P; ++e) w_cur[c][j][e] = w_nxt[c][j][e];
        s_cur[c] = s_nxt[c];
      }
      asm volatile("s_barrier" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      stage ^= (uint32_t)kStageBytes;
    }
    if (first < G) {
      if constexpr (kPieces) remove_in_pieces(first, last);
      else remove_in_fp32(first, last);
    }
  }

  // ---- rows in original token order.  Of a row tile of 32 a lane holds rows 8 (i >> 2) + 4 hh + (i & 3), i = 0 .. 15, and
  // columns 32 c + l31: stored from there an instruction writes two pieces of 128 bytes (from the layout of 16 x 16 tiles, four
  // of 64, it took 32 cycles each, 16400 a tile).  So 16 rows at a time go through the wavefront's own part of the stages
  // (free behind the last barrier; LDS operations of a wavefront execute in order): an instruction then writes four
  // rows of 256 bytes, or one where rows are not 16-byte aligned or two parts of K add. ----
  constexpr int kRow = 64 + 4;  // floats between rows
  float* const own = reinterpret_cast<float*>(smem) + wave * (16 * kRow);
  const int64_t col0 = (int64_t)ntile_n * kBN + 64 * wave;
  const bool wide = !accumulate && (M.N & 3) == 0 && (reinterpret_cast<uintptr_t>(out) & 15) == 0;
  float f[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) f[c] = m_cur[c] * (1.f / 64.f);  // true units
#pragma unroll
  for (int a = 0; a < MR; ++a) {
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int i = 0; i < 8; ++i)
        own[(8 * (i >> 2) + 4 * hh + (i & 3)) * kRow + 32 * c + l31] = acc[a >> 1][c][8 * (a & 1) + i] * f[c];
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (wide) {
      floatx4 v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = *reinterpret_cast<const floatx4*>(own + (4 * i + kq) * kRow + 4 * l15);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = 16 * a + 4 * i + kq;
        if (r < rows && col0 + 4 * l15 < M.N)
          *reinterpret_cast<floatx4*>(out + (int64_t)s_token[r] * M.N + col0 + 4 * l15) = v[i];
      }
    } else if (col0 + lane < M.N) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int r = 16 * a + i;
        if (r < rows) {
          float* y = out + (int64_t)s_token[r] * M.N + col0 + lane;
          const float v = own[i * kRow + lane];
          if (accumulate) unsafeAtomicAdd(y, v);  // cleared by the pre-kernel
          else *y = v;
        }
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  }
}

__global__ __launch_bounds__(256, 2) void prefill_kernel(const uint16_t* __restrict__ X, int64_t K, int KB, int gather,
                                                         const float* __restrict__ Sx, const Group grp) {
  __shared__ __attribute__((aligned(1024))) char smem[2 * kStageBytes + kSumsBytes + kRowsBytes];
  int j = 0;
#pragma unroll
  for (int i = 1; i < MBQ_MAX_GROUP; ++i)
    if (i < grp.n && (int)blockIdx.x >= grp.p[i].block_begin) j = i;
  const Proj& M = grp.p[j];
  // (tile row, tile column, K split): workgroups of one tile row are neighbours (they share activations)
  const int block = (int)blockIdx.x - M.block_begin, splits = M.splits;
  const int per_mt = M.cols * splits;
  const int mt = block / per_mt, ntile_n = (block % per_mt) / splits, split = block % splits;
  const int Gtot = (int)(K / kGroup);
  const int g0 = (int)((int64_t)split * Gtot / splits);
  const int Gs = (int)((int64_t)(split + 1) * Gtot / splits) - g0;
  int off[MBQ_N_PRECISIONS + 1];
#pragma unroll
  for (int q = 0; q <= MBQ_N_PRECISIONS; ++q) off[q] = M.offsets[q];
  // The tiles of a matrix by falling cost, so that the launch does not end on a long one: from the highest precision
  // down, then the remainders of up to 64 tokens.  (Ascending precisions, the 8-bit remainder last: 315 us instead of
  // 237 for 11008 x 4096 at 2048 tokens.)
  int p = -1, row0 = 0, rows = 0, idx = mt;
#pragma unroll
  for (int q = MBQ_N_PRECISIONS - 1; q >= 0; --q) {
    const int large = (off[q + 1] - off[q] + 63) / kBM;  // full tiles and a remainder of more than 64
    if (p < 0) {
      if (idx < large) {
        p = q;
        row0 = off[q] + idx * kBM;
        rows = min(kBM, off[q + 1] - row0);
      } else {
        idx -= large;
      }
    }
  }
#pragma unroll
  for (int q = MBQ_N_PRECISIONS - 1; q >= 0; --q) {
    const int rem = (off[q + 1] - off[q]) % kBM;
    if (p < 0 && rem > 0 && rem <= 64) {
      if (idx == 0) {
        p = q;
        row0 = off[q + 1] - rem;
        rows = rem;
      } else {
        --idx;
      }
    }
  }
  if (p < 0) return;
  // part s goes to array s mod slots; an array that two parts share is added into
  const int slot = split % M.slots;
  float* const out = slot == 0 ? M.Y : M.slot + (slot - 1) * M.slot_floats;
  const bool shared = slot + M.slots < splits;
  const bool halfway = splits > 1 && Gs <= 16;  // for this and `few` see remove_in_pieces
#define MBQ_TILE(PP, MM, PI) tile<PP, MM, PI>(X, K, KB, gather != 0, M, Sx, row0, rows, ntile_n, smem, g0, Gs, halfway, out, shared)
#define MBQ_ROWS(PP, PI)                     \
  do {                                       \
    if (rows > 96) MBQ_TILE(PP, 8, PI);      \
    else if (rows > 64) MBQ_TILE(PP, 6, PI); \
    else if (rows > 32) MBQ_TILE(PP, 4, PI); \
    else MBQ_TILE(PP, 2, PI);                \
  } while (0)
  const bool few = Gs <= 8;
  switch (p) {
    case 0:
      if (few) MBQ_ROWS(0, false);
      else MBQ_ROWS(0, true);
      break;
    case 1:
      if (few) MBQ_ROWS(1, false);
      else MBQ_ROWS(1, true);
      break;
    case 2:
      if (few) MBQ_ROWS(2, false);
      else MBQ_ROWS(2, true);
      break;
    default: MBQ_ROWS(3, false); break;
  }
#undef MBQ_ROWS
#undef MBQ_TILE
}

}  // namespace pf

static inline int64_t prefill_ld(int64_t T) { return (T + 32 + 63) / 64 * 64; }
static inline size_t prefill_copy_bytes(int64_t T, int64_t K) {
  return ((size_t)(T + pf::kPadRows) * K * sizeof(uint16_t) + 255) / 256 * 256;
}

// group sums, and room for a sorted copy of the activations or, where none is made, for arrays of partial sums
size_t prefill_workspace_bytes(int64_t T, const Shape& sh) {
  const size_t xs = (size_t)(T + pf::kPadRows) * sh.K * sizeof(uint16_t);
  const size_t sx = (size_t)sh.G * prefill_ld(T) * sizeof(float);
  return xs + sx + 256;
}

// How a matrix is cut along K: a launch with few tiles leaves compute units idle, so each tile is cut into `parts`
// workgroups.  Part s stores into array s mod `slots` - Y, then arrays of the workspace -, an array that two parts share
// is cleared ahead and added into (two addends: their order does not matter), and a last launch adds the arrays to Y in
// order.  So results do not depend on which workgroup comes first.  Arrays lie where the sorted copy of the activations
// would (below 4 GiB none is made); where there is no room for one a matrix is cut in two at most.
// (Parts that all added into Y, in whatever order they came, took 69 us instead of 79 for 4096 x 11008 at 256 tokens, 47
// instead of 54 at 96, and 91 instead of 72 for 3000 and 1000 x 2176 at 777, where four parts did not fit.)
struct Split {
  int parts, slots;
};
static inline int64_t slot_floats(int64_t T, int64_t N) { return (T * N + 3) / 4 * 4; }
static Split split_into(int parts, int64_t T, int64_t K, int64_t N, int64_t area_floats) {
  const int64_t room = 1 + area_floats / slot_floats(T, N);
  if (parts > 2 * room) parts = (int)(2 * room);
  while (parts > 1 && K / kGroup / parts < 4) --parts;
  return Split{parts, parts <= 2 ? 1 : parts < room ? parts : (int)room};
}
// An estimate of a launch, in units of what a compute unit needs for two whole tiles side by side (17 ns x K): with r =
// tiles x parts / workgroups resident at a time, the rounds cost 0.82 + 0.36 r up to one round (a workgroup alone on
// its unit is hardly faster than one of two) and 1.48 + w (r - 1) beyond (tiles differ in cost and are started by
// falling cost, so rounds are not in step; w: below 333 tokens the tiles of four buckets are half empty); a part costs
// its share of the K axis and eight groups for its prologue, zero-point term and stores; adding costs 350 / K for every
// output tile's worth of rows and part over the resident workgroups, the last launch 135 / K.
static double split_cost(Split sp, int64_t T, int64_t K, int64_t cols) {
  const int64_t rows = T / pf::kBM + 2 > 4 ? T / pf::kBM + 2 : 4;  // a bucket ends on a partial tile
  const double column_parts = (double)(cols * sp.parts) / (2.0 * device_compute_units());
  const double r = (double)rows * column_parts, w = T < 333 ? 0.55 + 0.45 * (double)T / 333.0 : 1.0;
  const double rounds = r <= 1.0 ? 0.82 + 0.36 * r : 1.48 + w * (r - 1.0);
  return rounds * (1.0 / sp.parts + 8.0 * kGroup / (double)K) +
         (sp.parts > 1 ? 350.0 * (double)T / pf::kBM * column_parts / (double)K : 0.0) +
         (sp.slots > 1 ? 135.0 / (double)K : 0.0);
}
// The cut that minimises the estimate, among those of at most `most` parts. Fitted to 1..8 parts on twenty shapes from
// 1000 x 2176 to 28672 x 8192, alone and in groups of two and three, at 65..4096 tokens: 1.0 % above the best cut alone
// on average (17 % on the worst), 0.6 % (13 %) in groups; of the tile kernel as it is now, 39 calls, 2.1 % above the best cut
// on average (19 % on the worst, 4096 x 14336 at 300 tokens 91 in eight parts, 76 in four; next 4096 x 11008 at 512 tokens 102,
// 89 in three, and 2048 x 8192 at 700 tokens 72, 62 in four; constants fitted anew came to 1.5 %, so they stay). For instance (us, 1 / 2 / 4 / 8 parts; * taken) 4096 x 11008 at 256 tokens 177 / 97 / 74 / 66*, at
// 2048 tokens 311 / 260* / 287 / -, 4096 x 4096 at 160 tokens 68 / 40 / 33*, 11008 x 4096 at 256 tokens 77 / 62*, at 777
// tokens 118* / 150.
// pairs: a matrix with as many rows as columns or more has company more often than not (q, k, v of an attention; gate
// and up of a gated MLP, with twice as many rows or more), and one or two parts have to be the same in company and
// alone (choose_splits): the product of the estimates alone and, `pairs` times, as a pair decides (14336 x 4096 at 160
// tokens, 1 / 2 parts: alone 76 / 53*, as a pair 115 / 110*; at 256 tokens as a pair 117* / 130).
// knob 5 forces the number of parts.
static Split choose_split(int64_t T, int64_t K, int64_t N, int64_t cols, int pairs, int most, int64_t area_floats) {
  if (knob(5) >= 1 && knob(5) <= pf::kMaxSplits) return split_into(knob(5), T, K, N, area_floats);
  Split best{1, 1};
  double best_cost = 0.0;
  for (int s = 1; s <= most; ++s) {
    const Split sp = split_into(s, T, K, N, area_floats);
    if (sp.parts != s) continue;
    double cost = split_cost(sp, T, K, cols);
    for (int i = 0; i < pairs; ++i) cost *= split_cost(sp, T, K, 2 * cols);
    if (s == 1 || cost < 0.98 * best_cost) {
      best_cost = cost;
      best = sp;
    }
  }
  return best;
}
// The cuts of the n matrices of a call. One or two parts: the matrix alone decides, so that a call for several matrices
// gives the bits of separate calls. More: a group that fills the chip needs fewer (three of 4096 x 4096 at 256 tokens:
// 72 us in two parts each, 157 in four and one launch after the other), and the matrices share the room for arrays.
static void choose_splits(int64_t T, int64_t K, int n, const Shape* shapes, int64_t area_floats, Split* out) {
  auto columns = [](const Shape& sh) { return (sh.N + pf::kBN - 1) / pf::kBN; };
  int64_t all = 0;
  for (int i = 0; i < n; ++i) all += columns(shapes[i]);
  for (int i = 0; i < n; ++i) {
    const int64_t N = shapes[i].N, cols = columns(shapes[i]);
    out[i] = choose_split(T, K, N, cols, 0, pf::kMaxSplits, area_floats);
    if (N >= K && out[i].parts == 2) out[i] = choose_split(T, K, N, cols, N >= 2 * K ? 2 : 1, 2, area_floats);
    if (n > 1 && out[i].parts > 2) out[i] = choose_split(T, K, N, all, 0, out[i].parts, area_floats / n);
  }
}

// ---- the launch that adds the arrays of a matrix that is cut along K ----
static_assert(pf::kMaxSplits <= kMaxKSplit, "arrays that it takes");
__global__ __launch_bounds__(256) void fold_kernel(const Fold f) {
  const int j = blockIdx.y;
  float* __restrict__ Y = f.Y[j];
  const float* __restrict__ array = f.array[j];
  const int64_t n = f.n[j], at = (int64_t)blockIdx.x * 256 + threadIdx.x, step = (int64_t)gridDim.x * 256;
  const int extra = f.arrays[j] - 1;
  if (extra <= 0) return;
  const bool wide = (reinterpret_cast<uintptr_t>(Y) & 15) == 0;  // (the arrays of the workspace always are)
  const int64_t n4 = wide ? n >> 2 : 0;
  for (int64_t i = at; i < n4; i += step) {
    floatx4 v[kMaxKSplit];  // all on their way before the first is used
    v[0] = reinterpret_cast<const floatx4*>(Y)[i];
#pragma unroll
    for (int e = 1; e < kMaxKSplit; ++e)
      if (e <= extra) v[e] = reinterpret_cast<const floatx4*>(array + (e - 1) * f.array_floats[j])[i];
#pragma unroll
    for (int e = 1; e < kMaxKSplit; ++e)
      if (e <= extra) v[0] += v[e];
    reinterpret_cast<floatx4*>(Y)[i] = v[0];
  }
  for (int64_t i = 4 * n4 + at; i < n; i += step) {
    float v = Y[i];
    for (int e = 0; e < extra; ++e) v += array[e * f.array_floats[j] + i];
    Y[i] = v;
  }
}

mbq_status launch_fold(const Fold& f, int n, hipStream_t stream) {
  int64_t most = 0;
  for (int i = 0; i < n; ++i)
    if (f.arrays[i] > 1 && f.n[i] > most) most = f.n[i];
  if (most == 0) return MBQ_OK;
  int64_t blocks = (most / 4 + 255) / 256;  // four floats a thread and pass
  if (blocks < 1) blocks = 1;
  if (blocks > 8 * device_compute_units()) blocks = 8 * device_compute_units();
  hipLaunchKernelGGL(fold_kernel, dim3((unsigned)blocks, (unsigned)n), dim3(256), 0, stream, f);
  return hip_status(hipGetLastError(), "fold_kernel launch");
}

// offsets of rows are 32-bit: from 4 GiB of activations on a sorted copy is made, one matrix at a time
static bool prefill_gathers(int64_t T, int64_t K) { return (uint64_t)T * (uint64_t)K * 2u <= 0xFFFFFFFFull; }
static float* prefill_sums(void* ws, int64_t T, int64_t K) {
  return reinterpret_cast<float*>(reinterpret_cast<char*>(ws) + prefill_copy_bytes(T, K));
}
// the cuts of a call's matrices, and what its pre-kernel clears: outputs, arrays of the workspace that two parts add into
static void prefill_cuts(int64_t T, int n, const Shape* shapes, float* const* Y, void* ws, Split* split, ZeroList* zl,
                         ZeroList* zs) {
  const int64_t K = shapes[0].K;
  // without a sorted copy its room takes arrays of partial sums
  const int64_t area = prefill_gathers(T, K) ? (int64_t)(prefill_copy_bytes(T, K) / sizeof(float)) : 0;
  choose_splits(T, K, n, shapes, area, split);
  float* slot = reinterpret_cast<float*>(ws);
  for (int i = 0; i < MBQ_MAX_GROUP; ++i) {
    const int j = i < n ? i : 0;
    const int64_t floats = slot_floats(T, shapes[j].N);
    const int twice = split[j].parts - split[j].slots;  // arrays with two parts: the first ones
    zl->p[i] = (i < n && twice > 0) ? Y[j] : nullptr;
    zl->n[i] = (i < n && twice > 0) ? (long long)T * shapes[j].N : 0;
    zs->p[i] = (i < n && twice > 1) ? slot : nullptr;
    zs->n[i] = (i < n && twice > 1) ? (long long)((twice - 1) * floats) : 0;
    if (i < n) slot += (split[j].slots - 1) * floats;
  }
}
bool prefill_prep_of(const uint16_t* X, int64_t T, int n, const Shape* shapes, float* const* Y, void* ws, PrefillPrep* prep) {
  if (!prefill_gathers(T, shapes[0].K)) return false;
  Split split[MBQ_MAX_GROUP];
  prep->X = X;
  prep->Sx = prefill_sums(ws, T, shapes[0].K);
  prefill_cuts(T, n, shapes, Y, ws, split, &prep->zl, &prep->zs);
  return true;
}

// The matrices share X; one launch for all of them, so that a stage has one ragged end.
mbq_status launch_linear_prefill_group(const uint16_t* X, int64_t T, int n, const void* const* blobs, const Shape* shapes,
                                       const int32_t* const* perm, const int32_t* const* offsets, float* const* Y, void* ws,
                                       hipStream_t stream, bool prepared) {
  const int64_t K = shapes[0].K;
  const bool gather = prefill_gathers(T, K);
  uint16_t* Xs = reinterpret_cast<uint16_t*>(ws);
  if (!gather && n > 1) {
    for (int i = 0; i < n; ++i) {
      mbq_status st = launch_linear_prefill_group(X, T, 1, blobs + i, shapes + i, perm + i, offsets + i, Y + i, ws, stream);
      if (st != MBQ_OK) return st;
    }
    return MBQ_OK;
  }
  Split split[MBQ_MAX_GROUP];
  PrefillPrep prep;
  prep.X = X;
  prep.Sx = prefill_sums(ws, T, K);
  prefill_cuts(T, n, shapes, Y, ws, split, &prep.zl, &prep.zs);
  const int64_t m_tiles_max = T / pf::kBM + MBQ_N_PRECISIONS;
  pf::Group g;
  Fold fold;
  int64_t blocks = 0;
  float* slot = reinterpret_cast<float*>(ws);
  for (int i = 0; i < MBQ_MAX_GROUP; ++i) {
    const int j = i < n ? i : 0;
    const Shape& sh = shapes[j];
    const Split sp = split[j];
    const int64_t floats = slot_floats(T, sh.N);
    pf::Proj& m = g.p[i];
    m.codes = reinterpret_cast<const uint32_t*>(blobs[j]);
    m.slice_words = sh.slice_words;
    m.meta = reinterpret_cast<const float2*>(reinterpret_cast<const char*>(blobs[j]) + sh.meta_offset);
    m.perm = perm[j];
    m.offsets = offsets[j];
    m.Y = Y[j];
    m.N = sh.N;
    m.slot = slot;
    m.slot_floats = floats;
    m.NT = sh.NT;
    m.cols = (int)((sh.N + pf::kBN - 1) / pf::kBN);
    m.splits = sp.parts;
    m.slots = sp.slots;
    m.block_begin = (int)blocks;
    fold.Y[i] = Y[j];
    fold.array[i] = slot;
    fold.array_floats[i] = floats;
    fold.n[i] = T * sh.N;
    fold.arrays[i] = i < n ? sp.slots : 1;
    if (i < n) {
      blocks += m_tiles_max * m.cols * sp.parts;
      slot += (sp.slots - 1) * floats;
    }
  }
  g.n = n;
  mbq_status st = MBQ_OK;
  if (!prepared || !gather) {
    hipLaunchKernelGGL(pf::prefill_prep_kernel, dim3((unsigned)T), dim3(256), 0, stream, prep, K, gather ? nullptr : perm[0],
                       gather ? nullptr : Xs);
    st = hip_status(hipGetLastError(), "prefill_prep_kernel launch");
    if (st != MBQ_OK) return st;
  }
  hipLaunchKernelGGL(pf::prefill_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, gather ? X : Xs, K, shapes[0].KB,
                     gather ? 1 : 0, prep.Sx, g);
  st = hip_status(hipGetLastError(), "prefill_kernel launch");
  return st == MBQ_OK ? launch_fold(fold, n, stream) : st;
}

mbq_status launch_linear_prefill(const uint16_t* X, int64_t T, const void* blob, const Shape& sh, const int32_t* perm,
                                 const int32_t* offsets, float* Y, void* ws, hipStream_t stream) {
  return launch_linear_prefill_group(X, T, 1, &blob, &sh, &perm, &offsets, &Y, ws, stream);
}

}  // namespace mbq
