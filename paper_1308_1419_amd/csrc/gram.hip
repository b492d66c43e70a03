// Gram-form EDM on the MFMA units (gfx950), packed output.
//
//   D_ij^2 = ||x_i||^2 + ||x_j||^2 - 2 x_i . x_j
//
// A prologue rounds X to BF16 (round to nearest even), pads the features to
// a multiple of 16 with zeros and the points to a multiple of 256, and
// computes the squared norms of the rounded points in FP32.  The products
// are taken by v_mfma_f32_32x32x16_bf16 on 32 x 32 output blocks (BF16
// products are exact in FP32, the sums accumulate in FP32).  The epilogue
// forms G = n_i + n_j - 2 acc and, when G <= theta (n_i + n_j) (theta =
// 1/4: the pair is close relative to its norms, where the Gram form
// cancels), recomputes the distance exactly in FP32 difference form from the
// FP32 points; otherwise it stores sqrt(G).
//
// Two kernels walk the triangle by g(lambda) (Sec. II-A, Eq. (2)) and
// compute every 32 x 32 block with the same instructions in the same order,
// so their outputs are equal bit for bit:
//   - gram_block_kernel: eight waves on 128 x 256 cells, each wave 64 x 64,
//     so an operand byte read from LDS feeds twice the products of a 32 x 32
//     wave block;
//   - gram_strip_kernel: eight waves on a 32-row strip of a 256 x 256 tile,
//     the strips of a tile row taken strip by strip across the row (the
//     order of the FP32 strips), so that the writes in flight stay in a
//     compact window of the packed output and small N makes more
//     work-groups.
// Measured (us, blocks / strips, prologue included, launches back to back on
// one box, the larger outputs 5 to 10 % more on others): N = 100000, d = 64
// 4052 / 3665 (BF16), 4300 / 4772 (split); N = 50000, d = 256 1390 / 1886; N =
// 30011, d = 200 split 739 / 853; N = 2000, d = 100 15.8 / 10.7.  The autotuner
// times both.  With row-major operands, staged through LDS in the strips and
// loaded by every lane on its own in 128 x 128 tiles, the same sizes took, in
// the faster of the two and on the same box, 3973, 6271, 2833, 1858 and 15.0 us.
//
// Split mode (precision BF16X3): each point is held as x = hi + lo with
// hi = bf16(x) and lo = bf16(x - hi) (x - hi is exact in FP32, and hi + lo
// is exact in FP32), the norms are those of hi + lo, and the dot product is
// hi.hi' + hi.lo' + lo.hi', three MFMA products into the same FP32
// accumulator; only lo.lo' (below 2^-16 of |x||y|) is dropped.
#include <type_traits>

#include "device.h"
#include "kernels.h"

namespace tdmap {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kGramPad = 256;   // operand rows are padded to this
constexpr float kGramTheta = 0.25f;

__device__ __forceinline__ uint16_t bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// The operands sit in memory as the MFMA instruction takes them.  A fragment
// holds 32 points x 16 features, 1 KB: lane l = p mod 32 + 32 h of the wave
// that multiplies it finds the features 8 h .. 8 h + 7 of point p at
// 16-byte chunk l.  Fragment (p / 32, k / 16) is number (p / 32) KS + k / 16
// (KS = KP / 16), so a wave loads one with a single 1 KB contiguous
// instruction, into registers or LDS alike, and reads it back from LDS
// without bank conflicts.
constexpr int kFragElems = 512;

// The BF16 copy (zero padded) and the squared norms of the represented
// points; with Xlo != nullptr also the low parts.  A work-group takes 32
// points: thread t converts the 8-feature chunks t / 32, t / 32 + 8, ... of
// point t mod 32 and writes each as one 16-byte store (a wave writes two
// chunks of 32 points, 1 KB).  VEC: whole chunks are read as two 16-byte
// loads.  The chunk sums of a point are kept by chunk modulo 256 and added
// in that order.
template <bool VEC>
__global__ __launch_bounds__(256) void gram_prologue_kernel(const float *__restrict__ X, int64_t N, int d,
                                                            int64_t ldx, uint16_t *__restrict__ Xb,
                                                            uint16_t *__restrict__ Xlo,
                                                            float *__restrict__ nrm, int KP) {
  typedef uint32_t u4 __attribute__((ext_vector_type(4)));
  extern __shared__ float part[];  // [min(KP / 8, 256)][32]
  const int cpp = KP >> 3;
  const int t = threadIdx.x;
  const int pl = t & 31;
  const int64_t p = (int64_t)blockIdx.x * 32 + pl;
  const float *__restrict__ x = X + p * ldx;
  uint16_t *__restrict__ hi = Xb + (int64_t)blockIdx.x * (KP >> 4) * kFragElems + pl * 8;
  uint16_t *__restrict__ lp =
      Xlo != nullptr ? Xlo + (int64_t)blockIdx.x * (KP >> 4) * kFragElems + pl * 8 : nullptr;
  for (int c = t >> 5; c < cpp; c += 8) {
    float v[8];
    if (VEC && p < N && 8 * c + 8 <= d) {
      const f4 q0 = *reinterpret_cast<const f4 *>(x + 8 * c);
      const f4 q1 = *reinterpret_cast<const f4 *>(x + 8 * c + 4);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        v[u] = q0[u];
        v[4 + u] = q1[u];
      }
    } else {
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = (p < N && 8 * c + u < d) ? x[8 * c + u] : 0.0f;
    }
    uint16_t hb[8], lb[8];
    const int slot = (c & 255) * 32 + pl;
    float s = c < 256 ? 0.0f : part[slot];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      hb[u] = bf16_rne(v[u]);
      float r = bf16_to_f32(hb[u]);
      if (Xlo != nullptr) {
        lb[u] = bf16_rne(v[u] - r);
        r += bf16_to_f32(lb[u]);
      }
      s = __builtin_fmaf(r, r, s);
    }
    part[slot] = s;
    u4 h, lo;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      h[e] = (uint32_t)hb[2 * e] | ((uint32_t)hb[2 * e + 1] << 16);
      lo[e] = (uint32_t)lb[2 * e] | ((uint32_t)lb[2 * e + 1] << 16);
    }
    // chunk c: half c mod 2 of fragment c / 2
    const int64_t at = (int64_t)(c >> 1) * kFragElems + (c & 1) * 256;
    *reinterpret_cast<u4 *>(hi + at) = h;
    if (Xlo != nullptr) *reinterpret_cast<u4 *>(lp + at) = lo;
  }
  __syncthreads();
  if (t < 32) {
    float n = 0.0f;
    const int m = cpp < 256 ? cpp : 256;
    for (int c = 0; c < m; ++c) n += part[c * 32 + t];
    nrm[p] = n;
  }
}

// FP32 difference form with eight interleaved partial sums combined as a
// tree, which keeps the rounding error of the squared distance near
// (d/8 + 6) units of roundoff.  Eight consecutive lanes take one pair: lane u
// of them sums the features u, u + 8, ..., so that a group's loads are 32
// consecutive bytes of each point, and the tree runs over lane moves; every
// lane of the group receives the distance.
__device__ __forceinline__ float exact_dist8(const float *__restrict__ X, int64_t ldx, int d, int64_t i,
                                             int64_t j) {
  const int u = threadIdx.x & 7;
  const float *xi = X + i * ldx;
  const float *xj = X + j * ldx;
  float s = 0.0f;
#pragma unroll 4
  for (int k = u; k < d; k += 8) {
    const float t = xi[k] - xj[k];
    s = __builtin_fmaf(t, t, s);
  }
  auto move = [](float v, auto ctrl) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v),
                                                                 decltype(ctrl)::value, 0xF,
                                                                 0xF, true));
  };
  s += move(s, std::integral_constant<int, 0xB1>());   // quad_perm [1,0,3,2]: 0+1, 2+3, ...
  s += move(s, std::integral_constant<int, 0x4E>());   // quad_perm [2,3,0,1]: (0+1)+(2+3), ...
  s += move(s, std::integral_constant<int, 0x141>());  // row_half_mirror: the other four
  return __builtin_amdgcn_sqrtf(s);
}

// Accumulator v of a 32 x 32 block holds row (v/4)*8 + (l/32)*4 + v%4 of
// the block and column l % 32.
__device__ __forceinline__ int acc_row(int v, int l) { return (v >> 2) * 8 + (l >> 5) * 4 + (v & 3); }

// The epilogue of one pair from its accumulator and the two squared norms:
// G (or sqrt(G)), and the lane's bit of `low` set for a pair to be recomputed (its
// square root, possibly of a negative G, is replaced then).
__device__ __forceinline__ float gram_square(float acc, float ni, float nj, uint64_t &low) {
  const float sn = ni + nj;
  const float G = __builtin_fmaf(-2.0f, acc, sn);
  low |= __builtin_amdgcn_ballot_w64(G <= kGramTheta * sn);
  return G;
}
__device__ __forceinline__ float gram_value(float acc, float ni, float nj, uint64_t &low) {
  return __builtin_amdgcn_sqrtf(gram_square(acc, ni, nj, low));
}
// Whether it is one of those.
__device__ __forceinline__ bool gram_close(float acc, float ni, float nj) {
  const float sn = ni + nj;
  return __builtin_fmaf(-2.0f, acc, sn) <= kGramTheta * sn;
}

// Pairs of a wave to be recomputed, as they are found: positions (row * 256 +
// column) in the wave's part of the staged output.  Recomputed lane by lane a
// wave waits for a pair's loads once per accumulator in which some lane has
// one (N = 60000, d = 10 BF16, where one pair in 170 is recomputed: 2540 us;
// 1425 with the list); the list spreads the pairs over the wave, eight lanes
// a pair.
constexpr int kListLen = 128;  // 63 left over and the 64 of one step

// Recomputes the first n pairs of the list (cells of the triangle, j < i):
// at(pos) is the staged position, i0 and j0 the pair of position 0.
template <bool COUNT, typename At>
__device__ __forceinline__ void recompute_pairs(const GramArgs &a, const uint16_t *list, int n, int64_t i0,
                                                int64_t j0, At at, uint32_t &nrec) {
  const int l = threadIdx.x & 63;
  for (int e0 = 0; e0 < n; e0 += 8) {
    const int e = e0 + (l >> 3);
    if (e < n) {
      const int pos = list[e];
      const float v = exact_dist8(a.X, a.ldx, a.d, i0 + (pos >> 8), j0 + (pos & 255));
      if ((l & 7) == 0) {
        if (COUNT) ++nrec;
        *at(pos) = v;
      }
    }
  }
}

// Recomputes a wave's close pairs where they are, for up to F features (feature
// k belongs to partial sum k mod 8, as in exact_dist8): bit m of the mask as in
// recompute_close, a column of pairs to 16 bits.  A lane keeps its column's
// point, and the row points are the same in each half of the wave, so a step
// loads two points' rows for up to 64 pairs where the list's eight lanes a pair
// load 16 for 8; but every step with a pair in some lane is taken.  In place /
// from the list / (before the list) lane by lane without a kept point, N =
// 12000, strips, us: N(3, 1), where 86 to 100 % of the pairs are close, d = 1
// 96 / 472 / 121, 4 127 / 507 / 303, 9 117 / 585 / 561, 16 248 / 594 / 2125; N(0, 1),
// 23, 4 and 0.6 %, d = 1 96 / 175 / 121, 4 120 / 81 / 142, 8 104 / 58 / 125.  Hence
// the line in the caller, by features and the fullest lane's pairs.  With 32
// features a lane's point costs spills (d = 32, half the pairs close: 737 against
// 548 from the list).  There the list stays, slower than lane by lane only where
// nearly every pair is close and the pitch odd (d = 33 2664 against 2409 in the
// faster kernel; d = 17, N = 513 53 against 42), at even pitches several times
// as fast (d = 64 1522, 8638).
template <bool COUNT, int BITS, int F, typename Pos, typename At>
__device__ __forceinline__ void recompute_in_place(const GramArgs &a, uint32_t mask, int64_t i0, int64_t j0,
                                                   Pos pos, At at, uint32_t &nrec) {
  const int d = a.d;
  float xj[F];
#pragma unroll 1
  for (int m = 0; m < BITS; ++m) {
    const int p = pos(m);
    if (m % 16 == 0 && (mask >> m & 0xffffu) != 0) {
      const float *x = a.X + (j0 + (p & 255)) * a.ldx;
#pragma unroll
      for (int k = 0; k < F; ++k)
        if (k < d) xj[k] = x[k];
    }
    if ((mask >> m & 1u) == 0) continue;
    const float *x = a.X + (i0 + (p >> 8)) * a.ldx;
    float s[8] = {};
#pragma unroll
    for (int k = 0; k < F; ++k)
      if (k < d) {
        const float t = x[k] - xj[k];
        s[k % 8] = __builtin_fmaf(t, t, s[k % 8]);
      }
    if (COUNT) ++nrec;
    *at(p) = __builtin_amdgcn_sqrtf(((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7])));
  }
}

// Recomputes a wave's close pairs: bit m of a lane's mask is its pair at
// position pos(m).  A point with itself, most of the recomputed cells, is
// exactly 0 and needs no loads; a cell outside the triangle is not stored and
// set to 0 (both only in blocks that touch the diagonal or the last point,
// `edge`).  The lanes then hand in one pair each per step, as many steps as
// the fullest lane has pairs.
template <bool COUNT, int BITS, bool FEW, typename Pos, typename At>
__device__ __forceinline__ void recompute_close(const GramArgs &a, uint16_t *list, uint32_t mask, bool edge,
                                                int64_t i0, int64_t j0, Pos pos, At at, uint32_t &nrec) {
  const int l = threadIdx.x & 63;
  if (edge) {
    uint32_t pairs = 0;
#pragma unroll
    for (int m = 0; m < BITS; ++m) {
      const int p = pos(m);
      const int64_t i = i0 + (p >> 8), j = j0 + (p & 255);
      pairs |= (uint32_t)(i < a.N && j < i) << m;
    }
    uint32_t other = mask & ~pairs;
    mask &= pairs;
    while (other != 0) {
      const int p = pos(__builtin_ctz(other));
      other &= other - 1;
      if (COUNT) nrec += i0 + (p >> 8) < a.N && i0 + (p >> 8) == j0 + (p & 255);
      *at(p) = 0.0f;
    }
  }
  // few features and many pairs (in the fullest lane)
  if constexpr (FEW) {
    const int many = a.d < 12 ? 4 + 5 * a.d / 8 : 11;
    if (a.d <= 16 && __builtin_amdgcn_ballot_w64(__builtin_popcount(mask) > many * (BITS / 16)) != 0) {
      if (a.d <= 8)
        recompute_in_place<COUNT, BITS, 8>(a, mask, i0, j0, pos, at, nrec);
      else
        recompute_in_place<COUNT, BITS, 16>(a, mask, i0, j0, pos, at, nrec);
      return;
    }
  }
  int count = 0;  // list entries, the same in every lane
  for (;;) {
    const uint64_t have = __builtin_amdgcn_ballot_w64(mask != 0);
    if (have == 0) break;
    if (mask != 0) {
      list[count + __builtin_amdgcn_mbcnt_hi((uint32_t)(have >> 32),
                                             __builtin_amdgcn_mbcnt_lo((uint32_t)have, 0))] =
          (uint16_t)pos(__builtin_ctz(mask));
      mask &= mask - 1;
    }
    count += __builtin_popcountll(have);
    __builtin_amdgcn_wave_barrier();  // the wave reads its own LDS writes
    if (count >= 64) {
      recompute_pairs<COUNT>(a, list, 64, i0, j0, at, nrec);
      count -= 64;
      __builtin_amdgcn_wave_barrier();
      const uint16_t rest = list[64 + l];
      __builtin_amdgcn_wave_barrier();
      list[l] = rest;
      __builtin_amdgcn_wave_barrier();
    }
  }
  recompute_pairs<COUNT>(a, list, count, i0, j0, at, nrec);
}

// One 1 KB fragment from global memory straight into LDS: lane l's 16 bytes
// land at dst + 16 l.
__device__ __forceinline__ void load_fragment(const uint16_t *src, unsigned char *dst) {
  __builtin_amdgcn_global_load_lds(
      (const __attribute__((address_space(1))) void *)(src + (threadIdx.x & 63) * 8),
      (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
}

// Lane l's part of fragment f of an LDS area.
__device__ __forceinline__ bf16x8 lds_fragment(const unsigned char *ops, int f) {
  return *reinterpret_cast<const bf16x8 *>(ops + f * 1024 + (threadIdx.x & 63) * 16);
}

// One k-step of a 32 x 32 block; split: lo.hi', hi.lo', hi.hi' in that
// order.  Steps run in increasing feature order in every kernel, so a block
// has the same bits wherever it is computed.
template <bool SPLIT>
__device__ __forceinline__ f32x16 gram_step(f32x16 acc, bf16x8 ah, bf16x8 al, bf16x8 bh, bf16x8 bl) {
  if constexpr (SPLIT) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl, acc, 0, 0, 0);
  }
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh, acc, 0, 0, 0);
}

// ---------------------------------------------------------------------------
// block kernel: eight waves, 128 x 256 cells
// ---------------------------------------------------------------------------

// Eight waves as 2 x 4, each on 64 x 64 cells (2 x 2 MFMA blocks).  Stage s
// holds the fragments of the work-group's 12 point blocks for two k-steps
// (split: the high and low parts of one), 24 KB, loaded straight into LDS:
// three buffers, one barrier a stage, two work-groups per CU.  The loads are
// issued two stages ahead, but the compiler, which cannot tell the buffers
// apart, waits for all of them in front of a stage's first LDS read, so they
// have one stage of products to land in.  (Three arrays, without that wait: 711
// against 697 us, N = 30011, d = 200 split.)  Three buffers start with two
// stages in flight; two, and loads one stage ahead: 755 against 729 us there,
// 1552 against 1478 at N = 50000, d = 256, but 4836 against 4902 at N = 100000,
// d = 64 split, where a block has four stages.
constexpr int kBlkRows = 128;
constexpr int kBlkFrags = 2 * (kBlkRows / 32 + 8);  // per stage
constexpr int kBlkStage = kBlkFrags * 1024;
constexpr int kBlkLoads = kBlkFrags / 8;            // per wave and stage
static_assert(8 * 32 * 64 * 4 <= 3 * kBlkStage, "the staged output overlays the operands");

template <bool SPLIT, bool COUNT>
__global__ __launch_bounds__(512, 4) void gram_block_kernel(GramArgs a, uint32_t w0, uint32_t nblk) {
  __shared__ __align__(16) unsigned char ops[3 * kBlkStage];
  __shared__ uint16_t list[8][kListLen];
  __shared__ float nrow[kBlkRows];
  const uint32_t w = w0 + xcd_contiguous(blockIdx.x, nblk);
  // g places 256 x 256 tiles, the two 128-row halves of a tile inner: its
  // column points then serve 256 rows from L2 (N = 50000, d = 256: 1704 us
  // against 1741 with the upper halves of a tile row before the lower ones and
  // 1777 with 512 x 512 squares, four bands inner)
  uint32_t I2, J;
  g_lambda_uniform(w >> 1, I2, J);
  const int64_t N = a.N;
  const int64_t r0 = (int64_t)I2 * 256 + (w & 1) * kBlkRows;
  const int64_t c0 = (int64_t)J * 256;
  if (r0 >= N) return;  // uniform
  const int q = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l = threadIdx.x & 63;
  const int lr = l & 31;
  const int KS = a.KP >> 4;
  const int wr = q >> 2, wc = q & 3;
  const int64_t cw = c0 + 64 * wc;
  const int stages = SPLIT ? KS : (KS + 1) >> 1;
  // the norms, loaded ahead of the operands: nothing waits for them later
  float nc[2];
#pragma unroll
  for (int y = 0; y < 2; ++y) nc[y] = a.nrm[cw + 32 * y + lr];
  if (threadIdx.x < kBlkRows) nrow[threadIdx.x] = a.nrm[r0 + threadIdx.x];

  // fragment f of a stage: point block f / 2 (rows first), f odd: the second
  // k-step (absent when KS is odd and the stage the last) or the low part
  auto load_stage = [&](int s) {
    unsigned char *buf = ops + (s % 3) * kBlkStage;
#pragma unroll
    for (int m = 0; m < kBlkLoads; ++m) {
      const int f = q + 8 * m;
      const int pb = f >> 1, odd = f & 1;
      const int64_t g = pb < kBlkRows / 32 ? (r0 >> 5) + pb : (c0 >> 5) + (pb - kBlkRows / 32);
      const uint16_t *src = (SPLIT && odd) ? a.Xlo : a.Xb;
      int ks = SPLIT ? s : 2 * s + odd;
      ks = ks < KS ? ks : KS - 1;  // (loaded, not used)
      load_fragment(src + (g * KS + ks) * kFragElems, buf + f * 1024);
    }
  };
  f32x16 acc[2][2];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[x][y][v] = 0.0f;

  load_stage(0);
  if (stages > 1) load_stage(1);
  for (int s = 0; s < stages; ++s) {
    // this wave's share of stage s has landed (the loads complete in order) and
    // its reads of stage s - 1 have returned
    if (s + 1 < stages)
      __builtin_amdgcn_s_waitcnt(0x0070 | kBlkLoads);  // vmcnt(kBlkLoads) lgkmcnt(0)
    else
      __builtin_amdgcn_s_waitcnt(0x0070);
    // ... and every wave's (no fence: it would wait for the loads in flight; the
    // empty asm keeps the LDS reads below)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    const unsigned char *buf = ops + (s % 3) * kBlkStage;
    bf16x8 av[2][2], bv[2][2];  // [block][k-step or part]
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        av[x][h] = lds_fragment(buf, 2 * (2 * wr + x) + h);
        bv[x][h] = lds_fragment(buf, 2 * (kBlkRows / 32 + 2 * wc + x) + h);
      }
    // (behind the LDS reads in the queues they share: 732 us against 750 with
    // N = 30011, d = 200 split)
    if (s + 2 < stages) load_stage(s + 2);
    if constexpr (SPLIT) {
#pragma unroll
      for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int y = 0; y < 2; ++y)
            acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[x][p == 0], bv[y][p == 1], acc[x][y],
                                                                0, 0, 0);
    } else {
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (2 * s + h < KS)
#pragma unroll
          for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y)
              acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[x][h], bv[y][h], acc[x][y], 0, 0, 0);
    }
  }
  __syncthreads();  // the operands are read

  // Output, 32 rows x 64 columns at a time, in whole rows of 64 cells (256
  // contiguous bytes per store).  Accumulator v of the two column blocks holds
  // the halves of rows R and R + 4: one swap of wave halves makes each a row of
  // 64 columns, stored from the register.  Blocks with pairs to recompute, at
  // the diagonal or past the last point go through the wave's own 8 KB of LDS
  // instead (when all of them did: 788 us against 750, same case; LDS feeds
  // the products too).
  float *st = reinterpret_cast<float *>(ops) + q * 32 * 64;
  uint32_t nrec = 0;
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    const int64_t rw = r0 + 64 * wr + 32 * x;
    if (rw >= N || cw > rw + 31) continue;  // no cell of the triangle (uniform)
    const bool edge = cw + 63 > rw || rw + 32 > N;
    uint64_t low = 0;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const float ni = nrow[64 * wr + 32 * x + acc_row(v, l)];
#pragma unroll
      for (int y = 0; y < 2; ++y) {
        const float e = acc[x][y][v];  // (copied out: a bit cast of a vector element is avoided)
        acc[x][y][v] = gram_square(e, ni, nc[y], low);
      }
    }
    // row rw + r starts at T(rw) + r rw + r (r + 1) / 2
    float *__restrict__ o = a.D + tri64((uint64_t)rw) + (uint64_t)cw;
    const uint32_t rwu = (uint32_t)rw;
    if (low == 0 && !edge) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const float e0 = acc[x][0][v], e1 = acc[x][1][v];
        const auto w2 = __builtin_amdgcn_permlane32_swap(
            __builtin_bit_cast(uint32_t, __builtin_amdgcn_sqrtf(e0)),
            __builtin_bit_cast(uint32_t, __builtin_amdgcn_sqrtf(e1)), false, false);
        const uint32_t b0 = w2[0], b1 = w2[1];
        const uint32_t r = (v >> 2) * 8 + (v & 3);
        (o + r * rwu + ((r * (r + 1)) >> 1))[l] = __builtin_bit_cast(float, b0);
        (o + (r + 4) * rwu + (((r + 4) * (r + 5)) >> 1))[l] = __builtin_bit_cast(float, b1);
      }
      continue;
    }
    uint32_t mask = 0;
#pragma unroll
    for (int m = 0; m < 32; ++m) {
      const int rr = acc_row(m & 15, l);
      const float G = acc[x][m >> 4][m & 15];
      mask |= (uint32_t)(G <= kGramTheta * (nrow[64 * wr + 32 * x + rr] + nc[m >> 4])) << m;
      st[rr * 64 + 32 * (m >> 4) + lr] = __builtin_amdgcn_sqrtf(G);
    }
    if (low != 0)
      recompute_close<COUNT, 32, true>(
          a, list[q], mask, edge, rw, cw, [&](int m) { return acc_row(m & 15, l) * 256 + 32 * (m >> 4) + lr; },
          [&](int p) { return st + (p >> 8) * 64 + (p & 255); }, nrec);
    __builtin_amdgcn_wave_barrier();  // the wave reads its own LDS writes
    for (uint32_t r = 0; r < 32; ++r)
      if (rw + r < N && cw + l <= rw + r) (o + r * rwu + ((r * (r + 1)) >> 1))[l] = st[r * 64 + l];
    __builtin_amdgcn_wave_barrier();
  }
  if (COUNT && nrec) atomicAdd(a.rec_count, (unsigned long long)nrec);
}

// ---------------------------------------------------------------------------
// strip kernel: eight waves, one 32-row strip of a 256 x 256 tile
// ---------------------------------------------------------------------------

// Tile row I (256 rows) is cut into kStripsPerTile strips of 32 rows and a
// work-group computes one strip of one tile, 32 x 256 cells.  What bounds it
// is the write stream (N = 100000, d = 64 BF16, tiles in groups of eight: 4.4
// ms, without the products 4.0, without the stores 1.45; 3.9 in bands), and
// with it the order in which the strips of a tile row are taken,
// u = 0 .. 8 (I + 1) - 1:
//   - up to 64 features (split: 32): two bands of kStripBand strips, swept
//     across the tile row with the strip inner, so that a band's rows are
//     written end to end, and three work-groups per CU for large outputs (the
//     fewer bytes being written at a time, the better: 4.16 ms with four; at two
//     the loads are no longer hidden, 4.34; kStripIdle).  N = 100000, d = 40:
//     3856 us, 4355 in column groups; N = 20000 159 and 182;
//   - more: column groups of kStripGroup tiles, group outer, strip next, tile
//     inner: a group's column points then stay in L2 across its 8 strips,
//     which the wider operands need more (d = 64 split: 5.05 ms, 5.25 in
//     bands, 5.4 with three work-groups per CU).
//
// Operands: wave q computes the 32 x 32 block of columns [32 q, 32 q + 32)
// and is the only one to use their fragments, so it loads those straight
// into registers; the fragments of the 32 row points, which all eight waves
// use, go to LDS, as many k-steps a pass as the area holds.  A work-group's
// loads are thus one round up to 256 features (split) or 512.
//
// Output: the distances of the strip are staged in LDS (over the operand
// area) and each wave writes whole packed rows q, q + 8, q + 16, q + 24:
// lane l owns columns l + 64 c and every 4-byte store instruction writes 256
// contiguous bytes.  The LDS footprint (33 KB) leaves four work-groups per
// CU.
constexpr int kStripRows = 32;
constexpr int kStripsPerTile = 256 / kStripRows;
constexpr int kStripWaves = 8;
constexpr int kStripPitch = 260;  // floats per staged output row
constexpr int kStripBytes = kStripRows * kStripPitch * 4;
constexpr int kStripFrags = kStripBytes / 1024;  // fragments that fit the area
constexpr uint32_t kStripGroup = 8;
constexpr uint32_t kStripBand = 4;
// (KPC: the padded feature count of an instance; those up to 64 all have one)
template <bool SPLIT, int KPC>
constexpr bool kStripBands = KPC != 0 && KPC * (SPLIT ? 2 : 1) <= 64;
// Three work-groups per CU instead of four, by dynamic LDS that no thread uses:
// in bands with more than 16 features (parts counted), for outputs from 64 MB
// on.  Three / four, us: d = 64 BF16 N = 3500 13.3 / 11.7, 4096 14.0 / 14.9,
// 5300 17.8 / 16.9, 5793 18.8 / 19.7, 8192 29.4 / 30.5, 11585 56.7 / 55.6, 16384
// 111 / 118, 46000 797 / 862; d = 32 split 5793 19.5 / 20.4, 46000 800 / 849; d =
// 16 split 8192 28.8 / 27.3, 16384 113 / 120, 46000 889 / 897.  A single step of
// 16 features loads too little to be hidden by fewer: d = 8 BF16 5793 19.7 /
// 18.5, 11585 53.1 / 48.0, 16384 107 / 110, 46000 809 / 801, 80000 2459 / 2423.
template <bool SPLIT, int KPC>
constexpr bool kStripIdle = kStripBands<SPLIT, KPC> && KPC * (SPLIT ? 2 : 1) > 16;
constexpr uint32_t kStripIdleLds = 16 * 1024;
constexpr uint64_t kStripSmall = (uint64_t)64 << 20;  // output bytes

template <bool BANDS>
__device__ __forceinline__ void strip_order(uint32_t w, uint32_t &I, uint32_t &k, uint32_t &J) {
  uint32_t Jt;
  g_lambda_uniform(w / kStripsPerTile, I, Jt);
  // u: this work-group's place among the 8 (I + 1) strips of tile row I
  const uint32_t u = kStripsPerTile * Jt + w % kStripsPerTile;
  if constexpr (BANDS) {
    uint32_t r;
    const uint32_t b = div_uniform(u, kStripBand * (I + 1), r);
    J = r / kStripBand;
    k = b * kStripBand + r % kStripBand;
    return;
  }
  constexpr uint32_t span = kStripGroup * kStripsPerTile;
  const uint32_t g = u / span, r = u % span;
  const uint32_t left = I + 1 - g * kStripGroup;  // tiles from this group on
  if (left >= kStripGroup) {
    k = r / kStripGroup;
    J = g * kStripGroup + r % kStripGroup;
  } else {  // the last, narrower group
    k = div_uniform(r, left, J);
    J += g * kStripGroup;
  }
}

template <bool SPLIT, int KPC, bool COUNT>
__global__ __launch_bounds__(kStripWaves * 64, 8) void gram_strip_kernel(GramArgs a, uint32_t w0,
                                                                         uint32_t nblk) {
  __shared__ __align__(16) unsigned char ops[kStripBytes];
  __shared__ float nrow[kStripRows];
  __shared__ uint16_t list[kStripWaves][kListLen];
  float *st = reinterpret_cast<float *>(ops);  // after the products
  const uint32_t w = w0 + xcd_contiguous(blockIdx.x, nblk);
  uint32_t I, k, J;
  strip_order<kStripBands<SPLIT, KPC>>(w, I, k, J);
  const int64_t N = a.N;
  const int64_t r0 = (int64_t)I * 256 + (int64_t)k * kStripRows;
  if (r0 >= N) return;  // a strip past the last point (uniform)
  const int64_t c0 = (int64_t)J * 256;
  const bool diag = I == J;
  const int t = threadIdx.x;
  const int q = __builtin_amdgcn_readfirstlane(t >> 6);
  const int l = t & 63;
  const int lr = l & 31;
  const int KS = (KPC ? KPC : a.KP) >> 4;
  if (t < kStripRows) nrow[t] = a.nrm[r0 + t];
  const float ncol = a.nrm[c0 + 32 * q + lr];

  constexpr int PARTS = SPLIT ? 2 : 1;
  constexpr int KA = kStripFrags / PARTS / 4 * 4;  // k-steps per pass
  constexpr int CH = SPLIT && KPC == 0 ? 2 : 4;      // k-steps loaded together (64 VGPRs)
  static_assert(KA >= CH, "a pass holds a chunk");
  const int64_t ra = (r0 >> 5) * KS;
  const int64_t rb = ((c0 >> 5) + q) * KS;
  const uint16_t *__restrict__ Bh = a.Xb + rb * kFragElems + l * 8;
  const uint16_t *__restrict__ Bl = SPLIT ? a.Xlo + rb * kFragElems + l * 8 : nullptr;
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
  bf16x8 bh[CH], bl[CH];
  auto load_chunk = [&](int ks, int n) {
#pragma unroll
    for (int u = 0; u < CH; ++u)
      if (u < n) {
        bh[u] = *reinterpret_cast<const bf16x8 *>(Bh + (int64_t)(ks + u) * kFragElems);
        if constexpr (SPLIT) bl[u] = *reinterpret_cast<const bf16x8 *>(Bl + (int64_t)(ks + u) * kFragElems);
      }
  };
  for (int k0 = 0; k0 < KS; k0 += KA) {
    const int na = KS - k0 < KA ? KS - k0 : KA;
    if (k0 > 0) __syncthreads();  // the previous pass is read
    for (int f = q; f < na * PARTS; f += kStripWaves) {
      const int part = f >= na ? 1 : 0;
      load_fragment((SPLIT && part ? a.Xlo : a.Xb) + (ra + k0 + f - part * na) * kFragElems, ops + f * 1024);
    }
    load_chunk(k0, na);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the wave's fragments have landed
    __syncthreads();
    for (int ks = 0; ks < na; ks += CH) {
      const int n = na - ks < CH ? na - ks : CH;
      if (ks > 0) load_chunk(k0 + ks, n);
#pragma unroll
      for (int u = 0; u < CH; ++u)
        if (u < n) {
          const bf16x8 av = lds_fragment(ops, ks + u);
          bf16x8 al = av;
          if constexpr (SPLIT) al = lds_fragment(ops, na + ks + u);
          acc = gram_step<SPLIT>(acc, av, al, bh[u], SPLIT ? bl[u] : bh[u]);
        }
    }
  }
  __syncthreads();  // the operands are read: the output may overwrite them

  // epilogue: the wave's 32 x 32 block into the staged output
  const int col = 32 * q + lr;
  uint64_t low = 0;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int rr = acc_row(v, l);
    const float e = acc[v];  // (copied out: a bit cast of a vector element is avoided)
    st[rr * kStripPitch + col] = gram_value(e, nrow[rr], ncol, low);
  }
  uint32_t nrec = 0;
  if (low != 0) {
    uint32_t mask = 0;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const float e = acc[v];
      mask |= (uint32_t)gram_close(e, nrow[acc_row(v, l)], ncol) << v;
    }
    recompute_close<COUNT, 16, KPC == 16>(
        a, list[q], mask, diag || r0 + kStripRows > N, r0, c0 + 32 * q,
        [&](int v) { return acc_row(v, l) * 256 + lr; },
        [&](int p) { return st + (p >> 8) * kStripPitch + 32 * q + (p & 255); }, nrec);
  }
  if (COUNT && nrec) atomicAdd(a.rec_count, (unsigned long long)nrec);
  __syncthreads();

  // Strip row r starts at T(r0 + r) + c0 = T(r0) + c0 + r r0 + r(r+1)/2: a
  // uniform 64-bit base and a 32-bit offset (r r0 < 32 N).
  float *__restrict__ outb = a.D + tri64((uint64_t)r0) + (uint64_t)c0;
  const uint32_t r0u = (uint32_t)r0;
  auto row_off = [&](uint32_t r) { return r * r0u + ((r * (r + 1)) >> 1); };
  if (!diag && r0 + kStripRows <= N) {
#pragma unroll
    for (int m = 0; m < kStripRows / kStripWaves; ++m) {
      const int r = q + kStripWaves * m;
      float *o = outb + row_off(r);
#pragma unroll
      for (int c = 0; c < 4; ++c) o[l + 64 * c] = st[r * kStripPitch + l + 64 * c];
    }
  } else {
    // diagonal or edge strip: rows below N, cells with j <= i
    for (int m = 0; m < kStripRows / kStripWaves; ++m) {
      const int r = q + kStripWaves * m;
      const int64_t i = r0 + r;
      if (i >= N) break;
      const int64_t jmax = diag ? i - c0 : 255;
      float *o = outb + row_off(r);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int cc = l + 64 * c;
        if (cc <= jmax) o[cc] = st[r * kStripPitch + cc];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

template <bool SPLIT, int KPC, bool COUNT>
static void launch_strip_kernel(dim3 grid, hipStream_t stream, const GramArgs &a, uint32_t w0) {
  const uint64_t N = (uint64_t)a.N;
  const uint32_t lds = kStripIdle<SPLIT, KPC> && N * (N + 1) * 2 >= kStripSmall ? kStripIdleLds : 0;
  hipLaunchKernelGGL((gram_strip_kernel<SPLIT, KPC, COUNT>), grid, dim3(kStripWaves * 64), lds, stream, a, w0,
                     grid.x);
}

template <bool SPLIT, bool COUNT>
static void launch_gram_strips(int KP, dim3 grid, hipStream_t stream, const GramArgs &a, uint32_t w0) {
  switch (KP) {
    case 16: return launch_strip_kernel<SPLIT, 16, COUNT>(grid, stream, a, w0);
    case 32: return launch_strip_kernel<SPLIT, 32, COUNT>(grid, stream, a, w0);
    case 48: return launch_strip_kernel<SPLIT, 48, COUNT>(grid, stream, a, w0);
    case 64: return launch_strip_kernel<SPLIT, 64, COUNT>(grid, stream, a, w0);
    case 128: return launch_strip_kernel<SPLIT, 128, COUNT>(grid, stream, a, w0);
    default: return launch_strip_kernel<SPLIT, 0, COUNT>(grid, stream, a, w0);
  }
}

static int64_t gram_npad(int64_t N) { return (N + kGramPad - 1) / kGramPad * kGramPad; }

size_t gram_workspace_bytes(int64_t N, int d, bool split) {
  const int64_t KP = (d + 15) / 16 * 16;
  const int64_t Npad = gram_npad(N);
  return (size_t)Npad * (size_t)KP * 2 * (split ? 2 : 1) + (size_t)Npad * 4;
}

// Work-groups of the block kernel: two per 256 x 256 tile.
static uint64_t gram_blocks(int64_t N) {
  const uint64_t nb = (uint64_t)((N + 255) / 256);
  return nb * (nb + 1);
}

bool gram_supported(int64_t N, int ts) {
  if (ts == 128) return gram_blocks(N) <= 0xffffffffull;
  if (ts == 256) {
    const uint64_t nb = (uint64_t)((N + 255) / 256);
    return (uint64_t)kStripsPerTile * (nb * (nb + 1) / 2) <= 0xffffffffull;
  }
  return false;
}

template <bool COUNT>
static hipError_t launch_gram_t(const float *X, int64_t N, int d, int64_t ldx, float *D, void *ws,
                                bool split, int ts, unsigned long long *count, hipStream_t stream,
                                uint32_t shard = 0, uint32_t nshards = 1) {
  if (N == 0) return hipSuccess;
  const int64_t Npad = gram_npad(N);
  const int KP = (d + 15) / 16 * 16;
  // workspace: hi parts, [lo parts,] norms
  uint16_t *Xb = reinterpret_cast<uint16_t *>(ws);
  uint16_t *Xlo = split ? Xb + (size_t)Npad * KP : nullptr;
  float *nrm = reinterpret_cast<float *>(reinterpret_cast<char *>(ws) +
                                         (size_t)Npad * KP * 2 * (split ? 2 : 1));
  const int cpp = KP / 8;
  const size_t lds = (size_t)(cpp < 256 ? cpp : 256) * 32 * sizeof(float);
  const bool vec = ldx % 4 == 0 && (reinterpret_cast<uintptr_t>(X) & 15) == 0;
  const dim3 pgrid((uint32_t)(Npad / 32));
  if (vec)
    hipLaunchKernelGGL(gram_prologue_kernel<true>, pgrid, dim3(256), lds, stream, X, N, d, ldx, Xb, Xlo, nrm, KP);
  else
    hipLaunchKernelGGL(gram_prologue_kernel<false>, pgrid, dim3(256), lds, stream, X, N, d, ldx, Xb, Xlo, nrm, KP);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  GramArgs a{X, N, d, ldx, Xb, Xlo, nrm, KP, D, count};
  if (ts == 256) {
    const uint64_t nb = (uint64_t)(Npad / 256);
    const uint64_t W = (uint64_t)kStripsPerTile * (nb * (nb + 1) / 2);
    uint64_t lo, hi;
    shard_range(W, shard, nshards, lo, hi);
    const uint64_t max_blocks = (((uint64_t)1 << 32) - 1) / (kStripWaves * 64);
    for (uint64_t w0 = lo; w0 < hi; w0 += max_blocks) {
      const uint64_t c = hi - w0 < max_blocks ? hi - w0 : max_blocks;
      if (split)
        launch_gram_strips<true, COUNT>(KP, dim3((uint32_t)c), stream, a, (uint32_t)w0);
      else
        launch_gram_strips<false, COUNT>(KP, dim3((uint32_t)c), stream, a, (uint32_t)w0);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
  }
  if (ts != 128) return hipErrorInvalidValue;
  const uint64_t T = gram_blocks(N);
  uint64_t lo, hi;
  shard_range(T, shard, nshards, lo, hi);
  const uint64_t max_blocks = (((uint64_t)1 << 32) - 1) / 512;
  for (uint64_t l0 = lo; l0 < hi; l0 += max_blocks) {
    const uint64_t c = hi - l0 < max_blocks ? hi - l0 : max_blocks;
    if (split)
      hipLaunchKernelGGL((gram_block_kernel<true, COUNT>), dim3((uint32_t)c), dim3(512), 0, stream, a,
                         (uint32_t)l0, (uint32_t)c);
    else
      hipLaunchKernelGGL((gram_block_kernel<false, COUNT>), dim3((uint32_t)c), dim3(512), 0, stream, a,
                         (uint32_t)l0, (uint32_t)c);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_gram(const float *X, int64_t N, int d, int64_t ldx, float *D, void *ws, bool split,
                       int ts, hipStream_t stream, uint32_t shard, uint32_t nshards) {
  return launch_gram_t<false>(X, N, d, ldx, D, ws, split, ts, nullptr, stream, shard, nshards);
}

hipError_t launch_gram_count(const float *X, int64_t N, int d, int64_t ldx, float *D, void *ws,
                             bool split, int ts, unsigned long long *count, hipStream_t stream) {
  hipError_t e = launch_fill(reinterpret_cast<float *>(count), 2, 0.0f, stream);
  if (e != hipSuccess) return e;
  return launch_gram_t<true>(X, N, d, ldx, D, ws, split, ts, count, stream);
}

}  // namespace tdmap
