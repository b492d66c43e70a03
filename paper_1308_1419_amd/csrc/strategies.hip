// The five space-of-computation strategies as the paper launches them
// (Sec. II-A, Sec. III-B): rho x rho threads per block, one cell per
// thread, the same per-pair function everywhere (so every strategy writes
// bit-identical values).  The maps are arithmetic only: no lookup tables,
// no auxiliary global memory (the restriction of Sec. III-B).
//
// With more than four features, LTM, BB and REC blocks stage their points
// (wide_cell_kernel), and large LTM launches give a work-group several
// blocks of one block column (wide_rows_kernel).
//
// Each kernel has two twins that evaluate the same map and filters: one
// counts blocks / fully idle blocks / idle threads instead of storing (one
// block per work-group, as for up to four features and in wide_cell_kernel;
// the work-groups of wide_rows_kernel are not counted), the other is the
// paper's dummy kernel (Sec. III-A, Sec. IV), which measures the cost of the
// map alone.
#include <type_traits>

#include "device.h"
#include "kernels.h"

namespace tdmap {

enum { kLTM = 0, kBB = 1, kUTM = 2, kRB = 3, kREC = 4 };
enum { kModeStore = 0, kModeCount = 1, kModeDummy = 2 };

template <int D, int LAYOUT, int MODE>
__device__ __forceinline__ void finish_cell(const EdmArgs &a, bool live, int64_t i, int64_t j,
                                            unsigned long long *counts) {
  if constexpr (MODE == kModeCount) {
    count_block(counts, live ? 1 : 0, (int)(blockDim.x * blockDim.y));
  } else if constexpr (MODE == kModeDummy) {
    // the mapping-cost kernel: the cell's i + j is "written" only when it
    // equals a run-time value no cell has, which keeps every step of the map
    // live without a store per thread to one address
    if (live && (uint32_t)(i + j) == a.never) a.sink[0] = (uint32_t)(i + j);
  } else {
    if (live) a.D[out_index<LAYOUT>(i, j, a.ldd)] = cell_dist<D>(a.X, a.ldx, a.d, i, j);
  }
}

// LTM: a 1D grid of exactly n(n+1)/2 blocks; block lambda covers block row
// and column g(lambda) (Sec. II-A, Eq. (2)).  Only the n diagonal blocks
// (and the edge when rho does not divide N) filter threads.
template <int D, int LAYOUT, int MODE>
__global__ void ltm_cell_kernel(EdmArgs a, uint32_t lam0, unsigned long long *counts) {
  uint32_t bi, bj;
  if constexpr (MODE == kModeDummy)
    g_lambda_variant(lam0 + blockIdx.x, a.variant, bi, bj);
  else
    g_lambda(lam0 + blockIdx.x, bi, bj);
  const int64_t i = (int64_t)bi * blockDim.y + threadIdx.y;
  const int64_t j = (int64_t)bj * blockDim.x + threadIdx.x;
  finish_cell<D, LAYOUT, MODE>(a, i < a.N && j <= i, i, j, counts);
}

// BB: an n x n grid (x = block column, y = block row).  A block above the
// diagonal returns before computing any thread coordinate; the others keep
// cells with j <= i < N (Sec. III-B).
template <int D, int LAYOUT, int MODE>
__global__ void bb_cell_kernel(EdmArgs a, unsigned long long *counts) {
  const uint32_t bx = blockIdx.x, by = blockIdx.y;
  // the timed kernels (EDM and dummy) discard the block at once; the
  // counting variant keeps every thread for the block-wide count
  if constexpr (MODE != kModeCount) {
    if (bx > by) return;
  }
  const int64_t i = (int64_t)by * blockDim.y + threadIdx.y;
  const int64_t j = (int64_t)bx * blockDim.x + threadIdx.x;
  finish_cell<D, LAYOUT, MODE>(a, bx <= by && i < a.N && j <= i, i, j, counts);
}

// UTM (Avril et al., Sec. III-B): thread k of a 1D grid takes the k-th pair
// (a, b), 1 <= a < b <= n, of the strictly upper triangle of an n x n
// matrix, with n = N + 1 so that there are exactly N(N+1)/2 pairs:
//   a = floor(((2n+1) - sqrt((2n-1)^2 - 8k)) / 2),
//   b = (a+1) + k - (a-1)(2n-a)/2.
// The square root is single precision; two integer conditionals repair a
// row that is off by one.  The pair is half-turned onto the lower triangle
// with the diagonal: (i, j) = (N - a, N + 1 - b), which keeps consecutive
// threads on one output row.
template <int D, int LAYOUT, int MODE>
__global__ void utm_cell_kernel(EdmArgs a, uint64_t k0, unsigned long long *counts) {
  const uint32_t lanes = blockDim.x * blockDim.y;
  const uint64_t k = k0 + (uint64_t)blockIdx.x * lanes + threadIdx.y * blockDim.x + threadIdx.x;
  const int64_t N = a.N;
  const uint64_t P = (uint64_t)N * (uint64_t)(N + 1) / 2;
  bool live = k < P;
  int64_t i = 0, j = 0;
  if (live) {
    const int64_t n = N + 1;
    const int64_t disc = (2 * n - 1) * (2 * n - 1) - 8 * (int64_t)k;
    const float sq = __builtin_amdgcn_sqrtf((float)disc);
    int64_t r = (int64_t)__builtin_floorf(((float)(2 * n + 1) - sq) * 0.5f);
    // start(a) = (a-1)(2n-a)/2 is the index of the first pair of row a
    const int64_t kk = (int64_t)k;
    if ((r - 1) * (2 * n - r) / 2 > kk) {
      --r;
    } else if (r * (2 * n - r - 1) / 2 <= kk) {
      ++r;
    }
    const int64_t b = (r + 1) + kk - (r - 1) * (2 * n - r) / 2;
    i = N - r;
    j = N + 1 - b;
    // a guess more than one row off would land outside the triangle: such
    // a thread stores nothing (the coverage tests would then fail)
    live = i >= 0 && i < N && j >= 0 && j <= i;
  }
  finish_cell<D, LAYOUT, MODE>(a, live, i, j, counts);
}

// RB (Jung et al., Sec. III-B): the threads form a rectangle; for even N
// it has N+1 rows and N/2 columns, the part above its diagonal being the
// turned-over sub-triangle of columns >= N/2.  Below the diagonal
// (ty > tx): (i, j) = (ty - 1, tx); on or above: (N - 1 - ty, N - 1 - tx).
// Odd N cuts at floor(N/2): N rows, floor(N/2)+1 columns, (ty, tx) when
// ty >= tx, else (N - 1 - ty, N - tx).
template <int D, int LAYOUT, int MODE>
__global__ void rb_cell_kernel(EdmArgs a, unsigned long long *counts) {
  const int64_t N = a.N;
  const int64_t ty = (int64_t)blockIdx.y * blockDim.y + threadIdx.y;
  const int64_t tx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool even = (N & 1) == 0;
  const int64_t rows = even ? N + 1 : N;
  const int64_t cols = even ? N / 2 : N / 2 + 1;
  const bool live = ty < rows && tx < cols;
  int64_t i, j;
  if (even) {
    if (ty > tx) {
      i = ty - 1;
      j = tx;
    } else {
      i = N - 1 - ty;
      j = N - 1 - tx;
    }
  } else {
    if (ty >= tx) {
      i = ty;
      j = tx;
    } else {
      i = N - 1 - ty;
      j = N - tx;
    }
  }
  finish_cell<D, LAYOUT, MODE>(a, live, i, j, counts);
}

// REC (Ries et al., Sec. III-B), in block units: the side is padded to
// m 2^k blocks (m <= 16).  mode 0 is the diagonal pass: 2^k base squares of
// m x m blocks, each a small bounding box (grid m x (m 2^k)).  mode 1 is one
// level of the bottom-up recursion with squares of side s = m 2^l: square q
// sits at block rows [(2q+1)s, (2q+2)s) and block columns [2qs, (2q+1)s)
// (grid s x (s * 2^(k-1-l))).  Block coordinates are computed at run time,
// not looked up.  Blocks past the real side nb are idle.
template <int D, int LAYOUT, int MODE>
__global__ void rec_cell_kernel(EdmArgs a, int mode, uint32_t side, uint32_t nb,
                                unsigned long long *counts) {
  const uint32_t q = blockIdx.y / side;
  const uint32_t lby = blockIdx.y - q * side;
  uint32_t R, C;
  bool blk_live;
  if (mode == 0) {
    R = q * side + lby;
    C = q * side + blockIdx.x;
    blk_live = blockIdx.x <= lby;
  } else {
    R = (2 * q + 1) * side + lby;
    C = 2 * q * side + blockIdx.x;
    blk_live = true;
  }
  blk_live = blk_live && R < nb;
  if constexpr (MODE != kModeCount) {
    if (!blk_live) return;
  }
  const int64_t i = (int64_t)R * blockDim.y + threadIdx.y;
  const int64_t j = (int64_t)C * blockDim.x + threadIdx.x;
  finish_cell<D, LAYOUT, MODE>(a, blk_live && i < a.N && j <= i, i, j, counts);
}

// ---------------------------------------------------------------------------
// more than four features: the same blocks, points staged per block
// ---------------------------------------------------------------------------

// Lane K of each 16-lane row, in every lane of the row (row_newbcast folds
// into the subtraction that consumes it).
template <int K>
__device__ __forceinline__ float row_lane(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x150 + K,
                                                               0xF, 0xF, true));
}

typedef float f4 __attribute__((ext_vector_type(4)));

// Four features of the pair sum, in feature order (the operation order of
// pair_dist).
template <int K>
__device__ __forceinline__ float add_features(float s, float row, f4 c) {
  const float c0 = c[0], c1 = c[1], c2 = c[2], c3 = c[3];
  float t = row_lane<K>(row) - c0;
  s = __builtin_fmaf(t, t, s);
  t = row_lane<K + 1>(row) - c1;
  s = __builtin_fmaf(t, t, s);
  t = row_lane<K + 2>(row) - c2;
  s = __builtin_fmaf(t, t, s);
  t = row_lane<K + 3>(row) - c3;
  return __builtin_fmaf(t, t, s);
}

// LTM, BB and REC blocks (rho x rho threads on a rho x rho square of cells,
// one cell per thread) for d > 4.  A thread that reads its two points on its
// own issues 2 d loads, and a wave's 64 column loads touch 16 to 32 rows of
// X each: at N = 8000, d = 16, rho = 16 (full layout, LTM) the launch took
// 907 us, bound by those uncoalesced loads; this one takes 92 us, bound by
// the placing of its block (wide_rows_kernel below takes such sizes).
// Here a block takes the features 16 at a time:
// its rho column points are loaded once, coalesced, into LDS (pitch 20
// floats: the 16-byte reads of 16 lanes cover every bank once), the next 16
// features being loaded before the current ones are used.  rho 16 and 32:
// lane l holds feature l mod 16 of its row's point and the row_newbcast lane
// move hands it to the row's 16 lanes, so the row points need no LDS read;
// rho 8 (two rows in 16 lanes) reads them from LDS.  Features past d are 0
// in both points and add an exact 0, so the sum has the bits of
// pair_dist_rt.  LTM takes one contiguous range of lambda per XCD: the two
// 64-byte pieces of an output line then meet in one L2.  ROUTE is the
// strategy (the enum above).
template <int RHO, int LAYOUT, int ROUTE>
__global__ __launch_bounds__(RHO *RHO) void wide_cell_kernel(EdmArgs a, uint32_t lam0, int mode,
                                                             uint32_t side, uint32_t nb) {
  constexpr int F = 16;       // features per step
  constexpr int PITCH = 20;   // floats per staged point
  constexpr int NT = RHO * RHO;
  constexpr int PER = RHO * F >= NT ? RHO * F / NT : 1;  // staged values per thread
  constexpr bool ALL = RHO * F >= NT;                    // every thread stages
  uint32_t bi, bj;
  if constexpr (ROUTE == kLTM) {
    g_lambda_uniform(lam0 + xcd_contiguous(blockIdx.x, gridDim.x), bi, bj);
  } else if constexpr (ROUTE == kBB) {
    bj = blockIdx.x;
    bi = blockIdx.y;
    if (bj > bi) return;
  } else {
    const uint32_t q = blockIdx.y / side;
    const uint32_t lby = blockIdx.y - q * side;
    bi = (mode == 0 ? q : 2 * q + 1) * side + lby;
    bj = (mode == 0 ? q : 2 * q) * side + blockIdx.x;
    if (bi >= nb || (mode == 0 && blockIdx.x > lby)) return;
  }
  const uint32_t tx = threadIdx.x, ty = threadIdx.y;
  const uint32_t t = ty * RHO + tx;
  const int d = a.d;
  // the 32-bit block index keeps N below 92682 rho
  const uint32_t N = (uint32_t)a.N, i0 = bi * RHO, j0 = bj * RHO;
  const uint32_t ni = N - i0 < RHO ? N - i0 : RHO;  // points of the block that exist
  const uint32_t nj = N - j0 < RHO ? N - j0 : RHO;
  const float *__restrict__ Xi = a.X + i0 * a.ldx;
  const float *__restrict__ Xj = a.X + j0 * a.ldx;
  __shared__ __align__(16) float xc[2][RHO * PITCH];
  __shared__ __align__(16) float xr[RHO == 8 ? 2 : 1][RHO == 8 ? RHO * PITCH : 4];

  // the thread's staged elements: point (t + NT m) / 16, feature t mod 16;
  // its row element: point ty (rho 8: as staged), the same feature
  const uint32_t f = RHO == 8 ? t % F : tx % F;
  uint64_t co[PER];
#pragma unroll
  for (int m = 0; m < PER; ++m) co[m] = (uint64_t)((RHO == 16 ? ty : t / F) + NT / F * m) * (uint64_t)a.ldx + f;
  const uint64_t ro = RHO == 16 ? co[0] : (uint64_t)ty * (uint64_t)a.ldx + f;
  const bool whole = ni == RHO && nj == RHO;
  float cv[PER], rv[PER];
  auto load = [&](int k0) {
    if (whole && k0 + F <= d) {
#pragma unroll
      for (int m = 0; m < PER; ++m) {
        if (ALL || t < RHO * F) {
          cv[m] = Xj[co[m] + k0];
          if constexpr (RHO == 8) rv[m] = Xi[co[m] + k0];
        }
      }
      if constexpr (RHO != 8) rv[0] = Xi[ro + k0];
      return;
    }
    const bool kok = k0 + (int)f < d;
#pragma unroll
    for (int m = 0; m < PER; ++m) {
      const uint32_t p = t / F + NT / F * m;
      cv[m] = kok && p < nj ? Xj[co[m] + k0] : 0.0f;
      if constexpr (RHO == 8) rv[m] = kok && p < ni ? Xi[co[m] + k0] : 0.0f;
    }
    if constexpr (RHO != 8) rv[0] = kok && ty < ni ? Xi[ro + k0] : 0.0f;
  };
  load(0);
  float s = 0.0f;
  for (int k0 = 0, b = 0; k0 < d; k0 += F, b ^= 1) {
    const float row = rv[0];
    if (ALL || t < RHO * F) {
#pragma unroll
      for (int m = 0; m < PER; ++m) {
        const uint32_t at = (t / F + NT / F * m) * PITCH + f;
        xc[b][at] = cv[m];
        if constexpr (RHO == 8) xr[b][at] = rv[m];
      }
    }
    if (k0 + F < d) load(k0 + F);
    // the other buffer's readers passed the previous step's barrier
    __syncthreads();
    const f4 *c = reinterpret_cast<const f4 *>(&xc[b][tx * PITCH]);
    if constexpr (RHO == 8) {
      const f4 *r = reinterpret_cast<const f4 *>(&xr[b][ty * PITCH]);
#pragma unroll
      for (int q = 0; q < F / 4; ++q) {
        if (k0 + 4 * q < d) {
          const f4 u = r[q], v = c[q];
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const float x = u[k], y = v[k];
            const float tt = x - y;
            s = __builtin_fmaf(tt, tt, s);
          }
        }
      }
    } else {
      s = add_features<0>(s, row, c[0]);
      if (k0 + 4 < d) s = add_features<4>(s, row, c[1]);
      if (k0 + 8 < d) s = add_features<8>(s, row, c[2]);
      if (k0 + 12 < d) s = add_features<12>(s, row, c[3]);
    }
  }
  const float v = __builtin_amdgcn_sqrtf(s);
  // cell (i0 + ty, j0 + tx): the block's first cell and a lane offset
  // (packed: T(i0 + ty) = T(i0) + ty i0 + ty (ty + 1) / 2, ty i0 < 2^32)
  float *__restrict__ o = a.D + out_index<LAYOUT>((uint64_t)i0, (uint64_t)j0, a.ldd);
  uint64_t lo;
  if constexpr (LAYOUT == kLayoutFull)
    lo = (uint64_t)ty * (uint64_t)a.ldd + tx;
  else
    lo = ty * i0 + ((ty * (ty + 1)) >> 1) + tx;
  if (bj < bi && ni == RHO)
    o[lo] = v;
  else if (ty < ni && j0 + tx <= i0 + ty)
    o[lo] = v;
}

// The LTM launches of wide_cell_kernel with enough blocks.  Placing a block
// costs each of its waves about 110 scalar instructions and its column points
// four 16-byte LDS reads a lane, against 32 vector instructions of sum per 16
// features; so a work-group does W block rows of one block column in turn,
// with the column's features in registers for all of them and only the row
// points read anew, all W loaded before the first is used.  Work-group u: with
// (I, J) = g(u / W), block column W J + u mod W of block rows W I ..
// W I + W - 1; consecutive work-groups are neighbouring columns of the same
// rows, and each XCD takes one contiguous range of u, as there.  Bound by the
// vector instructions of the sums (26 us at the size below).  N = 8000,
// d = 16, full layout: rho 16 45 us (wide_cell_kernel 92), rho 8 58 (117);
// packed, rho 32 53 (107).  Rho 8 takes W = 4: its row points (64 of them at
// W = 8) are read from LDS, and 100 registers and 5.8 KB leave 64 us.
// Offsets are 32 bits from uniform addresses (both pitches below 2^22).
template <int RHO, int LAYOUT, int W>
__global__ __launch_bounds__(RHO *RHO) void wide_rows_kernel(EdmArgs a, uint32_t u0) {
  constexpr int F = 16;       // features per step
  constexpr int PITCH = F + 4;
  constexpr int NT = RHO * RHO;
  constexpr int PER = RHO * F >= NT ? RHO * F / NT : 1;  // staged column values per thread
  constexpr bool ALL = RHO * F >= NT;                    // every thread stages
  constexpr int STEP = RHO == 8 ? NT / F : RHO;          // between a thread's row points
  constexpr int NR = RHO * W / STEP;                     // a thread's row values
  const uint32_t u = u0 + xcd_contiguous(blockIdx.x, gridDim.x);
  uint32_t bi, bj;
  g_lambda_uniform(u / W, bi, bj);
  bi *= W;
  bj = bj * W + u % W;
  const uint32_t N = (uint32_t)a.N, end = (N - 1) / RHO;  // end: the last block row
  if (bj > end) return;
  const uint32_t tx = threadIdx.x, ty = threadIdx.y, t = ty * RHO + tx;
  const int d = a.d;
  __shared__ __align__(16) float xc[RHO * PITCH];
  __shared__ __align__(16) float xr[RHO == 8 ? RHO * W * PITCH : 4];
  const uint32_t f = RHO == 8 ? t % F : tx % F;
  auto offset = [](uint32_t r, int64_t pitch, uint32_t c) {
    return ((r & 0xffu) * ((uint32_t)pitch & 0x3fffffu) + c) * 4u;
  };
  auto at = [](const float *base, uint32_t o) {
    return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(base) + o);
  };
  // points past the last are read as the last (their cells are not stored),
  // features past d as the last and taken as 0 when used
  const uint32_t ni = N - bi * RHO, nj = N - bj * RHO;
  const bool inner = ni >= RHO * W;
  uint32_t co[PER];
#pragma unroll
  for (int m = 0; m < PER; ++m) {
    const uint32_t r = (RHO == 16 ? ty : t / F) + NT / F * m;
    co[m] = offset(r < nj ? r : nj - 1, a.ldx, f);
  }
  const uint32_t rp = RHO == 8 ? t / F : ty;  // the thread's first row point
  const uint32_t ro = offset(rp, a.ldx, f);
  const float *__restrict__ xi = a.X + (uint64_t)(bi * RHO) * (uint64_t)a.ldx;
  const float *__restrict__ xj = a.X + (uint64_t)(bj * RHO) * (uint64_t)a.ldx;
  float cv[PER], rv[NR];
  auto load = [&](int k0) {
    const uint32_t lf = (uint32_t)(d - 1 - k0);
    const uint32_t back = lf < F - 1 && f > lf ? (f - lf) * 4u : 0u;
#pragma unroll
    for (int m = 0; m < PER; ++m)
      if (ALL || t < RHO * F) cv[m] = at(xj + k0, co[m] - back);
    if (inner) {
#pragma unroll
      for (int m = 0; m < NR; ++m) rv[m] = at(xi + (int64_t)(m * STEP) * a.ldx + k0, ro - back);
    } else {
#pragma unroll
      for (int m = 0; m < NR; ++m) {
        const uint32_t r = rp + m * STEP;
        rv[m] = at(xi + k0, offset(r < ni ? r : ni - 1, a.ldx, f) - back);
      }
    }
  };
  load(0);
  float s[W] = {};
  for (int k0 = 0;; k0 += F) {
    const bool over = k0 + F >= d;
    if (k0 + F > d && k0 + (int)f >= d) {
#pragma unroll
      for (int m = 0; m < PER; ++m) cv[m] = 0.0f;
#pragma unroll
      for (int m = 0; m < NR; ++m) rv[m] = 0.0f;
    }
    if (k0 > 0) __syncthreads();
    if (ALL || t < RHO * F) {
#pragma unroll
      for (int m = 0; m < PER; ++m) xc[(t / F + NT / F * m) * PITCH + f] = cv[m];
    }
    float row[RHO == 8 ? 1 : W];
#pragma unroll
    for (int m = 0; m < NR; ++m) {
      if constexpr (RHO == 8)
        xr[(rp + m * STEP) * PITCH + f] = rv[m];
      else
        row[m] = rv[m];
    }
    if (!over) load(k0 + F);
    __syncthreads();
    auto add = [&](auto q) {
      constexpr int Q = decltype(q)::value;
      const f4 c = *reinterpret_cast<const f4 *>(&xc[tx * PITCH + Q]);
#pragma unroll
      for (int w = 0; w < W; ++w) {
        if constexpr (RHO == 8) {
          const f4 r = *reinterpret_cast<const f4 *>(&xr[(w * RHO + ty) * PITCH + Q]);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const float tt = r[k] - c[k];
            s[w] = __builtin_fmaf(tt, tt, s[w]);
          }
        } else {
          s[w] = add_features<Q>(s[w], row[w], c);
        }
      }
    };
    add(std::integral_constant<int, 0>());
    if (k0 + 4 < d) add(std::integral_constant<int, 4>());
    if (k0 + 8 < d) add(std::integral_constant<int, 8>());
    if (k0 + 12 < d) add(std::integral_constant<int, 12>());
    if (over) break;
  }
  // cell (i0 + ty, j0 + tx): the block's first cell and a lane offset
  // (packed: T(i0 + ty) = T(i0) + ty i0 + ty (ty + 1) / 2, ty i0 < 2^30)
#pragma unroll
  for (int w = 0; w < W; ++w) {
    const uint32_t i = bi + w;
    if (i < bj || i > end) continue;
    float *__restrict__ o = a.D + out_index<LAYOUT>((uint64_t)(i * RHO), (uint64_t)(bj * RHO), a.ldd);
    uint32_t lo;
    if constexpr (LAYOUT == kLayoutFull)
      lo = offset(ty, a.ldd, tx);
    else
      lo = (ty * (i * RHO) + ((ty * (ty + 1)) >> 1) + tx) * 4u;
    float *__restrict__ cell = reinterpret_cast<float *>(reinterpret_cast<char *>(o) + lo);
    const float v = __builtin_amdgcn_sqrtf(s[w]);
    if (bj < i && i < end)
      *cell = v;
    else if (i * RHO + ty < N && bj * RHO + tx <= i * RHO + ty)
      *cell = v;
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

static void rec_shape(uint32_t nb, uint32_t &m, uint32_t &k) {
  uint64_t best = 0;
  for (uint32_t mm = 16; mm >= 1; --mm) {
    uint32_t kk = 0;
    while (((uint64_t)mm << kk) < nb) ++kk;
    const uint64_t side = (uint64_t)mm << kk;
    if (best == 0 || side < best) {
      best = side;
      m = mm;
      k = kk;
    }
  }
}

// The launches of the strategies whose blocks are rho x rho squares of
// cells (LTM, BB, REC): go(route, grid, lam0, mode, side) makes one launch,
// route an integral_constant of the strategy.
template <class Go>
static hipError_t launch_square_blocks(int strategy, int rho, const EdmArgs &a, Go go) {
  const uint64_t nb = (uint64_t)((a.N + rho - 1) / rho);
  // keep every launch below 2^32 work-items
  const uint64_t max_blocks = (((uint64_t)1 << 32) - 1) / ((uint64_t)rho * rho);
  hipError_t e = hipSuccess;
  switch (strategy) {
    case kLTM: {
      const uint64_t T = nb * (nb + 1) / 2;
      for (uint64_t l0 = 0; l0 < T; l0 += max_blocks) {
        const uint64_t c = T - l0 < max_blocks ? T - l0 : max_blocks;
        go(std::integral_constant<int, kLTM>(), dim3((uint32_t)c), (uint32_t)l0, 0, 0u);
        if ((e = hipGetLastError()) != hipSuccess) return e;
      }
      return e;
    }
    case kBB:
      go(std::integral_constant<int, kBB>(), dim3((uint32_t)nb, (uint32_t)nb), 0u, 0, 0u);
      return hipGetLastError();
    case kREC: {
      uint32_t m = 1, k = 0;
      rec_shape((uint32_t)nb, m, k);
      go(std::integral_constant<int, kREC>(), dim3(m, m << k), 0u, 0, m);
      if ((e = hipGetLastError()) != hipSuccess) return e;
      for (uint32_t lev = 0; lev < k; ++lev) {
        const uint32_t s = m << lev;
        const uint32_t squares = 1u << (k - 1 - lev);
        go(std::integral_constant<int, kREC>(), dim3(s, s * squares), 0u, 1, s);
        if ((e = hipGetLastError()) != hipSuccess) return e;
      }
      return e;
    }
    default:
      return hipErrorInvalidValue;
  }
}

// UTM and RB.
template <int D, int LAYOUT, int MODE>
static hipError_t launch_pair_blocks(int strategy, int rho, const EdmArgs &a,
                                     unsigned long long *counts) {
  const dim3 blk(rho, rho);
  const uint64_t lanes = (uint64_t)rho * rho;
  const uint64_t max_blocks = (((uint64_t)1 << 32) - 1) / lanes;
  hipError_t e = hipSuccess;
  if (strategy == kUTM) {
    const uint64_t P = (uint64_t)a.N * (uint64_t)(a.N + 1) / 2;
    const uint64_t blocks = (P + lanes - 1) / lanes;
    for (uint64_t b0 = 0; b0 < blocks; b0 += max_blocks) {
      const uint64_t c = blocks - b0 < max_blocks ? blocks - b0 : max_blocks;
      hipLaunchKernelGGL((utm_cell_kernel<D, LAYOUT, MODE>), dim3((uint32_t)c), blk, 0,
                         a.stream, a, b0 * lanes, counts);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return e;
  }
  if (strategy != kRB) return hipErrorInvalidValue;
  const int64_t rows = (a.N % 2 == 0) ? a.N + 1 : a.N;
  const int64_t cols = (a.N % 2 == 0) ? a.N / 2 : a.N / 2 + 1;
  const uint32_t gx = (uint32_t)((cols + rho - 1) / rho);
  const uint32_t gy = (uint32_t)((rows + rho - 1) / rho);
  if (gx == 0 || gy == 0) return hipSuccess;
  hipLaunchKernelGGL((rb_cell_kernel<D, LAYOUT, MODE>), dim3(gx, gy), blk, 0, a.stream, a,
                     counts);
  return hipGetLastError();
}

template <int D, int LAYOUT, int MODE>
static hipError_t launch_cell_t(int strategy, int rho, const EdmArgs &a,
                                unsigned long long *counts) {
  if (strategy == kUTM || strategy == kRB)
    return launch_pair_blocks<D, LAYOUT, MODE>(strategy, rho, a, counts);
  const uint32_t nb = (uint32_t)((a.N + rho - 1) / rho);
  return launch_square_blocks(
      strategy, rho, a, [&](auto route, dim3 grid, uint32_t lam0, int mode, uint32_t side) {
        const dim3 blk(rho, rho);
        if constexpr (route == kLTM)
          hipLaunchKernelGGL((ltm_cell_kernel<D, LAYOUT, MODE>), grid, blk, 0, a.stream, a, lam0,
                             counts);
        else if constexpr (route == kBB)
          hipLaunchKernelGGL((bb_cell_kernel<D, LAYOUT, MODE>), grid, blk, 0, a.stream, a, counts);
        else
          hipLaunchKernelGGL((rec_cell_kernel<D, LAYOUT, MODE>), grid, blk, 0, a.stream, a, mode,
                             side, nb, counts);
      });
}

template <int RHO, int LAYOUT, int W>
static hipError_t launch_wide_rows(const EdmArgs &a) {
  const uint64_t rows = (uint64_t)(a.N + RHO * W - 1) / (RHO * W), groups = W * rows * (rows + 1) / 2;
  // keep every launch below 2^32 work-items
  const uint64_t most = (((uint64_t)1 << 32) - 1) / (RHO * RHO);
  for (uint64_t u0 = 0; u0 < groups; u0 += most) {
    const uint64_t c = groups - u0 < most ? groups - u0 : most;
    hipLaunchKernelGGL((wide_rows_kernel<RHO, LAYOUT, W>), dim3((uint32_t)c), dim3(RHO, RHO), 0, a.stream, a,
                       (uint32_t)u0);
    if (const hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Cells (N^2 / 2) from which a work-group takes 4, and (rho 16 and 32) 8 block
// rows: below, the fewer work-groups leave the chip idle, the more so the longer
// a block takes (d, rho).  One / 4 rows, us, full layout, around 2^20 cells:
//   N = 1000   rho 8, d = 5 4.1 / 3.9, d = 64 5.8 / 6.7   rho 16, d = 32 4.3 / 4.8
//   N = 1200   rho 8, d = 5 4.8 / 3.7, d = 64 7.1 / 7.0   rho 16, d = 32 5.1 / 4.9
//   N = 1449   rho 8, d = 5 6.1 / 4.5, d = 64 9.0 / 9.0   rho 16, d = 32 6.4 / 6.1
//              rho 32, d = 5 6.3 / 5.1, d = 64 12.6 / 12.6
//   N = 2000   rho 8, d = 64 14.6 / 12.3   rho 32, d = 64 19.0 / 17.7
// 4 / 8 rows around 6 * 2^20:
//   N = 3000   rho 16, d = 5 9.2 / 8.9, d = 64 22.5 / 23.5   rho 32, d = 64 27.1 / 29.3
//   N = 3548   rho 16, d = 5 11.3 / 10.6, d = 64 29.2 / 29.0   rho 32, d = 5 14.0 / 13.4,
//              d = 64 36.2 / 37.3
//   N = 4500   rho 16, d = 64 43.5 / 42.8   rho 32, d = 64 54.0 / 52.3
constexpr uint64_t kWideRows4 = 1 << 20;
constexpr uint64_t kWideRows8 = 6 << 20;
template <int RHO, int LAYOUT>
static hipError_t launch_wide_t(int strategy, const EdmArgs &a) {
  const uint32_t nb = (uint32_t)((a.N + RHO - 1) / RHO);
  const uint64_t cells = (uint64_t)a.N * (uint64_t)a.N / 2;
  if (strategy == kLTM && cells >= kWideRows4 && a.ldx < (1 << 22) && (LAYOUT != kLayoutFull || a.ldd < (1 << 22))) {
    if (RHO > 8 && cells >= kWideRows8) return launch_wide_rows<RHO, LAYOUT, RHO == 8 ? 4 : 8>(a);
    return launch_wide_rows<RHO, LAYOUT, 4>(a);
  }
  return launch_square_blocks(
      strategy, RHO, a, [&](auto route, dim3 grid, uint32_t lam0, int mode, uint32_t side) {
        hipLaunchKernelGGL((wide_cell_kernel<RHO, LAYOUT, route>), grid, dim3(RHO, RHO), 0, a.stream,
                           a, lam0, mode, side, nb);
      });
}

template <int LAYOUT>
static hipError_t launch_wide(int strategy, int rho, const EdmArgs &a) {
  switch (rho) {
    case 8: return launch_wide_t<8, LAYOUT>(strategy, a);
    case 16: return launch_wide_t<16, LAYOUT>(strategy, a);
    case 32: return launch_wide_t<32, LAYOUT>(strategy, a);
    default: return hipErrorInvalidValue;
  }
}

template <int LAYOUT>
static hipError_t launch_cell_layout(int strategy, int rho, const EdmArgs &a) {
  switch (a.d) {
    case 1: return launch_cell_t<1, LAYOUT, kModeStore>(strategy, rho, a, nullptr);
    case 2: return launch_cell_t<2, LAYOUT, kModeStore>(strategy, rho, a, nullptr);
    case 3: return launch_cell_t<3, LAYOUT, kModeStore>(strategy, rho, a, nullptr);
    case 4: return launch_cell_t<4, LAYOUT, kModeStore>(strategy, rho, a, nullptr);
    default: break;
  }
  // more than four features: the square-block strategies stage the points;
  // UTM and RB blocks are not squares of cells (a block of UTM is a run of
  // pairs, one of RB may straddle the turned-over part)
  switch (strategy) {
    case kUTM:
    case kRB: return launch_pair_blocks<0, LAYOUT, kModeStore>(strategy, rho, a, nullptr);
    default: return launch_wide<LAYOUT>(strategy, rho, a);
  }
}

hipError_t launch_cell(int strategy, int rho, const EdmArgs &a, unsigned long long *counts) {
  if (a.N == 0) return hipSuccess;
  if (counts) return launch_cell_t<1, kLayoutPacked, kModeCount>(strategy, rho, a, counts);
  return a.layout == kLayoutFull ? launch_cell_layout<kLayoutFull>(strategy, rho, a)
                                 : launch_cell_layout<kLayoutPacked>(strategy, rho, a);
}

hipError_t launch_dummy(int strategy, int rho, const EdmArgs &a) {
  if (a.N == 0) return hipSuccess;
  return launch_cell_t<1, kLayoutPacked, kModeDummy>(strategy, rho, a, nullptr);
}

}  // namespace tdmap
