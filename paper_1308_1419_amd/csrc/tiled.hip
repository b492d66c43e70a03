// Coarsened EDM tiles for gfx950.
//
// The paper's point is that g(lambda) maps *blocks*, so the thread
// organisation inside a block is free (Sec. II-A; Sec. V notes this eases
// shared memory and thread coarsening).  Here a 256-thread work-group owns a
// TS x TS tile of cells:
//   - the tile's TS row points are staged once in LDS (read back with
//     broadcast, all lanes of a row share an address);
//   - each lane keeps its column points in registers;
//   - with VEC (full layout) a lane owns four consecutive columns and
//     stores them with one 16-byte store, so a wave writes TS/4-lane runs of
//     16 bytes: whole 64-byte segments of a row.  Without VEC a lane owns one
//     column and a wave writes 256 contiguous bytes.
// Full-layout stores are non-temporal (the output is written once and not
// re-read); packed-layout stores are plain (see put below).
//
// LTM launches exactly n(n+1)/2 work-groups, tile (I, J) = g(lambda) with
// lambda remapped so that every XCD owns one contiguous range of it
// (xcd_contiguous in device.h).  BB launches n x n and returns at once above
// the diagonal (Sec. III-B), with the same tile body, which makes the two
// directly comparable.
//
// TS = 256: edm_band_kernel below, which writes low, wide strips (no LDS, row
// points through the scalar cache).
// TS = 64 / 128: edm_tile_kernel.
#include "device.h"
#include "kernels.h"

namespace tdmap {

typedef float f4 __attribute__((ext_vector_type(4)));

// Output stores.  Full-layout rows are written whole by one tile each, so
// they bypass the caches (non-temporal).  Packed rows start at arbitrary
// offsets: the 16-byte chunks and cache lines at both ends of a tile's row
// segment are shared with the neighbouring tiles, and plain (cached) stores
// let those parts meet in L2 instead of reaching HBM as separate partial
// line writes (measured faster at every tile size).
template <int LAYOUT, typename T>
__device__ __forceinline__ void put(T v, T *p) {
  if constexpr (LAYOUT == kLayoutFull)
    __builtin_nontemporal_store(v, p);
  else
    *p = v;
}

template <int TS, int D, int LAYOUT, bool VEC, bool BB>
__global__ __launch_bounds__(256) void edm_tile_kernel(EdmArgs a, uint32_t lam0) {
  uint32_t I, J;
  if constexpr (BB) {
    J = blockIdx.x;
    I = blockIdx.y;
    if (J > I) return;
  } else {
    g_lambda(lam0 + xcd_contiguous(blockIdx.x, gridDim.x), I, J);
  }
  constexpr int V = VEC ? 4 : 1;    // cells per lane per row
  constexpr int LPR = TS / V;       // lanes per tile row
  static_assert(256 % LPR == 0, "tile row must divide the work-group");
  constexpr int RPP = 256 / LPR;    // rows per pass
  constexpr int PASSES = TS / RPP;

  const int t = threadIdx.x;
  const int lc = (t % LPR) * V;
  const int lr = t / LPR;
  const int64_t N = a.N;
  const int64_t row0 = (int64_t)I * TS;
  const int64_t col0 = (int64_t)J * TS;

  __shared__ float xs[TS * D];
  for (int e = t; e < TS * D; e += 256) {
    const int r = e / D;
    const int k = e - r * D;
    const int64_t p = row0 + r;
    xs[e] = p < N ? a.X[p * a.ldx + k] : 0.0f;
  }
  float xj[V][D];
#pragma unroll
  for (int q = 0; q < V; ++q) {
    const int64_t p = col0 + lc + q;
#pragma unroll
    for (int k = 0; k < D; ++k) xj[q][k] = p < N ? a.X[p * a.ldx + k] : 0.0f;
  }
  __syncthreads();

  float *__restrict__ out = a.D;
  const bool interior = (J < I) && (row0 + TS <= N);
  static_assert(!VEC || LAYOUT == kLayoutFull, "16-byte stores need the full layout");
  if (interior) {
#pragma unroll 8
    for (int ps = 0; ps < PASSES; ++ps) {
      const int r = lr + ps * RPP;
      float xi[D];
#pragma unroll
      for (int k = 0; k < D; ++k) xi[k] = xs[r * D + k];
      const uint64_t idx = out_index<LAYOUT>(row0 + r, col0 + lc, a.ldd);
      if constexpr (VEC) {
        f4 v;
        v.x = pair_dist<D>(xi, xj[0]);
        v.y = pair_dist<D>(xi, xj[1]);
        v.z = pair_dist<D>(xi, xj[2]);
        v.w = pair_dist<D>(xi, xj[3]);
        put<LAYOUT>(v, reinterpret_cast<f4 *>(out + idx));
      } else {
        put<LAYOUT>(pair_dist<D>(xi, xj[0]), out + idx);
      }
    }
  } else {
    // diagonal or edge tile: keep cells with j <= i < N (j < i for the
    // layout without the diagonal; j < N follows)
    for (int ps = 0; ps < PASSES; ++ps) {
      const int r = lr + ps * RPP;
      const int64_t i = row0 + r;
      if (i >= N) break;
      float xi[D];
#pragma unroll
      for (int k = 0; k < D; ++k) xi[k] = xs[r * D + k];
      const uint64_t idx = out_index<LAYOUT>(i, col0 + lc, a.ldd);
#pragma unroll
      for (int q = 0; q < V; ++q) {
        if (in_triangle<LAYOUT>(i, col0 + lc + q))
          put<LAYOUT>(pair_dist<D>(xi, xj[q]), out + idx + q);
      }
    }
  }
}

// rho = 256: rows written as strips.  W x W tiles are placed by g(lambda),
// tile row I is cut into S = W / H strips of H rows, and a 256-thread
// work-group writes one strip of one tile, H x W = 2048 cells: each wave two
// rows x 256 columns.  LTM: work-group w takes tile row I from g(w / S) (the
// paper's block map at the tile level); the S (I + 1) work-groups of tile
// row I are then numbered u = k (I + 1) + J, strip k outer and tile column J
// inner, so the work-groups in flight finish a few whole rows of the triangle
// before they move down instead of spreading over the many rows of whole
// tiles.  BB: an S n' x n grid, blockIdx.y = I, blockIdx.x = k n' + J,
// returning at once for J > I.  n' is n made odd: consecutive work-groups go to
// the eight XCDs in turn, so with an even n a tile column's strips would all go
// to some of them, and the low columns, which every row has, make those late
// (n = 8: column J on XCD J alone).  n' = n / n made odd, us: full, N = 8192, d =
// 1, 3, 4 35.6 / 24.7, 34.5 / 25.6, 38.4 / 25.6; packed, N = 12000 54.7 / 47.3,
// 54.5 / 47.8, 55.1 / 48.5; full, N = 9217 (n = 10) 43.5 / 45.1, 42.7 / 44.2.
// Turning the columns by k mod 8 instead breaks up the rows: full, N = 12000
// 64.7, 65.6, 55.5 against 58.3, 52.4, 50.9.
//
// VEC (full layout, D 16-byte aligned, ldd a multiple of 4): a lane owns
// four consecutive columns and each non-temporal 16-byte store writes a 1 KB
// row segment.  Otherwise rows start at any 4-byte boundary: a lane owns
// columns l, l + 64, l + 128, l + 192, each plain 4-byte store instruction
// writes 256 contiguous bytes, and the lines shared by neighbouring segments
// meet in L2 (neighbours in w are on one XCD); non-temporal stores would
// reach memory as partial lines (store-only, full layout: 395 against
// 345 us).  The row points are wave-uniform (scalar loads), and there is no
// LDS traffic and no barrier.
//
// What bounds it is the write stream, whose rate falls with the bytes that
// are being written at a time.  Store-only copies of the launch on the 30000
// points' triangle (1.8 GB): 325, 309, 292 and 319 us for one row of 1024
// columns per work-group at 8, 6, 5 and 4 work-groups per CU (full layout);
// a linear fill of as many bytes as the cells takes 253 to 270 us.  Hence the
// wide, low strips, and hence fewer work-groups per CU than would fit, by
// dynamic LDS that no thread uses, once the output is large (kCached).
// One row per wave loses more to the loads of its column points, which then
// serve four cells per lane, than it gains: 342 (full) and 360 us (packed)
// against 292 and 271.
// Measured at N = 30000 (us; before: 256-column strips of 8 rows at full
// residency, and 256-cell tiles for an unaligned full layout), d = 1, 2, 3, 4:
//   full                312 311 292 291   before 326 330 328 331
//   full, ldd odd       350   - 350 353   before 828 829 837 844
//   packed              272 271 271 272   before 286 288 278 292
// and at other sizes (us), full residency / kPerCu, d = 1, 3:
//   full, N = 8192      22.9 / 24.8   23.1 / 23.0
//   full, N = 11585     58.6 / 54.4   59.2 / 56.1
//   full, N = 46000     722 / 705     712 / 656
//   packed, N = 5793    13.5 / 13.5   13.7 / 13.5
//   packed, N = 16384   87.9 / 86.2   89.1 / 87.6
//   packed, N = 46000   651 / 644     629 / 614
//
// Up to kBandNarrow the aligned full layout takes strips of 256 columns: a
// small output pays for the upper half of wide diagonal tiles and for the
// longer column loads at its start.  256 against 1024 columns (d = 4: 512), d =
// 1, 2, 3, 4: N = 2100 4.1 4.1 4.2 4.5 against 4.6 4.3 4.3 4.6 us; 4097 8.3 8.3
// 8.5 9.2 against 9.5 8.4 8.6 9.5; beyond the line, 5000 12.0 12.0 12.0 12.4
// against 11.4 11.8 12.0 12.5.
//
// LTM leaves out the strips past the last point, up to a whole tile row less
// one strip (a fifth of the launch at 7200 points in 1024-column tiles).  With /
// without them, d = 1, 3: full, N = 4097 (1024 columns) 11.4 / 9.5 and 10.1 /
// 8.6 us, N = 6400 20.9 / 18.1 and 18.7 / 16.2; packed, N = 7200 19.7 / 17.7 and
// 19.9 / 18.0, N = 40000 494 / 484 and 489 / 480.  The aligned full layout keeps
// them above kBandWhole, where they leave the last of the eight XCDs with less
// to write and the others write faster: N = 9217 35.2 / 36.7 and 35.2 / 37.5,
// N = 22000 173 / 169 and 159 / 165, N = 8500 30.7 / 30.0 and 30.9 / 30.8.
template <int LAYOUT, bool VEC, int D, bool SMALL>
struct BandShape {
  // The strip is widest where rows are written end to end; packed rows are
  // adjacent, and unaligned full rows gain nothing from width.  At d = 4 the
  // column points of 1024 columns cost more than the width gives.  SMALL: see
  // above.
  static constexpr int W = VEC ? (SMALL ? 256 : D == 4 ? 512 : 1024) : (LAYOUT == kLayoutFull ? 256 : 512);
  static constexpr int kAcross = W / 256;     // waves across a strip
  static constexpr int kDown = 4 / kAcross;   // rows written at a time
  static constexpr int kRows = 2;             // rows per wave
  static constexpr int H = kDown * kRows;
  static constexpr int S = W / H;
  // work-groups per CU for a large output: fewer where a work-group's loads
  // (D floats per column) are over sooner
  static constexpr int kPerCu = VEC ? (D == 4 ? 6 : 4) : (LAYOUT == kLayoutFull ? 8 : (D <= 2 ? 6 : 7));
  // cells (bytes) from which they are fewer, N = 5793 or (d = 1, whose four
  // work-groups lose more up to there) 8689: see above
  static constexpr uint64_t kCached = (uint64_t)(VEC && D == 1 ? 144 : 64) << 20;
  // 160 KB of LDS in 2 KB steps, kPerCu to 8 work-groups of it
  static constexpr int kIdleLds = kPerCu == 8 ? 0 : (160 / kPerCu / 2 * 2 - 1) * 1024;
};
// Lines of the rules, in bytes of cells (4 N (N + 1) / 2).
constexpr uint64_t kBandNarrow = (uint64_t)40 << 20;  // N = 4579
constexpr uint64_t kBandWhole = (uint64_t)144 << 20;  // N = 8689
static uint64_t band_bytes(const EdmArgs &a) { return 2 * (uint64_t)a.N * ((uint64_t)a.N + 1); }

template <int D, int LAYOUT, bool VEC, bool SMALL, bool BB, bool DENSE>
__global__ __launch_bounds__(256) void edm_band_kernel(const float *__restrict__ X, uint32_t N,
                                                       int64_t ldx_, float *__restrict__ out,
                                                       int64_t ldd, uint32_t w0) {
  using B = BandShape<LAYOUT, VEC, D, SMALL>;
  constexpr uint32_t S = B::S;
  const int64_t ldx = DENSE ? D : ldx_;
  uint32_t I, J, k;
  if constexpr (BB) {
    I = blockIdx.y;
    const uint32_t cols = gridDim.y | 1;
    k = blockIdx.x / cols;
    J = blockIdx.x - k * cols;
    if (J > I) return;
  } else {
    const uint32_t w = w0 + xcd_contiguous(blockIdx.x, gridDim.x);
    uint32_t Jt;
    g_lambda_uniform(w / S, I, Jt);
    k = div_uniform(S * Jt + w % S, I + 1, J);
  }
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t l = threadIdx.x & 63;
  // the wave's first row and first column
  const uint32_t row0 = I * B::W + k * B::H + wv / B::kAcross;
  const uint32_t c = J * B::W + wv % B::kAcross * 256;
  const float *__restrict__ Xc = X + (uint64_t)c * (uint64_t)ldx;
  // the lane's columns, relative to c
  auto col = [&](int q) -> uint32_t { return VEC ? 4 * l + q : l + 64 * q; };
  auto load = [&](uint32_t j, float (&x)[D]) {
#pragma unroll
    for (int m = 0; m < D; ++m) x[m] = DENSE ? Xc[j * D + m] : Xc[(uint64_t)j * (uint64_t)ldx + m];
  };
  float xj[4][D];
  if (J < I && row0 + (B::kRows - 1) * B::kDown < N) {
#pragma unroll
    for (int q = 0; q < 4; ++q) load(col(q), xj[q]);
#pragma unroll
    for (int r = 0; r < B::kRows; ++r) {
      const uint32_t i = row0 + B::kDown * r;
      const float *__restrict__ Xi = X + (uint64_t)i * (uint64_t)ldx;
      float xi[D];
#pragma unroll
      for (int m = 0; m < D; ++m) xi[m] = Xi[m];
      float *__restrict__ o = out + out_index<LAYOUT>((uint64_t)i, (uint64_t)c, ldd);
      if constexpr (VEC) {
        f4 v;
        v.x = pair_dist<D>(xi, xj[0]);
        v.y = pair_dist<D>(xi, xj[1]);
        v.z = pair_dist<D>(xi, xj[2]);
        v.w = pair_dist<D>(xi, xj[3]);
        __builtin_nontemporal_store(v, reinterpret_cast<f4 *>(o + 4 * l));
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) o[l + 64 * q] = pair_dist<D>(xi, xj[q]);
      }
    }
    return;
  }
  // diagonal or edge strip: rows below N, cells of the triangle (columns
  // past the last point are read as the last point, and not written)
  if (c >= N) return;
  const uint32_t room = N - 1 - c;
#pragma unroll
  for (int q = 0; q < 4; ++q) load(col(q) < room ? col(q) : room, xj[q]);
#pragma unroll
  for (int r = 0; r < B::kRows; ++r) {
    const uint32_t i = row0 + B::kDown * r;
    if (i >= N || c > i) continue;
    const float *__restrict__ Xi = X + (uint64_t)i * (uint64_t)ldx;
    float xi[D], v[4];
#pragma unroll
    for (int m = 0; m < D; ++m) xi[m] = Xi[m];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = pair_dist<D>(xi, xj[q]);
    float *__restrict__ o = out + out_index<LAYOUT>((uint64_t)i, (uint64_t)c, ldd);
    if (VEC && in_triangle<LAYOUT>(i, c + 4 * l + 3)) {
      const f4 v4 = {v[0], v[1], v[2], v[3]};
      __builtin_nontemporal_store(v4, reinterpret_cast<f4 *>(o + 4 * l));
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (in_triangle<LAYOUT>(i, c + col(q))) o[col(q)] = v[q];
    }
  }
}

template <int D, int LAYOUT, bool VEC, bool SMALL, bool DENSE>
static hipError_t launch_band_t(bool bb, const EdmArgs &a) {
  using B = BandShape<LAYOUT, VEC, D, SMALL>;
  const uint64_t N = (uint64_t)a.N;
  const uint64_t nb = (N + B::W - 1) / B::W;
  const uint32_t lds = band_bytes(a) >= B::kCached ? B::kIdleLds : 0;
  if (bb) {
    hipLaunchKernelGGL((edm_band_kernel<D, LAYOUT, VEC, SMALL, true, DENSE>),
                       dim3((uint32_t)(B::S * (nb | 1)), (uint32_t)nb), dim3(256), lds, a.stream, a.X,
                       (uint32_t)a.N, a.ldx, a.D, a.ldd, 0u);
    return hipGetLastError();
  }
  // strips of the last tile row: those past the last point end the range of w
  // and are left out, except from a large aligned full output
  const uint64_t left = N - (nb - 1) * B::W;
  const uint64_t last = VEC && band_bytes(a) >= kBandWhole ? B::S : (left + B::H - 1) / B::H;
  const uint64_t W = B::S * (nb * (nb - 1) / 2) + last * nb;
  if (W > 0xffffffffull) return hipErrorInvalidValue;  // w is 32-bit (N above 4 million)
  uint64_t lo, hi;
  shard_range(W, a.shard, a.nshards, lo, hi);
  const uint64_t max_blocks = (((uint64_t)1 << 32) - 1) / 256;
  for (uint64_t w0 = lo; w0 < hi; w0 += max_blocks) {
    const uint64_t c = hi - w0 < max_blocks ? hi - w0 : max_blocks;
    hipLaunchKernelGGL((edm_band_kernel<D, LAYOUT, VEC, SMALL, false, DENSE>), dim3((uint32_t)c), dim3(256), lds,
                       a.stream, a.X, (uint32_t)a.N, a.ldx, a.D, a.ldd, (uint32_t)w0);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int D, int LAYOUT, bool VEC>
static hipError_t launch_band(bool bb, const EdmArgs &a) {
  const bool dense = a.ldx == D;
  if (VEC && band_bytes(a) < kBandNarrow)
    return dense ? launch_band_t<D, LAYOUT, VEC, VEC, true>(bb, a) : launch_band_t<D, LAYOUT, VEC, VEC, false>(bb, a);
  return dense ? launch_band_t<D, LAYOUT, VEC, false, true>(bb, a) : launch_band_t<D, LAYOUT, VEC, false, false>(bb, a);
}

template <int TS, int D, int LAYOUT, bool VEC>
static hipError_t launch_tiled_t(bool bb, const EdmArgs &a) {
  if constexpr (TS == 256) {
    return launch_band<D, LAYOUT, VEC>(bb, a);
  } else {
    const uint64_t nb = (uint64_t)((a.N + TS - 1) / TS);
    if (bb) {
      hipLaunchKernelGGL((edm_tile_kernel<TS, D, LAYOUT, VEC, true>),
                         dim3((uint32_t)nb, (uint32_t)nb), dim3(256), 0, a.stream, a, 0u);
      return hipGetLastError();
    }
    const uint64_t T = nb * (nb + 1) / 2;
    uint64_t lo, hi;
    shard_range(T, a.shard, a.nshards, lo, hi);
    const uint64_t max_blocks = (((uint64_t)1 << 32) - 1) / 256;
    for (uint64_t l0 = lo; l0 < hi; l0 += max_blocks) {
      const uint64_t c = hi - l0 < max_blocks ? hi - l0 : max_blocks;
      hipLaunchKernelGGL((edm_tile_kernel<TS, D, LAYOUT, VEC, false>), dim3((uint32_t)c), dim3(256),
                         0, a.stream, a, (uint32_t)l0);
      hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
}

template <int TS, int D>
static hipError_t launch_tiled_d(bool bb, const EdmArgs &a) {
  if (a.layout == kLayoutPacked) return launch_tiled_t<TS, D, kLayoutPacked, false>(bb, a);
  if (a.layout == kLayoutStrict) return launch_tiled_t<TS, D, kLayoutStrict, false>(bb, a);
  const bool aligned = (a.ldd % 4 == 0) && ((reinterpret_cast<uintptr_t>(a.D) & 15) == 0);
  return aligned ? launch_tiled_t<TS, D, kLayoutFull, true>(bb, a)
                 : launch_tiled_t<TS, D, kLayoutFull, false>(bb, a);
}

template <int TS>
static hipError_t launch_tiled_ts(bool bb, const EdmArgs &a) {
  switch (a.d) {
    case 1: return launch_tiled_d<TS, 1>(bb, a);
    case 2: return launch_tiled_d<TS, 2>(bb, a);
    case 3: return launch_tiled_d<TS, 3>(bb, a);
    case 4: return launch_tiled_d<TS, 4>(bb, a);
    default: return hipErrorInvalidValue;
  }
}

bool tiled_supported(int ts, int d) {
  return (ts == 64 || ts == 128 || ts == 256) && d >= 1 && d <= 4;
}

hipError_t launch_tiled(bool bb, int ts, const EdmArgs &a) {
  if (a.N == 0) return hipSuccess;
  switch (ts) {
    case 64: return launch_tiled_ts<64>(bb, a);
    case 128: return launch_tiled_ts<128>(bb, a);
    case 256: return launch_tiled_ts<256>(bb, a);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace tdmap
