// Packed-layout EDM as a linear sweep of the output.
//
// In the packed layout the index of cell (i, j) is i(i+1)/2 + j, which is
// exactly the block index lambda of Sec. II-A, Eq. (1) for blocks of one
// cell.  So g(lambda) with rho = 1 maps every output position back to its
// cell, and the output can be written in address order: each thread owns
// four consecutive positions (one aligned 16-byte store) and each
// work-group 1024 consecutive positions.  The map runs once per wave (a
// wave's 256 positions span at most a couple of rows); each lane then
// steps from the wave's first cell to its own.
//
// Without the diagonal (strict layout, index i(i-1)/2 + j, j < i) the same
// sweep maps positions with the paper's no-diagonal map (Sec. II-A,
// Eq. (10)); row i then holds i cells instead of i + 1.
//
// The batched variant sweeps the concatenation of every set's packed
// triangle; positions past the end of a set continue in the next one.  Its
// work-groups each own one contiguous stretch of the output and read the
// points of a set from LDS.
#include "device.h"
#include "kernels.h"

namespace tdmap {

typedef float f4 __attribute__((ext_vector_type(4)));

// g(lambda) for 64-bit lambda (packed indices pass 2^32 at N = 92682).  The
// single-precision guess of the row is within one for lambda < 2^40; the
// bounded loops make the result exact.
__device__ __forceinline__ void g_lambda64(uint64_t lam, uint64_t &i, uint64_t &j) {
  const float x = __builtin_fmaf(2.0f, (float)lam, 0.25f);
  const float s = x * __builtin_amdgcn_rsqf(x);
  uint64_t r = (uint64_t)__builtin_fmaxf(s - 0.5f, 0.0f);
  uint64_t t = tri64(r);
  while (t > lam) {
    --r;
    t -= r + 1;
  }
  while (t + r + 1 <= lam) {
    t += r + 1;
    ++r;
  }
  i = r;
  j = lam - t;
}

// Eq. (10) for 64-bit lambda: row i starts at S(i) = i(i-1)/2.
__device__ __forceinline__ void g_nodiag64(uint64_t lam, uint64_t &i, uint64_t &j) {
  const float x = __builtin_fmaf(2.0f, (float)lam, 0.25f);
  const float s = x * __builtin_amdgcn_rsqf(x);
  uint64_t r = (uint64_t)(s + 0.5f);
  if (r == 0) r = 1;
  uint64_t t = (r * (r - 1)) >> 1;
  while (t > lam) {
    --r;
    t -= r;
  }
  while (t + r <= lam) {
    t += r;
    ++r;
  }
  i = r;
  j = lam - t;
}

template <int D>
__device__ __forceinline__ void load_pt(const float *__restrict__ X, int64_t ldx, uint64_t p,
                                        float (&v)[D]) {
#pragma unroll
  for (int k = 0; k < D; ++k) v[k] = X[p * ldx + k];
}

// Column point c of a uniform base, addressed by a 32-bit byte offset
// (c * row_bytes < 2^32 is checked by the caller): the load then takes a
// scalar base and one vector offset, with no 64-bit index arithmetic.
template <int D>
__device__ __forceinline__ void load_pt32(const float *__restrict__ X, uint32_t row_bytes,
                                          uint32_t c, float (&v)[D]) {
  const float *p = reinterpret_cast<const float *>(reinterpret_cast<const char *>(X) + c * row_bytes);
#pragma unroll
  for (int k = 0; k < D; ++k) v[k] = p[k];
}

// One wave writes SW_G consecutive 1 KB pieces (SW_G float4 stores per
// lane, each covering 256 consecutive positions).  When the wave's first
// cell lies in a row of at least SW_G * 256 cells, its positions cover at
// most two rows: the two row points are uniform (scalar loads) and every
// column point load is issued before any arithmetic, so one memory latency
// covers the whole 4 KB.  Short rows (the first few hundred) and the tail
// of the array take a per-lane stepping path.
constexpr int SW_G = 4;
constexpr int SW_WAVE = 256 * SW_G;       // positions per wave
constexpr int SW_BLOCK = 4 * SW_WAVE;     // positions per work-group

// OFF32: contiguous points (ldx == D) and N * D * 4 < 2^32, so a column
// offset is a 32-bit multiple of the constant D * 4.
template <int D, bool STRICT, bool OFF32>
__global__ __launch_bounds__(256) void edm_sweep_kernel(const float *__restrict__ X, int64_t N,
                                                        int64_t ldx, float *__restrict__ out,
                                                        uint64_t total, uint64_t e_base) {
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint64_t ew = e_base + (uint64_t)blockIdx.x * SW_BLOCK + (uint64_t)w * SW_WAVE;
  if (ew >= total) return;
  // cells in row i
  auto row_len = [](uint64_t i) -> uint64_t { return STRICT ? i : i + 1; };
  uint64_t iw, jw;
  if constexpr (STRICT)
    g_nodiag64(ew, iw, jw);
  else
    g_lambda64(ew, iw, jw);
  const uint32_t l = threadIdx.x & 63;
  const uint64_t len_w = row_len(iw);
  if (len_w >= (uint64_t)SW_WAVE && ew + SW_WAVE <= total) {
    const uint64_t i1 = iw + 1 < (uint64_t)N ? iw + 1 : iw;  // row below (may be unused)
    float xa[D], xb[D];
    load_pt<D>(X, ldx, iw, xa);
    load_pt<D>(X, ldx, i1, xb);
    float xj[SW_G][4][D];
    bool lo[SW_G][4];
#pragma unroll
    for (int g = 0; g < SW_G; ++g)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if constexpr (OFF32) {
          // every column is below N < 2^31
          const uint32_t j = (uint32_t)jw + 256 * g + 4 * l + q;
          lo[g][q] = j < (uint32_t)len_w;
          load_pt32<D>(X, D * 4u, lo[g][q] ? j : j - (uint32_t)len_w, xj[g][q]);
        } else {
          const uint64_t j = jw + 256 * g + 4 * l + q;
          lo[g][q] = j < len_w;
          load_pt<D>(X, ldx, lo[g][q] ? j : j - len_w, xj[g][q]);
        }
      }
#pragma unroll
    for (int g = 0; g < SW_G; ++g) {
      f4 o;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float xi[D];
#pragma unroll
        for (int k = 0; k < D; ++k) xi[k] = lo[g][q] ? xa[k] : xb[k];
        o[q] = pair_dist<D>(xi, xj[g][q]);
      }
      __builtin_nontemporal_store(o, reinterpret_cast<f4 *>(out + ew + 256 * g + 4 * l));
    }
    return;
  }
  // general path: each lane steps from the wave's first cell to its own
  for (int g = 0; g < SW_G; ++g) {
    const uint64_t e0 = ew + 256 * g + 4 * l;
    if (e0 >= total) break;
    uint64_t i = iw, j = jw + 256 * g + 4 * l;
    while (j >= row_len(i)) {
      j -= row_len(i);
      ++i;
    }
    float xi[D];
    load_pt<D>(X, ldx, i, xi);
    float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (e0 + q >= total) break;
      if (j >= row_len(i)) {  // next row
        ++i;
        j = 0;
        load_pt<D>(X, ldx, i, xi);
      }
      float xj[D];
      load_pt<D>(X, ldx, j, xj);
      v[q] = pair_dist<D>(xi, xj);
      ++j;
    }
    if (e0 + 4 <= total) {
      f4 o = {v[0], v[1], v[2], v[3]};
      __builtin_nontemporal_store(o, reinterpret_cast<f4 *>(out + e0));
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (e0 + q < total) __builtin_nontemporal_store(v[q], out + e0 + q);
    }
  }
}

// Batched: the positions [out_off[0], out_off[S]) of the concatenated packed
// triangles.  A persistent grid of kBatchWgsPerCu 1024-thread work-groups per
// CU: work-group b of G owns the units [U b / G, U (b + 1) / G) of kBatchUnit
// positions, one contiguous stretch of the output, and walks it in chunks
// whose points it stages in LDS.  No wait for a global load then stands between
// a chunk's stores (vmcnt counts loads and stores alike, and a wait for a load
// waits for every store issued before it); what they do wait for is
// kBatchPending.  The chunks:
//   - a full chunk inside one set: the set's points, staged once when the walk
//     enters the set, 16 positions per lane in an unrolled loop;
//   - anything else (the end of a set, sets smaller than a chunk, the end of
//     the stretch): up to kBatchMulti positions over as many sets as the table
//     and the points' LDS hold.  Consecutive sets' points are adjacent in X,
//     so one pass of loads stages them all; each lane finds the set of its
//     first position by a search of the table in LDS, follows the table from
//     there, and maps every position on its own.
// A set too large for LDS maps each position on its own and reads global
// memory.  Lane l of wave w writes positions l + 64 q of the wave's stretch of
// the chunk: each 4-byte store instruction covers 256 contiguous bytes.
// Measured (us, d = 3): 3000 sets of 0 to 139 points 17.7 (57 when each
// position outside a full chunk searched its set and read global memory; the
// 64-cell tiles 40 with their prefix sums); 4096 sets of 8 to 32 points under
// 10.7, the time to issue the call (107); 500 sets of 250 to 1000 points 101
// (112); 1024 sets of 64 to 4096 points 2207 (2269; 1830 and 1928 where the
// output lies better), bound by the write rate of a persistent grid.
constexpr int kBatchThreads = 1024;
constexpr int kBatchPer = 16;                           // positions per lane per chunk
constexpr int kBatchChunk = kBatchThreads * kBatchPer;  // 16384 positions
constexpr int kBatchQuarter = kBatchChunk / 4;
constexpr int kBatchMulti = 2 * kBatchChunk;
constexpr int kBatchUnit = kBatchThreads;
constexpr int kBatchTable = kBatchThreads;              // sets of a chunk
constexpr int kBatchLdsFloats = 16384;                  // 64 KB
constexpr int kBatchWgsPerCu = 2;
// Stores a wave leaves unfinished when it goes on to the next (vmcnt): the
// write rate falls with the bytes that are being written at a time, and 32
// waves a CU with 16 stores of 256 bytes each would have 128 KB.  All on the
// same buffers in one process, us, no wait / 0, 1, 2, 3, 4, 8 stores (spread 1 %):
//   1024 sets of 64 to 4096 points, d = 1  2258 / 2266 2200 2199 2218 2237 2243
//                                   d = 2  2252 / 2270 2213 2197 2223 2250 2249
//                                   d = 3  2281 / 2296 2219 2209 2237 2264 2284
//                                   d = 4  2300 / 2330 2239 2225 2253 2285 2309
//   64 sets of 4096 points, d = 3           430 /  426  413  411  415  424  430
//   300 sets of 3000 points, d = 3         1067 / 1078 1049 1043 1050 1066 1065
//   500 sets of 250 to 1000 points, d = 3   103 /  105  102  102  103  103  103
constexpr int kBatchPending = 2;

// A point from LDS.  Four floats start on 16 bytes (points sit on multiples
// of D floats of an aligned area), which the compiler cannot see: read float
// by float the lanes' points meet in a quarter of the banks.  d = 4, 1024 sets
// of 64 to 4096 points 2471 us, 2236 as one read; 3000 of 0 to 139 19.0, 16.4.
template <int D>
__device__ __forceinline__ void lds_pt(const float *p, float (&v)[D]) {
  if constexpr (D == 4) {
    const f4 x = *reinterpret_cast<const f4 *>(p);
#pragma unroll
    for (int k = 0; k < D; ++k) v[k] = x[k];
  } else {
#pragma unroll
    for (int k = 0; k < D; ++k) v[k] = p[k];
  }
}

// PER x 1024 positions inside one set, from its position lam on; xp: the
// set's points in LDS, o: the position's cell.  The walk keeps the LDS
// offsets iD = i D and jD = j D (additions only; j > i is jD > iD, and a row
// of i + 1 cells is (i + 1) D floats).
template <int D, int PER>
__device__ __forceinline__ void set_chunk(const float *xp, uint32_t lam, float *__restrict__ o, uint32_t w,
                                          uint32_t l) {
  const uint32_t off = w * (64 * PER) + l;
  uint32_t i, j;
  g_lambda_small(lam + off, i, j);
  uint32_t iD = i * D, jD = j * D;
  float xi[D], xj[D];
  lds_pt<D>(xp + iD, xi);
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    if (q > 0) {
      jD += 64 * D;
      if (jD > iD) {
        do {
          iD += D;
          jD -= iD;
        } while (jD > iD);
        lds_pt<D>(xp + iD, xi);
      }
    }
    lds_pt<D>(xp + jD, xj);
    __builtin_nontemporal_store(pair_dist<D>(xi, xj), o + off + 64 * q);
    __builtin_amdgcn_s_waitcnt(0x0F70 | kBatchPending);
  }
}

template <int D>
__global__ __launch_bounds__(kBatchThreads, 8) void edm_batched_sweep_kernel(
    const float *__restrict__ X, const int64_t *__restrict__ point_off,
    const int64_t *__restrict__ oo, int32_t S, float *__restrict__ out) {
  // The table of a chunk comes first, within the reach of an instruction's
  // 16-bit offset: behind the points each array takes an address register of
  // its own, and d = 4 spills one (the reload waits for every store).
  struct Lds {
    // first position of each set (relative to the chunk's first; one more entry
    // ends the last) and its points' place in xs
    int32_t tab_o[kBatchTable + 1];
    int32_t tab_p[kBatchTable];
    __align__(16) float xs[kBatchLdsFloats];
  };
  __shared__ Lds lds;
  auto &xs = lds.xs;
  auto &tab_o = lds.tab_o;
  auto &tab_p = lds.tab_p;
  const uint64_t first = (uint64_t)oo[0];
  const uint64_t total = (uint64_t)oo[S];
  const uint64_t units = (total - first + kBatchUnit - 1) / kBatchUnit;
  const uint64_t G = gridDim.x;
  const uint64_t u0 = units * blockIdx.x / G, u1 = units * (blockIdx.x + 1) / G;
  if (u0 == u1) return;
  const uint64_t end = first + u1 * kBatchUnit < total ? first + u1 * kBatchUnit : total;
  uint64_t e = first + u0 * kBatchUnit;
  const uint32_t t = threadIdx.x;
  const uint32_t w = __builtin_amdgcn_readfirstlane(t >> 6), l = t & 63;

  // s: the largest set with out_off[s] <= e (so a set with cells), found by
  // all threads at once, 1024 candidates a round
  int32_t s = 0;
  for (int32_t n = S; n > 1;) {
    const int32_t step = (n + kBatchThreads - 1) / kBatchThreads;
    const int64_t k = (int64_t)t * step;
    const int32_t at = __syncthreads_count(k < n && (uint64_t)oo[s + k] <= e) - 1;
    s += at * step;
    n = n - at * step < step ? n - at * step : step;
  }
  // xs holds the points [have0, have1)
  int64_t have0 = 0, have1 = 0;
  // makes it hold [q0, q1), keeping what is there if both fit; the caller has
  // passed a barrier since the last use of xs and passes one before the next
  auto stage = [&](int64_t q0, int64_t q1) {
    if (q0 >= have0 && q1 <= have1) return;
    int64_t from = have1;
    if (q0 < have0 || q0 > have1 || q1 - have0 > kBatchLdsFloats / D) have0 = from = q0;
    // eight loads in flight per thread
    const float *__restrict__ src = X + from * D;
    float *dst = xs + (int)(from - have0) * D;
    const int len = (int)(q1 - from) * D;
    for (int m0 = (int)t; m0 < len; m0 += 8 * kBatchThreads) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (m0 + u * kBatchThreads < len) v[u] = src[m0 + u * kBatchThreads];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (m0 + u * kBatchThreads < len) dst[m0 + u * kBatchThreads] = v[u];
    }
    have1 = q1;
  };
  // set s: its positions [s_beg, s_end), first point and number of points
  uint64_t s_beg, s_end;
  int64_t p0, n;
  auto enter = [&]() {
    s_beg = (uint64_t)oo[s];
    s_end = (uint64_t)oo[s + 1];
    p0 = point_off[s];
    n = point_off[s + 1] - p0;
  };
  // goes on to the set of position e if it is not s
  auto advance = [&]() {
    if (e >= end || e < s_end) return;
    do ++s;
    while ((uint64_t)oo[s + 1] <= e);  // past empty sets
    enter();
  };
  enter();
  while (e < end) {
    // chunks end on units: a full chunk's 256-byte stores then cover whole
    // lines (non-temporal stores of split lines cost 1.3 times the time)
    const uint32_t past = (uint32_t)(e - first) % kBatchUnit;
    const uint64_t inside = s_end < end ? s_end : end;
    // what the full chunks of set s may take (a set smaller than a chunk
    // shares one with its neighbours)
    const uint64_t room = s_end - s_beg >= kBatchChunk && n <= kBatchLdsFloats / D ? inside - e : 0;
    if (past == 0 && room >= kBatchQuarter) {
      if (p0 < have0 || p0 + n > have1) {
        __syncthreads();  // every wave is done with the previous points
        stage(p0, p0 + n);
        __syncthreads();
      }
      const float *xp = xs + (uint32_t)(p0 - have0) * D;
      if (room >= kBatchChunk) {
        set_chunk<D, kBatchPer>(xp, (uint32_t)(e - s_beg), out + e, w, l);
        e += kBatchChunk;
      } else {
        set_chunk<D, kBatchPer / 4>(xp, (uint32_t)(e - s_beg), out + e, w, l);
        e += kBatchQuarter;
      }
      advance();
      continue;
    }
    // as many sets from s on as start before the limit and fit; the limit is
    // the next unit if full chunks of set s follow, the one after the end of
    // set s if full chunks of the next set do
    uint64_t lim = e - past + kBatchMulti;
    if (room >= kBatchUnit - past + kBatchQuarter)
      lim = e - past + kBatchUnit;
    else if (s + 2 <= S && (uint64_t)oo[s + 2] - s_end >= (uint64_t)(kBatchChunk + kBatchUnit))
      lim = s_end + (kBatchUnit - 1 - (s_end - first + kBatchUnit - 1) % kBatchUnit);
    if (lim > end) lim = end;
    const int64_t k = (int64_t)s + t;
    int64_t o = 0, o1 = 0, p = 0, p1 = 0;
    bool fits = false;
    if (k < S) {
      o = oo[k];
      o1 = oo[k + 1];
      p = point_off[k];
      p1 = point_off[k + 1];
      fits = (uint64_t)o < lim && p1 - p0 <= kBatchLdsFloats / D;
    }
    const int32_t count = __syncthreads_count(fits);
    if (count == 0) {
      // set s is too large for LDS
      const uint64_t stop = s_end < lim ? s_end : lim;
      const float *__restrict__ Xl = X + p0 * D;
      for (uint64_t pos = e + t; pos < stop; pos += kBatchThreads) {
        uint64_t i, j;
        g_lambda64(pos - s_beg, i, j);
        float xi[D], xj[D];
        load_pt<D>(Xl, D, i, xi);
        load_pt<D>(Xl, D, j, xj);
        __builtin_nontemporal_store(pair_dist<D>(xi, xj), out + pos);
      }
      e = stop;
      advance();
      continue;
    }
    stage(p0, point_off[s + count]);
    if ((int32_t)t < count) {
      tab_o[t] = (int32_t)(o - (int64_t)e);
      tab_p[t] = (int32_t)(p - have0);
      if ((int32_t)t == count - 1) tab_o[count] = (int32_t)(o1 - (int64_t)e);
    }
    __syncthreads();
    const uint64_t last = (uint64_t)oo[s + count];
    const int32_t len = (int32_t)((last < lim ? last : lim) - e);
    // the lanes sit on multiples of 64 positions, the first of them up to 63
    // before e
    const int32_t shift = (int32_t)(past % 64);
    const int32_t per = (len + shift + kBatchThreads - 1) / kBatchThreads;
    const int32_t begin = (int32_t)(w * 64) * per - shift;
    const int32_t stop = begin + 64 * per < len ? begin + 64 * per : len;
    int32_t pos = begin + (int32_t)l;
    if (pos < 0) pos += 64;
    if (pos < stop) {
      int32_t a = 0, b = count;  // largest a with tab_o[a] <= pos
      while (b - a > 1) {
        const int32_t mid = (a + b) >> 1;
        if (tab_o[mid] <= pos) a = mid; else b = mid;
      }
      float *__restrict__ op = out + e;
      int32_t beg = tab_o[a], next = tab_o[a + 1];
      const float *xp = xs + (uint32_t)tab_p[a] * D;
      // four positions at a time, each mapped on its own: no step waits for
      // the one before it (rows are short here, so stepping from row to row
      // would loop, and lanes would wait for one another)
      constexpr int R = 4;
      for (; pos < stop; pos += 64 * R) {
        float xi[R][D], xj[R][D];
#pragma unroll
        for (int u = 0; u < R; ++u) {
          // (past the stretch: its last position, not stored)
          const int32_t at = pos + 64 * u < stop ? pos + 64 * u : stop - 1;
          if (at >= next) {
            do {
              ++a;
              beg = next;
              next = tab_o[a + 1];
            } while (next <= at);
            xp = xs + (uint32_t)tab_p[a] * D;
          }
          uint32_t i, j;
          g_lambda_small((uint32_t)(at - beg), i, j);
          lds_pt<D>(xp + i * D, xi[u]);
          lds_pt<D>(xp + j * D, xj[u]);
        }
#pragma unroll
        for (int u = 0; u < R; ++u)
          if (pos + 64 * u < stop)
            __builtin_nontemporal_store(pair_dist<D>(xi[u], xj[u]), op + pos + 64 * u);
      }
    }
    e += (uint64_t)len;
    if (count > 1) {
      s += count - 1;  // the last set of the chunk
      enter();
    }
    advance();
  }
}

template <int D, bool STRICT, bool OFF32>
static hipError_t launch_sweep_t(const EdmArgs &a) {
  const uint64_t total = STRICT ? (uint64_t)a.N * (uint64_t)(a.N - 1) / 2
                                : (uint64_t)a.N * (uint64_t)(a.N + 1) / 2;
  const uint64_t per_launch = (uint64_t)SW_BLOCK * (((uint64_t)1 << 31) / 256);
  for (uint64_t b = 0; b < total; b += per_launch) {
    const uint64_t c = total - b < per_launch ? total - b : per_launch;
    hipLaunchKernelGGL((edm_sweep_kernel<D, STRICT, OFF32>), dim3((uint32_t)((c + SW_BLOCK - 1) / SW_BLOCK)),
                       dim3(256), 0, a.stream, a.X, a.N, a.ldx, a.D, b + c, b);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int D>
static hipError_t launch_sweep_d(const EdmArgs &a) {
  const bool strict = a.layout == kLayoutStrict;
  const bool off32 = a.ldx == D && (uint64_t)a.N * D * 4u < ((uint64_t)1 << 32);
  if (strict)
    return off32 ? launch_sweep_t<D, true, true>(a) : launch_sweep_t<D, true, false>(a);
  return off32 ? launch_sweep_t<D, false, true>(a) : launch_sweep_t<D, false, false>(a);
}

bool sweep_supported(const EdmArgs &a) {
  return (a.layout == kLayoutPacked || a.layout == kLayoutStrict) && a.d >= 1 && a.d <= 4 &&
         (reinterpret_cast<uintptr_t>(a.D) & 15) == 0;
}

hipError_t launch_sweep(const EdmArgs &a) {
  if (a.N == 0) return hipSuccess;
  switch (a.d) {
    case 1: return launch_sweep_d<1>(a);
    case 2: return launch_sweep_d<2>(a);
    case 3: return launch_sweep_d<3>(a);
    case 4: return launch_sweep_d<4>(a);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_batched_sweep(const BatchArgs &a) {
  if (a.num_sets == 0) return hipSuccess;
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      cus <= 0)
    cus = 256;
  const dim3 grid((uint32_t)(cus * kBatchWgsPerCu));
#define TD_BSWEEP(DD)                                                                          \
  hipLaunchKernelGGL(edm_batched_sweep_kernel<DD>, grid, dim3(kBatchThreads), 0, a.stream, a.X, \
                     a.point_off, a.out_off, a.num_sets, a.D)
  switch (a.d) {
    case 1: TD_BSWEEP(1); break;
    case 2: TD_BSWEEP(2); break;
    case 3: TD_BSWEEP(3); break;
    case 4: TD_BSWEEP(4); break;
    default: return hipErrorInvalidValue;
  }
#undef TD_BSWEEP
  return hipGetLastError();
}

}  // namespace tdmap
