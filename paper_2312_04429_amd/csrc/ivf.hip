// Inverted-file (IVF) approximate search over the cached prompt embeddings:
// the indexed vector-DB search the paper's system runs (Sec. 5.3, Sec. 6),
// built and searched on the GPU.  The rows are partitioned into L lists
// around unit centroids; a query ranks the lists by its score against their
// centroids and scans the rows of the best nprobe.
//
// Every score is the canonical one of the exact lookup (float64 sum of exact
// products, left to right), every order is total (ties to the lower list /
// row), and the centroid update sums in a fixed order, so an index and each
// search result are reproducible bit for bit.
//   build:  centroids = rows at caller-drawn indices; `iters` Lloyd steps
//           (assign every row with the exact lookup, then the normalised float64
//           mean of each non-empty list, rows in ascending order, rounded to
//           float32 and on to the cache type); a final assignment; the rows
//           sorted by list (a stable counting sort: ascending rows within a list),
//           list offsets, and a copy of the rows in list order, so a probe
//           reads one contiguous block.
//   search: canonical centroid scores per (query, list) (products in parallel, the
//           ordered sum by one lane per centroid); the best nprobe lists per query (a
//           radix select in one workgroup); per (query, probe, 256 rows) the best
//           row: float64 dots in another order, each within 2^-40 |q| |c| of the
//           canonical score (2 d 2^-53 |q| |c| for any two orders of exact products, d
//           <= 2048), rule out the rows that cannot be best, and those left are
//           summed canonically; a final pass merges the blocks' rows; float32
//           similarity and the selector's K.
#include <algorithm>
#include <cmath>
#include <vector>

#include "common.h"

using namespace nv;

namespace nv {
namespace {
constexpr int ASSIGN_BATCH = 1024;  // rows per exact-lookup call in the assignment

__device__ inline float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

__device__ inline uint16_t f32_to_bf16_rne_i(float f) {
  const uint32_t u = __float_as_uint(f);
  return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

// (score, id) order: higher score first, lower id on ties
__device__ inline bool better_pair(double s, int64_t i, double bs, int64_t bi) {
  return s > bs || (s == bs && i < bi);
}

__global__ void __launch_bounds__(256) gather_rows_k(const void* __restrict__ src, int bf, int d,
                                                     const int64_t* __restrict__ idx, int64_t cnt,
                                                     void* __restrict__ dst) {
  const int64_t words = (int64_t)d * (bf ? 2 : 4) / 4;
  for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < cnt * words;
       t += (int64_t)gridDim.x * 256) {
    const int64_t r = t / words, w = t % words;
    ((uint32_t*)dst)[r * words + w] = ((const uint32_t*)src)[idx[r] * words + w];
  }
}

__global__ void __launch_bounds__(256) rows_to_f32_k(const void* __restrict__ src, int bf, int d,
                                                     int64_t r0, int cnt, float* __restrict__ out) {
  const int64_t total = (int64_t)cnt * d;
  for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < total;
       t += (int64_t)gridDim.x * 256) {
    const int64_t e = r0 * d + t;
    out[t] = bf ? bf16_to_f32(((const uint16_t*)src)[e]) : ((const float*)src)[e];
  }
}

// Stable counting sort of the rows by list (L <= 4096 lists): the rows are cut
// into nb consecutive blocks of R rows; list_count_k counts each block's rows
// per list, list_scan_k turns the counts into list offsets and, per (block,
// list), the position of the block's first row of that list; list_scatter_k
// walks each block's rows in ascending order, 64 at a time, and places row r
// of list l at that position plus the number of earlier rows of l in the
// block.  Ties keep row order, so every list holds its rows ascending.
// A list id outside [0, L) cannot come from the assignment (a lookup over L >= 1
// centroids always names one); it is clamped so no access leaves the arrays.
constexpr int MAX_LISTS = 4096;
constexpr int64_t SORT_MIN_ROWS = 4096;  // rows per block at least
constexpr int64_t SORT_MAX_BLOCKS = 1024;

__device__ inline int list_of(const int64_t* lists, int64_t r, int L) {
  const int64_t l = lists[r];
  return l < 0 ? 0 : (l >= L ? L - 1 : (int)l);
}

__global__ void __launch_bounds__(256) list_count_k(const int64_t* __restrict__ lists, int64_t n,
                                                    int L, int64_t R,
                                                    int32_t* __restrict__ counts) {
  __shared__ int32_t h[MAX_LISTS];
  for (int l = threadIdx.x; l < L; l += 256) h[l] = 0;
  __syncthreads();
  const int64_t r0 = (int64_t)blockIdx.x * R, r1 = min(n, r0 + R);
  for (int64_t r = r0 + threadIdx.x; r < r1; r += 256) atomicAdd(&h[list_of(lists, r, L)], 1);
  __syncthreads();
  for (int l = threadIdx.x; l < L; l += 256) counts[(int64_t)blockIdx.x * L + l] = h[l];
}

// One workgroup: column sums over the blocks (exclusive, in place), list
// totals, their exclusive scan into off[0..L], then off added to every column.
__global__ void __launch_bounds__(1024) list_scan_k(int32_t* __restrict__ counts, int nb, int L,
                                                    int64_t* __restrict__ off) {
  __shared__ int64_t tot[MAX_LISTS];
  for (int l = threadIdx.x; l < L; l += 1024) {
    int64_t run = 0;
    for (int b = 0; b < nb; ++b) {
      const int32_t c = counts[(int64_t)b * L + l];
      counts[(int64_t)b * L + l] = (int32_t)run;
      run += c;
    }
    tot[l] = run;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t run = 0;
    for (int l = 0; l < L; ++l) {
      const int64_t c = tot[l];
      tot[l] = run;
      off[l] = run;
      run += c;
    }
    off[L] = run;
  }
  __syncthreads();
  for (int l = threadIdx.x; l < L; l += 1024) {
    const int64_t base = tot[l];
    for (int b = 0; b < nb; ++b) counts[(int64_t)b * L + l] += (int32_t)base;
  }
}

// One wave per block of rows: the next free position of each list in LDS; per
// 64 rows, a lane's rank among earlier lanes of its list (readlane sweep), then
// the last lane of each list advances that list's position.
__global__ void __launch_bounds__(64) list_scatter_k(const int64_t* __restrict__ lists, int64_t n,
                                                     int L, int64_t R,
                                                     const int32_t* __restrict__ base,
                                                     int64_t* __restrict__ perm) {
  __shared__ int32_t next[MAX_LISTS];
  const int lane = threadIdx.x;
  for (int l = lane; l < L; l += 64) next[l] = base[(int64_t)blockIdx.x * L + l];
  __syncthreads();
  const int64_t r0 = (int64_t)blockIdx.x * R, r1 = min(n, r0 + R);
  for (int64_t c = r0; c < r1; c += 64) {
    const int64_t r = c + lane;
    const bool live = r < r1;
    const int l = live ? list_of(lists, r, L) : -1;
    int rank = 0, same = 0;
    for (int j = 0; j < 64; ++j) {
      const int lj = __builtin_amdgcn_readlane(l, j);
      const bool eq = live && lj == l;
      rank += (eq && j < lane) ? 1 : 0;
      same += eq ? 1 : 0;
    }
    const int pos = live ? next[l] + rank : 0;
    __builtin_amdgcn_wave_barrier();
    if (live) perm[pos] = r;
    if (live && rank == same - 1) next[l] = pos + 1;
    __builtin_amdgcn_wave_barrier();
  }
}

inline int64_t sort_rows_per_block(int64_t n) {
  return std::max<int64_t>(SORT_MIN_ROWS, ceil_div(n, SORT_MAX_BLOCKS));
}

// sums[l][k] = sum over the rows of list l, in ascending row order, of row[k] (float64)
__global__ void __launch_bounds__(64) list_sums_k(const void* __restrict__ rows, int bf, int d,
                                                  const int64_t* __restrict__ perm,
                                                  const int64_t* __restrict__ off,
                                                  double* __restrict__ sums) {
  const int l = blockIdx.x;
  const int k = blockIdx.y * 64 + threadIdx.x;
  if (k >= d) return;
  double s = 0.0;
  for (int64_t j = off[l]; j < off[l + 1]; ++j) {
    const int64_t r = perm[j];
    s += bf ? (double)bf16_to_f32(((const uint16_t*)rows)[r * d + k])
            : (double)((const float*)rows)[r * d + k];
  }
  sums[(int64_t)l * d + k] = s;
}

// centroid l = sums[l] / sqrt(left-to-right sum of squares), float32 then cache type
__global__ void __launch_bounds__(256) list_normalise_k(const double* __restrict__ sums, int d,
                                                        const int64_t* __restrict__ off, int bf,
                                                        void* __restrict__ cents) {
  __shared__ double nrm;
  const int l = blockIdx.x;
  if (off[l + 1] == off[l]) return;  // empty list keeps its centroid
  const double* s = sums + (int64_t)l * d;
  if (threadIdx.x == 0) {
    double a = 0.0;
    for (int k = 0; k < d; ++k) a = __dadd_rn(a, __dmul_rn(s[k], s[k]));
    // the correctly rounded square root: of sqrt's result and its two neighbours,
    // the one whose square is nearest a
    const double r = sqrt(a);
    double best = r, err = fabs(fma(r, r, -a));
    const double cand[2] = {nextafter(r, 0.0), nextafter(r, INFINITY)};
    for (int c = 0; c < 2; ++c) {
      const double e = fabs(fma(cand[c], cand[c], -a));
      if (e < err) {
        best = cand[c];
        err = e;
      }
    }
    nrm = best;
  }
  __syncthreads();
  for (int k = threadIdx.x; k < d; k += 256) {
    const float v = (float)(s[k] / nrm);
    if (bf)
      ((uint16_t*)cents)[(int64_t)l * d + k] = f32_to_bf16_rne_i(v);
    else
      ((float*)cents)[(int64_t)l * d + k] = v;
  }
}

// Doubles of the query in LDS, zero padded to whole 64-value slices.
__host__ __device__ inline int q_padded(int d) { return (d + 63) / 64 * 64; }
__device__ inline void load_query(double* qd, const float* __restrict__ q, int d) {
  for (int k = threadIdx.x; k < q_padded(d); k += blockDim.x) qd[k] = k < d ? (double)q[k] : 0.0;
}

// cs[j][l]: canonical score of query j against centroid l, 64 centroids per
// block of four waves.  The serial part of a canonical sum is one float64
// addition per element; everything else is shared out: in slices of 64 values,
// all four waves load, convert and multiply (exact in float64) into one LDS
// buffer while lane r of the first wave adds row r's products of the previous
// slice from the other.  With one thread per row doing all of it, 1024
// centroids took 52 us (28 without its barriers).
constexpr int PROW = 66;  // products per LDS row (64, and room against bank conflicts)

__global__ void __launch_bounds__(256) cent_scores_k(const float* __restrict__ q, int d,
                                                     const void* __restrict__ cents, int bf,
                                                     int L, double* __restrict__ cs) {
  extern __shared__ __align__(16) unsigned char smem[];
  double* qd = (double*)smem;             // [q_padded(d)]
  double* prod = qd + q_padded(d);        // [2][64][PROW]
  const int j = blockIdx.y, l0 = blockIdx.x * 64, t = threadIdx.x;
  const int nrows = min(64, L - l0);
  const int slices = q_padded(d) / 64;
  // thread t: row t / 4, 16 values from (t % 4) * 16 of every slice
  const int row = t >> 2, k0 = (t & 3) * 16;
  const bool live = row < nrows;
  float v[2][16];
  auto fetch = [&](int sl, float(&x)[16]) {
    const int k = sl * 64 + k0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      u32x4 w0 = {0u, 0u, 0u, 0u}, w1 = {0u, 0u, 0u, 0u};
      if (live && k + 8 * h < d) {  // d is a multiple of 8
        if (bf) {
          w0 = *(const u32x4*)((const uint16_t*)cents + (int64_t)(l0 + row) * d + k + 8 * h);
        } else {
          const float* c = (const float*)cents + (int64_t)(l0 + row) * d + k + 8 * h;
          w0 = *(const u32x4*)c;
          w1 = *(const u32x4*)(c + 4);
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t a = w0[e], b = w1[e];
        if (bf) {
          x[8 * h + 2 * e] = __uint_as_float(a << 16);
          x[8 * h + 2 * e + 1] = __uint_as_float(a & 0xFFFF0000u);
        } else {
          x[8 * h + e] = __uint_as_float(a);
          x[8 * h + 4 + e] = __uint_as_float(b);
        }
      }
    }
  };
  fetch(0, v[0]);
  fetch(1, v[1]);
  load_query(qd, q + (int64_t)j * d, d);
  __syncthreads();
  double s = 0.0;
  auto turn = [&](int sl, float(&x)[16]) {
    if (sl < slices) {
      double* p = prod + (sl & 1) * 64 * PROW + row * PROW + k0;
#pragma unroll
      for (int e = 0; e < 16; ++e) p[e] = qd[sl * 64 + k0 + e] * (double)x[e];
      fetch(sl + 2, x);
    }
    if (sl > 0 && t < 64) {
      const double2* p = (const double2*)(prod + ((sl - 1) & 1) * 64 * PROW + t * PROW);
#pragma unroll 8
      for (int e = 0; e < 32; ++e) {
        const double2 y = p[e];
        s = __dadd_rn(s, y.x);
        s = __dadd_rn(s, y.y);
      }
    }
    __syncthreads();
  };
  for (int sl = 0; sl <= slices; sl += 2) {
    turn(sl, v[0]);
    if (sl + 1 <= slices) turn(sl + 1, v[1]);
  }
  if (t < nrows) cs[(int64_t)j * L + l0 + t] = s;
}

// the nprobe best lists of query j in rank order (higher score first, lower
// list on ties).  Scores map to order-preserving 64-bit keys; a most-
// significant-byte-first radix select finds the nprobe-th largest key K*
// (eight 256-bin histograms in LDS); the lists above K*, and the lowest-
// numbered lists equal to it (an index-order prefix count), are compacted and
// each is placed at its rank among the selected.
constexpr int TOP_MAX_L = 4096;
constexpr int TOP_PER_T = TOP_MAX_L / 256;

__device__ inline uint64_t order_key(double x) {
  const uint64_t u = (uint64_t)__double_as_longlong(x);
  return (u >> 63) ? ~u : (u | (uint64_t(1) << 63));
}

// exclusive prefix sum over the block of one value per thread (256 threads)
__device__ inline int block_excl_scan(int v, int* sh) {
  const int t = threadIdx.x;
  sh[t] = v;
  __syncthreads();
  for (int o = 1; o < 256; o <<= 1) {
    const int a = t >= o ? sh[t - o] : 0;
    __syncthreads();
    sh[t] += a;
    __syncthreads();
  }
  const int incl = sh[t];
  __syncthreads();
  return incl - v;
}

__global__ void __launch_bounds__(256) top_lists_k(const double* __restrict__ cs, int L,
                                                   int nprobe, int32_t* __restrict__ probed) {
  __shared__ int hist[256];
  __shared__ int scan_sh[256];
  __shared__ uint64_t sel_key[256];
  __shared__ int sel_idx[256];
  __shared__ uint64_t kstar_sh;
  __shared__ int need_sh;
  const int j = blockIdx.x, t = threadIdx.x;
  // thread t owns lists t * TOP_PER_T .. (index order within and across threads)
  uint64_t key[TOP_PER_T];
#pragma unroll
  for (int e = 0; e < TOP_PER_T; ++e) {
    const int l = t * TOP_PER_T + e;
    key[e] = l < L ? order_key(cs[(int64_t)j * L + l]) : 0;
  }
  uint64_t prefix = 0, mask = 0;
  int need = nprobe;  // how many of the remaining candidates to take from the top
  for (int byte = 7; byte >= 0; --byte) {
    hist[t] = 0;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < TOP_PER_T; ++e) {
      const int l = t * TOP_PER_T + e;
      if (l < L && (key[e] & mask) == prefix)
        atomicAdd(&hist[(key[e] >> (8 * byte)) & 255], 1);
    }
    __syncthreads();
    // thread t's bin is the one where the count of larger-or-equal keys passes
    // `need` (a suffix sum: within waves by shuffles, then over waves; one thread
    // walking the bins took 6 us a byte)
    {
      const int own = hist[t];
      int suf = own;
      const int lane = t & 63;
      for (int o = 1; o < 64; o <<= 1) {
        const int x = __shfl_down(suf, o, 64);
        if (lane + o < 64) suf += x;
      }
      if (lane == 0) scan_sh[t >> 6] = suf;
      __syncthreads();
      for (int w = (t >> 6) + 1; w < 4; ++w) suf += scan_sh[w];
      if (suf >= need && suf - own < need) {
        need_sh = need - (suf - own);
        kstar_sh = prefix | ((uint64_t)t << (8 * byte));
      }
    }
    __syncthreads();
    need = need_sh;
    prefix = kstar_sh;
    mask |= (uint64_t)255 << (8 * byte);
    __syncthreads();
  }
  const uint64_t kstar = prefix;  // the nprobe-th largest key; take `need` lists equal to it
  int eq = 0;
#pragma unroll
  for (int e = 0; e < TOP_PER_T; ++e) {
    const int l = t * TOP_PER_T + e;
    eq += (l < L && key[e] == kstar);
  }
  int eq_before = block_excl_scan(eq, scan_sh);
  int take = 0;
#pragma unroll
  for (int e = 0; e < TOP_PER_T; ++e) {
    const int l = t * TOP_PER_T + e;
    if (l < L && (key[e] > kstar || (key[e] == kstar && eq_before++ < need))) ++take;
  }
  int pos = block_excl_scan(take, scan_sh);
  eq_before = block_excl_scan(eq, scan_sh);
#pragma unroll
  for (int e = 0; e < TOP_PER_T; ++e) {
    const int l = t * TOP_PER_T + e;
    if (l < L && (key[e] > kstar || (key[e] == kstar && eq_before++ < need))) {
      sel_key[pos] = key[e];
      sel_idx[pos] = l;
      ++pos;
    }
  }
  __syncthreads();
  if (t < nprobe) {
    const uint64_t k = sel_key[t];
    const int l = sel_idx[t];
    int rank = 0;
    for (int o = 0; o < nprobe; ++o)
      rank += sel_key[o] > k || (sel_key[o] == k && sel_idx[o] < l);
    probed[(int64_t)j * nprobe + rank] = l;
  }
}

// Canonical score of one row by one thread, straight from global memory, 64 values
// requested ahead of those being added.
__device__ inline double canon_thread(const double* qd, const char* __restrict__ rows, int r,
                                      int bf, int d) {
  double s = 0.0;
  const int nch = d >> 3;  // chunks of 8 values
  auto add8 = [&](int c, const float(&x)[8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e) s = __dadd_rn(s, qd[c * 8 + e] * (double)x[e]);
  };
  if (bf) {
    const u32x4* p = (const u32x4*)((const uint16_t*)rows + (int64_t)r * d);
    u32x4 v[2][8];
    auto fetch = [&](int c0, u32x4(&w)[8]) {
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (c0 + u < nch) w[u] = p[c0 + u];
    };
    auto sum = [&](int c0, const u32x4(&w)[8]) {
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (c0 + u >= nch) break;
        float x[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t a = w[u][e];
          x[2 * e] = __uint_as_float(a << 16);
          x[2 * e + 1] = __uint_as_float(a & 0xFFFF0000u);
        }
        add8(c0 + u, x);
      }
    };
    fetch(0, v[0]);
    for (int c0 = 0; c0 < nch; c0 += 16) {
      fetch(c0 + 8, v[1]);
      sum(c0, v[0]);
      fetch(c0 + 16, v[0]);
      sum(c0 + 8, v[1]);
    }
  } else {
    const u32x4* p = (const u32x4*)((const float*)rows + (int64_t)r * d);
    u32x4 v[2][8];  // 4 chunks of 8 values each
    auto fetch = [&](int c0, u32x4(&w)[8]) {
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (c0 + u < nch) {
          w[2 * u] = p[2 * (c0 + u)];
          w[2 * u + 1] = p[2 * (c0 + u) + 1];
        }
    };
    auto sum = [&](int c0, const u32x4(&w)[8]) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (c0 + u >= nch) break;
        float x[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t a = w[2 * u][e], b = w[2 * u + 1][e];
          x[e] = __uint_as_float(a);
          x[4 + e] = __uint_as_float(b);
        }
        add8(c0 + u, x);
      }
    };
    fetch(0, v[0]);
    for (int c0 = 0; c0 < nch; c0 += 8) {
      fetch(c0 + 4, v[1]);
      sum(c0, v[0]);
      fetch(c0 + 8, v[0]);
      sum(c0 + 4, v[1]);
    }
  }
  return s;
}

// Best probed row per (query, probe, chunk of 256 list positions).  Groups of 8
// lanes take float64 dots of the rows in another summation order, each within
// tol = 2^-40 |q| |c| of the canonical score (2 d 2^-53 |q| |c| at most, d <=
// 2048, and room for the norms' own rounding); the rows that can still hold
// the block's best canonical score (dot + tol reaches the largest dot - tol)
// are summed canonically, usually one: exact products into LDS by its wave,
// then the additions in order.  The result is the best (score, lowest row) of
// the block, as if every row had been summed (one query, 32 lists of about a
// thousand rows: 54 us with a canonical sum per row against 29).
// A score that is not a number is neither above nor below another, so with one
// among the rows the result depends on the order of the comparisons: every row of
// such a block is summed and the scores are compared in the fixed tree of
// probe_final_k over list positions.
constexpr int PS_T = 512;
// Rows to sum beyond which every row gets a thread of its own: a wave's sum of a row
// costs about as much as a thread's of all rows of its wave, and four waves share the
// rows, so past two rows a wave the threads win (200000 x 768 bf16, one query equal
// to that many rows, 16 of 256 lists, waves against threads: 16 rows 67 and 68 us, 64
// rows 84 and 69, 120 rows 89 and 69, 300 rows 377 and 71, 20000 rows 1495 and 164;
// no equal rows 63; f32, 384 wide, 300 rows 174 and 53).
constexpr int PS_FEW = 8;

__global__ void __launch_bounds__(PS_T) probe_scan_k(const float* __restrict__ q, int d,
                                                     const void* __restrict__ lrows, int bf,
                                                     const int64_t* __restrict__ perm,
                                                     const int64_t* __restrict__ off,
                                                     const int32_t* __restrict__ probed,
                                                     int nprobe, int chunks,
                                                     double* __restrict__ ps,
                                                     int64_t* __restrict__ pi) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int NWV = PS_T / 64;
  double* qd = (double*)smem;                     // [q_padded(d)]
  double* prods = qd + q_padded(d);               // [NWV / 2][q_padded(d)]
  __shared__ double fast[256], tols[256];
  __shared__ double red[NWV], rs[NWV];
  __shared__ int64_t ri[NWV];
  __shared__ int64_t ids[256];
  __shared__ int surv[256];
  __shared__ int n_surv, n_nan;
  const int jp = blockIdx.x, ch = blockIdx.y, t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int j = jp / nprobe;
  const int l = probed[jp];
  const int64_t p0 = off[l] + (int64_t)ch * 256;
  const int nrows = (int)max<int64_t>(0, min<int64_t>(256, off[l + 1] - p0));
  if (nrows == 0) {  // past the list's end
    if (t == 0) {
      ps[(int64_t)jp * chunks + ch] = -INFINITY;
      pi[(int64_t)jp * chunks + ch] = -1;
    }
    return;
  }
  const char* rows = (const char*)lrows + p0 * d * (bf ? 2 : 4);
  load_query(qd, q + (int64_t)j * d, d);
  if (t == 0) n_surv = n_nan = 0;
  if (t < 256) ids[t] = t < nrows ? perm[p0 + t] : -1;
  __syncthreads();
  double qq = 0.0;
  for (int k = t; k < d; k += PS_T) qq = fma(qd[k], qd[k], qq);
  for (int o = 32; o > 0; o >>= 1) qq += __shfl_xor(qq, o, 64);
  if (lane == 0) red[wave] = qq;
  // 64 groups of 8 lanes; lane l8 takes chunks l8, l8 + 8, ... of 8 values
  const int g = t >> 3, l8 = t & 7, nch = d >> 3;
  for (int r = g; r < nrows; r += PS_T / 8) {
    double a0 = 0.0, a1 = 0.0;
    float nn = 0.f;
    for (int c0 = l8; c0 < nch; c0 += 48) {
      u32x4 v[6][2];
#pragma unroll
      for (int u = 0; u < 6; ++u) {
        const int c = c0 + 8 * u;
        if (c < nch) {
          if (bf) {
            v[u][0] = *(const u32x4*)((const uint16_t*)rows + (int64_t)r * d + c * 8);
          } else {
            v[u][0] = *(const u32x4*)((const float*)rows + (int64_t)r * d + c * 8);
            v[u][1] = *(const u32x4*)((const float*)rows + (int64_t)r * d + c * 8 + 4);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < 6; ++u) {
        const int c = c0 + 8 * u;
        if (c >= nch) break;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float x, y;
          if (bf) {
            const uint32_t w = v[u][0][e];
            x = __uint_as_float(w << 16);
            y = __uint_as_float(w & 0xFFFF0000u);
          } else {
            const uint32_t w0 = v[u][e >> 1][2 * (e & 1)], w1 = v[u][e >> 1][2 * (e & 1) + 1];
            x = __uint_as_float(w0);
            y = __uint_as_float(w1);
          }
          nn = fmaf(x, x, nn);
          nn = fmaf(y, y, nn);
          a0 = fma(qd[c * 8 + 2 * e], (double)x, a0);
          a1 = fma(qd[c * 8 + 2 * e + 1], (double)y, a1);
        }
      }
    }
    double s = a0 + a1;
    s += __shfl_xor(s, 1, 64);
    s += __shfl_xor(s, 2, 64);
    s += __shfl_xor(s, 4, 64);
    nn += __shfl_xor(nn, 1, 64);
    nn += __shfl_xor(nn, 2, 64);
    nn += __shfl_xor(nn, 4, 64);
    if (l8 == 0) {
      fast[r] = s;
      tols[r] = sqrt((double)nn * 1.001 + 0x1p-120);  // at least the row's norm
    }
  }
  __syncthreads();
  qq = 0.0;
  for (int w = 0; w < NWV; ++w) qq += red[w];
  const double scale = 0x1p-40 * sqrt(qq) * (1.0 + 0x1p-40);
  // the block's best canonical score is at least the largest dot - tol
  double lo = -INFINITY;
  if (t < nrows) {
    lo = fast[t] - (scale * tols[t] + 0x1p-1000);
    // the products decide whether a sum is a number, whatever its order
    if (isnan(fast[t])) n_nan = 1;
  }
  for (int o = 32; o > 0; o >>= 1) lo = fmax(lo, __shfl_xor(lo, o, 64));
  if (lane == 0) rs[wave] = lo;
  __syncthreads();
  for (int w = 0; w < NWV; ++w) lo = fmax(lo, rs[w]);
  const bool any_nan = n_nan != 0;
  // a bound that is not a number rules nothing out
  if (t < nrows && (any_nan || !(fast[t] + (scale * tols[t] + 0x1p-1000) < lo)))
    surv[atomicAdd(&n_surv, 1)] = t;
  __syncthreads();
  double bs = -INFINITY;
  int64_t bi = -1;
  const int ns = n_surv;
  if (ns > PS_FEW) {
    if (t < ns) {
      const int r = surv[t];
      const double s = canon_thread(qd, rows, r, bf, d);
      if (any_nan) {
        fast[r] = s;
      } else {
        bs = s;
        bi = ids[r];
      }
    }
    for (int o = 32; o > 0; o >>= 1) {
      const double s2 = __shfl_xor(bs, o, 64);
      const int64_t i2 = __shfl_xor(bi, o, 64);
      if (i2 >= 0 && (bi < 0 || better_pair(s2, i2, bs, bi))) {
        bs = s2;
        bi = i2;
      }
    }
  } else if (wave < NWV / 2) {
    double* prod = prods + (size_t)wave * q_padded(d);
    for (int i = wave; i < ns; i += NWV / 2) {
      const int r = surv[i];
      for (int c = lane; c < nch; c += 64)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int k = c * 8 + e;
          const float x = bf ? __uint_as_float((uint32_t)((const uint16_t*)rows)[(int64_t)r * d + k] << 16)
                             : ((const float*)rows)[(int64_t)r * d + k];
          prod[k] = qd[k] * (double)x;
        }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      double s = 0.0;
      for (int k = 0; k < d; k += 8)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const double2 y = *(const double2*)&prod[k + 2 * e];
          s = __dadd_rn(s, y.x);
          s = __dadd_rn(s, y.y);
        }
      __builtin_amdgcn_wave_barrier();
      const int64_t row = ids[r];
      if (any_nan) {
        if (lane == 0) fast[r] = s;
      } else if (bi < 0 || better_pair(s, row, bs, bi)) {
        bs = s;
        bi = row;
      }
    }
  }
  __syncthreads();  // rs held the bounds
  if (any_nan) {
    for (int w = 128; w > 0; w >>= 1) {
      if (t < w && ids[t + w] >= 0 &&
          (ids[t] < 0 || better_pair(fast[t + w], ids[t + w], fast[t], ids[t]))) {
        fast[t] = fast[t + w];
        ids[t] = ids[t + w];
      }
      __syncthreads();
    }
    if (t == 0) {
      ps[(int64_t)jp * chunks + ch] = fast[0];
      pi[(int64_t)jp * chunks + ch] = ids[0];
    }
    return;
  }
  if (lane == 0) {
    rs[wave] = bs;
    ri[wave] = bi;
  }
  __syncthreads();
  if (t == 0) {
    for (int w = 1; w < NWV / 2; ++w)
      if (ri[w] >= 0 && (bi < 0 || better_pair(rs[w], ri[w], bs, bi))) {
        bs = rs[w];
        bi = ri[w];
      }
    ps[(int64_t)jp * chunks + ch] = bs;
    pi[(int64_t)jp * chunks + ch] = bi;
  }
}

struct Sel {
  float t[16];
  int32_t k[16];
  int J;
};

__global__ void __launch_bounds__(256) probe_final_k(const double* __restrict__ ps,
                                                     const int64_t* __restrict__ pi, int per_q,
                                                     Sel sel, int64_t* __restrict__ idx,
                                                     float* __restrict__ sim,
                                                     int32_t* __restrict__ kk) {
  __shared__ double rs[256];
  __shared__ int64_t ri[256];
  const int j = blockIdx.x, t = threadIdx.x;
  double bs = -INFINITY;
  int64_t bi = -1;
  for (int c = t; c < per_q; c += 256) {
    const int64_t i = pi[(int64_t)j * per_q + c];
    const double s = ps[(int64_t)j * per_q + c];
    if (i >= 0 && (bi < 0 || better_pair(s, i, bs, bi))) {
      bs = s;
      bi = i;
    }
  }
  rs[t] = bs;
  ri[t] = bi;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (t < w && ri[t + w] >= 0 && (ri[t] < 0 || better_pair(rs[t + w], ri[t + w], rs[t], ri[t]))) {
      rs[t] = rs[t + w];
      ri[t] = ri[t + w];
    }
    __syncthreads();
  }
  if (t == 0) {
    const int64_t b = ri[0];
    const float s = b >= 0 ? (float)rs[0] : -INFINITY;
    int32_t k = 0;
    if (b >= 0)
      for (int a = 0; a < sel.J; ++a)
        if (s > sel.t[a]) {
          k = sel.k[a];
          break;
        }
    idx[j] = b;
    sim[j] = s;
    kk[j] = k;
  }
}

struct BuildWs {
  size_t qf, lk, idx_tmp, sim_tmp, k_tmp, init_idx, sums, counts, total;
  size_t lk_bytes;
};

inline BuildWs plan_build(int64_t n, int d, int L) {
  BuildWs w{};
  size_t o = 0;
  auto take = [&](size_t bytes) {
    const size_t at = o;
    o = align_up(o + bytes, 256);
    return at;
  };
  w.lk_bytes = nv_cache_lookup_workspace(ASSIGN_BATCH, L, d);
  w.qf = take((size_t)ASSIGN_BATCH * d * 4);
  w.lk = take(w.lk_bytes);
  w.idx_tmp = take((size_t)ASSIGN_BATCH * 8);
  w.sim_tmp = take((size_t)ASSIGN_BATCH * 4);
  w.k_tmp = take((size_t)ASSIGN_BATCH * 4);
  w.init_idx = take((size_t)std::max<int64_t>(L, 1) * 8);
  w.sums = take((size_t)L * d * 8);
  w.counts = take((size_t)ceil_div(n, sort_rows_per_block(n)) * L * 4);
  w.total = o;
  return w;
}

}  // namespace
}  // namespace nv

extern "C" size_t nv_ivf_build_workspace(int64_t n, int32_t d, int32_t L) {
  if (n < 1 || d < 1 || L < 1) return 0;
  return plan_build(n, d, L).total;
}

extern "C" int32_t nv_ivf_build(const void* cache, int32_t c_dtype, int64_t n, int32_t d,
                                const int64_t* init, int32_t L, int32_t iters, void* cents,
                                int64_t* lists, int64_t* perm, int64_t* offsets, void* ivf_rows,
                                int64_t* max_list, void* workspace, size_t workspace_bytes,
                                void* stream) {
  clear_error();
  NV_CHECK_ARG(cache && init && cents && lists && perm && offsets && ivf_rows && max_list,
               "null argument");
  NV_CHECK_ARG(c_dtype == NV_F32 || c_dtype == NV_BF16, "c_dtype must be NV_F32 or NV_BF16");
  NV_CHECK_ARG(n >= 1 && n < (int64_t(1) << 31), "n must be in [1, 2^31)");
  NV_CHECK_ARG(L >= 1 && L <= 4096 && L <= n, "L must be in [1, min(n, 4096)]");
  NV_CHECK_ARG(iters >= 0 && iters <= 100, "iters must be in [0, 100]");
  if (d % 8 != 0 || d < 8 || d > 2048) {
    set_error("d must be a multiple of 8 in [8, 2048]");
    return NV_ERR_UNSUPPORTED;
  }
  const BuildWs w = plan_build(n, d, L);
  if (!workspace || workspace_bytes < w.total || ((uintptr_t)workspace & 255)) {
    set_error("ivf build workspace missing, misaligned or smaller than nv_ivf_build_workspace()");
    return NV_ERR_WORKSPACE;
  }
  for (int l = 0; l < L; ++l) NV_CHECK_ARG(init[l] >= 0 && init[l] < n, "init out of range");
  hipStream_t s = (hipStream_t)stream;
  char* ws = (char*)workspace;
  const int bf = c_dtype == NV_BF16;
  int64_t* init_idx = (int64_t*)(ws + w.init_idx);
  // initial centroids: the rows at init (host indices staged through the key buffer)
  NV_HIP_TRY(hipMemcpyAsync(init_idx, init, (size_t)L * 8, hipMemcpyHostToDevice, s));
  hipLaunchKernelGGL(gather_rows_k, dim3((unsigned)std::min<int64_t>(ceil_div((int64_t)L * d, 256), 4096)),
                     dim3(256), 0, s, cache, bf, d, (const int64_t*)init_idx, (int64_t)L, cents);
  NV_LAUNCH_CHECK("gather_rows_k");
  const float thr_none[1] = {1e30f};
  const int32_t k_none[1] = {0};
  auto assign = [&]() -> int32_t {
    for (int64_t r0 = 0; r0 < n; r0 += ASSIGN_BATCH) {
      const int cnt = (int)std::min<int64_t>(ASSIGN_BATCH, n - r0);
      hipLaunchKernelGGL(rows_to_f32_k, dim3((unsigned)std::min<int64_t>(ceil_div((int64_t)cnt * d, 256), 2048)),
                         dim3(256), 0, s, cache, bf, d, r0, cnt, (float*)(ws + w.qf));
      NV_LAUNCH_CHECK("rows_to_f32_k");
      const int32_t st = nv_cache_lookup((const float*)(ws + w.qf), cnt, cents, c_dtype, L, d,
                                         thr_none, k_none, 1, lists + r0,
                                         (float*)(ws + w.sim_tmp), (int32_t*)(ws + w.k_tmp),
                                         ws + w.lk, w.lk_bytes, stream);
      if (st != NV_OK) return st;
    }
    return NV_OK;
  };
  auto sort_lists = [&]() -> int32_t {
    const int64_t R = sort_rows_per_block(n);
    const int nb = (int)ceil_div(n, R);
    int32_t* counts = (int32_t*)(ws + w.counts);
    hipLaunchKernelGGL(list_count_k, dim3((unsigned)nb), dim3(256), 0, s, (const int64_t*)lists,
                       n, L, R, counts);
    NV_LAUNCH_CHECK("list_count_k");
    hipLaunchKernelGGL(list_scan_k, dim3(1), dim3(1024), 0, s, counts, nb, L, offsets);
    NV_LAUNCH_CHECK("list_scan_k");
    hipLaunchKernelGGL(list_scatter_k, dim3((unsigned)nb), dim3(64), 0, s, (const int64_t*)lists,
                       n, L, R, (const int32_t*)counts, perm);
    NV_LAUNCH_CHECK("list_scatter_k");
    return NV_OK;
  };
  for (int it = 0; it < iters; ++it) {
    int32_t st = assign();
    if (st != NV_OK) return st;
    st = sort_lists();
    if (st != NV_OK) return st;
    hipLaunchKernelGGL(list_sums_k, dim3((unsigned)L, (unsigned)ceil_div(d, 64)), dim3(64), 0, s,
                       cache, bf, d, (const int64_t*)perm, (const int64_t*)offsets,
                       (double*)(ws + w.sums));
    NV_LAUNCH_CHECK("list_sums_k");
    hipLaunchKernelGGL(list_normalise_k, dim3((unsigned)L), dim3(256), 0, s,
                       (const double*)(ws + w.sums), d, (const int64_t*)offsets, bf, cents);
    NV_LAUNCH_CHECK("list_normalise_k");
  }
  int32_t st = assign();
  if (st != NV_OK) return st;
  st = sort_lists();
  if (st != NV_OK) return st;
  hipLaunchKernelGGL(gather_rows_k, dim3(4096), dim3(256), 0, s, cache, bf, d,
                     (const int64_t*)perm, n, ivf_rows);
  NV_LAUNCH_CHECK("gather_rows_k");
  std::vector<int64_t> off(L + 1);
  NV_HIP_TRY(hipMemcpyAsync(off.data(), offsets, (size_t)(L + 1) * 8, hipMemcpyDeviceToHost, s));
  NV_HIP_TRY(hipStreamSynchronize(s));
  int64_t mx = 0;
  for (int l = 0; l < L; ++l) mx = std::max(mx, off[l + 1] - off[l]);
  *max_list = mx;
  return NV_OK;
}

extern "C" size_t nv_ivf_search_workspace(int32_t m, int32_t L, int32_t nprobe, int64_t max_list) {
  if (m < 1 || L < 1 || nprobe < 1 || max_list < 0) return 0;
  const int64_t chunks = std::max<int64_t>(1, ceil_div(max_list, 256));
  return align_up((size_t)m * L * 8, 256) + align_up((size_t)m * nprobe * 4, 256) +
         2 * align_up((size_t)m * nprobe * chunks * 8, 256);
}

extern "C" int32_t nv_ivf_search(const float* queries, int32_t m, int32_t d, const void* cents,
                                 int32_t L, const void* ivf_rows, int32_t c_dtype,
                                 const int64_t* perm, const int64_t* offsets, int64_t max_list,
                                 int32_t nprobe, const float* thresholds, const int32_t* k_values,
                                 int32_t J, int64_t* idx_out, float* sim_out, int32_t* k_out,
                                 int32_t* probed_out, void* workspace, size_t workspace_bytes,
                                 void* stream) {
  clear_error();
  NV_CHECK_ARG(queries && cents && ivf_rows && perm && offsets && idx_out && sim_out && k_out,
               "null argument");
  NV_CHECK_ARG(m >= 1 && m <= 4096, "m must be in [1, 4096]");
  NV_CHECK_ARG(c_dtype == NV_F32 || c_dtype == NV_BF16, "c_dtype must be NV_F32 or NV_BF16");
  NV_CHECK_ARG(L >= 1 && L <= 4096, "L must be in [1, 4096]");
  NV_CHECK_ARG(nprobe >= 1 && nprobe <= L && nprobe <= 256, "nprobe must be in [1, min(L, 256)]");
  NV_CHECK_ARG(max_list >= 0 && max_list < (int64_t(1) << 31), "bad max_list");
  NV_CHECK_ARG(thresholds && k_values && J >= 1 && J <= 16, "need 1..16 thresholds");
  if (d % 8 != 0 || d < 8 || d > 2048) {
    set_error("d must be a multiple of 8 in [8, 2048]");
    return NV_ERR_UNSUPPORTED;
  }
  Sel sel{};
  sel.J = J;
  for (int a = 0; a < J; ++a) {
    NV_CHECK_ARG(std::isfinite(thresholds[a]), "thresholds must be finite");
    NV_CHECK_ARG(a == 0 || thresholds[a] < thresholds[a - 1], "thresholds must descend");
    NV_CHECK_ARG(k_values[a] >= 0, "k_values must be >= 0");
    sel.t[a] = thresholds[a];
    sel.k[a] = k_values[a];
  }
  const size_t need = nv_ivf_search_workspace(m, L, nprobe, max_list);
  if (!workspace || workspace_bytes < need || ((uintptr_t)workspace & 255)) {
    set_error("ivf search workspace missing, misaligned or too small");
    return NV_ERR_WORKSPACE;
  }
  const int chunks = (int)std::max<int64_t>(1, ceil_div(max_list, 256));
  NV_CHECK_ARG((int64_t)m * nprobe <= 65535 * 64 && chunks <= 65535, "search too large");
  hipStream_t s = (hipStream_t)stream;
  char* ws = (char*)workspace;
  double* cs = (double*)ws;
  int32_t* probed = probed_out ? probed_out
                               : (int32_t*)(ws + align_up((size_t)m * L * 8, 256));
  char* after = ws + align_up((size_t)m * L * 8, 256) + align_up((size_t)m * nprobe * 4, 256);
  double* ps = (double*)after;
  int64_t* pi = (int64_t*)(after + align_up((size_t)m * nprobe * chunks * 8, 256));
  const int bf = c_dtype == NV_BF16;
  // at most 84 KB and 82 KB of LDS (d = 2048)
  const size_t clds = (size_t)q_padded(d) * 8 + (size_t)2 * 64 * PROW * 8;
  const size_t plds = (size_t)q_padded(d) * 8 * (1 + PS_T / 128);
  NV_HIP_TRY(hipFuncSetAttribute((const void*)cent_scores_k,
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)clds));
  NV_HIP_TRY(hipFuncSetAttribute((const void*)probe_scan_k,
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)plds));
  hipLaunchKernelGGL(cent_scores_k, dim3((unsigned)ceil_div(L, 64), (unsigned)m), dim3(256),
                     (uint32_t)clds, s, queries, d, cents, bf, L, cs);
  NV_LAUNCH_CHECK("cent_scores_k");
  hipLaunchKernelGGL(top_lists_k, dim3((unsigned)m), dim3(256), 0, s, (const double*)cs, L, nprobe,
                     probed);
  NV_LAUNCH_CHECK("top_lists_k");
  hipLaunchKernelGGL(probe_scan_k, dim3((unsigned)(m * nprobe), (unsigned)chunks), dim3(PS_T),
                     (uint32_t)plds, s,
                     queries, d, ivf_rows, bf, perm, offsets, (const int32_t*)probed, nprobe,
                     chunks, ps, pi);
  NV_LAUNCH_CHECK("probe_scan_k");
  hipLaunchKernelGGL(probe_final_k, dim3((unsigned)m), dim3(256), 0, s, (const double*)ps,
                     (const int64_t*)pi, nprobe * chunks, sel, idx_out, sim_out, k_out);
  NV_LAUNCH_CHECK("probe_final_k");
  return NV_OK;
}
