// Matrix-core GEMM / implicit-GEMM convolution for the UNet (float16 operands,
// float32 accumulation, v_mfma_f32_16x16x32_f16).
//
//   C[m][n] = sum_k A[m][k] * W[n][k]       (both operands K-contiguous)
//
// A comes from one of two loaders:
//   dense : A[m][k] = k < C1 ? src1[m][k] : src2[m][k - C1]  (channel concat)
//   conv3 : 3x3 convolution over NHWC activations, k = (ky, kx, ci) with ci
//           fastest; input pixel (oy*s + ky - 1, ox*s + kx - 1), or for a fused
//           nearest x2 upsample ((oy + ky - 1) >> 1, (ox + kx - 1) >> 1) inside
//           the 2H x 2W grid; out-of-range pixels read zero (padding 1); the
//           channel may come from either of two concatenated sources.
// Epilogue (in this order): + bias[n], + rowvec[row / rows_div][n], SiLU,
// + residual[m][n]; or GEGLU: the weight rows are packed in groups of 32 as
// (16 "a" rows, 16 "g" rows) and output column j of group j/16 is
// a * GELU_erf(g).  Output float16 or float32.
//
// Three kernels:
//   gemm_f16  any K and channel counts in multiples of 8: global -> registers ->
//             LDS double buffer, 4 waves in 2 x 2, each (BM/2) x (BN/2) as 16x16
//             MFMA blocks, one barrier per 64-deep k tile; LDS rows are padded to 144
//             bytes so the 16 rows read by a quarter-wave land in distinct 16-byte
//             bank groups (9r mod 16 is a permutation).  The conv loader walks (tap,
//             ci) incrementally: no integer division in the k loop.
//   gemm_s    every 64-deep k tile in one source and tap: global -> LDS without
//             registers, small wave tiles; what it runs now is split K, products
//             whose outputs the row-staged epilogue cannot take, and small GEGLU grids.
//   gemm_w    the same products otherwise: larger wave tiles, or k shared out over
//             wave groups, and the row-staged epilogue.
// gemm_rule.h chooses between the last two.  Split K leaves float32 partials, summed
// in a fixed order by splitk_reduce, which applies the epilogue (deterministic).
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "gelu.h"
#include "gemm.h"
#include "gemm_rule.h"
#include "trace.h"

namespace nv {
namespace {

constexpr int BK = 64;
constexpr int ROW = BK + 8;  // halfs per LDS row

constexpr uint32_t OOB = 0x80000000u;  // offset past every descriptor's range

// ring depth of the streamed kernel per tile shape (LDS: depth x (BM + BN) x 128 bytes)
#ifndef GEMM_S128
#define GEMM_S128 2
#endif
#ifndef GEMM_S64
#define GEMM_S64 3
#endif

__device__ inline __amdgpu_buffer_rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}
__device__ inline uint4 bload(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
  return make_uint4(v[0], v[1], v[2], v[3]);
}

struct DeviceMath {
  static __device__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
  static __device__ float exp2(float x) { return __builtin_amdgcn_exp2f(x); }
};
__device__ __forceinline__ void gelu4(const float (&x)[4], float (&y)[4]) {
  gelu_quad<DeviceMath>(x, y);
}
__device__ inline float silu(float x) { return x / (1.0f + __expf(-x)); }

// Epilogue of 4 consecutive columns n..n+3 of row m (non-GEGLU): + bias,
// + rowvec, SiLU, + residual, then float16 or float32 out.  vec: the quad is
// inside N and every row stride keeps it 8-byte (float16) / 16-byte (float32)
// aligned, so it moves as one vector; otherwise element by element.
__device__ inline void store_out4(const GemmArgs& g, int64_t m, int n, float (&v)[4], bool vec) {
  const int nn = vec ? 4 : max(0, min(4, g.N - n));
  if (g.bias) {
    if (vec) {
      const float4 b = *(const float4*)(g.bias + n);
      v[0] += b.x; v[1] += b.y; v[2] += b.z; v[3] += b.w;
    } else {
      for (int r = 0; r < nn; ++r) v[r] += g.bias[n + r];
    }
  }
  if (g.rowvec) {
    const float* rv = g.rowvec + (m / g.rows_div) * (int64_t)g.ld_rowvec + n;
    for (int r = 0; r < nn; ++r) v[r] += rv[r];
  }
  if (g.silu)
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = silu(v[r]);
  if (g.vt && n >= g.vt_col0) {  // transposed columns (no residual on these)
    _Float16* o = g.vt + (int64_t)(n - g.vt_col0) * g.vt_ld + (m / g.vt_div) * g.vt_stride +
                  m % g.vt_div;
    for (int r = 0; r < nn; ++r) o[(int64_t)r * g.vt_ld] = (_Float16)v[r];
    return;
  }
  if (g.residual) {
    const _Float16* rp = g.residual + m * g.ld_res + n;
    if (vec) {
      const half4 h = *(const half4*)rp;
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] += (float)h[r];
    } else {
      for (int r = 0; r < nn; ++r) v[r] += (float)rp[r];
    }
  }
  if (g.out_f32) {
    float* o = (float*)g.out + m * g.ldo + n;
    if (vec)
      *(float4*)o = make_float4(v[0], v[1], v[2], v[3]);
    else
      for (int r = 0; r < nn; ++r) o[r] = v[r];
  } else {
    _Float16* o = (_Float16*)g.out + m * g.ldo + n;
    if (vec) {
      half4 h;
#pragma unroll
      for (int r = 0; r < 4; ++r) h[r] = (_Float16)v[r];
      *(half4*)o = h;
    } else {
      for (int r = 0; r < nn; ++r) o[r] = (_Float16)v[r];
    }
  }
}

// GEGLU quad: na is the packed column of the first "a" value (gates sit 16
// columns later); output columns oc..oc+3 with oc = (na / 32) * 16 + na % 32.
__device__ inline void store_geglu4(const GemmArgs& g, int64_t m, int na, const float (&a)[4],
                                    const float (&gt)[4], bool vec) {
  float av[4], gv[4], y[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    av[r] = a[r];
    gv[r] = gt[r];
    if (g.bias) {
      av[r] += g.bias[na + r];
      gv[r] += g.bias[na + 16 + r];
    }
  }
  gelu4(gv, y);
#pragma unroll
  for (int r = 0; r < 4; ++r) y[r] *= av[r];
  const int oc = (na >> 5) * 16 + (na & 15);
  _Float16* o = (_Float16*)g.out + m * g.ldo + oc;
  if (vec) {
    half4 h;
#pragma unroll
    for (int r = 0; r < 4; ++r) h[r] = (_Float16)y[r];
    *(half4*)o = h;
  } else {
    for (int r = 0; r < 4; ++r) o[r] = (_Float16)y[r];
  }
}

// Epilogue of a wave's FM x FN quads (row m = mb + i * 16 + li, columns n =
// nb + j * 16 + kc * 4 ..+3), the same arithmetic as store_out4 /
// store_geglu4.  The stores could alias the loaded operands as far as the
// compiler knows, so quad by quad every load (bias, row vector, residual)
// would cost a memory round trip; here each row block's loads are issued
// together, unconditionally from clamped addresses, before its stores.
template <int FM, int FN>
__device__ inline void epilogue_tile(const GemmArgs& g, int64_t mb, int nb, int li, int kc,
                                  floatx4 (&acc)[FM][FN]) {
  const bool vec = g.vec_ok;
  // bias per column quad, loaded once
  float bq[FN][4];
#pragma unroll
  for (int j = 0; j < FN; ++j) {
    const int n = nb + j * 16 + kc * 4;
#pragma unroll
    for (int r = 0; r < 4; ++r) bq[j][r] = 0.f;
    if (g.bias) {
      if (vec && n + 4 <= g.N) {
        const float4 b = *(const float4*)(g.bias + n);
        bq[j][0] = b.x; bq[j][1] = b.y; bq[j][2] = b.z; bq[j][3] = b.w;
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) bq[j][r] = g.bias[n + r < g.N ? n + r : 0];
      }
    }
  }
  if (g.geglu) {  // quad j = 2 jj holds "a" columns na.., j = 2 jj + 1 the gates na + 16..
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const int64_t m = mb + i * 16 + li;
      if (m >= g.M) continue;
#pragma unroll
      for (int jj = 0; jj < FN / 2; ++jj) {
        const int na = nb + 2 * jj * 16 + kc * 4;
        if (na + 16 >= g.N) continue;
        float av[4], gv[4], y[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          av[r] = acc[i][2 * jj][r];
          gv[r] = acc[i][2 * jj + 1][r];
          if (g.bias) {
            av[r] += bq[2 * jj][r];
            gv[r] += bq[2 * jj + 1][r];
          }
        }
        gelu4(gv, y);
#pragma unroll
        for (int r = 0; r < 4; ++r) y[r] *= av[r];
        const int oc = (na >> 5) * 16 + (na & 15);
        _Float16* o = (_Float16*)g.out + m * g.ldo + oc;
        if (vec) {
          half4 h;
#pragma unroll
          for (int r = 0; r < 4; ++r) h[r] = (_Float16)y[r];
          *(half4*)o = h;
        } else {
          for (int r = 0; r < 4; ++r) o[r] = (_Float16)y[r];
        }
      }
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int64_t m = mb + i * 16 + li;
    const int64_t mc = m < g.M ? m : 0;  // a row every load may use
    float rv[FN][4];
    half4 res[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int n = nb + j * 16 + kc * 4;
      const bool qv = vec && n + 4 <= g.N;
#pragma unroll
      for (int r = 0; r < 4; ++r) rv[j][r] = 0.f;
      if (g.rowvec) {
        const float* p = g.rowvec + (mc / g.rows_div) * (int64_t)g.ld_rowvec;
#pragma unroll
        for (int r = 0; r < 4; ++r) rv[j][r] = p[n + r < g.N ? n + r : 0];
      }
      res[j] = half4{};
      if (g.residual && !(g.vt && n >= g.vt_col0)) {
        const _Float16* p = g.residual + mc * g.ld_res;
        if (qv) {
          res[j] = *(const half4*)(p + n);
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r) res[j][r] = p[n + r < g.N ? n + r : 0];
        }
      }
    }
    if (m >= g.M) continue;
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int n = nb + j * 16 + kc * 4;
      if (n >= g.N) continue;
      const bool qv = vec && n + 4 <= g.N;
      const int nn = qv ? 4 : min(4, g.N - n);
      float w[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        w[r] = acc[i][j][r];
        if (g.bias) w[r] += bq[j][r];
        if (g.rowvec) w[r] += rv[j][r];
        if (g.silu) w[r] = silu(w[r]);
      }
      if (g.vt && n >= g.vt_col0) {  // transposed columns (no residual on these)
        _Float16* o = g.vt + (int64_t)(n - g.vt_col0) * g.vt_ld + (m / g.vt_div) * g.vt_stride +
                      m % g.vt_div;
        for (int r = 0; r < nn; ++r) o[(int64_t)r * g.vt_ld] = (_Float16)w[r];
        continue;
      }
      if (g.residual)
#pragma unroll
        for (int r = 0; r < 4; ++r) w[r] += (float)res[j][r];
      if (g.out_f32) {
        float* o = (float*)g.out + m * g.ldo + n;
        if (qv)
          *(float4*)o = make_float4(w[0], w[1], w[2], w[3]);
        else
          for (int r = 0; r < nn; ++r) o[r] = w[r];
      } else {
        _Float16* o = (_Float16*)g.out + m * g.ldo + n;
        if (qv) {
          half4 h;
#pragma unroll
          for (int r = 0; r < 4; ++r) h[r] = (_Float16)w[r];
          *(half4*)o = h;
        } else {
          for (int r = 0; r < nn; ++r) o[r] = (_Float16)w[r];
        }
      }
    }
  }
}

// Epilogue through LDS: the tile's float32 sums are staged row by row (IB
// 16-row blocks of every wave row per pass), then each thread finishes 8
// consecutive columns of one row, so that bias, row vector and residual are
// read and the float16 result is written as 16-byte pieces of whole lines.
// Straight from the accumulators a wave's store touches 16 rows in 32-byte
// pieces: the last tiles of a 256 x 256 grid then take 27 us to drain.
// GEGLU quads are combined in registers (as in epilogue_tile) and staged at
// half the columns, where a wave holds all of K and whole 32-column groups
// (KG == 1, FN even); the launcher gives the other forms none.  With KG > 1 wave
// group kg holds its share of K's sums: the groups add theirs to the staged rows in
// group order.  The arithmetic and
// its order are those of store_out4 / store_geglu4; the transposed columns (vt)
// go out as 8 consecutive tokens of one channel.
// st: LDSB bytes of LDS that no wave reads or loads into any more.  With LN,
// ln[r] holds (mean, 1 / sqrt(var + eps)) of tile row r: the sums become
// rstd * (sum - mean * ln_c1[n]) first.
template <int BM, int BN, int WGM, int WGN, int KG, int LDSB, bool LN, int FM, int FN>
__device__ __forceinline__ void epilogue_rows(const GemmArgs& g, float* st, int64_t m0, int n0, int kg,
                                              int wm, int wn, int li, int kc,
                                              floatx4 (&acc)[FM][FN], const float2* ln) {
  constexpr int NT = KG * WGM * WGN * 64, WM = BM / WGM, WN = BN / WGN;
  constexpr int SR = BN + 4;                   // staged row stride (floats)
  constexpr int FIT = LDSB / (WGM * 16 * SR * 4);
  constexpr int IB = FIT < FM ? FIT : FM;      // 16-row blocks per wave row and pass
  static_assert(IB >= 1, "staging needs one 16-row block per wave row");
  constexpr int ROWS = WGM * 16 * IB;
  const int tid = threadIdx.x;
  const int M = (int)min(g.M - m0, (int64_t)BM);  // rows of the tile inside the product
  const int vt0 = g.vt ? g.vt_col0 : g.N;         // first transposed column
  // GEGLU: quads combined in registers and staged as the finished float16
  // outputs, BN / 2 columns a row
  if constexpr (KG == 1 && FN % 2 == 0) {
    if (g.geglu) {
      constexpr int SH = BN / 2 + 8;  // staged row stride (halfs)
      static_assert((size_t)BM * SH * 2 <= LDSB, "staged GEGLU tile");
      _Float16* sh = (_Float16*)st;
      float4 ba[FN / 2], bg[FN / 2];
      floatx4 ca[FN / 2], cg[FN / 2];
#pragma unroll
      for (int jj = 0; jj < FN / 2; ++jj) {
        const int na = n0 + wn * WN + 2 * jj * 16 + kc * 4;
        const bool in = g.bias && na + 16 < g.N;
        ba[jj] = in ? *(const float4*)(g.bias + na) : make_float4(0.f, 0.f, 0.f, 0.f);
        bg[jj] = in ? *(const float4*)(g.bias + na + 16) : make_float4(0.f, 0.f, 0.f, 0.f);
        if (LN) {
          const bool cin = na + 16 < g.N;
          ca[jj] = cin ? *(const floatx4*)(g.ln_c1 + na) : floatx4{0.f, 0.f, 0.f, 0.f};
          cg[jj] = cin ? *(const floatx4*)(g.ln_c1 + na + 16) : floatx4{0.f, 0.f, 0.f, 0.f};
        }
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int jj = 0; jj < FN / 2; ++jj) {
          floatx4 a = acc[i][2 * jj], t = acc[i][2 * jj + 1];
          if (LN) {
            const float2 s = ln[wm * WM + i * 16 + li];
            a = s.y * (a - s.x * ca[jj]);
            t = s.y * (t - s.x * cg[jj]);
          }
          const float gv[4] = {t[0] + bg[jj].x, t[1] + bg[jj].y, t[2] + bg[jj].z, t[3] + bg[jj].w};
          float y[4];
          gelu4(gv, y);
          half4 h;
          h[0] = (_Float16)((a[0] + ba[jj].x) * y[0]);
          h[1] = (_Float16)((a[1] + ba[jj].y) * y[1]);
          h[2] = (_Float16)((a[2] + ba[jj].z) * y[2]);
          h[3] = (_Float16)((a[3] + ba[jj].w) * y[3]);
          *(half4*)&sh[(wm * WM + i * 16 + li) * SH + wn * (WN / 2) + jj * 16 + kc * 4] = h;
        }
      __syncthreads();
      constexpr int CH = BN / 16;
      const int nout = g.N / 2 - n0 / 2;
      for (int e = tid; e < BM * CH; e += NT) {
        const int r = e / CH, c = (e % CH) * 8;
        if (r < M && c < nout)
          *(half8*)((_Float16*)g.out + (m0 + r) * g.ldo + (n0 >> 1) + c) = *(const half8*)&sh[r * SH + c];
      }
      return;
    }
  }
#pragma unroll
  for (int i0 = 0; i0 < FM; i0 += IB) {
#pragma unroll
    for (int k = 0; k < KG; ++k) {
      __syncthreads();
      if (kg == k)
#pragma unroll
        for (int i = i0; i < i0 + IB && i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j) {
            floatx4* p = (floatx4*)&st[((wm * IB + i - i0) * 16 + li) * SR + wn * WN + j * 16 + kc * 4];
            *p = k == 0 ? acc[i][j] : *p + acc[i][j];
          }
    }
    __syncthreads();
    auto row_of = [&](int r) { return (r / (16 * IB)) * WM + i0 * 16 + r % (16 * IB); };
    auto live = [&](int r) { return i0 + (r % (16 * IB)) / 16 < FM && row_of(r) < M; };
    constexpr int CH = BN / 8;
    for (int e = tid; e < ROWS * CH; e += NT) {
      const int r = e / CH, c = e % CH;
      const int n = n0 + c * 8;
      if (!live(r) || n >= vt0) continue;
      const int64_t m = m0 + row_of(r);
      half8 res = {};
      if (g.residual) res = *(const half8*)(g.residual + m * g.ld_res + n);
      const float4* p = (const float4*)&st[r * SR + c * 8];
      float4 v[2] = {p[0], p[1]};
      if (LN) {
        const float2 s = ln[row_of(r)];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const float4 c1 = *(const float4*)(g.ln_c1 + n + 4 * q);
          v[q].x = s.y * (v[q].x - s.x * c1.x); v[q].y = s.y * (v[q].y - s.x * c1.y);
          v[q].z = s.y * (v[q].z - s.x * c1.z); v[q].w = s.y * (v[q].w - s.x * c1.w);
        }
      }
      if (g.bias) {
        const float4* b = (const float4*)(g.bias + n);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const float4 t = b[q];
          v[q].x += t.x; v[q].y += t.y; v[q].z += t.z; v[q].w += t.w;
        }
      }
      if (g.rowvec) {
        const float* rv = g.rowvec + (int64_t)((uint32_t)m / (uint32_t)g.rows_div) * g.ld_rowvec + n;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          v[q].x += rv[4 * q]; v[q].y += rv[4 * q + 1]; v[q].z += rv[4 * q + 2]; v[q].w += rv[4 * q + 3];
        }
      }
      float w[8] = {v[0].x, v[0].y, v[0].z, v[0].w, v[1].x, v[1].y, v[1].z, v[1].w};
      half8 h;
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        if (g.silu) w[q] = silu(w[q]);
        if (g.residual) w[q] += (float)res[q];
        h[q] = (_Float16)w[q];
      }
      *(half8*)((_Float16*)g.out + m * g.ldo + n) = h;
    }
    if (n0 + BN > vt0) {  // 8 tokens of one transposed column per thread
      constexpr int RG = ROWS / 8;
      for (int e = tid; e < BN * RG; e += NT) {
        const int c = e / RG, r = (e % RG) * 8;
        const int n = n0 + c;
        if (n < vt0 || n >= g.N || !live(r)) continue;
        const float b = g.bias ? g.bias[n] : 0.f;
        const float c1 = LN ? g.ln_c1[n] : 0.f;
        half8 h;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          float v = st[(r + q) * SR + c];
          if (LN) {
            const float2 s = ln[row_of(r + q)];
            v = s.y * (v - s.x * c1);
          }
          if (g.bias) v += b;
          if (g.silu) v = silu(v);
          h[q] = (_Float16)v;
        }
        const uint32_t m = (uint32_t)(m0 + row_of(r));
        const uint32_t img = m / (uint32_t)g.vt_div, at = m - img * (uint32_t)g.vt_div;
        // M, vt_div and the strides are multiples of 8
        *(half8*)(g.vt + (int64_t)(n - vt0) * g.vt_ld + img * g.vt_stride + at) = h;
      }
    }
  }
}

template <int MODE, int BM, int BN, bool DUAL>
__global__ void __launch_bounds__(256) gemm_f16(GemmArgs g, int kt_per_split) {
  constexpr int WM = BM / 2, WN = BN / 2;
  constexpr int FM = WM / 16, FN = WN / 16;
  constexpr int A_CH = BM * 8 / 256;  // 16-byte chunks per thread per k tile
  constexpr int B_CH = BN * 8 / 256;
  extern __shared__ __align__(16) unsigned char smem[];
  _Float16* sA = (_Float16*)smem;                 // [2][BM][ROW]
  _Float16* sB = sA + 2 * BM * ROW;               // [2][BN][ROW]

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int li = lane & 15, kc = lane >> 4;
  // 1-D grid of tiles; each XCD owns a contiguous range of logical tiles.  When
  // the activations are the larger operand an XCD owns M-rows (N fastest), else
  // it owns weight columns (M fastest), so the big operand is read once.
  const int ntn = (g.N + BN - 1) / BN;
  const int mtn = (int)((g.M + BM - 1) / BM);
  const int tile = xcd_remap(blockIdx.x, gridDim.x);
  const int64_t m0 = (int64_t)(g.n_major ? tile % mtn : tile / ntn) * BM;
  const int n0 = (g.n_major ? tile / mtn : tile % ntn) * BN;
  const int nk = (g.K + BK - 1) / BK;
  const int kt0 = blockIdx.z * kt_per_split;
  const int kt1 = min(nk, kt0 + kt_per_split);
  const int cch = tid & 7;   // chunk column of this thread (k offset cch*8)
  const int rr = tid >> 3;   // first row of this thread (+32 per chunk)

  // Row geometry of this thread's A rows.
  int64_t a_m[A_CH];
  int a_b[A_CH], a_oy[A_CH], a_ox[A_CH];
  bool a_ok[A_CH];
#pragma unroll
  for (int i = 0; i < A_CH; ++i) {
    a_m[i] = m0 + rr + 32 * i;
    a_ok[i] = a_m[i] < g.M;
    a_b[i] = a_oy[i] = a_ox[i] = 0;
    if (MODE == 1 && a_ok[i]) {
      const int hw = g.Ho * g.Wo;
      a_b[i] = (int)(a_m[i] / hw);
      const int p = (int)(a_m[i] - (int64_t)a_b[i] * hw);
      a_oy[i] = p / g.Wo;
      a_ox[i] = p - a_oy[i] * g.Wo;
    }
  }
  // conv: (tap, ci) of this thread's chunk at the current k tile
  const int cin = g.C1 + g.C2;
  int tap = 0, ci = 0;
  if (MODE == 1) {
    const int k = kt0 * BK + cch * 8;
    tap = k / cin;
    ci = k - tap * cin;
  }

  // Two register stages: the global loads of tile kt+2 are issued while tile
  // kt is multiplied from LDS and tile kt+1 waits in the other stage.
  uint4 ra0[A_CH], rb0[B_CH];
  // Buffer loads with range descriptors: an invalid element gets an
  // out-of-range offset and the hardware returns zeros, so no load result is
  // touched before it is stored to LDS and both pipeline stages stay in flight.
  const __amdgpu_buffer_rsrc_t rs1 = make_rsrc(g.src1, g.bytes1);
  const __amdgpu_buffer_rsrc_t rs2 = make_rsrc(g.src2 ? g.src2 : g.src1, g.src2 ? g.bytes2 : 0);
  const __amdgpu_buffer_rsrc_t rsw = make_rsrc(g.w, (uint32_t)((int64_t)g.N * g.ldw * 2));
  // !DUAL: one source per 64-channel k tile (C1, and for convs Cin, multiples of 64)
  constexpr bool uni = !DUAL;
  // Incremental addressing (one source and one tap per 64-deep k tile): the
  // per-row byte offsets are recomputed only when the tile enters a new tap or
  // source, and otherwise advance by 128 bytes; out-of-range rows carry an
  // offset past the descriptor's range, which stays out of range.
  int t_k0 = kt0 * BK;
  int t_tap = 0, t_ci = 0;
  bool t_first = true;
  uint32_t aoff[A_CH], boff[B_CH];
  auto a_offsets = [&]() {
    if (MODE == 0) {
      t_first = t_k0 < g.C1;
#pragma unroll
      for (int i = 0; i < A_CH; ++i) {
        const bool ok = a_ok[i] && t_k0 < g.K;
        aoff[i] = !ok ? OOB
                : t_first ? (uint32_t)((a_m[i] * g.lda1 + t_k0 + cch * 8) * 2)
                          : (uint32_t)((a_m[i] * g.lda2 + (t_k0 - g.C1) + cch * 8) * 2);
      }
    } else {
      t_first = t_ci < g.C1;
      const int ky = (t_tap * 11) >> 5, kx = t_tap - 3 * ((t_tap * 11) >> 5);
      const int ld = t_first ? g.C1 : g.C2;
      const int cs = (t_first ? t_ci : t_ci - g.C1) + cch * 8;
#pragma unroll
      for (int i = 0; i < A_CH; ++i) {
        int iy, ix;
        bool in;
        if (g.upsample) {
          const int uy = a_oy[i] + ky - 1, ux = a_ox[i] + kx - 1;
          in = uy >= 0 && ux >= 0 && uy < 2 * g.Hin && ux < 2 * g.Win;
          iy = uy >> 1;
          ix = ux >> 1;
        } else {
          iy = a_oy[i] * g.stride + ky - 1;
          ix = a_ox[i] * g.stride + kx - 1;
          in = iy >= 0 && ix >= 0 && iy < g.Hin && ix < g.Win;
        }
        const bool ok = a_ok[i] && in && t_tap < 9;
        const int64_t pix = ((int64_t)a_b[i] * g.Hin + iy) * g.Win + ix;
        aoff[i] = ok ? (uint32_t)((pix * ld + cs) * 2) : OOB;
      }
    }
  };
  if (!DUAL) {
    if (MODE == 1) {
      t_tap = t_k0 / cin;
      t_ci = t_k0 - t_tap * cin;
    }
    a_offsets();
#pragma unroll
    for (int i = 0; i < B_CH; ++i) {
      const int n = n0 + rr + 32 * i;
      boff[i] = (n < g.N) ? (uint32_t)(((int64_t)n * g.ldw + t_k0 + cch * 8) * 2) : OOB;
    }
  }
  auto load_inc = [&](uint4 (&ra)[A_CH], uint4 (&rb)[B_CH]) {
    const __amdgpu_buffer_rsrc_t rsa = t_first ? rs1 : rs2;
#pragma unroll
    for (int i = 0; i < A_CH; ++i) ra[i] = bload(rsa, aoff[i]);
#pragma unroll
    for (int i = 0; i < B_CH; ++i) rb[i] = bload(rsw, boff[i]);
    // advance to the next tile
    t_k0 += BK;
#pragma unroll
    for (int i = 0; i < B_CH; ++i) boff[i] += 2 * BK;
    bool fresh;
    if (MODE == 0) {
      fresh = t_k0 == g.C1 || t_k0 >= g.K;
    } else {
      t_ci += BK;
      fresh = false;
      if (t_ci >= cin) {
        t_ci -= cin;
        ++t_tap;
        fresh = true;
      }
      if (t_ci == g.C1) fresh = true;
    }
    if (fresh) {
      a_offsets();
    } else {
#pragma unroll
      for (int i = 0; i < A_CH; ++i) aoff[i] += 2 * BK;
    }
  };
  auto load_tile = [&](int kt, uint4 (&ra)[A_CH], uint4 (&rb)[B_CH]) {
    const int k = kt * BK + cch * 8;
    const bool kok = k < g.K;
    if (MODE == 0) {
      const bool first = k < g.C1;
#pragma unroll
      for (int i = 0; i < A_CH; ++i) {
        const bool ok = a_ok[i] && kok;
        const uint32_t o1 = ok && first ? (uint32_t)((a_m[i] * g.lda1 + k) * 2) : OOB;
        if (uni) {
          const uint32_t o2 = ok && !first ? (uint32_t)((a_m[i] * g.lda2 + (k - g.C1)) * 2) : OOB;
          ra[i] = bload((kt * BK < g.C1) ? rs1 : rs2, (kt * BK < g.C1) ? o1 : o2);
        } else {
          const uint32_t o2 = ok && !first ? (uint32_t)((a_m[i] * g.lda2 + (k - g.C1)) * 2) : OOB;
          const uint4 v1 = bload(rs1, o1), v2 = bload(rs2, o2);
          ra[i] = make_uint4(v1.x | v2.x, v1.y | v2.y, v1.z | v2.z, v1.w | v2.w);
        }
      }
    } else {
      const int ky = (tap * 11) >> 5, kx = tap - 3 * ((tap * 11) >> 5);
      const bool first = ci < g.C1;
#pragma unroll
      for (int i = 0; i < A_CH; ++i) {
        int iy, ix;
        bool in;
        if (g.upsample) {
          const int uy = a_oy[i] + ky - 1, ux = a_ox[i] + kx - 1;
          in = uy >= 0 && ux >= 0 && uy < 2 * g.Hin && ux < 2 * g.Win;
          iy = uy >> 1;
          ix = ux >> 1;
        } else {
          iy = a_oy[i] * g.stride + ky - 1;
          ix = a_ox[i] * g.stride + kx - 1;
          in = iy >= 0 && ix >= 0 && iy < g.Hin && ix < g.Win;
        }
        const bool ok = a_ok[i] && kok && in;
        const int64_t pix = ((int64_t)a_b[i] * g.Hin + iy) * g.Win + ix;
        const uint32_t o1 = ok && first ? (uint32_t)((pix * g.C1 + ci) * 2) : OOB;
        const uint32_t o2 = ok && !first ? (uint32_t)((pix * g.C2 + (ci - g.C1)) * 2) : OOB;
        if (uni) {
          const bool f0 = __builtin_amdgcn_readfirstlane(first ? 1 : 0) != 0;
          ra[i] = bload(f0 ? rs1 : rs2, f0 ? o1 : o2);
        } else {
          const uint4 v1 = bload(rs1, o1), v2 = bload(rs2, o2);
          ra[i] = make_uint4(v1.x | v2.x, v1.y | v2.y, v1.z | v2.z, v1.w | v2.w);
        }
      }
      ci += BK;
      if (uni) {  // cin % 64 == 0: at most one tap boundary per tile
        if (ci >= cin) {
          ci -= cin;
          ++tap;
        }
      } else {
        while (ci >= cin) {
          ci -= cin;
          ++tap;
        }
      }
    }
#pragma unroll
    for (int i = 0; i < B_CH; ++i) {
      const int n = n0 + rr + 32 * i;
      const bool ok = n < g.N && kok;
      rb[i] = bload(rsw, ok ? (uint32_t)(((int64_t)n * g.ldw + k) * 2) : OOB);
    }
  };
  auto store_tile = [&](int buf, const uint4 (&ra)[A_CH], const uint4 (&rb)[B_CH]) {
    _Float16* a = sA + buf * BM * ROW;
    _Float16* b = sB + buf * BN * ROW;
#pragma unroll
    for (int i = 0; i < A_CH; ++i) *(uint4*)&a[(rr + 32 * i) * ROW + cch * 8] = ra[i];
#pragma unroll
    for (int i = 0; i < B_CH; ++i) *(uint4*)&b[(rr + 32 * i) * ROW + cch * 8] = rb[i];
  };

  floatx4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  auto compute = [&](int buf) {
    const _Float16* a = sA + buf * BM * ROW;
    const _Float16* b = sB + buf * BN * ROW;
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
      half8 fa[FM], fb[FN];
#pragma unroll
      for (int i = 0; i < FM; ++i)
        fa[i] = *(const half8*)&a[(wm * WM + i * 16 + li) * ROW + sub * 32 + kc * 8];
#pragma unroll
      for (int j = 0; j < FN; ++j)
        fb[j] = *(const half8*)&b[(wn * WN + j * 16 + li) * ROW + sub * 32 + kc * 8];
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fb[j], fa[i], acc[i][j], 0, 0, 0);
    }
  };

  // Pipeline, two tiles deep: while tile kt is multiplied from LDS stage kt&1,
  // tile kt+1 waits in one register set and tile kt+2 is being fetched into
  // the other; loads past the last tile re-read the last tile (never used).
  uint4 ra1[A_CH], rb1[B_CH];
  const int klast = max(kt0, kt1 - 1);
  auto fetch = [&](int kt, uint4 (&ra)[A_CH], uint4 (&rb)[B_CH]) {
    if (DUAL)
      load_tile(kt, ra, rb);
    else
      load_inc(ra, rb);  // tiles arrive in order; fetches past the last tile are unused
  };
  fetch(kt0, ra0, rb0);
  store_tile(0, ra0, rb0);
  fetch(min(kt0 + 1, klast), ra1, rb1);
  __syncthreads();
  int kt = kt0;
  for (; kt + 1 < kt1; kt += 2) {
    fetch(min(kt + 2, klast), ra0, rb0);
    compute(0);
    store_tile(1, ra1, rb1);
    __syncthreads();
    fetch(min(kt + 3, klast), ra1, rb1);
    compute(1);
    store_tile(0, ra0, rb0);
    __syncthreads();
  }
  if (kt < kt1) compute(0);

  // Operands are swapped in the multiply (weights as the row operand), so lane
  // (li, kc) of block (i, j) holds row m = ... + i * 16 + li and the four
  // consecutive columns n = ... + j * 16 + kc * 4 + r.
  if (gridDim.z > 1) {
    float* part = g.partial + (int64_t)blockIdx.z * g.M * g.N;
    const bool pv = (g.N & 3) == 0;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const int64_t m = m0 + wm * WM + i * 16 + li;
      if (m >= g.M) continue;
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const int n = n0 + wn * WN + j * 16 + kc * 4;
        if (n >= g.N) continue;
        float* pp = part + m * g.N + n;
        if (pv)
          *(float4*)pp = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
        else
          for (int r = 0; r < 4 && n + r < g.N; ++r) pp[r] = acc[i][j][r];
      }
    }
    return;
  }
  epilogue_tile<FM, FN>(g, m0 + wm * WM, n0 + wn * WN, li, kc, acc);
}

// ---------------------------------------------------------------------------
// Streamed variant for shapes whose every 64-deep k tile lies inside one
// source and one tap (dense: C1 and K multiples of 64; conv: C1 and C2
// multiples of 64).  Tiles move global -> LDS with 16-byte buffer loads that
// write LDS directly (no registers, no LDS store instructions) into a ring of
// STAGES buffers; a wave waits for its own loads of the tile it is about to
// multiply (vmcnt), one barrier per tile publishes everyone's, and the tile
// STAGES - 1 ahead is requested right after it.  Rows are 128 bytes with the
// 16-byte chunk c of row r stored at chunk c ^ (r & 7): the 16 rows a quarter
// wave reads at one k offset hit distinct bank groups.  Out-of-range rows and
// padding taps use an offset past the descriptor's range and land as zeros.
__device__ inline void lds_dma16(__amdgpu_buffer_rsrc_t r, uint32_t off, void* lds_wave_base,
                                 uint32_t soff = 0) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)lds_wave_base,
                                           16, off, soff, 0, 0);
}

// s_waitcnt with only vmcnt limited (expcnt, lgkmcnt at their maxima; gfx9 encoding).
template <int N>
__device__ inline void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// Workgroup barrier for the ring: each wave has already waited (vmcnt) for its
// own loads of the tile about to be read, so the barrier alone publishes the
// tile; no memory fence, which would also wait for the loads still in flight
// into the other buffers.  The empty asm statements keep the compiler from
// moving LDS accesses across it.
__device__ inline void ring_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// One 64-deep k tile: wave tile (FM x 16) rows by (FN x 16) columns.  The
// tile's LDS buffers are read through restrict-qualified pointers: while this
// runs, only other ring buffers are being written (by loads in flight).
template <int FM, int FN>
__device__ __forceinline__ void mma_tile(const _Float16* __restrict__ a,
                                         const _Float16* __restrict__ b, int arow0, int brow0,
                                         int li, int kc, floatx4 (&acc)[FM][FN]) {
#pragma unroll
  for (int sub = 0; sub < 2; ++sub) {
    const int c = sub * 4 + kc;
    half8 fa[FM], fb[FN];
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const int r = arow0 + i * 16 + li;
      fa[i] = *(const half8*)(a + r * 64 + ((c ^ (r & 7)) << 3));
    }
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int r = brow0 + j * 16 + li;
      fb[j] = *(const half8*)(b + r * 64 + ((c ^ (r & 7)) << 3));
    }
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fb[j], fa[i], acc[i][j], 0, 0, 0);
  }
}

// NW waves: 2 x 2 wave tiles (4) or 2 x 4 (8, half the columns per wave).
template <int MODE, int BM, int BN, int STAGES, bool LN, int U, int NW>
__global__ void __launch_bounds__(NW * 64) gemm_s(GemmArgs g, int kt_per_split) {
  static_assert(U >= 1 && STAGES >= 2 * U, "ring must hold two groups of U tiles");
  static_assert(NW == 4 || NW == 8, "waves per workgroup");
  constexpr int WM = BM / 2, WN = BN / (NW / 2);
  constexpr int FM = WM / 16, FN = WN / 16;
  constexpr int AJ = BM / (8 * NW), BJ = BN / (8 * NW);  // 8-row groups per wave per tile
  constexpr int OPS = AJ + BJ;               // loads per wave per tile
  constexpr int TILE_H = (BM + BN) * 64;     // halfs per ring buffer
  extern __shared__ __align__(16) unsigned char smem[];
  _Float16* ring = (_Float16*)smem;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: LDS bases in SGPRs
  const int wm = wave / (NW / 2), wn = wave % (NW / 2);
  const int li = lane & 15, kc = lane >> 4;
  const int ntn = (g.N + BN - 1) / BN;
  const int mtn = (int)((g.M + BM - 1) / BM);
  const int tile = xcd_remap(blockIdx.x, gridDim.x);
  const int64_t m0 = (int64_t)(g.n_major ? tile % mtn : tile / ntn) * BM;
  const int n0 = (g.n_major ? tile / mtn : tile % ntn) * BN;
  const int nk = g.K / 64;
  const int kt0 = blockIdx.z * kt_per_split;
  const int kt1 = min(nk, kt0 + kt_per_split);
  // loader geometry: group j of this wave covers rows (j * NW + wave) * 8 ..+8;
  // lane l loads row +l/8, chunk slot l%8, i.e. k chunk (l%8) ^ (l/8)
  const int lrow = lane >> 3;
  const int cch = (lane & 7) ^ lrow;
  const __amdgpu_buffer_rsrc_t rs1 = make_rsrc(g.src1, g.bytes1);
  const __amdgpu_buffer_rsrc_t rs2 = make_rsrc(g.src2 ? g.src2 : g.src1, g.src2 ? g.bytes2 : 0);
  const __amdgpu_buffer_rsrc_t rsw = make_rsrc(g.w, (uint32_t)((int64_t)g.N * g.ldw * 2));

  int64_t a_m[AJ];
  int a_b[AJ], a_oy[AJ], a_ox[AJ];
#pragma unroll
  for (int j = 0; j < AJ; ++j) {
    a_m[j] = m0 + (j * NW + wave) * 8 + lrow;
    a_b[j] = a_oy[j] = a_ox[j] = 0;
    if (MODE == 1 && a_m[j] < g.M) {
      const int hw = g.Ho * g.Wo;
      a_b[j] = (int)(a_m[j] / hw);
      const int p = (int)(a_m[j] - (int64_t)a_b[j] * hw);
      a_oy[j] = p / g.Wo;
      a_ox[j] = p - a_oy[j] * g.Wo;
    }
  }
  const int cin = g.C1 + g.C2;
  int t_k0 = kt0 * 64, t_tap = 0, t_ci = 0;
  bool t_first = true;
  if (MODE == 1) {
    t_tap = t_k0 / cin;
    t_ci = t_k0 - t_tap * cin;
  }
  uint32_t aoff[AJ], boff[BJ];
  auto a_offsets = [&]() {
    if (MODE == 0) {
      t_first = t_k0 < g.C1;
#pragma unroll
      for (int j = 0; j < AJ; ++j) {
        const bool ok = a_m[j] < g.M && t_k0 < g.K;
        aoff[j] = !ok ? OOB
                : t_first ? (uint32_t)((a_m[j] * g.lda1 + t_k0 + cch * 8) * 2)
                          : (uint32_t)((a_m[j] * g.lda2 + (t_k0 - g.C1) + cch * 8) * 2);
      }
    } else {
      t_first = t_ci < g.C1;
      const int ky = (t_tap * 11) >> 5, kx = t_tap - 3 * ((t_tap * 11) >> 5);
      const int ld = t_first ? g.C1 : g.C2;
      const int cs = (t_first ? t_ci : t_ci - g.C1) + cch * 8;
#pragma unroll
      for (int j = 0; j < AJ; ++j) {
        int iy, ix;
        bool in;
        if (g.upsample) {
          const int uy = a_oy[j] + ky - 1, ux = a_ox[j] + kx - 1;
          in = uy >= 0 && ux >= 0 && uy < 2 * g.Hin && ux < 2 * g.Win;
          iy = uy >> 1;
          ix = ux >> 1;
        } else {
          iy = a_oy[j] * g.stride + ky - 1;
          ix = a_ox[j] * g.stride + kx - 1;
          in = iy >= 0 && ix >= 0 && iy < g.Hin && ix < g.Win;
        }
        const bool ok = a_m[j] < g.M && in && t_tap < 9;
        const int64_t pix = ((int64_t)a_b[j] * g.Hin + iy) * g.Win + ix;
        aoff[j] = ok ? (uint32_t)((pix * ld + cs) * 2) : OOB;
      }
    }
  };
  a_offsets();
#pragma unroll
  for (int j = 0; j < BJ; ++j) {
    const int n = n0 + (j * NW + wave) * 8 + lrow;
    boff[j] = (n < g.N) ? (uint32_t)(((int64_t)n * g.ldw + t_k0 + cch * 8) * 2) : OOB;
  }
  // request the next tile in k order into ring buffer `buf`, then advance
  auto issue = [&](int buf) {
    _Float16* A = ring + buf * TILE_H;
    _Float16* Bt = A + BM * 64;
    // the source is uniform: branch on it (made visibly uniform), so each
    // descriptor stays in SGPRs (a selected one would sit in VGPRs and need a
    // readfirstlane loop around every load)
    if (__builtin_amdgcn_readfirstlane((int)t_first) != 0) {
#pragma unroll
      for (int j = 0; j < AJ; ++j) lds_dma16(rs1, aoff[j], A + (j * NW + wave) * 512);
    } else {
#pragma unroll
      for (int j = 0; j < AJ; ++j) lds_dma16(rs2, aoff[j], A + (j * NW + wave) * 512);
    }
#pragma unroll
    for (int j = 0; j < BJ; ++j) lds_dma16(rsw, boff[j], Bt + (j * NW + wave) * 512);
    t_k0 += 64;
#pragma unroll
    for (int j = 0; j < BJ; ++j) boff[j] += 128;
    bool fresh;
    if (MODE == 0) {
      fresh = t_k0 == g.C1 || t_k0 >= g.K;
    } else {
      t_ci += 64;
      fresh = false;
      if (t_ci >= cin) {
        t_ci -= cin;
        ++t_tap;
        fresh = true;
      }
      if (t_ci == g.C1) fresh = true;
    }
    if (fresh) {
      a_offsets();
    } else {
#pragma unroll
      for (int j = 0; j < AJ; ++j) aoff[j] += 128;
    }
  };

  floatx4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  // Prologue: tiles kt0 .. kt0 + STAGES - U - 1.  Requests past kt1 fetch
  // tiles that are never multiplied (in range or zero-filled), which keeps the
  // per-wave count of loads in flight fixed for the waits below.  Each pass of
  // the main loop multiplies U tiles behind one barrier.
#pragma unroll
  for (int s = 0; s < STAGES - U; ++s) issue(s);
  // Folded LayerNorm: TPR threads per A row each sum CPT of the row's eight
  // 16-byte chunks per k tile, shifted by the row's first value (k = 0, in
  // chunk slot r & 7) so that the one-pass variance does not cancel: the
  // shifted pair d (float16) enters sum d and sum d^2 through float32 dot2.
  constexpr int TPR = NW * 64 / BM, CPT = 8 / TPR;
  const int st_row = tid / TPR, st_slot = (tid % TPR) * CPT;
  half2v st_shift = {(_Float16)0.f, (_Float16)0.f};
  const half2v st_one = {(_Float16)1.f, (_Float16)1.f};
  float st_s1 = 0.f, st_s2 = 0.f;
  // the folded LayerNorm's column sums c1 of this wave's columns, requested
  // now so that the epilogue does not wait for them
  float c1v[LN ? FN : 1][4];
  if (LN)
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int n = n0 + wn * WN + j * 16 + kc * 4;
#pragma unroll
      for (int r = 0; r < 4; ++r) c1v[j][r] = n + r < g.N ? g.ln_c1[n + r] : 0.f;
    }
  for (int kt = kt0; kt < kt1; kt += U) {
    wait_vmcnt<(STAGES - 2 * U) * OPS>();  // this wave's loads of tiles kt .. kt+U-1 have landed
    ring_barrier();                        // everyone's have; the previous U buffers are free
#pragma unroll
    for (int u = 0; u < U; ++u) issue((kt - kt0 + STAGES - U + u) % STAGES);
#pragma unroll
    for (int u = 0; u < U; ++u) {
    const int ktu = kt + u;
    if (U > 1 && ktu >= kt1) break;
    const _Float16* A = ring + ((ktu - kt0) % STAGES) * TILE_H;
    mma_tile<FM, FN>(A, A + BM * 64, wm * WM, wn * WN, li, kc, acc);
    if (LN) {
      const _Float16* ar = A + st_row * 64;
      if (ktu == 0) st_shift = half2v{ar[(st_row & 7) * 8], ar[(st_row & 7) * 8]};
#pragma unroll
      for (int c = 0; c < CPT; ++c) {
        const half8 h = *(const half8*)(ar + (st_slot + c) * 8);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const half2v d = half2v{h[2 * e], h[2 * e + 1]} - st_shift;
          st_s1 = __builtin_amdgcn_fdot2(d, st_one, st_s1, false);
          st_s2 = __builtin_amdgcn_fdot2(d, d, st_s2, false);
        }
      }
    }
    }
  }
  wait_vmcnt<0>();  // drain the requests past the last tile before the workgroup ends
  if (LN) {
    __shared__ float2 lnst[BM];  // (mean, 1 / sqrt(var + eps)) per tile row
#pragma unroll
    for (int o = 1; o < TPR; o <<= 1) {
      st_s1 += __shfl_xor(st_s1, o, 64);
      st_s2 += __shfl_xor(st_s2, o, 64);
    }
    if (tid % TPR == 0) {
      const float inv_k = 1.0f / (float)g.K;
      const float mu = st_s1 * inv_k;
      const float var = fmaxf(st_s2 * inv_k - mu * mu, 0.f);
      lnst[st_row] = make_float2((float)st_shift[0] + mu, rsqrtf(var + g.ln_eps));
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const float2 st = lnst[wm * WM + i * 16 + li];
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[i][j][r] = st.y * (acc[i][j][r] - st.x * c1v[j][r]);
    }
  }

  // Operands are swapped in the multiply (weights as the row operand), so lane
  // (li, kc) of block (i, j) holds row m = ... + i * 16 + li and the four
  // consecutive columns n = ... + j * 16 + kc * 4 + r.
  if (gridDim.z > 1) {
    float* part = g.partial + (int64_t)blockIdx.z * g.M * g.N;
    const bool pv = (g.N & 3) == 0;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const int64_t m = m0 + wm * WM + i * 16 + li;
      if (m >= g.M) continue;
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const int n = n0 + wn * WN + j * 16 + kc * 4;
        if (n >= g.N) continue;
        float* pp = part + m * g.N + n;
        if (pv)
          *(float4*)pp = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
        else
          for (int r = 0; r < 4 && n + r < g.N; ++r) pp[r] = acc[i][j][r];
      }
    }
    return;
  }
  epilogue_tile<FM, FN>(g, m0 + wm * WM, n0 + wn * WN, li, kc, acc);
}

// ---------------------------------------------------------------------------
// Wide tiles and k sharing for whole-chip grids.  The kernels above multiply
// 32 x 32 to 64 x 32 wave tiles: LDS bandwidth (fragment reads and tile writes)
// bounds them at half the matrix rate, and a grid that leaves a CU with one
// workgroup leaves its SIMDs one or two waves.  Here
//   - wave tiles are up to 128 x 64 (half the fragment bytes per multiply);
//   - where a grid of small tiles fills the chip only once, the waves of a
//     workgroup share out k instead of the tile: KH = 2 groups take the two
//     32-deep halves of every 64-deep tile, KT = 2 teams alternate tiles, and the
//     groups' sums meet in the row-staged epilogue;
//   - 64-deep k tiles (128-byte rows: whole L2 lines; 32-deep rows measured 10 %
//     slower) move through a ring of STAGES buffers per team, and the loop is
//     rotated: the fragments of the next half (or tile) are read while the
//     current ones are multiplied, so a tile's buffer is free again at the
//     barrier that follows its last fragment read.
// LDS row layout as in gemm_s (16-byte chunk c of row r at slot c ^ (r & 7)).
template <int FM, int FN>
__device__ __forceinline__ void read_frags(const _Float16* __restrict__ t, int aoff, int boff,
                                           half8 (&fa)[FM], half8 (&fb)[FN]) {
#pragma unroll
  for (int j = 0; j < FN; ++j) fb[j] = *(const half8*)(t + boff + j * 1024);
#pragma unroll
  for (int i = 0; i < FM; ++i) fa[i] = *(const half8*)(t + aoff + i * 1024);
}

template <int N>
__device__ inline void wait_vm_lgkm0() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));
}

template <int MODE, int BM, int BN, int WGM, int WGN, int KH, int KT, int STAGES, bool LN>
__global__ void __launch_bounds__(KT * KH * WGM * WGN * 64, 2) gemm_w(GemmArgs g) {
  static_assert(KH == 1 || KH == 2, "halves of a k tile");
  constexpr int NL = KH * WGM * WGN;  // waves of a team; they load its tiles
  constexpr int WM = BM / WGM, WN = BN / WGN, FM = WM / 16, FN = WN / 16;
  constexpr int GA = BM / 8, NG = GA + BN / 8;  // 8-row groups of a tile (1 KB of LDS each)
  constexpr int PER = (NG + NL - 1) / NL;       // groups a wave loads (the last may be missing)
  constexpr int TILE_H = (BM + BN) * 64;        // halfs per ring buffer
  static_assert(WM % 16 == 0 && WN % 16 == 0 && STAGES >= 2, "wave tile");
  static_assert((STAGES - 1) * PER < 64, "requests in flight per wave");
  extern __shared__ __align__(16) unsigned char smem[];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int team = KT == 1 ? 0 : wave_all / NL, wave = KT == 1 ? wave_all : wave_all % NL;
  const int kh = KH == 1 ? 0 : wave / (WGM * WGN), wt = KH == 1 ? wave : wave % (WGM * WGN);
  const int wm = wt / WGN, wn = wt % WGN;
  _Float16* ring = (_Float16*)smem + team * STAGES * TILE_H;
  const int li = lane & 15, kc = lane >> 4;
  const int ntn = (g.N + BN - 1) / BN;
  const int mtn = (int)((g.M + BM - 1) / BM);
  const int tile = xcd_remap(blockIdx.x, gridDim.x);
  const int64_t m0 = (int64_t)(g.n_major ? tile % mtn : tile / ntn) * BM;
  const int n0 = (g.n_major ? tile / mtn : tile % ntn) * BN;
  // this team's 64-deep k tiles: kt0, kt0 + KT, ...; every team runs
  // the steps of team 0, its last one may find no tile left
  const int nk = g.K / 64, kt0 = team < nk ? team : 0;  // no tile: tile 0, never multiplied
  const int n_steps = (nk + KT - 1) / KT;
  const int my_steps = KT == 1 ? n_steps : (nk - team + KT - 1) / KT;
  const __amdgpu_buffer_rsrc_t rs1 = make_rsrc(g.src1, g.bytes1);
  const __amdgpu_buffer_rsrc_t rs2 = make_rsrc(g.src2 ? g.src2 : g.src1, g.src2 ? g.bytes2 : 0);
  const __amdgpu_buffer_rsrc_t rsw = make_rsrc(g.w, (uint32_t)((int64_t)g.N * g.ldw * 2));

  // loader: group j of this wave is rows (j * NL + wave) * 8 ..+8 of the tile
  // (A rows, then B rows); lane l loads row l / 8, slot l % 8
  const int lrow = lane >> 3;
  const int cch = (lane & 7) ^ lrow;
  const bool last = NG % NL == 0 || (PER - 1) * NL + wave < NG;  // this wave has a PER-th group
  auto is_a = [&](int j) {  // known at compile time unless group j straddles A and B rows
    return (j + 1) * NL <= GA || (j * NL < GA && j * NL + wave < GA);
  };
  auto has = [&](int j) { return j + 1 < PER || last; };
  int a_b[PER], a_oy[PER], a_ox[PER];  // conv: image, output row and column; dense: row; -1: none
  uint32_t voff[PER];
  const int cin = g.C1 + g.C2;
  int t_tap = 0, t_ci = kt0 * 64;  // dense: t_ci walks [0, K)
  if (MODE == 1) {
    t_tap = t_ci / cin;
    t_ci -= t_tap * cin;
  }
  bool t_first = true;
  uint32_t soffA = 0, soffB = (uint32_t)kt0 * 128;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int gi = j * NL + wave;
    a_b[j] = -1;
    a_oy[j] = a_ox[j] = 0;
    voff[j] = OOB;
    if (is_a(j)) {
      const int64_t m = m0 + gi * 8 + lrow;
      if (m < g.M) {
        if (MODE == 1) {
          const int hw = g.Ho * g.Wo;
          a_b[j] = (int)((uint32_t)m / (uint32_t)hw);
          const int p = (int)m - a_b[j] * hw;
          a_oy[j] = p / g.Wo;
          a_ox[j] = p - a_oy[j] * g.Wo;
        } else {
          a_b[j] = (int)m;
        }
      }
    } else {
      const int n = n0 + (gi - GA) * 8 + lrow;
      if (has(j) && n < g.N) voff[j] = (uint32_t)(((int64_t)n * g.ldw + cch * 8) * 2);
    }
  }
  // offsets of the A rows at the start of the current tap and source
  auto a_offsets = [&]() {
    t_first = t_ci < g.C1;
    soffA = (uint32_t)(t_first ? t_ci : t_ci - g.C1) * 2;
    const int ky = (t_tap * 11) >> 5, kx = t_tap - 3 * ky;
    const int ld = MODE == 1 ? (t_first ? g.C1 : g.C2) : (t_first ? g.lda1 : g.lda2);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      if (!is_a(j)) continue;
      if (MODE == 0) {
        voff[j] = a_b[j] >= 0 ? (uint32_t)(((int64_t)a_b[j] * ld + cch * 8) * 2) : OOB;
      } else {
        int iy, ix;
        bool in;
        if (g.upsample) {
          const int uy = a_oy[j] + ky - 1, ux = a_ox[j] + kx - 1;
          in = uy >= 0 && ux >= 0 && uy < 2 * g.Hin && ux < 2 * g.Win;
          iy = uy >> 1;
          ix = ux >> 1;
        } else {
          iy = a_oy[j] * g.stride + ky - 1;
          ix = a_ox[j] * g.stride + kx - 1;
          in = iy >= 0 && ix >= 0 && iy < g.Hin && ix < g.Win;
        }
        // below 2^31 bytes for the rows that are loaded
        const uint32_t pix = (uint32_t)((a_b[j] * g.Hin + iy) * g.Win + ix);
        voff[j] = a_b[j] >= 0 && in ? (pix * (uint32_t)ld + cch * 8) * 2 : OOB;
      }
    }
  };
  a_offsets();
  int t_next = 0;  // tiles requested
  // request the team's next tile into ring buffer `slot`; past its last tile
  // the last one is requested again (never multiplied), so every wave's count
  // of requests in flight stays fixed for the waits below
  auto issue = [&](int slot) {
    _Float16* dst = ring + slot * TILE_H;
    // the source is uniform: branch on it, so each descriptor stays in SGPRs
    if (__builtin_amdgcn_readfirstlane((int)t_first) != 0) {
#pragma unroll
      for (int j = 0; j < PER; ++j)
        if (is_a(j)) lds_dma16(rs1, voff[j], dst + (j * NL + wave) * 512, soffA);
    } else {
#pragma unroll
      for (int j = 0; j < PER; ++j)
        if (is_a(j)) lds_dma16(rs2, voff[j], dst + (j * NL + wave) * 512, soffA);
    }
#pragma unroll
    for (int j = 0; j < PER; ++j)
      if (!is_a(j) && has(j)) lds_dma16(rsw, voff[j], dst + (j * NL + wave) * 512, soffB);
    if (++t_next >= my_steps) return;
    soffB += 128 * KT;
    soffA += 128 * KT;
    const bool was_first = t_ci < g.C1;
    t_ci += 64 * KT;
    bool fresh = was_first && t_ci >= g.C1;
    if (MODE == 1)
      while (t_ci >= cin) {
        t_ci -= cin;
        ++t_tap;
        fresh = true;
      }
    if (fresh) a_offsets();
  };
  // all but the newest N tiles of this wave's requests have landed
  auto wait_tiles = [&](auto n, bool lgkm) {
    constexpr int N = decltype(n)::value;
    if (NG % NL == 0 || last) {
      if (lgkm) wait_vm_lgkm0<N * PER>();
      else wait_vmcnt<N * PER>();
    } else {
      if (lgkm) wait_vm_lgkm0<N * (PER - 1)>();
      else wait_vmcnt<N * (PER - 1)>();
    }
  };

  // Folded LayerNorm: TPR threads of the team per A row each sum CPT of its
  // eight 16-byte chunks per tile, shifted by the row's first value so that the
  // one-pass variance does not cancel (float16 shift, float32 dot2); the teams'
  // sums meet in LDS after the loop.
  constexpr int TPR = NL * 64 / BM, CPT = TPR > 0 ? 8 / TPR : 1;
  static_assert(!LN || (TPR >= 1 && TPR <= 8 && 8 % TPR == 0), "LayerNorm rows per team");
  const int ttid = tid % (NL * 64), st_row = LN ? ttid / TPR : 0, st_slot = LN ? (ttid % TPR) * CPT : 0;
  half2v st_shift = {(_Float16)0.f, (_Float16)0.f};
  float st_s1 = 0.f, st_s2 = 0.f;
  if (LN && m0 + st_row < g.M) {
    const _Float16 x0 = g.src1[(m0 + st_row) * g.lda1];
    st_shift = half2v{x0, x0};
  }
  auto stats = [&](int sl) {
    if constexpr (LN) {
      const _Float16* ar = ring + sl * TILE_H + st_row * 64;
      const half2v one = {(_Float16)1.f, (_Float16)1.f};
#pragma unroll
      for (int c = 0; c < CPT; ++c) {
        const half8 x = *(const half8*)(ar + (st_slot + c) * 8);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const half2v d = half2v{x[2 * e], x[2 * e + 1]} - st_shift;
          st_s1 = __builtin_amdgcn_fdot2(d, one, st_s1, false);
          st_s2 = __builtin_amdgcn_fdot2(d, d, st_s2, false);
        }
      }
    }
  };

  floatx4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  const int arow = (wm * WM + li) * 64, brow = (BM + wn * WN + li) * 64;
  const int s0 = ((kh * 4 + kc) ^ (li & 7)) << 3;  // slot of this group's (first) half
  const int s1 = ((4 + kc) ^ (li & 7)) << 3;       // second half (KH == 1)
  half8 fa0[FM], fb0[FN], fa1[FM], fb1[FN];
#pragma unroll
  for (int s = 0; s < STAGES; ++s) issue(s);
  wait_tiles(std::integral_constant<int, STAGES - 1>{}, false);
  ring_barrier();
  read_frags<FM, FN>(ring, arow + s0, brow + s0, fa0, fb0);
  int slot = 0;  // ring buffer of the tile being multiplied
  if (LN && my_steps > 0) stats(0);
  // multiply the current fragments while the next ones are read (the reads go
  // out between the first multiplies)
  auto mma = [&](half8 (&ca)[FM], half8 (&cb)[FN]) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(cb[j], ca[i], acc[i][j], 0, 0, 0);
    constexpr int PER_READ = (FM * FN * 3 / 4) / (FM + FN) > 0 ? (FM * FN * 3 / 4) / (FM + FN) : 1;
#pragma unroll
    for (int r = 0; r < FM + FN; ++r) {
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);         // one LDS read
      __builtin_amdgcn_sched_group_barrier(0x008, PER_READ, 0);  // multiplies
    }
  };
  // this wave's reads of the current tile are done and its part of the next
  // one has landed; after the barrier that holds for every wave
  auto turn = [&]() {
    wait_tiles(std::integral_constant<int, STAGES - 2>{}, true);
    ring_barrier();
    issue(slot);
    slot = slot + 1 == STAGES ? 0 : slot + 1;
  };
  if constexpr (KH == 1) {
    for (int t = 0; t < n_steps; ++t) {
      read_frags<FM, FN>(ring + slot * TILE_H, arow + s1, brow + s1, fa1, fb1);
      if (KT == 1 || t < my_steps) mma(fa0, fb0);
      turn();
      read_frags<FM, FN>(ring + slot * TILE_H, arow + s0, brow + s0, fa0, fb0);
      if (KT == 1 || t < my_steps) mma(fa1, fb1);
      if (LN && t + 1 < my_steps) stats(slot);
    }
  } else {
    auto step = [&](int t, half8 (&ca)[FM], half8 (&cb)[FN], half8 (&na)[FM], half8 (&nb)[FN]) {
      turn();
      read_frags<FM, FN>(ring + slot * TILE_H, arow + s0, brow + s0, na, nb);
      if (KT == 1 || t < my_steps) mma(ca, cb);
      if (LN && t + 1 < my_steps) stats(slot);
    };
    int t = 0;
    for (; t + 1 < n_steps; t += 2) {
      step(t, fa0, fb0, fa1, fb1);
      step(t + 1, fa1, fb1, fa0, fb0);
    }
    if (t < n_steps) step(t, fa0, fb0, fa1, fb1);
  }
  wait_vmcnt<0>();  // drain the requests past the last tile before LDS is reused

  __shared__ float2 lnst[LN ? KT * BM : 1];
  if constexpr (LN) {
#pragma unroll
    for (int o = 1; o < TPR; o <<= 1) {
      st_s1 += __shfl_xor(st_s1, o, 64);
      st_s2 += __shfl_xor(st_s2, o, 64);
    }
    if (ttid % TPR == 0) lnst[team * BM + st_row] = make_float2(st_s1, st_s2);
    __syncthreads();
    if (team == 0 && ttid % TPR == 0) {
      float2 u = lnst[st_row];
#pragma unroll
      for (int k = 1; k < KT; ++k) {
        u.x += lnst[k * BM + st_row].x;
        u.y += lnst[k * BM + st_row].y;
      }
      const float inv_k = 1.0f / (float)g.K;
      const float mu = u.x * inv_k;
      const float var = fmaxf(u.y * inv_k - mu * mu, 0.f);
      lnst[st_row] = make_float2((float)st_shift[0] + mu, rsqrtf(var + g.ln_eps));
    }  // published by the epilogue's first barrier
    if (g.geglu) __syncthreads();  // whose GEGLU form reads the rows before it
  }
  epilogue_rows<BM, BN, WGM, WGN, KH * KT, KT * STAGES * TILE_H * 2, LN>(
      g, (float*)smem, m0, n0, team * KH + kh, wm, wn, li, kc, acc, lnst);
}

// Sum split-K partials in split order and apply the epilogue, four
// consecutive columns per thread (N % 4 == 0, checked by the launcher).  The
// loads of up to RED_CHUNK splits are issued together before their adds (a
// loop of load-then-add would pay one memory round trip per split); the adds
// still run in split order, so the sum does not change.
constexpr int RED_CHUNK = 8;

// NQ quads at p + k * off (k < NQ), each summed over splits s_lo .. splits - 1
// into v[k].
template <int NQ>
__device__ inline void sum_splits(const float* __restrict__ p, int off, int64_t MN, int splits,
                                  float (&v)[NQ][4], int s_lo = 0) {
  constexpr int CH = RED_CHUNK / NQ;
  for (int s0 = s_lo; s0 < splits; s0 += CH) {
    float4 q[CH][NQ];
#pragma unroll
    for (int u = 0; u < CH; ++u)
#pragma unroll
      for (int k = 0; k < NQ; ++k)
        if (s0 + u < splits) q[u][k] = *(const float4*)(p + (s0 + u) * MN + k * off);
#pragma unroll
    for (int u = 0; u < CH; ++u)
#pragma unroll
      for (int k = 0; k < NQ; ++k)
        if (s0 + u < splits) {
          v[k][0] += q[u][k].x; v[k][1] += q[u][k].y; v[k][2] += q[u][k].z; v[k][3] += q[u][k].w;
        }
  }
}

// P threads (adjacent lanes) per output quad where more than RED_CHUNK splits
// would take a second round of loads: lane j of the P sums its share of the
// splits in one round, and the shares are added in a fixed tree (lane pairs,
// then pairs of pairs), so the result stays the same from call to call.
template <int P>
__global__ void __launch_bounds__(256) splitk_reduce(GemmArgs g, int splits) {
  static_assert(P == 1 || P == 2 || P == 4, "threads per quad");
  const int64_t MN = g.M * (int64_t)g.N;
  const int nq = g.N / 4;
  const int64_t total = g.geglu ? g.M * (int64_t)(g.N / 32) * 4 : g.M * (int64_t)nq;
  const int sub = threadIdx.x % P, per = (splits + P - 1) / P;
  for (int64_t e = ((int64_t)blockIdx.x * 256 + threadIdx.x) / P; e < total;
       e += (int64_t)gridDim.x * (256 / P)) {
    if (g.geglu) {  // e -> (row, 32-column group, quad of the 16 "a" columns)
      const int per_row = (g.N / 32) * 4;
      const int64_t m = e / per_row;
      const int rem = (int)(e - m * per_row);
      const int na = (rem >> 2) * 32 + (rem & 3) * 4;
      float ag[2][4] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};  // "a", gate
      sum_splits<2>(g.partial + m * g.N + na, 16, MN, splits, ag);
      store_geglu4(g, m, na, ag[0], ag[1], g.vec_ok);
    } else {
      const int64_t m = e / nq;
      const int n = (int)(e - m * nq) * 4;
      // the epilogue's operands first: their loads overlap those of the partials
      float b[4] = {0.f, 0.f, 0.f, 0.f}, rv[4] = {0.f, 0.f, 0.f, 0.f};
      half4 res = {};
      if (g.bias) {
        const float4 q = *(const float4*)(g.bias + n);
        b[0] = q.x; b[1] = q.y; b[2] = q.z; b[3] = q.w;
      }
      if (g.rowvec) {
        const float* p = g.rowvec + (m / g.rows_div) * (int64_t)g.ld_rowvec + n;
#pragma unroll
        for (int r = 0; r < 4; ++r) rv[r] = p[r];
      }
      const bool vtc = g.vt && n >= g.vt_col0;
      if (g.residual && !vtc) {
        const _Float16* p = g.residual + m * g.ld_res + n;
        if (g.vec_ok) {
          res = *(const half4*)p;
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r) res[r] = p[r];
        }
      }
      float v[1][4] = {{0.f, 0.f, 0.f, 0.f}};
      if (P == 1) {
        sum_splits<1>(g.partial + m * g.N + n, 0, MN, splits, v);
      } else {
        sum_splits<1>(g.partial + m * g.N + n, 0, MN, min(splits, (sub + 1) * per), v, sub * per);
#pragma unroll
        for (int o = 1; o < P; o <<= 1)
#pragma unroll
          for (int r = 0; r < 4; ++r) v[0][r] += __shfl_xor(v[0][r], o, 64);
        if (sub != 0) continue;
      }
      float w[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        w[r] = v[0][r];
        if (g.bias) w[r] += b[r];
        if (g.rowvec) w[r] += rv[r];
        if (g.silu) w[r] = silu(w[r]);
      }
      if (vtc) {  // transposed columns (no residual on these)
        _Float16* o = g.vt + (int64_t)(n - g.vt_col0) * g.vt_ld + (m / g.vt_div) * g.vt_stride +
                      m % g.vt_div;
#pragma unroll
        for (int r = 0; r < 4; ++r) o[(int64_t)r * g.vt_ld] = (_Float16)w[r];
        continue;
      }
      if (g.residual)
#pragma unroll
        for (int r = 0; r < 4; ++r) w[r] += (float)res[r];
      if (g.out_f32) {
        float* o = (float*)g.out + m * g.ldo + n;
        if (g.vec_ok)
          *(float4*)o = make_float4(w[0], w[1], w[2], w[3]);
        else
          for (int r = 0; r < 4; ++r) o[r] = w[r];
      } else {
        _Float16* o = (_Float16*)g.out + m * g.ldo + n;
        if (g.vec_ok) {
          half4 h;
#pragma unroll
          for (int r = 0; r < 4; ++r) h[r] = (_Float16)w[r];
          *(half4*)o = h;
        } else {
          for (int r = 0; r < 4; ++r) o[r] = (_Float16)w[r];
        }
      }
    }
  }
}

// Split-K reduction: one thread per output quad up to RED_CHUNK splits, two
// or four beyond (each then loads its share in one round).
hipError_t reduce_launch(const GemmArgs& g, int splits, hipStream_t s) {
  const int P = g.geglu || splits <= RED_CHUNK ? 1 : splits <= 2 * RED_CHUNK ? 2 : 4;
  const int64_t total = g.M * (int64_t)(g.N / 4) * P;
  const unsigned blocks = (unsigned)std::min<int64_t>(ceil_div(total, 256), 4096);
  if (P == 1)
    hipLaunchKernelGGL(splitk_reduce<1>, dim3(blocks), dim3(256), 0, s, g, splits);
  else if (P == 2)
    hipLaunchKernelGGL(splitk_reduce<2>, dim3(blocks), dim3(256), 0, s, g, splits);
  else
    hipLaunchKernelGGL(splitk_reduce<4>, dim3(blocks), dim3(256), 0, s, g, splits);
  return hipGetLastError();
}

template <int MODE, int BM, int BN, bool DUAL>
hipError_t launch_t(const GemmArgs& g, int splits, hipStream_t s) {
  if (g.bytes1 >= 0x80000000u || g.bytes2 >= 0x80000000u ||
      (int64_t)g.N * g.ldw * 2 >= 0x80000000ll)
    return hipErrorInvalidValue;  // descriptors address at most 2 GiB
  const size_t lds = (size_t)2 * (BM + BN) * ROW * 2;
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void*)gemm_f16<MODE, BM, BN, DUAL>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const int nk = (g.K + BK - 1) / BK;
  const int kps = (nk + splits - 1) / splits;
  splits = (nk + kps - 1) / kps;
  if (splits > 1 && (!g.partial || (size_t)splits * g.M * g.N * 4 > g.partial_bytes))
    return hipErrorInvalidValue;  // split-K partials must fit the scratch
  dim3 grid((unsigned)(ceil_div(g.M, BM) * ceil_div(g.N, BN)), 1, (unsigned)splits);
  const int fam = MODE == 1 ? NV_FAM_CONV : NV_FAM_LINEAR;
  const double flops = 2.0 * (double)g.M * g.N * g.K;
  const double bytes = (double)g.bytes1 + g.bytes2 + (double)g.N * g.K * 2 +
                       (double)g.M * (g.geglu ? g.N / 2 : g.N) * (g.out_f32 ? 4 : 2);
  const TraceEv ev =
      trace_begin(fam, flops, bytes, TraceShape{g.M, g.N, g.K, BM * 10000 + BN * 10 + splits});
  hipExtLaunchKernelGGL((gemm_f16<MODE, BM, BN, DUAL>), grid, dim3(256), (uint32_t)lds, s, ev.a,
                        ev.b, 0u, g, kps);
  if (splits > 1) return reduce_launch(g, splits, s);
  return hipGetLastError();
}

template <int MODE, int BM, int BN, int STAGES, bool LN, int U = 1, int NW = 4>
hipError_t launch_s_t(const GemmArgs& g, int splits, hipStream_t s) {
  // the GEGLU epilogue pairs a wave's 16-column quads: at least 32 columns per wave
  if (g.geglu && splits <= 1 && BN / (NW / 2) < 32) return hipErrorInvalidValue;
  if (g.bytes1 >= 0x80000000u || g.bytes2 >= 0x80000000u ||
      (int64_t)g.N * g.ldw * 2 >= 0x80000000ll)
    return hipErrorInvalidValue;  // descriptors address less than 2 GiB (gemm_launch chunks)
  const size_t lds = (size_t)STAGES * (BM + BN) * 64 * 2;
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void*)gemm_s<MODE, BM, BN, STAGES, LN, U, NW>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const int nk = g.K / 64;
  const int kps = (nk + splits - 1) / splits;
  splits = (nk + kps - 1) / kps;
  if (splits > 1 && (!g.partial || (size_t)splits * g.M * g.N * 4 > g.partial_bytes))
    return hipErrorInvalidValue;  // split-K partials must fit the scratch
  dim3 grid((unsigned)(ceil_div(g.M, BM) * ceil_div(g.N, BN)), 1, (unsigned)splits);
  const int fam = MODE == 1 ? NV_FAM_CONV : NV_FAM_LINEAR;
  const double flops = 2.0 * (double)g.M * g.N * g.K;
  const double bytes = (double)g.bytes1 + g.bytes2 + (double)g.N * g.K * 2 +
                       (double)g.M * (g.geglu ? g.N / 2 : g.N) * (g.out_f32 ? 4 : 2);
  const TraceEv ev =
      trace_begin(fam, flops, bytes, TraceShape{g.M, g.N, g.K, BM * 10000 + BN * 10 + splits});
  hipExtLaunchKernelGGL((gemm_s<MODE, BM, BN, STAGES, LN, U, NW>), grid, dim3(NW * 64),
                        (uint32_t)lds, s, ev.a, ev.b, 0u, g, kps);
  if (splits > 1) return reduce_launch(g, splits, s);
  return hipGetLastError();
}

// A folded LayerNorm needs every k tile of a row in one workgroup: no split.
template <int MODE, int BM, int BN, int STAGES, int U = 1, int NW = 4>
hipError_t launch_s(const GemmArgs& g, int splits, hipStream_t s) {
  if constexpr (MODE == 0)
    if (g.ln_c1) return launch_s_t<0, BM, BN, STAGES, true, U, NW>(g, 1, s);
  return launch_s_t<MODE, BM, BN, STAGES, false, U, NW>(g, splits, s);
}

template <int MODE, int BM, int BN, int WGM, int WGN, int KH, int KT, int STAGES, bool LN>
hipError_t launch_w_t(const GemmArgs& g, hipStream_t s) {
  constexpr int NW = KT * KH * WGM * WGN;
  if (!g.rows_ok || g.K % 64 != 0) return hipErrorInvalidValue;
  // epilogue_rows pairs GEGLU's quads in the registers of one wave
  if (g.geglu && (KH * KT != 1 || (BN / WGN / 16) % 2 != 0)) return hipErrorInvalidValue;
  if (g.bytes1 >= 0x80000000u || g.bytes2 >= 0x80000000u ||
      (int64_t)g.N * g.ldw * 2 >= 0x80000000ll)
    return hipErrorInvalidValue;  // descriptors address less than 2 GiB (gemm_launch chunks)
  constexpr size_t lds = (size_t)KT * STAGES * (BM + BN) * 64 * 2;
  static_assert(lds <= 160 * 1024, "LDS per workgroup");
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void*)gemm_w<MODE, BM, BN, WGM, WGN, KH, KT, STAGES, LN>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  dim3 grid((unsigned)(ceil_div(g.M, BM) * ceil_div(g.N, BN)));
  const int fam = MODE == 1 ? NV_FAM_CONV : NV_FAM_LINEAR;
  const double flops = 2.0 * (double)g.M * g.N * g.K;
  const double bytes = (double)g.bytes1 + g.bytes2 + (double)g.N * g.K * 2 +
                       (double)g.M * (g.geglu ? g.N / 2 : g.N) * 2;
  const TraceEv ev =
      trace_begin(fam, flops, bytes,
                  TraceShape{g.M, g.N, g.K, KH * KT * 100000000ll + BM * 10000 + BN * 10 + 1});
  hipExtLaunchKernelGGL((gemm_w<MODE, BM, BN, WGM, WGN, KH, KT, STAGES, LN>), grid, dim3(NW * 64),
                        (uint32_t)lds, s, ev.a, ev.b, 0u, g);
  return hipGetLastError();
}

template <int MODE, int BM, int BN, int WGM, int WGN, int KH, int KT, int STAGES>
hipError_t launch_w(const GemmArgs& g, hipStream_t s) {
  if constexpr (MODE == 0)
    if (g.ln_c1) return launch_w_t<0, BM, BN, WGM, WGN, KH, KT, STAGES, true>(g, s);
  return launch_w_t<MODE, BM, BN, WGM, WGN, KH, KT, STAGES, false>(g, s);
}

// Streamed kernel when every 64-deep k tile lies inside one source and tap.
template <int MODE>
bool streamable(const GemmArgs& g) {
  if (g.C1 % 64 != 0) return false;
  return MODE == 0 ? (g.K % 64 == 0) : ((g.C1 + g.C2) % 64 == 0);
}

template <int MODE, int BM, int BN>
hipError_t launch(const GemmArgs& g, int splits, hipStream_t s) {
  // the incremental single-source path needs every 64-deep tile inside one
  // source and inside K: C1 and K (dense) or C1 and Cin (conv) multiples of 64
  const bool dual = (g.C1 % BK) != 0 || (MODE == 0 && (g.K % BK) != 0) ||
                    (MODE == 1 && ((g.C1 + g.C2) % BK) != 0);
  return dual ? launch_t<MODE, BM, BN, true>(g, splits, s)
              : launch_t<MODE, BM, BN, false>(g, splits, s);
}

template <int MODE>
hipError_t dispatch_wide(const GemmArgs& g, int form, hipStream_t s) {
  switch (form) {  // in the order of WIDE
    case 0: return launch_w<MODE, 256, 256, 2, 4, 1, 1, 2>(g, s);
    case 1: return launch_w<MODE, 256, 160, 4, 2, 1, 1, 2>(g, s);
    case 2: return launch_w<MODE, 128, 160, 4, 2, 1, 1, 2>(g, s);
    case 3: return launch_w<MODE, 128, 160, 2, 2, 2, 1, 3>(g, s);
    case 4: return launch_w<MODE, 128, 128, 2, 4, 1, 1, 2>(g, s);
    case 5: return launch_w<MODE, 128, 80, 4, 1, 2, 1, 3>(g, s);
    case 6: return launch_w<MODE, 64, 128, 2, 2, 2, 1, 3>(g, s);
    case 7: return launch_w<MODE, 64, 80, 2, 1, 2, 2, 3>(g, s);
    case 8: return launch_w<MODE, 64, 64, 2, 2, 2, 1, 4>(g, s);
    default: return hipErrorInvalidValue;
  }
}

// Streamed products: the form is stream_plan's choice (gemm_rule.h).
template <int MODE>
hipError_t dispatch_streamed(const GemmArgs& g, hipStream_t s) {
  const StreamPlan p =
      stream_plan({g.M, g.N, g.K, MODE == 1, g.geglu != 0, g.ln_c1 != nullptr, g.rows_ok != 0,
                   g.partial ? g.partial_bytes : 0});
  if (p.wide >= 0) return dispatch_wide<MODE>(g, p.wide, s);
  if (p.bm == 128)
    return p.waves == 8 ? launch_s<MODE, 128, 128, GEMM_S128, 1, 8>(g, p.splits, s)
                        : launch_s<MODE, 128, 128, GEMM_S128>(g, p.splits, s);
  if (p.bn == 128) return launch_s<MODE, 64, 128, 2, 1, 8>(g, p.splits, s);
  return p.waves == 8 ? launch_s<MODE, 64, 64, 4, 1, 8>(g, p.splits, s)
                      : launch_s<MODE, 64, 64, GEMM_S64>(g, p.splits, s);
}

template <int MODE>
hipError_t dispatch(const GemmArgs& g, hipStream_t s) {
  if (g.ln_c1 && (MODE != 0 || g.src2 || !streamable<MODE>(g))) return hipErrorInvalidValue;
  if (streamable<MODE>(g)) return dispatch_streamed<MODE>(g, s);
  // Larger tiles move fewer bytes per flop (64, 43 and 32 flop per byte of
  // L2 traffic for 128x128, 128x64, 64x64).  At these problem sizes a
  // workgroup is bound by load latency (about one wave per SIMD), so K is
  // split until about two workgroups per CU are resident, keeping at least
  // MIN_KT k tiles per split.
  constexpr int64_t MIN_WG = 128;
  constexpr int64_t TARGET = 512;
  const int nk = (g.K + BK - 1) / BK;
  const int64_t t128 = ceil_div(g.M, 128) * ceil_div(g.N, 128);
  const int64_t t12864 = ceil_div(g.M, 128) * ceil_div(g.N, 64);
  const int64_t t64 = ceil_div(g.M, 64) * ceil_div(g.N, 64);
  const bool n_fits_128 = g.N % 128 == 0 || g.N > 512;
  auto split_for = [&](int64_t tiles, int min_kt) {
    int sp = 1;
    if (!g.partial || (g.N & 3) != 0) return 1;
    while (tiles * sp < TARGET && nk / (sp + 1) >= min_kt &&
           (size_t)(sp + 1) * g.M * g.N * 4 <= g.partial_bytes)
      ++sp;
    return sp;
  };
  if (t128 >= MIN_WG && n_fits_128) return launch<MODE, 128, 128>(g, split_for(t128, 8), s);
  if (t12864 >= MIN_WG) return launch<MODE, 128, 64>(g, split_for(t12864, 8), s);
  return launch<MODE, 64, 64>(g, split_for(t64, 4), s);
}

hipError_t gemm_launch_one(const GemmArgs& gin, hipStream_t s) {
  GemmArgs g = gin;
  // byte extents of the A sources for the range descriptors
  if (g.conv) {
    const int64_t rows = g.M / ((int64_t)g.Ho * g.Wo);
    const int64_t pix = rows * g.Hin * g.Win;
    g.bytes1 = (uint64_t)(pix * g.C1 * 2);
    g.bytes2 = g.src2 ? (uint64_t)(pix * g.C2 * 2) : 0;
  } else {
    g.bytes1 = (uint64_t)(((g.M - 1) * g.lda1 + g.C1) * 2);
    g.bytes2 = g.src2 ? (uint64_t)(((g.M - 1) * g.lda2 + g.C2) * 2) : 0;
  }
  g.n_major = (int64_t)g.N >= g.M;  // weights at least as large as the activation rows
  // quads of 4 output columns move as vectors when every row stride and base
  // keeps them aligned (8 bytes float16, 16 bytes float32 / bias)
  auto al = [](const void* p, int a) { return ((uintptr_t)p & (a - 1)) == 0; };
  g.vec_ok = (g.N % 4 == 0) && (g.ldo % 4 == 0) && al(g.out, g.out_f32 ? 16 : 8) &&
             (!g.bias || al(g.bias, 16)) &&
             (!g.residual || ((g.ld_res % 4 == 0) && al(g.residual, 8)));
  g.rows_ok = row_epilogue_ok(g);
  return g.conv ? dispatch<1>(g, s) : dispatch<0>(g, s);
}

}  // namespace

// The buffer descriptors address less than 2 GiB (the out-of-range offset is
// 2^31), so a product whose A source reaches that runs as a sequence of row
// chunks below it, each a product of its own on the same stream.  Chunks hold
// whole units: one sample's output pixels for a convolution, and for a dense
// product the rows that share a row-vector entry or a transposed-output
// column block (both indexed per sample).  Weights of 2 GiB or more, or a
// single unit that large, are rejected.
hipError_t gemm_launch(const GemmArgs& g, hipStream_t s) {
  constexpr uint64_t LIMIT = 0x80000000ull;
  if ((uint64_t)g.N * (uint64_t)g.ldw * 2 >= LIMIT) return hipErrorInvalidValue;
  int64_t unit = 1;
  uint64_t ub1 = 0, ub2 = 0, src_u1 = 0, src_u2 = 0;  // bytes / halfs of source per unit
  if (g.conv) {
    unit = (int64_t)g.Ho * g.Wo;
    if (unit <= 0 || g.M % unit) return hipErrorInvalidValue;
    src_u1 = (uint64_t)g.Hin * g.Win * g.C1;
    src_u2 = (uint64_t)g.Hin * g.Win * g.C2;
  } else {
    auto lcm = [](int64_t a, int64_t b) { return a / std::__gcd(a, b) * b; };
    if (g.rowvec && g.rows_div > 1) unit = lcm(unit, g.rows_div);
    if (g.vt && g.vt_div > 1) unit = lcm(unit, g.vt_div);
    src_u1 = (uint64_t)unit * g.lda1;
    src_u2 = g.src2 ? (uint64_t)unit * g.lda2 : 0;
  }
  ub1 = src_u1 * 2;
  ub2 = src_u2 * 2;
  const uint64_t ub = std::max(ub1, ub2);
  const int64_t units = ceil_div(g.M, unit);
  if (ub == 0 || (uint64_t)units * ub < LIMIT) return gemm_launch_one(g, s);
  const int64_t per = (int64_t)((LIMIT - 1) / ub);  // units per chunk
  if (per < 1) return hipErrorInvalidValue;
  const size_t osz = g.out_f32 ? 4 : 2;
  for (int64_t u0 = 0; u0 < units; u0 += per) {
    const int64_t m0 = u0 * unit;
    GemmArgs c = g;
    c.M = std::min<int64_t>(g.M - m0, per * unit);
    c.src1 = g.src1 + u0 * src_u1;
    if (g.src2) c.src2 = g.src2 + u0 * src_u2;
    c.out = (char*)g.out + (size_t)m0 * g.ldo * osz;
    if (g.residual) c.residual = g.residual + m0 * g.ld_res;
    if (g.rowvec) c.rowvec = g.rowvec + (m0 / g.rows_div) * g.ld_rowvec;
    if (g.vt) c.vt = g.vt + (m0 / g.vt_div) * g.vt_stride;
    const hipError_t e = gemm_launch_one(c, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace nv
