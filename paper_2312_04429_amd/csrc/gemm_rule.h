// Which kernel form a product whose every 64-deep k tile lies in one source takes
// (host only; no HIP in this file).
#pragma once
#include <cstddef>
#include <cstdint>

namespace nv {

struct StreamShape {
  int64_t M;
  int N, K;              // K a multiple of 64
  bool conv, geglu, ln;  // ln: LayerNorm of the rows folded in (one workgroup needs all of K)
  bool rows_ok;          // the row-staged epilogue of the wide kernel applies
  size_t partial_bytes;  // split-K scratch, 0 without
};

// Whether the row-staged epilogue (epilogue_rows) takes a product: 8 float16
// columns, or 8 tokens of a transposed column, move as one 16-byte access.  It adds
// neither a row vector nor a residual to transposed columns; the other epilogues
// add the row vector there, so a product with both is theirs.  Args: GemmArgs
// (vec_ok filled in).
template <typename Args>
inline bool row_epilogue_ok(const Args& g) {
  auto aligned = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
  constexpr int64_t LIMIT = int64_t(1) << 31;
  return g.vec_ok && !g.out_f32 && g.M < LIMIT && g.N % (g.geglu ? 32 : 8) == 0 &&
         g.ldo % 8 == 0 && aligned(g.out) && (!g.rowvec || g.rows_div < LIMIT) &&
         (!g.residual || (g.ld_res % 8 == 0 && aligned(g.residual))) &&
         (!g.vt || (!g.geglu && !g.rowvec && g.M % 8 == 0 && g.vt_col0 % 8 == 0 &&
                    g.vt_ld % 8 == 0 && g.vt_div % 8 == 0 && g.vt_div < LIMIT &&
                    g.vt_stride % 8 == 0 && aligned(g.vt)));
}

// wide: index into WIDE (one share of K; waves unused), or -1: gemm_s with bm x
// bn tiles, `waves` waves and `splits` shares of K (the launcher rounds the shares
// to whole k tiles, which can leave fewer).
struct StreamPlan {
  int wide, bm, bn, waves, splits;
};

// Forms of the wide kernel and their cost in us: a launch costs 5, a single
// round of tiles f1 + s1 per 64-deep k tile, and each of several rounds f2 + s2
// per k tile.  A round is 256 tiles with one workgroup per CU, 512 with two (its
// last one, if it has at most 256 tiles, costs f1 and s1).  The constants were
// fitted, first of all so that the chosen form costs least, to 1124 graph-timed
// products (the UNet's layers at other resolutions, batches and channel counts: 16
// to 65536 rows, 1 to 360 k tiles, weights warm and streaming from HBM) and 363
// layers timed inside networks (78 with a folded LayerNorm): the choice takes 0.4 to
// 1 % more than the fastest form on average, and 0.6 % on 497 further products.  The
// small-tile kernels alone take 17 % longer; 15 of the 1984 lose more than 3 %
// against them, 16 % at most.
struct WideForm {
  int bm, bn, shares, per_cu;  // shares: wave groups that share out k (KH * KT)
  float f1, s1, f2, s2;
};
constexpr WideForm WIDE[] = {
    {256, 256, 1, 1, 11.10f, 1.354f, 12.18f, 1.105f},  // 0: 8 waves of 128 x 64
    {256, 160, 1, 1, 9.27f, 0.856f, 11.09f, 0.807f},   // 1: 8 waves of 64 x 80
    {128, 160, 1, 2, 4.43f, 0.590f, 5.20f, 0.909f},    // 2: 8 waves of 32 x 80
    {128, 160, 2, 1, 4.23f, 0.517f, 6.00f, 0.585f},    // 3: 2 k halves x 4 waves of 64 x 80
    {128, 128, 1, 2, 1.60f, 0.699f, 6.03f, 0.743f},    // 4: 8 waves of 64 x 32
    {128, 80, 2, 2, 0.94f, 0.401f, 4.39f, 0.615f},     // 5: 2 k halves x 4 waves of 32 x 80
    {64, 128, 2, 2, 0.34f, 0.324f, 2.45f, 0.527f},     // 6: 2 k halves x 4 waves of 32 x 64
    {64, 80, 4, 1, 1.27f, 0.247f, 1.20f, 0.215f},      // 7: 2 k halves x 2 teams x 2 waves of 32 x 80
    {64, 64, 2, 2, 0.22f, 0.240f, 1.81f, 0.357f},      // 8: 2 k halves x 4 waves of 32 x 32
};
constexpr int WIDE_FORMS = sizeof(WIDE) / sizeof(WIDE[0]);
constexpr int CUS = 256;

inline int64_t tiles_of(const StreamShape& g, int bm, int bn) {
  return ((g.M + bm - 1) / bm) * (((int64_t)g.N + bn - 1) / bn);
}

inline float wide_cost(const WideForm& w, const StreamShape& g) {
  const int64_t tiles = tiles_of(g, w.bm, w.bn);
  const float n = (float)(g.K / 64), one = w.f1 + n * w.s1, each = w.f2 + n * w.s2;
  if (w.per_cu == 1) return 5.0f + (tiles <= CUS ? one : (float)((tiles + CUS - 1) / CUS) * each);
  const int64_t rem = tiles % (2 * CUS);
  return 5.0f + (float)(tiles / (2 * CUS)) * each + (rem == 0 ? 0.f : rem <= CUS ? one : each);
}

// GEGLU pairs its quads in registers: forms whose waves hold all of k and
// whole 32-column groups.
inline bool wide_takes(const WideForm& w, const StreamShape& g) {
  return !g.geglu || (w.shares == 1 && w.bn % 160 != 0);
}

// Tiles and split of gemm_s (GPU time measured on the UNet's shapes).  A
// workgroup here is bound by the latency of its k-tile loads (about 0.4 us per
// tile), so small tiles and many resident workgroups win: K is split when it is
// long (> 40 tiles) or the grid is tiny, keeping >= MIN_KT tiles per split.
// Unsplit forms serve what the row-staged epilogue does not take (column counts
// off the grid of 8, float32 outputs, unaligned buffers) and small GEGLU grids;
// large grids of those take tiles of 128 x 128 where very wide or deep and up to
// 320 columns, 64 x 128 otherwise.
inline StreamPlan gemm_s_plan(const StreamShape& g) {
  constexpr int MIN_KT = 10;
  const int nk = g.K / 64;
  const int64_t t128 = tiles_of(g, 128, 128), t64 = tiles_of(g, 64, 64);
  auto split_to = [&](int64_t tiles, int64_t target) {
    int sp = 1;
    if (g.partial_bytes == 0 || g.N % 4 != 0 || g.ln) return 1;
    while (tiles * (sp + 1) <= target && nk / (sp + 1) >= MIN_KT &&
           (size_t)(sp + 1) * g.M * g.N * 4 <= g.partial_bytes)
      ++sp;
    return sp;
  };
  if (t64 >= 1024) {
    const bool big = (g.N >= 2560 && t128 >= 1536) || g.K >= 8192 || g.N <= 320 ||
                     (g.M >= 4096 && g.N >= 2560 && g.K >= 1280) ||
                     (g.M >= 4096 && g.N >= 1280 && g.K >= 4096) ||
                     (!g.conv && g.M >= 8192 && g.N >= 960);
    return big ? StreamPlan{-1, 128, 128, 8, 1} : StreamPlan{-1, 64, 128, 8, 1};
  }
  if (t128 >= 128 && nk >= 128) return {-1, 128, 128, 4, split_to(t128, 512)};
  // deep convolutions over mid-sized grids (batch 1 at 32 x 32 and 16 x 16):
  // 128 x 128 tiles halve the bytes per flop, split K refills the chip
  // (graph-timed 47 against 64 us at 32 x 32 with 1280 input channels); eight
  // waves (b1 guided step 5.296 -> 5.279 ms against four)
  if (g.conv && t128 >= 32 && t128 <= 128 && nk >= 80)
    return {-1, 128, 128, 8, split_to(t128, 700)};
  const bool split = nk > 40 || t64 < 100;
  if (!split && t64 >= 768 && g.N >= 1920) return {-1, 64, 128, 8, 1};
  // convolutions aim at fewer workgroups in total: fewer float32 partials to
  // write and sum (b1 guided step: the batch-1 8 x 8 convolutions at 12 splits
  // instead of 17, 5.365 -> 5.318 ms; 15 splits 5.360, 10 splits 5.346)
  const int spl = split ? split_to(t64, g.conv ? 480 : 700) : 1;
  // up to about two workgroups per CU: eight waves in 2 x 4 wave tiles of
  // 32 x 16 and a four-tile ring, 64 KB, two workgroups per CU (b1 guided step
  // 5.208 -> 5.117 ms).  The GEGLU epilogue pairs 16-column quads inside a wave and
  // keeps four.
  return {-1, 64, 64, !g.geglu && t64 * spl <= 512 ? 8 : 4, spl};
}

// Cost in us of a split plan: the products' workgroups, bound by their k tiles
// in turn or by the chip's rate over all of them, and the reduction (its launch
// and the partials).  Fitted to the 227 shapes of those above that split.
inline float split_cost(const StreamPlan& p, const StreamShape& g) {
  struct C { float fix, tile, wg, wg_tile, red, red_mb; };
  const C c = p.bm == 64 ? (p.waves == 8 ? C{0.35f, 0.222f, 1.345f, 0.230f, 2.616f, 1.169f}
                                         : C{0.00f, 0.591f, 1.943f, 0.070f, 2.861f, 1.440f})
                         : (p.waves == 8 ? C{2.53f, 1.099f, 2.987f, 0.530f, 5.532f, 0.f}
                                         : C{0.00f, 0.981f, 7.183f, 0.473f, 0.000f, 0.998f});
  const int nk = g.K / 64, per = (nk + p.splits - 1) / p.splits, splits = (nk + per - 1) / per;
  const float wgs = (float)(tiles_of(g, p.bm, p.bn) * splits) / CUS;
  const float chain = per * c.tile, rate = wgs * (c.wg + per * c.wg_tile);
  return 5.0f + c.fix + (chain > rate ? chain : rate) + c.red +
         (float)splits * (float)g.M * (float)g.N * 1e-6f * c.red_mb;
}

// The cheapest wide form, unless gemm_s would split K (2 shares or more) for less:
// a dense product if its estimate is 1 us or more below that form's (its second
// launch costs as much again where launches are not captured), a convolution
// if it is up to 6 % above (the estimates are good to about 10 % each, and the
// timings above had the fewest wrong choices there).  Unsplit gemm_s is not
// priced: the wide forms are its equals or better wherever both apply, but for
// GEGLU, whose two forms have few tiles and are slower up to 320 of 128 x 128 (inside
// the network 128 x 10240 x 1280, 80 tiles, 19.0 us on small tiles, 26.3 on form 4;
// 512 x 5120 x 640, 160 tiles, 14.1 and 14.9; 512 x 10240 x 1280, 320 tiles, 31.6 and
// 31.8; 768 x 10240 x 1280, 480 tiles, 44.0 and 31.7).
inline StreamPlan stream_plan(const StreamShape& g) {
  const StreamPlan s = gemm_s_plan(g);
  if (!g.rows_ok || (g.geglu && tiles_of(g, 128, 128) <= 320)) return s;
  int best = -1;
  float cost = 0.f;
  for (int i = 0; i < WIDE_FORMS; ++i) {
    if (!wide_takes(WIDE[i], g)) continue;
    // the fits hold no GEGLU products, whose gates cost form 4 more (1024 x 10240 x
    // 1280 52.3 us against 45.9 of form 0, 8192 x 5120 x 640 79.1 against 76.1, both
    // estimated about equal)
    const float c = wide_cost(WIDE[i], g) * (g.geglu && WIDE[i].bm == 128 ? 1.06f : 1.0f);
    if (best < 0 || c < cost) {
      best = i;
      cost = c;
    }
  }
  if (s.splits > 1 && !g.geglu &&
      (g.conv ? split_cost(s, g) + 0.5f < 1.06f * cost : split_cost(s, g) + 1.0f < cost))
    return s;
  return {best, WIDE[best].bm, WIDE[best].bn, 0, 1};
}

}  // namespace nv
