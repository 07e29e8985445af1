// Which bf16 scan a lookup takes (host only; no HIP in this file).
#pragma once
#include <cstdint>

namespace nv {

// Two scans read a bf16 cache of padded width dp <= 768 in tiles of 128 rows:
// one holds a tile's rows in registers and streams the queries past them (two
// workgroups per CU, so 512 tiles at once; the cache is read once for any
// number of queries), the other holds 16 * blocks queries per wave and streams
// the rows (one persistent workgroup per CU; the cache is read, and every query
// slot multiplied, once per pass of 64 * blocks queries).  Which one is faster
// follows from how well m fills the passes: over 4 M x 768 rows 65 queries take
// 1161 us row-resident against 1192, 128 queries 1489 against 1261, 129 to 256
// queries 1625 to 2286 against 1582 to 1749, but 272 queries 2403 against 3336
// and 512 queries 3713 against 3545; over 1 M x 384 rows 144 queries 219 against
// 275; over 2 M x 256 rows 256 queries 386 against 428.
//
// Costs in us, fitted to 468 timings (3000 to 4 M rows, widths 256 to 768, 48
// to 1024 queries; the choice is within 2.1 % of the row-resident time in all
// of them and 0.2 % from the faster form on average): a round of 512 tiles takes
// row + block us per 16 queries row-resident; a round of 256 tiles takes pass2 or
// pass4 us with two or four query blocks per wave, and pair2 or pair4 for two
// passes (narrow rows leave registers and LDS for two workgroups per CU, which
// then run two passes at once; twice one pass otherwise).
struct ScanCost {
  int dp;
  float row, block, pass2, pair2, pass4, pair4;
};
constexpr ScanCost SCAN_COST[] = {{256, 3.5f, 0.54f, 5.3f, 7.2f, 6.5f, 9.4f},
                                  {384, 6.5f, 0.76f, 6.3f, 9.0f, 8.4f, 16.8f},
                                  {512, 7.2f, 1.06f, 6.5f, 13.0f, 8.4f, 16.8f},
                                  {640, 11.1f, 1.42f, 9.4f, 18.8f, 11.4f, 22.8f},
                                  {768, 13.9f, 1.42f, 10.2f, 20.4f, 12.7f, 25.4f}};

// Query blocks per wave (2 or 4) of the query-resident scan, or 0 for the
// row-resident one.  tiles: 128-row tiles of the cache.  Up to 64 queries the
// row-resident scan is as fast or faster everywhere, and up to 128 wide too (the
// ring then holds few bytes in flight: 200 k x 64, 65 queries 31 us against 52).
inline int resident_query_blocks(int64_t tiles, int dp, int m) {
  if (m <= 64 || tiles <= 0) return 0;
  const ScanCost* c = nullptr;
  for (const ScanCost& s : SCAN_COST)
    if (s.dp == dp) c = &s;
  if (!c) return 0;
  // row-resident: whole rounds run two workgroups per CU, a last one part filled;
  // a workgroup that has its CU to itself takes 0.55 of the time
  const float t = (float)tiles;
  float row = c->row + c->block * (float)((m + 15) / 16);
  if (tiles <= 256)
    row *= 0.55f;
  else if (tiles < 512)
    row *= 0.55f + 0.45f * (t - 256.0f) / 256.0f;
  row *= t / 512.0f + 0.31f > 1.0f ? t / 512.0f + 0.31f : 1.0f;
  auto resident = [&](int blocks, float pass, float pair) {
    const int64_t passes = (m + 64 * blocks - 1) / (64 * blocks);
    // fewer tiles than CUs: the passes run side by side
    if (tiles < 256) return (float)((tiles * passes + 255) / 256) * pass;
    return (float)((tiles + 255) / 256) * ((float)(passes / 2) * pair + (float)(passes % 2) * pass);
  };
  const float q2 = resident(2, c->pass2, c->pair2), q4 = resident(4, c->pass4, c->pair4);
  if ((q2 < q4 ? q2 : q4) * 1.03f >= row) return 0;
  return q2 <= q4 ? 2 : 4;
}

}  // namespace nv
