// Which kernel a call takes: rules on sizes alone, on the host.
#pragma once

#include <stdint.h>

namespace fp8q {

struct GemmSize {
  int64_t M, N, K;
};

constexpr int kCUs = 256;
constexpr int kBlockK = 128;  // depth of a K block

// The kernels of gemm.hip.  All but the last three sum an output's K blocks
// in one order.
enum GemmRoute {
  kLargeTiles,  // 256 x 256 tiles, eight waves of 128 x 64
  kMidTiles,    // 128 x 128 tiles, four waves of 64 x 64, two workgroups per CU
  kEightWaves,  // 128 x 128 tiles, eight waves of 32 x 64
  kSmallTiles,  // 64 x 64 tiles, four waves of 32 x 32, two workgroups per CU
  kTwoKGroups,  // the same with two groups of waves on every other K block each
  kThinTiles,   // 16 x 16 to 64 x 64 tiles, every wave its own K blocks
  kSplitK       // 128 x 128 tiles, the K blocks over several workgroups
};

// Thin tiles of kThinM x kThinN outputs.
enum { kThin16x16, kThin16x32, kThin32x32, kThin32x64, kThin64x64, kThinConfigs };
constexpr int kThinM[kThinConfigs] = {16, 16, 32, 32, 64}, kThinN[kThinConfigs] = {16, 32, 32, 64, 64};

inline int64_t tile_count(const GemmSize& s, int bm, int bn) { return ((s.M + bm - 1) / bm) * ((s.N + bn - 1) / bn); }

// The grid of a large launch of `total` 256 x 256 tiles: `full` whole tiles,
// then the rest in `parts` (see large_tiles).  The last round is cut when its
// parts fit in one round of the CUs: up to a quarter of them in four, up to
// half in two; a fuller last round keeps whole tiles.
struct LargePlan {
  int full, parts, grid;
};
inline LargePlan large_plan(int64_t total) {
  const int rest = (int)(total % kCUs), rounds = (int)(total / kCUs);
  LargePlan p;
  p.parts = rest == 0 || rest > kCUs / 2 ? 1 : (rest <= kCUs / 4 ? 4 : 2);
  p.full = p.parts == 1 ? (int)total : rounds * kCUs;
  p.grid = p.full + (p.parts == 1 ? 0 : rest * p.parts);
  return p;
}

// Whether a launch of `outputs` outputs takes less time in `big` tiles of 256
// x 256 than in `mid` tiles of 128 x 128 (four waves).  Estimates in ns, fitted
// to both kernels' times at 4600 random sizes with more than 256 of the latter
// (K 128 to 25600, every pair; 7% from them, their ratio 5%): a round of kCUs
// large tiles, or of two 128 x 128 tiles per CU, takes a constant and a time
// per K block (kBlockNs); a last round a share of that which grows with how
// full it is.  Short K is the 128 x 128 tiles': a large tile's first loads and
// its epilogue overlap nothing (16384 x 128 x 6144, 1x128 x 1x128: 64.1 us on
// large tiles, 49.7 on the others; 3000 x 128 x 8192, 1x128 x 128x128: 15.5 and
// 12.4; at K = 4096 1x128 x 1x128 455 and 400 the other way).  Within a few
// percent the side that holds on more of the sizes: large from 512 tiles on,
// where they fill whole rounds or a last one in halves, and for one long round
// that more than 512 of the others would need two for (K >= 3072; measured
// 0.85 to 0.98 of them, not with 1x128 x 1x128 scales: 0.92 to 1.04).  1% of
// those sizes are more than 2.5% slower than with the rule "large from 512
// tiles on, 1x128 x 1x128 never"; 15% were with estimates of K = 4096 for
// every K.  Those were bursts on codes of random bits; run for long on
// quantized normal values, at the clock that the power limit holds, the 128 x
// 128 tiles take up to 3% longer beside the large ones with 1x128 x 1x128
// scales and quantized output (6528 x 1280 x 16384 178 us, large 168; 2500 x
// 2048 x 8192 quantized 55.1 and 51.8), and their times per K block here are
// those.
struct BlockNs {
  int large, mid;
};
constexpr BlockNs kBlockNs[6] = {{1614, 892},   // tensor
                                 {1614, 892},   // row
                                 {1814, 1031},  // 1x128 x 128x128
                                 {2204, 1180},  // 1x128 x 1x128
                                 {1708, 983},   // power-of-two scales
                                 {1944, 1100}}; // quantized output
// forms: the GemmPair values, then
constexpr int kFormQuantized = 5;

inline bool takes_large(int form, int64_t big, int64_t mid, int64_t outputs, int64_t K) {
  // (one round of halves alone: 2 to 11% slower at every K)
  if (mid <= kCUs || big <= kCUs / 2) return false;
  const double kb = (double)(K / kBlockK), common = form == kFormQuantized ? 2890 + outputs * (8240 / 16777216.0)
                                                                           : 2161 + outputs * (4506 / 16777216.0);
  const double l = kBlockNs[form].large * kb, m = kBlockNs[form].mid * kb;
  const int64_t rest = big % kCUs, rest_mid = mid % (2 * kCUs);
  const double fill = rest / (double)kCUs, fill_mid = rest_mid / (2.0 * kCUs);
  double large = common + (big / kCUs) * (2757 + l), tiled = common + (mid / (2 * kCUs)) * (641 + m);
  if (rest > kCUs / 2)
    large += 2452 + l * (0.566 + 0.357 * fill);
  else if (rest > kCUs / 4)
    large += 1561 + l * (0.486 + 0.159 * fill);
  else if (rest > 0)
    large += 1884 + l * (0.201 + 0.416 * fill);
  if (rest_mid > kCUs)
    tiled += 1043 + m * (0.897 + 0.109 * fill_mid);
  else if (rest_mid > 0)
    tiled += 1404 + m * (0.472 + 0.099 * fill_mid);
  const bool one_long = big < kCUs && mid > 2 * kCUs && K >= 24 * kBlockK && form != 3;
  const bool even = rest == 0 || (rest > kCUs / 4 && rest <= kCUs / 2 && K >= 8 * kBlockK);
  return large < tiled * (one_long ? 1.05 : big >= 2 * kCUs || even ? 1.02 : 0.98);
}

// Two K groups per 64 x 64 tile (one workgroup of 8 waves per CU) when there
// are at most 256 such tiles, so that a CU would hold one workgroup anyway,
// and the K blocks split evenly; more tiles keep two 4-wave workgroups per
// CU (their combined 4-stage rings already keep the loads in flight;
// measured faster there).
inline bool k_groups(const GemmSize& s) { return tile_count(s, 64, 64) <= kCUs && (s.K / kBlockK) % 2 == 0; }

// Time of the kernels for problems of at most kCUs 128 x 128 tiles, in ns: a
// constant, and for each round of one tile per CU a constant (first loads,
// epilogue, the meeting of partial tiles), a step per K block of a wave's
// chain, and the bytes that the CU loads, (bm + bn) K.  Fitted to all of these
// kernels' times at 8700 random sizes (K 128 to 25600, every pair, weights
// rotated through 3 x up to 160 MB), to choose well among them: the choice is
// 1.2% above the best of them on average (1.8% with the operand rows per CU
// alone, which sent short K to thin tiles: 192 x 128 x 8192 7.7 us, here 4.2;
// 27% with no thin tiles).
struct TileCost {
  int bm, bn, chain;  // chain: K blocks of one step of every wave
  int base, round, step, load;  // load: per 100 KB
};
constexpr TileCost kEightWavesCost = {128, 128, 1, 1468, 1889, 350, 337};
constexpr TileCost kTwoKGroupsCost = {64, 64, 2, 826, 2050, 0, 36};  // (step: kTwoKGroupsStep)
constexpr TileCost kSmallTilesCost = {64, 64, 1, 2185, 489, 220, 62};
constexpr TileCost kThinCost[kThinConfigs] = {{16, 16, 8, 2342, 156, 195, 233},
                                              {16, 32, 8, 2336, 94, 245, 597},
                                              {32, 32, 8, 2160, 554, 325, 717},
                                              {32, 64, 8, 1056, 1577, 488, 705},
                                              {64, 64, 8, 820, 2569, 685, 727}};

// Two K groups' step by form (the pairs' vector operations show there): thin
// 64 x 64 tiles, which take as long at K = 8192 with block scales, do so from
// 17408 with tensor and row scales.
constexpr int kTwoKGroupsStep[6] = {385, 385, 416, 400, 416, 416};

// `rounds`: of one tile per CU
inline double tile_ns(const TileCost& c, double rounds, int64_t K) {
  const int64_t steps = (K / kBlockK + c.chain - 1) / c.chain;
  return c.base + rounds * (c.round + c.step * (double)steps + c.load * (c.bm + c.bn) * (K / 1e5));
}

// The thin tile that takes the least time for the problems of one launch (of
// one K), and that time.
inline int thin_config(const GemmSize* probs, int count, double& ns) {
  int best = 0;
  for (int c = 0; c < kThinConfigs; ++c) {
    int64_t tiles = 0;
    for (int i = 0; i < count; ++i) tiles += tile_count(probs[i], kThinM[c], kThinN[c]);
    const double t = tile_ns(kThinCost[c], (double)((tiles + kCUs - 1) / kCUs), probs[0].K);
    if (c == 0 || t < ns) {
      best = c;
      ns = t;
    }
  }
  return best;
}

// Few rows against weights too large to stay in the last-level cache between
// calls: thin tiles, which read each weight row in pieces of 1 KB or less,
// take this much longer (33 to 80 x 25600 x 5120: 40-48 us, split 37-44; 24 x
// 12288 x 12288: 35, with two K groups 32; 128 x 25600 x 5120: 62, with two K
// groups 65).
inline double thin_from_memory(const GemmSize& s) { return s.M <= 96 && (s.M + s.N) * s.K > 80000000 ? 1.2 : 1.0; }

// Whether a problem too small for the 128 x 128 tiles of four waves is thin:
// against the kernel it takes else (see gemm_route).  Of 64 x 64 tiles without
// K groups two workgroups share a CU and even out.
inline bool is_thin(int form, const GemmSize& s) {
  const int64_t t64 = tile_count(s, 64, 64), mid = tile_count(s, 128, 128);
  double tiled, thin;
  if (k_groups(s))
    tiled = tile_ns(kTwoKGroupsCost, 1.0, s.K) + kTwoKGroupsStep[form] * (double)(s.K / (2 * kBlockK));
  else if (mid >= 128)
    tiled = tile_ns(kEightWavesCost, 1.0, s.K);
  else
    tiled = tile_ns(kSmallTilesCost, t64 > kCUs ? t64 / (double)kCUs : 1.0, s.K);
  thin_config(&s, 1, thin);
  return thin * thin_from_memory(s) < tiled;
}

// 256 x 256 tiles (8 waves of 128 x 64, see large_tiles) where they take less
// time than 128 x 128 tiles (see takes_large); else 128 x 128 tiles (4 waves
// of 64 x 64, two workgroups per CU) when there are more than one per CU;
// else, for skinny problems such as a decode step, whose time goes into
// streaming the weights: thin tiles (is_thin), 64 x 64 tiles with two K groups
// when those fit (k_groups), 128 x 128 tiles of 8 waves of 32 x 64 with a
// four-stage ring (one workgroup per CU) when there are 128 to 256 of them
// (1024 x 4096 x 4096, 256 tiles: 22.2 us, with 4 waves 24.6), and 64 x 64
// tiles (4 waves of 32 x 32) below that.
inline GemmRoute gemm_route(int form, const GemmSize& s) {
  const int64_t mid = tile_count(s, 128, 128);
  if (takes_large(form, tile_count(s, 256, 256), mid, s.M * s.N, s.K)) return kLargeTiles;
  if (mid > kCUs) return kMidTiles;
  if (is_thin(form, s)) return kThinTiles;
  if (k_groups(s)) return kTwoKGroups;
  return mid >= 128 ? kEightWaves : kSmallTiles;
}

// Quantized output needs whole 128-column units in a tile and must repeat the
// plain call's sums: 256 or 128 tiles; thin tiles of 32 x 128 where the plain
// call takes thin tiles (64 x 4096 x 4096, 32 tiles of 128 x 128: 24.8 us,
// thin 10.9); and where it takes two K groups, eight-wave 128 x 128 tiles that
// keep both groups' sums (64 x 4096 x 12288 20.4 us, with one sum 20.5; 250 x
// 512 x 4096 7.2, with one 7.0).
inline GemmRoute gemm_quantized_route(const GemmSize& s) {
  const GemmRoute r = gemm_route(kFormQuantized, s);
  return r == kSmallTiles ? kEightWaves : r;
}

// Split-K over `splits` workgroups per 128 x 128 tile, or thin tiles where
// they take less time.  A split's time in ns, fitted to 3000 random sizes (11%
// from them): its share of the K steps, and about 8 us and 0.8 per part for
// the partial tiles' way through memory; the thin tiles' waves meet in LDS.
// 256 x 12288 x 4096: split over four 24.9 us, thin 64 x 64 tiles 21.9; 64 x
// 25600 x 5120: split over four 42.0, thin 49.6.  More than 32 rows, whose
// thin tiles read the weights more than once or in 64-column strips, lose more
// against weights from memory than fewer do (33 x 25600 x 5120: split 39.4,
// thin 47.0; 64 x 17408 x 5120: 32.4 and 35.6).  The choice is 0.4% above the
// better on average (2.8% with a rule on bytes per CU alone).
inline GemmRoute gemm_splitk_route(int form, const GemmSize& s, int splits) {
  if (splits <= 1) return gemm_route(form, s);
  double thin;
  thin_config(&s, 1, thin);
  thin *= thin_from_memory(s) > 1.0 && s.M > 32 ? 1.4 : thin_from_memory(s);
  return thin < 7850 + 530.0 * (s.K / kBlockK) / splits + 811.0 * splits ? kThinTiles : kSplitK;
}

// 1x128 quantization, plain layout: two rows a thread instead of eight.  Up
// to kFewTiles tiles of 32 x 512, where the few waves of the other kernel and
// its long encode between loads and stores show (16384 x 4096, the largest
// measured, 37.4 -> 35.7 us); of many short rows a wave covers two instead of
// eight, and past these lines that is slower (131072 x 128 20.8 us with eight
// rows, 23.7 with two; 40000 x 128 8.65 and 9.26; 8192 x 128 3.80 and 3.51;
// 131072 x 512 33.4 and 34.3; 40000 x 512 12.1 and 11.8).
constexpr int kQuantRows = 32, kQuantCols = 512;  // a tile of the eight-row kernel
constexpr int64_t kFewTiles = 4096;
inline bool takes_few_rows(int64_t rows, int64_t cols) {
  const int64_t tiles = ((cols + kQuantCols - 1) / kQuantCols) * ((rows + kQuantRows - 1) / kQuantRows);
  return tiles <= kFewTiles && rows <= (cols < kQuantCols ? 8192 : 65536);
}

}  // namespace fp8q
