// Which kernel a GEMM takes: rules on sizes alone, on the host.
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
// 12.4; at K = 4096 1x128 x 1x128 455 and 400 the other way).  Within 2% the
// side that holds on more of the sizes: large from 512 tiles on and where they
// fill whole rounds.  1% of those sizes are more than 2.5% slower than with the
// rule "large from 512 tiles on, 1x128 x 1x128 never"; 15% were with estimates
// of K = 4096 for every K.
struct BlockNs {
  int large, mid;
};
constexpr BlockNs kBlockNs[6] = {{1614, 892},   // tensor
                                 {1614, 892},   // row
                                 {1814, 1031},  // 1x128 x 128x128
                                 {2204, 1152},  // 1x128 x 1x128
                                 {1708, 983},   // power-of-two scales
                                 {1944, 1072}}; // quantized output
constexpr int kFormQuantized = 5;  // after the GemmPair values

inline bool takes_large(int form, int64_t big, int64_t mid, int64_t outputs, int64_t K) {
  if (mid <= kCUs) return false;
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
  return large < tiled * (big >= 2 * kCUs || rest == 0 ? 1.02 : 0.98);
}

// Two K groups per 64 x 64 tile (one workgroup of 8 waves per CU) when there
// are at most 256 such tiles, so that a CU would hold one workgroup anyway,
// and the K blocks split evenly; more tiles keep two 4-wave workgroups per
// CU (their combined 4-stage rings already keep the loads in flight;
// measured faster there).
inline bool k_groups(const GemmSize& s) { return tile_count(s, 64, 64) <= kCUs && (s.K / kBlockK) % 2 == 0; }

// Operand rows (of K bytes) that the busiest CU loads: its tiles times a
// tile's rows of A (none past M) and of B.
inline int64_t cu_rows(int64_t tiles, int64_t rows) { return (tiles + kCUs - 1) / kCUs * rows; }

// The thin tile whose busiest CU loads the fewest rows, for the problems of
// one launch (one K).  64 x 64, whose partial tiles take longest to meet,
// from eight K blocks a wave on (256 x 12288 x 4096: 21.8 us against 23.5
// with two K groups; 64 x 4096 x 12288: 12.6 against 10.9).
inline int thin_config(const GemmSize* probs, int count, int64_t& rows) {
  int best = 0;
  for (int c = 0; c < kThinConfigs; ++c) {
    if (c == kThin64x64 && probs[0].K < 8 * 8 * kBlockK) continue;
    int64_t tiles = 0, most = 0;
    for (int i = 0; i < count; ++i) {
      tiles += tile_count(probs[i], kThinM[c], kThinN[c]);
      const int64_t per = (probs[i].M < kThinM[c] ? probs[i].M : kThinM[c]) + kThinN[c];
      most = per > most ? per : most;
    }
    const int64_t r = cu_rows(tiles, most);
    if (c == 0 || r < rows) {
      best = c;
      rows = r;
    }
  }
  return best;
}

// Whether a problem too small for the 128 x 128 tiles of four waves is thin:
// the tile kernels load fewer rows per CU only where they have tiles for most
// of the CUs, and take longer per row: 1.13 times for 64 x 64 with two K
// groups, 1.2 for 64 x 64 without (two workgroups per CU, which even out),
// 1.33 for 128 x 128 with eight waves (measured: 75, 70 and 64 KB a
// microsecond and CU against 85).  64 x 4096 x 12288 (192 tiles of 64 x 64)
// stays: 10.9 us, thin 32 x 32 13.2; 128 x 4096 x 12288 (384 of 64 x 64):
// 15.1, thin 19.2; 256 x 4096 x 12288 (192 of 128 x 128): 19.4, thin 26.9; 64
// x 12288 x 4096 (64 tiles) 22.2 and 11.9.
inline bool is_thin(const GemmSize& s) {
  const int64_t t64 = tile_count(s, 64, 64), mid = tile_count(s, 128, 128);
  const int64_t rows64 = (s.M < 64 ? s.M : 64) + 64;
  int64_t tiled;  // in percent
  if (k_groups(s))
    tiled = cu_rows(t64, rows64) * 113;
  else if (mid >= 128)
    tiled = cu_rows(mid, (s.M < 128 ? s.M : 128) + 128) * 133;
  else
    tiled = t64 > kCUs ? t64 * rows64 * 120 / kCUs : rows64 * 120;
  int64_t rows;
  thin_config(&s, 1, rows);
  return rows * 100 < tiled;
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
  if (is_thin(s)) return kThinTiles;
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
// they take less time: a split loads 256 K / S bytes per CU and then pays
// about 10 us (900 KB of loads) for the partial tiles' way through memory; the
// thin tiles' waves meet in LDS.  256 x 12288 x 4096: split over four 24.9 us,
// thin 64 x 64 tiles 21.9; 256 x 25600 x 5120 stays split.
inline GemmRoute gemm_splitk_route(int form, const GemmSize& s, int splits) {
  if (splits <= 1) return gemm_route(form, s);
  int64_t rows;
  thin_config(&s, 1, rows);
  return rows * s.K < 256 * s.K / splits + 900000 ? kThinTiles : kSplitK;
}

}  // namespace fp8q
