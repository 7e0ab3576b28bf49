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
  int full, parts, grid, cost;
};
inline LargePlan large_plan(int64_t total) {
  const int rest = (int)(total % kCUs), rounds = (int)(total / kCUs);
  LargePlan p;
  p.parts = rest == 0 || rest > kCUs / 2 ? 1 : (rest <= kCUs / 4 ? 4 : 2);
  p.full = p.parts == 1 ? (int)total : rounds * kCUs;
  p.grid = p.full + (p.parts == 1 ? 0 : rest * p.parts);
  p.cost = 100 * rounds + (rest == 0 ? 0 : p.parts == 4 ? 40 : p.parts == 2 ? 62 : 90);
  return p;
}

// Whether `big` 256 x 256 tiles run before `mid` 128 x 128 tiles (the same
// outputs) would: both in percent of a whole 256 x 256 tile's time.  512 of
// the 128 x 128 tiles (four waves, two workgroups per CU) take 59, up to 256
// (one per CU) 37; a last round of whole 256 x 256 tiles on part of the chip
// 90 (measured at K = 4096: 192 tiles 47 us, 256 tiles 56 us, 512 of 128 x
// 128 33 us, 256 of them 20.6 us).
inline bool takes_large(int64_t big, int64_t mid) {
  if (big > 0x3fffffff / 100) return true;
  const int64_t rest = mid % (2 * kCUs);
  const int64_t cost_mid = 59 * (mid / (2 * kCUs)) + (rest == 0 ? 0 : rest <= kCUs ? 37 : 59);
  return large_plan(big).cost < cost_mid;
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
inline GemmRoute gemm_route(const GemmSize& s) {
  const int64_t mid = tile_count(s, 128, 128);
  if (takes_large(tile_count(s, 256, 256), mid)) return kLargeTiles;
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
  const GemmRoute r = gemm_route(s);
  return r == kSmallTiles ? kEightWaves : r;
}

// Split-K over `splits` workgroups per 128 x 128 tile, or thin tiles where
// they take less time: a split loads 256 K / S bytes per CU and then pays
// about 10 us (900 KB of loads) for the partial tiles' way through memory; the
// thin tiles' waves meet in LDS.  256 x 12288 x 4096: split over four 24.9 us,
// thin 64 x 64 tiles 21.9; 256 x 25600 x 5120 stays split.
inline GemmRoute gemm_splitk_route(const GemmSize& s, int splits) {
  if (splits <= 1) return gemm_route(s);
  int64_t rows;
  thin_config(&s, 1, rows);
  return rows * s.K < 256 * s.K / splits + 900000 ? kThinTiles : kSplitK;
}

}  // namespace fp8q
