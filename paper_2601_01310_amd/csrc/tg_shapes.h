// How a grouped GEMM launch is cut into tiles: the census of the slots' rows
// and the choice of a tile shape, made by the dispatch for the GEMMs of the
// same call, or by a GEMM itself where there was none.
#pragma once

#include "tg_device.h"
#include "tg_launch.h"

namespace tg {

// Sum (or maximum) over the wave, uniform: row shifts and row broadcasts
// leave it in lane 63.
template <bool MAX>
__device__ __forceinline__ int wave_reduce(int v) {
#define TG_DPP_RED(ctrl, rows)                                              \
  do {                                                                      \
    const int o = __builtin_amdgcn_update_dpp(0, v, ctrl, rows, 0xF, false); \
    v = MAX ? max(v, o) : v + o;                                            \
  } while (0)
  TG_DPP_RED(0x111, 0xF);  // row_shr 1, 2, 4, 8
  TG_DPP_RED(0x112, 0xF);
  TG_DPP_RED(0x114, 0xF);
  TG_DPP_RED(0x118, 0xF);
  TG_DPP_RED(0x142, 0xA);  // row_bcast 15 into rows 1 and 3
  TG_DPP_RED(0x143, 0xC);  // row_bcast 31 into rows 2 and 3
#undef TG_DPP_RED
  return __builtin_amdgcn_readlane(v, kWave - 1);
}

// Row blocks of one launch at each tile height, its slots with rows, and its
// largest slot.
struct Census {
  int b32, b64, b128, b256, slots, max_rows;
};
// count(s): rows of slot s.
template <typename Count>
__device__ __forceinline__ Census census(int S, Count count) {
  const int lane = lane_id();
  int b32 = 0, b64 = 0, b128 = 0, b256 = 0, slots = 0, mx = 0;
  for (int base = 0; base < S; base += kWave) {
    const int s = base + lane;
    const int cnt = s < S ? count(s) : 0;
    b32 += (cnt + 31) / 32;
    b64 += (cnt + 63) / 64;
    b128 += (cnt + 127) / 128;
    b256 += (cnt + 255) / 256;
    slots += cnt > 0;
    mx = max(mx, cnt);
  }
  return {wave_reduce<false>(b32), wave_reduce<false>(b64), wave_reduce<false>(b128),
          wave_reduce<false>(b256), wave_reduce<false>(slots), wave_reduce<true>(mx)};
}

// Which tiles a launch runs as, in TG_TILES_AUTO: the base shapes (256-row
// walk; 32 x 256 or 32 x 128 tiles), or one of the middle shapes, which
// split a launch with too few base tiles for the chip, or too few rows for
// 256-row tiles, more finely.
enum Shape { k32x64, k32x32, k64x128, k64x64, k128x128, k128x64, k128x256, k32, k256 };

// log2 BM - 5 and log2 BN - 5 (BN: weight rows) of the shapes before k256.
__device__ __forceinline__ int shape_bm(int s) { return (0x02221100 >> (4 * s)) & 3; }
template <bool SWIGLU>
__device__ __forceinline__ int shape_bn(int s) {
  return ((SWIGLU ? 0x33121201 : 0x23121201) >> (4 * s)) & 3;
}

// Estimated time of a launch: sqrt(rounds^2 + loads^2 + weights^2) + 3 us.
//   rounds   ceil(tiles / blocks) x (K stages x the shape's stage time + 2.2 us)
//   loads    bytes staged by all tiles at 39 TB/s (L2 -> LDS over the chip)
//   weights  the touched slots' weights at 6.5 TB/s
// The stage times are one fit of all shapes over 66 repeated launches (one to
// 32 slots of 1 to 1024 rows; both Mixtral and DeepSeek-V3 experts and five
// smaller ones; 10 % rms). A middle shape is taken when its estimate is under
// 0.92 of the base shape's: over those launches the choice is 1.5 % slower than
// the best shape of each and 1.23 times as fast as the base shapes. Over 144
// calls of both projections it is 1.47 times as fast as they are with weights
// from HBM and 1.32 repeated, and 2 % slower at worst: where it keeps a base
// shape for a short launch, and for 700 rows of a Mixtral expert (128 x 128).
//
// Lane s estimates shape s: these instructions are fetched cold, so they are
// few. In a GEMM's own start census and choice cost about 1 us; the forward
// and the replay have them made by the dispatch, in waves that have nothing
// else to do.
template <bool SWIGLU, bool TAIL>
__device__ __forceinline__ Shape choose_shape(const Census& cs, int G, int K, int cols) {
  constexpr int H = SWIGLU ? 1 : 0;  // log2 of the weight rows per output column
  constexpr float kRound = 2.2f, kLoad = 128.0f / 3.9e7f;
  const float nk = (float)(K / 64), g = (float)G, inv_g = __builtin_amdgcn_rcpf(g);
  const int s = lane_id() & 7;
  const int bm = shape_bm(s), bn = shape_bn<SWIGLU>(s);
  // Stage times in ns.
  const uint64_t t03 = 0x00e6017c008000aeull;
  const uint64_t t47 = (uint64_t)(SWIGLU ? 575 : 315) << 48 | 0x0000035c013b01f9ull;
  const int ns = (int)((s < 4 ? t03 : t47) >> (16 * (s & 3))) & 0xffff;
  const int blocks = bm == 0 ? cs.b32 : bm == 1 ? cs.b64 : cs.b128;
  const int cl = 5 + bn - H;  // log2 of the output columns per tile
  // Squared estimate without the weights.
  auto squared = [&](float n, float rounds, float stage_us, float rows) {
    const float r = rounds * (nk * stage_us + kRound), l = n * nk * rows * kLoad;
    return r * r + l * l;
  };
  const float n = (float)(blocks * ((cols + (1 << cl) - 1) >> cl));
  float least =
      squared(n, ceilf(n * inv_g), (float)ns * 1e-3f, (float)((32 << bm) + (32 << bn)));
  // Base shape. Gate/up: rounds of tiles over the grid at each height; a
  // 32-row round costs about two thirds of a 256-row round (it streams the
  // same weight panel with an eighth of the MFMA work). Down (32 x 128 tiles,
  // two per 256-column panel): 32-row tiles when no slot exceeds 32 rows, or
  // when they fit in one round.
  const int NT = (cols + (256 >> H) - 1) >> (8 - H);
  const float n256 = (float)(cs.b256 * NT), n32 = (float)(cs.b32 * NT);
  const float rf = ceilf(n256 * inv_g);
  const bool small = TAIL ? (cs.max_rows <= 32 || 2.0f * n32 <= g)
                          : 2.0f * ceilf(n32 * inv_g) < 3.0f * rf;
  float base;
  if (small) {
    base = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(least), 7));
  } else {
    // Tiles of at most 128 rows cost about 0.7 of a full one; the spilled
    // last round of the down projection runs as 128 x 128 pieces, two or
    // four per tile.
    const float full =
        (float)(cs.b128 - cs.b256) * __builtin_amdgcn_rcpf((float)max(cs.b256, 1));
    const float stage = 1.37f * (0.7f + 0.3f * full);
    base = squared(n256, rf, stage, 512.0f);
    if (TAIL) {
      const float rem = n256 - floorf(n256 * inv_g) * g;
      if (rem > 0.0f && 2.0f * rem <= g) {
        const float pieces = ceilf(2.0f * rem * (1.0f + full) * inv_g);
        const float r = (rf - 1.0f) * (nk * stage + kRound) + pieces * (nk * 0.58f + kRound);
        const float l = n256 * nk * 512.0f * kLoad;
        base = r * r + l * l;
      }
    }
  }
  // The best of lanes 0 .. 6, in every row of 16 lanes (lane 7's is the base).
  int best = s;
  if (s == 7) least = 3.4e38f;
#define TG_DPP_LEAST(ctrl)                                                                      \
  do {                                                                                          \
    const float ol = __int_as_float(                                                            \
        __builtin_amdgcn_update_dpp(0, __float_as_int(least), ctrl, 0xF, 0xF, false));          \
    const int ob = __builtin_amdgcn_update_dpp(0, best, ctrl, 0xF, 0xF, false);                 \
    const bool less = ol < least || (ol == least && ob < best);                                 \
    least = less ? ol : least;                                                                  \
    best = less ? ob : best;                                                                    \
  } while (0)
  TG_DPP_LEAST(0xB1);   // xor 1
  TG_DPP_LEAST(0x4E);   // xor 2
  TG_DPP_LEAST(0x141);  // half-row mirror
#undef TG_DPP_LEAST
  const float wt = (float)cs.slots * ((float)K * (float)cols * (float)(2 << H) / 6.5e6f);
  const bool take = __builtin_amdgcn_sqrtf(least + wt * wt) + 3.0f <
                    0.92f * (__builtin_amdgcn_sqrtf(base + wt * wt) + 3.0f);
  return (Shape)__builtin_amdgcn_readfirstlane(take ? best : small ? (int)k32 : (int)k256);
}

}  // namespace tg
