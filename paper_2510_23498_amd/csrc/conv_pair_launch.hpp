// Launchers of conv_pair.hpp, one per number of channel blocks and precision, each in a translation unit of its own.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>

#include "conv_pair.hpp"

namespace rampde {

// (blocks of 16 pixels per wavefront in the first and the second convolution) that the kernel is built for
constexpr int kPairTiles[][2] = {{1, 1}, {2, 1}, {2, 2}, {3, 2}, {4, 4}, {5, 4}, {7, 7}, {9, 8}};

// Tiles of `lines` image lines, or none (tiles = 0): more pixels than a workgroup multiplies, or more lines than LDS holds
inline ConvPairShape conv_pair_tiles(int C32, int lines, int H, int Wd, int64_t images) {
  ConvPairShape t{};
  t.lines = lines;
  t.per_image = (H + lines - 1) / lines;
  t.magic = (65536 + Wd - 1) / Wd;
  const int hidden = t.per_image == 1 ? H : std::min(H, lines + (t.per_image == 2 ? 1 : 2));
  const int want1 = (hidden * Wd + 63) / 64, want2 = (std::min(lines, H) * Wd + 63) / 64;
  for (auto& m : kPairTiles)
    if (!t.mt1 && m[0] >= want1 && m[1] >= want2) {
      t.mt1 = m[0];
      t.mt2 = m[1];
    }
  if (t.mt1 && conv_pair_lds_bytes(C32, lines, Wd) <= (t.mt1 <= 5 ? 78 : 156) * 1024) t.tiles = (int)(images * t.per_image);
  return t;
}
// The tiles of least estimated time, from launches of every possible height on nine shapes (us per evaluation with the
// next stage's input; 64 channels unless noted): a launch takes about 8 us (6 with 32 channels), a tile 1.1 (0.5) per
// block of 16 pixels and wavefront, a little less where two workgroups share a compute unit (up to 5 blocks; the larger
// tiles have it alone), which also waits less for memory.  128 x 32 x 32 with 4 / 8 / 16 lines 39.1 / 29.7 / 35.2;
// 128 x 16 x 16 with 2 / 4 / 8 / 16 25.5 / 17.4 / 15.1 / 18.2; 60 x 14 x 14 with 1 / 2 / 4 / 7 / 14 23.3 / 15.6 / 12.6 /
// 13.2 / 17.3; 16 x 64 x 64 with 1 / 2 / 4 / 7 38.4 / 26.7 / 27.0 / 31.4; 32 channels, 20 x 28 x 28 with 1 / 2 / 4 / 7 / 14
// 8.2 / 7.6 / 7.9 / 9.5 / 12.7, 128 x 32 x 32 with 2 / 4 / 8 / 16 24.2 / 17.3 / 16.8 / 18.8.
inline ConvPairShape conv_pair_shape(int C32, int H, int Wd, int64_t images, int cus) {
  ConvPairShape best{};
  double least = 0;
  for (int lines = 1; lines <= std::min(H, 576 / Wd); ++lines) {
    const ConvPairShape t = conv_pair_tiles(C32, lines, H, Wd, images);
    if (!t.tiles) continue;
    const double rounds = (double)((t.tiles + cus - 1) / cus), block = (C32 == 1 ? 0.5 : 1.1) * (t.mt1 + t.mt2);
    const double cost = t.mt1 > 5 ? rounds * ((C32 == 1 ? 6 : 8) + 1.2 * block)
                                  : (C32 == 1 ? 6 : 8) + rounds * ((rounds > 1 ? 0.85 : 1.0) * block + 1.2);
    if (!best.tiles || cost < least) {
      best = t;
      least = cost;
    }
  }
  return best;
}

#define RAMPDE_DECLARE_CONV_PAIR(c32)                                                                                          \
  hipError_t conv_pair_launch_##c32##_f16(const ConvPair& g, const ConvPairShape& sh, bool vjp, hipStream_t st);               \
  hipError_t conv_pair_launch_##c32##_bf16(const ConvPair& g, const ConvPairShape& sh, bool vjp, hipStream_t st);
RAMPDE_DECLARE_CONV_PAIR(1)
RAMPDE_DECLARE_CONV_PAIR(2)
#undef RAMPDE_DECLARE_CONV_PAIR

inline hipError_t conv_pair_launch(int C32, bool bf16, const ConvPair& g, const ConvPairShape& sh, bool vjp, hipStream_t st) {
  if (C32 == 1) return bf16 ? conv_pair_launch_1_bf16(g, sh, vjp, st) : conv_pair_launch_1_f16(g, sh, vjp, st);
  return bf16 ? conv_pair_launch_2_bf16(g, sh, vjp, st) : conv_pair_launch_2_f16(g, sh, vjp, st);
}

}  // namespace rampde
