// Launchers of conv_pair.hpp and conv_pass.hpp, one per number of channel blocks and precision, each in a translation unit of its own.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>

#include "conv_pass.hpp"

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
// The tiles of least estimated time, fitted to launches of every possible height on nine shapes, of which it picks the best
// or one within 3 %: a fixed part, a part per block of 16 pixels and wavefront, a little less of it where two workgroups
// share a compute unit (up to 5 blocks; the larger tiles have it alone), which also wait less for memory.  us per
// evaluation with the next stage's input, 64 channels: 128 x 32 x 32 with 4 / 8 / 16 lines 30.9 / 25.6 / 29.1; 128 x 16 x 16
// with 2 / 4 / 8 / 16 22.3 / 13.2 / 10.6 / 13.0; 60 x 14 x 14 with 2 / 4 / 7 / 14 11.7 / 8.4 / 9.1 / 12.1; 16 x 64 x 64 with 1 /
// 2 / 4 / 7 31.5 / 22.3 / 22.4 / 24.8; 32 channels, 20 x 28 x 28 with 1 / 2 / 4 / 7 / 14 7.0 / 5.7 / 5.3 / 6.7 / 9.8, 128 x 32 x 32
// with 2 / 4 / 8 / 16 20.0 / 14.4 / 13.0 / 15.7.
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

constexpr int kPassTiles = 4;  // blocks of 16 pixels per wavefront, at most
// Tiles for the launches of conv_pass.hpp: all workgroups of a launch run at once, two on a compute unit.
inline PassShape conv_pass_tiles(int C32, int lines, int H, int Wd, int64_t images, int cus) {
  PassShape t{};
  t.mt = (std::min(lines, H) * Wd + 63) / 64;
  t.lines = lines;
  t.per_image = (H + lines - 1) / lines;
  t.magic = (65536 + Wd - 1) / Wd;
  if (t.mt > kPassTiles || t.per_image > 2 * cus || pass_lds_bytes(C32, lines, Wd) > 79 * 1024) return PassShape{};
  const int64_t most = 2 * cus / t.per_image, rounds = (images + most - 1) / most;
  t.slots = (int)((images + rounds - 1) / rounds);
  return t;
}
// The least estimated time of an evaluation, from (us, forward / recomputation; workgroups):
// 64 channels, 128 x 32 x 32, tiles of 4 lines (2 rounds of 512) 36.9 / 36.8, of 6 (2 of 384) 40.4 / 35.5, of 8 (512)
// 30.6 / 23.3; 64 x 16 x 16, 4 lines (256) 9.6 / 9.9, 8 (128) 10.5 / 10.6, 16 (64) 14.8 / 11.9; 32 channels, 20 x 28 x 28,
// 2 lines (280) 6.8 / 8.3, 4 (140) 6.2 / 7.3, 7 (80) 7.5 / 8.5; 128 x 32 x 32, 4 lines (2 of 512) 15.6 / 15.5, 8 (512) 10.2 / 11.1.
inline double conv_pass_cost(const PassShape& t, int C32, int64_t images, int cus) {
  const double rounds = (double)((images + t.slots - 1) / t.slots), shared = t.slots * t.per_image > cus ? (C32 == 1 ? 1.35 : 1.75) : 1.0;
  return rounds * shared * (C32 == 1 ? 5.3 + 0.6 * t.mt : 8.2 + 1.4 * t.mt);
}
inline PassShape conv_pass_shape(int C32, int H, int Wd, int64_t images, int cus) {
  PassShape best{};
  for (int lines = 1; lines <= std::min(H, 64 * kPassTiles / Wd); ++lines) {
    const PassShape t = conv_pass_tiles(C32, lines, H, Wd, images, cus);
    if (t.lines && (!best.lines || conv_pass_cost(t, C32, images, cus) < conv_pass_cost(best, C32, images, cus))) best = t;
  }
  return best;
}

enum ConvPassKind { kPassForward, kPassRecompute, kPassChain };
struct ConvLaunch {
  bool vjp;             // conv_pair
  ConvPassKind kind;    // conv_pass
  bool backward;        // conv_redo
  unsigned grid;
  hipStream_t st;
};

#define RAMPDE_DECLARE_CONV(c32, low)                                                                        \
  hipError_t conv_pair_launch_##c32##_##low(const ConvPair& g, const ConvPairShape& sh, const ConvLaunch& l); \
  hipError_t conv_pass_launch_##c32##_##low(const ConvPass& g, const PassShape& sh, const ConvLaunch& l);     \
  hipError_t conv_redo_launch_##c32##_##low(const ConvRedo& g, const ConvLaunch& l);
RAMPDE_DECLARE_CONV(1, f16)
RAMPDE_DECLARE_CONV(1, bf16)
RAMPDE_DECLARE_CONV(2, f16)
RAMPDE_DECLARE_CONV(2, bf16)
#undef RAMPDE_DECLARE_CONV

inline hipError_t conv_pair_launch(int C32, bool bf16, const ConvPair& g, const ConvPairShape& sh, bool vjp, hipStream_t st) {
  const ConvLaunch l{vjp, kPassForward, false, (unsigned)sh.tiles, st};
  if (C32 == 1) return bf16 ? conv_pair_launch_1_bf16(g, sh, l) : conv_pair_launch_1_f16(g, sh, l);
  return bf16 ? conv_pair_launch_2_bf16(g, sh, l) : conv_pair_launch_2_f16(g, sh, l);
}
inline hipError_t conv_pass_launch(int C32, bool bf16, const ConvPass& g, const PassShape& sh, ConvPassKind kind, hipStream_t st) {
  const ConvLaunch l{false, kind, false, (unsigned)(sh.slots * sh.per_image), st};
  if (C32 == 1) return bf16 ? conv_pass_launch_1_bf16(g, sh, l) : conv_pass_launch_1_f16(g, sh, l);
  return bf16 ? conv_pass_launch_2_bf16(g, sh, l) : conv_pass_launch_2_f16(g, sh, l);
}
inline hipError_t conv_redo_launch(int C32, bool bf16, const ConvRedo& g, bool backward, unsigned grid, hipStream_t st) {
  const ConvLaunch l{false, kPassForward, backward, grid, st};
  if (C32 == 1) return bf16 ? conv_redo_launch_1_bf16(g, l) : conv_redo_launch_1_f16(g, l);
  return bf16 ? conv_redo_launch_2_bf16(g, l) : conv_redo_launch_2_f16(g, l);
}

}  // namespace rampde
