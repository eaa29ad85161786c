// 3x3 zero-padded convolution (and its transpose: the same kernel with the flipped, transposed
// weights) on channels-last rows, for at most 64 channels: the velocity evaluations, their
// recomputation and the input-cotangent products of the convolutional velocity (paper Alg. 1, the
// low-precision evaluation of Phi; eq. (vjp)) as one persistent kernel per call.
//
// A workgroup keeps the whole weight tensor of the layer (9 taps x channels x channels, low precision) in LDS for as long
// as it lives and walks over tiles of PR whole image lines of one image, at most 256 pixels.  Per tile the input lines
// with a halo of one line above and below and one zero column left and right are staged in LDS once; every tap is then
// the same tile read at a shifted pixel address, and a wavefront computes 32 pixels x 32 output channels per block with
// v_mfma_f32_32x32x16 (weights as the first operand, so a lane ends with 4 consecutive output channels of a pixel:
// 8-byte stores and loads in the epilogue).  The next tile's input is fetched into registers while the current one is
// being multiplied.  Epilogue as in gemm_nt: bias, time-channel term (tabulated by border class), tanh or the tanh'
// factor from the stored activation, rounding, overflow detector.
//
// Any image height, any width up to 64 (padded channels: 64): the pixel of a lane and the staged chunks of a thread are the
// same in every tile, so the divisions by the width are done once per launch.  NA output blocks of 32 channels and KC
// blocks of 16 input channels are multiplied; networks of at most 32 channels take 1 and 2 (a quarter of the padded
// work; columns past 32 are not written, nothing reads them across columns), others 2 and 4.  AW = 2: the two
// output blocks go to two wavefronts, for tiles of at most 128 pixels.
#pragma once
#include "fused.hpp"
#include "gemm.hpp"

namespace rampde {

constexpr int CT_TILE = 256;      // pixels per tile, at most

struct ConvTileShape {
  int lines, per_image, tiles;    // image lines of a tile, tiles of an image, tiles in all
  int blocks, aw;
};
constexpr int conv_tile_pitch(int KC) { return 16 * KC + 8; }  // elements per LDS row of one pixel's (one output's) channels
inline size_t conv_tile_lds_bytes(int NA, int KC, int lines, int Wd) {
  return (size_t)(9 * 32 * NA + (lines + 2) * (Wd + 2)) * conv_tile_pitch(KC) * 2 + (16 + 10) * 32 * NA * 4;
}
inline bool conv_tile_applies(int Cpad, int N, int Wd) { return Cpad == 64 && N == 64 && Wd >= 1 && Wd <= 64; }
// Tiles of as few lines as the number of rounds over the compute units that the largest tile needs allows: 20 images of
// 28 x 28 in 200 tiles of 3 lines (one round) and not in 80 of 7.
inline ConvTileShape conv_tile_shape(int NA, int KC, int H, int Wd, int64_t images, int cus) {
  int most = std::min(H, CT_TILE / Wd);
  while (most > 1 && conv_tile_lds_bytes(NA, KC, most, Wd) > 156 * 1024) --most;
  auto rounds = [&](int lines) { return (images * ((H + lines - 1) / lines) + cus - 1) / cus; };
  int lines = 1;
  while (lines < most && (rounds(lines) > rounds(most) || (lines * Wd < 32 && lines < most))) ++lines;
  ConvTileShape t;
  t.lines = lines;
  t.per_image = (H + lines - 1) / lines;
  t.tiles = (int)(images * t.per_image);
  t.blocks = std::min(t.tiles, cus);
  t.aw = NA == 2 && lines * Wd <= CT_TILE / 2 ? 2 : 1;
  return t;
}

// What a tile reads and writes goes through buffer descriptors of its own image lines: a lane without a pixel reads zeros
// and stores nowhere, and every lane issues the same number of loads and stores.  Loads and stores share a counter, so
// only then can the compiler wait for the next tile's input without waiting for this tile's stores.
//
// The loads are not in flight beside the matrix instructions: the activations of the tanh' factor have arrived before the
// multiplication, the next tile's input is requested behind it and arrives during the epilogue.  Some cards run the two
// together slower than one after the other.  64 channels, 32 x 32, 128 images, 16 RK4 steps, ms per training pass on four
// cards (equal in a plain copy and a plain matrix product) with the kernel for powers of two that this one replaced /
// all loads in flight beside the multiplication / as here: 13.1 / 12.4 / 12.3, 13.6 / 13.9 / 13.0, 13.7 / 14.1 / 13.2,
// 14.2 / 14.8 / 13.7.
constexpr int kOutside = 0x40000000;  // (a byte offset past every window)
template <class E>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t window(const E* p, int elements) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<E*>(p), 0, elements * (int)sizeof(E), 0x00020000);
}

// 8 wavefronts: pixel block (wave / AW), output blocks (wave % AW) * NB ...
// nothing, tanh, tanh' of the stored activation, nothing and the next stage input, nothing and the next slope cotangent.
// The last two read 2 or 4 bytes and write 2 per element that a pass of their own would have read and written again
// (us per training pass without / with: 24 x 28 x 28, 20 images, 8 Heun steps 1064 / 955; 64 x 32 x 32, 128 images, 16
// RK4 steps, as shares of the same pass before on the same card: 0.961 / 0.943)
enum ConvEpilogue { kConvPlain, kConvTanh, kConvFactor, kConvStage, kConvCotangent };
template <class T, int NA, int KC, int AW, int EPI>
__global__ __launch_bounds__(512) void conv3x3_tile(GemmNT g, ConvTileShape sh) {
  constexpr int NT = 512;
  constexpr int NB = NA / AW;                        // output blocks of a wavefront
  constexpr int NCH = 32 * NA;                       // output channels
  constexpr int C8 = 2 * KC;                         // 16-byte chunks of a pixel
  constexpr int PITCH = conv_tile_pitch(KC);
  constexpr int MAXC = (CT_TILE + 2 * 64) * C8 / NT; // input chunks of a thread and tile
  if (g.ctl && g.ctl->poison) return;
  extern __shared__ __attribute__((aligned(16))) uint16_t ct_smem[];
  const int W = g.Wd, H = g.H, PR = sh.lines;
  const int LW = W + 2;                              // staged pixels per line
  uint16_t* sW = ct_smem;                            // [9][NCH][PITCH]
  uint16_t* sIn = ct_smem + 9 * NCH * PITCH;         // [PR + 2][W + 2][PITCH]
  float* s_tt = reinterpret_cast<float*>(sIn + (PR + 2) * LW * PITCH);  // [16][NCH]: bias + time term by border class
  float* s_wt = s_tt + 16 * NCH;                                        // [9][NCH] time-channel weights, [NCH] bias
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // ---- input chunks of a tile: chunk id -> (staged line ly, pixel x, 8 channels c8), the same in every tile
  int c_ly[MAXC], c_src[MAXC], c_dst[MAXC];          // ly = 0 is the line above the tile; -1: no chunk; c_src in bytes
#pragma unroll
  for (int i = 0; i < MAXC; ++i) {
    const int id = tid + NT * i;
    const int c8 = id % C8, px = id / C8;
    const int ly = px / W, x = px - ly * W;
    c_ly[i] = px < (PR + 2) * W ? ly : -1;
    c_src[i] = (ly * W + x) * g.lda * 2 + c8 * 16;
    c_dst[i] = (ly * LW + x + 1) * PITCH + c8 * 8;
  }
  u16x8 reg[MAXC];
  auto load_tile = [&](int t) __attribute__((always_inline)) {
    const int img = t / sh.per_image, y0 = (t - img * sh.per_image) * PR;
    // lines first .. y0 + PR of the image, those of them that it has
    const int first = y0 > 0 ? y0 - 1 : 0, lines = min(y0 + PR + 1, H) - first;
    const auto src = window(g.A + ((size_t)img * H + first) * W * g.lda, lines * W * g.lda);
    const int skip = (first - (y0 - 1)) * W * g.lda * 2;
#pragma unroll
    for (int i = 0; i < MAXC; ++i) {
      const int y = y0 + c_ly[i] - 1;
      const int off = c_ly[i] >= 0 && y >= 0 && y < H ? c_src[i] - skip : kOutside;
      reg[i] = __builtin_bit_cast(u16x8, __builtin_amdgcn_raw_buffer_load_b128(src, off, 0, 0));
    }
  };
  auto store_tile = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < MAXC; ++i)
      if (c_ly[i] >= 0) *reinterpret_cast<u16x8*>(&sIn[c_dst[i]]) = reg[i];
  };

  // wait for the requested input: where no stores were issued behind the request
  auto settle = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < MAXC; ++i) asm volatile("" : "+v"(reg[i]));
  };

  // (the first tile's input is requested before the weights: both are in flight together)
  load_tile(blockIdx.x);  // (the grid has at most sh.tiles workgroups)

  // ---- once per workgroup: weights, zero halo columns, time-term table
  {
    // (all loads of a thread are issued before the first is stored: one memory latency, not one per chunk)
    constexpr int TOTAL = 9 * NCH * C8, NWC = (TOTAL + NT - 1) / NT;
    u16x8 wr[NWC];
#pragma unroll
    for (int i = 0; i < NWC; ++i) {
      const int id = tid + NT * i;
      const int c8 = id % C8, co = (id / C8) % NCH, tap = id / (C8 * NCH);
      if (TOTAL % NT == 0 || id < TOTAL) wr[i] = *reinterpret_cast<const u16x8*>(g.W + (size_t)co * g.ldw + tap * 64 + c8 * 8);
    }
#pragma unroll
    for (int i = 0; i < NWC; ++i) {
      const int id = tid + NT * i;
      const int c8 = id % C8, row = id / C8;
      if (TOTAL % NT == 0 || id < TOTAL) *reinterpret_cast<u16x8*>(&sW[row * PITCH + c8 * 8]) = wr[i];
    }
  }
  for (int id = tid; id < (PR + 2) * 2 * C8; id += NT) {
    const int c8 = id % C8, side = (id / C8) & 1, ly = id / (2 * C8);
    const u16x8 z = {0, 0, 0, 0, 0, 0, 0, 0};
    *reinterpret_cast<u16x8*>(&sIn[(ly * LW + (side ? W + 1 : 0)) * PITCH + c8 * 8]) = z;
  }
  // (one global load per thread, then the table from LDS: a chain of dependent global loads per
  // table entry would cost more than the tile's multiplication)
  for (int i = tid; i < 10 * NCH; i += NT) {
    const int t = i / NCH, n = i % NCH;
    float v = 0.f;
    if (t < 9) {
      if (g.wt) v = g.wt[t * g.N + n];
    } else if (g.bias) {
      v = g.bias[n];
    }
    s_wt[i] = v;
  }
  __syncthreads();
  for (int i = tid; i < 16 * NCH; i += NT) {
    const int combo = i / NCH, n = i % NCH;
    float sum = 0.f;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      const int dy = t / 3 - 1, dx = t % 3 - 1;
      const bool ok = (dy >= 0 || (combo & 8)) && (dy <= 0 || (combo & 4)) && (dx >= 0 || (combo & 2)) &&
                      (dx <= 0 || (combo & 1));
      sum += ok ? s_wt[t * NCH + n] * g.tau : 0.f;
    }
    s_tt[i] = s_wt[9 * NCH + n] + sum;
  }

  // this lane's pixel (operand B) and weight rows (operand A)
  const int fk = (lane >> 5) * 8;
  const int pb = wave / AW, a0 = (wave % AW) * NB;    // pixel block, first output block
  const int p = pb * 32 + (lane & 31);
  const bool on = p < PR * W;
  const int ly = on ? p / W : 0, x = on ? p - ly * W : 0;
  const int in_base = ((ly + 1) * LW + x + 1) * PITCH + fk;
  const int w_base = (a0 * 32 + (lane & 31)) * PITCH + fk;
  const int n0 = a0 * 32 + 4 * (lane >> 5);           // this lane's first output channel

  bool bad = false;
  const float S = EPI == kConvCotangent ? g.ctl->S : 0.f;
  settle();
  for (int t = blockIdx.x; t < sh.tiles; t += gridDim.x) {
    __syncthreads();  // the previous tile's fragments have been read (and the tables are written)
    store_tile();
    __syncthreads();
    const int img = t / sh.per_image, y0 = (t - img * sh.per_image) * PR, y = y0 + ly;
    const bool live = on && y < H;
    const size_t row0 = ((size_t)img * H + y0) * W;
    const int pixels = min(PR, H - y0) * W;  // of the tile; lanes past them read zeros and their stores go nowhere
    // the stored activations for the tanh' factor of this lane's outputs
    uint2 dv[NB][4];
    if constexpr (EPI == kConvFactor) {
      const auto act = window(g.dact + row0 * g.ldd, pixels * g.ldd);
#pragma unroll
      for (int a = 0; a < NB; ++a)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4)
          dv[a][q4] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(act, (p * g.ldd + n0 + a * 32 + 8 * q4) * 2, 0, 0));
    }
    // ... the stored state or the adjoint at them
    float4 av4[NB][4];
    if constexpr (EPI == kConvStage) {
      const auto base = window(g.base + row0 * g.d, pixels * g.d);
#pragma unroll
      for (int a = 0; a < NB; ++a)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const int n = n0 + a * 32 + 8 * q4;
          dv[a][q4] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(base, n < g.d ? (p * g.d + n) * 2 : kOutside, 0, 0));
        }
    }
    if constexpr (EPI == kConvCotangent) {
      const auto adj = window(g.adj + row0 * g.d, pixels * g.d);
#pragma unroll
      for (int a = 0; a < NB; ++a)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const int n = n0 + a * 32 + 8 * q4;
          av4[a][q4] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(adj, n < g.d ? (p * g.d + n) * 4 : kOutside, 0, 0));
        }
    }
    if (pb * 32 >= PR * W) {  // (uniform: no pixel block for this wavefront)
      if (t + (int)gridDim.x < sh.tiles) load_tile(t + gridDim.x);
      settle();
      continue;
    }

    f32x16 acc[NB];
#pragma unroll
    for (int a = 0; a < NB; ++a)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[a][q] = 0.f;
    // 9 KC k-blocks of 16 (9 taps x 16 KC channels); the fragments of block i + 1 are read from LDS
    // before the MFMAs of block i are issued (a workgroup is alone on its CU: nothing else hides
    // the LDS latency)
    auto load_frags = [&](int it, u16x8 (&fa)[NB], u16x8& fb) __attribute__((always_inline)) {
      const int tap = it / KC, kk = it % KC;
      const int shift = ((tap / 3 - 1) * LW + (tap % 3 - 1)) * PITCH;
#pragma unroll
      for (int a = 0; a < NB; ++a)
        fa[a] = *reinterpret_cast<const u16x8*>(&sW[(tap * NCH + a * 32) * PITCH + w_base + kk * 16]);
      fb = *reinterpret_cast<const u16x8*>(&sIn[in_base + shift + kk * 16]);
    };
    if constexpr (EPI == kConvFactor || EPI == kConvStage) {  // (wait for them)
#pragma unroll
      for (int a = 0; a < NB; ++a)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) asm volatile("" : "+v"(dv[a][q4].x), "+v"(dv[a][q4].y));
    }
    if constexpr (EPI == kConvCotangent) {
#pragma unroll
      for (int a = 0; a < NB; ++a)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) asm volatile("" : "+v"(av4[a][q4].x), "+v"(av4[a][q4].y), "+v"(av4[a][q4].z), "+v"(av4[a][q4].w));
    }
    u16x8 fa[2][NB], fb[2];
    load_frags(0, fa[0], fb[0]);
#pragma unroll
    for (int it = 0; it < 9 * KC; ++it) {
      if (it + 1 < 9 * KC) load_frags(it + 1, fa[(it + 1) & 1], fb[(it + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);  // (keep the reads of block i + 1 ahead of the MFMAs of block i)
#pragma unroll
      for (int a = 0; a < NB; ++a) acc[a] = Low<T>::mfma32(fa[it & 1][a], fb[it & 1], acc[a]);
      __builtin_amdgcn_sched_barrier(0);
    }

    if (t + (int)gridDim.x < sh.tiles) load_tile(t + gridDim.x);

    // ---- epilogue: accumulator row = output channel 8 (q / 4) + 4 (lane / 32) + q % 4 of block a,
    //      column = pixel lane % 32
    const auto out = window(g.C + row0 * g.ldc, pixels * g.ldc);
    __amdgpu_buffer_rsrc_t next;
    if constexpr (EPI >= kConvStage) next = window(g.next + row0 * g.ldc, pixels * g.ldc);
    int combo = 0;
    if (g.wt) combo = ((y > 0) << 3) | ((y < H - 1) << 2) | ((x > 0) << 1) | (x < W - 1 ? 1 : 0);
    float4 tv[NB][4];
#pragma unroll
    for (int a = 0; a < NB; ++a)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
        tv[a][q4] = *reinterpret_cast<const float4*>(&s_tt[combo * NCH + n0 + a * 32 + 8 * q4]);
#pragma unroll
    for (int a = 0; a < NB; ++a)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = acc[a][q4 * 4 + r];
        v[0] += tv[a][q4].x; v[1] += tv[a][q4].y; v[2] += tv[a][q4].z; v[3] += tv[a][q4].w;
        if constexpr (EPI == kConvTanh) {
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = tanh_fast(v[r]);
        }
        if constexpr (EPI == kConvFactor) {
          float av[4];
          unpack4<T>(dv[a][q4], av);
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = v[r] * (1.f - av[r] * av[r]);
        }
        const uint2 q = pack4<T>(v);
        bad |= live & any_nonfinite4<T>(q);
        const int n = n0 + a * 32 + 8 * q4;
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, q), out, (p * g.ldc + n) * 2, 0, 0);
        if constexpr (EPI >= kConvStage) {
          float f[4], x[4];
          unpack4<T>(q, f);
          if constexpr (EPI == kConvStage) {
            float yh[4];
            unpack4<T>(dv[a][q4], yh);
#pragma unroll
            for (int r = 0; r < 4; ++r) x[r] = fmaf(g.h, g.coef * f[r], yh[r]);
          } else {
            const float4 av = av4[a][q4];
            const float sa[4] = {S * av.x, S * av.y, S * av.z, S * av.w};
            const uint2 lq = pack4<T>(sa);
            bad |= live & any_nonfinite4<T>(lq);
            float lam[4];
            unpack4<T>(lq, lam);
#pragma unroll
            for (int r = 0; r < 4; ++r) x[r] = fmaf(g.h, g.coef * f[r], g.bw * lam[r]);
          }
          uint2 xq = pack4<T>(x);
          if (n >= g.d) xq = make_uint2(0u, 0u);
          if constexpr (EPI == kConvCotangent) bad |= live & any_nonfinite4<T>(xq);
          __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, xq), next, (p * g.ldc + n) * 2, 0, 0);
        }
      }
  }
  if (g.detect) raise_if_any(bad, g.ctl);
}

}  // namespace rampde
