// Both 3x3 zero-padded convolutions of the two-convolution velocity in one launch, on channels-last rows of at most 64
// channels: an evaluation k = W2 * tanh(W1 * z + ...) + ... (paper Alg. 1, the low-precision evaluation of Phi) and its
// vector-Jacobian product zbar = W1^T * (W2^T * kbar . (1 - act^2)) (eq. (vjp); the transposed convolution is the same
// kernel with the flipped, transposed weights).
//
// A workgroup of four wavefronts owns `lines` whole image lines of one image.  The input lines with a halo of two above and
// below are staged in LDS, the first convolution is formed on the tile's lines and one more on either side (the same sums
// as in the neighbouring tile, bit for bit), rounded and put where the input was: all of its sums are in registers by
// then.  The second convolution reads it from there, and its result leaves through LDS too, so that every access to
// memory is 16 bytes per lane and whole pixels.
//
// v_mfma_f32_16x16x32 with the weights as the first operand: a lane ends with 4 consecutive output channels of one pixel.
// A wavefront multiplies all output channels with its MT blocks of 16 pixels: per contraction block of 32 input channels
// of one tap NCT weight fragments, which come from memory in the order in which they are used (1 KB each, three
// blocks ahead), and MT pixel fragments from LDS (a tap is a shifted pixel address) for NCT MT matrix instructions.
//
// It runs where conv_pass.hpp, which keeps a tile's state on chip over whole steps, does not: channel counts that are no
// multiple of 8, tableaux whose stages are no chain, dL/dt, calls in place, passes that are redone.  What bounds a launch
// (64 channels, 16 lines of 32 pixels, cycles of 75000 before the time channel became a block of the contraction): the
// input's arrival 13000, the two contractions 12700 and 11300 (10400 and 9200 of matrix instructions), tanh 10900, the output
// 15000: the memory's share moves 75 MB per evaluation of 128 images, 130 MB per vector-Jacobian product.
#pragma once
#include <type_traits>

#include "fused.hpp"

namespace rampde {

struct ConvPairShape {
  int lines, per_image, tiles;  // image lines of a tile, tiles of an image, tiles in all
  int mt1, mt2;                 // blocks of 16 pixels per wavefront: first, second convolution
  int magic;                    // p / W = p magic >> 16 for the pixels of a tile
};
struct ConvPair {
  const uint16_t* A;                 // [rows][64] stage input / slope cotangent
  const uint16_t *W1, *W2;           // weight fragments of the first and the second convolution (see cast_conv_layer)
  const uint16_t *T1, *T2;           // their time-channel weights and biases: [2][64][8], contraction index 0-8: tap, 9: bias
  const float *X1, *X2;              // the time-channel weights [9][64] in 32 bits ...
  const float *F1, *F2;              // ... and which outputs [64] have one that is not finite: 1 or 0 (see PairTime::odd)
  uint32_t tau;                      // stage time, low-precision bits
  const uint16_t* act;               // VJP: [rows][64] stored hidden activation
  uint16_t* mid;                     // [rows][64] hidden activation / its cotangent, or null: not kept
  uint16_t* C;                       // [rows][64] slope / cotangent of the stage input, or null: the hidden activation alone
  // what the next evaluation of a chained tableau reads, formed where its input is written (d a multiple of 8): the stage
  // input Q(base + h coef C) (base: the stored state) or the slope cotangent Q(bw Q(S adj) + h coef C) of the stage
  // before (adj: the fp32 adjoint).  base and adj have pitch d; the pad columns of next are zeroed.
  uint16_t* next;
  const uint16_t* base;
  const float* adj;
  int d;
  float h, coef, bw;
  Ctl* ctl;                          // may be null (forward pass)
  int detect;
  int H, Wd;
};

constexpr int conv_pair_pitch(int C32) { return 32 * C32 + 8; }  // elements per LDS row of one pixel's channels
inline size_t conv_pair_lds_bytes(int C32, int lines, int Wd) {
  return (size_t)(lines + 4) * (Wd + 2) * conv_pair_pitch(C32) * 2;
}
inline bool conv_pair_applies(int Cpad, int Wd) { return Cpad == 64 && Wd >= 1 && Wd <= 64; }
typedef uint32_t u32x4p __attribute__((ext_vector_type(4)));

template <class E>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t pair_window(const E* p, int elements) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<E*>(p), 0, elements * (int)sizeof(E), 0x00020000);
}

// The contraction: acc[m][t] += weights of output channels 16 t .. x pixels of block m.  base: LDS element of the block's
// pixel (this lane's) and channel chunk.  The first two lines of taps are one loop body: unrolled over all nine taps, a
// launch fetched more instructions that it executes once.
// LA: contraction blocks of weights in flight.
template <class T, int C32, int MT, int LA = 3>
struct PairGemm {
  static constexpr int NCT = 2 * C32, U = 3 * C32, PITCH = conv_pair_pitch(C32), FR = U % 2 ? 3 : 2;
  u16x8 w[LA][NCT];
  __amdgpu_buffer_rsrc_t frags;
  int at;  // bytes into the fragments
  __device__ __forceinline__ void load_w(int u, u16x8 (&dst)[NCT]) {
#pragma unroll
    for (int t = 0; t < NCT; ++t)
      dst[t] = __builtin_bit_cast(u16x8, __builtin_amdgcn_raw_buffer_load_b128(frags, (threadIdx.x & 63) * 16 + t * 1024, at + (u / C32 * 8 + u % C32 * 4) * 1024, 0));
  }
  __device__ __forceinline__ void start(const uint16_t* W) {
    frags = pair_window(W, 64 * 576);
    at = 0;
#pragma unroll
    for (int i = 0; i < LA; ++i) load_w(i, w[i]);
  }
  // One line of taps.  The lines are multiplied in the order dy = 0, -1, 1, in which the weights lie.  b: LDS element of
  // the blocks' pixels at the line's first tap; fb[0]: the pixels' first fragments.  AHEAD: those of the next line, `shift`
  // elements on, are read too.  LAST: no weights follow.
  template <bool AHEAD, bool LAST>
  __device__ __forceinline__ void line(const uint16_t* in, int (&b)[MT], int shift, u16x8 (&fb)[FR][MT], f32x4 (&acc)[MT][NCT]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (AHEAD && u + 1 == U) {
#pragma unroll
        for (int m = 0; m < MT; ++m) b[m] += shift;
      }
      if (AHEAD || u + 1 < U) load_b(in, b, (u + 1) % U, fb[(u + 1) % FR]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int t = 0; t < NCT; ++t) acc[m][t] = Low<T>::mfma16(w[u % LA][t], fb[u % FR][m], acc[m][t]);
      if (u + LA == U) at += 3 * 8 * 1024;
      if (!LAST || u + LA < U) load_w((u + LA) % U, w[u % LA]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  __device__ __forceinline__ void load_b(const uint16_t* in, const int (&b)[MT], int u, u16x8 (&fb)[MT]) {
#pragma unroll
    for (int m = 0; m < MT; ++m) fb[m] = *reinterpret_cast<const u16x8*>(&in[b[m] + u / C32 * PITCH + u % C32 * 32]);
  }
  // between: issues what the epilogue needs from memory, before the last line of taps (loads return in order: issued
  // earlier, the first weights behind them would wait for them)
  template <class Between>
  __device__ __forceinline__ void run(const uint16_t* in, const int (&base)[MT], int LW, f32x4 (&acc)[MT][NCT], const Between& between) {
    int b[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) b[m] = base[m] - PITCH;
    u16x8 fb[FR][MT];
    load_b(in, b, 0, fb[0]);
#pragma unroll 1
    for (int i = 0; i < 2; ++i) line<true, false>(in, b, (3 * i - 1) * LW * PITCH, fb, acc);
    between();
    __builtin_amdgcn_sched_barrier(0);
    line<false, true>(in, b, 0, fb, acc);
  }
};

// One more contraction block in front: the time channel (the stage time where the tap is inside the image) and the bias.
template <class T, int NCT>
struct PairTime {
  u16x8 w[NCT];
  __device__ __forceinline__ void start(const uint16_t* W) {
    const auto win = pair_window(W, 2 * 64 * 8);  // (contraction indices 16 and up: zeros)
#pragma unroll
    for (int t = 0; t < NCT; ++t)
      w[t] = __builtin_bit_cast(u16x8, __builtin_amdgcn_raw_buffer_load_b128(win, ((threadIdx.x & 63) / 16 * 64 + t * 16 + (threadIdx.x & 15)) * 16, 0, 0));
  }
  // edges: bits 0 to 3, the pixel is not in the image's first line, last line, first column, last column
  __device__ __forceinline__ void run(uint32_t tau, unsigned edges, f32x4 (&acc)[NCT]) {
    constexpr uint32_t one = std::is_same<T, BF16>::value ? 0x3f80u : 0x3c00u;
    const bool t = edges & 1, b = edges & 2, l = edges & 4, r = edges & 8;
    auto two = [&](bool lo, bool hi) __attribute__((always_inline)) { return (lo ? tau : 0u) | (hi ? tau << 16 : 0u); };
    uint4 q = make_uint4(two(t & l, t), two(t & r, l), two(true, r), two(b & l, b));
    if (threadIdx.x & 16) q.x = two(b & r, false) | one << 16;  // (lanes of contraction indices 8 to 15)
#pragma unroll
    for (int o = 0; o < NCT; ++o) acc[o] = Low<T>::mfma16(w[o], __builtin_bit_cast(u16x8, q), f32x4{0.f, 0.f, 0.f, 0.f});
  }
  // Time weights that are not finite once rounded are zeros among the fragments: a tap outside the image leaves its weight
  // out of the sum, where a product with zero would be NaN.  Whether there are any (uniform; flag: that of output
  // threadIdx.x % 64), and their terms.
  static __device__ __forceinline__ bool odd(float flag) { return __builtin_amdgcn_ballot_w64(flag != 0.f) != 0; }
  static __device__ __forceinline__ void add_odd(const float* X, uint32_t tau, unsigned edges, f32x4 (&acc)[NCT]) {
    const float time = Low<T>::to_f32((uint16_t)tau);
#pragma unroll 1
    for (int tap = 0; tap < 9; ++tap) {
      const bool inside = (tap / 3 > 0 || edges & 1) && (tap / 3 < 2 || edges & 2) && (tap % 3 > 0 || edges & 4) && (tap % 3 < 2 || edges & 8);
#pragma unroll
      for (int o = 0; o < NCT; ++o) {
        const float4 x = *reinterpret_cast<const float4*>(X + tap * 64 + o * 16 + (threadIdx.x & 63) / 16 * 4);
        const float v[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[o][r] += inside && !__builtin_isfinite(v[r]) ? time * v[r] : 0.f;
      }
    }
  }
};

// One tile.  With a control block nothing is done once a cotangent chain has been rejected.
template <class T, int C32, int MT1, int MT2, bool VJP>
__device__ __forceinline__ void pair_tile(const ConvPair& g, const ConvPairShape& sh, int tile, uint16_t* sIn) {
  constexpr int NT = 256, NCT = 2 * C32, C8 = 4 * C32, PITCH = conv_pair_pitch(C32);
  constexpr int MAXC = ((64 * MT1 + 128) * C8 + NT - 1) / NT;  // staged chunks of a thread: at most 2 lines of 64 more than the hidden tile
  constexpr int MAXO = (64 * MT2 * C8 + NT - 1) / NT;          // ... of the tile's own lines
  const int W = g.Wd, H = g.H, PR = sh.lines, LW = W + 2;              // sIn: [PR + 4][W + 2][PITCH]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fl = lane & 15, fg = lane >> 4;

  const int img = tile / sh.per_image, y0 = (tile - img * sh.per_image) * PR;
  const int rows = min(PR, H - y0);
  const int f0 = max(y0 - 2, 0), f1 = min(y0 + rows + 2, H);  // staged image lines
  const int h0 = max(y0 - 1, 0), h1 = min(y0 + rows + 1, H);  // lines of the first convolution
  const size_t line0 = (size_t)img * H;
  const int staged = (f1 - f0) * W, n1 = (h1 - h0) * W, n2 = rows * W;
  auto edges_of = [&](int y, int x) __attribute__((always_inline)) {
    return (unsigned)((y > 0) | (y < H - 1) << 1 | (x > 0) << 2 | (x < W - 1) << 3);
  };
  auto line_of = [&](int p) __attribute__((always_inline)) { return (p * sh.magic) >> 16; };
  auto lds_at = [&](int p, int first) __attribute__((always_inline)) {  // pixel p of the lines from image line `first` on
    const int l = line_of(p);
    return ((first - y0 + 2 + l) * LW + p - l * W + 1) * PITCH;
  };

  // (see PairTime::odd; behind the contraction, where registers are free)
  auto add_odd = [&](const float* X, int n, int first, auto& acc) __attribute__((always_inline)) {
    constexpr int MT = sizeof(acc) / sizeof(acc[0]);
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      const int p = (wave * MT + m) * 16 + fl, pc = p < n ? p : 0, l = line_of(pc);
      PairTime<T, NCT>::add_odd(X, g.tau, edges_of(first + l, pc - l * W), acc[m]);
    }
  };

  // ---- the input lines (past the window: zeros)
  u16x8 reg[MAXC];
  {
    const auto src = pair_window(g.A + (line0 + f0) * W * 64, staged * 64);
#pragma unroll
    for (int i = 0; i < MAXC; ++i) {
      const int id = tid + NT * i;
      reg[i] = __builtin_bit_cast(u16x8, __builtin_amdgcn_raw_buffer_load_b128(src, (id / C8) * 128 + (id % C8) * 16, 0, 0));
    }
  }
  if (g.ctl && g.ctl->poison) return;
  PairGemm<T, C32, MT1> first;
  first.start(g.W1);

  PairTime<T, NCT> time;
  float odd1 = 0.f, odd2 = 0.f;
  if constexpr (!VJP) {
    time.start(g.T1);
    odd1 = g.F1[lane];
    odd2 = g.F2[lane];
  }

  // ---- zero columns and lines
  const u16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int id = tid; id < (PR + 4) * 2 * C8; id += NT) {
    const int c8 = id % C8, side = (id / C8) & 1, l = id / (2 * C8);
    *reinterpret_cast<u16x8*>(&sIn[(l * LW + (side ? W + 1 : 0)) * PITCH + c8 * 8]) = zero;
  }
  if (h0 == 0)
    for (int id = tid; id < W * C8; id += NT)
      *reinterpret_cast<u16x8*>(&sIn[((1 - y0) * LW + 1 + id / C8) * PITCH + (id % C8) * 8]) = zero;
  if (h1 == H)
    for (int id = tid; id < W * C8; id += NT)
      *reinterpret_cast<u16x8*>(&sIn[((H - y0 + 2) * LW + 1 + id / C8) * PITCH + (id % C8) * 8]) = zero;
#pragma unroll
  for (int i = 0; i < MAXC; ++i) {
    const int id = tid + NT * i, px = id / C8;
    if (px < staged) *reinterpret_cast<u16x8*>(&sIn[lds_at(px, f0) + (id % C8) * 8]) = reg[i];
  }
  __syncthreads();
  uint32_t bad = 0u;  // (kNonfiniteBits of it)
  auto watch = [&](uint2 q) __attribute__((always_inline)) { return Low<T>::nonfinite2(q.x) | Low<T>::nonfinite2(q.y); };
  // ---- first convolution
  {
    int base[MT1];
    f32x4 acc[MT1][NCT];
    uint2 dv[VJP ? MT1 : 1][NCT];
#pragma unroll
    for (int m = 0; m < MT1; ++m) {
      const int p = (wave * MT1 + m) * 16 + fl, pc = p < n1 ? p : 0, l = line_of(pc);
      base[m] = lds_at(pc, h0) + fg * 8;
      if constexpr (!VJP) {
        time.run(g.tau, edges_of(h0 + l, pc - l * W), acc[m]);
      } else {
#pragma unroll
        for (int t = 0; t < NCT; ++t) acc[m][t] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    }
    first.run(sIn, base, LW, acc, []() {});
    if (!VJP && time.odd(odd1)) add_odd(g.X1, n1, h0, acc);
    if constexpr (VJP) {  // the stored activations for the tanh' factor (requested any earlier, beside the multiplication, they slow it down by more)
      const auto act = pair_window(g.act + (line0 + h0) * W * 64, n1 * 64);
#pragma unroll
      for (int m = 0; m < MT1; ++m)
#pragma unroll
        for (int t = 0; t < NCT; ++t)
          dv[m][t] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(act, ((wave * MT1 + m) * 16 + fl) * 128 + t * 32 + fg * 8, 0, 0));
    }
    __syncthreads();  // the input has been read
#pragma unroll
    for (int m = 0; m < MT1; ++m) {
      const bool on = (wave * MT1 + m) * 16 + fl < n1;
#pragma unroll
      for (int t = 0; t < NCT; ++t) {
        const int n = t * 16 + fg * 4;
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = acc[m][t][r];
        if constexpr (VJP) {
          float av[4];
          unpack4<T>(dv[m][t], av);
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = v[r] * (1.f - av[r] * av[r]);
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = tanh_fast(v[r]);
        }
        const uint2 q = pack4<T>(v);
        if constexpr (VJP) bad |= on ? watch(q) : 0u;
        if (on) *reinterpret_cast<uint2*>(&sIn[base[m] - fg * 8 + n]) = q;
      }
    }
  }
  PairGemm<T, C32, MT2> second;
  if (g.C) {
    second.start(g.W2);
    if constexpr (!VJP) time.start(g.T2);
  }
  __syncthreads();
  if (g.mid) {
    const auto out = pair_window(g.mid + (line0 + y0) * W * 64, n2 * 64);
#pragma unroll
    for (int i = 0; i < MAXO; ++i) {
      const int id = tid + NT * i, px = id / C8;
      const u16x8 q = *reinterpret_cast<const u16x8*>(&sIn[lds_at(px < n2 ? px : 0, y0) + (id % C8) * 8]);
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4p, q), out, px * 128 + (id % C8) * 16, 0, 0);
    }
  }
  // ---- second convolution
  if (g.C) {
    int base[MT2];
    f32x4 acc[MT2][NCT];
#pragma unroll
    for (int m = 0; m < MT2; ++m) {
      const int p = (wave * MT2 + m) * 16 + fl, pc = p < n2 ? p : 0, l = line_of(pc);
      base[m] = lds_at(pc, y0) + fg * 8;
      if constexpr (!VJP) {
        time.run(g.tau, edges_of(y0 + l, pc - l * W), acc[m]);
      } else {
#pragma unroll
        for (int t = 0; t < NCT; ++t) acc[m][t] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    }
    // what the next evaluation's input is formed from: the stored state in flight beside the multiplication, the adjoint
    // behind it (without `next` nothing is read; a chunk past the d columns reads zeros)
    const int dst0 = tid % C8 * 16, n = tid % C8 * 8, outside = n < g.d ? 0 : 0x40000000;
    uint4 ahead[MAXO][VJP ? 2 : 1];
    auto fetch = [&]() __attribute__((always_inline)) {
      const int live = g.next ? n2 * g.d : 0;
      if constexpr (VJP) {
        const auto adj = pair_window(g.adj + (g.next ? (line0 + y0) * W * g.d : 0), live);
#pragma unroll
        for (int i = 0; i < MAXO; ++i)
#pragma unroll
          for (int e = 0; e < 2; ++e)
            ahead[i][e] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(adj, ((tid + NT * i) / C8 * g.d + n + 4 * e) * 4 | outside, 0, 0));
      } else {
        const auto ybase = pair_window(g.base + (g.next ? (line0 + y0) * W * g.d : 0), live);
#pragma unroll
        for (int i = 0; i < MAXO; ++i)
          ahead[i][0] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(ybase, ((tid + NT * i) / C8 * g.d + n) * 2 | outside, 0, 0));
      }
    };
    if constexpr (VJP) {
      second.run(sIn, base, LW, acc, []() {});
      fetch();
    } else {
      second.run(sIn, base, LW, acc, fetch);
    }
    if (!VJP && time.odd(odd2)) add_odd(g.X2, n2, y0, acc);
    __syncthreads();
#pragma unroll
    for (int m = 0; m < MT2; ++m) {
      const bool on = (wave * MT2 + m) * 16 + fl < n2;
#pragma unroll
      for (int t = 0; t < NCT; ++t) {
        const float v[4] = {acc[m][t][0], acc[m][t][1], acc[m][t][2], acc[m][t][3]};
        if (on) *reinterpret_cast<uint2*>(&sIn[base[m] - fg * 8 + t * 16 + fg * 4]) = pack4<T>(v);
      }
    }
    __syncthreads();
    const auto out = pair_window(g.C + (line0 + y0) * W * 64, n2 * 64);
    if (!g.next) {
#pragma unroll
      for (int i = 0; i < MAXO; ++i) {
        const int id = tid + NT * i, px = id / C8;
        const uint4 q = *reinterpret_cast<const uint4*>(&sIn[lds_at(px < n2 ? px : 0, y0) + n]);
        if constexpr (VJP) bad |= watch(make_uint2(q.x, q.y)) | watch(make_uint2(q.z, q.w));  // (past the tile: its first pixel)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4p, q), out, px * 128 + dst0, 0, 0);
      }
    } else {
      const auto next = pair_window(g.next + (line0 + y0) * W * 64, n2 * 64);
      const float S = VJP ? g.ctl->S : 0.f;
#pragma unroll
      for (int i = 0; i < MAXO; ++i) {
        const int id = tid + NT * i, px = id / C8;
        const uint4 q = *reinterpret_cast<const uint4*>(&sIn[lds_at(px < n2 ? px : 0, y0) + n]);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4p, q), out, px * 128 + dst0, 0, 0);
        const uint2 half[2] = {make_uint2(q.x, q.y), make_uint2(q.z, q.w)};
        uint4 xq;
        if constexpr (VJP) {
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            float fe[4], lam[4], xe[4];
            const float4 a = __builtin_bit_cast(float4, ahead[i][e]);
            const float sa[4] = {S * a.x, S * a.y, S * a.z, S * a.w};
            const uint2 lq = pack4<T>(sa);
            unpack4<T>(half[e], fe);
            unpack4<T>(lq, lam);
#pragma unroll
            for (int r = 0; r < 4; ++r) xe[r] = fmaf(g.h, g.coef * fe[r], g.bw * lam[r]);
            uint2 z = pack4<T>(xe);
            if (n >= g.d) z = make_uint2(0u, 0u);
            bad |= px < n2 ? watch(half[e]) | watch(lq) | watch(z) : 0u;
            if (e == 0) { xq.x = z.x; xq.y = z.y; } else { xq.z = z.x; xq.w = z.y; }
          }
        } else {
          const uint4 yq = ahead[i][0];
          const uint2 yh[2] = {make_uint2(yq.x, yq.y), make_uint2(yq.z, yq.w)};
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            float fe[4], ye[4], xe[4];
            unpack4<T>(half[e], fe);
            unpack4<T>(yh[e], ye);
#pragma unroll
            for (int r = 0; r < 4; ++r) xe[r] = fmaf(g.h, g.coef * fe[r], ye[r]);
            uint2 z = pack4<T>(xe);
            if (n >= g.d) z = make_uint2(0u, 0u);
            if (e == 0) { xq.x = z.x; xq.y = z.y; } else { xq.z = z.x; xq.w = z.y; }
          }
        }
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4p, xq), next, px * 128 + dst0, 0, 0);
      }
    }
  }
  if (g.detect) raise_if_any((bad & kNonfiniteBits) != 0u, g.ctl);
}

template <class T, int C32, int MT1, int MT2, bool VJP>
__global__ __launch_bounds__(256, MT1 <= 5 ? 2 : 1) void conv_pair(ConvPair g, ConvPairShape sh) {
  extern __shared__ __attribute__((aligned(16))) uint16_t cp_smem[];
  pair_tile<T, C32, MT1, MT2, VJP>(g, sh, blockIdx.x, cp_smem);
}

}  // namespace rampde
