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
// of one tap NCT weight fragments, which come from memory in the order in which they are used (1 KB each, four blocks
// ahead), and MT pixel fragments from LDS (a tap is a shifted pixel address) for NCT MT matrix instructions.
#pragma once
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
  const float *bias1, *wt1, *bias2, *wt2;  // fp32 (rounded) biases [64], time-channel weights [9][64] (null: none)
  float tau;                         // stage time, already rounded to low
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
  return (size_t)(lines + 4) * (Wd + 2) * conv_pair_pitch(C32) * 2 + 2 * (16 + 10) * 32 * C32 * 4;
}
inline bool conv_pair_applies(int Cpad, int Wd) { return Cpad == 64 && Wd >= 1 && Wd <= 64; }
typedef uint32_t u32x4p __attribute__((ext_vector_type(4)));
constexpr int kPairLookahead = 3;  // contraction blocks of weights in flight

template <class E>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t pair_window(const E* p, int elements) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<E*>(p), 0, elements * (int)sizeof(E), 0x00020000);
}

// The contraction: acc[m][t] += weights of output channels 16 t .. x pixels of block m.  base: LDS element of the block's
// pixel (this lane's) and channel chunk.
template <class T, int C32, int MT>
struct PairGemm {
  static constexpr int NCT = 2 * C32, NB = 9 * C32, PITCH = conv_pair_pitch(C32);
  u16x8 w[kPairLookahead][NCT];
  const uint16_t* Wf;
  __device__ __forceinline__ void load_w(int it, u16x8 (&dst)[NCT]) {
    const int tap = it / C32, kk = it % C32;
#pragma unroll
    for (int t = 0; t < NCT; ++t) dst[t] = *reinterpret_cast<const u16x8*>(Wf + ((tap * 2 + kk) * 4 + t) * 512);
  }
  __device__ __forceinline__ void start(const uint16_t* frags) {
    Wf = frags + (threadIdx.x & 63) * 8;
#pragma unroll
    for (int i = 0; i < kPairLookahead; ++i) load_w(i, w[i]);
  }
  __device__ __forceinline__ void run(const uint16_t* in, const int (&base)[MT], int LW, f32x4 (&acc)[MT][NCT]) {
    auto load_b = [&](int it, u16x8 (&fb)[MT]) __attribute__((always_inline)) {
      const int tap = it / C32, kk = it % C32;
      const int shift = ((tap / 3 - 1) * LW + (tap % 3 - 1)) * PITCH;
#pragma unroll
      for (int m = 0; m < MT; ++m) fb[m] = *reinterpret_cast<const u16x8*>(&in[base[m] + shift + kk * 32]);
    };
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int t = 0; t < NCT; ++t) acc[m][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    u16x8 fb[2][MT];
    load_b(0, fb[0]);
#pragma unroll
    for (int it = 0; it < NB; ++it) {
      u16x8 cur[NCT];
#pragma unroll
      for (int t = 0; t < NCT; ++t) cur[t] = w[it % kPairLookahead][t];
      if (it + 1 < NB) load_b(it + 1, fb[(it + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int t = 0; t < NCT; ++t) acc[m][t] = Low<T>::mfma16(cur[t], fb[it & 1][m], acc[m][t]);
      if (it + kPairLookahead < NB) load_w(it + kPairLookahead, w[it % kPairLookahead]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
};

template <class T, int C32, int MT1, int MT2, bool VJP>
__global__ __launch_bounds__(256, MT1 <= 5 ? 2 : 1) void conv_pair(ConvPair g, ConvPairShape sh) {
  constexpr int NT = 256, NCT = 2 * C32, C8 = 4 * C32, NCH = 32 * C32, PITCH = conv_pair_pitch(C32);
  constexpr int MAXC = ((64 * MT1 + 128) * C8 + NT - 1) / NT;  // staged chunks of a thread: at most 2 lines of 64 more than the hidden tile
  constexpr int MAXO = (64 * MT2 * C8 + NT - 1) / NT;          // ... of the tile's own lines
  extern __shared__ __attribute__((aligned(16))) uint16_t cp_smem[];
  const int W = g.Wd, H = g.H, PR = sh.lines, LW = W + 2;
  uint16_t* sIn = cp_smem;                                               // [PR + 4][W + 2][PITCH]
  float* s_tt = reinterpret_cast<float*>(sIn + (PR + 4) * LW * PITCH);   // [2][16][NCH]: bias + time term by border class
  float* s_wt = s_tt + 2 * 16 * NCH;                                     // [2][10][NCH]: time-channel weights, bias
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fl = lane & 15, fg = lane >> 4;

  const int img = blockIdx.x / sh.per_image, y0 = (blockIdx.x - img * sh.per_image) * PR;
  const int rows = min(PR, H - y0);
  const int f0 = max(y0 - 2, 0), f1 = min(y0 + rows + 2, H);  // staged image lines
  const int h0 = max(y0 - 1, 0), h1 = min(y0 + rows + 1, H);  // lines of the first convolution
  const size_t line0 = (size_t)img * H;
  const int staged = (f1 - f0) * W, n1 = (h1 - h0) * W, n2 = rows * W;
  auto line_of = [&](int p) __attribute__((always_inline)) { return (p * sh.magic) >> 16; };
  auto lds_at = [&](int p, int first) __attribute__((always_inline)) {  // pixel p of the lines from image line `first` on
    const int l = line_of(p);
    return ((first - y0 + 2 + l) * LW + p - l * W + 1) * PITCH;
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

  // ---- time terms, zero columns and lines
  if constexpr (!VJP) {
    for (int i = tid; i < 2 * 10 * NCH; i += NT) {
      const int layer = i / (10 * NCH), t = i / NCH % 10, n = i % NCH;
      const float* wt = layer ? g.wt2 : g.wt1;
      s_wt[i] = t == 9 ? (layer ? g.bias2 : g.bias1)[n] : wt ? wt[t * 64 + n] : 0.f;
    }
  }
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
  if constexpr (!VJP) {
    for (int i = tid; i < 2 * 16 * NCH; i += NT) {
      const int layer = i / (16 * NCH), combo = i / NCH % 16, n = i % NCH;
      const float* wt = s_wt + layer * 10 * NCH;
      float sum = 0.f;
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        const int dy = t / 3 - 1, dx = t % 3 - 1;
        const bool ok = (dy >= 0 || (combo & 8)) && (dy <= 0 || (combo & 4)) && (dx >= 0 || (combo & 2)) && (dx <= 0 || (combo & 1));
        sum += ok ? wt[t * NCH + n] * g.tau : 0.f;
      }
      s_tt[i] = wt[9 * NCH + n] + sum;
    }
  }
  auto border = [&](int y, int x) __attribute__((always_inline)) {
    return ((y > 0) << 3) | ((y < H - 1) << 2) | ((x > 0) << 1) | (x < W - 1 ? 1 : 0);
  };

  bool bad = false;
  // ---- first convolution
  {
    int base[MT1], combo[MT1];
    uint2 dv[VJP ? MT1 : 1][NCT];
#pragma unroll
    for (int m = 0; m < MT1; ++m) {
      const int p = (wave * MT1 + m) * 16 + fl, pc = p < n1 ? p : 0, l = line_of(pc);
      base[m] = lds_at(pc, h0) + fg * 8;
      if constexpr (!VJP) combo[m] = border(h0 + l, pc - l * W);
    }
    if constexpr (VJP) {  // the stored activations for the tanh' factor
      const auto act = pair_window(g.act + (line0 + h0) * W * 64, n1 * 64);
#pragma unroll
      for (int m = 0; m < MT1; ++m)
#pragma unroll
        for (int t = 0; t < NCT; ++t)
          dv[m][t] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(act, ((wave * MT1 + m) * 16 + fl) * 128 + t * 32 + fg * 8, 0, 0));
    }
    f32x4 acc[MT1][NCT];
    first.run(sIn, base, LW, acc);
    __syncthreads();  // the input has been read (and the time terms are written)
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
          const float4 tv = *reinterpret_cast<const float4*>(&s_tt[combo[m] * NCH + n]);
          v[0] = tanh_fast(v[0] + tv.x); v[1] = tanh_fast(v[1] + tv.y);
          v[2] = tanh_fast(v[2] + tv.z); v[3] = tanh_fast(v[3] + tv.w);
        }
        const uint2 q = pack4<T>(v);
        if constexpr (VJP) bad |= on & any_nonfinite4<T>(q);
        if (on) *reinterpret_cast<uint2*>(&sIn[base[m] - fg * 8 + n]) = q;
      }
    }
  }
  PairGemm<T, C32, MT2> second;
  if (g.C) second.start(g.W2);
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
    int base[MT2], combo[MT2];
#pragma unroll
    for (int m = 0; m < MT2; ++m) {
      const int p = (wave * MT2 + m) * 16 + fl, pc = p < n2 ? p : 0, l = line_of(pc);
      base[m] = lds_at(pc, y0) + fg * 8;
      if constexpr (!VJP) combo[m] = border(y0 + l, pc - l * W);
    }
    f32x4 acc[MT2][NCT];
    second.run(sIn, base, LW, acc);
    __syncthreads();
#pragma unroll
    for (int m = 0; m < MT2; ++m) {
      const bool on = (wave * MT2 + m) * 16 + fl < n2;
#pragma unroll
      for (int t = 0; t < NCT; ++t) {
        const int n = t * 16 + fg * 4;
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = acc[m][t][r];
        if constexpr (!VJP) {
          const float4 tv = *reinterpret_cast<const float4*>(&s_tt[(16 + combo[m]) * NCH + n]);
          v[0] += tv.x; v[1] += tv.y; v[2] += tv.z; v[3] += tv.w;
        }
        if (on) *reinterpret_cast<uint2*>(&sIn[base[m] - fg * 8 + n]) = pack4<T>(v);
      }
    }
    __syncthreads();
    const auto out = pair_window(g.C + (line0 + y0) * W * 64, n2 * 64);
    const int dst0 = tid % C8 * 16, n = tid % C8 * 8;
    if (!g.next) {
#pragma unroll
      for (int i = 0; i < MAXO; ++i) {
        const int id = tid + NT * i, px = id / C8;
        const uint4 q = *reinterpret_cast<const uint4*>(&sIn[lds_at(px < n2 ? px : 0, y0) + n]);
        if constexpr (VJP) bad |= px < n2 & (any_nonfinite4<T>(make_uint2(q.x, q.y)) | any_nonfinite4<T>(make_uint2(q.z, q.w)));
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4p, q), out, px * 128 + dst0, 0, 0);
      }
    } else {
      const auto next = pair_window(g.next + (line0 + y0) * W * 64, n2 * 64);
      // (a chunk past the d columns reads and keeps zeros)
      const int outside = n < g.d ? 0 : 0x40000000;
      const auto ybase = pair_window(g.base + (VJP ? 0 : (line0 + y0) * W * g.d), VJP ? 0 : n2 * g.d);
      const auto adj = pair_window(g.adj + (VJP ? (line0 + y0) * W * g.d : 0), VJP ? n2 * g.d : 0);
      const float S = VJP ? g.ctl->S : 0.f;
#pragma unroll
      for (int i = 0; i < MAXO; ++i) {
        const int id = tid + NT * i, px = id / C8;
        const uint4 q = *reinterpret_cast<const uint4*>(&sIn[lds_at(px < n2 ? px : 0, y0) + n]);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4p, q), out, px * 128 + dst0, 0, 0);
        const uint2 half[2] = {make_uint2(q.x, q.y), make_uint2(q.z, q.w)};
        uint4 xq;
        if constexpr (VJP) {
          float a[8];
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const float4 v = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(adj, (px * g.d + n + 4 * e) * 4 | outside, 0, 0));
            a[4 * e] = v.x; a[4 * e + 1] = v.y; a[4 * e + 2] = v.z; a[4 * e + 3] = v.w;
          }
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            float fe[4], lam[4], xe[4];
            const float sa[4] = {S * a[4 * e], S * a[4 * e + 1], S * a[4 * e + 2], S * a[4 * e + 3]};
            const uint2 lq = pack4<T>(sa);
            unpack4<T>(half[e], fe);
            unpack4<T>(lq, lam);
#pragma unroll
            for (int r = 0; r < 4; ++r) xe[r] = fmaf(g.h, g.coef * fe[r], g.bw * lam[r]);
            uint2 z = pack4<T>(xe);
            if (n >= g.d) z = make_uint2(0u, 0u);
            bad |= px < n2 & (any_nonfinite4<T>(half[e]) | any_nonfinite4<T>(lq) | any_nonfinite4<T>(z));
            if (e == 0) { xq.x = z.x; xq.y = z.y; } else { xq.z = z.x; xq.w = z.y; }
          }
        } else {
          const uint4 yq = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(ybase, (px * g.d + n) * 2 | outside, 0, 0));
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
  if (g.detect) raise_if_any(bad, g.ctl);
}

}  // namespace rampde
