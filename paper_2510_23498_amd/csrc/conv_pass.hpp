// The convolutional velocity with at most 64 channels over whole steps: a workgroup keeps its image lines' state on chip
// and the evaluations of all stages (forward: of all steps) follow one another in one launch.
//
// What this is for: an evaluation per launch (conv_pair.hpp) reads and writes the stage's tensors of the whole batch, all
// workgroups at the same time, with the matrix units idle: 75 MB per evaluation and 130 MB per vector-Jacobian product of
// 64 x 32 x 32, 128 images, where two thirds of a launch are not multiplication.  Here the stage input is in LDS, the sums
// over the stages are in registers in the order in which the matrix instructions leave them, and a forward pass writes the
// stored states and nothing else.
//
// A workgroup of four wavefronts owns `lines` lines of an image, at most 256 pixels, so that two run on a compute unit and
// the arithmetic of one runs beside the multiplication of the other.  The tiles of an image exchange their first and last
// lines in front of each convolution: as 64-bit words {a pair of values, number of the exchange}, stored and loaded as
// device-scope atomics, so a word is known to have arrived by its own number and nothing else has to be ordered.  There are
// two sets of words, used in turn: a tile stores exchange e + 2 after it has seen its neighbours' e + 1, which they store
// after they have read its e.  While the words are on their way the three taps of the middle line are multiplied.
//
// The tiles of an image have to run at the same time: a launch has at most as many workgroups as the device runs at once.
// If others hold the device a wait ends after kPassWaitTicks; the launch then raises `stalled`, and conv_redo_* behind it do the
// work again, one workgroup per image (nothing is left of a launch that was given up: they start from its inputs).  Each group
// of adjoint steps has a flag of its own: the groups behind a redone one run on these kernels again.  A pass
// under overflow detection is redone by way of the host instead.  Time weights that are not finite go the same way from the
// start (pass_reset): beside the contractions here their terms (PairTime::add_odd) cost registers, 137 spilled instead of 5 in
// the recomputation of 64 channels.
//
// Measured, us per evaluation of 64 x 32 x 32, 128 images (512 workgroups of 8 lines): forward 30.1, recomputation 22.9, chain
// 36 (conv_pair.hpp with the passes over memory that it needs beside it 31, 28 and 45); 32 channels 10.2, 11.1 and 13.5;
// 32 channels, 20 x 28 x 28, 4 lines 6.2, 7.3 and 9.4.  Cycles per convolution and workgroup in the first: arithmetic of the
// epilogue 7100 (tanh, roundings, the next stage's input), matrix instructions 9000 (both workgroups of a compute unit at
// once), stores and the exchange's 3400, waiting for the neighbours 2800, barriers 1800.  Without any exchange (wrong results)
// it would be 20.3 per evaluation.  Words stored chunk by chunk instead of word by word cost 2.5 us more; plain stores
// between tiles that share an XCD's L2 gained 0.3; tiles of 16 lines, one workgroup to a compute unit, do not fit the
// registers (55); wavefronts that wait for a line each for themselves, and a head start for half of the workgroups, gained
// nothing.
#pragma once
#include "conv_pair.hpp"

namespace rampde {

constexpr int kPassStages = 4;
// How long a workgroup waits for a neighbour's words, of the 100 MHz counter: 20 ms.  (Workgroups start in order, so what
// it waits for comes as soon as others make room, unless two such launches each hold what the other one needs.)
constexpr unsigned long long kPassWaitTicks = 2000ull * 1000;
constexpr int kPassEvaluations = 96;  // per launch of a forward pass and round over the images: about 3 ms
struct PassShape {
  int lines, per_image, slots;  // lines of a tile, tiles of an image, images (or images x steps) at once
  int mt, magic;                // blocks of 16 pixels per wavefront; p / W = p magic >> 16
};
struct ConvPass {
  const uint16_t *W1, *W2;      // weight fragments in the order of use: forward W_1, W_2, chain W_2^T, W_1^T
  const uint16_t *T1, *T2;      // time-channel weights and biases (forward)
  const float *X1, *X2, *F1, *F2;  // (see ConvPair)
  const float* steptab;         // [N][1 + s]: step size, stage times rounded to low
  unsigned long long* words;    // [workgroups][2][2][Wd x 16-byte chunks of a pixel x 4]
  uint32_t first;               // number of the launch's first exchange
  uint32_t give_up_at;          // number of the exchange at which no workgroup looks for words (RAMPDE_NO_WAITS), 0: none
  int* stalled;
  int H, Wd, d, s, images;
  int64_t n;                    // elements from one stored state to the next
  float sub[kPassStages], b[kPassStages];  // a_{j+1, j}, b_j of the (chained) tableau
  int step, nsteps;             // forward: the steps step, step + 1, ... of N; else step, step - 1, ...
  int N;
  uint16_t* ckpt;
  // forward
  const float* y0;              // [image][d][H Wd]
  float* y;                     // [rows][d]
  float* yN;                    // like y0
  // backward: buffers of a step's stages [nsets][s][rows][64], step i in set (step - i) + set0
  uint16_t *Z, *ACT, *KBAR, *DELTA;
  int64_t stage_stride;
  int set0;
  const float* a_in;            // [rows][d]
  float* a_out;
  const float* gys;             // [rows][d] running-cost cotangent of the (one) step, or null
  unsigned* amax;               // [workgroups] max |a_out| bits
  Ctl* ctl;
  int detect;
};

constexpr int pass_words(int C32, int Wd) { return 4 * Wd * 4 * C32 * 4; }  // 64-bit words of a workgroup
inline size_t pass_lds_bytes(int C32, int lines, int Wd) { return (size_t)((lines + 2) * (Wd + 2) + 1) * conv_pair_pitch(C32) * 2; }

template <class T, int C32, int MT>
struct PassTile {
  static constexpr int NT = 256, NCT = 2 * C32, C8 = 4 * C32, PITCH = conv_pair_pitch(C32);
  using Gemm = PairGemm<T, C32, MT, C32 == 2 && MT <= 4 ? 2 : 3>;  // (registers: see the kernels)
  uint16_t* in;                 // LDS [lines + 2][W + 2][PITCH]
  const ConvPass& g;
  int W, LW, tid, wave, fl, fg;
  int y0, rows, n2, magic;
  int base[MT];                 // LDS element of this lane's pixels
  int spare;                    // ... of a place behind the tile, where lanes without a pixel write
  unsigned edges;               // 4 bits per block: pixel not in the image's first line, last line, first column, last column
  bool up, down;
  unsigned long long* mine;
  int pitch;                    // words of a workgroup
  uint32_t tag;

  __device__ __forceinline__ PassTile(const ConvPass& a, const PassShape& sh, uint16_t* lds) : in(lds), g(a) {
    W = g.Wd; LW = W + 2; magic = sh.magic;
    tid = threadIdx.x; wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    fl = tid & 15; fg = (tid >> 4) & 3;
    const int tile = blockIdx.x % sh.per_image;
    y0 = tile * sh.lines;
    rows = min(sh.lines, g.H - y0);
    n2 = rows * W;
    up = tile > 0;
    down = tile + 1 < sh.per_image;
    pitch = pass_words(C32, W);
    mine = g.words + (size_t)blockIdx.x * pitch;
    tag = g.first;
    edges = 0;
    spare = (sh.lines + 2) * LW * PITCH;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      const int p = pixel(m), pc = p < n2 ? p : 0, l = line_of(pc), x = pc - l * W, yy = y0 + l;
      base[m] = ((l + 1) * LW + x + 1) * PITCH;
      edges |= ((yy > 0) | (yy < g.H - 1) << 1 | (x > 0) << 2 | (x < W - 1) << 3) << (4 * m);
    }
    const u16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int i = tid * 8; i < (sh.lines + 2) * LW * PITCH; i += NT * 8) *reinterpret_cast<u16x8*>(&in[i]) = zero;
    __syncthreads();
  }
  // the thread's number as a value that the compiler does not know: what is computed from it is not kept in registers
  // over the loops of a launch
  __device__ __forceinline__ int me() const {
    int v = tid;
    asm volatile("" : "+v"(v));
    return v;
  }
  __device__ __forceinline__ int line_of(int p) const { return (p * magic) >> 16; }
  __device__ __forceinline__ int pixel(int m) const { return (wave * MT + m) * 16 + fl; }
  // this lane's place in row-major arrays of the tile's pixels, `ld` elements each: element of its first pixel's first
  // channel; + (16 m) ld + 16 t.  (A pixel past the tile is past the arrays' windows, or past `outside`)
  __device__ __forceinline__ int place(int ld) const {
    const int v = me();
    return (wave * MT * 16 + (v & 15)) * ld + ((v >> 4) & 3) * 4;
  }
  // the same with an offset past every window for the channels from d on
  template <class F>
  __device__ __forceinline__ void for_each(int ld, int size, const F& f) const {
    const int at = place(ld), first = (me() >> 4 & 3) * 4;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int t = 0; t < NCT; ++t) f(m, t, first + 16 * t < g.d ? (at + 16 * m * ld + 16 * t) * size : 0x40000000);
  }
  __device__ __forceinline__ bool on(int m) const { return pixel(m) < n2; }
  __device__ __forceinline__ int channel(int t) const { return t * 16 + fg * 4; }
  __device__ __forceinline__ void put(int m, int t, uint2 q) const {
    *reinterpret_cast<uint2*>(&in[(on(m) ? base[m] : spare) + channel(t)]) = q;  // (no branch: a store each)
  }
  // the tile's lines to rows of `ld` elements (the tile's first pixel at dst), the first `cols` channels
  __device__ __forceinline__ void store(uint16_t* dst, int ld, int cols) const {
    const auto win = pair_window(dst, n2 * ld);
    const int me0 = me();
#pragma unroll
    for (int i = 0; i < (64 * MT * C8 + NT - 1) / NT; ++i) {
      const int id = me0 + NT * i, px = id / C8, c = id % C8 * 8, pc = px < n2 ? px : 0, l = line_of(pc);
      const u16x8 q = *reinterpret_cast<const u16x8*>(&in[((l + 1) * LW + pc - l * W + 1) * PITCH + c]);
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4p, q), win, c < cols ? (px * ld + c) * 2 : 0x40000000, 0, 0);
    }
  }
  __device__ __forceinline__ void publish() const {
    unsigned long long* set = mine + (tag & 1) * (pitch / 2);
    const int side_words = pitch / 4;
    for (int id = me(); id < 2 * W * C8; id += NT) {
      const int side = id >= W * C8, c = id - side * W * C8;
      if (side ? !down : !up) continue;
      const uint4 q = *reinterpret_cast<const uint4*>(&in[((side ? rows : 1) * LW + c / C8 + 1) * PITCH + c % C8 * 8]);
      unsigned long long* w = set + side * side_words + c;
      const unsigned long long t = (unsigned long long)tag << 32;
      __hip_atomic_store(w, t | q.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(w + W * C8, t | q.y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(w + 2 * W * C8, t | q.z, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(w + 3 * W * C8, t | q.w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  // the neighbours' lines; false: a wait of this thread ran out
  __device__ __forceinline__ bool collect() const {
    const int side_words = pitch / 4, chunks = W * C8, me0 = me();
    bool late = tag == g.give_up_at;
    unsigned long long t0 = 0, v[2][4];
    for (int first = 0; first < 2 * chunks; first += 2 * NT) {
      const unsigned long long* w[2];
      bool want[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int id = first + i * NT + me0, side = id >= chunks;
        want[i] = id < 2 * chunks && (side ? down : up);
        // (above: the last line of the workgroup before, below: the first of the one behind)
        w[i] = want[i] ? (side ? mine + pitch : mine - pitch + side_words) + (tag & 1) * (pitch / 2) + (id - side * chunks) : mine;
      }
      for (;;) {
        bool there = true;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int k = 0; k < 4; ++k) v[i][k] = __hip_atomic_load(w[i] + k * chunks, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int k = 0; k < 4; ++k) there &= !want[i] | ((uint32_t)(v[i][k] >> 32) == tag);
        if (there || late) break;
        if (t0 == 0) t0 = wall_clock64();
        late = wall_clock64() - t0 >= kPassWaitTicks;
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int id = first + i * NT + me0, side = id >= chunks, c = id - side * chunks;
        if (want[i])
          *reinterpret_cast<uint4*>(&in[((side ? rows + 1 : 0) * LW + c / C8 + 1) * PITCH + c % C8 * 8]) =
              make_uint4((uint32_t)v[i][0], (uint32_t)v[i][1], (uint32_t)v[i][2], (uint32_t)v[i][3]);
      }
    }
    return !late;
  }
  // One convolution of the lines in LDS (written by all threads; `w` has been started): `kept` runs behind the barrier in
  // front of it, `between` before the last line of taps.  Ends behind a barrier; false (for all threads): a wait ran out.
  template <class Kept, class Between>
  __device__ __forceinline__ bool convolve(Gemm& w, f32x4 (&acc)[MT][NCT], const Kept& kept, const Between& between) {
    __syncthreads();
    if (up || down) publish();
    kept();
    int b[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) b[m] = base[m] + fg * 8 - PITCH;
    u16x8 fb[Gemm::FR][MT];
    w.load_b(in, b, 0, fb[0]);
    w.template line<false, false>(in, b, 0, fb, acc);
    bool ok = true;
    if (up || down) {
      ok = collect();
      ++tag;
      __syncthreads();
    }
#pragma unroll
    for (int m = 0; m < MT; ++m) b[m] -= LW * PITCH;
    w.load_b(in, b, 0, fb[0]);
    w.template line<true, false>(in, b, 2 * LW * PITCH, fb, acc);
    between();
    __builtin_amdgcn_sched_barrier(0);
    w.template line<false, true>(in, b, 0, fb, acc);
    return __syncthreads_or(ok ? 0 : 1) == 0;  // (and the lines have been read)
  }
  __device__ __forceinline__ void time_terms(PairTime<T, NCT>& time, uint32_t tau, f32x4 (&acc)[MT][NCT]) const {
    unsigned e = edges;
    asm volatile("" : "+v"(e));  // (see me())
#pragma unroll
    for (int m = 0; m < MT; ++m) time.run(tau, e >> (4 * m), acc[m]);
  }
  __device__ __forceinline__ void tanh_to_lds(f32x4 (&acc)[MT][NCT]) const {
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int t = 0; t < NCT; ++t) {
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = tanh_fast(acc[m][t][r]);
        put(m, t, pack4<T>(v));
      }
  }
  // whether the launch goes on (uniform)
  __device__ __forceinline__ bool alive() const {
    const int lost = tid == 0 ? __hip_atomic_load(g.stalled, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    return __syncthreads_or(lost) == 0;
  }
  __device__ __forceinline__ void give_up() const {
    if (tid != 0) return;
    __hip_atomic_store(g.stalled, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (g.detect) {  // (poison: every later kernel of the pass does nothing)
      __hip_atomic_store(&g.ctl->stalled, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&g.ctl->poison, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  __device__ __forceinline__ int64_t row0(int img) const { return ((int64_t)img * g.H + y0) * W; }
};

// Both convolutions of a stage whose input is in LDS; false: a wait ran out.  keep_z / keep_act store what the backward
// pass reads; last: the hidden activation alone.  acc: the slope.
template <class T, int C32, int MT, class KeepZ, class KeepAct>
__device__ __forceinline__ bool pass_stage(PassTile<T, C32, MT>& t, uint32_t tau, bool last, f32x4 (&acc)[MT][2 * C32],
                                           const KeepZ& keep_z, const KeepAct& keep_act) {
  typename PassTile<T, C32, MT>::Gemm w;
  PairTime<T, 2 * C32> time;
  w.start(t.g.W1);
  time.start(t.g.T1);
  t.time_terms(time, tau, acc);
  if (!t.convolve(w, acc, keep_z, []() {})) return false;
  if (!last) w.start(t.g.W2);
  t.tanh_to_lds(acc);
  if (last) {
    __syncthreads();
    keep_act();
    return true;
  }
  time.start(t.g.T2);
  t.time_terms(time, tau, acc);
  return t.convolve(w, acc, keep_act, []() {});
}

// a packed value that stays packed over a loop (its unpacked form is twice the registers)
__device__ __forceinline__ uint2 packed(uint2 q) {
  asm volatile("" : "+v"(q.x), "+v"(q.y));
  return q;
}
template <class T>
__device__ __forceinline__ uint32_t low_bits(float x) { return Low<T>::from_f32(x); }

// ---- the forward pass (Alg. 1)
template <class T, int C32, int MT>
__global__ __launch_bounds__(256, MT <= 4 ? 2 : 1) void conv_pass_forward(ConvPass g, PassShape sh) {
  constexpr int NCT = 2 * C32;
  extern __shared__ __attribute__((aligned(16))) uint16_t pass_smem[];
  PassTile<T, C32, MT> t(g, sh, pass_smem);
  const int HW = g.H * g.Wd;
  for (int img = blockIdx.x / sh.per_image; img < g.images; img += sh.slots) {
    if (!t.alive()) return;
    const int64_t r0 = t.row0(img);
    const auto y = pair_window(g.y + r0 * g.d, t.n2 * g.d);
    f32x4 sum[MT][NCT];
    if (g.step == 0) {
      const auto y0 = pair_window(g.y0 + (size_t)img * g.d * HW, g.d * HW);
      const int v0 = t.me(), p0 = t.wave * MT * 16 + (v0 & 15), n0 = (v0 >> 4 & 3) * 4;
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int c = 0; c < NCT; ++c) {
          float v[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int n = n0 + 16 * c + r;
            v[r] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(y0, n < g.d && t.on(m) ? (n * HW + t.y0 * g.Wd + p0 + 16 * m) * 4 : 0x40000000, 0, 0));
          }
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4p, make_float4(v[0], v[1], v[2], v[3])), y,
                                                 n0 + 16 * c < g.d ? ((p0 + 16 * m) * g.d + n0 + 16 * c) * 4 : 0x40000000, 0, 0);
          t.put(m, c, pack4<T>(v));
        }
    } else {  // (the state of an earlier launch)
      t.for_each(g.d, 4, [&](int m, int c, int o) __attribute__((always_inline)) {
        sum[m][c] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(y, o, 0, 0));
      });
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int c = 0; c < NCT; ++c) {
          const float v[4] = {sum[m][c][0], sum[m][c][1], sum[m][c][2], sum[m][c][3]};
          t.put(m, c, pack4<T>(v));
        }
    }
    for (int i = g.step; i < g.step + g.nsteps; ++i) {
      const float* tab = g.steptab + (size_t)i * (1 + g.s);
      const float h = tab[0];
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int c = 0; c < NCT; ++c) sum[m][c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
      for (int j = 0; j < g.s; ++j) {
        f32x4 acc[MT][NCT];
        if (!pass_stage(t, low_bits<T>(tab[1 + j]), false, acc, [&]() __attribute__((always_inline)) {
              if (j == 0) t.store(g.ckpt + (size_t)i * g.n + r0 * g.d, g.d, g.d);
            }, []() {})) {
          t.give_up();
          return;
        }
        const float b = g.b[j], coef = g.sub[j];
        const bool more = j + 1 < g.s;
        // (the stored state comes back from memory: it does not fit in registers beside the sums)
        uint2 yh[MT][NCT];
        const auto state = pair_window(g.ckpt + (size_t)i * g.n + r0 * g.d, t.n2 * g.d);
        t.for_each(g.d, 2, [&](int m, int c, int o) __attribute__((always_inline)) {
          yh[m][c] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(state, o, 0, 0));
        });
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
          for (int c = 0; c < NCT; ++c) {
            const float v[4] = {acc[m][c][0], acc[m][c][1], acc[m][c][2], acc[m][c][3]};
            float k[4], x[4];
            unpack4<T>(pack4<T>(v), k);
            unpack4<T>(yh[m][c], x);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              sum[m][c][r] = fmaf(b, k[r], sum[m][c][r]);
              x[r] = fmaf(h, coef * k[r], x[r]);
            }
            if (more) t.put(m, c, pack4<T>(x));
          }
      }
      // y <- y + h sum, the next step's state
      f32x4 v[MT][NCT];
      t.for_each(g.d, 4, [&](int m, int c, int o) __attribute__((always_inline)) {
        v[m][c] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(y, o, 0, 0));
      });
      t.for_each(g.d, 4, [&](int m, int c, int o) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 4; ++r) v[m][c][r] = fmaf(h, sum[m][c][r], v[m][c][r]);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4p, v[m][c]), y, o, 0, 0);
        const float x[4] = {v[m][c][0], v[m][c][1], v[m][c][2], v[m][c][3]};
        t.put(m, c, pack4<T>(x));
      });
      if (i + 1 == g.N) {
        const auto yN = pair_window(g.yN + (size_t)img * g.d * HW, g.d * HW);
        const int v0 = t.me(), p0 = t.wave * MT * 16 + (v0 & 15), n0 = (v0 >> 4 & 3) * 4;
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
          for (int c = 0; c < NCT; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int n = n0 + 16 * c + r;
              __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, (float)v[m][c][r]), yN,
                                                    n < g.d && t.on(m) ? (n * HW + t.y0 * g.Wd + p0 + 16 * m) * 4 : 0x40000000, 0, 0);
            }
      }
    }
    __syncthreads();
    if (g.step + g.nsteps == g.N) t.store(g.ckpt + (size_t)g.N * g.n + r0 * g.d, g.d, g.d);
    __syncthreads();  // (the next image's state goes where this one is being read)
  }
}

// ---- stage inputs and hidden activations of the steps step, step - 1, ... from the stored states
template <class T, int C32, int MT>
__global__ __launch_bounds__(256, MT <= 4 ? 2 : 1) void conv_pass_recompute(ConvPass g, PassShape sh) {
  constexpr int NCT = 2 * C32;
  if (g.ctl->poison) return;
  extern __shared__ __attribute__((aligned(16))) uint16_t pass_smem[];
  PassTile<T, C32, MT> t(g, sh, pass_smem);
  for (int item = blockIdx.x / sh.per_image; item < g.images * g.nsteps; item += sh.slots) {
    if (!t.alive()) return;
    const int q = item / g.images, img = item - q * g.images;
    const float* tab = g.steptab + (size_t)(g.step - q) * (1 + g.s);
    const float h = tab[0];
    const int64_t r0 = t.row0(img);
    const uint16_t* ck = g.ckpt + (size_t)(g.step - q) * g.n + r0 * g.d;
    const size_t set = (size_t)(g.set0 + q) * g.s * g.stage_stride + r0 * 64;
    uint2 yh[MT][NCT];
    const auto state = pair_window(ck, t.n2 * g.d);
    auto load_state = [&]() __attribute__((always_inline)) {
      t.for_each(g.d, 2, [&](int m, int c, int o) __attribute__((always_inline)) {
        yh[m][c] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(state, o, 0, 0));
      });
    };
    load_state();
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int c = 0; c < NCT; ++c) t.put(m, c, yh[m][c]);
#pragma unroll 1
    for (int j = 0; j < g.s; ++j) {
      f32x4 acc[MT][NCT];
      const bool last = j + 1 == g.s;
      const size_t at = set + j * g.stage_stride;
      if (!pass_stage(t, low_bits<T>(tab[1 + j]), last, acc, [&]() __attribute__((always_inline)) { t.store(g.Z + at, 64, 64); },
                      [&]() __attribute__((always_inline)) { t.store(g.ACT + at, 64, 64); })) {
        t.give_up();
        return;
      }
      if (last) break;
      const float coef = g.sub[j];
      load_state();
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int c = 0; c < NCT; ++c) {
          const float v[4] = {acc[m][c][0], acc[m][c][1], acc[m][c][2], acc[m][c][3]};
          float k[4], x[4];
          unpack4<T>(pack4<T>(v), k);
          unpack4<T>(yh[m][c], x);
#pragma unroll
          for (int r = 0; r < 4; ++r) x[r] = fmaf(h, coef * k[r], x[r]);
          t.put(m, c, pack4<T>(x));
        }
    }
    __syncthreads();  // (the next item's state goes where this one's activation is being read)
  }
}

// ---- cotangent chains of the steps step, step - 1, ... and the adjoint behind them (Alg. 2 without its decisions: under
// overflow detection a launch is one step, and pass_decide follows it)
template <class T, int C32, int MT>
__global__ __launch_bounds__(256, MT <= 4 ? 2 : 1) void conv_pass_chain(ConvPass g, PassShape sh) {
  constexpr int NCT = 2 * C32;
  if (g.ctl->poison) return;
  extern __shared__ __attribute__((aligned(16))) uint16_t pass_smem[];
  __shared__ unsigned wave_max[4];
  PassTile<T, C32, MT> t(g, sh, pass_smem);
  const float S = g.ctl->S;
  uint32_t bad = 0u;
  unsigned bits = 0;
  auto watch = [&](uint2 q) __attribute__((always_inline)) { bad |= Low<T>::nonfinite2(q.x) | Low<T>::nonfinite2(q.y); };
  for (int img = blockIdx.x / sh.per_image; img < g.images; img += sh.slots) {
    if (!t.alive()) return;
    const int64_t r0 = t.row0(img);
    for (int q = 0; q < g.nsteps; ++q) {
      const float h = g.steptab[(size_t)(g.step - q) * (1 + g.s)];
      const float* a = (q == 0 ? g.a_in : g.a_out) + r0 * g.d;
      const size_t set = (size_t)(g.set0 + q) * g.s * g.stage_stride + r0 * 64;
      uint2 lam[MT][NCT];
      f32x4 sum[MT][NCT];
      {
        const auto adj = pair_window(a, t.n2 * g.d);
        t.for_each(g.d, 4, [&](int m, int c, int o) __attribute__((always_inline)) {
          sum[m][c] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(adj, o, 0, 0));
        });
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
          for (int c = 0; c < NCT; ++c) {
            float v[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = S * sum[m][c][r];
            lam[m][c] = pack4<T>(v);
            watch(lam[m][c]);
            unpack4<T>(lam[m][c], v);
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = g.b[g.s - 1] * v[r];
            const uint2 kq = pack4<T>(v);
            watch(kq);
            t.put(m, c, kq);
            sum[m][c] = f32x4{0.f, 0.f, 0.f, 0.f};
          }
      }
#pragma unroll 1
      for (int j = g.s - 1; j >= 0; --j) {
        const size_t at = set + j * g.stage_stride;
        f32x4 acc[MT][NCT];
        uint2 dv[MT][NCT];
        typename PassTile<T, C32, MT>::Gemm w;
        auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
          for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int c = 0; c < NCT; ++c) acc[m][c] = f32x4{0.f, 0.f, 0.f, 0.f};
        };
        w.start(g.W1);
        clear();
        bool ok = t.convolve(w, acc, [&]() __attribute__((always_inline)) { t.store(g.KBAR + at, 64, 64); },
                             []() {});
        if (ok) {
          const auto act = pair_window(g.ACT + at, t.n2 * 64);
          const int o = t.place(64) * 2;
#pragma unroll
          for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int c = 0; c < NCT; ++c)
              dv[m][c] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(act, o + m * 2048 + c * 32, 0, 0));
          w.start(g.W2);
#pragma unroll
          for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int c = 0; c < NCT; ++c) {
              float v[4], f[4];
              unpack4<T>(dv[m][c], f);
#pragma unroll
              for (int r = 0; r < 4; ++r) v[r] = acc[m][c][r] * (1.f - f[r] * f[r]);
              const uint2 dq = pack4<T>(v);
              if (t.on(m)) watch(dq);
              t.put(m, c, dq);
            }
          clear();
          ok = t.convolve(w, acc, [&]() __attribute__((always_inline)) { t.store(g.DELTA + at, 64, 64); }, []() {});
        }
        if (!ok) {
          t.give_up();
          return;
        }
        const float coef = j > 0 ? g.sub[j - 1] : 0.f, bw = j > 0 ? g.b[j - 1] : 0.f;
        const int first = (t.me() >> 4 & 3) * 4;  // this lane's first channel
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
          for (int c = 0; c < NCT; ++c) {
            const float v[4] = {acc[m][c][0], acc[m][c][1], acc[m][c][2], acc[m][c][3]};
            const uint2 zq = pack4<T>(v);
            float f[4], l[4], x[4];
            unpack4<T>(zq, f);
            unpack4<T>(packed(lam[m][c]), l);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              sum[m][c][r] += f[r];
              x[r] = fmaf(h, coef * f[r], bw * l[r]);
            }
            uint2 kq = pack4<T>(x);
            if (first + 16 * c >= g.d) kq = make_uint2(0u, 0u);  // (an infinite slope cotangent times the zero weights of pad channels: NaN)
            if (t.on(m)) {
              watch(zq);
              if (j > 0) watch(kq);
            }
            if (j > 0) t.put(m, c, kq);
          }
      }
      const float hs = h / S;
      const auto adj = pair_window(a, t.n2 * g.d), next = pair_window(g.a_out + r0 * g.d, t.n2 * g.d),
                 cost = pair_window(g.gys + (g.gys ? r0 * g.d : 0), g.gys ? t.n2 * g.d : 0);
      f32x4 v[MT][NCT];
      t.for_each(g.d, 4, [&](int m, int c, int o) __attribute__((always_inline)) {
        v[m][c] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(adj, o, 0, 0));
      });
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int c = 0; c < NCT; ++c)
#pragma unroll
          for (int r = 0; r < 4; ++r) v[m][c][r] = fmaf(hs, t.on(m) ? sum[m][c][r] : 0.f, v[m][c][r]);
      if (g.gys)
        t.for_each(g.d, 4, [&](int m, int c, int o) __attribute__((always_inline)) {
          v[m][c] += __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(cost, o, 0, 0));
        });
      t.for_each(g.d, 4, [&](int m, int c, int o) __attribute__((always_inline)) {
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4p, v[m][c]), next, o, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) bits = max(bits, __builtin_bit_cast(unsigned, fabsf(v[m][c][r])));
      });
    }
    __syncthreads();  // (the next image's cotangent goes where this one's is being read)
  }
  if (!g.detect) return;
  raise_if_any((bad & kNonfiniteBits) != 0u, g.ctl);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) bits = max(bits, (unsigned)__shfl_xor((int)bits, o));
  if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = bits;
  __syncthreads();
  if (threadIdx.x == 0) g.amax[blockIdx.x] = max(max(wave_max[0], wave_max[1]), max(wave_max[2], wave_max[3]));
}

// ---- a launch that was given up, again: one workgroup per image, tile after tile through memory
template <class T, int C32>
__device__ __forceinline__ void redo_tiles(const ConvPair& p, const ConvPairShape& sh, int img, bool vjp, uint16_t* lds) {
  for (int tile = 0; tile < sh.per_image; ++tile) {
    __syncthreads();  // (the tile before has been read; what the stage before wrote is there)
    if (vjp) pair_tile<T, C32, 3, 2, true>(p, sh, img * sh.per_image + tile, lds);
    else pair_tile<T, C32, 3, 2, false>(p, sh, img * sh.per_image + tile, lds);
  }
  __threadfence();
  __syncthreads();
}
struct ConvRedo {
  ConvPass g;
  ConvPairShape sh;                // tiles of one line
  const uint16_t *V1, *V2;         // backward: the transposed fragments W_2^T, W_1^T (g.W1, g.W2: the forward ones)
  uint16_t *Z2, *K, *ZBAR;         // [rows][64]: a second stage input (forward); slopes and cotangents of a step's stages
  int* redone;
};

template <class T, int C32>
__global__ __launch_bounds__(256, 1) void conv_redo_forward(ConvRedo a) {
  const ConvPass& g = a.g;
  if (!*g.stalled) return;
  if (blockIdx.x == 0 && threadIdx.x == 0) ++*a.redone;
  extern __shared__ __attribute__((aligned(16))) uint16_t pass_smem[];
  const int HW = g.H * g.Wd;
  for (int img = blockIdx.x; img < g.images; img += gridDim.x) {
    const size_t r0 = (size_t)img * HW;
    for (int e = threadIdx.x; e < HW * 64; e += 256) {
      const int p = e / 64, c = e % 64;
      const float v = c < g.d ? g.y0[((size_t)img * g.d + c) * HW + p] : 0.f;
      const uint16_t q = Low<T>::from_f32(v);
      if (c < g.d) {
        g.y[(r0 + p) * g.d + c] = v;
        g.ckpt[(r0 + p) * g.d + c] = q;
      }
      g.Z[(r0 + p) * 64 + c] = q;
    }
    __threadfence();
    for (int i = 0; i < g.N; ++i) {
      const float* tab = g.steptab + (size_t)i * (1 + g.s);
      for (int j = 0; j < g.s; ++j) {
        ConvPair p{};
        p.A = j % 2 ? a.Z2 : g.Z;
        p.W1 = g.W1; p.W2 = g.W2; p.T1 = g.T1; p.T2 = g.T2;
        p.X1 = g.X1; p.X2 = g.X2; p.F1 = g.F1; p.F2 = g.F2;
        p.tau = low_bits<T>(tab[1 + j]);
        p.C = a.K + (size_t)j * g.stage_stride;
        if (j + 1 < g.s) {
          p.next = j % 2 ? g.Z : a.Z2;
          p.base = g.ckpt + (size_t)i * g.n;
          p.d = g.d; p.h = tab[0]; p.coef = g.sub[j];
        }
        p.H = g.H; p.Wd = g.Wd;
        redo_tiles<T, C32>(p, a.sh, img, false, pass_smem);
      }
      for (int e = threadIdx.x; e < HW * g.d; e += 256) {
        const int p = e / g.d, c = e - p * g.d;
        float sum = 0.f;
        for (int j = 0; j < g.s; ++j) sum = fmaf(g.b[j], Low<T>::to_f32(a.K[(size_t)j * g.stage_stride + (r0 + p) * 64 + c]), sum);
        const float v = fmaf(tab[0], sum, g.y[(r0 + p) * g.d + c]);
        const uint16_t q = Low<T>::from_f32(v);
        g.y[(r0 + p) * g.d + c] = v;
        g.ckpt[(size_t)(i + 1) * g.n + (r0 + p) * g.d + c] = q;
        g.Z[(r0 + p) * 64 + c] = q;
        if (i + 1 == g.N) g.yN[((size_t)img * g.d + c) * HW + p] = v;
      }
      __threadfence();
    }
  }
}

template <class T, int C32>
__global__ __launch_bounds__(256, 1) void conv_redo_backward(ConvRedo a) {
  const ConvPass& g = a.g;
  if (!*g.stalled) return;
  if (blockIdx.x == 0 && threadIdx.x == 0) ++*a.redone;
  extern __shared__ __attribute__((aligned(16))) uint16_t pass_smem[];
  const int HW = g.H * g.Wd;
  const float S = g.ctl->S;
  for (int img = blockIdx.x; img < g.images; img += gridDim.x) {
    const size_t r0 = (size_t)img * HW;
    for (int q = 0; q < g.nsteps; ++q) {
      const int step = g.step - q;
      const float* tab = g.steptab + (size_t)step * (1 + g.s);
      const size_t set = (size_t)(g.set0 + q) * g.s * g.stage_stride;
      const float* adj = q == 0 ? g.a_in : g.a_out;
      for (int e = threadIdx.x; e < HW * 64; e += 256) {
        const int p = e / 64, c = e % 64;
        uint16_t z = 0, k = 0;
        if (c < g.d) {
          z = g.ckpt[(size_t)step * g.n + (r0 + p) * g.d + c];
          k = Low<T>::from_f32(g.b[g.s - 1] * Low<T>::to_f32(Low<T>::from_f32(S * adj[(r0 + p) * g.d + c])));
        }
        g.Z[set + (r0 + p) * 64 + c] = z;
        g.KBAR[set + (size_t)(g.s - 1) * g.stage_stride + (r0 + p) * 64 + c] = k;
      }
      __threadfence();
      for (int j = 0; j < g.s; ++j) {
        ConvPair p{};
        p.A = g.Z + set + (size_t)j * g.stage_stride;
        p.W1 = g.W1; p.W2 = g.W2; p.T1 = g.T1; p.T2 = g.T2;
        p.X1 = g.X1; p.X2 = g.X2; p.F1 = g.F1; p.F2 = g.F2;
        p.tau = low_bits<T>(tab[1 + j]);
        p.mid = g.ACT + set + (size_t)j * g.stage_stride;
        if (j + 1 < g.s) {
          p.C = a.K;
          p.next = g.Z + set + (size_t)(j + 1) * g.stage_stride;
          p.base = g.ckpt + (size_t)step * g.n;
          p.d = g.d; p.h = tab[0]; p.coef = g.sub[j];
        }
        p.H = g.H; p.Wd = g.Wd;
        redo_tiles<T, C32>(p, a.sh, img, false, pass_smem);
      }
      for (int j = g.s - 1; j >= 0; --j) {
        ConvPair p{};
        p.A = g.KBAR + set + (size_t)j * g.stage_stride;
        p.W1 = a.V1; p.W2 = a.V2;
        p.act = g.ACT + set + (size_t)j * g.stage_stride;
        p.mid = g.DELTA + set + (size_t)j * g.stage_stride;
        p.C = a.ZBAR + (size_t)j * g.stage_stride;
        if (j > 0) {
          p.next = g.KBAR + set + (size_t)(j - 1) * g.stage_stride;
          p.adj = adj;
          p.d = g.d; p.h = tab[0]; p.coef = g.sub[j - 1]; p.bw = g.b[j - 1];
        }
        p.ctl = g.ctl;
        p.H = g.H; p.Wd = g.Wd;
        redo_tiles<T, C32>(p, a.sh, img, true, pass_smem);
      }
      for (int e = threadIdx.x; e < HW * g.d; e += 256) {
        const int p = e / g.d, c = e - p * g.d;
        float sum = 0.f;
        for (int j = g.s - 1; j >= 0; --j) sum += Low<T>::to_f32(a.ZBAR[(size_t)j * g.stage_stride + (r0 + p) * 64 + c]);
        float v = fmaf(tab[0] / S, sum, adj[(r0 + p) * g.d + c]);
        if (g.gys) v += g.gys[(r0 + p) * g.d + c];
        g.a_out[(r0 + p) * g.d + c] = v;
      }
      __threadfence();
      __syncthreads();
    }
  }
}

// In front of a pass: no exchange has taken place, nothing is given up (`stalled`: `flags` of them) unless the kernels cannot
// do the work (F1, F2: see ConvPair), and the head of the step table.
__global__ __launch_bounds__(256) inline void pass_reset(uint4* words, size_t n, int* stalled, int flags, const float* F1, const float* F2, Ctl* ctl,
                                                         int detect, FloatChunk c, float* table, int count) {
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i < count; i += 256) table[i] = c.v[i];
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) words[i] = make_uint4(0u, 0u, 0u, 0u);
  if (blockIdx.x != 0 || threadIdx.x >= 64) return;
  const bool odd = __builtin_amdgcn_ballot_w64(F1[threadIdx.x] + F2[threadIdx.x] != 0.f) != 0;
  for (int i = threadIdx.x; i < flags; i += 64) stalled[i] = odd;
  if (threadIdx.x != 0) return;
  ctl->redone = 0;
  if (odd && detect) ctl->stalled = ctl->poison = 1;
}

// Behind the chain of a step under overflow detection: accept or reject it, the scale of the next (Alg. 2).  256 threads.
__global__ __launch_bounds__(256) inline void pass_decide(Ctl* ctl, float* scale_hist, int step, int p_bits, int dynamic, int raw_norm,
                                                          const unsigned* __restrict__ slots, int nslots) {
  if (ctl->poison) return;
  __shared__ unsigned wave_max[4];
  unsigned bits = 0;
  for (int i = threadIdx.x; i < nslots; i += 256) bits = max(bits, slots[i]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) bits = max(bits, (unsigned)__shfl_xor((int)bits, o));
  if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = bits;
  __syncthreads();
  if (threadIdx.x != 0) return;
  if (ctl->nonfinite) {
    ctl->poison = 1;
    ctl->failed_step = step;
    return;
  }
  const float S = ctl->S, amax = __builtin_bit_cast(float, max(max(wave_max[0], wave_max[1]), max(wave_max[2], wave_max[3])));
  ctl->S_step = S;
  scale_hist[step] = S;
  ctl->s_min = fminf(ctl->s_min, S);
  ctl->s_max = fmaxf(ctl->s_max, S);
  if (dynamic && ctl->attempt == 1) {
    const float test = raw_norm ? amax : S * amax;
    if (test <= ldexpf(1.f, p_bits - 1) && S < ldexpf(1.f, 126)) ctl->S = 2.f * S;
  }
  ctl->attempt = 1;
}

}  // namespace rampde
