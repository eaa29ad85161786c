// Row-tile kernels for dense networks with ONE hidden layer: the velocity of a normalising flow with its exact trace row,
// dl/dt = -sum_h c_h (1 - a_h^2) (paper Sec. 6.1; TRACE), up to 64 state columns and 1024 hidden units, and plain networks
// (the same, or up to 128 state columns and 512 hidden units).
//
// Every wavefront owns a slice of the hidden layer and keeps the slices of both weight matrices in registers.  With the
// weight fragment as first operand a lane ends a 16 x 16 tile with 4 consecutive hidden columns of one row; two tiles
// are 8 values of that row, which is exactly a lane's part of the second operand of a 32-deep contraction -- over the
// hidden columns in the order (16 p + 4 q + 0..3, 16 (p + 1) + 4 q + 0..3), so the second matrix's fragments are laid
// out in that order (CastLayer.perm_f, perm_t) and the activation never leaves the registers.  What the wavefronts
// exchange is the sum of their contributions to the 64 state columns: fp32 through LDS, added in wavefront order.
//
// Bound: tanh (and the trace's two multiply-adds) on 16 rows x 1024 columns per compute unit, 1.3 us per evaluation,
// plus the exchange; a tile per 16 rows, so 512 rows occupy 32 compute units.  At 1024 columns the forward and the
// transposed slices (128 registers each) do not fit together, and in one kernel the recomputation and the cotangent
// chain of a step load their own (2 x 256 KB from L2 per step).  So a group of steps runs in two launches as in
// resident.hpp, scale exchange included: all stages side by side, then the chain; the one-launch kernel is left to
// single steps and to tiles of narrow networks that fill the device.  Measured on flows of 63 features, width 1024,
// fp16, 16 RK4 steps of 512 rows: 793 -> 584 us per pass; one launch per layer, 900 launches, 6456 to 6514 us.
#pragma once
#include "resident.hpp"

namespace rampde {

template <int NTL, int HP>
struct ShallowShape {
  static constexpr int NW = HP <= 128 ? 4 : 8;      // wavefronts
  static constexpr int NT = 64 * NW;
  static constexpr int TPW = HP / 16 / NW;          // hidden column tiles of a wavefront (even)
  static constexpr int KP = TPW / 2;                // k-blocks of 32 of its part of the contraction over the hidden layer
  static constexpr int KS = 2 * NTL;                // k-blocks of a contraction over the state
  static constexpr int NS = 4 * NTL;                // state column tiles
  static constexpr int EPT = 16 * 64 * NTL / NT;    // state elements of a thread: row tid / (NT / 16), consecutive columns
  static constexpr int LDZ = 64 * NTL + 8;          // 16-bit elements
  static constexpr int LDS_ = 64 * NTL + 4;         // floats
  static constexpr bool ACT_LDS = HP <= 512;        // activations of a step kept in LDS for the tanh' factors
  static constexpr bool PHASED = TPW * KS + NS * KP > 24;
};

struct ShallowLds {
  lds_f32 *b1, *wt, *cf, *b2, *coef, *rows, *part, *tr;
  lds_u16 *z, *act;
  template <int NTL, int HP>
  static constexpr size_t bytes(bool adjoint, int s) {
    using Sh = ShallowShape<NTL, HP>;
    return 4 * (size_t)(3 * HP + 64 * NTL + 32 + Sh::NW * 16 * (Sh::LDS_ + 1)) + 2 * (size_t)16 * Sh::LDZ +
           (adjoint && Sh::ACT_LDS ? 2 * (size_t)s * 16 * (HP + 8) : 0);
  }
  template <int NTL, int HP>
  __device__ __forceinline__ void carve(lds_u16* smem) {
    using Sh = ShallowShape<NTL, HP>;
    b1 = (lds_f32*)smem;
    wt = b1 + HP;
    cf = wt + HP;
    b2 = cf + HP;
    coef = b2 + 64 * NTL;
    rows = coef + 16;
    part = rows + 16;
    tr = part + Sh::NW * 16 * Sh::LDS_;
    z = (lds_u16*)(tr + Sh::NW * 16);
    act = z + 16 * Sh::LDZ;
  }
};

struct ShallowArgs {
  ResidentArgs r;
  const float* trace_c;  // [HP] c_h (TRACE)
};

// N state elements c..c+N-1 of row `row` (columns >= d and rows >= R: zero / not written)
template <int N>
__device__ __forceinline__ void load_elems(const float* p, int64_t row, int64_t R, int c, int d, float (&v)[N]) {
#pragma unroll
  for (int e = 0; e < N; ++e) v[e] = 0.f;
  if (row >= R) return;
#pragma unroll
  for (int e = 0; e < N; ++e)
    if (c + e < d) v[e] = p[(size_t)row * d + c + e];
}
template <int N>
__device__ __forceinline__ void store_elems(float* p, int64_t row, int64_t R, int c, int d, const float (&v)[N]) {
  if (row >= R) return;
#pragma unroll
  for (int e = 0; e < N; ++e)
    if (c + e < d) p[(size_t)row * d + c + e] = v[e];
}
template <int N>
__device__ __forceinline__ void store_elems(uint16_t* p, int64_t row, int64_t R, int c, int d, const uint16_t (&v)[N]) {
  if (row >= R) return;
#pragma unroll
  for (int e = 0; e < N; ++e)
    if (c + e < d) p[(size_t)row * d + c + e] = v[e];
}
// ... branch-free (clamped addresses): requested at the head of a stage's body, see StepRows
template <int N>
__device__ __forceinline__ void load_elems_clamped(const uint16_t* p, int64_t row, int64_t R, int c, int d, uint16_t (&v)[N]) {
  const int64_t r = row < R ? row : R - 1;
#pragma unroll
  for (int e = 0; e < N; ++e) {
    const uint16_t x = p[(size_t)r * d + min(c + e, d - 1)];
    v[e] = (row < R && c + e < d) ? x : (uint16_t)0;
  }
}
template <int N>
__device__ __forceinline__ void put_z(lds_u16* z, const uint16_t (&v)[N]) {
#pragma unroll
  for (int e = 0; e < N; e += 2) *(RAMPDE_LDS uint32_t*)(z + e) = (uint32_t)v[e] | ((uint32_t)v[e + 1] << 16);
}

template <class T, int NTL, int HP>
struct ShallowTile {
  using Sh = ShallowShape<NTL, HP>;
  // W[t][kb]: state -> own hidden tiles; V[n][p]: own hidden columns -> state tiles
  struct Weights {
    u16x8 W[Sh::TPW][Sh::KS];
    u16x8 V[Sh::NS][Sh::KP];
    template <bool AGAIN>
    __device__ __forceinline__ void load(const u16x8* wf, const u16x8* vf, int wave, int lane) {
      if constexpr (AGAIN) asm volatile("" : "+v"(lane));  // (see ResidentWeights)
      const glb_u16x8* w = (const glb_u16x8*)wf + lane;
      const glb_u16x8* v = (const glb_u16x8*)vf + lane;
#pragma unroll
      for (int t = 0; t < Sh::TPW; ++t)
#pragma unroll
        for (int kb = 0; kb < Sh::KS; ++kb) W[t][kb] = w[(size_t)(kb * (HP / 16) + wave * Sh::TPW + t) * 64];
#pragma unroll
      for (int n = 0; n < Sh::NS; ++n)
#pragma unroll
        for (int p = 0; p < Sh::KP; ++p) V[n][p] = v[(size_t)((wave * Sh::KP + p) * Sh::NS + n) * 64];
    }
  };
  static __device__ __forceinline__ void read_z(u16x8 (&a)[Sh::KS], const lds_u16* z, int lane) {
#pragma unroll
    for (int kb = 0; kb < Sh::KS; ++kb) a[kb] = *(const lds_u16x8*)(z + (lane & 15) * Sh::LDZ + (lane >> 4) * 8 + kb * 32);
  }
  static __device__ __forceinline__ u16x8 operand(uint2 lo, uint2 hi) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 v = {lo.x, lo.y, hi.x, hi.y};
    return __builtin_bit_cast(u16x8, v);
  }
  // this wavefront's contributions to the state columns
  template <int COPIES = 1>
  static __device__ __forceinline__ void put_part(const f32x4 (&out)[Sh::NS], const ShallowLds& l, int wave, int lane) {
    lds_f32* p = l.part + ((size_t)wave * 16 + (lane & 15) / COPIES) * Sh::LDS_ + (lane >> 4) * 4;
    if (COPIES == 1 || lane % COPIES == 0)
#pragma unroll
      for (int n = 0; n < Sh::NS; ++n) *(RAMPDE_LDS f32x4*)(p + n * 16) = out[n];
  }
  // ---- COPIES = 2, 4: tiles of 16 / COPIES rows, where those of 16 leave compute units idle.  A tile's 16 rows are copies of
  // them, in neighbouring lanes, and copy c of a row does the tanh arithmetic of a share of the hidden units: of a lane's
  // eight of a block of 32 (the four words of its operand) those of word c, or words 2c and 2c + 1.  The other words come
  // from the lanes beside it (DPP within four lanes), so that every copy has the whole operand and the sums, trace included,
  // are those of the 16-row tiles, bit for bit.  (With zeros for the other words and the copies' sums added up at the end
  // the recomputation, which has no copies, summed in another order, and an infinite output weight gave NaN.)  Forward pass,
  // up to 64 state columns and more than 256 hidden units (16 RK4 steps, us): 40 features, width 700, 64 rows, trace row 165
  // -> 135 (130 with every copy's share of the trace sum); 50 -> 1000 -> 50, 800 rows 134 -> 109; training pass of 63
  // features, width 1024, 512 rows 559 -> 527.  Not with fewer hidden units or more state columns, where a version that added
  // up the copies' sums lost (training pass, 128 -> 512 -> 128, 1024 rows 391 -> 410; flow of 8 features, width 100, 2048 rows
  // 281 -> 289; this one is not measured there), and not in the chain, where that version lost on shapes outside this range
  // (128 -> 512 -> 128, 1024 rows 410 -> 433: more tiles exchange the scale) and was not tried by itself within it.
  static constexpr int words(int COPIES) { return 4 / COPIES; }
  // this copy's of a lane's eight hidden units: pair u of words(COPIES)
  template <int COPIES>
  static __device__ __forceinline__ void own(const f32x4 (&acc)[2], int copy, int u, float (&v)[2]) {
    if constexpr (COPIES == 2) {
#pragma unroll
      for (int r = 0; r < 2; ++r) v[r] = copy ? acc[1][2 * u + r] : acc[0][2 * u + r];
    } else {
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const float lo = copy & 1 ? acc[0][2 + r] : acc[0][r], hi = copy & 1 ? acc[1][2 + r] : acc[1][r];
        v[r] = copy & 2 ? hi : lo;
      }
    }
  }
  // word K of the operand, from the copy that has it
  template <int COPIES, int K>
  static __device__ __forceinline__ uint32_t word(const uint32_t (&w)[words(COPIES)]) {
    constexpr int owner = K / words(COPIES), other = COPIES == 4 ? owner : owner + 2;  // (lanes 0, 1 and 2, 3 of four)
    return __builtin_amdgcn_update_dpp(0, (int)w[K % words(COPIES)], owner * 5 + other * 0x50, 0xf, 0xf, false);
  }
  template <int COPIES>
  static __device__ __forceinline__ void whole(const uint32_t (&w)[words(COPIES)], uint32_t (&v)[4]) {
    v[0] = word<COPIES, 0>(w);
    v[1] = word<COPIES, 1>(w);
    v[2] = word<COPIES, 2>(w);
    v[3] = word<COPIES, 3>(w);
  }
  static __device__ __forceinline__ void sum_parts(float (&v)[Sh::EPT], const ShallowLds& l, int row, int c) {
#pragma unroll
    for (int w = 0; w < Sh::NW; ++w) {
      const lds_f32* p = l.part + ((size_t)w * 16 + row) * Sh::LDS_ + c;
#pragma unroll
      for (int e = 0; e < Sh::EPT; ++e) v[e] = w == 0 ? p[e] : v[e] + p[e];
    }
  }
  static __device__ __forceinline__ void fill(const ShallowArgs& sa, const ShallowLds& l, bool trace) {
    const FusedArgs& g = sa.r.f;
    for (int i = threadIdx.x; i < HP; i += Sh::NT) {
      l.b1[i] = g.layer[0].bias[i];
      l.wt[i] = g.layer[0].wt ? g.layer[0].wt[i] : 0.f;
      l.cf[i] = trace ? sa.trace_c[i] : 0.f;
    }
    for (int i = threadIdx.x; i < 64 * NTL; i += Sh::NT) l.b2[i] = g.layer[1].bias[i];
    if (threadIdx.x < 16) {  // as in ResidentLds::fill
      const int j = threadIdx.x >> 2, e = threadIdx.x & 3;
      float c = 0.f;
      if (j < g.s) c = e == 0 ? (j + 1 < g.s ? g.A[(j + 1) * g.s + j] : 0.f) : e == 1 ? g.b[j] : 0.f;
      l.coef[threadIdx.x] = c;
    }
  }
  // pre-activations of hidden tiles 2p, 2p + 1
  static __device__ __forceinline__ void pre(f32x4 (&acc)[2], const Weights& w, const u16x8 (&a)[Sh::KS], int p) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int kb = 0; kb < Sh::KS; ++kb) acc[h] = Low<T>::mfma16(w.W[2 * p + h][kb], a[kb], acc[h]);
  }
  static __device__ __forceinline__ void start(f32x4 (&acc)[2], const ShallowLds& l, float tau, int nh, int p) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const f32x4 b = *(const RAMPDE_LDS f32x4*)(l.b1 + nh + (2 * p + h) * 16);
      const f32x4 w = *(const RAMPDE_LDS f32x4*)(l.wt + nh + (2 * p + h) * 16);
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[h][r] = fmaf(w[r], tau, b[r]);
    }
  }
  // sum of a row's trace terms over the four lanes that share it -> LDS
  template <int COPIES = 1>
  static __device__ __forceinline__ void put_trace(float tr, const ShallowLds& l, int wave, int lane) {
    tr += __shfl_xor(tr, 16);
    tr += __shfl_xor(tr, 32);
    if (lane < 16 && lane % COPIES == 0) l.tr[wave * 16 + lane / COPIES] = tr;
  }
  static __device__ __forceinline__ float trace_of(const ShallowLds& l, int row) {
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < Sh::NW; ++w) v += l.tr[w * 16 + row];
    return v;
  }
};

template <class T, int NTL, int HP, bool TRACE, int COPIES>
__global__ __launch_bounds__((ShallowShape<NTL, HP>::NT), (HP <= 128 ? 1 : 2)) void mlp_forward_shallow(ShallowArgs sa) {
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  using Sh = ShallowShape<NTL, HP>;
  using Tile = ShallowTile<T, NTL, HP>;
  constexpr int EPT = Sh::EPT;
  const FusedArgs& g = sa.r.f;
  ShallowLds l;
  l.carve<NTL, HP>((lds_u16*)smem);
  constexpr int ROWS = 16 / COPIES, WORDS = Tile::words(COPIES);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, copy = lane % COPIES;
  const int nh = wave * Sh::TPW * 16 + (lane >> 4) * 4;
  const int er = tid / (Sh::NT / 16), ec = (tid % (Sh::NT / 16)) * EPT;  // this thread's state elements
  const int64_t row = COPIES == 1 || er < ROWS ? (int64_t)blockIdx.x * ROWS + er : g.R;
  const int64_t n_state = g.R * g.d;
  const int s = g.s;
  typename Tile::Weights w;
  w.template load<false>(g.layer[0].Wf, g.layer[1].Wf, wave, lane);
  Tile::fill(sa, l, TRACE);
  const StepRows rows{l.rows};
  rows.put(0, rows.load(g, 0));
  float y[EPT], yh[EPT], bs[EPT], b2[EPT];
  uint16_t q[EPT];
  load_elems(g.y0, row, g.R, ec, g.d, y);
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    q[e] = Low<T>::from_f32(y[e]);
    yh[e] = Low<T>::to_f32(q[e]);
    if (g.round_incr & 2) y[e] = yh[e];
  }
  store_elems(g.ckpt, row, g.R, ec, g.d, q);
  put_z(l.z + er * Sh::LDZ + ec, q);
  __syncthreads();
#pragma unroll
  for (int e = 0; e < EPT; ++e) b2[e] = l.b2[ec + e];

  for (int i = 0; i < g.N; ++i) {
    const float h = rows.h(i);
    const int i_next = min(i + 1, g.N - 1);
#pragma unroll
    for (int e = 0; e < EPT; ++e) bs[e] = 0.f;
#pragma unroll 1
    for (int j = 0; j < s; ++j) {
      const bool last_stage = j + 1 == s;
      const float row_next = rows.load(g, i_next);
      const float tau = rows.tau(i, j);
      u16x8 a[Sh::KS];
      Tile::read_z(a, l.z, (lane & 0x30) | (lane & 15) / COPIES);
      f32x4 out[Sh::NS];
#pragma unroll
      for (int n = 0; n < Sh::NS; ++n) out[n] = f32x4{0.f, 0.f, 0.f, 0.f};
      float tr = 0.f;
#pragma unroll
      for (int p = 0; p < Sh::KP; ++p) {
        f32x4 acc[2];
        Tile::start(acc, l, tau, nh, p);
        Tile::pre(acc, w, a, p);
        uint2 hq[2];
        if constexpr (COPIES > 1) {
          uint32_t mine[WORDS], op[4];
#pragma unroll
          for (int u = 0; u < WORDS; ++u) {
            float v[2];
            Tile::template own<COPIES>(acc, copy, u, v);
            mine[u] = Low<T>::pack2(tanh_fast(v[0]), tanh_fast(v[1]));
          }
          Tile::template whole<COPIES>(mine, op);
          hq[0] = make_uint2(op[0], op[1]);
          hq[1] = make_uint2(op[2], op[3]);
        }
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
          float v[4];
          if constexpr (COPIES == 1) {
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = tanh_fast(acc[hh][r]);
            hq[hh] = pack4<T>(v);
          }
          if constexpr (TRACE) {
            const f32x4 c = *(const RAMPDE_LDS f32x4*)(l.cf + nh + (2 * p + hh) * 16);
            unpack4<T>(hq[hh], v);
#pragma unroll
            for (int r = 0; r < 4; ++r) tr = fmaf(c[r], fmaf(-v[r], v[r], 1.f), tr);
          }
        }
        const u16x8 op = Tile::operand(hq[0], hq[1]);
#pragma unroll
        for (int n = 0; n < Sh::NS; ++n) out[n] = Low<T>::mfma16(w.V[n][p], op, out[n]);
      }
      Tile::template put_part<COPIES>(out, l, wave, lane);
      if constexpr (TRACE) Tile::template put_trace<COPIES>(tr, l, wave, lane);
      rows.put(i + 1, row_next);
      const float cz = l.coef[j * 4], cb = l.coef[j * 4 + 1];
      __syncthreads();
      float v[EPT];
      Tile::sum_parts(v, l, er, ec);
      float trace = 0.f;
      if constexpr (TRACE) trace = Tile::trace_of(l, er);
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        float k = v[e] + b2[e];
        if constexpr (TRACE) k = ec + e == g.d - 1 ? -trace : k;
        k = Low<T>::to_f32(Low<T>::from_f32(k));
        bs[e] = fmaf(cb, k, bs[e]);
        if (!last_stage) {
          q[e] = Low<T>::from_f32(fmaf(h, cz * k, yh[e]));
        } else {
          if (g.round_incr & 1) bs[e] = Low<T>::to_f32(Low<T>::from_f32(bs[e]));
          y[e] = fmaf(h, bs[e], y[e]);
          q[e] = Low<T>::from_f32(y[e]);
          yh[e] = Low<T>::to_f32(q[e]);
          if (g.round_incr & 2) y[e] = yh[e];
        }
      }
      put_z(l.z + er * Sh::LDZ + ec, q);
      if (last_stage) store_elems(g.ckpt + (size_t)(i + 1) * n_state, row, g.R, ec, g.d, q);
      __syncthreads();
    }
  }
  store_elems(g.y, row, g.R, ec, g.d, y);
}

// Stage recomputation of the g.nsteps steps g.step, g.step - 1, ... (the counterpart of mlp_recompute_resident).
template <class T, int NTL, int HP, bool TRACE>
__global__ __launch_bounds__((ShallowShape<NTL, HP>::NT), (HP <= 128 ? 1 : 2)) void mlp_recompute_shallow(ShallowArgs sa) {
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  using Sh = ShallowShape<NTL, HP>;
  using Tile = ShallowTile<T, NTL, HP>;
  constexpr int EPT = Sh::EPT;
  const FusedArgs& g = sa.r.f;
  if (g.ctl->poison) return;
  ShallowLds l;
  l.carve<NTL, HP>((lds_u16*)smem);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lm = lane & 15;
  const int nh = wave * Sh::TPW * 16 + (lane >> 4) * 4;
  const int er = tid / (Sh::NT / 16), ec = (tid % (Sh::NT / 16)) * EPT;
  const int s = g.s, tiles = (int)((g.R + 15) / 16), total = tiles * g.nsteps;
  const size_t tile_bytes = (size_t)g.ldk * 32, stage_bytes = (size_t)g.Rp * 8;
  const bool copies = tid < 256 * NTL;  // (threads that copy a word of the stage-input tile, see mlp_chain_shallow)
  typename Tile::Weights w;
  w.template load<false>(g.layer[0].Wf, g.layer[1].Wf, wave, lane);
  Tile::fill(sa, l, TRACE);
  uint16_t yh_next[EPT];
  auto fetch_state = [&](int idx) __attribute__((always_inline)) {
    load_elems_clamped(g.ckpt + (size_t)(g.step - idx / tiles) * g.ckpt_stride, (int64_t)(idx % tiles) * 16 + er, g.R, ec, g.d, yh_next);
  };
  fetch_state(min((int)blockIdx.x, total - 1));
  __syncthreads();
  float b2[EPT];
#pragma unroll
  for (int e = 0; e < EPT; ++e) b2[e] = l.b2[ec + e];
#pragma unroll 1
  for (int idx = blockIdx.x; idx < total; idx += gridDim.x) {
    const int step = g.step - idx / tiles;
    const int64_t row0 = (int64_t)(idx % tiles) * 16;
    const float* st = g.steptab + (size_t)step * (1 + s);
    const float h = st[0];
    float taus[kResidentStages];
#pragma unroll
    for (int j = 0; j < kResidentStages; ++j) taus[j] = st[1 + min(j, s - 1)];
    const int64_t set_off = (int64_t)(step % g.nsets) * g.set_stride;
    char* const ZT = (char*)(g.ZT + set_off);
    char* const ACTT = (char*)(g.ACTT[0] + set_off);
    const uint32_t off_h = (uint32_t)(((size_t)(nh >> 2) * g.ldk + row0 + lm) * 8);
    const uint32_t mask = row0 + lm < g.R ? 0xFFFFFFFFu : 0u;
    const uint32_t off_z = (uint32_t)(((size_t)(tid >> 4) * g.ldk + row0 + (tid & 15)) * 8);
    const uint32_t mask_z = row0 + (tid & 15) < g.R ? 0xFFFFFFFFu : 0u;
    float yh[EPT];
    uint16_t q[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      q[e] = yh_next[e];
      yh[e] = Low<T>::to_f32(q[e]);
    }
    put_z(l.z + er * Sh::LDZ + ec, q);
    __syncthreads();
    fetch_state(min(idx + (int)gridDim.x, total - 1));
#pragma unroll 1
    for (int j = 0; j < s; ++j) {
      const float tau = j == 0 ? taus[0] : j == 1 ? taus[1] : j == 2 ? taus[2] : taus[3];
      u16x8 a[Sh::KS];
      Tile::read_z(a, l.z, lane);
      if (copies) store_word(ZT + j * stage_bytes, off_z, lds_load_u2(l.z + (tid & 15) * Sh::LDZ + (tid >> 4) * 4), mask_z);
      f32x4 out[Sh::NS];
#pragma unroll
      for (int n = 0; n < Sh::NS; ++n) out[n] = f32x4{0.f, 0.f, 0.f, 0.f};
      float tr = 0.f;
      char* gout = ACTT + j * stage_bytes;
#pragma unroll
      for (int p = 0; p < Sh::KP; ++p) {
        f32x4 acc[2];
        Tile::start(acc, l, tau, nh, p);
        Tile::pre(acc, w, a, p);
        uint2 hq[2];
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
          float v[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = tanh_fast(acc[hh][r]);
          hq[hh] = pack4<T>(v);
          store_word(gout + (2 * p + hh) * tile_bytes, off_h, hq[hh], mask);
          if constexpr (TRACE) {
            const f32x4 c = *(const RAMPDE_LDS f32x4*)(l.cf + nh + (2 * p + hh) * 16);
            unpack4<T>(hq[hh], v);
#pragma unroll
            for (int r = 0; r < 4; ++r) tr = fmaf(c[r], fmaf(-v[r], v[r], 1.f), tr);
          }
        }
        const u16x8 op = Tile::operand(hq[0], hq[1]);
#pragma unroll
        for (int n = 0; n < Sh::NS; ++n) out[n] = Low<T>::mfma16(w.V[n][p], op, out[n]);
      }
      if (j + 1 == s) break;  // (the slope of the last stage is not needed)
      Tile::put_part(out, l, wave, lane);
      if constexpr (TRACE) Tile::put_trace(tr, l, wave, lane);
      const float cz = l.coef[j * 4];
      __syncthreads();
      float v[EPT];
      Tile::sum_parts(v, l, er, ec);
      float trace = 0.f;
      if constexpr (TRACE) trace = Tile::trace_of(l, er);
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        float k = v[e] + b2[e];
        if constexpr (TRACE) k = ec + e == g.d - 1 ? -trace : k;
        k = Low<T>::to_f32(Low<T>::from_f32(k));
        q[e] = Low<T>::from_f32(fmaf(h, cz * k, yh[e]));
      }
      put_z(l.z + er * Sh::LDZ + ec, q);
      __syncthreads();
    }
    __syncthreads();  // (the stage-input tile is free again)
  }
}

// The cotangent chain of a group of adjoint steps of a tile, without the time-grid gradient (the counterpart of
// mlp_chain_resident: the outcome of the step before is looked at after a step's first stage).  Activations are requested
// a stage ahead.
template <class T, int NTL, int HP, bool TRACE>
__global__ __launch_bounds__((ShallowShape<NTL, HP>::NT), (HP <= 128 ? 1 : 2)) void mlp_chain_shallow(ShallowArgs sa) {
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  using Sh = ShallowShape<NTL, HP>;
  using Tile = ShallowTile<T, NTL, HP>;
  constexpr int EPT = Sh::EPT;
  const FusedArgs& g = sa.r.f;
  if (g.ctl->poison) return;
  ShallowLds l;
  l.carve<NTL, HP>((lds_u16*)smem);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lm = lane & 15;
  const int nh = wave * Sh::TPW * 16 + (lane >> 4) * 4;
  const int er = tid / (Sh::NT / 16), ec = (tid % (Sh::NT / 16)) * EPT;
  const int64_t row0 = (int64_t)blockIdx.x * 16, row = row0 + er;
  const int s = g.s;
  StepExchange ex(sa.r);

  typename Tile::Weights wb;
  wb.template load<false>(g.layer[1].WTf, g.layer[0].WTf, wave, lane);
  Tile::fill(sa, l, TRACE);
  const uint32_t off_h = (uint32_t)(((size_t)(nh >> 2) * g.ldk + row0 + lm) * 8);
  const size_t tile_bytes = (size_t)g.ldk * 32, stage_bytes = (size_t)g.Rp * 8;
  const uint32_t mask = row0 + lm < g.R ? 0xFFFFFFFFu : 0u;
  const uint32_t emask = row < g.R ? 0xFFFFu : 0u;
  // the 8-byte word of the state-shaped operand arrays that this thread copies out of the stage-input tile
  const bool copies = tid < 256 * NTL;
  const uint32_t off_z = (uint32_t)(((size_t)(tid >> 4) * g.ldk + row0 + (tid & 15)) * 8);
  const uint32_t mask_z = row0 + (tid & 15) < g.R ? 0xFFFFFFFFu : 0u;
  float av[EPT], a_old[EPT];
  load_elems(g.a_in, row, g.R, ec, g.d, av);
  uint2 act[Sh::TPW];
  auto fetch_act = [&](uint2 (&w)[Sh::TPW], int step, int j) __attribute__((always_inline)) {
    const char* base = (const char*)(g.ACTT[0] + (int64_t)(step % g.nsets) * g.set_stride) + j * stage_bytes;
#pragma unroll
    for (int t = 0; t < Sh::TPW; ++t) w[t] = *reinterpret_cast<const uint2*>(base + t * tile_bytes + off_h);
  };
  fetch_act(act, g.step, s - 1);
  float h_next = g.steptab[(size_t)g.step * (1 + s)];
  __syncthreads();

  bool rejected = false;
#pragma unroll 1
  for (int it = 0; it < g.nsteps; ++it) {
    const int step = g.step - it, step_next = it + 1 < g.nsteps ? step - 1 : step;
    const int64_t set_off = (int64_t)(step % g.nsets) * g.set_stride;
    char* const KBART = (char*)(g.KBART + set_off);
    char* const DELTAT = (char*)(g.DELTAT[0] + set_off);
    const float h = h_next;
    h_next = g.steptab[(size_t)step_next * (1 + s)];
    uint32_t big = 0;
    uint16_t q[EPT];
    float lam[EPT], zf[EPT], da[EPT];
    auto make_kbar = [&](int j) __attribute__((always_inline)) {
      const float ca = l.coef[j * 4], cb = l.coef[j * 4 + 1];
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        q[e] = Low<T>::from_f32(fmaf(h, ca * zf[e], cb * lam[e]));
        track(big, make_uint2(q[e], 0u));
      }
      put_z(l.z + er * Sh::LDZ + ec, q);
    };
    auto start = [&]() __attribute__((always_inline)) {
      big = 0;
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const uint16_t lq = Low<T>::from_f32(ex.S * av[e]);
        track(big, make_uint2(lq, 0u));
        lam[e] = Low<T>::to_f32(lq);
        zf[e] = da[e] = 0.f;
      }
      make_kbar(s - 1);
      __syncthreads();
    };
    start();
    bool open = it > 0 && g.detect;  // the outcome of the step before is not known yet
#pragma unroll 1
    for (int j = s - 1; j >= 0;) {
      uint2 act_next[Sh::TPW];
      fetch_act(act_next, j > 0 ? step : step_next, j > 0 ? j - 1 : s - 1);
      u16x8 a[Sh::KS];
      Tile::read_z(a, l.z, lane);
      float kl = 0.f;
      if constexpr (TRACE) kl = Low<T>::to_f32(l.z[lm * Sh::LDZ + g.d - 1]);
      if (copies) store_word(KBART + j * stage_bytes, off_z, lds_load_u2(l.z + (tid & 15) * Sh::LDZ + (tid >> 4) * 4), mask_z);
      f32x4 out[Sh::NS];
#pragma unroll
      for (int n = 0; n < Sh::NS; ++n) out[n] = f32x4{0.f, 0.f, 0.f, 0.f};
      char* gout = DELTAT + j * stage_bytes;
#pragma unroll
      for (int p = 0; p < Sh::KP; ++p) {
        f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
        Tile::pre(acc, wb, a, p);
        uint2 dq[2];
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
          float ac[4], v[4];
          unpack4<T>(act[2 * p + hh], ac);
          f32x4 c;
          if constexpr (TRACE) c = *(const RAMPDE_LDS f32x4*)(l.cf + nh + (2 * p + hh) * 16);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            float x = acc[hh][r];
            if constexpr (TRACE) x = fmaf(2.f * c[r] * ac[r], kl, x);
            v[r] = x * (1.f - ac[r] * ac[r]);
          }
          dq[hh] = pack4<T>(v);
          dq[hh].x &= mask;
          dq[hh].y &= mask;
          *reinterpret_cast<uint2*>(gout + (2 * p + hh) * tile_bytes + off_h) = dq[hh];
          track(big, dq[hh]);
        }
        const u16x8 op = Tile::operand(dq[0], dq[1]);
#pragma unroll
        for (int n = 0; n < Sh::NS; ++n) out[n] = Low<T>::mfma16(wb.V[n][p], op, out[n]);
      }
      Tile::put_part(out, l, wave, lane);
      __syncthreads();
      float v[EPT];
      Tile::sum_parts(v, l, er, ec);
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const uint16_t zq = Low<T>::from_f32(v[e]) & (uint16_t)emask;
        track(big, make_uint2(zq, 0u));
        zf[e] = Low<T>::to_f32(zq);
        da[e] += zf[e];
      }
      if (open) {
        open = false;
        const float used = ex.S;
        if (!ex.template decide<T>(g, step + 1)) {
          rejected = true;
          break;
        }
        if (ex.S != used) {
          start();
          continue;
        }
      }
      if (j > 0) make_kbar(j - 1);
      __syncthreads();
#pragma unroll
      for (int t = 0; t < Sh::TPW; ++t) {
        asm volatile("" : "+v"(act_next[t].x), "+v"(act_next[t].y));
        act[t] = act_next[t];
      }
      --j;
    }
    if (rejected) break;

    // ---- a <- a + (h / S) sum_j zbar_j (+ running-cost cotangent), fp32
    const float hs = h / ex.S;
    unsigned bits = 0;
    float gy[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) gy[e] = 0.f;
    if (g.gys) load_elems(g.gys - (int64_t)it * g.gys_stride, row, g.R, ec, g.d, gy);
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      a_old[e] = av[e];
      av[e] = fmaf(hs, da[e], av[e]) + gy[e];
      if (g.round_incr & 2) av[e] = Low<T>::to_f32(Low<T>::from_f32(av[e]));
      if (row < g.R && ec + e < g.d) bits = max(bits, __builtin_bit_cast(unsigned, fabsf(av[e])));
    }
    if (g.detect) ex.post(g, step, bits, tracked_nonfinite<T>(big));
    else ex.template decide<T>(g, step);
  }
  if (g.detect && !rejected) rejected = !ex.template decide<T>(g, g.step - g.nsteps + 1);
  if (ex.stalled) return;
#pragma unroll
  for (int e = 0; e < EPT; ++e) av[e] = rejected ? a_old[e] : av[e];
  store_elems(g.a_out, row, g.R, ec, g.d, av);
  ex.finish(g);
}

// A group of adjoint steps of a tile (the counterpart of mlp_adjoint_resident; without the time-grid gradient).
template <class T, int NTL, int HP, bool TRACE>
__global__ __launch_bounds__((ShallowShape<NTL, HP>::NT), (HP <= 128 ? 1 : 2)) void mlp_adjoint_shallow(ShallowArgs sa) {
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  using Sh = ShallowShape<NTL, HP>;
  using Tile = ShallowTile<T, NTL, HP>;
  constexpr int EPT = Sh::EPT;
  const FusedArgs& g = sa.r.f;
  if (g.ctl->poison) return;
  ShallowLds l;
  l.carve<NTL, HP>((lds_u16*)smem);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lm = lane & 15;
  const int nh = wave * Sh::TPW * 16 + (lane >> 4) * 4;
  const int er = tid / (Sh::NT / 16), ec = (tid % (Sh::NT / 16)) * EPT;
  const int64_t row0 = (int64_t)blockIdx.x * 16, row = row0 + er;
  const int s = g.s;
  StepExchange ex(sa.r);

  typename Tile::Weights wf, wb;
  if constexpr (!Sh::PHASED) {
    wf.template load<false>(g.layer[0].Wf, g.layer[1].Wf, wave, lane);
    wb.template load<false>(g.layer[1].WTf, g.layer[0].WTf, wave, lane);
  }
  Tile::fill(sa, l, TRACE);
  const StepRows rows{l.rows};
  rows.put(0, rows.load(g, g.step));
  const uint32_t off_h = (uint32_t)(((size_t)(nh >> 2) * g.ldk + row0 + lm) * 8);
  const size_t tile_bytes = (size_t)g.ldk * 32, stage_bytes = (size_t)g.Rp * 8;
  const uint32_t mask = row0 + lm < g.R ? 0xFFFFFFFFu : 0u;
  const uint32_t emask = row < g.R ? 0xFFFFu : 0u;
  // the 8-byte word of the state-shaped operand arrays that this thread copies out of the stage-input tile
  const bool copies = tid < 256 * NTL;
  const uint32_t off_z = (uint32_t)(((size_t)(tid >> 4) * g.ldk + row0 + (tid & 15)) * 8);
  const uint32_t mask_z = row0 + (tid & 15) < g.R ? 0xFFFFFFFFu : 0u;
  auto copy_z = [&](char* dst) __attribute__((always_inline)) {
    if (copies) store_word(dst, off_z, lds_load_u2(l.z + (tid & 15) * Sh::LDZ + (tid >> 4) * 4), mask_z);
  };
  float av[EPT], a_old[EPT], b2[EPT];
  load_elems(g.a_in, row, g.R, ec, g.d, av);
  uint16_t yh_next[EPT];
  load_elems_clamped(g.ckpt + (size_t)g.step * g.ckpt_stride, row, g.R, ec, g.d, yh_next);
  auto act_word = [&](int j, int t) __attribute__((always_inline)) { return l.act + ((size_t)j * 16 + lm) * (HP + 8) + nh + t * 16; };
  __syncthreads();
#pragma unroll
  for (int e = 0; e < EPT; ++e) b2[e] = l.b2[ec + e];

  bool rejected = false;
#pragma unroll 1
  for (int it = 0; it < g.nsteps; ++it) {
    const int step = g.step - it;
    const int step_next = it + 1 < g.nsteps ? step - 1 : step;
    const int64_t set_off = (int64_t)(step % g.nsets) * g.set_stride;
    char* const ZT = (char*)(g.ZT + set_off);
    char* const KBART = (char*)(g.KBART + set_off);
    char* const ACTT = (char*)(g.ACTT[0] + set_off);
    char* const DELTAT = (char*)(g.DELTAT[0] + set_off);
    if constexpr (Sh::PHASED) wf.template load<true>(g.layer[0].Wf, g.layer[1].Wf, wave, lane);
    float yh[EPT];
    uint16_t q[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      q[e] = yh_next[e];
      yh[e] = Low<T>::to_f32(q[e]);
    }
    put_z(l.z + er * Sh::LDZ + ec, q);
    __syncthreads();
    const float h = rows.h(it);

    // ---- stage recomputation
#pragma unroll 1
    for (int j = 0; j < s; ++j) {
      const bool last_stage = j + 1 == s;
      const float row_next = rows.load(g, step_next);
      load_elems_clamped(g.ckpt + (size_t)step_next * g.ckpt_stride, row, g.R, ec, g.d, yh_next);
      const float tau = rows.tau(it, j);
      u16x8 a[Sh::KS];
      Tile::read_z(a, l.z, lane);
      copy_z(ZT + j * stage_bytes);
      f32x4 out[Sh::NS];
#pragma unroll
      for (int n = 0; n < Sh::NS; ++n) out[n] = f32x4{0.f, 0.f, 0.f, 0.f};
      float tr = 0.f;
      char* gout = ACTT + j * stage_bytes;
#pragma unroll
      for (int p = 0; p < Sh::KP; ++p) {
        f32x4 acc[2];
        Tile::start(acc, l, tau, nh, p);
        Tile::pre(acc, wf, a, p);
        uint2 hq[2];
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
          float v[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = tanh_fast(acc[hh][r]);
          hq[hh] = pack4<T>(v);
          if constexpr (Sh::ACT_LDS) lds_store_u2(act_word(j, 2 * p + hh), hq[hh]);
          store_word(gout + (2 * p + hh) * tile_bytes, off_h, hq[hh], mask);
          if constexpr (TRACE) {
            const f32x4 c = *(const RAMPDE_LDS f32x4*)(l.cf + nh + (2 * p + hh) * 16);
            unpack4<T>(hq[hh], v);
#pragma unroll
            for (int r = 0; r < 4; ++r) tr = fmaf(c[r], fmaf(-v[r], v[r], 1.f), tr);
          }
        }
        const u16x8 op = Tile::operand(hq[0], hq[1]);
#pragma unroll
        for (int n = 0; n < Sh::NS; ++n) out[n] = Low<T>::mfma16(wf.V[n][p], op, out[n]);
      }
      rows.put(it + 1, row_next);
#pragma unroll
      for (int e = 0; e < EPT; ++e) asm volatile("" : "+v"(yh_next[e]));
      if (last_stage) break;  // (the slope of the last stage is not needed)
      Tile::put_part(out, l, wave, lane);
      if constexpr (TRACE) Tile::put_trace(tr, l, wave, lane);
      const float cz = l.coef[j * 4];
      __syncthreads();
      float v[EPT];
      Tile::sum_parts(v, l, er, ec);
      float trace = 0.f;
      if constexpr (TRACE) trace = Tile::trace_of(l, er);
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        float k = v[e] + b2[e];
        if constexpr (TRACE) k = ec + e == g.d - 1 ? -trace : k;
        k = Low<T>::to_f32(Low<T>::from_f32(k));
        q[e] = Low<T>::from_f32(fmaf(h, cz * k, yh[e]));
      }
      put_z(l.z + er * Sh::LDZ + ec, q);
      __syncthreads();
    }

    // ---- the previous step's outcome: its scale is needed from here on
    if (it > 0 && !ex.template decide<T>(g, step + 1)) {
      rejected = true;
      break;
    }
    if constexpr (Sh::PHASED) wb.template load<true>(g.layer[1].WTf, g.layer[0].WTf, wave, lane);

    // ---- cotangent chain
    uint32_t big = 0;
    float lam[EPT], zf[EPT], da[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const uint16_t lq = Low<T>::from_f32(ex.S * av[e]);
      track(big, make_uint2(lq, 0u));
      lam[e] = Low<T>::to_f32(lq);
      zf[e] = da[e] = 0.f;
    }
    auto make_kbar = [&](int j) __attribute__((always_inline)) {
      const float ca = l.coef[j * 4], cb = l.coef[j * 4 + 1];
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        q[e] = Low<T>::from_f32(fmaf(h, ca * zf[e], cb * lam[e]));
        track(big, make_uint2(q[e], 0u));
      }
      put_z(l.z + er * Sh::LDZ + ec, q);
    };
    __syncthreads();  // (all wavefronts are done reading the last stage's input)
    make_kbar(s - 1);
    __syncthreads();
#pragma unroll 1
    for (int j = s - 1; j >= 0; --j) {
      // activations: own words, from LDS or back from memory
      uint2 act[Sh::TPW];
#pragma unroll
      for (int t = 0; t < Sh::TPW; ++t) {
        if constexpr (Sh::ACT_LDS) act[t] = lds_load_u2(act_word(j, t));
        else act[t] = *reinterpret_cast<const uint2*>(ACTT + j * stage_bytes + t * tile_bytes + off_h);
      }
      u16x8 a[Sh::KS];
      Tile::read_z(a, l.z, lane);
      float kl = 0.f;
      if constexpr (TRACE) kl = Low<T>::to_f32(l.z[lm * Sh::LDZ + g.d - 1]);
      copy_z(KBART + j * stage_bytes);
      f32x4 out[Sh::NS];
#pragma unroll
      for (int n = 0; n < Sh::NS; ++n) out[n] = f32x4{0.f, 0.f, 0.f, 0.f};
      char* gout = DELTAT + j * stage_bytes;
#pragma unroll
      for (int p = 0; p < Sh::KP; ++p) {
        f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
        Tile::pre(acc, wb, a, p);
        uint2 dq[2];
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
          float ac[4], v[4];
          unpack4<T>(act[2 * p + hh], ac);
          f32x4 c;
          if constexpr (TRACE) c = *(const RAMPDE_LDS f32x4*)(l.cf + nh + (2 * p + hh) * 16);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            float x = acc[hh][r];
            if constexpr (TRACE) x = fmaf(2.f * c[r] * ac[r], kl, x);
            v[r] = x * (1.f - ac[r] * ac[r]);
          }
          dq[hh] = pack4<T>(v);
          dq[hh].x &= mask;
          dq[hh].y &= mask;
          *reinterpret_cast<uint2*>(gout + (2 * p + hh) * tile_bytes + off_h) = dq[hh];
          track(big, dq[hh]);
        }
        const u16x8 op = Tile::operand(dq[0], dq[1]);
#pragma unroll
        for (int n = 0; n < Sh::NS; ++n) out[n] = Low<T>::mfma16(wb.V[n][p], op, out[n]);
      }
      Tile::put_part(out, l, wave, lane);
      __syncthreads();
      float v[EPT];
      Tile::sum_parts(v, l, er, ec);
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const uint16_t zq = Low<T>::from_f32(v[e]) & (uint16_t)emask;
        track(big, make_uint2(zq, 0u));
        zf[e] = Low<T>::to_f32(zq);
        da[e] += zf[e];
      }
      if (j > 0) make_kbar(j - 1);
      __syncthreads();
    }

    // ---- a <- a + (h / S) sum_j zbar_j (+ running-cost cotangent), fp32
    const float hs = h / ex.S;
    unsigned bits = 0;
    float gy[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) gy[e] = 0.f;
    if (g.gys) load_elems(g.gys - (int64_t)it * g.gys_stride, row, g.R, ec, g.d, gy);
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      a_old[e] = av[e];
      av[e] = fmaf(hs, da[e], av[e]) + gy[e];
      if (g.round_incr & 2) av[e] = Low<T>::to_f32(Low<T>::from_f32(av[e]));
      if (row < g.R && ec + e < g.d) bits = max(bits, __builtin_bit_cast(unsigned, fabsf(av[e])));
    }
    if (g.detect) ex.post(g, step, bits, tracked_nonfinite<T>(big));
    else ex.template decide<T>(g, step);
  }
  if (g.detect && !rejected) rejected = !ex.template decide<T>(g, g.step - g.nsteps + 1);
  if (ex.stalled) return;
#pragma unroll
  for (int e = 0; e < EPT; ++e) av[e] = rejected ? a_old[e] : av[e];
  store_elems(g.a_out, row, g.R, ec, g.d, av);
  ex.finish(g);
}

// ---------------------------------------------------------------------------------------
// The trace row's share of dW1 and dW2 (see cnf.hpp): s_h = sum over stages and rows of kbar_l (1 - a_h^2) of every
// accepted step of a launch, times h / S, into slots [step][HP]; one wavefront per 4 hidden units and step.
struct TraceSums {
  const uint16_t* ACTT;   // set 0, feature-group-major
  const uint16_t* KBART;
  int64_t set_stride, ldk;
  int step, nsets, HP, l_col, s;
  const float* steptab;
  const float* scale_hist;
  float* slots;
};
template <class T>
__global__ __launch_bounds__(256) void cnf_trace_slots(TraceSums t) {
  const int lane = threadIdx.x & 63, grp = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int step = t.step - (int)blockIdx.y;
  const float S = t.scale_hist[step];
  if (S == 0.f || grp * 4 >= t.HP) return;
  const int64_t set = (int64_t)(step % t.nsets) * t.set_stride;
  const uint2* act = reinterpret_cast<const uint2*>(t.ACTT + set) + (size_t)grp * t.ldk;
  const uint16_t* kl = t.KBART + set + (size_t)(t.l_col >> 2) * t.ldk * 4 + (t.l_col & 3);
  float s[4] = {0.f, 0.f, 0.f, 0.f};
  for (int64_t k = lane; k < t.ldk; k += 64) {
    float a[4];
    unpack4<T>(act[k], a);
    const float x = Low<T>::to_f32(kl[k * 4]);
#pragma unroll
    for (int r = 0; r < 4; ++r) s[r] = fmaf(x, fmaf(-a[r], a[r], 1.f), s[r]);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r)
    for (int o = 32; o > 0; o >>= 1) s[r] += __shfl_xor(s[r], o);
  const float f = t.steptab[(size_t)step * (1 + t.s)] / S;
  if (lane == 0) *reinterpret_cast<float4*>(t.slots + (size_t)step * t.HP + grp * 4) = make_float4(f * s[0], f * s[1], f * s[2], f * s[3]);
}

// dW2[i][h] -= W1[h][i] s_h, dW1[h][i] -= W2[i][h] s_h with s_h summed over the N steps; one wavefront per h
template <class T>
__global__ __launch_bounds__(256) void cnf_trace_fold(const float* __restrict__ slots, int N, int HP, const float* __restrict__ W1,
                                                      const float* __restrict__ W2, int d, int H, int ld1, float* __restrict__ gW1,
                                                      float* __restrict__ gW2, const Ctl* ctl) {
  if (ctl->poison) return;
  const int lane = threadIdx.x & 63, h = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (h >= H) return;
  float f = 0.f;
  for (int n = lane; n < N; n += 64) f += slots[(size_t)n * HP + h];
  for (int o = 32; o > 0; o >>= 1) f += __shfl_xor(f, o);
  for (int i = lane; i < d; i += 64) {
    gW2[(size_t)i * H + h] -= f * Low<T>::to_f32(Low<T>::from_f32(W1[(size_t)h * ld1 + i]));
    gW1[(size_t)h * ld1 + i] -= f * Low<T>::to_f32(Low<T>::from_f32(W2[(size_t)i * H + h]));
  }
}

// c_h = sum_i W2[i][h] W1[h][i] from the rounded weights, fp32, in the order of i (zero past H); one thread per h
struct TraceCoef {
  const float *W1, *W2;
  float* c;
  int ld1, d, H, HP;  // HP = 0: none
};
template <class T>
__device__ __forceinline__ void trace_coefficient(const TraceCoef& t, int h) {
  if (h >= t.HP) return;
  float acc = 0.f;
  if (h < t.H) {
#pragma unroll 8
    for (int i = 0; i < t.d; ++i)
      acc = fmaf(Low<T>::to_f32(Low<T>::from_f32(t.W2[(size_t)i * t.H + h])), Low<T>::to_f32(Low<T>::from_f32(t.W1[(size_t)h * t.ld1 + i])), acc);
  }
  t.c[h] = acc;
}

}  // namespace rampde
