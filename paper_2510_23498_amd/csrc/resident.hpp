// Row-tile kernels for narrow dense networks (hidden widths up to 256, state width up to 64, two to four layers,
// up to four stages, a stage built from the one before it: Euler, midpoint, Heun, classic RK4) that keep every weight
// fragment in registers.
//
// What bounds the kernels of fused.hpp on these networks is the weight stream: a 16-row tile re-reads all weights from
// L2 in every velocity evaluation (196 KB for 64 -> 256 -> 256 -> 64, at the 64 B/clk that a compute unit gets from
// L2: 1.3 of the 3.1 us that an evaluation took), behind run-time layer and stage loops.  A compute unit's register
// file holds 512 KB: four wavefronts, one per SIMD, own a quarter of every layer's output columns each and hold their
// slices of all layers (196 KB forward, as much again transposed) for the whole launch.  What is left per evaluation is
// the matrix work, the tanh arithmetic (1024 values per SIMD and hidden layer of a tile, about 50 cycles per 64) and
// one LDS exchange with a barrier per layer; at one tile per compute unit that chain of latencies is the bound (1.5 us
// per evaluation, 0.55 of it tanh), in the adjoint kernel together with the hand-off to the gradient contraction
// (36 MB written per RK4 step of 4096 rows).  Measured, 64 -> 256 -> 256 -> 64, bf16, 32 RK4 steps of 4096 rows:
// forward 400 -> 218 us, adjoint 940 -> 491 us; fp16, 2 -> 32 -> 32 -> 2, 8 steps of 256 rows under dynamic scaling:
// forward 87 -> 27 us, adjoint 8 x 38 -> 64 us.  Of the steps on the way, each worth 5 to 15 % of the adjoint kernel:
// weights pinned to the accumulation registers so that a contraction's LDS reads are in flight together; no scalar
// loads in the stage loop; no wait for a load across a loop edge (it waits for every store as well); stores without
// branches or 64-bit lane addresses.
//
//   mlp_forward_resident : Algorithm 1, all steps of a tile in one launch
//   mlp_recompute_resident, mlp_chain_resident : Algorithm 2 for a group of steps in two launches: all steps' stages side
//     by side, then the cotangent chains one after the other.  50 -> 200 -> 200 -> 50, bf16, 1003 rows (63 tiles), 20
//     Heun steps with the time-grid gradient: 213 us in one kernel, pass 414 -> 347 us
//   mlp_adjoint_resident : the same in one launch (tiles that fill the device, single steps)
//     Both also under overflow detection.  The scale is the only thing that couples tiles between steps.  Every
//     workgroup posts max|a| and its overflow flag of a step as ONE 64-bit word (payload and tag together: no fence, no
//     second round trip).  It reads the others' words when it needs the next step's scale, which in one launch is not
//     before its last stage has been recomputed; the chain alone goes on with the scale at hand and looks after one
//     stage.  All workgroups fold the same words, so they take the same decision.
//
// The waits need the workgroups of a launch to run at the same time; the host launches no more of them than the device
// holds.  If others occupy the device (another stream's kernels), a wait ends after kWaitTicks, the launch raises
// Ctl.stalled, writes no result, and the host redoes the pass with one launch per step.  A word that is on its way comes
// within a step (at most about 0.1 ms); kernels that hold compute units for longer than 2 ms cost less as a redone pass
// (a few ms) than as a wait for their end.
#pragma once
#include "fused.hpp"

namespace rampde {

struct ResidentArgs {
  FusedArgs f;
  // [steps of the pass][workgroups] words {tag : 32, payload : 32}; payload = bits of max|a| of the tile after the
  // step, top bit: a value of the step's cotangent chain was not finite; tag = the attempt number (0: not posted)
  unsigned long long* slots;
  unsigned long long wait_ticks;  // how long a workgroup waits for a word; 0: it gives up without looking
};

constexpr int kResidentStages = 4;
constexpr unsigned long long kWaitTicks = 200ull * 1000;  // of the 100 MHz counter: 2 ms

template <int L, int HP>
struct ResidentShape {
  static constexpr int TPW = HP / 64;  // column tiles of 16 that a wavefront owns in a hidden layer
  static constexpr int KBH = HP / 32;  // k-blocks of 32 of a contraction over a hidden layer
  static constexpr int LDZ = 64 + 8, LDP = HP + 8;
  static constexpr int MIDS = L - 2;   // hidden -> hidden layers
};

// the wavefront's slices of all layers: FWD as they multiply forward, else transposed (cotangent chain)
// LAST_IN_LDS: the last slice (32 KB per workgroup at width 256) is kept in LDS and read when it is used
template <int L, int HP, bool LAST_IN_LDS = false>
struct ResidentWeights {
  using Sh = ResidentShape<L, HP>;
  u16x8 first[Sh::TPW][2];
  u16x8 mid[Sh::MIDS > 0 ? Sh::MIDS : 1][Sh::TPW][Sh::KBH];
  u16x8 last[1][Sh::KBH];
  lds_u16* last_lds;

  // AGAIN: called once per phase; the barrier keeps the compiler from holding both phases' slices over the whole loop
  template <bool FWD, int PINNED, bool AGAIN = false>
  __device__ __forceinline__ void load(const FusedArgs& g, int wave, int lane) {
    if constexpr (AGAIN) asm volatile("" : "+v"(lane));
    const glb_u16x8* f = (const glb_u16x8*)(FWD ? g.layer[0].Wf : g.layer[L - 1].WTf) + lane;
    const glb_u16x8* e = (const glb_u16x8*)(FWD ? g.layer[L - 1].Wf : g.layer[0].WTf) + lane;
#pragma unroll
    for (int t = 0; t < Sh::TPW; ++t)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) first[t][kb] = f[(size_t)(kb * (HP / 16) + wave * Sh::TPW + t) * 64];
#pragma unroll
    for (int m = 0; m < Sh::MIDS; ++m) {
      const glb_u16x8* w = (const glb_u16x8*)(FWD ? g.layer[m + 1].Wf : g.layer[m + 1].WTf) + lane;
#pragma unroll
      for (int t = 0; t < Sh::TPW; ++t)
#pragma unroll
        for (int kb = 0; kb < Sh::KBH; ++kb) mid[m][t][kb] = w[(size_t)(kb * (HP / 16) + wave * Sh::TPW + t) * 64];
    }
#pragma unroll
    for (int kb = 0; kb < Sh::KBH; ++kb) {
      if constexpr (LAST_IN_LDS) *(lds_u16x8*)(last_lds + ((size_t)(wave * Sh::KBH + kb) * 64 + lane) * 8) = e[(size_t)(kb * 4 + wave) * 64];
      else last[0][kb] = e[(size_t)(kb * 4 + wave) * 64];
    }
    // At width 256 the hidden layers' slices go to the accumulation half of the register file, from where matrix
    // instructions read them as well (left to itself the compiler fills the other half with them, and the activation
    // fragments of a contraction then share one register: every LDS read waits for its own round trip).  PINNED: how many
    // fragments per column tile; the accumulators need room there too.
    if constexpr (HP == 256) {
#pragma unroll
      for (int m = 0; m < Sh::MIDS; ++m)
#pragma unroll
        for (int t = 0; t < Sh::TPW; ++t)
#pragma unroll
          for (int kb = 0; kb < Sh::KBH; ++kb)
            if (m * Sh::KBH + kb < PINNED) asm volatile("" : "+a"(mid[m][t][kb]));
    }
  }
};

// the last slice as registers (before the barrier of the pass that multiplies by it)
template <int L, int HP, bool IN_LDS>
__device__ __forceinline__ void fetch_last(u16x8 (&r)[1][HP / 32], const ResidentWeights<L, HP, IN_LDS>& w, int wave, int lane) {
#pragma unroll
  for (int kb = 0; kb < HP / 32; ++kb) {
    if constexpr (IN_LDS) r[0][kb] = *(const lds_u16x8*)(w.last_lds + ((size_t)(wave * (HP / 32) + kb) * 64 + lane) * 8);
    else r[0][kb] = w.last[0][kb];
  }
}

// acc[t][mt] += (rows of `in`) x (weight slice w); in: LDS tile of 16 MT rows
template <class T, int MT, int NT, int KB>
__device__ __forceinline__ void resident_mma(f32x4 (&acc)[NT][MT], const u16x8 (&w)[NT][KB], const lds_u16* in, int pitch,
                                             int lane) {
  const lds_u16* a0 = in + (lane & 15) * pitch + (lane >> 4) * 8;
  u16x8 a[KB][MT];
#pragma unroll
  for (int kb = 0; kb < KB; ++kb)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) a[kb][mt] = *(const lds_u16x8*)(a0 + mt * 16 * pitch + kb * 32);
  __builtin_amdgcn_sched_barrier(0);  // all reads in flight before the first matrix instruction
  // (tile by tile: the arithmetic on a finished tile runs beside the matrix instructions of the next)
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[t][mt] = Low<T>::mfma16(w[t][kb], a[kb][mt], acc[t][mt]);
}

// the state-shaped contraction: one column tile per wavefront, two accumulators so that the dependent chain of matrix
// instructions is half as long
template <class T, int MT, int KB>
__device__ __forceinline__ void resident_mma_state(f32x4 (&out)[MT], const u16x8 (&w)[1][KB], const lds_u16* in, int pitch,
                                                   int lane) {
  const lds_u16* a0 = in + (lane & 15) * pitch + (lane >> 4) * 8;
  f32x4 odd[MT];
  u16x8 a[KB][MT];
#pragma unroll
  for (int kb = 0; kb < KB; ++kb)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) a[kb][mt] = *(const lds_u16x8*)(a0 + mt * 16 * pitch + kb * 32);
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) odd[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int kb = 0; kb < KB; kb += 2)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      out[mt] = Low<T>::mfma16(w[0][kb], a[kb][mt], out[mt]);
      if (kb + 1 < KB) odd[mt] = Low<T>::mfma16(w[0][kb + 1], a[kb + 1][mt], odd[mt]);
    }
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) out[mt] += odd[mt];
}

// (a branch around the assignment would put the array in scratch memory)
__device__ __forceinline__ void keep_if(bool c, uint2& dst, uint2 v) {
  dst.x = c ? v.x : dst.x;
  dst.y = c ? v.y : dst.y;
}

// The step table's rows (h, tau_1 .. tau_s) pass through LDS, two rows at a time: a scalar load in the stage loop would
// share its counter with the LDS reads, and every wait for an activation fragment would become a wait for it too.
// A stage's body requests the next step's row at its head and writes it to LDS at its end, in straight-line code: loads
// and stores share a counter, and a wait across a loop edge is a wait for every store that was issued meanwhile.
struct StepRows {
  lds_f32* tab;  // [2][8]
  __device__ __forceinline__ float load(const FusedArgs& g, int step) const {
    return g.steptab[(size_t)step * (1 + g.s) + min((int)threadIdx.x, g.s)];
  }
  __device__ __forceinline__ void put(int it, float v) const {
    if (threadIdx.x < 8) tab[(it & 1) * 8 + threadIdx.x] = v;
  }
  __device__ __forceinline__ float h(int it) const { return tab[(it & 1) * 8]; }
  __device__ __forceinline__ float tau(int it, int j) const { return tab[(it & 1) * 8 + 1 + j]; }
};

// one lane's 4 state columns of a stored state (columns >= d and rows >= R read as zero) without divergent branches
__device__ __forceinline__ uint2 load_state(const uint16_t* p, int64_t row, int64_t R, int c, int d) {
  const int64_t r = row < R ? row : R - 1;
  uint2 q;
  if ((d & 3) == 0) {
    q = *reinterpret_cast<const uint2*>(&p[(size_t)r * d + min(c, d - 4)]);
    if (c >= d) q = make_uint2(0u, 0u);
  } else {
    uint32_t e[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) e[i] = p[(size_t)r * d + min(c + i, d - 1)];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (c + i >= d) e[i] = 0;
    q = make_uint2(e[0] | (e[1] << 16), e[2] | (e[3] << 16));
  }
  if (row >= R) q = make_uint2(0u, 0u);
  return q;
}

// running maxima of |x| over the two 16-bit halves of packed words (as integers: inf and nan compare above everything)
__device__ __forceinline__ void track(uint32_t& m, uint2 q) {
  typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
  u16x2 a = __builtin_bit_cast(u16x2, m), x = __builtin_bit_cast(u16x2, q.x & 0x7FFF7FFFu), y = __builtin_bit_cast(u16x2, q.y & 0x7FFF7FFFu);
  a = __builtin_elementwise_max(a, __builtin_elementwise_max(x, y));
  m = __builtin_bit_cast(uint32_t, a);
}
template <class T>
__device__ __forceinline__ bool tracked_nonfinite(uint32_t m) {
  return Low<T>::nonfinite((uint16_t)m) || Low<T>::nonfinite((uint16_t)(m >> 16));
}

// 8-byte word at a wave-uniform base plus a 32-bit lane offset (bytes), zero for rows past the batch (they are the
// padding of the parameter-gradient contraction): no branch around the store, no 64-bit lane address
__device__ __forceinline__ void store_word(void* base, uint32_t lane_off, uint2 q, uint32_t mask) {
  q.x &= mask;
  q.y &= mask;
  *reinterpret_cast<uint2*>((char*)base + lane_off) = q;
}

// LDS: parameters (biases, time column), 16-entry coefficient tables, stage-input tile, then the kernel's own tiles
template <int L, int HP>
struct ResidentLds {
  using Sh = ResidentShape<L, HP>;
  static constexpr int NPARAM = HP * L + 64;  // (L - 1) hidden biases, the state bias, the time column
  lds_f32* bias;
  lds_f32* wt;
  lds_f32* coef;  // [4][4]: row j = a_{j+1,j}, b_j, c_j, a_{j,j-1} (zero where the tableau has no such entry)
  lds_f32* rows;  // [2][8] step table
  lds_u16* z;
  lds_u16* tiles;
  __device__ __forceinline__ ResidentLds(lds_u16* smem, int MT) {
    bias = (lds_f32*)smem;
    wt = bias + (L - 1) * HP + 64;
    coef = bias + NPARAM;
    rows = coef + 16;
    z = (lds_u16*)(rows + 16);
    tiles = z + 16 * MT * Sh::LDZ;
  }
  static constexpr size_t bytes(int MT, int ntiles) {
    return (size_t)(NPARAM + 32) * 4 + 2 * (size_t)(16 * MT) * (Sh::LDZ + (size_t)ntiles * Sh::LDP);
  }
  __device__ __forceinline__ void fill(const FusedArgs& g) {
#pragma unroll
    for (int l = 0; l < L; ++l) {
      const int n = l + 1 < L ? HP : 64;
      for (int i = threadIdx.x; i < n; i += 256) bias[l * HP + i] = g.layer[l].bias[i];
    }
    for (int i = threadIdx.x; i < HP; i += 256) wt[i] = g.layer[0].wt ? g.layer[0].wt[i] : 0.f;
    if (threadIdx.x < 16) {
      const int j = threadIdx.x >> 2, e = threadIdx.x & 3;
      float c = 0.f;
      if (j < g.s) c = e == 0 ? (j + 1 < g.s ? g.A[(j + 1) * g.s + j] : 0.f) : e == 1 ? g.b[j] : e == 2 ? g.c[j] : (j > 0 ? g.A[j * g.s + j - 1] : 0.f);
      coef[threadIdx.x] = c;
    }
  }
};

// hidden layer l: bias (+ time column) as the accumulators' start
template <int NT, int MT>
__device__ __forceinline__ void init_acc(f32x4 (&acc)[NT][MT], const lds_f32* bias, int n0) {
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const f32x4 b = *(const RAMPDE_LDS f32x4*)(bias + n0 + t * 16);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[t][mt] = b;
  }
}
template <int NT, int MT>
__device__ __forceinline__ void init_acc_time(f32x4 (&acc)[NT][MT], const lds_f32* bias, const lds_f32* wt, float tau, int n0) {
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    f32x4 b = *(const RAMPDE_LDS f32x4*)(bias + n0 + t * 16);
    const f32x4 w = *(const RAMPDE_LDS f32x4*)(wt + n0 + t * 16);
#pragma unroll
    for (int r = 0; r < 4; ++r) b[r] = fmaf(w[r], tau, b[r]);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[t][mt] = b;
  }
}
template <int NT, int MT>
__device__ __forceinline__ void zero_acc(f32x4 (&acc)[NT][MT]) {
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[t][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
}

// ---------------------------------------------------------------------------------------
// COPIES = 2, 4: tiles of 8 or 4 rows, where the 16-row tiles leave half or three quarters of the compute units idle.  The
// tile's 16 rows are then so many copies of them, and a copy of a row finishes its share of the wavefront's column tiles:
// half or a quarter of the tanh arithmetic per lane.  One row, 64 -> 256 -> 256 -> 64, f16, 32 RK4 steps: 203 -> 174 us per
// pass; 300 rows, one hidden layer, bf16 129 -> 111; 1024 rows, 64 -> 3 x 200 -> 64 271 -> 230; 2048 rows (two copies), two
// of 256 200 -> 182.
template <class T, int L, int HP, int MT, int COPIES>
__global__ __launch_bounds__(256, HP == 256 ? 1 : 2) void mlp_forward_resident(ResidentArgs ra) {
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  using Sh = ResidentShape<L, HP>;
  const FusedArgs& g = ra.f;
  ResidentLds<L, HP> lds((lds_u16*)smem, MT);
  static_assert(COPIES == 1 || MT == 1, "one tile");
  constexpr int ROWS = 16 / COPIES;               // of a tile of 16
  const int lane0 = threadIdx.x & 63, wave = threadIdx.x >> 6, copy = (lane0 & 15) / ROWS;
  const int lane = (lane0 & 0x30) | lane0 % ROWS, lm = lane & 15, lq = lane >> 4;  // (of the copied row)
  constexpr int TPW = Sh::TPW;
  const int64_t row0 = (int64_t)blockIdx.x * ROWS * MT;
  const int64_t n_state = g.R * g.d;
  const int s = g.s;
  const int ns = wave * 16 + lq * 4;              // the lane's state columns
  const int nh = wave * TPW * 16 + lq * 4;        // ... and its first hidden columns
  lds_u16* const buf[2] = {lds.tiles, lds.tiles + 16 * MT * Sh::LDP};

  ResidentWeights<L, HP> w;
  w.template load<true, MT == 1 ? 14 : 12>(g, wave, lane0);
  lds.fill(g);
  const StepRows rows{lds.rows};
  rows.put(0, rows.load(g, 0));
  // y, the stored state Q(y), and the running sum_j b_j k_j
  float yv[MT][4], yh[MT][4], bs[MT][4];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    load4f(g.y0, row0 + mt * 16 + lm, g.R, ns, g.d, yv[mt]);
    const uint2 q = pack4<T>(yv[mt]);
    if (g.round_incr & 2) unpack4<T>(q, yv[mt]);
    if (copy == 0) store4h(g.ckpt, row0 + mt * 16 + lm, g.R, ns, g.d, q);
    unpack4<T>(q, yh[mt]);
    lds_store_u2(&lds.z[(mt * 16 + lm) * Sh::LDZ + ns], q);
  }
  __syncthreads();

  auto store_tanh = [&](const f32x4 (&acc)[TPW][MT], lds_u16* out) __attribute__((always_inline)) {
    if constexpr (COPIES > 1) {
      constexpr int C = COPIES < TPW ? COPIES : TPW;  // (fewer column tiles than copies: two finish the same one)
#pragma unroll
      for (int u = 0; u < TPW / C; ++u) {
        const int t = copy % C;
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float x = acc[u * C][0][r];
#pragma unroll
          for (int q = 1; q < C; ++q) x = t == q ? acc[u * C + q][0][r] : x;
          v[r] = tanh_fast(x);
        }
        lds_store_u2(&out[lm * Sh::LDP + nh + (u * C + t) * 16], pack4<T>(v));
      }
      return;
    }
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = tanh_fast(acc[t][mt][r]);
        lds_store_u2(&out[(mt * 16 + lm) * Sh::LDP + nh + t * 16], pack4<T>(v));
      }
  };

  // (a pass's bias and coefficient reads are issued before the barrier that it waits at)
  f32x4 acc[TPW][MT];
  init_acc_time(acc, lds.bias, lds.wt, rows.tau(0, 0), nh);
  for (int i = 0; i < g.N; ++i) {
    const float h = rows.h(i);
    const int i_next = min(i + 1, g.N - 1);
    uint16_t* ck_next = g.ckpt + (size_t)(i + 1) * n_state;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r) bs[mt][r] = 0.f;
#pragma unroll 1
    for (int j = 0; j < s; ++j) {
      const bool last_stage = j + 1 == s;
      const float row_next = rows.load(g, i_next);
      resident_mma<T, MT>(acc, w.first, lds.z, Sh::LDZ, lane);
      store_tanh(acc, buf[0]);
      rows.put(i + 1, row_next);
      f32x4 ks[MT];
      const f32x4 bl = *(const RAMPDE_LDS f32x4*)(lds.bias + (L - 1) * HP + ns);
      const f32x4 cf = *(const RAMPDE_LDS f32x4*)(lds.coef + j * 4);
#pragma unroll
      for (int m = 0; m < Sh::MIDS; ++m) {
        init_acc(acc, lds.bias + (m + 1) * HP, nh);
        __syncthreads();
        resident_mma<T, MT>(acc, w.mid[m], buf[m & 1], Sh::LDP, lane);
        store_tanh(acc, buf[(m + 1) & 1]);
      }
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) ks[mt] = bl;
      __syncthreads();
      resident_mma_state<T, MT>(ks, w.last, buf[Sh::MIDS & 1], Sh::LDP, lane);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const float v[4] = {ks[mt][0], ks[mt][1], ks[mt][2], ks[mt][3]};
        const uint2 q = pack4<T>(v);
        float kf[4];
        unpack4<T>(q, kf);
#pragma unroll
        for (int r = 0; r < 4; ++r) bs[mt][r] = fmaf(cf[1], kf[r], bs[mt][r]);
        uint2 zq;
        if (!last_stage) {
          float z[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) z[r] = fmaf(h, cf[0] * kf[r], yh[mt][r]);
          zq = pack4<T>(z);
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            if (g.round_incr & 1) bs[mt][r] = Low<T>::to_f32(Low<T>::from_f32(bs[mt][r]));
            yv[mt][r] = fmaf(h, bs[mt][r], yv[mt][r]);
          }
          zq = pack4<T>(yv[mt]);
          if (g.round_incr & 2) unpack4<T>(zq, yv[mt]);
          unpack4<T>(zq, yh[mt]);
        }
        lds_store_u2(&lds.z[(mt * 16 + lm) * Sh::LDZ + ns], zq);
        if (last_stage && copy == 0) store4h(ck_next, row0 + mt * 16 + lm, g.R, ns, g.d, zq);
      }
      init_acc_time(acc, lds.bias, lds.wt, last_stage ? rows.tau(i + 1, 0) : rows.tau(i, j + 1), nh);
      __syncthreads();
    }
  }
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
    if (copy == 0) store4f(g.y, row0 + mt * 16 + lm, g.R, ns, g.d, yv[mt]);
}

// The accept / reject / grow bookkeeping of a launch that runs several steps (Algorithm 2), one object per thread with
// the same contents in every thread of every workgroup.
struct StepExchange {
  const ResidentArgs& ra;
  float S, s_min, s_max;
  int attempt;
  bool stalled = false;
  int me, posts;  // this workgroup's number among those that post
  __device__ __forceinline__ StepExchange(const ResidentArgs& r, int me_, int posts_)
      : ra(r), S(r.f.ctl->S), s_min(r.f.ctl->s_min), s_max(r.f.ctl->s_max), attempt(r.f.ctl->attempt), me(me_), posts(posts_) {}
  __device__ __forceinline__ StepExchange(const ResidentArgs& r) : StepExchange(r, blockIdx.x, gridDim.x) {}

  // post this workgroup's word of step `step`: bits of its max|a|, and whether its cotangent chain left the range
  __device__ __forceinline__ void post(const FusedArgs& g, int step, unsigned bits, bool nonfinite) {
    __shared__ unsigned s_post[16];
    if (nonfinite) bits |= 0x80000000u;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) bits = max(bits, (unsigned)__shfl_xor((int)bits, o));
    if ((threadIdx.x & 63) == 0) s_post[threadIdx.x >> 6] = bits;
    __syncthreads();
    if (threadIdx.x == 0) {
      unsigned m = 0;
      for (int w = 0; w < (int)(blockDim.x >> 6); ++w) m = max(m, s_post[w]);
      __hip_atomic_store(ra.slots + (size_t)step * posts + me, ((unsigned long long)attempt << 32) | m,
                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }

  // the outcome of step `step` over all tiles, from every workgroup's word.  Returns false if a wait ran out.
  __device__ __forceinline__ bool collect(int step, unsigned& pay) {
    __shared__ unsigned s_pay[16];
    __shared__ int s_late[16];
    const unsigned long long* row = ra.slots + (size_t)step * posts;
    unsigned m = 0;
    bool late = ra.wait_ticks == 0;
    unsigned long long t0 = 0;
    for (int q = threadIdx.x; q < posts; q += blockDim.x) {
      unsigned long long v = __hip_atomic_load(row + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      while ((int)(v >> 32) != attempt && !late) {
        if (t0 == 0) t0 = wall_clock64();
        __builtin_amdgcn_s_sleep(1);
        v = __hip_atomic_load(row + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        late = wall_clock64() - t0 >= ra.wait_ticks;
      }
      m = max(m, (unsigned)v);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = max(m, (unsigned)__shfl_xor((int)m, o));
    const int any_late = __any(late ? 1 : 0);
    if ((threadIdx.x & 63) == 0) {
      s_pay[threadIdx.x >> 6] = m;
      s_late[threadIdx.x >> 6] = any_late;
    }
    __syncthreads();
    bool ok = true;
    pay = 0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
      pay = max(pay, s_pay[w]);
      ok = ok && s_late[w] == 0;
    }
    return ok;  // (the next write to the shared words is a whole step of barriers away)
  }

  // accept / grow; false: the step is rejected, or the wait ran out (stalled)
  template <class T>
  __device__ __forceinline__ bool decide(const FusedArgs& g, int step) {
    const bool first = me == 0 && threadIdx.x == 0;
    if (g.detect) {
      unsigned pay;
      if (!collect(step, pay)) {
        stalled = true;
        if (threadIdx.x == 0) {  // (poison: every later kernel of the pass does nothing)
          __hip_atomic_store(&g.ctl->stalled, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(&g.ctl->poison, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        return false;
      }
      if (pay & 0x80000000u) {
        if (first) {
          g.ctl->poison = 1;
          g.ctl->failed_step = step;
        }
        return false;
      }
      s_min = fminf(s_min, S);
      s_max = fmaxf(s_max, S);
      if (first) {
        g.scale_hist[step] = S;
        g.ctl->S_step = S;
      }
      if (g.dynamic && attempt == 1) {
        const float amax = __builtin_bit_cast(float, pay);
        const float test = g.raw_norm ? amax : S * amax;
        if (test <= ldexpf(1.f, Low<T>::p_bits - 1) && S < ldexpf(1.f, 126)) S *= 2.f;
      }
      attempt = 1;
    } else if (first) {
      g.scale_hist[step] = S;
    }
    return true;
  }

  __device__ __forceinline__ void finish(const FusedArgs& g) {
    if (me == 0 && threadIdx.x == 0) {
      g.ctl->S = S;
      g.ctl->attempt = attempt;
      g.ctl->s_min = s_min;
      g.ctl->s_max = s_max;
    }
  }
};

// ---------------------------------------------------------------------------------------
// Stage recomputation of the g.nsteps steps g.step, g.step - 1, ... from their stored states: stage inputs and hidden
// activations into the steps' buffer sets.  The stored states are all known, so steps x tiles run side by side; a
// workgroup takes every gridDim.x-th of them and loads its weight slices once.  TG: also the slopes (g.KT), for the
// time-grid terms of the chain.
template <class T, int L, int HP, int MT, bool TG>
__global__ __launch_bounds__(256, HP == 256 ? 1 : 2) void mlp_recompute_resident(ResidentArgs ra) {
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  using Sh = ResidentShape<L, HP>;
  const FusedArgs& g = ra.f;
  if (g.ctl->poison) return;
  ResidentLds<L, HP> lds((lds_u16*)smem, MT);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lm = lane & 15, lq = lane >> 4;
  constexpr int TPW = Sh::TPW, TM = 16 * MT;
  const int s = g.s;
  const int ns = wave * 16 + lq * 4, nh = wave * TPW * 16 + lq * 4;
  lds_u16* const buf[2] = {lds.tiles, lds.tiles + TM * Sh::LDP};
  const int tiles = (int)((g.R + TM - 1) / TM), total = tiles * g.nsteps;
  const size_t tile_bytes = (size_t)g.ldk * 32, stage_bytes = (size_t)g.Rp * 8;

  ResidentWeights<L, HP> w;
  w.template load<true, MT == 1 ? 14 : 12>(g, wave, lane);
  lds.fill(g);
  uint2 yh_next[MT];
  auto fetch_state = [&](int idx) __attribute__((always_inline)) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      yh_next[mt] = load_state(g.ckpt + (size_t)(g.step - idx / tiles) * g.ckpt_stride, (int64_t)(idx % tiles) * TM + mt * 16 + lm, g.R, ns, g.d);
  };
  fetch_state(min((int)blockIdx.x, total - 1));
#pragma unroll 1
  for (int idx = blockIdx.x; idx < total; idx += gridDim.x) {
    const int step = g.step - idx / tiles;
    const int64_t row0 = (int64_t)(idx % tiles) * TM;
    const float* st = g.steptab + (size_t)step * (1 + s);
    const float h = st[0];
    float tau[kResidentStages];
#pragma unroll
    for (int j = 0; j < kResidentStages; ++j) tau[j] = st[1 + min(j, s - 1)];
    const int64_t set_off = (int64_t)(step % g.nsets) * g.set_stride;
    char* const ZT = (char*)(g.ZT + set_off);
    const uint32_t off_h = (uint32_t)(((size_t)(nh >> 2) * g.ldk + row0 + lm) * 8);
    const uint32_t off_s = (uint32_t)(((size_t)(ns >> 2) * g.ldk + row0 + lm) * 8);
    uint32_t mask[MT];
    float yh[MT][4];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      mask[mt] = row0 + mt * 16 + lm < g.R ? 0xFFFFFFFFu : 0u;
      unpack4<T>(yh_next[mt], yh[mt]);
      lds_store_u2(&lds.z[(mt * 16 + lm) * Sh::LDZ + ns], yh_next[mt]);
      store_word(ZT, off_s + mt * 128, yh_next[mt], mask[mt]);
    }
    __syncthreads();
    fetch_state(min(idx + (int)gridDim.x, total - 1));
    auto store_act = [&](const f32x4 (&acc)[TPW][MT], int j, int l) __attribute__((always_inline)) {
      char* gout = (char*)(g.ACTT[l] + set_off) + j * stage_bytes;
#pragma unroll
      for (int t = 0; t < TPW; ++t)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          float v[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = tanh_fast(acc[t][mt][r]);
          const uint2 q = pack4<T>(v);
          lds_store_u2(&buf[l & 1][(mt * 16 + lm) * Sh::LDP + nh + t * 16], q);
          store_word(gout + t * tile_bytes, off_h + mt * 128, q, mask[mt]);
        }
    };
    f32x4 acc[TPW][MT];
#pragma unroll 1
    for (int j = 0; j < s; ++j) {
      const bool last_stage = j + 1 == s;
      init_acc_time(acc, lds.bias, lds.wt, j == 0 ? tau[0] : j == 1 ? tau[1] : j == 2 ? tau[2] : tau[3], nh);
      resident_mma<T, MT>(acc, w.first, lds.z, Sh::LDZ, lane);
      store_act(acc, j, 0);
      f32x4 ks[MT];
      const f32x4 bl = *(const RAMPDE_LDS f32x4*)(lds.bias + (L - 1) * HP + ns);
      const f32x4 cf = *(const RAMPDE_LDS f32x4*)(lds.coef + j * 4);
#pragma unroll
      for (int m = 0; m < Sh::MIDS; ++m) {
        init_acc(acc, lds.bias + (m + 1) * HP, nh);
        __syncthreads();
        resident_mma<T, MT>(acc, w.mid[m], buf[m & 1], Sh::LDP, lane);
        store_act(acc, j, m + 1);
      }
      if (last_stage && !TG) break;  // (the slope of the last stage is not needed)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) ks[mt] = bl;
      __syncthreads();
      resident_mma_state<T, MT>(ks, w.last, buf[Sh::MIDS & 1], Sh::LDP, lane);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const float v[4] = {ks[mt][0], ks[mt][1], ks[mt][2], ks[mt][3]};
        const uint2 q = pack4<T>(v);
        float kf[4], z[4];
        unpack4<T>(q, kf);
        if constexpr (TG) store_word((char*)(g.KT + set_off) + j * stage_bytes, off_s + mt * 128, q, mask[mt]);
        if (!last_stage) {
#pragma unroll
          for (int r = 0; r < 4; ++r) z[r] = fmaf(h, cf[0] * kf[r], yh[mt][r]);
          const uint2 zq = pack4<T>(z);
          lds_store_u2(&lds.z[(mt * 16 + lm) * Sh::LDZ + ns], zq);
          store_word(ZT + (j + 1) * stage_bytes, off_s + mt * 128, zq, mask[mt]);
        }
      }
      __syncthreads();
    }
    __syncthreads();  // (the stage-input tile and the ping-pong tiles are free again)
  }
}

// ---------------------------------------------------------------------------------------
// The cotangent chain of a group of adjoint steps of a tile, from the stages that mlp_recompute_resident has stored.
// A step's scale depends on the outcome of the step before, which takes an exchange between all workgroups: the step
// starts with the scale at hand and looks at the outcome after its first stage; where that changed the scale, the stage
// is redone (everything that it has written is written again).
template <class T, int L, int HP, int MT, bool TG>
__global__ __launch_bounds__(256, HP == 256 ? 1 : 2) void mlp_chain_resident(ResidentArgs ra) {
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  using Sh = ResidentShape<L, HP>;
  const FusedArgs& g = ra.f;
  if (g.ctl->poison) return;
  ResidentLds<L, HP> lds((lds_u16*)smem, MT);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lm = lane & 15, lq = lane >> 4;
  constexpr int TPW = Sh::TPW, TM = 16 * MT;
  const int64_t row0 = (int64_t)blockIdx.x * TM;
  const int s = g.s;
  const int ns = wave * 16 + lq * 4, nh = wave * TPW * 16 + lq * 4;

  ResidentWeights<L, HP> wb;
  wb.template load<false, MT == 1 ? 14 : 12>(g, wave, lane);
  lds.fill(g);
  StepExchange ex(ra);
  float av[MT][4], a_old[MT][4];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) load4f(g.a_in, row0 + mt * 16 + lm, g.R, ns, g.d, av[mt]);
  // lane offsets (bytes) into the feature-group-major arrays: hidden and state columns, and the batch-row masks
  const uint32_t off_h = (uint32_t)(((size_t)(nh >> 2) * g.ldk + row0 + lm) * 8);
  const uint32_t off_s = (uint32_t)(((size_t)(ns >> 2) * g.ldk + row0 + lm) * 8);
  const size_t tile_bytes = (size_t)g.ldk * 32;  // 16 columns further
  const size_t stage_bytes = (size_t)g.Rp * 8;
  uint32_t mask[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) mask[mt] = row0 + mt * 16 + lm < g.R ? 0xFFFFFFFFu : 0u;
  // activations at the lane's own elements, requested a stage ahead
  uint2 act[L - 1][TPW][MT];
  auto fetch_act = [&](uint2 (&q)[L - 1][TPW][MT], int step, int j) __attribute__((always_inline)) {
#pragma unroll
    for (int l = 0; l < L - 1; ++l) {
      const char* base = (const char*)(g.ACTT[l] + (int64_t)(step % g.nsets) * g.set_stride) + j * stage_bytes;
#pragma unroll
      for (int t = 0; t < TPW; ++t)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) q[l][t][mt] = *reinterpret_cast<const uint2*>(base + t * tile_bytes + (off_h + mt * 128));
    }
  };
  fetch_act(act, g.step, s - 1);
  // cotangents of hidden layer l
  auto tile = [&](int l) __attribute__((always_inline)) { return lds.tiles + (size_t)l * TM * Sh::LDP; };
  float h_next = g.steptab[(size_t)g.step * (1 + s)];
  __syncthreads();

  bool rejected = false;
#pragma unroll 1
  for (int it = 0; it < g.nsteps; ++it) {
    const int step = g.step - it, step_next = it + 1 < g.nsteps ? step - 1 : step;
    const int64_t set_off = (int64_t)(step % g.nsets) * g.set_stride;
    char* const KBART = (char*)(g.KBART + set_off);
    const float h = h_next;
    h_next = g.steptab[(size_t)step_next * (1 + s)];
    float t_phia = 0.f, t_dt = 0.f, t_dh = 0.f;
    uint2 k[TG ? kResidentStages : 1][MT];  // slopes
    if constexpr (TG) {
#pragma unroll
      for (int j = 0; j < kResidentStages; ++j)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          k[j][mt] = *reinterpret_cast<const uint2*>((const char*)(g.KT + set_off) + min(j, s - 1) * stage_bytes + (off_s + mt * 128));
    }
    uint32_t big = 0;  // largest magnitudes of the step's cotangents
    uint2 lamq[MT];
    float zf[MT][4];  // cotangent of the stage input behind the slope at hand
    float da[MT][4];
    // cotangent of the slope of stage j:  kbar_j = Q( b_j lambda + h a_{j+1,j} zbar_{j+1} )
    auto make_kbar = [&](int j) __attribute__((always_inline)) {
      const f32x4 cf = *(const RAMPDE_LDS f32x4*)(lds.coef + j * 4);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        float lam[4], v[4];
        unpack4<T>(lamq[mt], lam);
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = fmaf(h, cf[0] * zf[mt][r], cf[1] * lam[r]);
        const uint2 q = pack4<T>(v);
        track(big, q);
        lds_store_u2(&lds.z[(mt * 16 + lm) * Sh::LDZ + ns], q);
        store_word(KBART + j * stage_bytes, off_s + mt * 128, q, mask[mt]);
      }
    };
    auto start = [&]() __attribute__((always_inline)) {
      big = 0;
      t_dt = t_dh = 0.f;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        float sa[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) sa[r] = ex.S * av[mt][r];
        lamq[mt] = pack4<T>(sa);
        track(big, lamq[mt]);
#pragma unroll
        for (int r = 0; r < 4; ++r) da[mt][r] = zf[mt][r] = 0.f;
      }
      make_kbar(s - 1);
      __syncthreads();
    };
    start();

    f32x4 acc[TPW][MT];
    auto store_delta = [&](int j, int l) __attribute__((always_inline)) {
      lds_u16* io = tile(l);
      char* gout = (char*)(g.DELTAT[l] + set_off) + j * stage_bytes;
#pragma unroll
      for (int t = 0; t < TPW; ++t)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          float a[4], v[4];
          unpack4<T>(act[l][t][mt], a);
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = acc[t][mt][r] * (1.f - a[r] * a[r]);
          uint2 q = pack4<T>(v);
          q.x &= mask[mt];
          q.y &= mask[mt];
          if constexpr (TG) {
            if (l == 0) {
              float dv[4];
              unpack4<T>(q, dv);
              const float4 tv = lds_load_f4(&lds.wt[nh + t * 16]);
              const float tb = dv[0] * tv.x + dv[1] * tv.y + dv[2] * tv.z + dv[3] * tv.w;
              t_dt += tb;
              t_dh = fmaf(lds.coef[j * 4 + 2], tb, t_dh);
            }
          }
          lds_store_u2(&io[(mt * 16 + lm) * Sh::LDP + nh + t * 16], q);
          *reinterpret_cast<uint2*>(gout + t * tile_bytes + (off_h + mt * 128)) = q;
          track(big, q);
        }
    };
    bool open = it > 0 && g.detect;  // the outcome of the step before is not known yet
#pragma unroll 1
    for (int j = s - 1; j >= 0;) {
      // (the next stage's activations: see StepRows)
      uint2 act_next[L - 1][TPW][MT];
      fetch_act(act_next, j > 0 ? step : step_next, j > 0 ? j - 1 : s - 1);
      zero_acc(acc);
      resident_mma<T, MT>(acc, wb.first, lds.z, Sh::LDZ, lane);
      store_delta(j, L - 2);
#pragma unroll
      for (int m = Sh::MIDS - 1; m >= 0; --m) {
        __syncthreads();
        zero_acc(acc);
        resident_mma<T, MT>(acc, wb.mid[m], tile(m + 1), Sh::LDP, lane);
        store_delta(j, m);
      }
      __syncthreads();
      f32x4 zs[MT];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) zs[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
      resident_mma_state<T, MT>(zs, wb.last, tile(0), Sh::LDP, lane);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const float v[4] = {zs[mt][0], zs[mt][1], zs[mt][2], zs[mt][3]};
        uint2 q = pack4<T>(v);
        q.x &= mask[mt];
        q.y &= mask[mt];
        track(big, q);
        unpack4<T>(q, zf[mt]);
#pragma unroll
        for (int r = 0; r < 4; ++r) da[mt][r] += zf[mt][r];
        if constexpr (TG) {
          if (j > 0) {
            const float a = lds.coef[j * 4 + 3];
            float kl[4];
            unpack4<T>(j == 1 ? k[0][mt] : j == 2 ? k[1][mt] : k[2][mt], kl);
#pragma unroll
            for (int r = 0; r < 4; ++r) t_dh = fmaf(a * kl[r], zf[mt][r], t_dh);
          }
        }
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
      if (j > 0) {
        make_kbar(j - 1);
        __syncthreads();
      }
#pragma unroll
      for (int l = 0; l < L - 1; ++l)
#pragma unroll
        for (int t = 0; t < TPW; ++t)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) {
            asm volatile("" : "+v"(act_next[l][t][mt].x), "+v"(act_next[l][t][mt].y));
            act[l][t][mt] = act_next[l][t][mt];
          }
      --j;
    }
    if (rejected) break;

    // ---- a <- a + (h / S) sum_j zbar_j (+ running-cost cotangent), fp32
    const float hs = h / ex.S;
    if constexpr (TG) {
#pragma unroll
      for (int j = 0; j < kResidentStages; ++j)
        if (j < s) {
          const float b = lds.coef[j * 4 + 1];
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) {
            float kf[4];
            unpack4<T>(k[j][mt], kf);
#pragma unroll
            for (int r = 0; r < 4; ++r) t_phia = fmaf(b * kf[r], av[mt][r], t_phia);
          }
        }
      block_sum2(fmaf(hs, t_dt - t_dh, -t_phia), fmaf(hs, t_dh, t_phia), g.tpart + 2 * ((size_t)it * gridDim.x + blockIdx.x));
    }
    unsigned bits = 0;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      float gy[4] = {0.f, 0.f, 0.f, 0.f};
      if (g.gys) load4f(g.gys - (int64_t)it * g.gys_stride, row0 + mt * 16 + lm, g.R, ns, g.d, gy);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        a_old[mt][r] = av[mt][r];
        av[mt][r] = fmaf(hs, da[mt][r], av[mt][r]) + gy[r];
        if (g.round_incr & 2) av[mt][r] = Low<T>::to_f32(Low<T>::from_f32(av[mt][r]));
        const unsigned bb = __builtin_bit_cast(unsigned, fabsf(av[mt][r]));
        if (mask[mt] && ns + r < g.d) bits = max(bits, bb);
      }
    }
    if (g.detect) ex.post(g, step, bits, tracked_nonfinite<T>(big));
    else ex.template decide<T>(g, step);
  }
  if (g.detect && !rejected) rejected = !ex.template decide<T>(g, g.step - g.nsteps + 1);
  if (ex.stalled) return;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    // (a rejected step leaves the adjoint as it was before it)
    if (rejected) {
#pragma unroll
      for (int r = 0; r < 4; ++r) av[mt][r] = a_old[mt][r];
    }
    store4f(g.a_out, row0 + mt * 16 + lm, g.R, ns, g.d, av[mt]);
  }
  ex.finish(g);
}

// ---------------------------------------------------------------------------------------
// A group of adjoint steps of a tile.  PHASED: the forward and the transposed slices do not fit in the registers
// together (four layers of 256): each phase of a step loads its own.
template <class T, int L, int HP, int MT, bool TG, bool PHASED>
__global__ __launch_bounds__(256, HP == 256 ? 1 : 2) void mlp_adjoint_resident(ResidentArgs ra) {
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  using Sh = ResidentShape<L, HP>;
  const FusedArgs& g = ra.f;
  if (g.ctl->poison) return;
  ResidentLds<L, HP> lds((lds_u16*)smem, MT);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lm = lane & 15, lq = lane >> 4;
  constexpr int TPW = Sh::TPW, TM = 16 * MT;
  const int64_t row0 = (int64_t)blockIdx.x * TM;
  const int s = g.s;
  const int ns = wave * 16 + lq * 4, nh = wave * TPW * 16 + lq * 4;

  // (the transposed last slice in LDS where it fits beside the activations: 32 registers for the rest)
  constexpr bool LDS_LAST = HP >= 128 && L >= 3 && MT == 1;
  ResidentWeights<L, HP> wf;
  ResidentWeights<L, HP, LDS_LAST> wb;
  wb.last_lds = lds.tiles + (size_t)s * (L - 1) * TM * Sh::LDP;
  if constexpr (!PHASED) {
    wf.template load<true, 8>(g, wave, lane);
    wb.template load<false, 6>(g, wave, lane);
  }
  lds.fill(g);
  StepExchange ex(ra);
  float av[MT][4], a_old[MT][4];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) load4f(g.a_in, row0 + mt * 16 + lm, g.R, ns, g.d, av[mt]);
  uint2 yh_next[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
    yh_next[mt] = load_state(g.ckpt + (size_t)g.step * g.ckpt_stride, row0 + mt * 16 + lm, g.R, ns, g.d);
  const StepRows rows{lds.rows};
  rows.put(0, rows.load(g, g.step));
  // lane offsets (bytes) into the feature-group-major arrays: hidden and state columns, and the batch-row masks
  const uint32_t off_h = (uint32_t)(((size_t)(nh >> 2) * g.ldk + row0 + lm) * 8);
  const uint32_t off_s = (uint32_t)(((size_t)(ns >> 2) * g.ldk + row0 + lm) * 8);
  const size_t tile_bytes = (size_t)g.ldk * 32;  // 16 columns further
  const size_t stage_bytes = (size_t)g.Rp * 8;
  uint32_t mask[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) mask[mt] = row0 + mt * 16 + lm < g.R ? 0xFFFFFFFFu : 0u;

  // activations (later: cotangents, in place) of stage j, hidden layer l
  auto tile = [&](int j, int l) __attribute__((always_inline)) { return lds.tiles + (size_t)(j * (L - 1) + l) * TM * Sh::LDP; };

  bool rejected = false;
#pragma unroll 1
  for (int it = 0; it < g.nsteps; ++it) {
    const int step = g.step - it;
    const int64_t set_off = (int64_t)(step % g.nsets) * g.set_stride;
    char* const ZT = (char*)(g.ZT + set_off);
    char* const KBART = (char*)(g.KBART + set_off);
    uint2 yhat[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) yhat[mt] = yh_next[mt];
    const int step_next = it + 1 < g.nsteps ? step - 1 : step;
    if constexpr (PHASED) wf.template load<true, MT == 1 ? 14 : 12, true>(g, wave, lane);
    float t_phia = 0.f, t_dt = 0.f, t_dh = 0.f;

    // ---- stage recomputation, keeping inputs and activations
    uint2 k0[MT], k1[MT], k2[MT];  // (slopes: for the time-grid terms only)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      if constexpr (TG) k0[mt] = k1[mt] = k2[mt] = make_uint2(0u, 0u);
      lds_store_u2(&lds.z[(mt * 16 + lm) * Sh::LDZ + ns], yhat[mt]);
      store_word(ZT, off_s + mt * 128, yhat[mt], mask[mt]);
    }
    __syncthreads();

    auto store_act = [&](const f32x4 (&acc)[TPW][MT], int j, int l) __attribute__((always_inline)) {
      lds_u16* out = tile(j, l);
      char* gout = (char*)(g.ACTT[l] + set_off) + j * stage_bytes;
#pragma unroll
      for (int t = 0; t < TPW; ++t)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          float v[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = tanh_fast(acc[t][mt][r]);
          const uint2 q = pack4<T>(v);
          lds_store_u2(&out[(mt * 16 + lm) * Sh::LDP + nh + t * 16], q);
          store_word(gout + t * tile_bytes, off_h + mt * 128, q, mask[mt]);
        }
    };
    f32x4 acc[TPW][MT];
    __syncthreads();
    const float h = rows.h(it);
    init_acc_time(acc, lds.bias, lds.wt, rows.tau(it, 0), nh);
#pragma unroll 1
    for (int j = 0; j < s; ++j) {
      const bool last_stage = j + 1 == s;
      // (the next step's row and stored state: see StepRows)
      const float row_next = rows.load(g, step_next);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        yh_next[mt] = load_state(g.ckpt + (size_t)step_next * g.ckpt_stride, row0 + mt * 16 + lm, g.R, ns, g.d);
      resident_mma<T, MT>(acc, wf.first, lds.z, Sh::LDZ, lane);
      store_act(acc, j, 0);
      rows.put(it + 1, row_next);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) asm volatile("" : "+v"(yh_next[mt].x), "+v"(yh_next[mt].y));
      f32x4 ks[MT];
      const f32x4 bl = *(const RAMPDE_LDS f32x4*)(lds.bias + (L - 1) * HP + ns);
      const f32x4 cf = *(const RAMPDE_LDS f32x4*)(lds.coef + j * 4);
#pragma unroll
      for (int m = 0; m < Sh::MIDS; ++m) {
        init_acc(acc, lds.bias + (m + 1) * HP, nh);
        __syncthreads();
        resident_mma<T, MT>(acc, wf.mid[m], tile(j, m), Sh::LDP, lane);
        store_act(acc, j, m + 1);
      }
      if (last_stage && !TG) break;  // (the slope of the last stage is not needed)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) ks[mt] = bl;
      __syncthreads();
      resident_mma_state<T, MT>(ks, wf.last, tile(j, L - 2), Sh::LDP, lane);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const float v[4] = {ks[mt][0], ks[mt][1], ks[mt][2], ks[mt][3]};
        const uint2 q = pack4<T>(v);
        float kf[4], yh[4], z[4];
        unpack4<T>(q, kf);
        if constexpr (TG) {
#pragma unroll
          for (int r = 0; r < 4; ++r) t_phia = fmaf(cf[1] * kf[r], av[mt][r], t_phia);
          keep_if(j == 0, k0[mt], q);
          keep_if(j == 1, k1[mt], q);
          keep_if(j == 2, k2[mt], q);
        }
        if (!last_stage) {
          unpack4<T>(yhat[mt], yh);
#pragma unroll
          for (int r = 0; r < 4; ++r) z[r] = fmaf(h, cf[0] * kf[r], yh[r]);
          const uint2 zq = pack4<T>(z);
          lds_store_u2(&lds.z[(mt * 16 + lm) * Sh::LDZ + ns], zq);
          store_word(ZT + (j + 1) * stage_bytes, off_s + mt * 128, zq, mask[mt]);
        }
      }
      if (!last_stage) init_acc_time(acc, lds.bias, lds.wt, rows.tau(it, j + 1), nh);
      __syncthreads();
    }

    // ---- the previous step's outcome: its scale is needed from here on
    if (it > 0 && !ex.template decide<T>(g, step + 1)) {
      rejected = true;
      break;
    }
    if constexpr (PHASED) wb.template load<false, MT == 1 ? 14 : 12, true>(g, wave, lane);

    // ---- cotangent chain, stages in reverse (eq. (vjp) pushed through the stage recursion)
    uint32_t big = 0;  // largest magnitudes of the step's cotangents
    uint2 lamq[MT];
    float zf[MT][4];  // cotangent of the stage input behind the slope at hand
    float da[MT][4];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      float sa[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) sa[r] = ex.S * av[mt][r];
      lamq[mt] = pack4<T>(sa);
      track(big, lamq[mt]);
#pragma unroll
      for (int r = 0; r < 4; ++r) da[mt][r] = zf[mt][r] = 0.f;
    }
    // cotangent of the slope of stage j:  kbar_j = Q( b_j lambda + h a_{j+1,j} zbar_{j+1} )
    auto make_kbar = [&](int j) __attribute__((always_inline)) {
      const f32x4 cf = *(const RAMPDE_LDS f32x4*)(lds.coef + j * 4);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        float lam[4], v[4];
        unpack4<T>(lamq[mt], lam);
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = fmaf(h, cf[0] * zf[mt][r], cf[1] * lam[r]);
        const uint2 q = pack4<T>(v);
        track(big, q);
        lds_store_u2(&lds.z[(mt * 16 + lm) * Sh::LDZ + ns], q);
        store_word(KBART + j * stage_bytes, off_s + mt * 128, q, mask[mt]);
      }
    };
    // (the stage input tile was last read by the last stage's first contraction: a barrier ago, except with two layers)
    if (L == 2 && !TG) __syncthreads();
    make_kbar(s - 1);
    __syncthreads();

    // activations at the lane's own elements of a tile (their cotangents take their place)
    auto load_own = [&](uint2 (&q)[TPW][MT], const lds_u16* io) __attribute__((always_inline)) {
#pragma unroll
      for (int t = 0; t < TPW; ++t)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) q[t][mt] = lds_load_u2(&io[(mt * 16 + lm) * Sh::LDP + nh + t * 16]);
    };
    auto store_delta = [&](const f32x4 (&acc)[TPW][MT], const uint2 (&act)[TPW][MT], int j, int l) __attribute__((always_inline)) {
      lds_u16* io = tile(j, l);
      char* gout = (char*)(g.DELTAT[l] + set_off) + j * stage_bytes;
#pragma unroll
      for (int t = 0; t < TPW; ++t)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          float a[4], v[4];
          unpack4<T>(act[t][mt], a);
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = acc[t][mt][r] * (1.f - a[r] * a[r]);
          uint2 q = pack4<T>(v);
          q.x &= mask[mt];
          q.y &= mask[mt];
          if constexpr (TG) {
            if (l == 0) {
              float dv[4];
              unpack4<T>(q, dv);
              const float4 tv = lds_load_f4(&lds.wt[nh + t * 16]);
              const float tb = dv[0] * tv.x + dv[1] * tv.y + dv[2] * tv.z + dv[3] * tv.w;
              t_dt += tb;
              t_dh = fmaf(lds.coef[j * 4 + 2], tb, t_dh);
            }
          }
          lds_store_u2(&io[(mt * 16 + lm) * Sh::LDP + nh + t * 16], q);
          *reinterpret_cast<uint2*>(gout + t * tile_bytes + (off_h + mt * 128)) = q;
          track(big, q);
        }
    };
#pragma unroll 1
    for (int j = s - 1; j >= 0; --j) {
      uint2 act[TPW][MT];
      load_own(act, tile(j, L - 2));
      zero_acc(acc);
      resident_mma<T, MT>(acc, wb.first, lds.z, Sh::LDZ, lane);
      store_delta(acc, act, j, L - 2);
#pragma unroll
      for (int m = Sh::MIDS - 1; m >= 0; --m) {
        load_own(act, tile(j, m));
        __syncthreads();
        zero_acc(acc);
        resident_mma<T, MT>(acc, wb.mid[m], tile(j, m + 1), Sh::LDP, lane);
        store_delta(acc, act, j, m);
      }
      u16x8 wl[1][Sh::KBH];
      fetch_last(wl, wb, wave, lane);
      __syncthreads();
      f32x4 zs[MT];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) zs[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
      resident_mma_state<T, MT>(zs, wl, tile(j, 0), Sh::LDP, lane);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const float v[4] = {zs[mt][0], zs[mt][1], zs[mt][2], zs[mt][3]};
        uint2 q = pack4<T>(v);
        q.x &= mask[mt];
        q.y &= mask[mt];
        track(big, q);
        unpack4<T>(q, zf[mt]);
#pragma unroll
        for (int r = 0; r < 4; ++r) da[mt][r] += zf[mt][r];
        if constexpr (TG) {
          if (j > 0) {
            const float a = lds.coef[j * 4 + 3];
            float kl[4];
            unpack4<T>(j == 1 ? k0[mt] : j == 2 ? k1[mt] : k2[mt], kl);
#pragma unroll
            for (int r = 0; r < 4; ++r) t_dh = fmaf(a * kl[r], zf[mt][r], t_dh);
          }
        }
      }
      if (j > 0) {
        make_kbar(j - 1);
        __syncthreads();
      }
    }

    // ---- a <- a + (h / S) sum_j zbar_j (+ running-cost cotangent), fp32
    const float hs = h / ex.S;
    if constexpr (TG)
      block_sum2(fmaf(hs, t_dt - t_dh, -t_phia), fmaf(hs, t_dh, t_phia), g.tpart + 2 * ((size_t)it * gridDim.x + blockIdx.x));
    unsigned bits = 0;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      float gy[4] = {0.f, 0.f, 0.f, 0.f};
      if (g.gys) load4f(g.gys - (int64_t)it * g.gys_stride, row0 + mt * 16 + lm, g.R, ns, g.d, gy);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        a_old[mt][r] = av[mt][r];
        av[mt][r] = fmaf(hs, da[mt][r], av[mt][r]) + gy[r];
        if (g.round_incr & 2) av[mt][r] = Low<T>::to_f32(Low<T>::from_f32(av[mt][r]));
        const unsigned bb = __builtin_bit_cast(unsigned, fabsf(av[mt][r]));
        if (mask[mt] && ns + r < g.d) bits = max(bits, bb);
      }
    }
    if (g.detect) ex.post(g, step, bits, tracked_nonfinite<T>(big));
    else ex.template decide<T>(g, step);
  }
  if (g.detect && !rejected) rejected = !ex.template decide<T>(g, g.step - g.nsteps + 1);
  if (ex.stalled) return;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    // (a rejected step leaves the adjoint as it was before it)
    if (rejected) {
#pragma unroll
      for (int r = 0; r < 4; ++r) av[mt][r] = a_old[mt][r];
    }
    store4f(g.a_out, row0 + mt * 16 + lm, g.R, ns, g.d, av[mt]);
  }
  ex.finish(g);
}

}  // namespace rampde
