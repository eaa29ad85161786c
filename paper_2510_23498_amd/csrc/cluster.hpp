// Dense networks with 512- to 1024-wide hidden layers and a batch that leaves most of the device idle in row tiles:
// CLUSTERS of workgroups that share a row tile.  (1024 rows of a 1024-wide network are 64 tiles of 16 rows, and each
// streams 3.15 MB of weights from its XCD's L2 per velocity evaluation at the 57 B/clk that a compute unit gets: 22.9 us.)
//
// A cluster is C = HP / 64 workgroups on one XCD.  Member m owns 64 output features of every hidden layer (and 32 of
// the state for one of the cluster's row tiles) and keeps its slices of ALL weight matrices in registers for the whole
// launch; what moves are activations.  Four wavefronts split the contraction: wavefront w holds the quarter w of the
// input features, reads exactly that quarter of the previous layer's activations, and the four partial sums of a 32-row
// tile are folded through LDS, each wavefront finishing a quarter of the member's outputs.
//
// Exchange.  A finished quarter is one 1 KB matrix-instruction operand fragment (the contraction order within 16 features
// is permuted to the accumulators' order, so a lane's results ARE its 16 bytes of the fragment), written by plain stores
// to the XCD's L2, and read back by loads that bypass the compute unit's own cache.  There are no flags: a buffer is
// filled with a word that no result has (all ones; results are kept off it) and a reader repeats its loads until none is
// left.  So a layer costs one trip through L2 instead of three (store, arrival counter, gather).  Every buffer exists
// kClusterRing times: a member clears its part of the buffers of evaluation e during evaluation e + 1, once that one's
// stage input is complete (which nobody publishes before everybody has read evaluation e), two evaluations before they are
// used again.  The clear lands in time: a wavefront's loads and stores complete in the order of issue, so that its wait
// for the stage input of e + 2 has retired the clear before it publishes anything of e + 2, and nobody looks into the
// buffers of e + 3 before all of e + 2 has been published.
// With several row tiles of 32 per cluster, one tile's exchange runs beside the next one's contraction.
//
//   mlp_forward_cluster : Algorithm 1, as many steps per launch as take about 3 ms (a launch holds the whole device; other
//                         streams' kernels get in between two of them), the fp32 state in yN from one to the next
//   mlp_chain_cluster   : Algorithm 2 for a group of steps whose stages have been recomputed (mlp_recompute_fused): the
//                         cotangent chain, the fp32 adjoint and the scale decisions (StepExchange of resident.hpp)
//
// Measured, 256 -> 1024 -> 1024 -> 256, f16, 1024 rows, 256 RK4 steps: forward 24.2 -> 7.7 ms (7.6 us per evaluation of 64
// rows, 5.7 of 32), cotangent chain 48 -> 10.3 ms, pass 95.6 -> 28.6 ms (72.3 with the recomputation ahead alone).  A phase
// (gather, contraction, fold, epilogue) of 64 rows takes 2 to 3 us: 128 KB from L2 per compute unit in 1.6 us, 0.85 us of
// matrix instructions, two LDS folds, and a trip through L2 of about 1 us that the other row tile hides in part.  Stores
// that go through to memory instead of the XCD's own L2 (workgroups anywhere on the device) made an exchange 3.8 us
// instead of 2.2.
//
// Members find each other at run time: a workgroup takes a ticket of the XCD that it runs on.  Waits end after
// kWaitTicks (the workgroups of a launch did not run at the same time), and a workgroup that finds its XCD's share of the
// launch taken gives up at once (the workgroups were not spread evenly over the XCDs): the launch then writes `stalled`
// and no result that is not overwritten, and the row-tile kernels redo its work: behind it on the stream, as launches that
// do nothing otherwise (forward, fixed scale), or by way of the host (under overflow detection).
#pragma once
#include "resident.hpp"

namespace rampde {

constexpr int kClusterRing = 3;
constexpr uint32_t kUnwritten = 0xFFFFFFFFu;

// sizes shared by host and device
template <int HP, int L, int NTL, int RTN>
struct ClusterShape {
  static constexpr int C = HP / 64;             // members
  static constexpr int KS1 = NTL, KSH = HP / 64;  // contraction steps of 16 per wavefront: over the state, over a hidden layer
  static constexpr int MIDS = L - 2;
  static constexpr int CTS = 2 * NTL;           // column tiles of 32 of the state
  // row tiles whose state-shaped passes run side by side (a power of two)
  static constexpr int APC = C / CTS >= 4 && RTN >= 4 ? 4 : C / CTS >= 2 && RTN >= 2 ? 2 : 1;
  static constexpr int NU = RTN / APC;          // ... one after the other in one member
  static_assert(APC >= 1 && RTN % APC == 0, "every state tile has a member");
  static constexpr int FRAGS = 2 * KS1 + MIDS * 2 * KSH + KSH;  // weight fragments of a wavefront
  static constexpr int ZF = 4 * KS1 * RTN, HF = 4 * KSH * RTN;  // fragments of an exchanged stage input / hidden layer
  static constexpr int SLOT = ZF + (L - 1) * HF;                // ... of one evaluation
  static constexpr size_t exchange_bytes = (size_t)kClusterRing * SLOT * 1024;  // per cluster
};

struct ClusterArgs {
  ResidentArgs r;          // (r.f: as for the row-tile kernels; r.slots: [N][clusters * C])
  const u16x8* W;          // [C][4 wavefronts][FRAGS][64 lanes]
  uint32_t* exchange;      // [clusters][kClusterRing][SLOT] KB
  unsigned* tickets;       // [8], zero at the start of the launch
  int* stalled;            // raised when a wait ran out; raised before the launch: nothing is done
  int clusters;
  int budget;              // evaluations of this launch after which it is given up (see RAMPDE_NO_WAITS_AFTER)
};

// theta (fp32) -> the wavefronts' weight fragments (transposed: as the cotangent chain multiplies by them)
struct ClusterCastLayer {
  const float* W;
  const float* b;
  float* bias_f;
  float* wt_f;
  int out, in, in_full, has_time, Npad;
};
struct ClusterCast {
  ClusterCastLayer layer[4];
  u16x8* W;
  int L, C, NTL, KSH, frags, transposed, write_bias;
};
template <class T>
__global__ __launch_bounds__(256) void cast_cluster_fragments(ClusterCast c) {
  const int lane = threadIdx.x & 63, lh = lane >> 5, lr = lane & 31;
  const int id = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (id < c.C * 4 * c.frags) {
    const int f = id % c.frags, wave = (id / c.frags) & 3, me = id / c.frags / 4;
    const int n1 = 2 * c.NTL, nm = 2 * c.KSH;
    int q, ks, ksn, n;  // position in the chain of contractions, contraction step, steps per wavefront, output feature
    if (f < n1) {
      q = 0; ksn = c.NTL; ks = f % ksn;
    } else if (f < n1 + (c.L - 2) * nm) {
      q = 1 + (f - n1) / nm; ksn = c.KSH; ks = (f - n1) % nm % ksn;
    } else {
      q = c.L - 1; ksn = c.KSH; ks = f - n1 - (c.L - 2) * nm;
    }
    if (q < c.L - 1) {
      // local column quarter p of the wavefront is finished by wavefront (wave + p) % 4
      const int ct = q == 0 ? f / ksn : (f - n1) % nm / ksn, lc = ct * 32 + lr;
      n = me * 64 + 16 * ((wave + lc / 16) & 3) + lc % 16;
    } else {
      n = me % (2 * c.NTL) * 32 + 8 * ((wave + lr / 8) & 3) + lr % 8;
    }
    const ClusterCastLayer& y = c.layer[c.transposed ? c.L - 1 - q : q];
    u16x8 v;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int k = (wave * ksn + ks) * 16 + 4 * lh + e + (e >= 4 ? 4 : 0);
      float x = 0.f;
      if (c.transposed) {
        if (k < y.out && n < y.in) x = y.W[(size_t)k * y.in_full + n];
      } else {
        if (n < y.out && k < y.in) x = y.W[(size_t)n * y.in_full + k];
      }
      v[e] = Low<T>::from_f32(x);
    }
    c.W[(size_t)id * 64 + lane] = v;
  }
  if (c.write_bias) {
    const int i = blockIdx.x * 256 + threadIdx.x, l = i / 1024, n = i % 1024;
    if (l < c.L && n < c.layer[l].Npad) {
      const ClusterCastLayer& y = c.layer[l];
      y.bias_f[n] = n < y.out ? Low<T>::to_f32(Low<T>::from_f32(y.b[n])) : 0.f;
      y.wt_f[n] = n < y.out && y.has_time ? Low<T>::to_f32(Low<T>::from_f32(y.W[(size_t)n * y.in_full + y.in])) : 0.f;
    }
  }
}

typedef uint32_t u32x4c __attribute__((ext_vector_type(4)));

// before a launch: nothing has been written, no ticket taken (skew: the first XCD's tickets start there, as if it had been
// given that many workgroups more)
__global__ __launch_bounds__(256) inline void cluster_reset(u32x4c* x, size_t n, unsigned* tickets, int* stalled, unsigned skew) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) x[i] = u32x4c{kUnwritten, kUnwritten, kUnwritten, kUnwritten};
  if (blockIdx.x == 0 && threadIdx.x < 8) tickets[threadIdx.x] = threadIdx.x == 0 ? skew : 0u;
  if (stalled && blockIdx.x == 0 && threadIdx.x == 0) *stalled = 0;
}

// What both kernels share: the member's place, its weights, the exchange and the passes.
template <class T, int HP, int L, int NTL, int RTN>
struct ClusterEngine {
  using Sh = ClusterShape<HP, L, NTL, RTN>;
  static constexpr int KS1 = Sh::KS1, KSH = Sh::KSH, MIDS = Sh::MIDS;
  int lane, wave, lr, lh, me, cl;
  int unit_ct, unit_rt;  // the member's state tile (its first row tile), unit_rt < 0: none
  __amdgpu_buffer_rsrc_t xr;
  int* stalled;
  unsigned long long ticks;
  lds_f32* red;   // [2][4 destinations][3][2][64 lanes] x 16 B: partial sums
  RAMPDE_LDS int* dead;
  bool lost = false;  // setup gave the launch up
  int par = 0;    // half of `red` in use
  u16x8 w1[2][KS1];
  u16x8 wm[MIDS > 0 ? MIDS : 1][2][KSH];
  u16x8 wl[KSH];

  // false: this workgroup has no part in the launch
  __device__ __forceinline__ bool setup(const ClusterArgs& a, lds_f32* red_, RAMPDE_LDS int* sh) {
    lane = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    lr = lane & 31;
    lh = lane >> 5;
    red = red_;
    dead = sh;
    stalled = a.stalled;
    ticks = a.r.wait_ticks;
    if (threadIdx.x == 0) {
      // XCC_ID: the XCD that the workgroup runs on
      const int xcd = __builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11)) & 7;
      sh[1] = xcd;
      sh[2] = (int)atomicAdd(a.tickets + xcd, 1u);
      sh[0] = __hip_atomic_load(a.stalled, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    const int rank = __builtin_amdgcn_readfirstlane(sh[2]);
    cl = __builtin_amdgcn_readfirstlane(sh[1]) + 8 * (rank / Sh::C);
    me = rank % Sh::C;
    if (sh[0]) return false;
    // (more workgroups here than an XCD's share: others have fewer, and a cluster that nobody joins has nobody to notice)
    lost = a.budget <= 0 || rank >= (a.clusters + 7) / 8 * Sh::C;
    if (lost) give_up();
    if (lost || cl >= a.clusters) return false;
    unit_ct = me % Sh::CTS;
    unit_rt = me / Sh::CTS < Sh::APC ? me / Sh::CTS : -1;
    xr = __builtin_amdgcn_make_buffer_rsrc((char*)a.exchange + (size_t)cl * Sh::exchange_bytes, 0, (int)Sh::exchange_bytes, 0x00020000);
    const glb_u16x8* w = (const glb_u16x8*)a.W + (size_t)(me * 4 + wave) * Sh::FRAGS * 64 + lane;
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
#pragma unroll
      for (int ks = 0; ks < KS1; ++ks) w1[ct][ks] = w[(size_t)(ct * KS1 + ks) * 64];
#pragma unroll
    for (int m = 0; m < MIDS; ++m)
#pragma unroll
      for (int ct = 0; ct < 2; ++ct)
#pragma unroll
        for (int ks = 0; ks < KSH; ++ks) wm[m][ct][ks] = w[(size_t)(2 * KS1 + (m * 2 + ct) * KSH + ks) * 64];
#pragma unroll
    for (int ks = 0; ks < KSH; ++ks) wl[ks] = w[(size_t)(2 * KS1 + MIDS * 2 * KSH + ks) * 64];
#pragma unroll
    for (int m = 0; m < MIDS; ++m)
#pragma unroll
      for (int ct = 0; ct < 2; ++ct)
#pragma unroll
        for (int ks = 0; ks < KSH; ++ks) asm volatile("" : "+a"(wm[m][ct][ks]));
    return true;
  }

  // fragment numbers within the exchange buffer of evaluation e (modulo the ring): stage input, output of hidden layer q
  __device__ __forceinline__ int zfrag(int e, int ks, int rt) const { return (e % kClusterRing) * Sh::SLOT + ks * RTN + rt; }
  __device__ __forceinline__ int hfrag(int e, int q, int ks, int rt) const {
    return (e % kClusterRing) * Sh::SLOT + Sh::ZF + q * Sh::HF + ks * RTN + rt;
  }
  // loads that bypass the compute unit's cache (sc1): they see what the XCD's L2 holds
  __device__ __forceinline__ u16x8 take(int frag) const {
    return __builtin_bit_cast(u16x8, __builtin_amdgcn_raw_buffer_load_b128(xr, lane * 16, frag * 1024, 16));
  }
  __device__ __forceinline__ void publish16(int frag, uint2 a, uint2 b) const {
    const u32x4c v = {min(a.x, kUnwritten - 1), min(a.y, kUnwritten - 1), min(b.x, kUnwritten - 1), min(b.y, kUnwritten - 1)};
    __builtin_amdgcn_raw_buffer_store_b128(v, xr, lane * 16, frag * 1024, 0);
  }
  __device__ __forceinline__ void publish8(int frag, int half, uint2 a) const {
    const u32x2 v = {min(a.x, kUnwritten - 1), min(a.y, kUnwritten - 1)};
    __builtin_amdgcn_raw_buffer_store_b64(v, xr, lane * 16 + half * 8, frag * 1024, 0);
  }
  __device__ __forceinline__ void clear16(int frag) const {
    const u32x4c v = {kUnwritten, kUnwritten, kUnwritten, kUnwritten};
    __builtin_amdgcn_raw_buffer_store_b128(v, xr, lane * 16, frag * 1024, 0);
  }
  __device__ __forceinline__ void clear8(int frag, int half) const {
    const u32x2 v = {kUnwritten, kUnwritten};
    __builtin_amdgcn_raw_buffer_store_b64(v, xr, lane * 16 + half * 8, frag * 1024, 0);
  }
  __device__ __forceinline__ void gather_z(u16x8 (&f)[KS1], int e, int rt) const {
    asm volatile("" ::: "memory");
#pragma unroll
    for (int ks = 0; ks < KS1; ++ks) f[ks] = take(zfrag(e, wave * KS1 + ks, rt));
  }
  __device__ __forceinline__ void gather_h(u16x8 (&f)[KSH], int e, int q, int rt) const {
    asm volatile("" ::: "memory");
#pragma unroll
    for (int ks = 0; ks < KSH; ++ks) f[ks] = take(hfrag(e, q, wave * KSH + ks, rt));
  }
  template <int N>
  __device__ __forceinline__ static bool missing(const u16x8 (&f)[N], int k0, int k1) {
    uint32_t m = 0;
#pragma unroll
    for (int ks = 0; ks < N; ++ks)
      if (ks >= k0 && ks < k1) {
        const u32x4c v = __builtin_bit_cast(u32x4c, f[ks]);
        m = max(max(m, max(v[0], v[1])), max(v[2], v[3]));
      }
    return __any(m == kUnwritten);
  }
  // repeats the loads of contraction steps k0 .. k1 until they have all been written; again(ks): the step's fragment number
  template <int N, class Again>
  __device__ __forceinline__ void complete(u16x8 (&f)[N], int k0, int k1, Again again) {
    unsigned long long t0 = 0;
    while (missing(f, k0, k1)) {
      const unsigned long long now = wall_clock64();
      if (t0 == 0) t0 = now;
      if (now - t0 >= ticks) {
        *dead = 1;
        break;
      }
      asm volatile("" ::: "memory");
#pragma unroll
      for (int ks = 0; ks < N; ++ks)
        if (ks >= k0 && ks < k1) f[ks] = take(again(ks));
    }
  }

  // partial sums of 64 features x 32 rows -> the lane's 8 finished values (features me * 64 + 16 wave + 4 lh + 0..3, + 8);
  // mid(): after the partial sums are on their way.  false: a wait ran out
  template <class Mid>
  __device__ __forceinline__ bool fold_hidden(f32x16 (&acc)[2], float (&v)[8], Mid mid) {
    RAMPDE_LDS f32x4* const base = (RAMPDE_LDS f32x4*)red + par * (4 * 3 * 2 * 64) + lane;
#pragma unroll
    for (int q = 1; q < 4; ++q)
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const int i = (q & 1) * 8 + p * 4;
        base[((((wave + q) & 3) * 3 + q - 1) * 2 + p) * 64] = f32x4{acc[q >> 1][i], acc[q >> 1][i + 1], acc[q >> 1][i + 2], acc[q >> 1][i + 3]};
      }
    mid();
    __syncthreads();
    const bool ok = *dead == 0;
    f32x4 s[2] = {{acc[0][0], acc[0][1], acc[0][2], acc[0][3]}, {acc[0][4], acc[0][5], acc[0][6], acc[0][7]}};
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int p = 0; p < 2; ++p) s[p] += base[((wave * 3 + q) * 2 + p) * 64];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = s[i >> 2][i & 3];
    par ^= 1;
    return ok;
  }
  // ... of 32 state features x 32 rows -> 4 values (features unit_ct * 32 + 8 wave + 4 lh + 0..3)
  __device__ __forceinline__ bool fold_state(const f32x16& acc, float (&v)[4]) {
    RAMPDE_LDS f32x4* const base = (RAMPDE_LDS f32x4*)red + par * (4 * 3 * 2 * 64) + lane;
#pragma unroll
    for (int q = 1; q < 4; ++q)
      base[(((wave + q) & 3) * 3 + q - 1) * 2 * 64] = f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
    __syncthreads();
    const bool ok = *dead == 0;
    f32x4 s = {acc[0], acc[1], acc[2], acc[3]};
#pragma unroll
    for (int q = 0; q < 3; ++q) s += base[(wave * 3 + q) * 2 * 64];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = s[i];
    par ^= 1;
    return ok;
  }
  template <int N>
  __device__ __forceinline__ static void zero(f32x16 (&acc)[N]) {
#pragma unroll
    for (int c = 0; c < N; ++c)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[c][i] = 0.f;
  }

  // One evaluation e of the chain of contractions.  hid(q, rt, v) -> two words: the epilogue of hidden pass q (0 .. L - 2)
  // for the lane's 8 values of row tile rt; st(u, rt, v): the state-shaped epilogue of the member's u-th row tile, which
  // publishes the next stage input itself.  started(): once the first loads have arrived.  false: a wait ran out
  template <class Hid, class St, class Started>
  __device__ __forceinline__ bool evaluate(int e, Hid hid, St st, Started started) {
    u16x8 fz[KS1];
    u16x8 fh[KSH];
    gather_z(fz, e, 0);
#pragma unroll
    for (int rt = 0; rt < RTN; ++rt) {
      complete(fz, 0, KS1, [&](int ks) { return zfrag(e, wave * KS1 + ks, rt); });
      if (rt == 0) started();
      f32x16 acc[2];
      zero(acc);
#pragma unroll
      for (int ks = 0; ks < KS1; ++ks)
#pragma unroll
        for (int ct = 0; ct < 2; ++ct) acc[ct] = Low<T>::mfma32(w1[ct][ks], fz[ks], acc[ct]);
      float v[8];
      if (!fold_hidden(acc, v, [&]() {
            if (rt + 1 < RTN) gather_z(fz, e, rt + 1);
            else if (RTN > 1) gather_h(fh, e, 0, next_rt(0));
          }))
        return false;
      uint2 lo, hi;
      hid(0, rt, v, lo, hi);
      publish16(hfrag(e, 0, me * 4 + wave, rt), lo, hi);
      if (RTN == 1) gather_h(fh, e, 0, 0);
      // (a complete stage input: every member has read all of the evaluation before)
      if (rt + 1 == RTN && e > 0) clear_hidden(e - 1);
    }
#pragma unroll
    for (int m = 0; m < MIDS; ++m) {
#pragma unroll
      for (int rt = 0; rt < RTN; ++rt) {
        f32x16 acc[2];
        zero(acc);
#pragma unroll
        for (int k0 = 0; k0 < KSH; k0 += 4) {
          complete(fh, k0, k0 + 4, [&](int ks) { return hfrag(e, m, wave * KSH + ks, rt); });
#pragma unroll
          for (int ks = k0; ks < k0 + 4; ++ks)
#pragma unroll
            for (int ct = 0; ct < 2; ++ct) acc[ct] = Low<T>::mfma32(wm[m][ct][ks], fh[ks], acc[ct]);
        }
        float v[8];
        if (!fold_hidden(acc, v, [&]() {
              if (rt + 1 < RTN) gather_h(fh, e, m, rt + 1);
              else if (RTN > 1) gather_h(fh, e, m + 1, next_rt(m + 1));
            }))
          return false;
        uint2 lo, hi;
        hid(m + 1, rt, v, lo, hi);
        publish16(hfrag(e, m + 1, me * 4 + wave, rt), lo, hi);
        if (RTN == 1) gather_h(fh, e, m + 1, 0);
      }
    }
    if (unit_rt >= 0) {
#pragma unroll
      for (int u = 0; u < Sh::NU; ++u) {
        const int rt = unit_rt + u * Sh::APC;
        if (u > 0) gather_h(fh, e, L - 2, rt);
        f32x16 acc[1];
        zero(acc);
#pragma unroll
        for (int k0 = 0; k0 < KSH; k0 += 4) {
          complete(fh, k0, k0 + 4, [&](int ks) { return hfrag(e, L - 2, wave * KSH + ks, rt); });
#pragma unroll
          for (int ks = k0; ks < k0 + 4; ++ks) acc[0] = Low<T>::mfma32(wl[ks], fh[ks], acc[0]);
        }
        float v[4];
        if (!fold_state(acc[0], v)) return false;
        clear8(zfrag(e, unit_ct * 2 + (wave >> 1), rt), wave & 1);
        st(u, rt, v);
      }
    }
    return true;
  }
  // row tile with which the pass over hidden output q starts: the member's own in the state-shaped pass
  __device__ __forceinline__ int next_rt(int q) const { return q == L - 2 ? max(unit_rt, 0) : 0; }
  __device__ __forceinline__ void clear_hidden(int e) const {
#pragma unroll
    for (int q = 0; q < L - 1; ++q)
#pragma unroll
      for (int rt = 0; rt < RTN; ++rt) clear16(hfrag(e, q, me * 4 + wave, rt));
  }
  __device__ __forceinline__ void publish_z(int e, int rt, uint2 q) const {
    publish8(zfrag(e, unit_ct * 2 + (wave >> 1), rt), wave & 1, q);
  }
  __device__ __forceinline__ void give_up() const {
    if (threadIdx.x == 0) __hip_atomic_store(stalled, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
};

constexpr size_t kClusterLds = 2 * 4 * 3 * 2 * 64 * 16;

// ---------------------------------------------------------------------------------------
template <class T, int HP, int L, int NTL, int RTN>
__global__ __launch_bounds__(256, 1) void mlp_forward_cluster(ClusterArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  __shared__ int sh_[4];
  using Eng = ClusterEngine<T, HP, L, NTL, RTN>;
  constexpr int NU = Eng::Sh::NU, APC = Eng::Sh::APC;
  const FusedArgs& g = a.r.f;
  Eng c;
  if (!c.setup(a, (lds_f32*)(lds_u16*)smem, (RAMPDE_LDS int*)sh_)) return;
  const int s = g.s;
  const int64_t row0 = (int64_t)c.cl * 32 * RTN, n_state = g.R * g.d;
  const int nh = c.me * 64 + 16 * c.wave + 4 * c.lh;           // the lane's hidden features: nh .. nh + 3, nh + 8 .. nh + 11
  const int ns = c.unit_ct * 32 + 8 * c.wave + 4 * c.lh;       // ... and state features
  float bias[L - 1][8], wt[8], bl[4];
#pragma unroll
  for (int q = 0; q < L - 1; ++q)
#pragma unroll
    for (int i = 0; i < 8; ++i) bias[q][i] = g.layer[q].bias[nh + i + (i >= 4 ? 4 : 0)];
#pragma unroll
  for (int i = 0; i < 8; ++i) wt[i] = g.layer[0].wt ? g.layer[0].wt[nh + i + (i >= 4 ? 4 : 0)] : 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) bl[i] = g.layer[L - 1].bias[ns + i];
  float y[NU][4], yh[NU][4], bs[NU][4];
  if (c.unit_rt >= 0) {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int rt = c.unit_rt + u * APC;
      const int64_t row = row0 + rt * 32 + c.lr;
      load4f(g.step > 0 ? g.y : g.y0, row, g.R, ns, g.d, y[u]);
      const uint2 q = pack4<T>(y[u]);
      if (g.round_incr & 2) unpack4<T>(q, y[u]);
      unpack4<T>(q, yh[u]);
      if (g.step == 0) store4h(g.ckpt, row, g.R, ns, g.d, q);
      c.publish_z(0, rt, q);
    }
  }
  int e = 0;
#pragma unroll 1
  for (int i = g.step; i < g.step + g.nsteps; ++i) {
    const float* stp = g.steptab + (size_t)i * (1 + s);
    const float h = stp[0];
#pragma unroll
    for (int u = 0; u < NU; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) bs[u][r] = 0.f;
#pragma unroll 1
    for (int j = 0; j < s; ++j, ++e) {
      const bool last_stage = j + 1 == s;
      const float tau = stp[1 + j], bj = g.b[j], aj = last_stage ? 0.f : g.A[(j + 1) * s + j];
      auto hid = [&](int q, int, float (&v)[8], uint2& lo, uint2& hi) __attribute__((always_inline)) {
        float x[2][4];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          float p = v[k] + bias[q][k];
          if (q == 0) p = fmaf(wt[k], tau, p);
          x[k >> 2][k & 3] = tanh_fast(p);
        }
        lo = pack4<T>(x[0]);
        hi = pack4<T>(x[1]);
      };
      auto st = [&](int u, int rt, float (&v)[4]) __attribute__((always_inline)) {
        const int64_t row = row0 + rt * 32 + c.lr;
        float kf[4], z[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] += bl[r];
        unpack4<T>(pack4<T>(v), kf);
#pragma unroll
        for (int r = 0; r < 4; ++r) bs[u][r] = fmaf(bj, kf[r], bs[u][r]);
        uint2 zq;
        if (!last_stage) {
#pragma unroll
          for (int r = 0; r < 4; ++r) z[r] = fmaf(h, aj * kf[r], yh[u][r]);
          zq = pack4<T>(z);
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            if (g.round_incr & 1) bs[u][r] = Low<T>::to_f32(Low<T>::from_f32(bs[u][r]));
            y[u][r] = fmaf(h, bs[u][r], y[u][r]);
          }
          zq = pack4<T>(y[u]);
          if (g.round_incr & 2) unpack4<T>(zq, y[u]);
          unpack4<T>(zq, yh[u]);
        }
        c.publish_z(e + 1, rt, zq);
        if (last_stage) store4h(g.ckpt + (size_t)(i + 1) * n_state, row, g.R, ns, g.d, zq);
      };
      if (e == a.budget || !c.evaluate(e, hid, st, []() {})) {
        c.give_up();
        return;
      }
    }
  }
  if (c.unit_rt >= 0) {
#pragma unroll
    for (int u = 0; u < NU; ++u) store4f(g.y, row0 + (c.unit_rt + u * APC) * 32 + c.lr, g.R, ns, g.d, y[u]);
  }
}

// ---------------------------------------------------------------------------------------
// The cotangent chain of a group of steps whose stage inputs and activations are in their buffer sets.
template <class T, int HP, int L, int NTL, int RTN>
__global__ __launch_bounds__(256, 1) void mlp_chain_cluster(ClusterArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  __shared__ int sh_[4];
  using Eng = ClusterEngine<T, HP, L, NTL, RTN>;
  constexpr int NU = Eng::Sh::NU, APC = Eng::Sh::APC;
  const FusedArgs& g = a.r.f;
  if (g.ctl->poison) return;
  Eng c;
  const bool part = c.setup(a, (lds_f32*)(lds_u16*)smem, (RAMPDE_LDS int*)sh_);
  // under overflow detection nobody redoes a launch that was given up but the host, with the whole pass
  auto lost = [&]() {
    c.give_up();
    if (g.detect && threadIdx.x == 0) {
      __hip_atomic_store(&g.ctl->stalled, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&g.ctl->poison, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  };
  if (!part) {
    if (c.lost) lost();
    return;
  }
  const int s = g.s;
  const int64_t row0 = (int64_t)c.cl * 32 * RTN;
  const int nh = c.me * 64 + 16 * c.wave + 4 * c.lh, ns = c.unit_ct * 32 + 8 * c.wave + 4 * c.lh;
  const bool owner = c.unit_rt >= 0;
  StepExchange ex(a.r, c.cl * Eng::Sh::C + c.me, a.clusters * Eng::Sh::C);
  float av[NU][4], a_old[NU][4], da[NU][4], zf[NU][4];
  uint2 lamq[NU];
  uint32_t mask_h[RTN], mask_u[NU];
#pragma unroll
  for (int rt = 0; rt < RTN; ++rt) mask_h[rt] = row0 + rt * 32 + c.lr < g.R ? 0xFFFFFFFFu : 0u;
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int64_t row = row0 + (max(c.unit_rt, 0) + u * APC) * 32 + c.lr;
    mask_u[u] = row < g.R ? 0xFFFFFFFFu : 0u;
    load4f(g.a_in, row, g.R, ns, g.d, av[u]);
  }
  // row tiles past the padded batch (64-row units; clusters have 32, 64 or 128 rows): nothing to read or write there
  auto inside = [&](int rt) __attribute__((always_inline)) { return RTN <= 2 || row0 + rt * 32 < g.Rp; };
  // lane offsets (bytes) into the feature-group-major arrays
  const uint32_t off_h = (uint32_t)(((size_t)(nh >> 2) * g.ldk + row0 + c.lr) * 8);
  const uint32_t off_s = (uint32_t)(((size_t)(ns >> 2) * g.ldk + row0 + c.lr) * 8);
  const size_t two_groups = (size_t)g.ldk * 16, stage_bytes = (size_t)g.Rp * 8;
  // the lane's activations of an evaluation, for the tanh' factors: requested one evaluation ahead
  uint2 act[L - 1][RTN][2];
  auto fetch_act = [&](uint2 (&q)[L - 1][RTN][2], int step, int j) __attribute__((always_inline)) {
#pragma unroll
    for (int l = 0; l < L - 1; ++l) {
      const char* base = (const char*)(g.ACTT[l] + (int64_t)(step % g.nsets) * g.set_stride) + j * stage_bytes;
#pragma unroll
      for (int rt = 0; rt < RTN; ++rt)
#pragma unroll
        for (int p = 0; p < 2; ++p) q[l][rt][p] = *reinterpret_cast<const uint2*>(base + p * two_groups + (off_h + (inside(rt) ? rt * 256 : 0)));
    }
  };
  fetch_act(act, g.step, s - 1);

  bool rejected = false;
  int e = 0;
#pragma unroll 1
  for (int it = 0; it < g.nsteps; ++it) {
    const int step = g.step - it;
    if (it > 0 && !ex.template decide<T>(g, step + 1)) {
      rejected = true;
      break;
    }
    const float h = g.steptab[(size_t)step * (1 + s)];
    const int64_t set_off = (int64_t)(step % g.nsets) * g.set_stride;
    char* const KBART = (char*)(g.KBART + set_off);
    uint32_t big = 0;  // largest magnitudes of the step's cotangents
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      float sa[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) sa[r] = ex.S * av[u][r];
      lamq[u] = pack4<T>(sa);
      if (owner) track(big, lamq[u]);
#pragma unroll
      for (int r = 0; r < 4; ++r) da[u][r] = zf[u][r] = 0.f;
    }
    // cotangent of the slope of stage j:  kbar_j = Q( b_j lambda + h a_{j+1,j} zbar_{j+1} )
    auto make_kbar = [&](int ev, int u, int rt, int j) __attribute__((always_inline)) {
      const float bj = g.b[j], aj = j + 1 < s ? g.A[(j + 1) * s + j] : 0.f;
      float lam[4], v[4];
      unpack4<T>(lamq[u], lam);
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = fmaf(h, aj * zf[u][r], bj * lam[r]);
      uint2 q = pack4<T>(v);
      q.x &= mask_u[u];
      q.y &= mask_u[u];
      track(big, q);
      c.publish_z(ev, rt, q);
      if (inside(rt)) *reinterpret_cast<uint2*>(KBART + j * stage_bytes + (off_s + rt * 256)) = q;
    };
    if (owner) {
#pragma unroll
      for (int u = 0; u < NU; ++u) make_kbar(e, u, c.unit_rt + u * APC, s - 1);
    }
#pragma unroll 1
    for (int j = s - 1; j >= 0; --j, ++e) {
      const int j_next = j > 0 ? j - 1 : s - 1, step_next = j > 0 ? step : max(step - 1, g.step - g.nsteps + 1);
      uint2 act_next[L - 1][RTN][2];
      auto hid = [&](int q, int rt, float (&v)[8], uint2& lo, uint2& hi) __attribute__((always_inline)) {
        const int l = L - 2 - q;
        float x[2][4];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          float t[4];
          unpack4<T>(act[l][rt][p], t);
#pragma unroll
          for (int r = 0; r < 4; ++r) x[p][r] = v[4 * p + r] * (1.f - t[r] * t[r]);
        }
        lo = pack4<T>(x[0]);
        hi = pack4<T>(x[1]);
        lo.x &= mask_h[rt]; lo.y &= mask_h[rt];
        hi.x &= mask_h[rt]; hi.y &= mask_h[rt];
        track(big, lo);
        track(big, hi);
        char* out = (char*)(g.DELTAT[l] + set_off) + j * stage_bytes;
        if (inside(rt)) {
          *reinterpret_cast<uint2*>(out + (off_h + rt * 256)) = lo;
          *reinterpret_cast<uint2*>(out + two_groups + (off_h + rt * 256)) = hi;
        }
      };
      auto st = [&](int u, int rt, float (&v)[4]) __attribute__((always_inline)) {
        uint2 q = pack4<T>(v);
        q.x &= mask_u[u];
        q.y &= mask_u[u];
        track(big, q);
        unpack4<T>(q, zf[u]);
#pragma unroll
        for (int r = 0; r < 4; ++r) da[u][r] += zf[u][r];
        if (j > 0) make_kbar(e + 1, u, rt, j - 1);
      };
      if (e == a.budget || !c.evaluate(e, hid, st, [&]() { fetch_act(act_next, step_next, j_next); })) {
        lost();
        return;
      }
#pragma unroll
      for (int l = 0; l < L - 1; ++l)
#pragma unroll
        for (int rt = 0; rt < RTN; ++rt)
#pragma unroll
          for (int p = 0; p < 2; ++p) act[l][rt][p] = act_next[l][rt][p];
    }
    // ---- a <- a + (h / S) sum_j zbar_j (+ running-cost cotangent), fp32
    const float hs = h / ex.S;
    unsigned bits = 0;
    if (owner) {
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        float gy[4] = {0.f, 0.f, 0.f, 0.f};
        const int64_t row = row0 + (c.unit_rt + u * APC) * 32 + c.lr;
        if (g.gys) load4f(g.gys - (int64_t)it * g.gys_stride, row, g.R, ns, g.d, gy);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          a_old[u][r] = av[u][r];
          av[u][r] = fmaf(hs, da[u][r], av[u][r]) + gy[r];
          if (g.round_incr & 2) av[u][r] = Low<T>::to_f32(Low<T>::from_f32(av[u][r]));
          const unsigned bb = __builtin_bit_cast(unsigned, fabsf(av[u][r]));
          if (mask_u[u] && ns + r < g.d) bits = max(bits, bb);
        }
      }
    }
    if (g.detect) ex.post(g, step, bits, tracked_nonfinite<T>(big));
    else ex.template decide<T>(g, step);
  }
  if (g.detect && !rejected) rejected = !ex.template decide<T>(g, g.step - g.nsteps + 1);
  if (ex.stalled) return;
  if (owner) {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      // (a rejected step leaves the adjoint as it was before it)
      if (rejected) {
#pragma unroll
        for (int r = 0; r < 4; ++r) av[u][r] = a_old[u][r];
      }
      store4f(g.a_out, row0 + (c.unit_rt + u * APC) * 32 + c.lr, g.R, ns, g.d, av[u]);
    }
  }
  ex.finish(g);
}

}  // namespace rampde
