// Launchers of the kernels of resident.hpp, one per (padded) hidden width and precision, each in a translation unit of
// its own.
#pragma once
#include <hip/hip_runtime.h>

#include "resident.hpp"

namespace rampde {

enum ResidentKind { kResidentForward, kResidentAdjoint, kResidentRecompute, kResidentChain };
struct ResidentLaunch {
  ResidentKind kind;
  int bf16;
  int MT;        // row tile = 16 MT rows; 2 only at hidden width 256
  int copies;    // forward pass, hidden width 128 or 256, MT = 1: tiles of 16 / copies rows (1, 2, 4)
  unsigned grid;
  hipStream_t stream;
};

#define RAMPDE_DECLARE_RESIDENT(hp)                                                        \
  hipError_t resident_launch_hp##hp##_f16(const ResidentLaunch& l, const ResidentArgs& a); \
  hipError_t resident_launch_hp##hp##_bf16(const ResidentLaunch& l, const ResidentArgs& a);
RAMPDE_DECLARE_RESIDENT(64)
RAMPDE_DECLARE_RESIDENT(128)
RAMPDE_DECLARE_RESIDENT(256)
#undef RAMPDE_DECLARE_RESIDENT

inline hipError_t resident_launch(int hp, const ResidentLaunch& l, const ResidentArgs& a) {
  switch (hp) {
    case 64: return l.bf16 ? resident_launch_hp64_bf16(l, a) : resident_launch_hp64_f16(l, a);
    case 128: return l.bf16 ? resident_launch_hp128_bf16(l, a) : resident_launch_hp128_f16(l, a);
    case 256: return l.bf16 ? resident_launch_hp256_bf16(l, a) : resident_launch_hp256_f16(l, a);
    default: return hipErrorInvalidValue;
  }
}

// LDS of a launch: s * (L - 1) activation tiles in the adjoint kernel, two ping-pong tiles (three in the chain of
// four layers) in the others
inline size_t resident_lds_bytes(int hp, int L, int s, int MT, bool adjoint) {
  const size_t param = ((size_t)hp * L + 64 + 32) * 4, rows = 16 * (size_t)MT;
  const size_t tiles = adjoint ? (size_t)s * (L - 1) : L > 2 ? L - 1 : 2;
  const size_t last = adjoint && hp >= 128 && L >= 3 && MT == 1 ? 64 * (size_t)hp * 2 : 0;  // (the transposed last slice)
  return param + 2 * rows * (64 + 8 + tiles * (hp + 8)) + last;
}
// workgroups that a compute unit runs at once: the register bound of the kernels (one of 512 registers at width 256,
// two of 256 below) and the LDS
inline int resident_per_cu(int hp, size_t lds_bytes) {
  const int by_lds = (int)((size_t)159 * 1024 / (lds_bytes + 256));
  const int by_regs = hp == 256 ? 1 : 2;
  return by_lds < by_regs ? by_lds : by_regs;
}

}  // namespace rampde
