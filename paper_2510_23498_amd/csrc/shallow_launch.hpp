// Launchers of the kernels of shallow.hpp, one per (padded) hidden width and precision, each in a translation unit of its own.
#pragma once
#include <hip/hip_runtime.h>

#include "resident_launch.hpp"
#include "shallow.hpp"

namespace rampde {

struct ShallowLaunch {
  ResidentKind kind;
  int bf16;
  int NTL;    // state width / 64 (padded)
  int trace;  // normalising flow with the trace row
  int copies; // forward pass, NTL = 1, hidden width above 256: tiles of 16 / copies rows (1, 2, 4)
  unsigned grid;
  hipStream_t stream;
};

#define RAMPDE_DECLARE_SHALLOW(hp)                                                       \
  hipError_t shallow_launch_hp##hp##_f16(const ShallowLaunch& l, const ShallowArgs& a);  \
  hipError_t shallow_launch_hp##hp##_bf16(const ShallowLaunch& l, const ShallowArgs& a);
RAMPDE_DECLARE_SHALLOW(128)
RAMPDE_DECLARE_SHALLOW(256)
RAMPDE_DECLARE_SHALLOW(512)
RAMPDE_DECLARE_SHALLOW(1024)
#undef RAMPDE_DECLARE_SHALLOW

inline hipError_t shallow_launch(int hp, const ShallowLaunch& l, const ShallowArgs& a) {
  switch (hp) {
    case 128: return l.bf16 ? shallow_launch_hp128_bf16(l, a) : shallow_launch_hp128_f16(l, a);
    case 256: return l.bf16 ? shallow_launch_hp256_bf16(l, a) : shallow_launch_hp256_f16(l, a);
    case 512: return l.bf16 ? shallow_launch_hp512_bf16(l, a) : shallow_launch_hp512_f16(l, a);
    case 1024: return l.bf16 ? shallow_launch_hp1024_bf16(l, a) : shallow_launch_hp1024_f16(l, a);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace rampde
