// One translation unit per hidden width and precision: compile with
// -DRAMPDE_INST_HP={128,256,512,1024} -DRAMPDE_INST_BF16={0,1}.
#include "shallow_launch.hpp"

#if !defined(RAMPDE_INST_HP) || !defined(RAMPDE_INST_BF16)
#error "define RAMPDE_INST_HP and RAMPDE_INST_BF16"
#endif
#define RAMPDE_CAT2(a, b) a##b
#define RAMPDE_CAT(a, b) RAMPDE_CAT2(a, b)

namespace rampde {

namespace {

constexpr int HP = RAMPDE_INST_HP;

template <int NTL, class Kern>
hipError_t launch_kernel(Kern kern, const ShallowLaunch& l, const ShallowArgs& a) {
  const size_t lds = ShallowLds::bytes<NTL, HP>(l.kind == kResidentAdjoint, a.r.f.s);
  if (lds > 48 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  kern<<<l.grid, ShallowShape<NTL, HP>::NT, lds, l.stream>>>(a);
  return hipGetLastError();
}

template <class T, int NTL, bool TRACE>
hipError_t pick_kind(const ShallowLaunch& l, const ShallowArgs& a) {
  switch (l.kind) {
    case kResidentForward:
      if constexpr (NTL == 1 && HP > 256) {
        if (l.copies == 4) return launch_kernel<NTL>(mlp_forward_shallow<T, NTL, HP, TRACE, 4>, l, a);
        if (l.copies == 2) return launch_kernel<NTL>(mlp_forward_shallow<T, NTL, HP, TRACE, 2>, l, a);
      }
      return l.copies == 1 ? launch_kernel<NTL>(mlp_forward_shallow<T, NTL, HP, TRACE, 1>, l, a) : hipErrorInvalidValue;
    case kResidentChain: return launch_kernel<NTL>(mlp_chain_shallow<T, NTL, HP, TRACE>, l, a);
    case kResidentRecompute: return launch_kernel<NTL>(mlp_recompute_shallow<T, NTL, HP, TRACE>, l, a);
    default: return launch_kernel<NTL>(mlp_adjoint_shallow<T, NTL, HP, TRACE>, l, a);
  }
}

// (plain networks up to 256 wide with up to 64 state columns are those of resident.hpp)
template <class T>
hipError_t pick(const ShallowLaunch& l, const ShallowArgs& a) {
  if (l.NTL == 1 && l.trace) return pick_kind<T, 1, true>(l, a);
  if constexpr (HP >= 512)
    if (l.NTL == 1) return pick_kind<T, 1, false>(l, a);
  if constexpr (HP == 256 || HP == 512)
    if (l.NTL == 2 && !l.trace) return pick_kind<T, 2, false>(l, a);
  return hipErrorInvalidValue;
}

}  // namespace

#if RAMPDE_INST_BF16
hipError_t RAMPDE_CAT(RAMPDE_CAT(shallow_launch_hp, RAMPDE_INST_HP), _bf16)(const ShallowLaunch& l, const ShallowArgs& a) {
  return pick<BF16>(l, a);
}
#else
hipError_t RAMPDE_CAT(RAMPDE_CAT(shallow_launch_hp, RAMPDE_INST_HP), _f16)(const ShallowLaunch& l, const ShallowArgs& a) {
  return pick<F16>(l, a);
}
#endif

}  // namespace rampde
