// One translation unit per hidden width and precision: compile with
// -DRAMPDE_INST_HP={64,128,256} -DRAMPDE_INST_BF16={0,1}.
#include "resident_launch.hpp"

#if !defined(RAMPDE_INST_HP) || !defined(RAMPDE_INST_BF16)
#error "define RAMPDE_INST_HP and RAMPDE_INST_BF16"
#endif
#define RAMPDE_CAT2(a, b) a##b
#define RAMPDE_CAT(a, b) RAMPDE_CAT2(a, b)

namespace rampde {

namespace {

constexpr int HP = RAMPDE_INST_HP;

template <class Kern>
hipError_t launch_kernel(Kern kern, const ResidentLaunch& l, const ResidentArgs& a) {
  const size_t lds = l.kind == kResidentAdjoint ? resident_lds_bytes(HP, a.f.L, a.f.s, l.MT, true) : resident_lds_bytes(HP, a.f.L, 0, l.MT, false);
  if (lds > 48 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  kern<<<l.grid, 256, lds, l.stream>>>(a);
  return hipGetLastError();
}

template <class T, int L, int MT>
hipError_t pick_kernel(const ResidentLaunch& l, const ResidentArgs& a) {
  // forward and transposed weight slices together: 384 of 512 registers at three layers of 256, 640 at four; 192 of
  // 256 at four layers of 128
  constexpr bool phased = (HP == 256 && (L == 4 || MT == 2)) || (HP == 128 && L == 4);
  if (l.kind == kResidentForward) {
    if constexpr (MT == 1 && HP >= 128) {
      if (l.copies == 4) return launch_kernel(mlp_forward_resident<T, L, HP, MT, 4>, l, a);
      if (l.copies == 2) return launch_kernel(mlp_forward_resident<T, L, HP, MT, 2>, l, a);
    }
    return l.copies == 1 ? launch_kernel(mlp_forward_resident<T, L, HP, MT, 1>, l, a) : hipErrorInvalidValue;
  }
  if (l.kind == kResidentRecompute)
    return a.f.KT ? launch_kernel(mlp_recompute_resident<T, L, HP, MT, true>, l, a) : launch_kernel(mlp_recompute_resident<T, L, HP, MT, false>, l, a);
  if (l.kind == kResidentChain)
    return a.f.KT ? launch_kernel(mlp_chain_resident<T, L, HP, MT, true>, l, a) : launch_kernel(mlp_chain_resident<T, L, HP, MT, false>, l, a);
  if (a.f.tpart) return launch_kernel(mlp_adjoint_resident<T, L, HP, MT, true, phased>, l, a);
  return launch_kernel(mlp_adjoint_resident<T, L, HP, MT, false, phased>, l, a);
}

template <class T, int MT>
hipError_t pick_layers(const ResidentLaunch& l, const ResidentArgs& a) {
  switch (a.f.L) {
    case 2: return pick_kernel<T, 2, MT>(l, a);
    case 3: return pick_kernel<T, 3, MT>(l, a);
    case 4: return pick_kernel<T, 4, MT>(l, a);
    default: return hipErrorInvalidValue;
  }
}

template <class T>
hipError_t pick_rows(const ResidentLaunch& l, const ResidentArgs& a) {
  if (l.MT == 1) return pick_layers<T, 1>(l, a);
  if constexpr (HP == 256)
    if (l.MT == 2) return pick_layers<T, 2>(l, a);
  return hipErrorInvalidValue;
}

}  // namespace

#if RAMPDE_INST_BF16
hipError_t RAMPDE_CAT(RAMPDE_CAT(resident_launch_hp, RAMPDE_INST_HP), _bf16)(const ResidentLaunch& l, const ResidentArgs& a) {
  return pick_rows<BF16>(l, a);
}
#else
hipError_t RAMPDE_CAT(RAMPDE_CAT(resident_launch_hp, RAMPDE_INST_HP), _f16)(const ResidentLaunch& l, const ResidentArgs& a) {
  return pick_rows<F16>(l, a);
}
#endif

}  // namespace rampde
