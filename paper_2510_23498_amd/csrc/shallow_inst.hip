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
  const size_t lds = ShallowLds::bytes<NTL, HP>(l.adjoint != 0, a.r.f.s);
  if (lds > 48 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  kern<<<l.grid, ShallowShape<NTL, HP>::NT, lds, l.stream>>>(a);
  return hipGetLastError();
}

// (plain networks up to 256 wide with up to 64 state columns are those of resident.hpp)
template <class T>
hipError_t pick(const ShallowLaunch& l, const ShallowArgs& a) {
  if (l.NTL == 1 && l.trace)
    return l.adjoint ? launch_kernel<1>(mlp_adjoint_shallow<T, 1, HP, true>, l, a) : launch_kernel<1>(mlp_forward_shallow<T, 1, HP, true>, l, a);
  if constexpr (HP >= 512)
    if (l.NTL == 1)
      return l.adjoint ? launch_kernel<1>(mlp_adjoint_shallow<T, 1, HP, false>, l, a) : launch_kernel<1>(mlp_forward_shallow<T, 1, HP, false>, l, a);
  if constexpr (HP == 256 || HP == 512)
    if (l.NTL == 2 && !l.trace)
      return l.adjoint ? launch_kernel<2>(mlp_adjoint_shallow<T, 2, HP, false>, l, a) : launch_kernel<2>(mlp_forward_shallow<T, 2, HP, false>, l, a);
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
