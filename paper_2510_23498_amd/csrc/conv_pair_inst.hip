// One translation unit per number of 32-channel blocks and precision: compile with
// -DRAMPDE_INST_C32={1,2} -DRAMPDE_INST_BF16={0,1}.
#include "conv_pair_launch.hpp"

#if !defined(RAMPDE_INST_C32) || !defined(RAMPDE_INST_BF16)
#error "define RAMPDE_INST_C32 and RAMPDE_INST_BF16"
#endif
#define RAMPDE_CAT2(a, b) a##b
#define RAMPDE_CAT(a, b) RAMPDE_CAT2(a, b)

namespace rampde {

namespace {

constexpr int C32 = RAMPDE_INST_C32;

template <class Kern, class... Args>
hipError_t launch_kernel(Kern kern, size_t lds, const ConvLaunch& l, Args... args) {
  if (lds > 48 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  kern<<<l.grid, 256, lds, l.st>>>(args...);
  return hipGetLastError();
}

template <class T, int I = 0>
hipError_t pick_pair(const ConvPair& g, const ConvPairShape& sh, const ConvLaunch& l) {
  if constexpr (I < (int)(sizeof(kPairTiles) / sizeof(kPairTiles[0]))) {
    constexpr int MT1 = kPairTiles[I][0], MT2 = kPairTiles[I][1];
    if (sh.mt1 != MT1 || sh.mt2 != MT2) return pick_pair<T, I + 1>(g, sh, l);
    return launch_kernel(l.vjp ? &conv_pair<T, C32, MT1, MT2, true> : &conv_pair<T, C32, MT1, MT2, false>,
                         conv_pair_lds_bytes(C32, sh.lines, g.Wd), l, g, sh);
  } else {
    return hipErrorInvalidValue;
  }
}

template <class T, int MT = 1>
hipError_t pick_pass(const ConvPass& g, const PassShape& sh, const ConvLaunch& l) {
  if constexpr (MT <= kPassTiles) {
    if (sh.mt != MT) return pick_pass<T, MT + 1>(g, sh, l);
    return launch_kernel(l.kind == kPassForward ? &conv_pass_forward<T, C32, MT>
                         : l.kind == kPassRecompute ? &conv_pass_recompute<T, C32, MT> : &conv_pass_chain<T, C32, MT>,
                         pass_lds_bytes(C32, sh.lines, g.Wd), l, g, sh);
  } else {
    return hipErrorInvalidValue;
  }
}

template <class T>
hipError_t pick_redo(const ConvRedo& a, const ConvLaunch& l) {
  return launch_kernel(l.backward ? &conv_redo_backward<T, C32> : &conv_redo_forward<T, C32>, conv_pair_lds_bytes(C32, a.sh.lines, a.g.Wd), l, a);
}

}  // namespace

#if RAMPDE_INST_BF16
#define RAMPDE_LOW BF16
#define RAMPDE_NAME(f) RAMPDE_CAT(RAMPDE_CAT(f, RAMPDE_INST_C32), _bf16)
#else
#define RAMPDE_LOW F16
#define RAMPDE_NAME(f) RAMPDE_CAT(RAMPDE_CAT(f, RAMPDE_INST_C32), _f16)
#endif
hipError_t RAMPDE_NAME(conv_pair_launch_)(const ConvPair& g, const ConvPairShape& sh, const ConvLaunch& l) { return pick_pair<RAMPDE_LOW>(g, sh, l); }
hipError_t RAMPDE_NAME(conv_pass_launch_)(const ConvPass& g, const PassShape& sh, const ConvLaunch& l) { return pick_pass<RAMPDE_LOW>(g, sh, l); }
hipError_t RAMPDE_NAME(conv_redo_launch_)(const ConvRedo& a, const ConvLaunch& l) { return pick_redo<RAMPDE_LOW>(a, l); }

}  // namespace rampde
