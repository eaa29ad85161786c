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

template <class T, int MT1, int MT2>
hipError_t launch_tiles(const ConvPair& g, const ConvPairShape& sh, bool vjp, hipStream_t st) {
  const size_t lds = conv_pair_lds_bytes(C32, sh.lines, g.Wd);
  auto kern = vjp ? &conv_pair<T, C32, MT1, MT2, true> : &conv_pair<T, C32, MT1, MT2, false>;
  if (lds > 48 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  kern<<<sh.tiles, 256, lds, st>>>(g, sh);
  return hipGetLastError();
}

template <class T, int I = 0>
hipError_t pick(const ConvPair& g, const ConvPairShape& sh, bool vjp, hipStream_t st) {
  if constexpr (I < (int)(sizeof(kPairTiles) / sizeof(kPairTiles[0]))) {
    if (sh.mt1 == kPairTiles[I][0] && sh.mt2 == kPairTiles[I][1])
      return launch_tiles<T, kPairTiles[I][0], kPairTiles[I][1]>(g, sh, vjp, st);
    return pick<T, I + 1>(g, sh, vjp, st);
  } else {
    return hipErrorInvalidValue;
  }
}

}  // namespace

#if RAMPDE_INST_BF16
hipError_t RAMPDE_CAT(RAMPDE_CAT(conv_pair_launch_, RAMPDE_INST_C32), _bf16)(const ConvPair& g, const ConvPairShape& sh, bool vjp, hipStream_t st) {
  return pick<BF16>(g, sh, vjp, st);
}
#else
hipError_t RAMPDE_CAT(RAMPDE_CAT(conv_pair_launch_, RAMPDE_INST_C32), _f16)(const ConvPair& g, const ConvPairShape& sh, bool vjp, hipStream_t st) {
  return pick<F16>(g, sh, vjp, st);
}
#endif

}  // namespace rampde
