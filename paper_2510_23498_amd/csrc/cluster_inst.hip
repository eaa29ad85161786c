// One translation unit per hidden width and precision: compile with
// -DRAMPDE_INST_HP={512,768,1024} -DRAMPDE_INST_BF16={0,1}.
#include "cluster_launch.hpp"

#if !defined(RAMPDE_INST_HP) || !defined(RAMPDE_INST_BF16)
#error "define RAMPDE_INST_HP and RAMPDE_INST_BF16"
#endif
#define RAMPDE_CAT2(a, b) a##b
#define RAMPDE_CAT(a, b) RAMPDE_CAT2(a, b)

namespace rampde {

namespace {

// a workgroup per member; every XCD (of eight) gets whole clusters
unsigned cluster_grid(int clusters) { return 8u * (RAMPDE_INST_HP / 64) * ((clusters + 7) / 8); }

template <class T, int L, int NTL, int RTN>
hipError_t launch_kernel(const ClusterLaunch& l, const ClusterArgs& a) {
  static_assert(ClusterShape<RAMPDE_INST_HP, L, NTL, RTN>::FRAGS > 0, "");
  auto kern = l.chain ? &mlp_chain_cluster<T, RAMPDE_INST_HP, L, NTL, RTN> : &mlp_forward_cluster<T, RAMPDE_INST_HP, L, NTL, RTN>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kClusterLds);
  if (e != hipSuccess) return e;
  kern<<<cluster_grid(a.clusters), 256, kClusterLds, l.stream>>>(a);
  return hipGetLastError();
}

template <class T, int L, int NTL>
hipError_t pick_rows(const ClusterLaunch& l, const ClusterArgs& a) {
  if constexpr (RAMPDE_INST_HP > 512 && L > 2)  // (128 rows: see choose_clusters)
    if (l.RTN == 4) return launch_kernel<T, L, NTL, 4>(l, a);
  return l.RTN == 1 ? launch_kernel<T, L, NTL, 1>(l, a) : l.RTN == 2 ? launch_kernel<T, L, NTL, 2>(l, a) : hipErrorInvalidValue;
}

template <class T, int L>
hipError_t pick_state(const ClusterLaunch& l, const ClusterArgs& a) {
  constexpr int lo = RAMPDE_INST_HP == 512 ? 1 : 2;
  return l.NTL == lo ? pick_rows<T, L, lo>(l, a) : l.NTL == 2 * lo ? pick_rows<T, L, 2 * lo>(l, a) : hipErrorInvalidValue;
}

template <class T>
hipError_t pick_layers(const ClusterLaunch& l, const ClusterArgs& a) {
  constexpr int lo = RAMPDE_INST_HP == 512 ? 3 : 2;
  return l.L == lo ? pick_state<T, lo>(l, a) : l.L == lo + 1 ? pick_state<T, lo + 1>(l, a) : hipErrorInvalidValue;
}

}  // namespace

#if RAMPDE_INST_BF16
hipError_t RAMPDE_CAT(RAMPDE_CAT(cluster_launch_hp, RAMPDE_INST_HP), _bf16)(const ClusterLaunch& l, const ClusterArgs& a) {
  return pick_layers<BF16>(l, a);
}
#else
hipError_t RAMPDE_CAT(RAMPDE_CAT(cluster_launch_hp, RAMPDE_INST_HP), _f16)(const ClusterLaunch& l, const ClusterArgs& a) {
  return pick_layers<F16>(l, a);
}
#endif

}  // namespace rampde
