// Launchers of the cluster kernels (cluster.hpp): one translation unit per hidden width and precision.
#pragma once
#include "cluster.hpp"

namespace rampde {

struct ClusterLaunch {
  int chain;    // 0: mlp_forward_cluster, 1: mlp_chain_cluster
  int bf16;
  int L, NTL;   // layers; dpad / 64
  int RTN;      // row tiles of 32 per cluster: 1, 2, or 4 (two hidden layers of more than 512)
  hipStream_t stream;
};

// networks that have kernels: hidden width (all hidden layers padded to it), layers, padded state width.  (Two 1024-wide
// layers between 256-wide states are 224 registers of weight fragments per lane, three would be 352; the other shapes
// that are left out would fit and have not been built)
inline bool cluster_shape(int hp, int L, int dpad) {
  return (hp == 512 && (L == 3 || L == 4) && (dpad == 64 || dpad == 128)) ||
         ((hp == 768 || hp == 1024) && (L == 2 || L == 3) && (dpad == 128 || dpad == 256));
}
inline int cluster_frags(int hp, int L, int dpad) { return 2 * (dpad / 64) + (L - 2) * 2 * (hp / 64) + hp / 64; }
inline size_t cluster_exchange_bytes(int hp, int L, int dpad, int RTN) {
  return (size_t)kClusterRing * 1024 * 4 * RTN * (dpad / 64 + (L - 1) * (hp / 64));
}

hipError_t cluster_launch_hp512_f16(const ClusterLaunch& l, const ClusterArgs& a);
hipError_t cluster_launch_hp512_bf16(const ClusterLaunch& l, const ClusterArgs& a);
hipError_t cluster_launch_hp768_f16(const ClusterLaunch& l, const ClusterArgs& a);
hipError_t cluster_launch_hp768_bf16(const ClusterLaunch& l, const ClusterArgs& a);
hipError_t cluster_launch_hp1024_f16(const ClusterLaunch& l, const ClusterArgs& a);
hipError_t cluster_launch_hp1024_bf16(const ClusterLaunch& l, const ClusterArgs& a);
inline hipError_t cluster_launch(int hp, const ClusterLaunch& l, const ClusterArgs& a) {
  if (hp == 512) return l.bf16 ? cluster_launch_hp512_bf16(l, a) : cluster_launch_hp512_f16(l, a);
  if (hp == 768) return l.bf16 ? cluster_launch_hp768_bf16(l, a) : cluster_launch_hp768_f16(l, a);
  if (hp == 1024) return l.bf16 ? cluster_launch_hp1024_bf16(l, a) : cluster_launch_hp1024_f16(l, a);
  return hipErrorInvalidValue;
}

}  // namespace rampde
