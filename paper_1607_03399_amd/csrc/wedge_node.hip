// Launches of the node-lane wedge kernel (wedge_node.hpp).
#include "wedge_node.hpp"

namespace wdg {
namespace {

// XCD-aware mapping of blocks to chunks (each XCD one contiguous range, so
// face neighbours share its L2)
__device__ __forceinline__ int xcd_chunk_n(int bid, int nb) {
  const int qd = nb / 8, rm = nb % 8, xcd = bid % 8, kk = bid / 8;
  return xcd < rm ? xcd * (qd + 1) + kk : rm * (qd + 1) + (xcd - rm) * qd + kk;
}

// at least two wavefronts per SIMD (at most 256 registers per lane)
template <int N, typename T, int MODE, int EPB>
__global__ void __launch_bounds__((NCfg<N, T, EPB>::BS), 2) wedge_node_stage(StageLaunch A) {
  wedge_node_chunk<N, T, MODE, EPB>(A, xcd_chunk_n(blockIdx.x, gridDim.x));
}

template <int N, typename T, int EPB>
__global__ void __launch_bounds__((NCfg<N, T, EPB>::BS), 2)
    wedge_node_batch(const StageLaunch* __restrict__ probs, const int2* __restrict__ work, int nwork) {
  const int w = xcd_chunk_n(blockIdx.x, gridDim.x);
  if (w >= nwork) return;
  const int2 it = work[w];
  wedge_node_chunk<N, T, 0, EPB>(probs[it.x], it.y);
}

template <int N, typename T, int EPB>
hipError_t launch_node_t(const StageLaunch& a, hipStream_t st) {
  using C = NCfg<N, T, EPB>;
  const int64_t nchunks = (a.Kw + EPB - 1) / EPB;
  if (nchunks <= 0) return hipSuccess;
  if (a.nmort > 0)
    hipLaunchKernelGGL((wedge_node_stage<N, T, 2, EPB>), dim3(unsigned(nchunks)), dim3(C::BS), 0, st, a);
  else if (a.Kt > 0)
    hipLaunchKernelGGL((wedge_node_stage<N, T, 1, EPB>), dim3(unsigned(nchunks)), dim3(C::BS), 0, st, a);
  else
    hipLaunchKernelGGL((wedge_node_stage<N, T, 0, EPB>), dim3(unsigned(nchunks)), dim3(C::BS), 0, st, a);
  return hipGetLastError();
}

template <int N, typename T, int EPB>
hipError_t launch_node_batch_t(const StageLaunch* probs, const int2* work, int nwork, hipStream_t st) {
  if (nwork <= 0) return hipSuccess;
  hipLaunchKernelGGL((wedge_node_batch<N, T, EPB>), dim3(unsigned(nwork)), dim3(NCfg<N, T, EPB>::BS), 0, st, probs,
                     work, nwork);
  return hipGetLastError();
}

}  // namespace

// Elements per block of the node-lane kernel (FP32): the candidates the batch
// autotuner tries (index 0 is the single-problem kernel's), lane counts
// EPB Np_tri close to whole wavefronts.
int wedge_node_epb(int N, int bits, int idx) {
  // index 0 is the default: the fastest shape measured for one problem (order 4
  // on 73 728 wedges: 121 / 125 / 125 / 124 us for 8 / 17 / 12 / 4 elements
  // per block, and 8 also beside tetrahedra; order 5: 213 us at 12, 239-244 at
  // 9, 6, 3)
  static const int e4[kNodeEpbVariants] = {8, 17, 12, 4}, e5[kNodeEpbVariants] = {12, 9, 6, 3};
  if (bits != 32 || idx < 0 || idx >= kNodeEpbVariants) return 0;
  return N == 4 ? e4[idx] : (N == 5 ? e5[idx] : 0);
}

#define WDG_NODE_EPB(n, CALL)                          \
  switch (epb) {                                       \
    case (n == 4 ? 12 : 9): CALL(n, (n == 4 ? 12 : 9)); break;   \
    case (n == 4 ? 8 : 6): CALL(n, (n == 4 ? 8 : 6)); break;     \
    case (n == 4 ? 4 : 3): CALL(n, (n == 4 ? 4 : 3)); break;     \
    case (n == 4 ? 17 : 12): CALL(n, (n == 4 ? 17 : 12)); break; \
    default: break;                                    \
  }

hipError_t launch_wedge_node_stage(int N, int bits, int epb, const StageLaunch& a, hipStream_t st) {
  hipError_t err = hipErrorInvalidValue;
  if (bits != 32) return err;
#define WDG_CALL(n, E) err = launch_node_t<n, float, E>(a, st)
  if (N == 4) {
    WDG_NODE_EPB(4, WDG_CALL)
  } else if (N == 5) {
    WDG_NODE_EPB(5, WDG_CALL)
  }
#undef WDG_CALL
  return err;
}

hipError_t launch_wedge_node_batch(int N, int bits, int epb, const StageLaunch* probs, const int2* work, int nwork,
                                   hipStream_t st) {
  hipError_t err = hipErrorInvalidValue;
  if (bits != 32) return err;
#define WDG_CALL(n, E) err = launch_node_batch_t<n, float, E>(probs, work, nwork, st)
  if (N == 4) {
    WDG_NODE_EPB(4, WDG_CALL)
  } else if (N == 5) {
    WDG_NODE_EPB(5, WDG_CALL)
  }
#undef WDG_CALL
  return err;
}
#undef WDG_NODE_EPB

}  // namespace wdg
