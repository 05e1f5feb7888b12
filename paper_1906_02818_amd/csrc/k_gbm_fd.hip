// Central finite differences of a GBM payoff on common random numbers, delta
// and vega in one pass over the paths. One draw of the normals serves all the
// bumped paths: the log-price relative to S0 does not depend on S0, so the
// two delta payoffs come from one path at the unbumped volatility (two spot
// prices, two barrier levels over one running maximum), and the two vega
// payoffs from a path each. The per-path differences are reduced in place;
// nothing is written per path.
//
// Bound: FP64 issue of Philox and Box-Muller, then the latency of the FP64
// chains. On the barrier call, 300007 paths x 52 steps, delta and vega: four
// bumped runs with their per-path values, and two difference kernels, took
// 160 us of kernels and six waits, this kernel and the price run 51 us; the call
// 252 -> 74 us.
#include "device/gbm.h"
#include "device/reduce.h"

namespace mcp {
namespace {

// DELTA, VEGA: the greeks wanted. Their moment vectors (one channel: the
// difference, a path counted when both its payoffs are finite) go to
// partials[greek][block].
template <uint32_t BIT, bool LOGS, bool DELTA, bool VEGA>
__global__ __launch_bounds__(kBlock) void gbm_fd_kernel(const GbmFdParams Q) {
  const GbmParams& P = Q.up[0];
  stamp(P.clock);
  constexpr bool BRIDGE = BIT == G_UOBB;
  typedef GbmStepper<double, BIT, LOGS> Stepper;
  __shared__ F64Tables tables;
  const PathMath<double> pm(tables);
  const PhiloxKeys keys = make_keys<false>(P.k0, P.k1);
  const Stepper base(Q.up[0], pm), up(Q.up[1], pm), down(Q.down[1], pm);
  ThreadSums<1> acc_d, acc_v;
  acc_d.zero();
  acc_v.zero();
  auto push = [](ThreadSums<1>& acc, double u, double d) {
    const double y[1] = {u - d};
    const bool finite = isfinite(y[0]) && isfinite(u) && isfinite(d);
    acc.push(y, finite, !finite);
  };
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  for (uint64_t pid = (uint64_t)blockIdx.x * kBlock + threadIdx.x; pid < P.n_paths;
       pid += stride) {
    const uint64_t path = P.path_offset + pid;
    with_uniform_high(path, [&](uint32_t hi) {
      GbmState<double> s0, su, sd;
      s0.start(LOGS);
      su.start(LOGS);
      sd.start(LOGS);
      walk_normals<double, BRIDGE>(P.n_steps, P.tag, (uint32_t)path, hi, keys, pm,
                                   [&](uint32_t i, double Z, uint32_t W) {
                                     if constexpr (DELTA) base.step(s0, Z, i, W);
                                     if constexpr (VEGA) {
                                       up.step(su, Z, i, W);
                                       down.step(sd, Z, i, W);
                                     }
                                   });
      auto pay = [&](const GbmParams& p, const GbmState<double>& s) {
        return payoff_of<double, BIT, LOGS>(p, s, LOGS ? Dom<double>::exp_(s.z, pm) : s.z, pm);
      };
      if constexpr (DELTA) push(acc_d, pay(Q.up[0], s0), pay(Q.down[0], s0));
      if constexpr (VEGA) push(acc_v, pay(Q.up[1], su), pay(Q.down[1], sd));
    });
  }
  double* out = Q.partials;
  if constexpr (DELTA) {
    PartSums<1> part = acc_d.part();
    block_reduce<1, kBlock>(part, out, blockIdx.x);
    out += (size_t)gridDim.x * PartSums<1>::M;
    __syncthreads();                       // the two reductions share their LDS
  }
  if constexpr (VEGA) {
    PartSums<1> part = acc_v.part();
    block_reduce<1, kBlock>(part, out, blockIdx.x);
  }
}

template <uint32_t BIT, bool LOGS>
hipError_t launch_bit(const GbmFdParams& p, bool delta, bool vega, hipStream_t s, uint32_t nb) {
  if (delta && vega)
    hipLaunchKernelGGL((gbm_fd_kernel<BIT, LOGS, true, true>), dim3(nb), dim3(kBlock), 0, s, p);
  else if (delta)
    hipLaunchKernelGGL((gbm_fd_kernel<BIT, LOGS, true, false>), dim3(nb), dim3(kBlock), 0, s, p);
  else if (vega)
    hipLaunchKernelGGL((gbm_fd_kernel<BIT, LOGS, false, true>), dim3(nb), dim3(kBlock), 0, s, p);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace

hipError_t launch_gbm_fd(const GbmFdParams& p, uint32_t bit, bool delta, bool vega, hipStream_t s,
                         uint32_t* n_blocks) {
  const uint64_t need = (p.up[0].n_paths + kBlock - 1) / kBlock;
  const uint32_t nb = (uint32_t)(need < kGbmMaxBlocks ? need : kGbmMaxBlocks);
  *n_blocks = nb;
  if (nb == 0) return hipErrorInvalidValue;
  const bool L = p.up[0].log_scheme != 0;
  switch (bit) {
#define MCP_FD_BIT(B)                                       \
  case B:                                                   \
    return L ? launch_bit<B, true>(p, delta, vega, s, nb)   \
             : launch_bit<B, false>(p, delta, vega, s, nb);
    MCP_FD_BIT(G_EURO)
    MCP_FD_BIT(G_ASIAN)
    MCP_FD_BIT(G_GEO)
    MCP_FD_BIT(G_UO)
#undef MCP_FD_BIT
    case G_UOBB: return L ? launch_bit<G_UOBB, true>(p, delta, vega, s, nb) : hipErrorInvalidValue;
  }
  return hipErrorInvalidValue;
}

}  // namespace mcp
