// One-dimensional GBM path kernel: Euler-Maruyama (Sec. II-A.1) for
// dS = r S dt + sigma S dW under the risk-neutral measure, fused with the
// path functionals, the payoffs and the first stage of the averaging
// reduction (Eq. 3). A thread prices one path at a time, its state in
// registers, nothing written to memory per step; over a persistent grid it
// prices several paths and keeps their moments in FP64 registers.
// The path itself: device/gbm.h.
//
// Bound: VALU issue. At 2^24 x 252 (Asian, geometric, barrier) a Philox block
// and its four steps are 117 cycles of Philox, 110 of Box-Muller and 82 of
// steps per wave (issue costs: device/rng.h; a transcendental 8.3, v_max3 and
// v_alignbit 4.2), 309 in all, and the kernel runs at 307 (1.98 ms).
#include <initializer_list>

#include "device/gbm.h"
#include "device/reduce.h"
#include "mc_internal.h"

namespace mcp {
namespace {

template <typename R, uint32_t MASK, bool LOGS, uint32_t CO>
__device__ __forceinline__ void simulate(const GbmParams& P,
                                         const GbmStepper<R, MASK, LOGS>& st,
                                         const PhiloxKeys& keys, uint32_t lo, uint32_t hi,
                                         double (&y)[gbm_channels(MASK)]) {
  const PathMath<R>& pm = st.pm;
  GbmState<R> s;
  s.start(LOGS);
  const uint32_t n = P.n_steps;
  if constexpr (CO > 1) {
    // Coupled coarse path: step i takes normals CO i .. CO i + CO - 1 of the
    // fine path, summed and scaled by 1/sqrt(CO) (same Brownian increment
    // over the coarse step). CO divides the 4 normals of a Philox block.
    static_assert(CO == 2 || CO == 4, "coupling factor");
    const PathRng pc = make_rng(lo, hi, P.tag, keys);
    const R rsc = CO == 2 ? R(0.70710678118654752440) : R(0.5);
    constexpr uint32_t SPB = 4 / CO;              // coarse steps per block
    const uint32_t nb = n / SPB;
    for (uint32_t j = 0; j < nb; ++j) {
      const Normals4<R> nz = normals4(philox(j, pc, keys), pm);
#pragma unroll
      for (uint32_t q = 0; q < SPB; ++q) {
        R Z = nz.z[q * CO];
#pragma unroll
        for (uint32_t t = 1; t < CO; ++t) Z += nz.z[q * CO + t];
        st.step(s, Z * rsc, SPB * j + q, 0u);
      }
    }
    if (n % SPB) {                                 // CO = 2, odd n: one step left
      const Normals4<R> nz = normals4(philox(nb, pc, keys), pm);
      st.step(s, (nz.z[0] + nz.z[1]) * rsc, n - 1, 0u);
    }
  } else {
    walk_normals<R, (MASK & G_UOBB) != 0>(n, P.tag, lo, hi, keys, pm,
                                          [&](uint32_t i, R Z, uint32_t W) { st.step(s, Z, i, W); });
  }

  // Terminal payoffs, discounted (e^{-rT}).
  const R S0 = (R)P.S0, K = (R)P.K, disc = (R)P.disc, inv_n = R(1) / (R)n;
  const R En = LOGS ? Dom<R>::exp_(s.z, pm) : s.z;    // S_n / S0
  const R ST = S0 * En;
  const R A = S0 * s.sumE * inv_n;
  int c = 0;
  if constexpr ((MASK & G_EURO) != 0) y[c++] = payoff_of<R, G_EURO, LOGS>(P, s, En, pm);
  if constexpr ((MASK & G_ASIAN) != 0) y[c++] = payoff_of<R, G_ASIAN, LOGS>(P, s, En, pm);
  if constexpr ((MASK & G_GEO) != 0) y[c++] = payoff_of<R, G_GEO, LOGS>(P, s, En, pm);
  if constexpr ((MASK & G_UO) != 0) y[c++] = payoff_of<R, G_UO, LOGS>(P, s, En, pm);
  if constexpr ((MASK & G_UOBB) != 0) y[c++] = payoff_of<R, G_UOBB, LOGS>(P, s, En, pm);
  if constexpr ((MASK & G_EURO_G) != 0) {
    const bool itm = ST > K;
    y[c++] = itm ? (double)(disc * En) : 0.0;     // dS_T/dS0 = S_T/S0
    const R dST = LOGS ? ST * (st.sdt * s.sumZ - st.sig * (R)P.T) : S0 * s.dsig;
    y[c++] = itm ? (double)(disc * dST) : 0.0;
  }
  if constexpr ((MASK & G_ASIAN_G) != 0) {
    const bool itm = A > K;
    y[c++] = itm ? (double)(disc * s.sumE * inv_n) : 0.0;
    y[c++] = itm ? (double)(disc * S0 * s.accV * inv_n) : 0.0;
  }
}

// Persistent grid: at most kGbmMaxBlocks workgroups (one wave of blocks at
// full occupancy); each thread prices paths pid, pid + stride, ... and keeps
// their moments in FP64 registers, so each block writes one moment vector.
template <typename R, uint32_t MASK, bool LOGS, uint32_t CO>
__global__ __launch_bounds__(kBlock) void gbm_path_kernel(const GbmParams P) {
  stamp(P.clock);
  constexpr int C = gbm_channels(MASK);
  __shared__ typename PathMath<R>::Shared shared;
  const PathMath<R> pm(shared);
  const GbmStepper<R, MASK, LOGS> st(P, pm);
  const PhiloxKeys keys = make_keys<sizeof(R) == 4>(P.k0, P.k1);
  ThreadSums<C> acc;
  acc.zero();
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  for (uint64_t pid = (uint64_t)blockIdx.x * kBlock + threadIdx.x; pid < P.n_paths;
       pid += stride) {
    double y[C];
    const uint64_t path = P.path_offset + pid;
    with_uniform_high(path, [&](uint32_t hi) {
      simulate<R, MASK, LOGS, CO>(P, st, keys, (uint32_t)path, hi, y);
    });
    bool finite = true;
#pragma unroll
    for (int c = 0; c < C; ++c) finite = finite && isfinite(y[c]);
    if (P.path_out != nullptr) {
#pragma unroll
      for (int c = 0; c < C; ++c) P.path_out[pid * C + c] = y[c];
    }
    acc.push(y, finite, !finite);
  }
  PartSums<C> part = acc.part();
  block_reduce<C, kBlock>(part, P.partials, blockIdx.x);
}

template <typename R, uint32_t MASK, bool LOGS, uint32_t CO = 1>
hipError_t launch_one(const GbmParams& p, hipStream_t s, uint32_t nb) {
  hipLaunchKernelGGL((gbm_path_kernel<R, MASK, LOGS, CO>), dim3(nb), dim3(kBlock), 0, s, p);
  return hipGetLastError();
}

// Coupled coarse paths (multilevel): every channel except the bridge barrier.
constexpr uint32_t kMaskCoupled = G_ALL & ~G_UOBB;

template <typename R, bool LOGS>
hipError_t launch_coupled(const GbmParams& p, hipStream_t s, uint32_t nb) {
  return p.coarsen == 2 ? launch_one<R, kMaskCoupled, LOGS, 2>(p, s, nb)
                        : launch_one<R, kMaskCoupled, LOGS, 4>(p, s, nb);
}

// Instantiated functional sets, smallest first. A call takes the first that
// covers what it wants: the functionals it does not want cost it time (a
// barrier on the all-functional kernel pays for the bridge's second Philox
// block, logarithm and square root and for an exponential per step: in FP64,
// 300007 paths x 52 steps, 187 us against 39 us on its own set).
constexpr uint32_t kMaskEuro = G_EURO;
constexpr uint32_t kMaskEuroG = G_EURO | G_EURO_G;
constexpr uint32_t kMaskAsianGeo = G_ASIAN | G_GEO;
constexpr uint32_t kMaskAsianG = G_ASIAN | G_ASIAN_G;
constexpr uint32_t kMaskPath3 = G_ASIAN | G_GEO | G_UO;
constexpr uint32_t kMaskS = G_ALL & ~G_UOBB;   // Euler on S

}  // namespace

uint32_t gbm_pick_mask(uint32_t want, bool fp64, bool log_scheme, uint32_t coarsen, bool rows) {
  if (coarsen != 1) {
    if (coarsen != 2 && coarsen != 4) return 0;
    return (want & ~kMaskCoupled) == 0 ? kMaskCoupled : 0;
  }
  auto first = [want](std::initializer_list<uint32_t> sets) -> uint32_t {
    for (uint32_t m : sets)
      if ((m & want) == want) return m;
    return 0;
  };
  if (!log_scheme) return first({kMaskS});
  // Rows of per-path values keep their documented channel sets.
  if (rows) return fp64 ? first({kMaskEuroG, G_ALL}) : first({kMaskEuro, kMaskEuroG, kMaskPath3, G_ALL});
  return fp64 ? first({kMaskEuroG, G_UO, G_UOBB, kMaskAsianGeo, kMaskAsianG, kMaskPath3, G_ALL})
              : first({kMaskEuro, kMaskEuroG, G_UO, G_UOBB, kMaskAsianGeo, kMaskAsianG, kMaskPath3,
                       G_ALL});
}

hipError_t launch_gbm(const GbmParams& p, uint32_t mask, bool fp64, hipStream_t s,
                      uint32_t* n_blocks) {
  const uint64_t need = (p.n_paths + kBlock - 1) / kBlock;
  const uint32_t nb = (uint32_t)(need < kGbmMaxBlocks ? need : kGbmMaxBlocks);
  *n_blocks = nb;
  const bool L = p.log_scheme != 0;
  if (p.coarsen != 1) {
    if (mask != kMaskCoupled || (p.coarsen != 2 && p.coarsen != 4)) return hipErrorInvalidValue;
    if (L) return fp64 ? launch_coupled<double, true>(p, s, nb) : launch_coupled<float, true>(p, s, nb);
    return fp64 ? launch_coupled<double, false>(p, s, nb) : launch_coupled<float, false>(p, s, nb);
  }
  if (!L) {
    if (mask != kMaskS) return hipErrorInvalidValue;
    return fp64 ? launch_one<double, kMaskS, false>(p, s, nb)
                : launch_one<float, kMaskS, false>(p, s, nb);
  }
  switch (mask) {
    case kMaskEuro: return fp64 ? hipErrorInvalidValue : launch_one<float, kMaskEuro, true>(p, s, nb);
#define MCP_GBM_SET(M)                                   \
  case M:                                                \
    return fp64 ? launch_one<double, M, true>(p, s, nb)  \
                : launch_one<float, M, true>(p, s, nb);
    MCP_GBM_SET(kMaskEuroG)
    MCP_GBM_SET(G_UO)
    MCP_GBM_SET(G_UOBB)
    MCP_GBM_SET(kMaskAsianGeo)
    MCP_GBM_SET(kMaskAsianG)
    MCP_GBM_SET(kMaskPath3)
    MCP_GBM_SET(G_ALL)
#undef MCP_GBM_SET
  }
  return hipErrorInvalidValue;
}

}  // namespace mcp
