// One path of geometric Brownian motion: its running state, its step, its
// normals and its payoffs, for the path kernel and the bumped-path kernel
// (Euler-Maruyama, Sec. II-A.1, for dS = r S dt + sigma S dW).
//
// Schemes: log-Euler on ln S (exact in law for every step count) and Euler
// on S (first-order weak error, Sec. V-B). In FP32 the log state is kept in
// base 2, z = log2(S/S0), so that S_i/S0 = exp2(z) is one v_exp_f32; in FP64
// it is the natural log.
#pragma once

#include "../mc_internal.h"
#include "rng.h"

namespace mcp {

template <typename R>
struct Dom;
template <>
struct Dom<float> {
  typedef PathMath<float> M;
  static __device__ __forceinline__ float exp_(float z, const M&) {
    return __builtin_amdgcn_exp2f(z);
  }
  // -log of the uniform of a word, in the kernel's log domain.
  static __device__ __forceinline__ float neg_log_(uint32_t w, const M&) {
    return -__builtin_amdgcn_logf(uniform_f32(w));
  }
  static __device__ __forceinline__ float max_(float a, float b) { return __builtin_fmaxf(a, b); }
  static __device__ __forceinline__ float sqrt_(float x) { return __builtin_amdgcn_sqrtf(x); }
};
template <>
struct Dom<double> {
  typedef PathMath<double> M;
  static __device__ __forceinline__ double exp_(double z, const M& m) { return exp_f64(z, m.t); }
  static __device__ __forceinline__ double neg_log_(uint32_t w, const M& m) {
    return 0.5 * neg2_log_f64(w, m.t);
  }
  static __device__ __forceinline__ double max_(double a, double b) { return __builtin_fmax(a, b); }
  static __device__ __forceinline__ double sqrt_(double x) { return sqrt(x); }
};

template <typename R>
__device__ __forceinline__ R pos(R x) {
  return x > R(0) ? x : R(0);
}

// Running state of one path.
template <typename R>
struct GbmState {
  R z;       // log scheme: log(S/S0) in the kernel's domain; Euler-S: S/S0
  R sumE;    // sum of S_i/S0            (Asian)
  R sumz;    // sum of log(S_i/S0)       (geometric Asian)
  R sumZ;    // sum of the normals       (vega)
  R dsig;    // Euler-S: d(S_i/S0)/dsigma
  R accV;    // sum of d(S_i/S0)/dsigma  (Asian vega)
  R top;     // running maximum of z (discrete barrier)
  R top_bb;  // running maximum of twice the bridge's maxima

  __device__ __forceinline__ void start(bool log_scheme) {
    z = log_scheme ? R(0) : R(1);
    sumE = sumz = sumZ = dsig = accV = R(0);
    top = top_bb = -R(__builtin_inff());
  }
};

template <typename R, uint32_t MASK, bool LOGS>
struct GbmStepper {
  // The barrier is watched through the running maximum: two dates per
  // v_max3_f32, where a compare and a mask update per date took twice as
  // long, and one maximum serves both levels of a bumped pair. (Folding the
  // volatility into Box-Muller's radius would save another multiply per step,
  // 3% of the FP32 kernel; it rounds every state differently, and single
  // paths then cross the barrier that did not before.)
  R dz, vz, cbb, sdt, sig, dt, rdt, vsdt;
  const PathMath<R>& pm;

  __device__ __forceinline__ GbmStepper(const GbmParams& P, const PathMath<R>& math) : pm(math) {
    dz = (R)P.drift_dom;
    vz = (R)P.vol_dom;
    cbb = (R)P.bridge_c;
    sdt = (R)P.sdt;
    sig = (R)P.sigma;
    dt = (R)P.dt;
    rdt = (R)P.r_dt;
    vsdt = (R)P.vol_sdt;
  }

  // Step i -> i+1 with normal Z (and the bridge's uniform of word W when
  // monitored).
  __device__ __forceinline__ void step(GbmState<R>& s, R Z, uint32_t i, uint32_t W) const {
    if constexpr (LOGS) {
      const R zp = s.z;
      s.z = s.z + dz + vz * Z;
      R E = R(0);
      if constexpr ((MASK & (G_ASIAN | G_ASIAN_G)) != 0) {
        E = Dom<R>::exp_(s.z, pm);
        s.sumE += E;
      }
      if constexpr ((MASK & G_GEO) != 0) s.sumz += s.z;
      if constexpr ((MASK & G_UO) != 0) s.top = Dom<R>::max_(s.top, s.z);
      if constexpr ((MASK & (G_EURO_G | G_ASIAN_G)) != 0) s.sumZ += Z;
      if constexpr ((MASK & G_ASIAN_G) != 0)
        s.accV += E * (sdt * s.sumZ - sig * (dt * (R)(i + 1)));
      if constexpr ((MASK & G_UOBB) != 0) {
        // Maximum of the Brownian bridge between z_i and z_{i+1}.
        const R d = zp - s.z;
        const R twice_max = zp + s.z + Dom<R>::sqrt_(d * d + cbb * Dom<R>::neg_log_(W, pm));
        s.top_bb = Dom<R>::max_(s.top_bb, twice_max);
      }
    } else {
      const R inc = rdt + vsdt * Z;           // S_{i+1}/S_i - 1
      if constexpr ((MASK & (G_EURO_G | G_ASIAN_G)) != 0) s.dsig = s.dsig * (R(1) + inc) + s.z * sdt * Z;
      s.z = s.z + s.z * inc;
      if constexpr ((MASK & (G_ASIAN | G_ASIAN_G)) != 0) s.sumE += s.z;
      if constexpr ((MASK & G_GEO) != 0) s.sumz += log(s.z);
      if constexpr ((MASK & G_UO) != 0) s.top = Dom<R>::max_(s.top, s.z);
      if constexpr ((MASK & G_ASIAN_G) != 0) s.accV += s.dsig;
    }
  }
};

// The normals of one path: step(q, Z, W) for q = 0 .. n - 1 in order, W the
// bridge's uniform word (BRIDGE).
template <typename R, bool BRIDGE, typename F>
__device__ __forceinline__ void walk_normals(uint32_t n, uint32_t tag, uint32_t lo, uint32_t hi,
                                             const PhiloxKeys& keys, const PathMath<R>& pm,
                                             F&& step) {
  const PathRng pc = make_rng(lo, hi, tag, keys);
  const PathRng pcb = make_rng(lo, hi, tag + 5u, keys);
  const uint32_t n_full = n >> 2, rem = n & 3u;
  for (uint32_t j = 0; j < n_full; ++j) {
    const Normals4<R> nz = normals4(philox(j, pc, keys), pm);
    Words4 wb{0, 0, 0, 0};
    if constexpr (BRIDGE) wb = philox(j, pcb, keys);
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) step(4 * j + q, nz.z[q], word_at(wb, q));
  }
  if (rem) {
    const Normals4<R> nz = normals4(philox(n_full, pc, keys), pm);
    Words4 wb{0, 0, 0, 0};
    if constexpr (BRIDGE) wb = philox(n_full, pcb, keys);
#pragma unroll
    for (uint32_t q = 0; q < 3; ++q) {
      if (q >= rem) break;
      step(4 * n_full + q, nz.z[q], word_at(wb, q));
    }
  }
}

// Discounted payoff of functional BIT (one bit) from a path's final state;
// En = S_n / S0; P supplies S0, strike, discount factor and barrier.
template <typename R, uint32_t BIT, bool LOGS>
__device__ __forceinline__ double payoff_of(const GbmParams& P, const GbmState<R>& s, R En,
                                            const PathMath<R>& pm) {
  const R S0 = (R)P.S0, K = (R)P.K, disc = (R)P.disc, inv_n = R(1) / (R)P.n_steps;
  const R ST = S0 * En;
  const R call = pos(ST - K);
  if constexpr (BIT == G_EURO) return (double)(disc * call);
  if constexpr (BIT == G_ASIAN) {
    const R A = S0 * s.sumE * inv_n;
    return (double)(disc * pos(A - K));
  }
  if constexpr (BIT == G_GEO) {
    const R G = LOGS ? S0 * Dom<R>::exp_(s.sumz * inv_n, pm)
                     : S0 * (R)exp((double)s.sumz / (double)P.n_steps);
    return (double)(disc * pos(G - K));
  }
  if constexpr (BIT == G_UO) {
    const R level = (R)(LOGS ? P.barrier_dom : P.barrier_rel);
    return s.top < level ? (double)(disc * call) : 0.0;
  }
  const R level = (R)P.barrier_dom;
  return s.top_bb < R(2) * level ? (double)(disc * call) : 0.0;
}

}  // namespace mcp
