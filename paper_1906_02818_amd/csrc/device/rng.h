// Device random numbers for the path kernels: Philox4x32-10, the open-interval
// uniform and Box-Muller (keyed counter-based PRNG of Sec. IV-A; Box-Muller as
// the paper uses it for Sobol points in Sec. VI-D).
//
// Counter layout: normal k of path p in stream `tag` is slot k mod 4 of the
// block with counter (floor(k/4), p mod 2^32, p >> 32, tag) and key
// (seed mod 2^32, seed >> 32). Words (w0, w1) give slots 0, 1 as
// r(w0) cos(2 pi u(w1)), r(w0) sin(2 pi u(w1)); (w2, w3) give slots 2, 3.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fp64.h"

namespace mcp {

constexpr uint32_t kPhiloxM0 = 0xD2511F53u;
constexpr uint32_t kPhiloxM1 = 0xCD9E8D57u;
constexpr uint32_t kPhiloxW0 = 0x9E3779B9u;
constexpr uint32_t kPhiloxW1 = 0xBB67AE85u;

struct Words4 {
  uint32_t w0, w1, w2, w3;
};

// The per-path part of the counter and the key. c1, c2, c3 do not change
// along a path, so the first round's product of c2 is loop invariant.
struct PathCounter {
  uint32_t c1, c2, c3;  // path lo, path hi, tag
  uint32_t k0, k1;      // key (uniform across the launch: scalar registers)
};

__device__ __forceinline__ PathCounter make_counter(uint64_t path, uint32_t tag,
                                                    uint32_t k0, uint32_t k1) {
  PathCounter pc;
  pc.c1 = (uint32_t)path;
  pc.c2 = (uint32_t)(path >> 32);
  pc.c3 = tag;
  pc.k0 = k0;
  pc.k1 = k1;
  return pc;
}

__device__ __forceinline__ void mul_hi_lo(uint32_t a, uint32_t b, uint32_t& hi,
                                          uint32_t& lo) {
  const uint64_t p = (uint64_t)a * (uint64_t)b;
  hi = (uint32_t)(p >> 32);
  lo = (uint32_t)p;
}

// Ten Philox rounds on counter (j, c1, c2, c3).
__device__ __forceinline__ Words4 philox(uint32_t j, const PathCounter& pc) {
  uint32_t c0 = j, c1 = pc.c1, c2 = pc.c2, c3 = pc.c3;
  uint32_t k0 = pc.k0, k1 = pc.k1;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    uint32_t hi0, lo0, hi1, lo1;
    mul_hi_lo(kPhiloxM0, c0, hi0, lo0);
    mul_hi_lo(kPhiloxM1, c2, hi1, lo1);
    // Three-input xors: one v_bitop3_b32 each (truth table 0x96 = a^b^c).
    const uint32_t n0 = __builtin_amdgcn_bitop3_b32(hi1, c1, k0, 0x96);
    const uint32_t n2 = __builtin_amdgcn_bitop3_b32(hi0, c3, k1, 0x96);
    c0 = n0;
    c1 = lo1;
    c2 = n2;
    c3 = lo0;
    k0 += kPhiloxW0;
    k1 += kPhiloxW1;
  }
  return Words4{c0, c1, c2, c3};
}

// The form of the path kernels, where a lane follows one path and every lane
// of the wave draws the same block index j at the same time.
//
// On gfx950 an FP32 fma / add / mul, a xor and a v_bitop3_b32 issue in about
// 2.5 cycles per wave when all their operands are VGPRs or constants, and in
// 4.3 (the rate of v_mad_u64_u32) as soon as one operand is an SGPR. The
// round keys are uniform, so the compiler would keep them in SGPRs; make_keys
// pins them in VGPRs (an asm statement hides the uniformity), 13 of the 17
// xors of a block take the fast form, and 4 fold one scalar.
//
// Of a block's 20 products, those of j and of the high word of the path index
// (uniform: see with_uniform_high) are scalar through the third round, and
// one of round 2 is a constant of the path: 15 remain.
//
// Measured on the Asian + geometric + barrier call of 2^24 GBM paths x 252
// steps: 2.21 ms with SGPR keys and 18 products (two of them as v_mul_lo /
// v_mul_hi pairs), 2.02 ms in this form. Per block and wave: 64 cycles of
// products, 53 of xors, of about 305 for the four steps.
struct PhiloxKeys {
  uint32_t a[10], b[10];   // round keys k0 + r W0, k1 + r W1
};

__device__ __forceinline__ uint32_t in_vgpr(uint32_t x) {
  uint32_t y;
  asm volatile("v_mov_b32 %0, %1" : "=v"(y) : "s"(x));
  return y;
}
__device__ __forceinline__ float in_vgpr(float x) {
  return __uint_as_float(in_vgpr(__float_as_uint(x)));
}

__device__ __forceinline__ uint64_t mul_wide(uint32_t a, uint32_t m) { return (uint64_t)a * m; }

// PIN = false leaves the keys to the compiler (SGPRs): double-precision
// kernels, where the 13 VGPRs cost more than the xors.
template <bool PIN>
__device__ __forceinline__ PhiloxKeys make_keys(uint32_t k0, uint32_t k1) {
  PhiloxKeys k;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    // Rounds 0 .. 2 and one key of round 3 enter scalar expressions.
    k.a[r] = k0 + (uint32_t)r * kPhiloxW0;
    k.b[r] = k1 + (uint32_t)r * kPhiloxW1;
    if (PIN && r >= 3) k.a[r] = in_vgpr(k.a[r]);
    if (PIN && r >= 4) k.b[r] = in_vgpr(k.b[r]);
  }
  return k;
}

// One path's generator: stream `tag`, path index (hi, lo), hi uniform.
struct PathRng {
  uint32_t tag, c1;        // uniform: the stream; low word of M1 hi
  uint32_t a_hi, a_lo;     // round 2's product of the path's word (per lane)
};

__device__ __forceinline__ PathRng make_rng(uint32_t lo, uint32_t hi, uint32_t tag,
                                            const PhiloxKeys& k) {
  PathRng g;
  uint32_t h1;
  mul_hi_lo(kPhiloxM1, hi, h1, g.c1);
  const uint64_t p = mul_wide(lo ^ (h1 ^ k.a[0]), kPhiloxM0);
  g.a_hi = (uint32_t)(p >> 32);
  g.a_lo = (uint32_t)p;
  g.tag = tag;
  return g;
}

// Ten Philox rounds on counter (j, path lo, path hi, tag), j uniform.
__device__ __forceinline__ Words4 philox(uint32_t j, const PathRng& g, const PhiloxKeys& k) {
  uint32_t jh, jl, bh, bl, ch, cl;
  mul_hi_lo(kPhiloxM0, j, jh, jl);                          // round 1, scalar
  mul_hi_lo(kPhiloxM1, jh ^ g.tag ^ k.b[0], bh, bl);        // round 2, scalar half
  mul_hi_lo(kPhiloxM0, bh ^ g.c1 ^ k.a[1], ch, cl);         // round 3, scalar half
  const uint64_t d = mul_wide(g.a_hi ^ (jl ^ k.b[1]), kPhiloxM1);
  uint32_t c0 = (uint32_t)(d >> 32) ^ (bl ^ k.a[2]);
  uint32_t c1 = (uint32_t)d;
  uint32_t c2 = g.a_lo ^ (ch ^ k.b[2]);
  uint64_t e = mul_wide(c0, kPhiloxM0), f = mul_wide(c2, kPhiloxM1);   // round 4
  c0 = __builtin_amdgcn_bitop3_b32((uint32_t)(f >> 32), c1, k.a[3], 0x96);
  c2 = (uint32_t)(e >> 32) ^ (cl ^ k.b[3]);
#pragma unroll
  for (int r = 4; r < 10; ++r) {
    const uint32_t c3 = (uint32_t)e;
    c1 = (uint32_t)f;
    e = mul_wide(c0, kPhiloxM0);
    f = mul_wide(c2, kPhiloxM1);
    c0 = __builtin_amdgcn_bitop3_b32((uint32_t)(f >> 32), c1, k.a[r], 0x96);
    c2 = __builtin_amdgcn_bitop3_b32((uint32_t)(e >> 32), c3, k.b[r], 0x96);
  }
  return Words4{c0, (uint32_t)f, c2, (uint32_t)e};
}

// Calls f(hi) for each lane's path index, hi its high word as a uniform
// value. The lanes of a wave hold consecutive paths in lane order, so a wave
// meets a second high word only where it straddles a multiple of 2^32; the
// lanes past it (low word wrapped) then take a second pass.
template <typename F>
__device__ __forceinline__ void with_uniform_high(uint64_t path, F&& f) {
  const uint32_t lo0 = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)path);
  const uint32_t hi0 = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(path >> 32));
  const bool wrapped = (uint32_t)path < lo0;
  const uint32_t passes = __ballot(wrapped) != 0ull ? 2u : 1u;
  for (uint32_t p = 0; p < passes; ++p)
    if (wrapped == (p != 0u)) f(hi0 + p);
}

// u(w) = (2 (w >> 9) + 1) 2^-24, exact in FP32: the top 23 bits fill the
// mantissa of a float in [1, 2), and subtracting 1 - 2^-24 is exact.
__device__ __forceinline__ float uniform_f32(uint32_t w) {
  // (0x7F:w) >> 9 = 0x3F800000 | (w >> 9) in one v_alignbit_b32.
  return __uint_as_float(__builtin_amdgcn_alignbit(0x7Fu, w, 9u)) - 0x1.fffffep-1f;
}

__device__ __forceinline__ double uniform_f64(uint32_t w) {
  return (double)(2u * (w >> 9) + 1u) * 0x1p-24;
}

// Box-Muller in FP32 on the hardware transcendental units:
// v_log_f32 is log2, so -2 ln u = (-2 ln 2) log2 u; v_sin_f32 / v_cos_f32
// take their argument in revolutions, so sin(2 pi u) is sin_rev(u).
__device__ __forceinline__ void box_muller_f32(uint32_t w_rad, uint32_t w_ang, float& z0,
                                               float& z1) {
  const float ur = uniform_f32(w_rad);
  const float ua = uniform_f32(w_ang);
  const float rad = __builtin_amdgcn_sqrtf(-1.38629436111989061883f * __builtin_amdgcn_logf(ur));
  z0 = rad * __builtin_amdgcn_cosf(ua);
  z1 = rad * __builtin_amdgcn_sinf(ua);
}

template <typename R>
struct Normals4 {
  R z[4];
};

// What a path's arithmetic in R needs beside its state: nothing in FP32 (the
// hardware's transcendental unit), the workgroup's tables in FP64.
template <typename R>
struct PathMath;
template <>
struct PathMath<float> {
  struct Shared {};
  __device__ __forceinline__ explicit PathMath(Shared&) {}
};
template <>
struct PathMath<double> {
  typedef F64Tables Shared;
  const F64Tables& t;
  // Fills the tables (every thread of the workgroup calls it).
  __device__ __forceinline__ explicit PathMath(Shared& s) : t(s) {
    f64_tables_fill(s);
    __syncthreads();
  }
};

__device__ __forceinline__ Normals4<float> normals4(const Words4& w) {
  Normals4<float> n;
  box_muller_f32(w.w0, w.w1, n.z[0], n.z[1]);
  box_muller_f32(w.w2, w.w3, n.z[2], n.z[3]);
  return n;
}
template <bool ROUND_ANGLE = false>
__device__ __forceinline__ Normals4<float> normals4(const Words4& w, const PathMath<float>&) {
  return normals4(w);
}
template <bool ROUND_ANGLE = false>
__device__ __forceinline__ Normals4<double> normals4(const Words4& w,
                                                     const PathMath<double>& pm) {
  Normals4<double> n;
  box_muller_f64<ROUND_ANGLE>(w.w0, w.w1, pm.t, n.z[0], n.z[1]);
  box_muller_f64<ROUND_ANGLE>(w.w2, w.w3, pm.t, n.z[2], n.z[3]);
  return n;
}

__device__ __forceinline__ uint32_t word_at(const Words4& w, uint32_t s) {
  return s == 0 ? w.w0 : s == 1 ? w.w1 : s == 2 ? w.w2 : w.w3;
}

}  // namespace mcp
