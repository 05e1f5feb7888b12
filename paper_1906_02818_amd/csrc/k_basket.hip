// Basket path kernel: d correlated GBM assets stepped by log-Euler (the
// multivariate Euler-Maruyama scheme of Sec. II-A.2). A step adds the
// correlated increment L' Z_i, L' = diag(sigma_a sqrt(dt)) L, to the vector of
// log-prices and the payoffs read only its last value, so
//     sum_i L' Z_i = L' (sum_i Z_i):
// every step's normals are drawn and summed, and the product with L' (the
// matrix-unit product of Sec. VI-A.2) is taken once per path, on the matrix
// cores, instead of once per step. The drift n (r - sigma_a^2/2) dt is added
// there too.
//
// Sums. A lane follows one path and a wave takes four assets (one Philox
// block) through all steps, so the block index is uniform (device/rng.h), four
// registers hold the sums, and any number of waves can share a tile of 64
// paths. The sums go to LDS as [asset][path]. Reduced precisions round each
// step's normals as an operand of their products would be rounded: to
// bfloat16 (two steps' normals per conversion, both added by one
// v_dot2_f32_bf16) or half. The sums are FP32 in every case.
//
// Product. X = L' S per tile by 16x16x32 MFMAs, rows = assets, columns = 16
// paths; wave w takes path columns w mod 4 and up to four 16-asset row blocks,
// paired so that every wave has the same share of the triangle. The FP32 sums
// enter as up to three terms of the 16-bit type (8 + 8 + 8 bits), and so does
// an FP32 L', with the products of terms above 2^-24 kept: the FP32 form is
// six bfloat16 MFMAs for the eight FP32 ones of the same block, 96 cycles
// against 256. Error of a path's value against 64 bits (root mean square over
// the paths, of their spread), product per step in FP32 -> here: portfolio of
// 112 assets x 50 steps 3.0e-7 -> 1.6e-7, 64 x 30 2.4e-7 -> 1.4e-7, 16 x 3
// 1.3e-7 -> 1.2e-7 (8 keys each); baskets of 16 to 256 assets 2.7e-7 to 3.0e-7
// -> 1.5e-7. Error of the portfolio's standard error: 2.6e-8 -> 1.8e-8.
//
// Bound: VALU issue of the normals, 222 cycles per block of four and wave in
// FP32, 244 in bfloat16 (issue costs: device/rng.h; 4.3 for a conversion or a
// v_dot2). Path kernel, product per step -> product per path: 2^18 paths x 100
// steps x 256 assets in bfloat16 3.70 -> 2.70 ms (2.60 ms of issue), the
// portfolio of 100003 x 50 x 112 in FP32 1.21 -> 0.26 ms (0.20 ms). A product
// per step spent 0.2 and 0.75 of its time in MFMAs, which on gfx950 do not run
// beside FP32 VALU work of the same SIMD: an MFMA stream and an FMA stream of
// 0.245 and 0.219 ms in different waves take 0.434 ms.
#include <type_traits>

#include "device/reduce.h"
#include "device/rng.h"
#include "mc_internal.h"

namespace mcp {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;

constexpr int kQmcWaves = 4;              // waves of a QMC workgroup: a tile each
constexpr int kTile = kBasketTile;        // paths per tile: one per lane
constexpr int kRow = kTile + 2;           // LDS row of an asset's sums: rows 8 apart
                                          // fall 16 banks apart (fragment reads)

// NL, NZ: terms of L' and of the sums; KEEP: a product of terms i and j is
// taken when i + j < KEEP.
template <int PREC>
struct Form;
template <>
struct Form<BK_FP32> {
  typedef bf16x8 V;
  static constexpr int NL = 3, NZ = 3, KEEP = 3;
};
template <>
struct Form<BK_BF16> {
  typedef bf16x8 V;
  static constexpr int NL = 1, NZ = 3, KEEP = 3;
};
template <>
struct Form<BK_BF16X2> {
  typedef bf16x8 V;
  static constexpr int NL = 2, NZ = 3, KEEP = 3;
};
template <>
struct Form<BK_FP16> {
  typedef f16x8 V;
  static constexpr int NL = 1, NZ = 2, KEEP = 2;
};

__device__ __forceinline__ void mma(f32x4& acc, const bf16x8& a, const bf16x8& b) {
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
}
__device__ __forceinline__ void mma(f32x4& acc, const f16x8& a, const f16x8& b) {
  acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, acc, 0, 0, 0);
}

// s += the normals of one or two steps (blocks a, b; two: b holds a step),
// rounded as PREC's operands are. FP32 sums the normals over sqrt(2 ln 2), the
// factor of every radius, which L' carries: one fma per normal.
template <int PREC>
__device__ __forceinline__ void add_steps(float (&s)[4], const Words4& a, const Words4& b,
                                          bool two) {
  if constexpr (PREC == BK_FP32) {
    auto add = [&](const Words4& w) {
      const uint32_t wr[2] = {w.w0, w.w2}, wa[2] = {w.w1, w.w3};
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const float ua = uniform_f32(wa[h]);
        const float rad = __builtin_amdgcn_sqrtf(-__builtin_amdgcn_logf(uniform_f32(wr[h])));
        s[2 * h] = __builtin_fmaf(rad, __builtin_amdgcn_cosf(ua), s[2 * h]);
        s[2 * h + 1] = __builtin_fmaf(rad, __builtin_amdgcn_sinf(ua), s[2 * h + 1]);
      }
    };
    add(a);
    if (two) add(b);
  } else {
    const Normals4<float> na = normals4(a);
    Normals4<float> nb = {{0.f, 0.f, 0.f, 0.f}};
    if (two) nb = normals4(b);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      if constexpr (PREC == BK_FP16) {
        // The FP32 normal rounds to half: not the exact product of its radius
        // and sine, which a v_fma_mixlo_f16 would round.
        float za = na.z[t], zb = nb.z[t];
        asm("" : "+v"(za));
        asm("" : "+v"(zb));
        s[t] += (float)(_Float16)za;
        s[t] += (float)(_Float16)zb;
      } else {
        const bf16x2 p = __builtin_convertvector((f32x2){na.z[t], nb.z[t]}, bf16x2);
        const bf16x2 one = {(__bf16)1.0f, (__bf16)1.0f};
        s[t] = __builtin_amdgcn_fdot2_f32_bf16(p, one, s[t], false);
      }
    }
  }
}

// Words of one block of four Sobol' dimensions (dims 4j .. 4j+3) for the
// points base + lane, each xored with its digital shift. V and shift are
// read as scalars; the bits of the point index that are the same for all
// lanes (above the sixth when the base is a multiple of 64) are folded on the
// scalar unit.
__device__ __forceinline__ Words4 sobol_words(const uint32_t* __restrict__ V,
                                              const uint32_t* __restrict__ shift, uint32_t j,
                                              uint32_t base, uint32_t lane) {
  const uint32_t* v = V + (size_t)j * 128u;
  const uint32_t last = base + 63u < base ? 0xFFFFFFFFu : base + 63u;   // points end at 2^32
  const uint32_t bits = 32u - (uint32_t)__builtin_clz(last | 63u);
  const uint32_t split = (base & 63u) == 0u ? 6u : bits;
  uint32_t u[4], x[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) u[t] = shift[4u * j + t];
  for (uint32_t b = split; b < bits; ++b) {
    const uint32_t m = 0u - ((base >> b) & 1u);
#pragma unroll
    for (int t = 0; t < 4; ++t) u[t] ^= m & v[32 * t + b];
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) x[t] = u[t];
  const uint32_t point = base + lane;
  for (uint32_t b = 0; b < split; ++b) {
    const uint32_t m = 0u - ((point >> b) & 1u);
#pragma unroll
    for (int t = 0; t < 4; ++t) x[t] ^= m & v[32 * t + b];
  }
  return Words4{x[0], x[1], x[2], x[3]};
}

// Term t of v in the 16-bit type: bfloat16 terms are each the rounding of what
// the earlier ones leave of the double (three: 26 bits); half has one.
__device__ __forceinline__ uint16_t to_bf16(float f) {
  const uint32_t u = __float_as_uint(f);
  return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}
template <int PREC>
__device__ __forceinline__ void split_terms(double v, uint16_t (&h)[Form<PREC>::NL]) {
  if constexpr (PREC == BK_FP16) {
    const _Float16 x = (_Float16)(float)v;
    __builtin_memcpy(&h[0], &x, 2);
  } else {
    double rest = v;
#pragma unroll
    for (int t = 0; t < Form<PREC>::NL; ++t) {
      h[t] = to_bf16((float)rest);
      rest -= (double)__uint_as_float((uint32_t)h[t] << 16);
    }
  }
}

// L' carries, in FP64, what is common to all sums: a constant applied to them
// in FP32 instead (sqrt(2 ln 2) of the FP32 form, 1.4e-8 off) shows in every
// standard deviation, where the roundings of single paths average out.
//
// One workgroup per four fragments of L' (a lane writes its eight entries of
// each term), one for the asset table, and the words to clear. Latency of a
// launch and of reads over PCIe; 4 us.
template <int PREC>
__global__ __launch_bounds__(256) void basket_pack_kernel(const BasketPack K) {
  constexpr int NL = Form<PREC>::NL;
  const uint32_t n_pairs = basket_pairs(K.d >> 4);
  const uint32_t gid = blockIdx.x * 256u + threadIdx.x;
  for (int z = 0; z < 2; ++z)
    for (uint32_t i = gid; i < K.zero[z].n; i += gridDim.x * 256u) K.zero[z].words[i] = 0u;
  if (blockIdx.x == gridDim.x - 1u) {
    for (uint32_t i = threadIdx.x; i < 4u * 256u; i += 256u)
      if ((i & 255u) < K.d) K.asset_out[i] = K.asset[i];
    return;
  }
  const uint32_t pair = gid >> 6, lane = gid & 63u;
  if (pair >= n_pairs) return;
  uint32_t rb = 0;
  while (basket_pairs(rb + 1u) <= pair) ++rb;
  const uint32_t kb = pair - basket_pairs(rb);
  const uint32_t a = 16u * rb + (lane & 15u), b0 = 32u * kb + 8u * (lane >> 4);
  const double scale = K.sigma[a] * K.step;
  uint16_t h[8][NL];
#pragma unroll
  for (uint32_t e = 0; e < 8u; ++e) {
    const uint32_t b = b0 + e;
    split_terms<PREC>(b <= a ? scale * K.L[(size_t)a * K.d + b] : 0.0, h[e]);
  }
#pragma unroll
  for (int t = 0; t < NL; ++t) {
    uint16_t* out = K.frag + (((size_t)t * n_pairs + pair) * 64u + lane) * 8u;
#pragma unroll
    for (uint32_t e = 0; e < 8u; ++e) out[e] = h[e][t];
  }
}

// Sums of the normals of assets 4q .. 4q + 3 over the steps, to their LDS rows;
// words(j): Philox or Sobol' block j.
template <int PREC, typename F>
__device__ __forceinline__ void sum_block(float* s_sum, uint32_t n, uint32_t nq, uint32_t q,
                                          int lane, F&& words) {
  float s[4] = {0.f, 0.f, 0.f, 0.f};
  uint32_t i = 0;
  for (; i + 1 < n; i += 2) {
    const Words4 a = words(i * nq + q), b = words((i + 1) * nq + q);
    add_steps<PREC>(s, a, b, true);
  }
  if (i < n) {
    const Words4 a = words(i * nq + q);
    add_steps<PREC>(s, a, a, false);
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) s_sum[(4u * q + t) * kRow + lane] = s[t];
}

// One step leaves sums of one term in the reduced precisions.
template <int PREC>
__device__ __forceinline__ uint32_t sum_terms(uint32_t n) {
  return n == 1u && PREC != BK_FP32 ? 1u : (uint32_t)Form<PREC>::NZ;
}

// Terminal values of the lane's four assets 16 rb + 4 (lane / 16) + 0..3 of a
// path: basket and geometric-basket sums (or the portfolio's value), and the
// growth of asset 0. QMC: the basket's sum is of S_a / S0_a - 1, whose FP32
// roundings are smaller (P.base, the sum of the ones, joins it in FP64): the
// standard error of a few replicates shows what does not average out (its
// error, 16 replicates of 2^16 points: 7.0e-7 without, 4.3e-7 with).
template <bool PORT, bool QMC>
__device__ __forceinline__ void terminal_rows(const BasketParams& P, const f32x4& x, uint32_t rb,
                                              uint32_t g4, float& bs, float& gs, float& e0) {
  // The four assets by themselves first: a lane has up to 32.
  float b = 0.f, g = 0.f;
#pragma unroll
  for (uint32_t r = 0; r < 4u; ++r) {
    const uint32_t a = 16u * rb + 4u * g4 + r;
    const float v = x[r] * P.x_scale + P.asset[a];        // log2(S_a / S0_a)
    const float E = __builtin_amdgcn_exp2f(v);
    if constexpr (PORT) {
      // Portfolio value of asset a: S0_a sum_k q_k (E - m_k)^+.
      float pv = 0.f;
      for (uint32_t k = 0; k < P.n_strikes; ++k) {
        const float itm = E - P.pm[k];
        pv = __builtin_fmaf(P.pq[k], itm > 0.f ? itm : 0.f, pv);
      }
      b = __builtin_fmaf(P.asset[768 + a], pv, b);
    } else {
      b += P.asset[256 + a] * (QMC ? E - 1.0f : E);
      g += P.asset[512 + a] * v;
      if (a == 0u) e0 = E;
    }
  }
  bs += b;
  gs += g;
}

// Channels of a path from its sums v.
template <bool PORT, bool QMC, int C, typename R>
__device__ __forceinline__ void channels(const BasketParams& P, const R (&v)[C],
                                         double (&y)[C]) {
  if constexpr (PORT) {
    y[0] = (double)v[0] * P.ratio - P.premium;
  } else {
    const double disc = P.disc, K = P.K;
    const double basket = QMC ? P.base + (double)v[0] : (double)v[0];
    const double geo = exp(P.geo0 + (double)v[1]);
    y[0] = disc * (basket > K ? basket - K : 0.0);
    y[1] = disc * (geo > K ? geo - K : 0.0);
    y[2] = basket > K ? disc * P.w0 * (double)v[2] : 0.0;
  }
}

// Row block i of the wave's set of the triangle's 16-row blocks, S sets per
// workgroup: consecutive pairs sum to a constant, so the sets have equal
// shares of the triangle.
template <int S>
__device__ __forceinline__ uint32_t row_block(uint32_t set, uint32_t i) {
  if constexpr (S == 1) return i;
  return 2u * S * (i >> 1) + ((i & 1u) ? 2u * S - 1u - set : set);
}

// RPW: 16-row blocks per wave (d <= 4 W RPW). SPLIT: the tiles from
// P.split_from on have P.split_parts workgroups each, of one Philox block of
// assets per wave; they put their sums in P.split_sums and the last to arrive
// takes the product.
template <int PREC, bool PORT, bool QMC, int W, int RPW, bool SPLIT = false>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(4))) void basket_kernel(const BasketParams P) {
  stamp(P.clock);
  typedef Form<PREC> F;
  typedef typename F::V V8;
  constexpr int SETS = W / 4, C = PORT ? 1 : 3;
  extern __shared__ float s_sum[];         // [d][kRow]
  // The sums over a path's lanes in FP64, where their rounding would be the
  // largest of a path: per path 3.0e-7 -> 1.5e-7 of the spread in FP32 (16 to
  // 256 assets), at the same time. In the reduced precisions, whose operands
  // round to 2e-4 and more, it costs 5% (basket, bfloat16: 2715 -> 2844 us) and
  // shows in no digit.
  constexpr bool kSums64 = QMC || PREC == BK_FP32;
  typedef typename std::conditional<kSums64, double, float>::type Sum;
  __shared__ Sum s_part[C][SETS][kTile];
  // The first wave's paths over the workgroup's tiles (in LDS: as registers
  // they would be held by every wave). About a shift: a lane takes 2^18 paths
  // of the longest runs, and a portfolio's values can be equal.
  __shared__ PartSums<C> s_acc[kTile];
  const int lane = threadIdx.x & 63;
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // Block blk of nblk of the launch, or of its replicate when replicates
  // share it.
  uint32_t blk = blockIdx.x, nblk = gridDim.x;
  const uint32_t* qshift = P.qshift;
  double* partials = P.partials;
  if constexpr (QMC) {
    if (P.q_rep_blocks != 0) {
      nblk = P.q_rep_blocks;
      const uint32_t rep = blockIdx.x / nblk;
      blk = blockIdx.x - rep * nblk;
      qshift += (size_t)rep * P.q_dims;
      partials += (size_t)rep * n_moments(C) * nblk;
    }
  }
  const uint32_t d = P.d, n = P.n_steps, nq = d >> 2, rows = d >> 4;
  const PhiloxKeys keys = make_keys<true>(P.k0, P.k1);
  if (threadIdx.x < kTile) s_acc[threadIdx.x].zero();

  const uint64_t tiles = (P.n_paths + kTile - 1) / kTile;
  uint32_t piece = ~0u;                    // SPLIT: the workgroup's part of its tile
  if constexpr (SPLIT) {
    nblk = (uint32_t)tiles;                // one tile, or part of one, per workgroup
    if (blk >= P.split_from) {
      const uint32_t i = blk - P.split_from;
      blk = P.split_from + i / P.split_parts;
      piece = i % P.split_parts;
    }
  }
  for (uint64_t tile = blk; tile < tiles; tile += nblk) {
    // ---- sums of the normals ----
    const uint64_t path = P.path_offset + tile * kTile + (uint64_t)lane;
    if constexpr (QMC) {
      const uint32_t base = (uint32_t)(P.path_offset + tile * kTile);
      for (uint32_t q = wave; q < nq; q += W)
        sum_block<PREC>(s_sum, n, nq, q, lane, [&](uint32_t j) {
          return sobol_words(P.qV, qshift, j, base, (uint32_t)lane);
        });
    } else {
      with_uniform_high(path, [&](uint32_t hi) {
        const PathRng g = make_rng((uint32_t)path, hi, P.tag, keys);
        if constexpr (SPLIT) {
          const bool whole = piece == ~0u;
          const uint32_t q0 = whole ? wave : piece * W + wave, q1 = whole ? nq : q0 + 1u;
          for (uint32_t q = q0; q < q1 && q < nq; q += W)
            sum_block<PREC>(s_sum, n, nq, q, lane, [&](uint32_t j) { return philox(j, g, keys); });
        } else {
          for (uint32_t q = wave; q < nq; q += W)
            sum_block<PREC>(s_sum, n, nq, q, lane, [&](uint32_t j) { return philox(j, g, keys); });
        }
      });
    }
    if constexpr (SPLIT) {
      if (piece != ~0u) {
        const uint32_t i = blk - P.split_from, q = piece * W + wave;
        float* rows_of = P.split_sums + (size_t)i * d * kTile;
        if (q < nq) {
#pragma unroll
          for (uint32_t t = 0; t < 4u; ++t)
            store_agent(&rows_of[(4u * q + t) * kTile + lane], s_sum[(4u * q + t) * kRow + lane]);
        }
        if (!arrives_last(&P.split_arrivals[i], P.split_parts)) return;
        for (uint32_t e = threadIdx.x; e < d * kTile; e += 64u * W)
          s_sum[(e / kTile) * kRow + e % kTile] = load_agent(&rows_of[e]);
      }
    }
    __syncthreads();

    // ---- X = L' S: columns `col` (16 paths), rows of the wave's set ----
    const uint32_t col = wave & 3u, set = wave >> 2;
    const uint32_t c16 = (uint32_t)lane & 15u, g4 = (uint32_t)lane >> 4;
    f32x4 x[RPW];
#pragma unroll
    for (int i = 0; i < RPW; ++i) x[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
    const uint32_t nz = sum_terms<PREC>(n);
    const uint32_t n_pairs = (uint32_t)basket_pairs(rows);
    for (uint32_t kb = 0; 32u * kb < d; ++kb) {
      // The column operand: sums of assets 32 kb + 8 g4 + 0..7, path c16.
      V8 z[F::NZ];
      {
        const uint32_t k0 = 32u * kb + 8u * g4;
        float r[8];
#pragma unroll
        for (uint32_t e = 0; e < 8u; ++e)
          r[e] = k0 < d ? s_sum[(k0 + e) * kRow + 16u * col + c16] * P.z_scale : 0.f;
#pragma unroll
        for (int t = 0; t < F::NZ; ++t)
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            z[t][e] = r[e];
            r[e] -= (float)z[t][e];
          }
      }
#pragma unroll
      for (uint32_t i = 0; i < (uint32_t)RPW; ++i) {
        const uint32_t rb = row_block<SETS>(set, i);
        if (rb < rows && 2u * kb <= rb) {
          const V8* a = (const V8*)P.Lfrag + ((size_t)basket_pairs(rb) + kb) * 64u + lane;
#pragma unroll
          for (int p = 0; p < F::NL; ++p) {
            const V8 l = a[(size_t)p * n_pairs * 64u];
#pragma unroll
            for (int t = 0; t < F::NZ; ++t)
              if (p + t < F::KEEP && (uint32_t)t < nz) mma(x[i], l, z[t]);
          }
        }
      }
    }

    // ---- terminal values: the lane holds assets 16 rb + 4 g4 + 0..3 of
    // path c16 of its column block ----
    float bs = 0.f, gs = 0.f, e0 = 0.f;
#pragma unroll
    for (uint32_t i = 0; i < (uint32_t)RPW; ++i) {
      const uint32_t rb = row_block<SETS>(set, i);
      if (rb < rows) terminal_rows<PORT, QMC>(P, x[i], rb, g4, bs, gs, e0);
    }
    Sum bsum, gsum = 0, esum = 0;
    if constexpr (kSums64) {
      bsum = lane_add<16>(lane_add<32>((double)bs));
      gsum = lane_add<16>(lane_add<32>((double)gs));
      esum = lane_add<16>(lane_add<32>((double)e0));
    } else {
#pragma unroll
      for (int off = 16; off < 64; off <<= 1) {
        bs += __shfl_xor(bs, off, 64);
        if constexpr (!PORT) {
          gs += __shfl_xor(gs, off, 64);
          e0 += __shfl_xor(e0, off, 64);   // one lane of the four holds it
        }
      }
      bsum = bs;
      gsum = gs;
      esum = e0;
    }
    if (g4 == 0u) {
      s_part[0][set][16u * col + c16] = bsum;
      if constexpr (!PORT) {
        s_part[1][set][16u * col + c16] = gsum;
        s_part[2][set][16u * col + c16] = esum;
      }
    }
    __syncthreads();                       // also: every wave has read s_sum
    const uint64_t pid = tile * kTile + (uint64_t)lane;
    if (wave == 0u && pid < P.n_paths) {
      Sum v[C];
#pragma unroll
      for (int c = 0; c < C; ++c) {
        v[c] = s_part[c][0][lane];
#pragma unroll
        for (int q = 1; q < SETS; ++q) v[c] += s_part[c][q][lane];
      }
      double y[C];
      channels<PORT, QMC>(P, v, y);
      bool finite = true;
#pragma unroll
      for (int c = 0; c < C; ++c) finite = finite && isfinite(y[c]);
      if (P.path_out != nullptr) {
#pragma unroll
        for (int c = 0; c < C; ++c) P.path_out[pid * C + c] = y[c];
      }
      s_acc[lane].push(y, finite, !finite);
    }
    // The next tile's terminal values are written two barriers from here.
  }
  PartSums<C> part;
  part.zero();
  if (wave == 0u) part = s_acc[lane];
  block_reduce<C, 64 * W>(part, partials, blk);
}

// Replicates of few Sobol' dimensions (n_steps d <= 64): a wave takes a tile of
// 64 consecutive points by itself, with no barrier between its stages. Lane l
// keeps the part of dimension l that the tile's points share, and moves it
// from one tile to the next by the bits of the point index that change; the
// part of the low six bits is the same in every tile and is read from LDS. The
// digital shifts are drawn here, one block per lane.
//
// Bound: VALU issue and the latency of the stages (16 dimensions: four blocks
// of Box-Muller, 24 MFMAs, an FP64 exponential per path). 16 replicates of
// 2^16 points x 16 assets: 74 us in the general kernel, whose waves share a
// tile and wait for each other three times, and a launch for the shifts; 42 us
// here.
template <int PREC>
__global__ __launch_bounds__(64 * kQmcWaves, 4) void qmc_tile_kernel(const BasketParams P) {
  stamp(P.clock);
  typedef Form<PREC> F;
  typedef typename F::V V8;
  constexpr int C = 3;
  // [dims / 4][64][4], read 16 bytes at a time, [32][dims], then the sums.
  extern __shared__ __attribute__((aligned(16))) uint32_t s_words[];
  const int lane = threadIdx.x & 63;
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t d = P.d, n = P.n_steps, nq = d >> 2, rows = d >> 4, dims = n * d;
  uint32_t* s_low = s_words;
  uint32_t* s_dir = s_words + 64u * dims;
  float* s_sum = (float*)(s_dir + 32u * dims) + wave * d * kRow;
  for (uint32_t i = threadIdx.x; i < 32u * dims; i += 64u * kQmcWaves)
    s_dir[(i & 31u) * dims + (i >> 5)] = P.qV[i];
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < 64u * dims; i += 64u * kQmcWaves) {
    const uint32_t l = (i >> 2) & 63u, dim = 4u * (i >> 8) + (i & 3u);
    uint32_t x = 0;
#pragma unroll
    for (uint32_t b = 0; b < 6u; ++b) x ^= (l >> b) & 1u ? s_dir[b * dims + dim] : 0u;
    s_low[i] = x;
  }
  __syncthreads();
  const uint32_t nblk = P.q_rep_blocks, rep = blockIdx.x / nblk, blk = blockIdx.x - rep * nblk;
  uint32_t high = 0;                       // dimension `lane`: shift and the bits of `at`
  if ((uint32_t)lane < dims)
    high = word_at(philox((uint32_t)lane >> 2, make_counter(rep, P.q_shift_tag, P.k0, P.k1)),
                   (uint32_t)lane & 3u);
  const uint64_t first = P.path_offset, last = first + P.n_paths;   // last <= 2^32
  const uint64_t base0 = first & ~63ull, tiles = (last - base0 + 63u) >> 6;
  uint32_t at = 0;
  PartSums<C> acc;
  acc.zero();
  for (uint64_t tile = (uint64_t)blk * kQmcWaves + wave; tile < tiles;
       tile += (uint64_t)nblk * kQmcWaves) {
    const uint32_t base = (uint32_t)(base0 + (tile << 6));
    for (uint32_t change = base ^ at; change != 0u; change &= change - 1u) {
      const uint32_t b = (uint32_t)__builtin_ctz(change);
      high ^= (uint32_t)lane < dims ? s_dir[b * dims + (uint32_t)lane] : 0u;
    }
    at = base;
    for (uint32_t q = 0; q < nq; ++q)
      sum_block<PREC>(s_sum, n, nq, q, lane, [&](uint32_t j) {
        const uint4 low = *(const uint4*)(s_low + (j * 64u + (uint32_t)lane) * 4u);
        auto of = [&](uint32_t t) {
          return (uint32_t)__builtin_amdgcn_readlane((int)high, (int)(4u * j + t));
        };
        return Words4{low.x ^ of(0), low.y ^ of(1), low.z ^ of(2), low.w ^ of(3)};
      });
    wave_sync();
    // The product as in basket_kernel, a row block at a time. (A function for
    // both costs that kernel 20 registers and spills.)
    const uint32_t c16 = (uint32_t)lane & 15u, g4 = (uint32_t)lane >> 4;
    const uint32_t nz = sum_terms<PREC>(n), n_pairs = basket_pairs(rows);
    double v[C] = {0.0, 0.0, 0.0};         // of path `lane`
#pragma unroll
    for (uint32_t col = 0; col < 4u; ++col) {
      float bs = 0.f, gs = 0.f, e0 = 0.f;
      for (uint32_t rb = 0; rb < rows; ++rb) {
        f32x4 x = {0.f, 0.f, 0.f, 0.f};
        for (uint32_t kb = 0; 2u * kb <= rb; ++kb) {
          const uint32_t k0 = 32u * kb + 8u * g4;
          V8 z[F::NZ];
          float r[8];
#pragma unroll
          for (uint32_t e = 0; e < 8u; ++e)
            r[e] = k0 < d ? s_sum[(k0 + e) * kRow + 16u * col + c16] * P.z_scale : 0.f;
#pragma unroll
          for (int t = 0; t < F::NZ; ++t)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              z[t][e] = r[e];
              r[e] -= (float)z[t][e];
            }
          const V8* a = (const V8*)P.Lfrag + ((size_t)basket_pairs(rb) + kb) * 64u + lane;
#pragma unroll
          for (int p = 0; p < F::NL; ++p) {
            const V8 l = a[(size_t)p * n_pairs * 64u];
#pragma unroll
            for (int t = 0; t < F::NZ; ++t)
              if (p + t < F::KEEP && (uint32_t)t < nz) mma(x, l, z[t]);
          }
        }
        terminal_rows<false, true>(P, x, rb, g4, bs, gs, e0);
      }
      // The last two sums in FP64: their rounding would be the largest of a path.
      const float t[C] = {bs, gs, e0};
#pragma unroll
      for (int c = 0; c < C; ++c) {
        const double w = lane_add<16>(lane_add<32>((double)t[c]));
        if (g4 == col) v[c] = w;
      }
    }
    wave_sync();                           // the sums are read before the next tile's
    const uint64_t point = (uint64_t)base + (uint64_t)lane;
    if (point >= first && point < last) {
      double y[C];
      channels<false, true>(P, v, y);
      bool finite = true;
#pragma unroll
      for (int c = 0; c < C; ++c) finite = finite && isfinite(y[c]);
      acc.push(y, finite, !finite);
    }
  }
  block_reduce<C, 64 * kQmcWaves>(acc, P.partials + (size_t)rep * n_moments(C) * nblk, blk);
}

template <int PREC>
hipError_t launch_qmc_tile(const BasketParams& p, hipStream_t s, uint32_t blocks) {
  const uint32_t dims = p.n_steps * p.d;
  const size_t lds = 96u * dims * sizeof(uint32_t) + (size_t)kQmcWaves * p.d * kRow * sizeof(float);
  if (dims > 64u) return hipErrorInvalidValue;
  if (lds > 32768) {
    const hipError_t e = hipFuncSetAttribute((const void*)qmc_tile_kernel<PREC>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(qmc_tile_kernel<PREC>, dim3(blocks), dim3(64 * kQmcWaves), lds, s, p);
  return hipGetLastError();
}

template <int PREC, bool PORT, bool QMC, int W, int RPW, bool SPLIT>
hipError_t launch_form(const BasketParams& p, hipStream_t s, uint32_t nb) {
  static_assert(kBasketMaxDim <= 4 * 8 * 8, "row blocks of the largest form");
  if (p.d > (uint32_t)(4 * W * RPW)) return hipErrorInvalidValue;
  const size_t lds = (size_t)p.d * kRow * sizeof(float);
  if (lds > 32768) {                       // above it: the default limit is 64 KB with the static part
    const hipError_t e = hipFuncSetAttribute((const void*)basket_kernel<PREC, PORT, QMC, W, RPW, SPLIT>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((basket_kernel<PREC, PORT, QMC, W, RPW, SPLIT>), dim3(nb), dim3(64 * W), lds, s, p);
  return hipGetLastError();
}

template <int PREC, bool PORT, bool QMC, int W, int RPW>
hipError_t launch_w(const BasketParams& p, hipStream_t s, uint32_t nb) {
  if constexpr (!QMC) {
    if (p.split_parts > 1u) {
      if (p.split_parts != (p.d / 4u + W - 1u) / W || p.split_from > nb ||
          p.split_sums == nullptr || p.split_arrivals == nullptr)
        return hipErrorInvalidValue;
      return launch_form<PREC, PORT, QMC, W, RPW, true>(
          p, s, p.split_from + (nb - p.split_from) * p.split_parts);
    }
  }
  return launch_form<PREC, PORT, QMC, W, RPW, false>(p, s, nb);
}

// Waves per tile and row blocks per wave. A CU holds 16 waves at the 128 VGPRs
// of the product phase; two or more workgroups of them should be resident so
// that one's product runs beside the other's sums. Measured (d = 112, FP32,
// 100003 x 50): 255 us in workgroups of 8 waves, 287 us in 4; capping the
// registers for 20 waves spills and gains nothing.
template <int PREC, bool PORT, bool QMC>
hipError_t launch_mode(const BasketParams& p, hipStream_t s, uint32_t nb) {
  if (p.d <= 64) return launch_w<PREC, PORT, QMC, 4, 4>(p, s, nb);
  if (p.d <= 128) return launch_w<PREC, PORT, QMC, 8, 4>(p, s, nb);
  return launch_w<PREC, PORT, QMC, 8, 8>(p, s, nb);
}

template <int PREC>
hipError_t launch_prec(const BasketParams& p, hipStream_t s, uint32_t nb) {
  const bool qmc = p.qV != nullptr, port = p.n_strikes != 0;
  if (qmc && port) return hipErrorInvalidValue;
  if constexpr (PREC == BK_FP32 || PREC == BK_FP16) {
    if (qmc) return launch_mode<PREC, false, true>(p, s, nb);
  }
  if constexpr (PREC != BK_BF16X2) {
    if (port) return launch_mode<PREC, true, false>(p, s, nb);
  }
  if (qmc || port) return hipErrorInvalidValue;
  return launch_mode<PREC, false, false>(p, s, nb);
}

// Shapes the kernel assumes.
bool shapes_ok(const BasketParams& p) {
  return p.d >= 16 && p.d <= (uint32_t)kBasketMaxDim && p.d % 16 == 0 && p.n_steps > 0 && p.n_paths > 0;
}

hipError_t launch_any(const BasketParams& p, int prec, hipStream_t s, uint32_t nb) {
  if (!shapes_ok(p)) return hipErrorInvalidValue;
  switch (prec) {
    case BK_FP32: return launch_prec<BK_FP32>(p, s, nb);
    case BK_BF16: return launch_prec<BK_BF16>(p, s, nb);
    case BK_FP16: return launch_prec<BK_FP16>(p, s, nb);
    case BK_BF16X2: return launch_prec<BK_BF16X2>(p, s, nb);
  }
  return hipErrorInvalidValue;
}

}  // namespace

int basket_l_terms(int prec) {
  return prec == BK_FP32 ? Form<BK_FP32>::NL : prec == BK_BF16X2 ? Form<BK_BF16X2>::NL : 1;
}

// The last workgroups of a launch with one tile each leave most CUs idle: 1563
// tiles are six on each of 256 CUs and 27 on 27 of them. Those past the last
// multiple of 256 are split, by asset blocks so that the sums keep their
// order, into parts of one block per wave. Portfolio kernel in FP32: 100003
// paths x 50 steps x 112 assets 266 -> 260 us, 5000 such paths (79 tiles)
// 56 -> 43 us, 20000 x 30 x 64 40 -> 34 us. Above 16 tiles a CU the tail is
// lost in the rest, a last round more than 7/8 full is left whole, and a tile
// of few asset blocks (d <= 16) has nothing to split.
BasketSplit basket_split(uint64_t n_paths, uint32_t n_steps, uint32_t d) {
  BasketSplit x;
  const uint64_t tiles = (n_paths + kTile - 1) / kTile;
  const uint32_t nb = basket_blocks(n_paths, n_steps, d);
  const uint32_t W = d <= 64 ? 4 : 8, parts = (d / 4 + W - 1) / W, tail = (uint32_t)(tiles % 256u);
  x.from = nb;
  if (nb != tiles || tiles > 16u * 256u || tail == 0 || tail > 224 || parts < 2) return x;
  x.parts = parts;
  x.from = nb - tail;
  x.sums = (size_t)tail * d * kTile;
  x.arrivals = tail;
  return x;
}

hipError_t launch_basket_pack(const BasketPack& k, int prec, hipStream_t s) {
  if (k.d < 16 || k.d > (uint32_t)kBasketMaxDim || k.d % 16 != 0) return hipErrorInvalidValue;
  const dim3 grid((basket_pairs(k.d / 16) + 3) / 4 + 1);
  switch (prec) {
#define MCP_PACK(P) \
  case P: hipLaunchKernelGGL(basket_pack_kernel<P>, grid, dim3(256), 0, s, k); break;
    MCP_PACK(BK_FP32) MCP_PACK(BK_BF16) MCP_PACK(BK_FP16) MCP_PACK(BK_BF16X2)
#undef MCP_PACK
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// A workgroup ends with a reduction and a moment vector, so it takes enough
// tiles to draw 64 Philox blocks per wave, as long as 1024 workgroups are left
// to fill the chip.
uint32_t basket_blocks(uint64_t n_paths, uint32_t n_steps, uint32_t d) {
  const uint64_t tiles = (n_paths + kTile - 1) / kTile;
  const uint64_t per_wave = (uint64_t)n_steps * (d / 4) / (d <= 64 ? 4 : 8);
  const uint64_t per_wg = per_wave >= 64 ? 1 : (64 + per_wave - 1) / (per_wave ? per_wave : 1);
  uint64_t nb = (tiles + per_wg - 1) / per_wg;
  if (nb < 1024) nb = tiles < 1024 ? tiles : 1024;
  return (uint32_t)(nb < kBasketMaxBlocks ? nb : kBasketMaxBlocks);
}

// Replicates whose points have few dimensions take the tile kernel, in about
// four tiles per wave with 1024 workgroups in all (a CU holds four).
bool qmc_tiles(const BasketParams& p, int prec) {
  return (uint64_t)p.n_steps * p.d <= 64u && (prec == BK_FP32 || prec == BK_FP16);
}

bool basket_qmc_draws_shifts(const BasketParams& p, int prec) { return qmc_tiles(p, prec); }

hipError_t launch_basket_qmc_batch(BasketParams p, int prec, uint32_t n_rep, hipStream_t s,
                                   uint32_t* blocks_per_rep) {
  if (n_rep == 0 || n_rep > kBasketMaxBlocks) return hipErrorInvalidValue;
  if (p.qV == nullptr || p.n_strikes != 0 || p.path_out != nullptr) return hipErrorInvalidValue;
  uint64_t nb, share;
  if (qmc_tiles(p, prec)) {
    nb = (p.n_paths + 64u * kQmcWaves - 1) / (64u * kQmcWaves);
    share = 1024 / n_rep;
  } else {
    nb = basket_blocks(p.n_paths, p.n_steps, p.d);
    share = kBasketMaxBlocks / 2 / n_rep;                 // 2048 workgroups in all
  }
  if (nb > share) nb = share ? share : 1;
  if (nb == 0) return hipErrorInvalidValue;
  *blocks_per_rep = (uint32_t)nb;
  p.q_rep_blocks = (uint32_t)nb;
  if (!qmc_tiles(p, prec)) return launch_any(p, prec, s, (uint32_t)(nb * n_rep));
  if (!shapes_ok(p)) return hipErrorInvalidValue;
  return prec == BK_FP32 ? launch_qmc_tile<BK_FP32>(p, s, (uint32_t)(nb * n_rep))
                         : launch_qmc_tile<BK_FP16>(p, s, (uint32_t)(nb * n_rep));
}

hipError_t launch_basket(const BasketParams& p, int prec, hipStream_t s, uint32_t* n_blocks) {
  const uint32_t nb = basket_blocks(p.n_paths, p.n_steps, p.d);
  *n_blocks = nb;
  if (nb == 0) return hipErrorInvalidValue;
  return launch_any(p, prec, s, nb);
}

}  // namespace mcp
