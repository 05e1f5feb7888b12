// Internal interface between the C ABI (api.hip) and the kernel translation
// units. Host-side declarations only; no torch types anywhere.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mcp {

constexpr int kBlock = 256;          // threads per path-kernel workgroup (4 waves)
#ifndef MCP_GBM_MAX_BLOCKS
#define MCP_GBM_MAX_BLOCKS 8192
#endif
// GBM grid cap: the persistent grid gives each thread several paths.
constexpr uint32_t kGbmMaxBlocks = MCP_GBM_MAX_BLOCKS;

// ---- GBM path functionals (bit mask -> per-path channels, in bit order) ----
enum : uint32_t {
  G_EURO = 1u << 0,     // "euro"
  G_ASIAN = 1u << 1,    // "asian"
  G_GEO = 1u << 2,      // "geo"
  G_UO = 1u << 3,       // "uo"
  G_UOBB = 1u << 4,     // "uo_bridge"
  G_EURO_G = 1u << 5,   // "euro_delta", "euro_vega"
  G_ASIAN_G = 1u << 6,  // "asian_delta", "asian_vega"
  G_ALL = 0x7Fu
};

__host__ __device__ constexpr int popcount_c(uint32_t m) {
  return m == 0 ? 0 : (int)(m & 1u) + popcount_c(m >> 1);
}
__host__ __device__ constexpr int gbm_channels(uint32_t mask) {
  return popcount_c(mask & 0x1Fu) + 2 * popcount_c(mask & 0x60u);
}
// Moment vector of C channels: [n_valid, n_nonfinite, mean y_c (C),
// co-moment sum (y_a - mean_a)(y_b - mean_b) (a <= b)]; block partials are
// block-major, [block][n_moments(C)] (device/reduce.h).
__host__ __device__ constexpr int n_moments(int C) { return 2 + C + C * (C + 1) / 2; }
constexpr int kMaxMomentChannels = 9;

struct GbmParams {
  uint64_t n_paths, path_offset;
  uint32_t n_steps, tag, k0, k1;
  int log_scheme;
  // Multilevel coupling: step i uses the normalised sum of normals
  // coarsen*i .. coarsen*i + coarsen - 1 (1, 2 or 4; 1 = plain).
  uint32_t coarsen;
  // Model constants, double on the host; kernels round them to their type.
  double S0, K, disc, T, dt, sdt, sigma;
  // Log scheme, in the kernel's log domain (log2 for FP32, ln for FP64):
  double drift_dom, vol_dom, barrier_dom, bridge_c;
  // Euler on S: increments of S/S0.
  double r_dt, vol_sdt, barrier_rel;
  double* partials;   // [n_blocks][n_moments]
  double* path_out;   // [n_paths][C] or nullptr
  uint64_t* clock;    // start stamp (device/reduce.h), or nullptr
};

// Launches the GBM path kernel for the instantiated mask `mask` (must be one
// returned by gbm_pick_mask). Returns the number of blocks via *n_blocks.
hipError_t launch_gbm(const GbmParams& p, uint32_t mask, bool fp64, hipStream_t s,
                      uint32_t* n_blocks);

// The bumped models of a finite-difference run, [0] for delta (S0) and [1]
// for vega (sigma). up[0] also carries what all of them share (paths, steps,
// key, tag, clock) and, as S0 does not enter a step, the unbumped dynamics.
struct GbmFdParams {
  GbmParams up[2], down[2];
  double* partials;   // [greeks][n_blocks][n_moments(1)]
};
hipError_t launch_gbm_fd(const GbmFdParams& p, uint32_t bit, bool delta, bool vega, hipStream_t s,
                         uint32_t* n_blocks);
// Smallest instantiated mask containing `want` for this precision/scheme
// and coupling factor, or 0 when none does. rows: the set whose channels a
// row of per-path values has (mc_path_channels).
uint32_t gbm_pick_mask(uint32_t want, bool fp64, bool log_scheme, uint32_t coarsen, bool rows);

// Moments of [a[ca] - b[cb], a[ca], b[cb]] over n paths of two per-path
// tables with Ca and Cb channels (multilevel correction); returns the block
// count.
hipError_t launch_diff_moments(const double* a, uint32_t Ca, uint32_t ca, const double* b,
                               uint32_t Cb, uint32_t cb, uint64_t n, double* partials,
                               hipStream_t s, uint32_t* n_blocks);
constexpr uint32_t kDiffMaxBlocks = 1024;

// ---- Heston ----
enum : uint32_t { H_EURO = 1u << 0, H_ASIAN = 1u << 1 };

// Heston kernels run on a persistent grid of at most this many workgroups
// (each thread prices several paths); partials are one moment vector per
// workgroup.
constexpr uint32_t kHestonMaxBlocks = 8192;
uint32_t heston_blocks(uint64_t n_paths);

struct HestonParams {
  uint64_t n_paths, path_offset;
  uint32_t n_steps, tag, k0, k1;
  double S0, K, disc, dt, sdt, r, v0, kappa, theta, xi, rho, rho_c;
  double* partials;
  double* path_out;
  uint64_t* clock;    // start stamp, or nullptr
};
hipError_t launch_heston(const HestonParams& p, uint32_t mask, bool fp64, hipStream_t s,
                         uint32_t* n_blocks);
// Price, pathwise delta and d/dv0 of one payoff by forward-mode tangents
// (channels: payoff, delta, d/dv0).
hipError_t launch_heston_tangent(const HestonParams& p, bool asian, bool fp64, hipStream_t s,
                                 uint32_t* n_blocks);

// The same channels in FP32 paths with the derivatives chained in FP64: one
// path per thread.
hipError_t launch_heston_pathwise(const HestonParams& p, bool asian, hipStream_t s,
                                  uint32_t* n_blocks);

// Pathwise adjoint (reverse sweep with checkpoints every `every` steps:
// even, 2..kCkptMax; kCkpt by default). A full (one-launch) sweep with at
// most kLdsCkpt checkpoints keeps them in LDS (2 kLdsCkpt floats per path,
// 32 KB per 256-path block) and needs no device buffer.
constexpr int kCkpt = 16;
constexpr int kCkptMax = 16;
constexpr int kLdsCkpt = 16;
struct AdjointParams {
  HestonParams h;
  int asian;            // 1: arithmetic-Asian call, 0: European call
  int phase;            // 0 full, 1 forward (write checkpoints), 2 reverse
  float* ckpt;          // [2*n_ckpt + 1][n_paths]: (z, v) per checkpoint, then terminal;
                        // nullptr for a full sweep with checkpoints in LDS
  uint32_t n_ckpt;
  uint32_t every;       // checkpoint period
  double grad_out;
};
hipError_t launch_heston_adjoint(const AdjointParams& p, hipStream_t s, uint32_t* n_blocks);

// ---- Basket (correlated GBM, MFMA product of the summed normals) ----
enum : int { BK_FP32 = 0, BK_BF16 = 1, BK_FP16 = 2, BK_BF16X2 = 3 };
constexpr int kBasketTile = 64;              // paths per tile, one per lane
constexpr int kBasketMaxDim = 256;
// Grid cap: a workgroup takes tiles blk, blk + grid, ... and writes one
// moment vector.
constexpr uint32_t kBasketMaxBlocks = 4096;
uint32_t basket_blocks(uint64_t n_paths, uint32_t n_steps, uint32_t d);
// Tiles of a run that are split: from tile `from`, into `parts` workgroups, and
// the scratch they take (floats, counters).
struct BasketSplit {
  uint32_t from = 0, parts = 1;
  size_t sums = 0;
  uint32_t arrivals = 0;
};
BasketSplit basket_split(uint64_t n_paths, uint32_t n_steps, uint32_t d);
// L' in MFMA operand order: for each 16-row block rb of the lower triangle its
// 32-column blocks kb = 0 .. rb / 2, fragment basket_pairs(rb) + kb = [64
// lanes][8] of the 16-bit type, lane l holding row 16 rb + l mod 16 and
// columns 32 kb + 8 (l / 16) + 0..7; one such array per term of L' (hi, mid,
// lo).
__host__ __device__ constexpr uint32_t basket_pairs(uint32_t rb) {   // fragments before block rb
  return (rb / 2) * (rb / 2 + 1) + (rb % 2) * (rb / 2 + 1);
}
int basket_l_terms(int prec);
struct BasketParams {
  uint64_t n_paths, path_offset;
  uint32_t n_steps, tag, k0, k1;
  uint32_t d;             // assets, multiple of 16, <= 256
  const void* Lfrag;      // [terms][basket_pairs(d / 16)][64][8] (device)
  // Scale of the sums as operands, and of the product: half precision takes the
  // sums times a power of two (|sum| < 5.8 n_steps stays below 2^15) and the
  // product over it; 1 in the other forms.
  float z_scale, x_scale;
  // Device [4][256]: n*mu_a (log2), w_a*S0_a / ratio, w_a*ln 2, S0_a / ratio; the
  // prices' ratio (near 1, see basket_setup) also divides K and w0, multiplies
  // disc, and its logarithm is taken off geo0.
  const float* asset;
  double disc, K, geo0, w0;
  // Call portfolio (risk mode): q_k calls of strike m_k S0_a on every asset;
  // the per-path value is sum_a S0_a sum_k q_k (S_a/S0_a - m_k)^+ - premium.
  uint32_t n_strikes;     // 0: basket-call mode
  float pm[8], pq[8];
  double premium;
  // Randomised quasi-Monte Carlo: when qV is set, normal block j of path p
  // comes from Sobol' point p (dimensions 4j..4j+3) shifted by qshift.
  const uint32_t* qV;     // [dims][32] direction words
  const uint32_t* qshift; // [dims], or [replicates][dims] with q_rep_blocks
  // Replicates in one launch: block b runs replicate b / q_rep_blocks with
  // shift row q_dims * replicate, and writes its moments to that
  // replicate's own [q_rep_blocks][moment] partials.
  uint32_t q_rep_blocks, q_dims;
  // Tiles split over workgroups (basket_split), or parts <= 1.
  uint32_t split_from, split_parts;
  float* split_sums;      // [tiles from split_from][d][kBasketTile]
  uint32_t* split_arrivals;   // [tiles from split_from], zero
  uint32_t q_shift_tag;   // stream of the shifts, where the kernel draws them itself
  double* partials;
  double* path_out;       // [n_paths][3] (basket) or [n_paths] (portfolio), or nullptr
  uint64_t* clock;        // start stamp, or nullptr
  double ratio;           // the prices', for the portfolio's value
  double base;            // sum of the table's w_a*S0_a / ratio
};
constexpr int kMaxStrikes = 8;
// Words a run's set-up launch clears for later kernels of the call (n <= 2^20).
struct BasketZero {
  uint32_t* words = nullptr;
  uint32_t n = 0;
};
// Packs L' = diag(sigma_a step) L into Lfrag form and copies the asset table
// from pinned memory. step: sqrt(dt) / ln 2, in FP32 times the factor
// sqrt(2 ln 2) that its sums of normals leave out.
struct BasketPack {
  const double* L;        // [d][d] lower factor (device)
  const double* sigma;    // [d] (pinned)
  const float* asset;     // [4][256] (pinned)
  double step;
  uint32_t d;
  uint16_t* frag;
  float* asset_out;
  BasketZero zero[2];
};
hipError_t launch_basket_pack(const BasketPack& k, int prec, hipStream_t s);
hipError_t launch_basket(const BasketParams& p, int prec, hipStream_t s, uint32_t* n_blocks);
// All n_rep randomised-QMC replicates of p in one launch (p.qshift holds
// n_rep rows of p.q_dims shifts); *blocks_per_rep = one replicate's blocks.
bool basket_qmc_draws_shifts(const BasketParams& p, int prec);   // p.qshift unused
hipError_t launch_basket_qmc_batch(BasketParams p, int prec, uint32_t n_rep, hipStream_t s,
                                   uint32_t* blocks_per_rep);

// Digital shifts of one randomised-QMC replicate: shift[j] = word (j mod 4)
// of Philox block (floor(j/4), replicate, tag) under key (k0, k1).
// Digital shifts of replicates replicate0 .. replicate0 + n_rep - 1:
// shift [n_rep][n_dims].
hipError_t launch_qmc_shifts(uint32_t k0, uint32_t k1, uint32_t tag, uint64_t replicate0,
                             uint32_t n_rep, uint32_t n_dims, uint32_t* shift, hipStream_t s);

// ---- Order statistic and tail mean of per-path values (risk metrics) ----
// Exact k-th smallest (1-based) of x[0..n) and the count and sum of the values
// below it (k_risk.hip). The state is zero in hist and arrivals before the
// first launch of a call and again after the last.
constexpr uint32_t kSelectDigit = 12;
constexpr uint32_t kSelectList = 2048;       // matches sorted in LDS
struct SelectState {
  uint32_t hist[1u << kSelectDigit];
  uint32_t arrivals, n_match;
  uint64_t prefix, mask;                     // digits fixed so far, and their bits
  uint64_t k;                                // 1-based rank still sought among the matches
  uint64_t key_min, key_max;                 // of the matches
};
constexpr uint32_t kSelectZeroWords = (1u << kSelectDigit) + 1;
constexpr size_t kSelectPartialBytes = 2 * 256 * sizeof(double);
struct SelectResult {                        // host memory
  uint64_t key;                              // of the k-th smallest
  double n_tail, tail_sum;                   // values strictly below it
  uint64_t end;                              // stamp
  uint32_t done;                             // 0: queue launch_select_rest
};
hipError_t launch_select(const double* x, uint64_t n, uint64_t k, SelectState* st, uint64_t* list,
                         double* partials, SelectResult* out, hipStream_t s, uint64_t* clock);
hipError_t launch_select_rest(const double* x, uint64_t n, SelectState* st, uint64_t* list,
                              double* partials, SelectResult* out, hipStream_t s);
// Value of a key.
double select_key_to_value(uint64_t key);

// ---- Longstaff-Schwartz regression (Bermudan options) ----
// d <= 4 correlated GBM assets with dividend yield, log-Euler in the log2
// domain: x_a = log2(S_a / K), so that y_a = S_a / K = exp2(x_a).
constexpr int kLsmMaxD = 4, kLsmMaxDates = 64, kLsmMaxFeat = 11;
// Moments per block: the upper triangle of u u^T, u = (features, cash flow),
// then the sum and the sum of squares of the cash flow and the number of
// paths in the money at the last date.
constexpr int kLsmMaxMom = (kLsmMaxFeat + 1) * (kLsmMaxFeat + 2) / 2 + 3;
constexpr uint32_t kLsmMaxBlocks = 2048;
enum : uint32_t { LSM_MAX_CALL = 1, LSM_BASKET_PUT = 2, LSM_BASKET_CALL = 3 };
struct LsmParams {
  uint64_t n_paths, path_offset;
  uint32_t tag, k0, k1;
  uint32_t d, degree, pay_feat;  // pay_feat: f/K appended to the features
  uint32_t kind, n_dates, spd;   // payoff, exercise dates, Euler steps per date
  uint32_t nf;                   // number of features
  float x0[kLsmMaxD];            // log2(S0_a / K)
  float drift[kLsmMaxD];         // (r - q - sigma_a^2 / 2) dt / ln 2
  float vol[kLsmMaxD][kLsmMaxD]; // sigma_a sqrt(dt) L_ab / ln 2 (lower triangle)
  double discK[kLsmMaxDates + 1];// K e^{-r t_j}, j = 0..n_dates
  uint64_t ystride;               // row stride of y and length of C: n_paths rounded up to 64
  float* y;                      // [n_dates][d][ystride]: S_a(t_j) / K
  float* C;                      // [ystride] discounted cash flow
  uint8_t* ex;                   // [n_paths] exercise date (0 = never), or nullptr
  const double* beta;            // [n_dates][kLsmMaxFeat]
  const int* valid;              // [n_dates]: 1 when date j has a regression
  double* partials;              // [n_mom][n_blocks]
  double* path_value;            // out-of-sample: [n_paths] values, or nullptr
  uint64_t* clock;               // start stamp, or nullptr
  uint32_t* arrivals;            // the reductions' counter, zeroed by the simulation
};
// Where a stage's reduction writes (device memory), and the copy of all
// results to the host at the end of a call's last one (host: nullptr before).
struct LsmReduce {
  double* sums;                  // [n_mom]
  double* beta;                  // [n_dates][kLsmMaxFeat]
  int* valid;                    // [n_dates]
  uint64_t* clock;               // [0] start, [1] end
  uint32_t* arrivals;            // workgroups that have written their rows; 0 between launches
  const double* results;         // n_results doubles: all of the above
  double* host;
  uint32_t n_results;
};
// Moments the kernels of this feature set write (see kLsmMaxMom).
uint32_t lsm_n_moments(uint32_t nf);
uint32_t lsm_n_features(uint32_t d, uint32_t degree, uint32_t pay_feat);
// Simulation of the stored paths (cash flows at t_M, Gram matrix of date
// n_dates - 1 and the exercise-at-maturity moments), the update of date j
// (exercise rule of date j, then the Gram matrix of date j - 1, or the
// price moments when j = 1), the reduction of a stage's block partials
// followed by the Cholesky solve of date j (none when j = 0), and the
// out-of-sample estimate on fresh paths.
hipError_t launch_lsm_sim(const LsmParams& p, hipStream_t s, uint32_t* n_blocks);
hipError_t launch_lsm_update(const LsmParams& p, uint32_t j, hipStream_t s, uint32_t* n_blocks);
hipError_t launch_lsm_reduce(const double* partials, uint32_t nb, uint32_t nmom, uint32_t nf,
                             uint32_t j, const LsmReduce& r, hipStream_t s);
hipError_t launch_lsm_oos(const LsmParams& p, hipStream_t s, uint32_t* n_blocks);

// ---- Learned martingale control variate (Heston Asian) ----
// Hedge network 4 -> 64 -> 64 -> 1 with tanh, run on MFMA for 32 paths per
// wave. Host-packed per-lane fragments (see api.hip, pack_mlp):
constexpr int kMlpH = 64;
constexpr int kMlpNParam = 4545;
// Row stride of the per-block gradient partials: whole 128-byte lines.
constexpr int kGradStride = (kMlpNParam + 31) / 32 * 32;
struct CvParams {
  HestonParams h;
  uint32_t hedge_every;      // rebalancing period m
  int bf16;                  // 1: BF16 MFMA operands, 0: FP32 MFMA
  const float* theta;        // [4545] flat weights (b3 is read from here)
  const float* w1f;          // [2 mb][64 lane][8]   layer-1 A fragments (W1 | b1 | 0)
  const void* w2f;           // [2 mb][4 kb][64][8]  layer-2 A fragments (permuted W2), in the
                             // operand type (BF16 or FP32)
  const void* w2tf;          // [2 mb][4 kb][64][8]  W2^T fragments for the backward pass
  const float* lanec;        // [2][2 halves][32]: b2 * (-2 / ln 2), then 2 W3, of a half's units
  const float* dfac;         // [n_steps + 1]: e^{r t_i}
  // training
  uint32_t val_blocks;       // blocks of the hedged-value kernel whose moment vectors
                             // (in `partials`) the backward sums for Ybar
  const double* y_path;      // per-path values of that pass, [n_paths][3] (Y is channel 2)
  double g_scale;            // -2 / B
  float* grad_partials;      // [n_blocks][kGradStride]: FP64 wave sums rounded to FP32
  double* partials;
  double* path_out;
  // Feature cache of the training paths, one entry per hedge segment k (the
  // network's inputs do not depend on its weights, so each training path is
  // simulated once per training run, not once per Adam step).
  float* c_phi;              // [n_seg][4][c_stride] features at the segment's opening date
  float* c_dst;              // [n_seg][c_stride] discounted price change over the segment
  double* c_pay;             // [c_stride] discounted payoff
  uint64_t c_stride;         // paths held by the cache
  uint64_t c_first;          // the minibatch's first path within the cache
  uint32_t n_seg;            // ceil(n_steps / hedge_every)
  uint32_t seg_split;        // backward: waves per 32-path tile, each taking a
                             // contiguous range of segments (set by its launcher)
};
constexpr int kCvPathsPerBlock = 256;       // evaluation: 4 waves of 64 paths
constexpr int kCvTrainPathsPerBlock = 128;  // training: 4 waves of 32 paths (/ split)
// Fragment layout of the weights, built on the device from theta.
constexpr int kW1fFloats = 2 * 64 * 8, kW2fFloats = 2 * 4 * 64 * 8, kLanecFloats = 2 * 2 * 32;
hipError_t launch_cv_pack(const float* theta, bool bf16, float* w1f, void* w2f, void* w2tf,
                          float* lanec, hipStream_t s);
hipError_t launch_cv_price(const CvParams& p, hipStream_t s, uint32_t* n_blocks);
// Training on the feature cache: fill it (h.n_paths paths from h.path_offset),
// the network along every 32-path tile of the minibatch with the per-path
// hedged values and their moments, and the gradient partials.
hipError_t launch_cv_cache(const CvParams& p, hipStream_t s);
hipError_t launch_cv_values(const CvParams& p, hipStream_t s, uint32_t* n_blocks);
hipError_t launch_cv_backward(const CvParams& p, hipStream_t s, uint32_t* n_blocks);
// Workgroups of the backward (the rows of its gradient partials) and of the
// hedged-value kernel (the rows of its block moments) for a minibatch of
// n_paths with n_seg hedge segments; *split (if given) receives the waves
// per 32-path tile.
uint32_t cv_bwd_blocks(uint64_t n_paths, uint32_t n_seg, uint32_t* split);
uint32_t cv_values_blocks(uint64_t n_paths, uint32_t n_seg, uint32_t* split);
constexpr int kCvValSlab = 16;  // segments a wave of a split tile holds (values)
// The hedged-value kernel's moment vectors (one per workgroup) and where
// their fixed-order merge (the minibatch's loss) goes.
struct CvValMoments {
  const double* partials;
  uint32_t n_blocks;
  double* out;
};
// Reduces the per-block gradient partials [n_blocks][kMlpNParam], takes one
// Adam step and refreshes the packed fragments, in one launch; or only
// reduces them into grad (the same fixed order). A workgroup of its own in
// the same launch merges the hedged values' moments into vm.out.
hipError_t launch_adam_pack(const float* partials, uint32_t n_blocks, const CvValMoments& vm,
                            double* grad, float* theta, float* m, float* v, int t, double lr,
                            double b1, double b2, double eps, bool bf16, float* w1f, void* w2f,
                            void* w2tf, float* lanec, hipStream_t s);
hipError_t launch_grad_sum(const float* partials, uint32_t n_blocks, const CvValMoments& vm,
                           double* grad, hipStream_t s);

// ---- reductions and diagnostics ----
// Moment vectors of C channels (1..kMaxMomentChannels): n_batch independent
// merges of block-major partials [batch][n_blocks][n_moments(C)] into
// out [batch][n_moments(C)] (device or pinned host memory), in a fixed order.
// A single batch of more than 4096 vectors merges in two stages and overwrites
// the partials' chunk heads. clock: start stamp of the merge, or nullptr.
hipError_t launch_final_merge(double* partials, uint32_t n_blocks, uint32_t C,
                              uint32_t n_batch, double* out, hipStream_t s,
                              uint64_t* clock = nullptr);
hipError_t launch_philox_words(uint32_t k0, uint32_t k1, uint32_t tag, uint64_t n,
                               const uint64_t* paths, const uint64_t* blocks, uint32_t* out,
                               hipStream_t s);
hipError_t launch_normals(uint32_t k0, uint32_t k1, uint32_t tag, uint64_t path,
                          uint64_t k_first, uint64_t count, bool fp64, double* out,
                          hipStream_t s);

}  // namespace mcp
