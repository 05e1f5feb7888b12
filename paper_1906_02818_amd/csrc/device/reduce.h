// Block reduction of per-path values into per-block moments, the first
// stage of the averaging reduction that ends every Monte Carlo estimate
// (Eq. 3) and of its variance term (Sec. V-B).
//
// A moment vector of C channels holds M = 2 + C + C (C+1)/2 doubles:
//   [0] valid paths, [1] non-finite paths, [2 .. 2+C) means,
//   then the co-moments M_ab = sum (y_a - mean_a)(y_b - mean_b), a <= b, in
//   row order.
// Block partials are block-major: block b writes partials[b M .. b M + M),
// one contiguous vector; the final merge combines them the same way.
//
// Parts are combined by the pairwise update of Chan, Golub and LeVeque,
// written about a shift: a part with n paths, mean m and co-moments M is
// held as (n, c, S1 = n (m - c), S2 = M + n (m - c)(m - c)^T) for a shift c
// that is itself one of the parts' means (a sample of the same spread).
// About a common shift, S1 and S2 add like plain sums, so paths, lanes,
// waves and blocks combine without a division; moving a part to another
// shift c' is exact algebra (S1' = S1 + n e, S2' = S2 + S1 e^T + e S1^T +
// n e e^T with e = c - c'), and the moments come back as m = c + S1 / n,
// M = S2 - S1 S1^T / n. All deviations are of the order of the spread, so a
// variance far below the square of the mean (a near-perfect control
// variate) keeps its digits. A thread of a persistent kernel sums its few
// paths about zero and enters as one part about its own mean (ThreadSums),
// which keeps the path loop's registers and code those of plain sums.
// Sums run in fixed orders (per-thread path order, xor butterfly, wave
// order, block order): results do not depend on scheduling.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mcp {

// What one workgroup hands to another of the same launch goes through loads
// and stores of device scope, past the dies' own L2 caches. (Plain stores and
// a fence per wave, which writes a whole L2 back, took a launch of 196
// workgroups from 5 to 30 us.)
template <typename T>
__device__ __forceinline__ T load_agent(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void store_agent(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The start of a launch on the device's constant clock, written by its first
// workgroup (clock: host memory, or nullptr). Two event records around a
// kernel cost a call 7.5 us (22.9 -> 15.3 us for a short kernel, a merge and
// the wait); a stamp costs nothing that shows.
__device__ __forceinline__ void stamp(uint64_t* clock) {
  if (clock != nullptr && threadIdx.x == 0 && blockIdx.x == 0 && blockIdx.y == 0)
    store_agent(clock, (uint64_t)wall_clock64());
}

// True in the last of n workgroups to arrive: every store_agent and
// device-scope atomic of the others is then visible to its load_agent. The
// counter, zero before the launch, is left at zero.
__device__ __forceinline__ bool arrives_last(uint32_t* arrivals, uint32_t n) {
  __shared__ uint32_t order;
  __builtin_amdgcn_s_waitcnt(0);           // this wave's stores have arrived
  __syncthreads();
  if (threadIdx.x == 0u) {
    order = __hip_atomic_fetch_add(arrivals, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (order == n - 1u) *arrivals = 0u;
  }
  __syncthreads();
  return order == n - 1u;
}

// v of the lane whose number differs in bit OFF (a power of two up to 32),
// added to v: one stage of a butterfly whose earlier stages ran over the
// larger offsets, so that lanes equal modulo 2 OFF hold the same v (a rotation
// of a row by 4 or 8 then reads the partner's). The moves between lanes are on
// the vector unit. Through LDS, whose pipe the waves of a CU share, the 132
// moves of a wave for three channels' moments cost a full grid 2.6 us (FP64
// European, 2^18 paths x 64: kernel 33.7 -> 31.1 us) and the merge of its
// 1024 vectors 1 us (6.0 -> 5.0 us).
template <int OFF>
__device__ __forceinline__ uint32_t lane_move(uint32_t x) {
  if constexpr (OFF == 8 || OFF == 4)        // row_ror
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x120 + OFF, 0xf, 0xf, true);
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, OFF == 2 ? 0x4E : 0xB1, 0xf, 0xf, true);
}
template <int OFF>
__device__ __forceinline__ double lane_add(double v) {
  const uint32_t hi = (uint32_t)__double2hiint(v), lo = (uint32_t)__double2loint(v);
  if constexpr (OFF >= 16) {                 // the two halves (pairs of rows), each to all lanes
    const auto h = OFF == 32 ? __builtin_amdgcn_permlane32_swap(hi, hi, false, false)
                             : __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    const auto l = OFF == 32 ? __builtin_amdgcn_permlane32_swap(lo, lo, false, false)
                             : __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
  } else {
    return v + __hiloint2double((int)lane_move<OFF>(hi), (int)lane_move<OFF>(lo));
  }
}

// Orders the wave's own LDS stores before its loads (lockstep wave).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Sum over the wave, the same in every lane (every lane active).
__device__ __forceinline__ double wave_sum(double v) {
  v = lane_add<32>(v);
  v = lane_add<16>(v);
  v = lane_add<8>(v);
  v = lane_add<4>(v);
  v = lane_add<2>(v);
  return lane_add<1>(v);
}

template <int C>
struct PartSums {
  static constexpr int NC = C * (C + 1) / 2;
  static constexpr int M = 2 + C + NC;     // doubles in a moment vector
  double n, bad, shift[C], s1[C], s2[NC];

  __device__ __forceinline__ void zero() {
    n = 0.0;
    bad = 0.0;
#pragma unroll
    for (int a = 0; a < C; ++a) shift[a] = s1[a] = 0.0;
#pragma unroll
    for (int k = 0; k < NC; ++k) s2[k] = 0.0;
  }

  // A part (nb paths, means mb, co-moments cb), in this part's shift; the
  // first non-empty part sets the shift.
  __device__ __forceinline__ void add(double nb, const double* mb, const double* cb) {
    if (nb == 0.0) return;
    if (n == 0.0) {
#pragma unroll
      for (int a = 0; a < C; ++a) shift[a] = mb[a];
    }
    double e[C];
#pragma unroll
    for (int a = 0; a < C; ++a) {
      e[a] = mb[a] - shift[a];
      s1[a] += nb * e[a];
    }
    int k = 0;
#pragma unroll
    for (int a = 0; a < C; ++a)
#pragma unroll
      for (int b = a; b < C; ++b, ++k) s2[k] += (cb ? cb[k] : 0.0) + nb * e[a] * e[b];
    n += nb;
  }

  // One path: counted as valid (its channels enter the moments) or not,
  // and as non-finite or not.
  __device__ __forceinline__ void push(const double (&y)[C], bool valid, bool nonfinite) {
    if (nonfinite) bad += 1.0;
    if (valid) add(1.0, y, nullptr);
  }

  // A stored moment vector [n, bad, means, co-moments].
  __device__ __forceinline__ void add_vector(const double* v) {
    bad += v[1];
    add(v[0], v + 2, v + 2 + C);
  }

  // The same part about the shift c.
  __device__ __forceinline__ void rebase(const double (&c)[C]) {
    double e[C];
#pragma unroll
    for (int a = 0; a < C; ++a) e[a] = n > 0.0 ? shift[a] - c[a] : 0.0;
    int k = 0;
#pragma unroll
    for (int a = 0; a < C; ++a)
#pragma unroll
      for (int b = a; b < C; ++b, ++k) s2[k] += s1[a] * e[b] + e[a] * s1[b] + n * e[a] * e[b];
#pragma unroll
    for (int a = 0; a < C; ++a) {
      s1[a] += n * e[a];
      shift[a] = c[a];
    }
  }
};

// Per-thread sums of a persistent kernel's paths, y and y y^T about zero, on
// grids of 2^21 threads: a few paths each (eight of 2^24, 2^15 of the longest
// run's 2^36), whose rounding errors average out across threads; the thread's
// part enters the reduction about its own mean (part()), and everything above
// the thread combines about shifts. The rounding is of the size of y^2: of
// equal values it can leave a negative sum of squares, which part() takes as 0.
template <int C>
struct ThreadSums {
  static constexpr int NC = C * (C + 1) / 2;
  double n, bad, s[C], ss[NC];

  __device__ __forceinline__ void zero() {
    n = 0.0;
    bad = 0.0;
#pragma unroll
    for (int a = 0; a < C; ++a) s[a] = 0.0;
#pragma unroll
    for (int k = 0; k < NC; ++k) ss[k] = 0.0;
  }

  __device__ __forceinline__ void push(const double (&y)[C], bool valid, bool nonfinite) {
    if (nonfinite) bad += 1.0;
    if (!valid) return;
    n += 1.0;
#pragma unroll
    for (int a = 0; a < C; ++a) s[a] += y[a];
    int k = 0;
#pragma unroll
    for (int a = 0; a < C; ++a)
#pragma unroll
      for (int b = a; b < C; ++b) ss[k++] += y[a] * y[b];
  }

  // (n, shift = mean, S1 = 0, S2 = co-moments).
  __device__ __forceinline__ PartSums<C> part() const {
    PartSums<C> p;
    p.n = n;
    p.bad = bad;
    const double r = n > 0.0 ? 1.0 / n : 0.0;
#pragma unroll
    for (int a = 0; a < C; ++a) {
      p.shift[a] = s[a] * r;
      p.s1[a] = 0.0;
    }
    int k = 0;
#pragma unroll
    for (int a = 0; a < C; ++a)
#pragma unroll
      for (int b = a; b < C; ++b, ++k) {
        const double m = ss[k] - s[a] * s[b] * r;
        p.s2[k] = n == 0.0 || (a == b && m < 0.0) ? 0.0 : m;   // a NaN stays
      }
    return p;
  }
};

// The block's moment vector from its threads' parts, written to
// out[block * M ...]: each wave moves its lanes to the shift of its first
// lane holding a path and sums them (xor butterfly); after one barrier every
// output component is computed by its own thread, moving the waves' sums to
// the shift of the first wave holding a path and adding them in wave order.
template <int C, int BLOCK>
__device__ __forceinline__ void block_reduce(PartSums<C>& t, double* __restrict__ out,
                                             uint32_t block) {
  constexpr int W = BLOCK / 64, NC = PartSums<C>::NC, M = PartSums<C>::M;
  constexpr int R = 2 + 2 * C + NC;        // n, bad, shift, S1, S2 of a wave
  __shared__ double red[W][R];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const unsigned long long holders = __ballot(t.n > 0.0);
  if (holders != 0ull) {                   // wave-uniform
    const int src = __ffsll((long long)holders) - 1;
    double c[C];
#pragma unroll
    for (int a = 0; a < C; ++a)
      c[a] = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(t.shift[a]), src),
                              __builtin_amdgcn_readlane(__double2loint(t.shift[a]), src));
    t.rebase(c);
  }
  t.n = wave_sum(t.n);
  t.bad = wave_sum(t.bad);
#pragma unroll
  for (int a = 0; a < C; ++a) t.s1[a] = wave_sum(t.s1[a]);
#pragma unroll
  for (int k = 0; k < NC; ++k) t.s2[k] = wave_sum(t.s2[k]);
  if (lane == 0) {
    red[wave][0] = t.n;
    red[wave][1] = t.bad;
#pragma unroll
    for (int a = 0; a < C; ++a) {
      red[wave][2 + a] = t.shift[a];
      red[wave][2 + C + a] = t.s1[a];
    }
#pragma unroll
    for (int k = 0; k < NC; ++k) red[wave][2 + 2 * C + k] = t.s2[k];
  }
  __syncthreads();
  for (int q = threadIdx.x; q < M; q += BLOCK) {
    int w0 = 0;
    while (w0 < W - 1 && red[w0][0] == 0.0) ++w0;   // first wave holding a path
    double n = 0.0, bad = 0.0;
    for (int w = 0; w < W; ++w) {
      n += red[w][0];
      bad += red[w][1];
    }
    // S1 of channel a about the common shift (wave order).
    auto S1 = [&](int a) {
      double s = 0.0;
      for (int w = 0; w < W; ++w)
        s += red[w][2 + C + a] + red[w][0] * (red[w][2 + a] - red[w0][2 + a]);
      return s;
    };
    double v;
    if (q == 0) {
      v = n;
    } else if (q == 1) {
      v = bad;
    } else if (q < 2 + C) {
      const int a = q - 2;
      v = n > 0.0 ? red[w0][2 + a] + S1(a) / n : 0.0;
    } else {
      int k = q - 2 - C, a = 0;
      while (k >= C - a) {
        k -= C - a;
        ++a;
      }
      const int b = a + k, kk = q - 2 - C;
      double s2 = 0.0;
      for (int w = 0; w < W; ++w) {
        const double nw = red[w][0];
        const double ea = red[w][2 + a] - red[w0][2 + a], eb = red[w][2 + b] - red[w0][2 + b];
        const double sa = red[w][2 + C + a], sb = red[w][2 + C + b];
        s2 += red[w][2 + 2 * C + kk] + sa * eb + ea * sb + nw * ea * eb;
      }
      v = n > 0.0 ? s2 - S1(a) * S1(b) / n : 0.0;
    }
    out[(size_t)block * M + q] = v;
  }
}

// One path per thread (y[] ignored unless valid).
template <int C, int BLOCK>
__device__ __forceinline__ void block_moments(const double (&y)[C], bool valid, bool nonfinite,
                                              double* __restrict__ partials,
                                              uint32_t block = ~0u) {
  PartSums<C> m;
  m.zero();
  m.push(y, valid, nonfinite);
  block_reduce<C, BLOCK>(m, partials, block == ~0u ? blockIdx.x : block);
}

// ---- Plain sums (counts, tail sums, Gram matrices): moment-major ----------

// Block sum of per-thread vectors, written to partials[m * n_blocks + block]
// (fixed wave butterfly and wave order).
template <int M, int BLOCK>
__device__ __forceinline__ void block_sum(const double (&acc)[M], double* __restrict__ partials,
                                          uint32_t n_blocks) {
  constexpr int W = BLOCK / 64;
  __shared__ double red[M][W];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const double v = wave_sum(acc[m]);
    if (lane == 0) red[m][wave] = v;
  }
  __syncthreads();
  for (int t = threadIdx.x; t < M; t += BLOCK) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < W; ++w) s += red[t][w];
    partials[(size_t)t * n_blocks + blockIdx.x] = s;
  }
}

// Block sum for long vectors (fixed order, like the above): per pass, each
// wave stores 16 entries of its 64 lanes in LDS; lane l adds the 16 values
// of entry l / 4 from lanes 16 (l mod 4) .. 16 (l mod 4) + 15, and two
// butterfly steps combine the four quarters. About a quarter of the
// instructions of a 6-step butterfly per entry.
template <int M, int BLOCK>
__device__ __forceinline__ void block_sum_wide(const double (&acc)[M],
                                               double* __restrict__ partials,
                                               uint32_t n_blocks) {
  constexpr int W = BLOCK / 64, CH = 16;
  __shared__ double buf[W][CH][64 + 1];
  __shared__ double red[M][W];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int c = lane >> 2, q = lane & 3;
#pragma unroll
  for (int m0 = 0; m0 < M; m0 += CH) {
#pragma unroll
    for (int j = 0; j < CH; ++j)
      if (m0 + j < M) buf[wave][j][lane] = acc[m0 + j];
    wave_sync();
    // Quarters 2 and 3 start with their upper half: with the same t in all
    // four, quarters 32 doubles apart met on one bank.
    const double* lower = &buf[wave][c][16 * q + 8 * (q >> 1)];
    const double* upper = &buf[wave][c][16 * q + 8 - 8 * (q >> 1)];
    double s = 0.0;
#pragma unroll
    for (int t = 0; t < 8; ++t) s += lower[t];
#pragma unroll
    for (int t = 0; t < 8; ++t) s += upper[t];
    s += __shfl_xor(s, 1, 64);
    s += __shfl_xor(s, 2, 64);
    if (q == 0 && m0 + c < M) red[m0 + c][wave] = s;
    wave_sync();
  }
  __syncthreads();
  for (int t = threadIdx.x; t < M; t += BLOCK) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < W; ++w) s += red[t][w];
    partials[(size_t)t * n_blocks + blockIdx.x] = s;
  }
}

}  // namespace mcp
