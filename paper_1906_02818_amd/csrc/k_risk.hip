// Risk metrics of a simulated P&L sample (Sec. VI-B.1): the exact order
// statistic behind Value-at-Risk, and the tail sum behind Conditional
// Value-at-Risk, over per-path values already in device memory.
//
// Selection is a most-significant-digit radix select on 64-bit keys that
// order like the doubles (flip every bit of a negative value, set the sign
// bit of a non-negative one), cut short by a sort. A histogram pass counts, in
// LDS, a 12-bit digit of the keys that match the prefix chosen so far; its
// last workgroup scans the 4096 counts, fixes the digit that holds the k-th
// key and the rank left inside it, and clears the counts. After two passes (24
// bits; three above 2^19 values) a few values match: the finishing pass lists
// them and sums the values below them, and its last workgroup sorts the list
// in LDS and takes the k-th key and the tail's remainder from it. When more
// match than the list holds and they are not all equal, the host queues the
// remaining digits and finishes again (select_done). Counts are integers and
// every sum runs in a fixed order: results do not depend on scheduling.
//
// Bound: the latency of dependent launches; the values, 0.8 MB at 100003, are
// read from the caches three times. There: 57 us as 19 launches of 8-bit
// digits with a scan launch each, 26 us as three.
#include "device/reduce.h"
#include "mc_internal.h"

namespace mcp {
namespace {

constexpr uint32_t kSelThreads = 512, kSelBlocks = 256;
constexpr uint32_t kBins = 1u << kSelectDigit;

__device__ __forceinline__ uint64_t order_key(double x) {
  const uint64_t b = (uint64_t)__double_as_longlong(x);
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}
__device__ __forceinline__ double key_value(uint64_t key) {
  return __longlong_as_double((long long)((key >> 63) ? (key & 0x7FFFFFFFFFFFFFFFull) : ~key));
}

// One digit, the `bits` bits from `shift`. first: k is the rank sought and no
// digit is fixed yet.
__global__ __launch_bounds__(kSelThreads) void select_digit_kernel(
    const double* __restrict__ x, uint64_t n, SelectState* st, uint32_t shift, uint32_t bits,
    uint64_t first_k, uint64_t* clock) {
  stamp(clock);
  __shared__ uint32_t h[kBins];
  for (uint32_t b = threadIdx.x; b < kBins; b += kSelThreads) h[b] = 0u;
  __syncthreads();
  const uint64_t prefix = first_k ? 0ull : st->prefix, mask = first_k ? 0ull : st->mask;
  const uint32_t digit_mask = (1u << bits) - 1u;
  const uint64_t stride = (uint64_t)gridDim.x * kSelThreads;
  for (uint64_t i = (uint64_t)blockIdx.x * kSelThreads + threadIdx.x; i < n; i += stride) {
    const uint64_t key = order_key(x[i]);
    if ((key & mask) == prefix) atomicAdd(&h[(uint32_t)(key >> shift) & digit_mask], 1u);
  }
  __syncthreads();
  for (uint32_t b = threadIdx.x; b < kBins; b += kSelThreads) {
    const uint32_t c = h[b];
    if (c) __hip_atomic_fetch_add(&st->hist[b], c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (!arrives_last(&st->arrivals, gridDim.x)) return;
  // Eight neighbouring bins per thread; the scan of the threads' counts by
  // waves, then over the waves.
  constexpr uint32_t PER = kBins / kSelThreads;
  uint64_t own[PER], sum = 0;
#pragma unroll
  for (uint32_t j = 0; j < PER; ++j) {
    own[j] = load_agent(&st->hist[threadIdx.x * PER + j]);
    sum += own[j];
  }
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  uint64_t incl = sum;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint64_t up = __shfl_up((unsigned long long)incl, off, 64);
    if (lane >= (uint32_t)off) incl += up;
  }
  __shared__ uint64_t wave_sum_[kSelThreads / 64];
  if (lane == 63u) wave_sum_[wave] = incl;
  const uint64_t k = first_k ? first_k : st->k;
  __syncthreads();
  uint64_t below = incl - sum;
  for (uint32_t w = 0; w < wave; ++w) below += wave_sum_[w];
#pragma unroll
  for (uint32_t j = 0; j < PER; ++j) {
    if (below < k && k <= below + own[j]) {        // in one bin of one thread
      st->prefix = prefix | ((uint64_t)(threadIdx.x * PER + j) << shift);
      st->mask = mask | ((uint64_t)digit_mask << shift);
      st->k = k - below;
      st->n_match = 0u;
      st->key_min = ~0ull;
      st->key_max = 0ull;
    }
    below += own[j];
    st->hist[threadIdx.x * PER + j] = 0u;
  }
}

// Lists the keys that match the prefix, sums and counts the values below
// them, and in the last workgroup finishes (see the head of the file).
__global__ __launch_bounds__(kSelThreads) void select_finish_kernel(
    const double* __restrict__ x, uint64_t n, SelectState* st, uint64_t* __restrict__ list,
    double* __restrict__ partials, SelectResult* out) {
  const uint64_t prefix = st->prefix, mask = st->mask;
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  double acc[2] = {0.0, 0.0};
  uint64_t lo = ~0ull, hi = 0ull;
  const uint64_t stride = (uint64_t)gridDim.x * kSelThreads;
  for (uint64_t i0 = (uint64_t)blockIdx.x * kSelThreads; i0 < n; i0 += stride) {
    const uint64_t i = i0 + threadIdx.x;
    const double v = i < n ? x[i] : 0.0;
    const uint64_t key = order_key(v);
    const bool match = i < n && (key & mask) == prefix;
    if (i < n && (key & mask) < prefix) {
      acc[0] += 1.0;
      acc[1] += v;
    }
    const uint64_t ballot = __ballot(match);
    if (ballot != 0ull) {
      uint32_t at = 0;
      if (lane == 0u)
        at = __hip_atomic_fetch_add(&st->n_match, (uint32_t)__popcll(ballot), __ATOMIC_RELAXED,
                                    __HIP_MEMORY_SCOPE_AGENT);
      at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) +
           (uint32_t)__popcll(ballot & ((1ull << lane) - 1ull));
      if (match) {
        if (at < kSelectList) store_agent(&list[at], key);
        lo = key < lo ? key : lo;
        hi = key > hi ? key : hi;
      }
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const uint64_t l = __shfl_xor((unsigned long long)lo, off, 64);
    const uint64_t h = __shfl_xor((unsigned long long)hi, off, 64);
    lo = l < lo ? l : lo;
    hi = h > hi ? h : hi;
  }
  if (lane == 0u && hi != 0ull) {          // keys of finite values are not 0
    __hip_atomic_fetch_min(&st->key_min, lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_max(&st->key_max, hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __shared__ double red[2][kSelThreads / 64];
  // Sum over the workgroup, waves in order, in its first thread.
  auto block_total = [&](double (&v)[2]) {
    v[0] = wave_sum(v[0]);
    v[1] = wave_sum(v[1]);
    if (lane == 0u) {
      red[0][wave] = v[0];
      red[1][wave] = v[1];
    }
    __syncthreads();
    if (threadIdx.x == 0u) {
      v[0] = v[1] = 0.0;
      for (uint32_t w = 0; w < kSelThreads / 64; ++w) {
        v[0] += red[0][w];
        v[1] += red[1][w];
      }
    }
  };
  block_total(acc);
  if (threadIdx.x == 0u) {
    store_agent(&partials[blockIdx.x], acc[0]);
    store_agent(&partials[gridDim.x + blockIdx.x], acc[1]);
  }
  if (!arrives_last(&st->arrivals, gridDim.x)) return;

  __shared__ uint64_t keys[kSelectList];
  const uint32_t m = load_agent(&st->n_match);
  const uint64_t k = st->k, k_min = load_agent(&st->key_min), k_max = load_agent(&st->key_max);
  const bool listed = m <= kSelectList;
  double tail[2] = {0.0, 0.0};
  for (uint32_t b = threadIdx.x; b < gridDim.x; b += kSelThreads) {
    tail[0] += load_agent(&partials[b]);
    tail[1] += load_agent(&partials[gridDim.x + b]);
  }
  uint64_t kth = k_min;                    // all matches equal
  if (listed && k_min != k_max) {
    uint32_t size = 2;
    while (size < m) size <<= 1;
    for (uint32_t i = threadIdx.x; i < size; i += kSelThreads) keys[i] = i < m ? load_agent(&list[i]) : ~0ull;
    __syncthreads();
    for (uint32_t run = 2; run <= size; run <<= 1)
      for (uint32_t step = run >> 1; step > 0; step >>= 1) {
        for (uint32_t p = threadIdx.x; p < size / 2; p += kSelThreads) {
          const uint32_t a = 2u * p - (p & (step - 1u)), b = a + step;
          const uint64_t ka = keys[a], kb = keys[b];
          if ((ka > kb) == ((a & run) == 0u)) {
            keys[a] = kb;
            keys[b] = ka;
          }
        }
        __syncthreads();
      }
    kth = keys[k - 1u];
    for (uint32_t i = threadIdx.x; i + 1u < k; i += kSelThreads)
      if (keys[i] < kth) {
        tail[0] += 1.0;
        tail[1] += key_value(keys[i]);
      }
  }
  block_total(tail);
  if (threadIdx.x != 0u) return;
  out->key = kth;
  out->n_tail = tail[0];
  out->tail_sum = tail[1];
  out->done = listed || k_min == k_max ? 1u : 0u;
  out->end = (uint64_t)wall_clock64();
}

uint32_t grid_for(uint64_t n) {
  const uint64_t need = (n + kSelThreads - 1) / kSelThreads;
  return (uint32_t)(need < kSelBlocks ? need : kSelBlocks);
}

hipError_t digits(const double* x, uint64_t n, uint64_t first_k, uint32_t from, uint32_t to,
                  SelectState* st, hipStream_t s, uint64_t* clock) {
  for (uint32_t done = from; done < to; done += kSelectDigit) {
    const uint32_t bits = 64u - done < kSelectDigit ? 64u - done : kSelectDigit;
    hipLaunchKernelGGL(select_digit_kernel, dim3(grid_for(n)), dim3(kSelThreads), 0, s, x, n, st,
                       64u - done - bits, bits, done == 0u ? first_k : 0ull,
                       done == 0u ? clock : nullptr);
  }
  return hipGetLastError();
}

hipError_t finish(const double* x, uint64_t n, SelectState* st, uint64_t* list, double* partials,
                  SelectResult* out, hipStream_t s) {
  hipLaunchKernelGGL(select_finish_kernel, dim3(grid_for(n)), dim3(kSelThreads), 0, s, x, n, st,
                     list, partials, out);
  return hipGetLastError();
}

// Digits before the first finishing pass: of 2^19 values, a few hundred share
// 24 leading bits, and of 2^31 as many share 36.
uint32_t first_digits(uint64_t n) { return n <= (1ull << 19) ? 2u : 3u; }

}  // namespace

static_assert(2 * kSelBlocks * sizeof(double) <= kSelectPartialBytes, "partials");

hipError_t launch_select(const double* x, uint64_t n, uint64_t k, SelectState* st, uint64_t* list,
                         double* partials, SelectResult* out, hipStream_t s, uint64_t* clock) {
  if (n == 0 || k == 0 || k > n) return hipErrorInvalidValue;
  const hipError_t e = digits(x, n, k, 0u, first_digits(n) * kSelectDigit, st, s, clock);
  return e != hipSuccess ? e : finish(x, n, st, list, partials, out, s);
}

hipError_t launch_select_rest(const double* x, uint64_t n, SelectState* st, uint64_t* list,
                              double* partials, SelectResult* out, hipStream_t s) {
  const hipError_t e = digits(x, n, 0u, first_digits(n) * kSelectDigit, 64u, st, s, nullptr);
  return e != hipSuccess ? e : finish(x, n, st, list, partials, out, s);
}

double select_key_to_value(uint64_t key) {
  const uint64_t b = (key >> 63) ? (key & 0x7FFFFFFFFFFFFFFFull) : ~key;
  double v;
  static_assert(sizeof(v) == sizeof(b), "double is 64-bit");
  __builtin_memcpy(&v, &b, sizeof(v));
  return v;
}

}  // namespace mcp
