// The fixed-order fp64 two-pass reduction (count, mean, unbiased variance) by
// one 256-thread workgroup, shared by the reduction kernels and the
// simulation kernel that reduces the previous run's outputs in an extra
// workgroup: both give the same bits. Order: thread-strided partial sums, a
// butterfly over each wavefront, then the four wavefronts in a fixed tree.
//
// Latency is all there is to it: it stands between the last replication and
// the host that waits for the interval, or at the end of the launch. So its
// loads are all in flight at once and kept for the second pass, there is one
// barrier in each pass, and the results go out in one store that needs no
// flag after it (a store to the host that something waits for takes 2 us).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mrip {

constexpr int RED_THREADS = 256;
constexpr int RED_KEEP = 8;  // values per thread and output kept between the passes

template <int K>
struct RedShared {
  double first[K][RED_THREADS / 64], second[K][RED_THREADS / 64];
  long long whole[K][RED_THREADS / 64];
};

// Sums over the workgroup, in every thread; `sh` is used once per launch or
// with a barrier between.
template <int K, class T>
__device__ __forceinline__ void red_block_sums(T (&v)[K], T (*sh)[RED_THREADS / 64]) {
#pragma unroll
  for (int k = 0; k < K; ++k) {
    for (int m = 1; m < 64; m <<= 1) v[k] += __shfl_xor(v[k], m, 64);
    if ((threadIdx.x & 63) == 0) sh[k][threadIdx.x >> 6] = v[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = (sh[k][0] + sh[k][1]) + (sh[k][2] + sh[k][3]);
}

// A sum's accumulator: int32 outputs are summed exactly for the mean.
template <class X>
struct RedSum {
  using type = double;
  template <int K>
  static __device__ __forceinline__ auto &shared(RedShared<K> &sh) { return sh.first; }
};
template <>
struct RedSum<int32_t> {
  using type = long long;
  template <int K>
  static __device__ __forceinline__ auto &shared(RedShared<K> &sh) { return sh.whole; }
};

// mean[k], var[k] of x[k][0..n), in every thread of a 256-thread workgroup.
template <int K, class X>
__device__ __forceinline__ void reduce_outputs(const X *const (&x)[K], uint64_t n, double (&mean)[K],
                                               double (&var)[K], RedShared<K> &sh) {
  using T = typename RedSum<X>::type;
  X kept[K][RED_KEEP];
  T s[K] = {};
#pragma unroll
  for (int i = 0; i < RED_KEEP; ++i) {
    const uint64_t j = threadIdx.x + (uint64_t)i * RED_THREADS;
#pragma unroll
    for (int k = 0; k < K; ++k) kept[k][i] = j < n ? x[k][j] : X(0);
  }
#pragma unroll
  for (int i = 0; i < RED_KEEP; ++i)
#pragma unroll
    for (int k = 0; k < K; ++k) s[k] += (T)kept[k][i];
  const uint64_t rest = threadIdx.x + (uint64_t)RED_KEEP * RED_THREADS;
  for (int k = 0; k < K; ++k)
#pragma unroll 8
    for (uint64_t j = rest; j < n; j += RED_THREADS) s[k] += (T)x[k][j];
  red_block_sums<K>(s, RedSum<X>::shared(sh));
  double ss[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    mean[k] = (double)s[k] / (double)n;
    ss[k] = 0.0;
#pragma unroll
    for (int i = 0; i < RED_KEEP; ++i) {
      const double d = (double)kept[k][i] - mean[k];
      if (threadIdx.x + (uint64_t)i * RED_THREADS < n) ss[k] += d * d;
    }
  }
  for (int k = 0; k < K; ++k)
#pragma unroll 8
    for (uint64_t j = rest; j < n; j += RED_THREADS) {
      const double d = (double)x[k][j] - mean[k];
      ss[k] += d * d;
    }
  red_block_sums<K>(ss, sh.second);
#pragma unroll
  for (int k = 0; k < K; ++k) {
    mean[k] = n > 0 ? mean[k] : 0.0;
    var[k] = n > 1 ? ss[k] / (double)(n - 1) : 0.0;
  }
}

// Write K outputs' results to the host: per output the mean, the variance,
// and each again with `tag` mixed in, four words, in one store. The words
// may become visible in any order: the host takes a value once its second
// word agrees with it under the run's own tag, and earlier runs of the slot
// had other tags, so a value that is still an earlier run's never agrees.
template <int K>
__device__ __forceinline__ void publish(uint64_t *out, const double (&mean)[K],
                                        const double (&var)[K], uint64_t tag) {
  const int t = threadIdx.x;
  if (t >= 4 * K) return;
  double v = mean[0];
#pragma unroll
  for (int k = 0; k < K; ++k)
    if (t >> 2 == k) v = t & 1 ? var[k] : mean[k];
  __hip_atomic_store(out + t, (uint64_t)__double_as_longlong(v) ^ (t & 2 ? tag : 0),
                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

}  // namespace mrip
