// Monte Carlo pi replication engines (paper section 5.1, first model).
//
// Point i of replication r is the pair of words 2(i&1), 2(i&1)+1 of Philox
// block (i>>1, 0, r, TAG_PI); a word's top 24 bits X give u = (X + 1/2)
// 2^-24 and the point is inside the quarter disc iff
// (2X+1)^2 + (2Y+1)^2 <= 2^50, an exact test on two v_mad_u64_u32.
//
// WAVE: one replication per wavefront (or per several workgroups of four,
// when replications are few: pi_parts_kernel), the lanes take interleaved
// blocks (four per lane per iteration). SIMT: one replication per lane
// (STRIDE 1) or per wavefront's first lane (STRIDE 64, the paper's WLP form).
//
// On taus88 streams point i takes outputs 2i and 2i+1 of the replication's
// stream; in the WAVE form lane l takes the contiguous run of points
// [l B, (l+1) B), B = ceil(points / 64), after jumping 2 l B outputs.
// With few replications pi_wide_taus_kernel<X> gives a replication X
// wavefronts (a workgroup). The hit count is an integer sum, identical
// however the points are shared out.
#include <algorithm>

#include "device.hpp"
#include "kernels.hpp"
#include "taus.hpp"

namespace mrip {

namespace {

__device__ __forceinline__ uint32_t inside(uint32_t wx, uint32_t wy) {
  const uint64_t a = 2u * (wx >> 8) + 1u, b = 2u * (wy >> 8) + 1u;
  return a * a + b * b <= (1ull << 50) ? 1u : 0u;
}

// hits of the two points of block k (the second only if it exists)
__device__ __forceinline__ uint32_t block_hits(uint64_t k, uint64_t points, uint32_t rep,
                                               uint32_t k0, uint32_t k1) {
  const Block4 b = philox((uint32_t)k, 0u, rep, TAG_PI, k0, k1);
  return inside(b.x, b.y) + ((2 * k + 1 < points) ? inside(b.z, b.w) : 0u);
}

// wx^2 + wy^2 modulo 2^64; `over` gets the lanes where the sum reached 2^64.
__device__ __forceinline__ uint64_t square_sum(uint32_t wx, uint32_t wy, uint64_t &over) {
  const uint64_t p = (uint64_t)wx * wx;
  uint64_t d;
  asm("v_mad_u64_u32 %0, %1, %2, %2, %3" : "=&v"(d), "=s"(over) : "v"(wy), "v"(p));
  return d;
}

__device__ __forceinline__ uint32_t min3u(uint32_t a, uint32_t b, uint32_t c) {
  return min(min(a, b), c);
}
__device__ __forceinline__ uint32_t max3u(uint32_t a, uint32_t b, uint32_t c) {
  return max(max(a, b), c);
}

// Hits of replication rep's points in blocks [b0, b1), by one wavefront with
// all lanes active (every lane gets the count).
//
// Bound: vector-ALU issue (one instruction per four cycles per SIMD), so
// the loop is written for few instructions: 21.4 per point (29.25 before).
// Each lane has four blocks in flight whose first Philox products advance by
// a 64-bit add. The inside test needs no masking, compare or per-lane count:
// on the whole words w = 2^8 X + low the squares' sum s = wx^2 + wy^2
// carries out of 64 bits when the point is outside, up to the low bits: the
// exact test compares m = sum of (2^8 X + 2^7)^2 with 2^64 (an odd multiple
// of 2^15, never equal), and |s - m| <= 2 * 2^7 * 2^33 = 2^41. So the carry
// is the answer unless s is within 2^41 of 2^64, which its high word shows
// (>= 2^32 - 512 or < 512); then (one iteration in ten thousand) the
// iteration is counted again by the exact test. The carries arrive as lane
// masks, which the scalar unit counts. The round keys are held in vector
// registers (1024 x 1e7 points: 7.87 ms before, 5.83 with scalar keys, 5.18
// with these; two blocks in flight 5.92).
__device__ __forceinline__ uint32_t pi_range(uint32_t b0, uint32_t b1, uint64_t points,
                                             uint32_t rep, uint32_t k0, uint32_t k1) {
  constexpr int U = 4;  // blocks in flight per lane
  k0 = in_vgpr(k0);
  k1 = in_vgpr(k1);
  const uint32_t lane = threadIdx.x & 63;
  // iterations of 64 U blocks of two points each
  const uint32_t whole = min(b1, (uint32_t)(points >> 1));
  const uint32_t iters = whole > b0 ? (whole - b0) / (64u * U) : 0u;
  uint64_t p[U];
#pragma unroll
  for (int j = 0; j < U; ++j) p[j] = (uint64_t)PHILOX_M0 * (b0 + 64u * j + lane);
  uint32_t outside = 0;  // scalar: of the iterations' points
  for (uint32_t it = 0; it < iters; ++it) {
    uint32_t lo = 0xFFFFFFFFu, hi = 0u, out = 0;
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const Block4 b = philox_from(p[j], 0u, rep, TAG_PI, k0, k1);
      p[j] += (uint64_t)PHILOX_M0 * (64u * U);
      uint64_t m0, m1;
      const uint32_t s0 = (uint32_t)(square_sum(b.x, b.y, m0) >> 32);
      const uint32_t s1 = (uint32_t)(square_sum(b.z, b.w, m1) >> 32);
      out += (uint32_t)__popcll(m0) + (uint32_t)__popcll(m1);
      lo = min3u(lo, s0, s1);
      hi = max3u(hi, s0, s1);
    }
    if (__builtin_amdgcn_ballot_w64(lo < 512u || hi >= 0xFFFFFE00u)) {
      uint32_t in = 0;
      for (uint32_t j = 0; j < U; ++j)
        in += block_hits(b0 + (it * U + j) * 64u + lane, points, rep, k0, k1);
      out = 128u * U - (uint32_t)__builtin_amdgcn_readfirstlane(group_sum_i((int)in, 64));
    }
    outside += out;
  }
  uint32_t rest = 0;
  for (uint32_t k = b0 + iters * 64u * U + lane; k < b1; k += 64)
    rest += block_hits(k, points, rep, k0, k1);
  return iters * 128u * U - outside + (uint32_t)group_sum_i((int)rest, 64);
}

__device__ __forceinline__ void write_pi(const PiArgs &a, uint64_t r, uint32_t total) {
  a.hits[r] = (int32_t)total;
  a.estimate[r] = (float)(4.0 * (double)(int32_t)total / (double)a.points);
}

__global__ __launch_bounds__(1024) void pi_wave_kernel(PiArgs a) {
  const uint64_t r = (uint64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (r >= a.n_reps) return;  // wave-uniform
  const uint32_t total = pi_range(0u, (uint32_t)((a.points + 1) / 2), a.points, (uint32_t)r,
                                  (uint32_t)a.seed, (uint32_t)(a.seed >> 32));
  if ((threadIdx.x & 63) == 0) write_pi(a, r, total);
}

// A replication shared by the four wavefronts of each of `parts` workgroups
// (part blockIdx.x / n_reps of replication blockIdx.x % n_reps), each
// wavefront a contiguous range of blocks. With several parts the counts
// meet in the replication's 64-bit slot, arrivals in its high bits: one
// device-scope atomic add both adds and tells the last workgroup that it is
// the last, with the total in its hand, so no fence is needed; it clears the
// slot for the next run. 30 x 1000001 points: 201 us in one 16-wavefront
// workgroup each, 28 spread like this.
__global__ __launch_bounds__(256) void pi_parts_kernel(PiArgs a, uint32_t parts, uint32_t per) {
  __shared__ uint32_t sh[4];
  const uint32_t wave = threadIdx.x >> 6, n = (uint32_t)a.n_reps;
  const uint32_t part = blockIdx.x / n, r = blockIdx.x % n;
  const uint32_t blocks = (uint32_t)((a.points + 1) / 2);
  const uint64_t first = (uint64_t)(part * 4u + wave) * per;
  const uint32_t b0 = (uint32_t)min((uint64_t)blocks, first);
  const uint32_t b1 = (uint32_t)min((uint64_t)blocks, first + per);
  const uint32_t mine =
      pi_range((uint32_t)__builtin_amdgcn_readfirstlane((int)b0),
               (uint32_t)__builtin_amdgcn_readfirstlane((int)b1), a.points, r, (uint32_t)a.seed,
               (uint32_t)(a.seed >> 32));
  if ((threadIdx.x & 63) == 0) sh[wave] = mine;
  __syncthreads();
  if (threadIdx.x != 0) return;
  const uint32_t sum = sh[0] + sh[1] + sh[2] + sh[3];
  if (parts == 1) {
    write_pi(a, r, sum);
    return;
  }
  const unsigned long long old =
      atomicAdd((unsigned long long *)a.slots + r, (1ull << 40) | (unsigned long long)sum);
  if ((old >> 40) == parts - 1) {
    atomicExch((unsigned long long *)a.slots + r, 0ull);
    write_pi(a, r, (uint32_t)old + sum);
  }
}

template <int STRIDE>
__global__ void pi_simt_kernel(PiArgs a) {
  if (threadIdx.x % STRIDE) return;
  const uint64_t r = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / STRIDE;
  if (r >= a.n_reps) return;
  const uint32_t k0 = (uint32_t)a.seed, k1 = (uint32_t)(a.seed >> 32);
  const uint64_t blocks = (a.points + 1) / 2;
  uint32_t hits = 0;
  for (uint64_t k = 0; k < blocks; ++k) hits += block_hits(k, a.points, (uint32_t)r, k0, k1);
  a.hits[r] = (int32_t)hits;
  a.estimate[r] = (float)(4.0 * (double)hits / (double)a.points);
}

// Hits of the next n points of one lane's stream. The test is pi_range's
// (the carry of the squares' sum, counted again exactly where the sum is
// within 2^41 of 2^64), four points an iteration. Vector instructions bound
// it: 21 per point, 41 with a step of the generator per output and the exact
// test throughout (1024 x 1e6 points: 0.70 ms, 1.30 before).
__device__ __forceinline__ uint32_t taus_hits(const Taus &t, uint64_t n) {
  TausStream ts(t);
  uint32_t out = 0, x[8];
  uint64_t i = 0;
  for (; i + 4 <= n; i += 4) {
    ts.next8(x);
    uint32_t s[4], here = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint64_t xx = (uint64_t)x[2 * k] * x[2 * k];
      const uint64_t sum = (uint64_t)x[2 * k + 1] * x[2 * k + 1] + xx;
      here += sum < xx;  // it reached 2^64
      s[k] = (uint32_t)(sum >> 32);
    }
    const uint32_t lo = min(min3u(s[0], s[1], s[2]), s[3]);
    const uint32_t hi = max(max3u(s[0], s[1], s[2]), s[3]);
    if (lo < 512u || hi >= 0xFFFFFE00u) {
      here = 4u;
#pragma unroll
      for (int k = 0; k < 4; ++k) here -= inside(x[2 * k], x[2 * k + 1]);
    }
    out += here;
  }
  uint32_t hits = (uint32_t)i - out;
  if (i < n) {
    ts.next8(x);
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (i + k < n) hits += inside(x[2 * k], x[2 * k + 1]);
  }
  return hits;
}

__global__ void pi_wave_taus_kernel(PiArgs a) {
  const int lane = threadIdx.x & 63;
  const uint64_t r = (uint64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (r >= a.n_reps) return;  // wave-uniform
  const uint32_t k0 = (uint32_t)a.seed, k1 = (uint32_t)(a.seed >> 32);
  const uint64_t per = (a.points + 63) / 64;
  const uint64_t p0 = min(a.points, (uint64_t)lane * per), p1 = min(a.points, p0 + per);
  Taus t = taus_seed(TAG_PI, 0u, (uint32_t)r, k0, k1);
  taus_skip(t, 2 * p0, a.taus);
  const uint32_t hits = taus_hits(t, p1 - p0);
  const int total = group_sum_i((int)hits, 64);
  if (lane == 0) {
    a.hits[r] = total;
    a.estimate[r] = (float)(4.0 * (double)total / (double)a.points);
  }
}

template <int STRIDE>
__global__ void pi_simt_taus_kernel(PiArgs a) {
  if (threadIdx.x % STRIDE) return;
  const uint64_t r = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / STRIDE;
  if (r >= a.n_reps) return;
  const uint32_t k0 = (uint32_t)a.seed, k1 = (uint32_t)(a.seed >> 32);
  Taus t = taus_seed(TAG_PI, 0u, (uint32_t)r, k0, k1);
  uint32_t hits = 0;
  for (uint64_t i = 0; i < a.points; ++i) {
    const uint32_t x = taus_next(t), y = taus_next(t);
    hits += inside(x, y);
  }
  a.hits[r] = (int32_t)hits;
  a.estimate[r] = (float)(4.0 * (double)hits / (double)a.points);
}

// taus88: a replication's X wavefronts (one workgroup), each lane a
// contiguous run of points reached by one jump.
template <int X>
__global__ __launch_bounds__(64 * X) void pi_wide_taus_kernel(PiArgs a) {
  constexpr uint32_t L = 64 * X;  // lanes per replication
  __shared__ uint32_t sh[X];
  const uint32_t tid = threadIdx.x;
  const uint64_t r = blockIdx.x;
  const uint32_t k0 = (uint32_t)a.seed, k1 = (uint32_t)(a.seed >> 32);
  const uint64_t per = (a.points + L - 1) / L;
  const uint64_t p0 = min(a.points, (uint64_t)tid * per), p1 = min(a.points, p0 + per);
  Taus t = taus_seed(TAG_PI, 0u, (uint32_t)r, k0, k1);
  taus_skip(t, 2 * p0, a.taus);
  const uint32_t hits = taus_hits(t, p1 - p0);
  const int wave_total = group_sum_i((int)hits, 64);
  if ((tid & 63) == 0) sh[tid >> 6] = (uint32_t)wave_total;
  __syncthreads();
  if (tid == 0) {
    uint32_t total = 0;
    for (int w = 0; w < X; ++w) total += sh[w];
    write_pi(a, r, total);
  }
}

template <int X>
hipError_t wide_taus_launch(const PiArgs &a, hipStream_t s) {
  hipLaunchKernelGGL(pi_wide_taus_kernel<X>, dim3((uint32_t)a.n_reps), dim3(64 * X), 0, s, a);
  return hipGetLastError();
}

}  // namespace

uint32_t pi_parts(uint64_t n_reps, uint64_t points, int rng) {
  if (rng != RNG_PHILOX || n_reps >= PI_PARTS_MAX_REPS || points < PI_PARTS_MIN_POINTS) return 0;
  // two workgroups per SIMD's worth of wavefronts (2048) if a wavefront then
  // keeps four iterations of 512 points, up to four times as many (which
  // evens out the last round) while it keeps eight
  const uint64_t some = std::min((PI_SOME_GROUPS + n_reps - 1) / n_reps, points / 8192);
  const uint64_t many = std::min((PI_MANY_GROUPS + n_reps - 1) / n_reps, points / 16384);
  return (uint32_t)std::max<uint64_t>(1, std::max(some, many));
}

hipError_t launch_pi_wave(const PiArgs &a, uint32_t wg, hipStream_t s) {
  // taus88: aim at about 4096 wavefronts (four per SIMD) when replications
  // are few and long enough to share out
  if (a.rng == RNG_TAUS88 && a.n_reps < 4096 && a.points >= 65536) {
    const uint64_t x = 4096 / a.n_reps;
    if (x >= 16) return wide_taus_launch<16>(a, s);
    if (x >= 8) return wide_taus_launch<8>(a, s);
    if (x >= 4) return wide_taus_launch<4>(a, s);
    if (x >= 2) return wide_taus_launch<2>(a, s);
  }
  if (const uint32_t parts = pi_parts(a.n_reps, a.points, a.rng)) {
    if (parts > 1 && (!a.slots || a.n_reps >= PI_MANY_GROUPS)) return hipErrorInvalidValue;
    // blocks per wavefront: a whole number of 256-block iterations
    const uint64_t blocks = (a.points + 1) / 2;
    const uint32_t per = (uint32_t)((blocks + 1024ull * parts - 1) / (1024ull * parts) * 256u);
    hipLaunchKernelGGL(pi_parts_kernel, dim3((uint32_t)a.n_reps * parts), dim3(256), 0, s, a,
                       parts, per);
    return hipGetLastError();
  }
  const uint32_t wpb = wg / 64;
  const uint64_t blocks = (a.n_reps + wpb - 1) / wpb;
  if (a.rng == RNG_TAUS88)
    hipLaunchKernelGGL(pi_wave_taus_kernel, dim3((uint32_t)blocks), dim3(wg), 0, s, a);
  else
    hipLaunchKernelGGL(pi_wave_kernel, dim3((uint32_t)blocks), dim3(wg), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_pi_simt(const PiArgs &a, bool one_lane, hipStream_t s) {
  const uint32_t wg = 64;
  const uint64_t threads = a.n_reps * (one_lane ? 64 : 1);
  const uint64_t blocks = (threads + wg - 1) / wg;
  const dim3 g((uint32_t)blocks), b(wg);
  if (a.rng == RNG_TAUS88) {
    if (one_lane) hipLaunchKernelGGL(pi_simt_taus_kernel<64>, g, b, 0, s, a);
    else hipLaunchKernelGGL(pi_simt_taus_kernel<1>, g, b, 0, s, a);
  } else {
    if (one_lane) hipLaunchKernelGGL(pi_simt_kernel<64>, g, b, 0, s, a);
    else hipLaunchKernelGGL(pi_simt_kernel<1>, g, b, 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace mrip
