// Forest-fire cellular automaton replication engines (Drossel-Schwabl,
// synchronous, torus, von Neumann neighbourhood).
//
// The grid is held as two bit planes, `tree` and `burning` (empty = neither),
// 32 cells per word, bit i of word k of a row = cell x = 32k + i. One step is
// then word-parallel logic:
//     nb      = burning shifted left/right (funnel shifts with wrap) | row above | row below
//     ignite  = tree & (nb | [u < TF])
//     grow    = empty & [u < TP]
//     burning' = ignite,  tree' = (tree & ~ignite) | grow,  burnt += popcount(ignite)
// and the random bits come one Philox block per 4 cells.
//
// WAVE mapping: one replication per workgroup of one to eight wavefronts;
// a thread keeps its words' trees in registers and trades burning words with
// its neighbours through LDS, so the grid never leaves the compute unit
// during the 2000 steps.
//
// SIMT mapping: one replication per lane. A 4 KiB grid per lane cannot stay
// in registers; it lives in global memory laid out [plane][row][word][rep]
// so that the 64 lanes of a wave touch 64 consecutive words, and is updated
// in place one row at a time (old rows y-1 and 0 are kept in registers).
#include "device.hpp"
#include "kernels.hpp"

namespace mrip {

namespace {

// mask = 2 mask + [u < t]: the borrow of u - t shifts straight into the mask
// (v_sub_co_u32 then v_addc_co_u32), two instructions per bit where a
// compare, a select and a shift-or would take three. A carry that the vector
// ALU writes to scalar registers may be read by it two wait states later at
// the earliest; the compiler sees to that for its own instructions only, so
// the steps alternate between two carries (c = vcc and %[c]), each read after
// the other one's two instructions, and the first and the last wait.
#define FF_LESS(c, u, t) "v_sub_co_u32 %[tmp], " c ", %[" u "], %[" t "]\n\t"
#define FF_SHIFT(c, m) "v_addc_co_u32 %[" m "], " c ", %[" m "], %[" m "], " c "\n\t"
#define FF_C0 "vcc"
#define FF_C1 "%[c]"

// Both masks of one block's four cells, cell 3 first.
__device__ __forceinline__ void shift_in_less(uint32_t &mp, uint32_t &mf, const Block4 &b,
                                              uint32_t tp, uint32_t tf) {
  uint32_t tmp;
  uint64_t c;
  asm(FF_LESS(FF_C0, "w", "tp") FF_LESS(FF_C1, "w", "tf") "s_nop 0\n\t"
      FF_SHIFT(FF_C0, "mp") FF_LESS(FF_C0, "z", "tp") FF_SHIFT(FF_C1, "mf") FF_LESS(FF_C1, "z", "tf")
      FF_SHIFT(FF_C0, "mp") FF_LESS(FF_C0, "y", "tp") FF_SHIFT(FF_C1, "mf") FF_LESS(FF_C1, "y", "tf")
      FF_SHIFT(FF_C0, "mp") FF_LESS(FF_C0, "x", "tp") FF_SHIFT(FF_C1, "mf") FF_LESS(FF_C1, "x", "tf")
      FF_SHIFT(FF_C0, "mp") "s_nop 0\n\t"
      FF_SHIFT(FF_C1, "mf")
      : [tmp] "=&v"(tmp), [mp] "+&v"(mp), [mf] "+&v"(mf), [c] "=&s"(c)
      : [w] "v"(b.w), [z] "v"(b.z), [y] "v"(b.y), [x] "v"(b.x), [tp] "v"(tp), [tf] "v"(tf)
      : "vcc");
}

// Bits [u < TP] and [u < TF] for the 32 cells of one word: cells
// 32k..32k+31 of row y use blocks q0..q0+7, word (cell & 3).
__device__ __forceinline__ void draw_masks(uint32_t t, uint32_t q0, uint32_t rep, uint32_t k0,
                                           uint32_t k1, uint32_t tp, uint32_t tf, uint32_t &ltp,
                                           uint32_t &ltf) {
  uint32_t mp = 0u, mf = 0u;
  // kept as a loop: eight inlined Philox blocks per word would stop the
  // callers' loops over the register-resident grid from unrolling
#pragma unroll 2
  for (int m = 7; m >= 0; --m)
    shift_in_less(mp, mf, philox(t, q0 + (uint32_t)m, rep, TAG_FF, k0, k1), tp, tf);
  ltp = mp;
  ltf = mf;
}

// bit x of the result = bit x-1 of the row (word k of DW, wrapping)
__device__ __forceinline__ uint32_t from_left(uint32_t cur, uint32_t prev_word) {
  return __builtin_amdgcn_alignbit(cur, prev_word, 31);
}
// bit x of the result = bit x+1 of the row
__device__ __forceinline__ uint32_t from_right(uint32_t next_word, uint32_t cur) {
  return __builtin_amdgcn_alignbit(next_word, cur, 1);
}

// The random words of 16 cells of one step: blocks c .. c + 3 of the lane's
// first block, c0_base the counter word 0 after round 1 of that block (the
// block number enters round 1 by xor alone, and the lane's first is a
// multiple of its block count).
struct Words16 {
  Block4 b[4];
};
__device__ __forceinline__ Words16 draw16(uint32_t c0_base, uint32_t c1, uint32_t c2, uint32_t c3,
                                          uint32_t c, uint32_t k0, uint32_t k1) {
  Words16 w;
#pragma unroll
  for (uint32_t j = 0; j < 4; ++j)
    w.b[j] = philox_rounds<1>(c0_base ^ (c + j), c1, c2, c3, k0, k1);
  return w;
}

// mask = the bits [u < t] of the 16 cells shifted in, cell 15 first.
__device__ __forceinline__ uint32_t less16(uint32_t mask, const Words16 &w, uint32_t t) {
  uint32_t tmp;
  uint64_t c;
#define FF_NEXT(u0, u1)                                                      \
  FF_SHIFT(FF_C0, "mask") FF_LESS(FF_C0, u0, "t") FF_SHIFT(FF_C1, "mask") \
      FF_LESS(FF_C1, u1, "t")
  asm(FF_LESS(FF_C0, "w3", "t") FF_LESS(FF_C1, "z3", "t") "s_nop 0\n\t"
      FF_NEXT("y3", "x3") FF_NEXT("w2", "z2") FF_NEXT("y2", "x2") FF_NEXT("w1", "z1")
      FF_NEXT("y1", "x1") FF_NEXT("w0", "z0") FF_NEXT("y0", "x0")
      FF_SHIFT(FF_C0, "mask") "s_nop 0\n\t"
      FF_SHIFT(FF_C1, "mask")
      : [tmp] "=&v"(tmp), [mask] "+&v"(mask), [c] "=&s"(c)
      : [w3] "v"(w.b[3].w), [z3] "v"(w.b[3].z), [y3] "v"(w.b[3].y), [x3] "v"(w.b[3].x),
        [w2] "v"(w.b[2].w), [z2] "v"(w.b[2].z), [y2] "v"(w.b[2].y), [x2] "v"(w.b[2].x),
        [w1] "v"(w.b[1].w), [z1] "v"(w.b[1].z), [y1] "v"(w.b[1].y), [x1] "v"(w.b[1].x),
        [w0] "v"(w.b[0].w), [z0] "v"(w.b[0].z), [y0] "v"(w.b[0].y), [x0] "v"(w.b[0].x), [t] "v"(t)
      : "vcc");
#undef FF_NEXT
  return mask;
}
#undef FF_LESS
#undef FF_SHIFT
#undef FF_C0
#undef FF_C1

__device__ __forceinline__ uint32_t min16(const Words16 &w) {
  uint32_t m = 0xFFFFFFFFu;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    m = min(min(m, w.b[j].x), w.b[j].y);
    m = min(min(m, w.b[j].z), w.b[j].w);
  }
  return m;
}

// The growth and lightning bits of the word whose first block is c (tp, tf:
// the thresholds, tf_s the latter in a scalar register).
template <bool RARE>
__device__ __forceinline__ void word_masks(uint32_t c0_base, uint32_t c1, uint32_t c2, uint32_t c3,
                                           uint32_t c, uint32_t k0, uint32_t k1, uint32_t tp,
                                           uint32_t tf, uint32_t tf_s, uint32_t &ltp,
                                           uint32_t &ltf) {
  ltp = ltf = 0u;
#pragma unroll
  for (int half = 1; half >= 0; --half) {
    const Words16 w = draw16(c0_base, c1, c2, c3, c + 4u * half, k0, k1);
    ltp = less16(ltp, w, tp);
    if (RARE) {
      uint32_t low = 0u;
      if (__builtin_amdgcn_ballot_w64(min16(w) < tf_s)) low = less16(0u, w, tf);
      ltf |= half ? low << 16 : low;
    } else {
      ltf = less16(ltf, w, tf);
    }
  }
}

// One replication over the THREADS = GRID * GRID / 32 / N threads of a
// workgroup, N consecutive words of a row each. Bound: vector-ALU issue (one
// instruction per four cycles per SIMD), so the step is written for few
// instructions per cell: 11.7 where lightning is rare, 13.6 before.
//  * Round 1 of Philox is the same for a thread's blocks up to an xor with
//    the block's number; rounds 2 and 3 share their products with word 2 and
//    word 0 across the blocks of a step. The round keys sit in vector
//    registers (9.37 ms against 9.97 with scalar keys, 4096 x 128 x 128 x 500).
//  * RARE: the lightning bits of 16 cells are built only if some lane has a
//    word below tf among them, which the minimum of the words shows in half
//    an instruction per cell instead of the two a bit costs.
//  * The burning plane lives in LDS, two copies by step parity, so one
//    barrier a step suffices: a thread draws its words' random masks, waits
//    for the others' burning words of the step before, applies the rule and
//    stores its own new ones into the other copy, whose readers passed this
//    barrier. The trees stay in registers.
// Several wavefronts per replication fill the chip when replications are few
// (alone on its SIMD a wavefront issues one instruction in five cycles) and
// even out the last round of workgroups when they are many.
// 128 x 128 x 200 steps, one wavefront per replication with 2 rows per lane
// in registers / four wavefronts / eight: 30 replications 1.17 / 0.319 / 0.285
// ms, 500 1.18 / 0.560 / 0.548, 700 1.18 / 0.778 / 0.787, 1500 2.00 / 1.42 /
// 1.43, 4096 3.76 / 3.64 / 3.70. 64 x 64, one / two: 256 0.311 / 0.176 ms, 1000
// 0.320 / 0.300, 1500 0.514 / 0.506, 2000 0.512 / 0.516, 4096 0.964 / 0.973.
template <int GRID, int N, bool RARE>
__global__ __launch_bounds__(GRID *GRID / 32 / N) void ff_wave_kernel(FfArgs a) {
  constexpr int DW = GRID / 32, WORDS = GRID * DW, THREADS = WORDS / N;
  static_assert(N <= DW && THREADS % 64 == 0, "whole wavefronts, words of one row per thread");
  __shared__ uint32_t fire[2][WORDS];
  __shared__ int sh_burnt[THREADS / 64];
  const int tid = threadIdx.x, w0 = tid * N;  // the thread's first word, row-major
  const int row = w0 / DW, col = w0 % DW;
  const int above0 = ((row + GRID - 1) % GRID) * DW + col, below0 = ((row + 1) % GRID) * DW + col;
  const int left = row * DW + (col + DW - 1) % DW, right = row * DW + (col + N) % DW;
  const uint32_t rep = (uint32_t)a.rep0 + blockIdx.x;
  const uint32_t k0 = in_vgpr((uint32_t)a.seed), k1 = in_vgpr((uint32_t)(a.seed >> 32));
  const uint64_t p1 = (uint64_t)PHILOX_M1 * rep;
  const uint32_t tp = in_vgpr(a.tp), tf = in_vgpr(a.tf);
  uint32_t c0_base = xor3((uint32_t)(p1 >> 32), (uint32_t)w0 * 8u, k0);

  uint32_t T[N], B[N];
#pragma unroll
  for (int j = 0; j < N; ++j) {
    T[j] = B[j] = 0u;
    fire[0][w0 + j] = 0u;
  }
  int burnt = 0;
  for (uint32_t t = 0; t < a.steps; ++t) {
    const uint64_t p0 = (uint64_t)PHILOX_M0 * t;
    const uint32_t c2 = xor3((uint32_t)(p0 >> 32), TAG_FF, k1), c3 = (uint32_t)p0;
    asm("" : "+v"(c0_base));  // keeps the blocks' first products out of registers
    uint32_t ltp[N], ltf[N];
#pragma unroll
    for (int j = 0; j < N; ++j)
      word_masks<RARE>(c0_base, (uint32_t)p1, c2, c3, 8u * j, k0, k1, tp, tf, a.tf, ltp[j], ltf[j]);
    __syncthreads();
    const uint32_t *old = fire[t & 1];
    uint32_t *now = fire[(t & 1) ^ 1];
    const uint32_t lw = old[left], rw = old[right];
    uint32_t nB[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const uint32_t nb = from_left(B[j], j == 0 ? lw : B[j - 1]) |
                          from_right(j == N - 1 ? rw : B[j + 1], B[j]) | old[above0 + j] |
                          old[below0 + j];
      const uint32_t ign = T[j] & (nb | ltf[j]);
      const uint32_t grow = ~(T[j] | B[j]) & ltp[j];
      nB[j] = ign;
      T[j] = (T[j] & ~ign) | grow;
      burnt += __popc(ign);
      now[w0 + j] = ign;
    }
#pragma unroll
    for (int j = 0; j < N; ++j) B[j] = nB[j];
  }
  burnt = group_sum_i(burnt, 64);
  if ((tid & 63) == 0) sh_burnt[tid >> 6] = burnt;
  __syncthreads();
  if (tid == 0) {
    int total = 0;
    for (int w = 0; w < THREADS / 64; ++w) total += sh_burnt[w];
    a.burnt[blockIdx.x] = total;
  }
}

// STRIDE = 1: one replication per lane; 64: one working lane per wavefront
// (the paper's WLP form).
template <int GRID, int STRIDE>
__global__ void ff_simt_kernel(FfArgs a) {
  constexpr int DW = GRID / 32;
  if (threadIdx.x % STRIDE) return;
  const uint64_t r = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / STRIDE;
  if (r >= a.n_reps) return;
  const uint64_t R = a.n_reps;
  const uint32_t k0 = (uint32_t)a.seed, k1 = (uint32_t)(a.seed >> 32);
  // word (plane p, row y, word k) of replication r
  auto at = [&](int p, uint32_t y, int k) -> uint32_t * {
    return a.state + (((uint64_t)p * GRID + y) * DW + k) * R + r;
  };
  for (uint32_t y = 0; y < (uint32_t)GRID; ++y)
    for (int k = 0; k < DW; ++k) {
      *at(0, y, k) = 0u;
      *at(1, y, k) = 0u;
    }
  int burnt = 0;
  for (uint32_t t = 0; t < a.steps; ++t) {
    uint32_t first[DW], prev[DW], cur[DW];
    for (int k = 0; k < DW; ++k) {
      first[k] = *at(1, 0, k);
      cur[k] = first[k];
      prev[k] = *at(1, GRID - 1, k);
    }
    for (uint32_t y = 0; y < (uint32_t)GRID; ++y) {
      uint32_t nxt[DW];
      for (int k = 0; k < DW; ++k) nxt[k] = (y == GRID - 1) ? first[k] : *at(1, y + 1, k);
      for (int k = 0; k < DW; ++k) {
        const uint32_t nb = from_left(cur[k], cur[(k + DW - 1) % DW]) |
                            from_right(cur[(k + 1) % DW], cur[k]) | prev[k] | nxt[k];
        uint32_t ltp, ltf;
        draw_masks(t, (y * GRID + 32u * k) >> 2, (uint32_t)r, k0, k1, a.tp, a.tf, ltp, ltf);
        const uint32_t tree = *at(0, y, k), burn = cur[k];
        const uint32_t ign = tree & (nb | ltf);
        const uint32_t grow = ~(tree | burn) & ltp;
        *at(0, y, k) = (tree & ~ign) | grow;
        *at(1, y, k) = ign;
        burnt += __popc(ign);
      }
      for (int k = 0; k < DW; ++k) {
        prev[k] = cur[k];
        cur[k] = nxt[k];
      }
    }
  }
  a.burnt[r] = burnt;
}

// Lightning thresholds below which a wavefront's 16 x 64 cells hold a strike
// seldom enough for the minimum to pay (300 steps, rare form against the
// other: f = 1e-4 5.7 / 6.2 ms, 3e-4 5.87 / 6.12, 6e-4 6.07 / 6.13, 1e-3
// 6.23 / 6.13).
constexpr uint32_t RARE_TF = 2147484u;  // f < 5e-4

template <int GRID, int N>
hipError_t wave_launch(const FfArgs &a, hipStream_t s) {
  // at most 2^22 workgroups, 2^31 lanes, per launch
  constexpr uint64_t MOST = 1ull << 22;
  for (uint64_t r0 = 0; r0 < a.n_reps; r0 += MOST) {
    FfArgs b = a;
    b.rep0 = a.rep0 + r0;
    b.n_reps = a.n_reps - r0 < MOST ? a.n_reps - r0 : MOST;
    b.burnt = a.burnt + r0;
    const dim3 g((uint32_t)b.n_reps), t(GRID * GRID / 32 / N);
    if (a.tf < RARE_TF) hipLaunchKernelGGL((ff_wave_kernel<GRID, N, true>), g, t, 0, s, b);
    else hipLaunchKernelGGL((ff_wave_kernel<GRID, N, false>), g, t, 0, s, b);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int GRID>
hipError_t simt_launch(const FfArgs &a, bool one_lane, hipStream_t s) {
  const uint32_t wg = 64;
  const uint64_t threads = a.n_reps * (one_lane ? 64 : 1);
  const uint64_t blocks = (threads + wg - 1) / wg;
  if (one_lane) hipLaunchKernelGGL((ff_simt_kernel<GRID, 64>), dim3((uint32_t)blocks), dim3(wg), 0, s, a);
  else hipLaunchKernelGGL((ff_simt_kernel<GRID, 1>), dim3((uint32_t)blocks), dim3(wg), 0, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_ff_wave(const FfArgs &a, hipStream_t s) {
  // one or two words per thread: the lines follow the times at ff_wave_kernel
  switch (a.grid) {
    case 64: return a.n_reps <= 1500 ? wave_launch<64, 1>(a, s) : wave_launch<64, 2>(a, s);
    case 128: return a.n_reps <= 512 ? wave_launch<128, 1>(a, s) : wave_launch<128, 2>(a, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_ff_simt(const FfArgs &a, bool one_lane, hipStream_t s) {
  switch (a.grid) {
    case 32: return simt_launch<32>(a, one_lane, s);
    case 64: return simt_launch<64>(a, one_lane, s);
    case 96: return simt_launch<96>(a, one_lane, s);
    case 128: return simt_launch<128>(a, one_lane, s);
    case 160: return simt_launch<160>(a, one_lane, s);
    case 192: return simt_launch<192>(a, one_lane, s);
    case 224: return simt_launch<224>(a, one_lane, s);
    case 256: return simt_launch<256>(a, one_lane, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace mrip
