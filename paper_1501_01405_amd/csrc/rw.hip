// Lattice random-walk replication engines (paper section 5.1, third model).
//
// WAVE mapping: one replication per wavefront, lane w = walker w. The
// replication's visited sites are a byte map in LDS (SiteMap) that every move
// marks with one byte store; at the end the lanes count it and sum squared
// displacements across the wave.
//
// With few replications that form leaves the chip idle and each wave walks
// its 1000 steps one after the other. The walk is a prefix sum of
// independent moves, so rw_seg_kernel cuts every walker's steps into 16
// segments, one lane each: pass 1 counts a segment's net displacement
// (popcounts of the move fields), a 16-lane
// exclusive scan gives each segment its start, and pass 2 replays the
// segment from there, marking the sites. Both forms give identical outputs;
// the launcher picks by the number of replications.
//
// Optionally every walker also marks a bitmap of its own, in global memory,
// and output 2 is the sum over walkers of their popcounts; those forms
// (rw_bits_kernel, rw_seg_sites_kernel) keep the union as a bitmap in LDS, as
// many short walks do (short_walks).
//
// SIMT mapping: one replication per lane; the lane walks its walkers one
// after the other and keeps the replication's bitmap in global memory, the
// per-thread state the paper's thread-per-replication form implies. The
// same kernel with one working lane per wavefront is the paper's own WLP.
//
// On taus88 streams (RNG = RNG_TAUS88) move t of walker w takes bits
// 2(t&15) of output w ceil(T/16) + (t>>4) of the replication's stream: each
// walker reads a contiguous run, so a WAVE lane jumps to its walker's run and
// a SIMT lane reads the stream in order, walker after walker.
#include <algorithm>

#include "device.hpp"
#include "kernels.hpp"
#include "taus.hpp"

namespace mrip {

namespace {

// Move d (0:+x 1:-x 2:+y 3:-y) as two sign-extended 2-bit fields of small
// tables: dx = field d of 0b00'00'11'01, dy = field d of 0b11'01'00'00.
__device__ __forceinline__ void step_delta(uint32_t d, int &dx, int &dy) {
  dx = __builtin_amdgcn_sbfe(0x0D, d << 1, 2);
  dy = __builtin_amdgcn_sbfe(0xD0, d << 1, 2);
}

// Set the visited bit of lattice site c (row-major) in an LDS bitmap.
__device__ __forceinline__ void mark(uint32_t *bm, int c) { atomicOr(&bm[c >> 5], 1u << (c & 31)); }

// Walker bitmap modes: none, owned by this lane (plain read-modify-write),
// shared by the walker's segment lanes (global atomic or).
enum : int { WB_NONE = 0, WB_OWN = 1, WB_SHARED = 2 };

template <int WB>
__device__ __forceinline__ void mark_walker(uint32_t *wb, int c, bool active) {
  if (WB == WB_OWN && active) wb[c >> 5] |= 1u << (c & 31);
  if (WB == WB_SHARED && active) atomicOr(&wb[c >> 5], 1u << (c & 31));
}

// One move of a walker at unwrapped position (X, Y); marks the wrapped site.
// LDS: inactive lanes or into `spare` (a word past the bitmaps), so the
// mark needs no branch.
template <int GRID, bool LDS, int WB>
__device__ __forceinline__ void move1(uint32_t d, bool active, int &X, int &Y, uint32_t *bm,
                                      uint32_t *spare, uint32_t *wb) {
  int dx, dy;
  step_delta(d, dx, dy);
  X += dx;
  Y += dy;
  const int c = (Y & (GRID - 1)) * GRID + (X & (GRID - 1));
  if (LDS) {
    atomicOr(active ? &bm[c >> 5] : spare, 1u << (c & 31));
  } else {
    bm[c >> 5] |= 1u << (c & 31);
  }
  mark_walker<WB>(wb, c, active);
}

// Up to 16 moves from one 32-bit word (2 bits each, lowest first): moves
// g .. min(g + 16, steps) - 1.
template <int GRID, bool LDS, int WB = WB_NONE>
__device__ __forceinline__ void walk16(uint32_t word, uint32_t g, uint32_t steps, bool active,
                                       int &X, int &Y, uint32_t *bm, uint32_t *spare,
                                       uint32_t *wb = nullptr) {
  if (g + 16u <= steps) {
#pragma unroll
    for (int i = 0; i < 16; ++i)
      move1<GRID, LDS, WB>((word >> (2 * i)) & 3u, active, X, Y, bm, spare, wb);
  } else {
    for (uint32_t i = 0; g + i < steps; ++i)
      move1<GRID, LDS, WB>((word >> (2 * i)) & 3u, active, X, Y, bm, spare, wb);
  }
}

// The walk's visited-site map of the forms without per-walker counts: one
// byte per site in 64 KiB of LDS, so that a mark is a plain byte store and
// its address costs one instruction. Byte 0 of the address holds x, byte 1
// holds y, each in the top bits of its byte: a move adds +-(1 << SH) to one
// of them and the torus wraps where the byte does. The low SH bits of the two
// bytes are free: they number the wavefronts (replications) that share the
// 64 KiB, so the space is full. Grids below 64 walk on the 64-torus and are
// folded when counted (a site is its copies modulo the grid).
template <int GRID>
struct SiteMap {
  static constexpr int SH = GRID == 128 ? 1 : 2;  // free low bits per byte
  static constexpr int TORUS = 256 >> SH;         // 128 or 64
  static constexpr int REPS = 1 << (2 * SH);      // replications that fit
  static constexpr uint32_t LOW = (1u << SH) - 1;
  // byte 0 and byte 1 of the address of site (x, y) of replication slot i
  // (in the low bytes; they run unwrapped above)
  static __device__ __forceinline__ int byte0(int x, uint32_t i) {
    return (int)((uint32_t)x << SH) | (int)(i & LOW);
  }
  static __device__ __forceinline__ int byte1(int y, uint32_t i) {
    return (int)((uint32_t)y << SH) | (int)((i >> SH) & LOW);
  }
};

// The address made of the low bytes of X and Y (which run unwrapped above).
__device__ __forceinline__ uint32_t map_address(int X, int Y) {
  return __builtin_amdgcn_perm((uint32_t)Y, (uint32_t)X, 0x0c0c0400u);
}

// Moves 0 .. n - 1 (n <= 16) of a word by one walker at (X, Y) (site << SH |
// slot bits), each marked in the map. Full words take four moves' deltas at
// once: the word's 2-bit fields, spread to bytes, select bytes of a table.
template <int SH>
__device__ __forceinline__ void walk_word(uint32_t word, uint32_t n, int &X, int &Y,
                                          uint8_t *map) {
  constexpr uint32_t P1 = 1u << SH, M1 = 256u - P1;  // +1 and -1 site, as bytes
  constexpr uint32_t TX = P1 | M1 << 8, TY = P1 << 16 | M1 << 24;
  if (n >= 16u) {
    uint32_t dx[4], dy[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t sel = (word >> (2 * k)) & 0x03030303u;  // moves k, 4 + k, 8 + k, 12 + k
      dx[k] = __builtin_amdgcn_perm(0u, TX, sel);
      dy[k] = __builtin_amdgcn_perm(0u, TY, sel);
    }
#pragma unroll
    for (int m = 0; m < 16; ++m) {
      X += (int)(int8_t)(dx[m & 3] >> (8 * (m >> 2)));
      Y += (int)(int8_t)(dy[m & 3] >> (8 * (m >> 2)));
      map[map_address(X, Y)] = 1;
    }
  } else {
    for (uint32_t m = 0; m < n; ++m) {
      int ddx, ddy;
      step_delta((word >> (2 * m)) & 3u, ddx, ddy);
      X += ddx << SH;
      Y += ddy << SH;
      map[map_address(X, Y)] = 1;
    }
  }
}

__device__ __forceinline__ uint32_t moves_left(uint32_t g, uint32_t end) {
  return g < end ? min(16u, end - g) : 0u;
}

// Moves g .. end - 1 (g a multiple of 64) of walker w of replication rep,
// from Philox blocks, word by word.
template <class Word>
__device__ __forceinline__ void each_word(uint32_t g, uint32_t end, uint32_t w, uint32_t rep,
                                          uint32_t k0, uint32_t k1, Word word) {
  for (; g + 64u <= end; g += 64) {
    const Block4 b = philox(g >> 6, w, rep, TAG_RW, k0, k1);
    word(b.x, 16u);
    word(b.y, 16u);
    word(b.z, 16u);
    word(b.w, 16u);
  }
  if (g < end) {
    const Block4 b = philox(g >> 6, w, rep, TAG_RW, k0, k1);
    word(b.x, moves_left(g, end));
    word(b.y, moves_left(g + 16, end));
    word(b.z, moves_left(g + 32, end));
    word(b.w, moves_left(g + 48, end));
  }
}

template <int SH>
__device__ __forceinline__ void walk_blocks(uint32_t g, uint32_t end, uint32_t w, uint32_t rep,
                                            uint32_t k0, uint32_t k1, int &X, int &Y,
                                            uint8_t *map) {
  each_word(g, end, w, rep, k0, k1,
            [&](uint32_t word, uint32_t n) { walk_word<SH>(word, n, X, Y, map); });
}

// Marked sites of replication slot i among those thread j of n counts.
template <int GRID>
__device__ __forceinline__ int count_sites(const uint8_t *map, uint32_t i, int j, int n) {
  using S = SiteMap<GRID>;
  // a row is 256 bytes: 16 vectors of 16 (TORUS / 16 sites each)
  constexpr int T = S::TORUS, COPIES = T / (GRID < T ? GRID : T);
  constexpr int VROW = 16 / COPIES, VECS = VROW * GRID;
  const uint32_t b = (i >> S::SH) & S::LOW;
  uint32_t acc = 0;
  for (int v = j; v < VECS; v += n) {
    const int vx = v % VROW, y = v / VROW;
    uint4 q = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int cy = 0; cy < COPIES; ++cy)
#pragma unroll
      for (int cx = 0; cx < COPIES; ++cx) {
        const uint32_t at = ((uint32_t)((y + cy * GRID) << S::SH) | b) << 8;
        const uint4 p = *(const uint4 *)(map + at + 16 * (vx + cx * VROW));
        q.x |= p.x;
        q.y |= p.y;
        q.z |= p.z;
        q.w |= p.w;
      }
    acc += (q.x + q.y) + (q.z + q.w);  // byte sums: at most 4 x 32 a byte and thread
  }
  acc >>= 8u * (i & S::LOW);
  if (S::SH == 1) return (int)((acc & 0xFFu) + ((acc >> 16) & 0xFFu));
  return (int)(acc & 0xFFu);
}

__device__ __forceinline__ void start_site(uint32_t w, int grid, int &x0, int &y0) {
  x0 = (int)(((w % 8u) * (grid / 8) + grid / 16) % grid);
  y0 = (int)(((w / 8u) * (grid / 8) + grid / 16) % grid);
}

// One replication per wavefront, lane w = walker w (fewer than 64 walkers:
// the other lanes are masked off for the whole walk). A move is 4.5
// vector instructions (its share of the deltas' tables, two adds, the
// address) and one byte store, where a bit map took 11.2 and one atomic or.
// Bound: LDS, 6.8 cycles a store and compute unit, of which 4.8 are bank
// conflicts of 64 walkers at random columns. 64 walkers x 1000 steps on 64 x
// 64: 16384 replications 0.289 ms before, 0.204 now; 35 walkers x 700, 8192
// replications 0.60 / 0.059 (no walkers' lanes marking a spare word).
template <int GRID, int RNG, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void rw_map_kernel(RwArgs a) {
  using S = SiteMap<GRID>;
  static_assert(WAVES <= S::REPS, "one map slot per wavefront");
  __shared__ __attribute__((aligned(16))) uint8_t map[65536];
  const int lane = threadIdx.x & 63;
  const uint32_t wave = threadIdx.x >> 6;
  const uint64_t r = (uint64_t)blockIdx.x * WAVES + wave;
  const uint32_t k0 = (uint32_t)a.seed, k1 = (uint32_t)(a.seed >> 32);
  for (int i = threadIdx.x; i < 65536 / 16; i += 64 * WAVES)
    ((uint4 *)map)[i] = uint4{0u, 0u, 0u, 0u};
  __syncthreads();
  int sd = 0;
  if (r < a.n_reps && (uint32_t)lane < a.walkers) {
    int x0, y0;
    start_site((uint32_t)lane, GRID, x0, y0);
    const int X0 = S::byte0(x0, wave), Y0 = S::byte1(y0, wave);
    int X = X0, Y = Y0;
    map[map_address(X, Y)] = 1;
    const uint32_t rep = (uint32_t)(a.rep0 + r);
    if (RNG == RNG_TAUS88) {
      Taus t = taus_seed(TAG_RW, 0u, rep, k0, k1);
      taus_jump(t, a.taus_walk + (uint64_t)lane * TAUS_COLS);  // to the walker's run
      uint32_t g = 0;
      for (; g + 16u <= a.steps; g += 16) walk_word<S::SH>(taus_next(t), 16u, X, Y, map);
      if (g < a.steps) walk_word<S::SH>(taus_next(t), a.steps - g, X, Y, map);
    } else {
      walk_blocks<S::SH>(0u, a.steps, (uint32_t)lane, rep, k0, k1, X, Y, map);
    }
    const int ux = (X - X0) >> S::SH, uy = (Y - Y0) >> S::SH;
    sd = ux * ux + uy * uy;
  }
  __syncthreads();
  const int cnt = group_sum_i(count_sites<GRID>(map, wave, lane, 64), 64);
  const int ssd = group_sum_i(sd, 64);
  if (lane == 0 && r < a.n_reps) {
    a.ssd[r] = ssd;
    a.distinct[r] = cnt;
  }
}

// Two moves a store. Every walker starts on a site with x + y even, so after
// an even number of moves it is on one again, and the site between is a
// neighbour of it: a byte per even site and direction says "was here and left
// that way", which marks both sites of a pair of moves. In the 64-torus map
// (SiteMap<64>) the direction takes byte 0's two free bits, so a site's four
// directions are one word; byte 1's two free bits and the parity of the
// sites used (a replication on the odd ones starts one site to the right)
// number eight replications in the 64 KiB.
struct PairMap {
  static constexpr int SH = 2;
  static constexpr uint32_t REPS = 8, ENDED = 2;  // ENDED: in direction 0's byte, the last site
  static __device__ __forceinline__ int byte0(int x, uint32_t i) {
    return (int)((uint32_t)x + (i >> 2)) << SH;
  }
  static __device__ __forceinline__ int byte1(int y, uint32_t i) {
    return (int)((uint32_t)y << SH | (i & 3u));
  }
};

// Moves 0 .. n - 1 (n <= 16) of a word by one walker at (X, Y), on an even
// site unless n was odd.
__device__ __forceinline__ void walk_pairs(uint32_t word, uint32_t n, int &X, int &Y,
                                           uint8_t *map) {
  constexpr uint32_t P1 = 1u << PairMap::SH, M1 = 256u - P1;
  constexpr uint32_t TX = P1 | M1 << 8, TY = P1 << 16 | M1 << 24;
  if (n >= 16u) {
    uint32_t d[4], dx[4], dy[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      d[k] = (word >> (2 * k)) & 0x03030303u;  // moves k, 4 + k, 8 + k, 12 + k
      asm("" : "+v"(d[k]));  // bytes to add, not bit fields to extract first
      dx[k] = __builtin_amdgcn_perm(0u, TX, d[k]);
      dy[k] = __builtin_amdgcn_perm(0u, TY, d[k]);
    }
#pragma unroll
    for (int m = 0; m < 16; ++m) {
      if (m % 2 == 0) map[map_address(X + (int)((d[m & 3] >> (8 * (m >> 2))) & 0xFFu), Y)] = 1;
      X += (int)(int8_t)(dx[m & 3] >> (8 * (m >> 2)));
      Y += (int)(int8_t)(dy[m & 3] >> (8 * (m >> 2)));
      asm("" : "+v"(X), "+v"(Y));  // one addition per move (of a byte), not two fields and a sum
    }
  } else {
    for (uint32_t m = 0; m < n; ++m) {
      const uint32_t d = (word >> (2 * m)) & 3u;
      if (m % 2 == 0) map[map_address(X + (int)d, Y)] = 1;
      int ddx, ddy;
      step_delta(d, ddx, ddy);
      X += ddx << PairMap::SH;
      Y += ddy << PairMap::SH;
    }
  }
}

// Visited sites of replication slot i among those lane j counts: even
// sites, each with its right neighbour, an odd one, which was visited if one
// of its four neighbours was left towards it.
template <int GRID>
__device__ __forceinline__ int count_pairs(const uint8_t *map, uint32_t i, int j) {
  constexpr int COPIES = 64 / GRID, HALF = GRID / 2;
  const auto odd_site = [](uint32_t left, uint32_t right, uint32_t below, uint32_t above) {
    return (left & 0x1u) | (right & 0x100u) | (below & 0x10000u) | (above & 0x1000000u);
  };
  if constexpr (COPIES == 1) {
    // a lane has two columns and half of the rows: its even sites and their
    // right neighbours' right neighbours, row by row, are all it reads (a row
    // is 1 KiB further on, so the addresses are constants)
    const int k = j & 31;
    const auto column = [&](int x, int p) {
      return map + map_address((x + p) << PairMap::SH, PairMap::byte1(0, i));
    };
    // rows whose even sites are the even columns (p = 0) and the odd ones
    const int odd_rows = (int)(i >> 2), y0 = (j >> 5) * 32 + odd_rows;  // y0: a p = 0 row
    const uint8_t *h0 = column(2 * k, 0), *r0 = column(2 * k, 2), *h1 = column(2 * k, 1),
                  *r1 = column(2 * k, 3);
    const auto at = [](const uint8_t *c, int y) {
      return *(const uint32_t *)(c + ((y & 63) << 10));
    };
    int cnt = 0;
    uint32_t below = at(h1, y0 - 1);  // the p = 1 row under the first
    for (int y = y0; y < y0 + 32; y += 2) {
      const uint32_t a = at(h0, y), b = at(r0, y);          // p = 0
      const uint32_t c = at(h1, y + 1), d = at(r1, y + 1);  // p = 1
      const uint32_t e = at(r0, y + 2);                     // p = 0 again
      cnt += (a != 0u) + (odd_site(a, b, below, c) != 0u);
      cnt += (c != 0u) + (odd_site(c, d, b, e) != 0u);
      below = c;
    }
    return cnt;
  }
  const auto word = [&](int x, int y) {  // a site's directions, over its copies
    uint32_t w = 0;
#pragma unroll
    for (int cy = 0; cy < COPIES; ++cy)
#pragma unroll
      for (int cx = 0; cx < COPIES; ++cx)
        w |= *(const uint32_t *)(map + map_address((x + cx * GRID) << PairMap::SH,
                                                   PairMap::byte1(y + cy * GRID, i)));
    return w;
  };
  int cnt = 0;
  for (int v = j; v < HALF * GRID; v += 64) {
    const int y = v / HALF, x = 2 * (v % HALF) + ((y + (int)(i >> 2)) & 1);
    const uint32_t here = word(x, y), right = word(x + 2, y), below = word(x + 1, y - 1),
                   above = word(x + 1, y + 1);
    cnt += (here != 0u) + (odd_site(here, right, below, above) != 0u);
  }
  return cnt;
}

// One replication per wavefront, as rw_map_kernel, two moves a store: half
// the stores (3.4 cycles a move and compute unit), and as many vector
// instructions (5 a move, four of them additions of a byte), which bound it.
// 16384 replications of 64 x 1000 on 64 x 64: 0.145 ms, 0.205 with a store
// per move.
template <int GRID, int RNG>
__global__ __launch_bounds__(64 * PairMap::REPS) void rw_pair_kernel(RwArgs a) {
  static_assert(GRID <= 64, "the 64-torus");
  constexpr int WAVES = (int)PairMap::REPS;
  __shared__ __attribute__((aligned(16))) uint8_t map[65536];
  const int lane = threadIdx.x & 63;
  const uint32_t wave = threadIdx.x >> 6;
  const uint64_t r = (uint64_t)blockIdx.x * WAVES + wave;
  const uint32_t k0 = (uint32_t)a.seed, k1 = (uint32_t)(a.seed >> 32);
  for (int i = threadIdx.x; i < 65536 / 16; i += 64 * WAVES)
    ((uint4 *)map)[i] = uint4{0u, 0u, 0u, 0u};
  __syncthreads();
  const bool active = r < a.n_reps && (uint32_t)lane < a.walkers;
  int sd = 0, X = 0, Y = 0;
  if (active) {
    int x0, y0;
    start_site((uint32_t)lane, GRID, x0, y0);
    const int X0 = PairMap::byte0(x0, wave), Y0 = PairMap::byte1(y0, wave);
    X = X0;
    Y = Y0;
    const uint32_t rep = (uint32_t)(a.rep0 + r);
    if (RNG == RNG_TAUS88) {
      Taus t = taus_seed(TAG_RW, 0u, rep, k0, k1);
      taus_jump(t, a.taus_walk + (uint64_t)lane * TAUS_COLS);  // to the walker's run
      uint32_t g = 0;
      for (; g + 16u <= a.steps; g += 16) walk_pairs(taus_next(t), 16u, X, Y, map);
      if (g < a.steps) walk_pairs(taus_next(t), a.steps - g, X, Y, map);
    } else {
      each_word(0u, a.steps, (uint32_t)lane, rep, k0, k1,
                [&](uint32_t word, uint32_t n) { walk_pairs(word, n, X, Y, map); });
    }
    const int ux = (X - X0) >> PairMap::SH, uy = (Y - Y0) >> PairMap::SH;
    sd = ux * ux + uy * uy;
  }
  __syncthreads();
  // a walk of an even number of moves ends on an even site that it does not leave
  if (active && a.steps % 2 == 0)
    atomicOr((uint32_t *)(map + map_address(X, Y)), PairMap::ENDED);
  __syncthreads();
  const int cnt = group_sum_i(count_pairs<GRID>(map, wave, lane), 64);
  const int ssd = group_sum_i(sd, 64);
  if (lane == 0 && r < a.n_reps) {
    a.ssd[r] = ssd;
    a.distinct[r] = cnt;
  }
}

// One replication per wavefront on a bitmap of the visited sites (grid^2
// bits) in LDS, set with atomic ors. PW: with per-walker site counts, a bitmap
// of its own per walker in global memory. Without, the form of short walks
// (short_walks): a walk clears and counts 2 KiB at most, not its share of the
// byte map's 64. Vector instructions bound it (some 12 a move).
template <int GRID, int RNG, bool PW>
__global__ __launch_bounds__(1024) void rw_bits_kernel(RwArgs a) {
  constexpr int WORDS = GRID * GRID / 32;
  constexpr int LOG_ROWB = GRID == 16 ? 1 : GRID == 32 ? 2 : GRID == 64 ? 3 : 4, ROWB = 1 << LOG_ROWB;
  constexpr int WB = PW ? WB_OWN : WB_NONE;
  extern __shared__ uint32_t lds[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t r = (uint64_t)blockIdx.x * (blockDim.x >> 6) + wave;
  const uint32_t k0 = (uint32_t)a.seed, k1 = (uint32_t)(a.seed >> 32);
  uint32_t *bm = lds + wave * WORDS;
  // in bytes; a power of two apart, so a word's address in the map is or-ed in
  const uint32_t base = (uint32_t)wave * (4 * WORDS);
  for (int i = lane; i < WORDS; i += 64) bm[i] = 0u;
  __syncthreads();

  const bool active = r < a.n_reps && (uint32_t)lane < a.walkers;
  const uint32_t w = (uint32_t)lane;
  int sd = 0, mine = 0;
  if (active) {
    int x0, y0;
    start_site(w, GRID, x0, y0);
    int X = x0;
    // this walker's own bitmap (global memory, owned by this lane)
    uint32_t *wb = nullptr;
    if (PW) {
      wb = a.walker_bitmaps + (r * a.walkers + w) * WORDS;
      for (int i = 0; i < WORDS; ++i) wb[i] = 0u;
      mark_walker<WB>(wb, y0 * GRID + x0, true);
    }
    // YB is Y in bytes of a row; the word that holds the walker's site, in
    // bytes, and the bits of it visited since the walker entered it: they reach
    // LDS when it leaves, which half the moves do not (x moves stay in a word
    // 31 times in 32)
    int YB = y0 * ROWB;
    const auto word_at = [&] {
      return (((uint32_t)YB & (uint32_t)(GRID * ROWB - 1) & ~(uint32_t)(ROWB - 1) & ~3u) | base) |
             (GRID > 32 ? __builtin_amdgcn_ubfe((uint32_t)X, 5, GRID == 128 ? 2 : 1) << 2 : 0u);
    };
    const auto bit = [&] {
      return 1u << (GRID > 16 ? (uint32_t)X & 31u : ((uint32_t)YB & 2u) << 3 | ((uint32_t)X & 15u));
    };
    uint32_t at = word_at(), bits = bit();
    const auto flush = [&] { atomicOr((uint32_t *)((char *)lds + at), bits); };
    const auto move = [&](int dx, int dy) {
      X += dx;
      YB += dy * ROWB;
      const uint32_t now = word_at();
      if (now != at) {
        flush();
        bits = 0u;
      }
      at = now;
      bits |= bit();
      if (PW) mark_walker<WB>(wb, ((YB >> LOG_ROWB) & (GRID - 1)) * GRID + (X & (GRID - 1)), true);
    };
    const auto walk = [&](uint32_t word, uint32_t n) {
      // the moves' dx and dy as 2-bit fields, each one extract away
      constexpr uint32_t M = 0x55555555u;
      const uint32_t lo = word & M, hi = (word >> 1) & M;
      const int DX = (int)((hi ^ M) | (lo & ~hi) << 1), DY = (int)(hi | (hi & lo) << 1);
      if (n >= 16u) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
          move(__builtin_amdgcn_sbfe(DX, 2 * i, 2), __builtin_amdgcn_sbfe(DY, 2 * i, 2));
      } else {
        for (uint32_t i = 0; i < n; ++i)
          move(__builtin_amdgcn_sbfe(DX, 2 * i, 2), __builtin_amdgcn_sbfe(DY, 2 * i, 2));
      }
    };
    const uint32_t rep = (uint32_t)(a.rep0 + r);
    if (RNG == RNG_TAUS88) {
      Taus t = taus_seed(TAG_RW, 0u, rep, k0, k1);
      taus_jump(t, a.taus_walk + (uint64_t)w * TAUS_COLS);  // to walker w's run
      for (uint32_t g = 0; g < a.steps; g += 16) walk(taus_next(t), a.steps - g);
    } else {
      each_word(0u, a.steps, w, rep, k0, k1, walk);
    }
    flush();
    const int ux = X - x0, uy = (YB >> LOG_ROWB) - y0;
    sd = ux * ux + uy * uy;
    if (PW)
      for (int i = 0; i < WORDS; ++i) mine += __popc(wb[i]);
  }
  __syncthreads();
  int cnt = 0;
  for (int i = lane; i < WORDS; i += 64) cnt += __popc(bm[i]);
  cnt = group_sum_i(cnt, 64);
  const int ssd = group_sum_i(sd, 64);
  if (PW) mine = group_sum_i(mine, 64);
  if (lane == 0 && r < a.n_reps) {
    a.ssd[r] = ssd;
    a.distinct[r] = cnt;
    if (PW) a.walker_sites[r] = mine;
  }
}

// STRIDE = 1: one replication per lane. STRIDE = 64: one replication per
// wavefront with only its first lane working (the paper's WLP form, 63 of
// 64 lanes idle).
template <int GRID, int STRIDE, int RNG, bool PW>
__global__ void rw_simt_kernel(RwArgs a) {
  constexpr int WORDS = GRID * GRID / 32;
  constexpr int WB = PW ? WB_OWN : WB_NONE;
  if (threadIdx.x % STRIDE) return;
  const uint64_t r = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / STRIDE;
  if (r >= a.n_reps) return;
  const uint32_t k0 = (uint32_t)a.seed, k1 = (uint32_t)(a.seed >> 32);
  uint32_t *bm = a.scratch_bitmaps + r * WORDS;
  for (int i = 0; i < WORDS; ++i) bm[i] = 0u;
  // one walker bitmap per replication, cleared for every walker
  uint32_t *wb = PW ? a.walker_bitmaps + r * WORDS : nullptr;
  int ssd = 0, mine = 0;
  Taus t;
  if (RNG == RNG_TAUS88) t = taus_seed(TAG_RW, 0u, (uint32_t)(a.rep0 + r), k0, k1);
  for (uint32_t w = 0; w < a.walkers; ++w) {
    const int x0 = (int)(((w % 8u) * (GRID / 8) + GRID / 16) % GRID);
    const int y0 = (int)(((w / 8u) * (GRID / 8) + GRID / 16) % GRID);
    int X = x0, Y = y0;
    bm[(y0 * GRID + x0) >> 5] |= 1u << ((y0 * GRID + x0) & 31);
    if (PW) {
      for (int i = 0; i < WORDS; ++i) wb[i] = 0u;
      mark_walker<WB>(wb, y0 * GRID + x0, true);
    }
    if (RNG == RNG_TAUS88) {
      for (uint32_t g = 0; g < a.steps; g += 16)
        walk16<GRID, false, WB>(taus_next(t), g, a.steps, true, X, Y, bm, nullptr, wb);
    } else {
      for (uint32_t g = 0; g < a.steps; g += 64) {
        const Block4 b = philox(g >> 6, w, (uint32_t)(a.rep0 + r), TAG_RW, k0, k1);
        walk16<GRID, false, WB>(b.x, g, a.steps, true, X, Y, bm, nullptr, wb);
        walk16<GRID, false, WB>(b.y, g + 16, a.steps, true, X, Y, bm, nullptr, wb);
        walk16<GRID, false, WB>(b.z, g + 32, a.steps, true, X, Y, bm, nullptr, wb);
        walk16<GRID, false, WB>(b.w, g + 48, a.steps, true, X, Y, bm, nullptr, wb);
      }
    }
    const int ux = X - x0, uy = Y - y0;
    ssd += ux * ux + uy * uy;
    if (PW)
      for (int i = 0; i < WORDS; ++i) mine += __popc(wb[i]);
  }
  int cnt = 0;
  for (int i = 0; i < WORDS; ++i) cnt += __popc(bm[i]);
  a.ssd[r] = ssd;
  a.distinct[r] = cnt;
  if (PW) a.walker_sites[r] = mine;
}

// Net displacement of moves g .. min(g + 16, steps) - 1 of one word.
__device__ __forceinline__ void word_displacement(uint32_t word, uint32_t g, uint32_t steps,
                                                  int &dx, int &dy) {
  const uint32_t n = g + 16u <= steps ? 16u : (g < steps ? steps - g : 0u);
  const uint32_t fields = n == 16u ? 0x55555555u : ((1u << (2u * n)) - 1u) & 0x55555555u;
  const uint32_t lo = word & fields, hi = (word >> 1) & fields;
  // d = 0: +x, 1: -x, 2: +y, 3: -y (hi:lo)
  dx += __popc(fields & ~hi & ~lo) - __popc(lo & ~hi);
  dy += __popc(hi & ~lo) - __popc(hi & lo);
}

// Sum of v over the workgroup (every thread gets it); `sh` holds one int per
// wavefront.
__device__ __forceinline__ int block_sum_i(int v, int *sh) {
  v = group_sum_i(v, 64);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  int t = 0;
  for (int i = 0; i < (int)(blockDim.x >> 6); ++i) t += sh[i];
  return t;
}

// Pass 1 of the segmented walk: the net displacement of walker w's moves
// t0 .. t1 - 1 (t0 a multiple of 64). The words of the first 64 moves are
// kept for pass 2 (for up to 1024 steps that is the whole segment, and pass
// 2 draws nothing).
struct Segment {
  int dx = 0, dy = 0;
  uint32_t first[4] = {0u, 0u, 0u, 0u};
  Taus after;  // taus88: the state after those words
};
template <int RNG>
__device__ __forceinline__ void words64(Taus &ts, uint32_t g, uint32_t t1, uint32_t w, uint32_t rep,
                                        uint32_t k0, uint32_t k1, uint32_t (&wd)[4]) {
  if (RNG == RNG_TAUS88) {
#pragma unroll
    for (int j = 0; j < 4; ++j) wd[j] = g + 16u * j < t1 ? taus_next(ts) : 0u;
  } else {
    const Block4 b = philox(g >> 6, w, rep, TAG_RW, k0, k1);
    wd[0] = b.x;
    wd[1] = b.y;
    wd[2] = b.z;
    wd[3] = b.w;
  }
}
template <int RNG>
__device__ __forceinline__ Segment segment_pass1(const RwArgs &a, uint32_t rep, uint32_t w,
                                                 uint32_t sgi, uint32_t t0, uint32_t t1,
                                                 uint32_t k0, uint32_t k1) {
  Segment s;
  Taus ts;
  if (RNG == RNG_TAUS88) {
    ts = taus_seed(TAG_RW, 0u, rep, k0, k1);
    // to walker w's run, then to this segment's start within it (w <= 63)
    taus_jump(ts, a.taus_walk + (uint64_t)w * TAUS_COLS);
    taus_jump(ts, a.taus_walk + (uint64_t)(TAUS_WALK_WALKERS + sgi) * TAUS_COLS);
  }
  s.after = ts;
  for (uint32_t g = t0; g < t1; g += 64) {
    uint32_t wd[4];
    words64<RNG>(ts, g, t1, w, rep, k0, k1, wd);
    if (g == t0) {
#pragma unroll
      for (int j = 0; j < 4; ++j) s.first[j] = wd[j];
      s.after = ts;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) word_displacement(wd[j], g + 16u * j, t1, s.dx, s.dy);
  }
  return s;
}
// Inclusive sum over the walker's 16 segments.
__device__ __forceinline__ int segment_scan(int v, uint32_t sgi) {
#pragma unroll
  for (int o = 1; o < 16; o <<= 1) {
    const int p = __shfl_up(v, o, 16);
    if ((int)sgi >= o) v += p;
  }
  return v;
}

// 16 lanes per walker, pass 2 marks the sites in the byte map. A workgroup
// takes `reps` replications of `threads` threads (whole wavefronts) each, one
// per map slot: the map fills the LDS of half a compute unit, so with few
// walkers a replication to a workgroup would leave most of it idle (4 walkers
// x 1000 steps, 600 replications: 12.2 us, 8.6 with several and their counting
// shared by idle wavefronts).
template <int GRID, int RNG, bool ONE>
__global__ __launch_bounds__(1024) void rw_seg_kernel(RwArgs a, uint32_t seg, uint32_t threads,
                                                      uint32_t reps) {
  using S = SiteMap<GRID>;
  __shared__ __attribute__((aligned(16))) uint8_t map[65536];
  __shared__ int sh_sd[16], sh_cnt[4][16];
  const int tid = threadIdx.x;
  // wave-uniform: the slot's replication and this thread's place in it
  if (ONE) {  // one replication to a workgroup
    threads = blockDim.x;
    reps = 1;
  }
  const uint32_t slot =
      ONE ? 0u : (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)tid / threads));
  const uint32_t t = (uint32_t)tid - slot * threads;
  const uint64_t r = slot < reps ? (uint64_t)blockIdx.x * reps + slot : a.n_reps;
  const uint32_t w = t >> 4, sgi = t & 15u;
  const uint32_t rep = (uint32_t)(a.rep0 + r);
  const uint32_t k0 = (uint32_t)a.seed, k1 = (uint32_t)(a.seed >> 32);
  // the rows of the slots in use (1 + LOW of them share rows)
  for (uint32_t b = 0; b < (reps + S::LOW) >> S::SH; ++b)
    for (uint32_t v = tid; v < 16u * S::TORUS; v += blockDim.x)
      *(uint4 *)(map + (((v >> 4) << S::SH | b) << 8) + 16 * (v & 15)) = uint4{0u, 0u, 0u, 0u};
  __syncthreads();
  const bool active = w < a.walkers && r < a.n_reps;
  const uint32_t t0 = min(a.steps, sgi * seg), t1 = active ? min(a.steps, t0 + seg) : t0;
  const Segment s1 = segment_pass1<RNG>(a, rep, w, sgi, t0, t1, k0, k1);
  const int sx = segment_scan(s1.dx, sgi), sy = segment_scan(s1.dy, sgi);
  if (active) {
    int x0, y0;
    start_site(w, GRID, x0, y0);
    if (sgi == 0) map[map_address(S::byte0(x0, slot), S::byte1(y0, slot))] = 1;
    // pass 2: the segment's moves from its (unwrapped) start
    int X = S::byte0(x0 + sx - s1.dx, slot);
    int Y = S::byte1(y0 + sy - s1.dy, slot);
    if (t0 < t1) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        walk_word<S::SH>(s1.first[j], moves_left(t0 + 16u * j, t1), X, Y, map);
      if (RNG == RNG_TAUS88) {
        Taus ts = s1.after;
        for (uint32_t g = t0 + 64; g < t1; g += 16)
          walk_word<S::SH>(taus_next(ts), moves_left(g, t1), X, Y, map);
      } else {
        walk_blocks<S::SH>(t0 + 64, t1, w, rep, k0, k1, X, Y, map);
      }
    }
  }
  __syncthreads();
  // the walkers' squared end displacements (the last segment's lane holds the
  // walker's total) and the marked sites: each replication's threads count
  // its own, or, if some wavefronts have none, all threads count all
  const int sd = group_sum_i((active && sgi == 15) ? sx * sx + sy * sy : 0, 64);
  const bool own = ONE || threads * reps == blockDim.x;
  for (uint32_t i = own ? slot : 0u; i < (own ? slot + 1 : reps); ++i) {
    const int cnt = group_sum_i(count_sites<GRID>(map, i, own ? (int)t : tid,
                                                  own ? (int)threads : (int)blockDim.x), 64);
    if ((tid & 63) == 0) sh_cnt[own ? 0 : i][tid >> 6] = cnt;
  }
  if ((tid & 63) == 0) sh_sd[tid >> 6] = sd;
  __syncthreads();
  if (t == 0 && r < a.n_reps) {
    int all = 0, sites = 0;
    const uint32_t first = (uint32_t)tid >> 6, last = first + threads / 64;
    for (uint32_t i = first; i < last; ++i) all += sh_sd[i];
    for (uint32_t i = own ? first : 0u; i < (own ? last : blockDim.x / 64); ++i)
      sites += sh_cnt[own ? 0 : slot][i];
    a.ssd[r] = all;
    a.distinct[r] = sites;
  }
}

// The segmented form with per-walker site counts: a bitmap in LDS for the
// union and one per walker, shared by its 16 lanes, in global memory.
template <int GRID, int RNG>
__global__ __launch_bounds__(1024) void rw_seg_sites_kernel(RwArgs a, uint32_t seg) {
  constexpr int WORDS = GRID * GRID / 32;
  __shared__ uint32_t bm[WORDS + 1];  // + the inactive lanes' spare word
  __shared__ int sh_red[16];
  const int tid = threadIdx.x;
  const uint32_t w = (uint32_t)tid >> 4, sgi = (uint32_t)tid & 15u;
  const uint64_t r = blockIdx.x;
  const uint32_t rep = (uint32_t)(a.rep0 + r);
  const uint32_t k0 = (uint32_t)a.seed, k1 = (uint32_t)(a.seed >> 32);
  for (int i = tid; i < WORDS; i += blockDim.x) bm[i] = 0u;
  const bool active = w < a.walkers;
  uint32_t *wb = nullptr;
  if (active) {
    wb = a.walker_bitmaps + (r * a.walkers + w) * WORDS;
    for (int i = (int)sgi; i < WORDS; i += 16) wb[i] = 0u;
  }
  __syncthreads();
  const uint32_t t0 = min(a.steps, sgi * seg), t1 = min(a.steps, t0 + seg);
  const Segment s1 = segment_pass1<RNG>(a, rep, w, sgi, t0, t1, k0, k1);
  const int sx = segment_scan(s1.dx, sgi), sy = segment_scan(s1.dy, sgi);
  int x0, y0;
  start_site(w, GRID, x0, y0);
  if (active && sgi == 0) {
    mark(bm, y0 * GRID + x0);
    mark_walker<WB_SHARED>(wb, y0 * GRID + x0, true);
  }
  // pass 2: the segment's moves from its (unwrapped) start
  int X = x0 + (sx - s1.dx), Y = y0 + (sy - s1.dy);
  if (t0 < t1) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      walk16<GRID, true, WB_SHARED>(s1.first[j], t0 + 16u * j, t1, active, X, Y, bm, &bm[WORDS],
                                    wb);
  }
  Taus ts = s1.after;
  for (uint32_t g = t0 + 64; g < t1; g += 64) {
    uint32_t wd[4];
    words64<RNG>(ts, g, t1, w, rep, k0, k1, wd);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      walk16<GRID, true, WB_SHARED>(wd[j], g + 16u * j, t1, active, X, Y, bm, &bm[WORDS], wb);
  }
  __syncthreads();
  int mine = 0;
  if (active) {
    // read the walker's words back through the atomic unit (where the other
    // segment lanes' ors were performed)
    for (int i = (int)sgi; i < WORDS; i += 16) mine += __popc(atomicOr(&wb[i], 0u));
  }
  const int sd = block_sum_i((active && sgi == 15) ? sx * sx + sy * sy : 0, sh_red);
  mine = block_sum_i(mine, sh_red);
  int cnt = 0;
  for (int i = tid; i < WORDS; i += blockDim.x) cnt += __popc(bm[i]);
  cnt = block_sum_i(cnt, sh_red);
  if (tid == 0) {
    a.ssd[r] = sd;
    a.distinct[r] = cnt;
    a.walker_sites[r] = mine;
  }
}

// Whether the segmented form is used, for walkers that take `waves`
// wavefronts per replication in it (16 lanes a walker). Up to 512
// replications (256 on taus88 streams, whose segment lanes jump to their
// place first, two tables of 88 columns) its own time is all there is, and
// only short walks are over before it. Beyond, a replication's share of the
// chip grows with its walkers, while the sequential forms take one wavefront
// whatever their number: up to four wavefronts the segmented form wins at any
// number of replications from some hundred moves on, with more only while
// they are few in all. Kernel times on 64 x 64, segmented / sequential (us), by
// walkers x moves: 64 x 1000, 300 replications 14.7 / 21.3, 768 20 / 21, 1000
// 24.6 / 21.2; 64 x 100, 300 14.7 / 7.4; 35 x 1000, 1000 17.4 / 21.2, 2000
// 28.8 / 26.5; 16 x 1000, 1000 11.1 / 21.4, 12288 62 / 110; 16 x 256, 600 9.6 /
// 9.2, 12288 49 / 37; 4 x 1000, 1000 8.5 / 36, 12288 24 / 117; 4 x 128, 1000
// 9.2 / 8.6; 4 x 64, 300 8.3 / 7.4. taus88: 16 x 600, 300 16.4 / 18.9, 1000
// 24.3 / 19.4; 16 x 3000, 4096 93 / 127; 4 x 256, 1000 15.5 / 17.0, 4096
// 24.5 / 21.7; 4 x 600, 4096 25.7 / 38.
bool use_segments(uint32_t waves, uint64_t n_reps, uint32_t steps, bool taus) {
  if (taus) {
    if (n_reps <= 256) return steps >= std::min(256u, 100u * waves);
    return n_reps <= 512 ? steps >= 128u * waves : waves <= 4 && steps >= 512u * waves;
  }
  if (n_reps <= 512) return steps >= std::min(160u, 40u * waves);
  return (waves <= 4 || n_reps * waves <= 12288u) &&
         steps >= std::min(1000u, 132u + 12u * waves * waves);
}
// ... and with per-walker site counts (1000 steps: 44 / 83 us at 1024
// replications, 79 / 87 at 2048, 149 / 146 at 4096; taus88 57 / 56 at 512).
constexpr uint64_t RW_SITES_SEG_MAX_REPS = 2048, RW_SITES_SEG_MAX_REPS_TAUS88 = 512;
// Replications from which a workgroup of the byte-map form takes eight
// wavefronts instead of four: four spread a run over the compute units (2500
// replications 47 us against 58 with eight), but two workgroups fill a
// compute unit's LDS, so eight keep more wavefronts on it (8192: 111 / 107).
constexpr uint64_t RW_MAP8_MIN_REPS = 4096;

// Moves up to which many replications walk on a bitmap: clearing and counting
// the byte map is most of a short walk's time, the more the larger the torus
// (of 128 x 128 four fill the map). Bitmap / byte map, 64 walkers (us):
// 64 x 64, 12288 replications of 10 moves 10.3 / 14.5, of 32 15.2 / 16.7, of 48
// 18.8 / 19.0, of 64 22.7 / 20.6; 4096 of 24 7.6 / 7.7, of 48 10.7 / 9.7; 128 x
// 128, 12288 of 10 10.5 / 25.7, of 100 31.5 / 38, of 128 38 / 39; 16 x 16, 40000
// of 10 22 / 46, of 48 53 / 60.
template <int GRID>
bool short_walks(uint64_t n_reps, uint32_t steps) {
  if (n_reps < 2000) return false;
  return n_reps < 8192 ? steps <= (GRID == 128 ? 80 : 24) : steps <= (GRID == 128 ? 120 : 48);
}

template <int GRID, int WAVES>
hipError_t map_launch(const RwArgs &a, hipStream_t s) {
  const dim3 g((uint32_t)((a.n_reps + WAVES - 1) / WAVES)), b(64 * WAVES);
  if (a.rng == RNG_TAUS88)
    hipLaunchKernelGGL((rw_map_kernel<GRID, RNG_TAUS88, WAVES>), g, b, 0, s, a);
  else
    hipLaunchKernelGGL((rw_map_kernel<GRID, RNG_PHILOX, WAVES>), g, b, 0, s, a);
  return hipGetLastError();
}

// Replications, and moves of all a replication's walkers, from which two
// moves are marked by one store: counting the sites costs more there, whatever
// the walkers (16384 replications of 64 walkers on 64 x 64: 100 moves 31.5 us
// with a store per move, 35.2 with one per two; 150 41 / 41; 200 50 / 47; 300
// 69 / 59; 1000 205 / 145; 12288 of 35 walkers: 256 moves 39 / 42, 600 76 / 75,
// 1000 117 / 112), and with few replications latency bounds the walk, not the
// stores (1024 of 1000 moves 21.5 / 22.0; 2000 of 400 17.8 / 15.6; 3000 of 200
// 16.0 / 16.4).
constexpr uint64_t RW_PAIR_MIN_REPS = 2000;
constexpr uint64_t RW_PAIR_MIN_MOVES = 64 * 256;  // a replication's, over all walkers

template <int GRID>
hipError_t pair_launch(const RwArgs &a, hipStream_t s) {
  const dim3 g((uint32_t)((a.n_reps + PairMap::REPS - 1) / PairMap::REPS)), b(64 * PairMap::REPS);
  if (a.rng == RNG_TAUS88)
    hipLaunchKernelGGL((rw_pair_kernel<GRID, RNG_TAUS88>), g, b, 0, s, a);
  else
    hipLaunchKernelGGL((rw_pair_kernel<GRID, RNG_PHILOX>), g, b, 0, s, a);
  return hipGetLastError();
}

template <int GRID, bool PW>
hipError_t bits_launch(const RwArgs &a, uint32_t wg, hipStream_t s) {
  const uint32_t wpb = wg / 64;
  const uint64_t blocks = (a.n_reps + wpb - 1) / wpb;
  const size_t lds = (size_t)wpb * (GRID * GRID / 32) * sizeof(uint32_t);
  const dim3 g((uint32_t)blocks), b(wg);
  if (a.rng == RNG_TAUS88)
    hipLaunchKernelGGL((rw_bits_kernel<GRID, RNG_TAUS88, PW>), g, b, lds, s, a);
  else
    hipLaunchKernelGGL((rw_bits_kernel<GRID, RNG_PHILOX, PW>), g, b, lds, s, a);
  return hipGetLastError();
}

template <int GRID>
hipError_t wave_launch(const RwArgs &a, uint32_t wg, hipStream_t s) {
  const bool sites = a.walker_sites != nullptr, taus = a.rng == RNG_TAUS88;
  // 16 lanes per walker; segments of whole Philox blocks (64 moves)
  const uint32_t threads = (16u * a.walkers + 63u) / 64u * 64u;
  const uint32_t seg = (a.steps + 16u * 64u - 1u) / (16u * 64u) * 64u;
  if (sites) {
    if (a.n_reps > (taus ? RW_SITES_SEG_MAX_REPS_TAUS88 : RW_SITES_SEG_MAX_REPS))
      return bits_launch<GRID, true>(a, wg, s);
    const dim3 g((uint32_t)a.n_reps), b(threads);
    if (taus) hipLaunchKernelGGL((rw_seg_sites_kernel<GRID, RNG_TAUS88>), g, b, 0, s, a, seg);
    else hipLaunchKernelGGL((rw_seg_sites_kernel<GRID, RNG_PHILOX>), g, b, 0, s, a, seg);
    return hipGetLastError();
  }
  const uint32_t waves = threads / 64;
  if (use_segments(waves, a.n_reps, a.steps, taus)) {
    // a workgroup's replications: as many as put two workgroups on each of 256
    // compute units, and fit; one alone has its map cleared by four wavefronts
    const uint32_t most = std::min<uint32_t>(1024u / threads, SiteMap<GRID>::REPS);
    const uint32_t reps = (uint32_t)std::min<uint64_t>(most, (a.n_reps + 511) / 512);
    const dim3 g((uint32_t)((a.n_reps + reps - 1) / reps));
    const dim3 b(std::max(threads * reps, 256u));
#define MRIP_SEG(RN, ONE) \
  hipLaunchKernelGGL((rw_seg_kernel<GRID, RN, ONE>), g, b, 0, s, a, seg, threads, reps)
    if (taus) { if (reps == 1) MRIP_SEG(RNG_TAUS88, true); else MRIP_SEG(RNG_TAUS88, false); }
    else { if (reps == 1) MRIP_SEG(RNG_PHILOX, true); else MRIP_SEG(RNG_PHILOX, false); }
#undef MRIP_SEG
    return hipGetLastError();
  }
  if (short_walks<GRID>(a.n_reps, a.steps)) return bits_launch<GRID, false>(a, wg, s);
  if constexpr (GRID < 128) {
    if (a.n_reps >= RW_PAIR_MIN_REPS && (uint64_t)a.steps * a.walkers >= RW_PAIR_MIN_MOVES) return pair_launch<GRID>(a, s);
    if (a.n_reps >= RW_MAP8_MIN_REPS) return map_launch<GRID, 8>(a, s);
  }
  return map_launch<GRID, 4>(a, s);
}

template <int GRID>
hipError_t simt_launch(const RwArgs &a, bool one_lane, hipStream_t s) {
  const uint32_t wg = 64;
  const uint64_t threads = a.n_reps * (one_lane ? 64 : 1);
  const uint64_t blocks = (threads + wg - 1) / wg;
  const dim3 g((uint32_t)blocks), b(wg);
#define MRIP_SIMT(ST, RN, PW) hipLaunchKernelGGL((rw_simt_kernel<GRID, ST, RN, PW>), g, b, 0, s, a)
  const bool pw = a.walker_sites != nullptr;
  if (a.rng == RNG_TAUS88) {
    if (one_lane) { if (pw) MRIP_SIMT(64, RNG_TAUS88, true); else MRIP_SIMT(64, RNG_TAUS88, false); }
    else { if (pw) MRIP_SIMT(1, RNG_TAUS88, true); else MRIP_SIMT(1, RNG_TAUS88, false); }
  } else {
    if (one_lane) { if (pw) MRIP_SIMT(64, RNG_PHILOX, true); else MRIP_SIMT(64, RNG_PHILOX, false); }
    else { if (pw) MRIP_SIMT(1, RNG_PHILOX, true); else MRIP_SIMT(1, RNG_PHILOX, false); }
  }
#undef MRIP_SIMT
  return hipGetLastError();
}

}  // namespace

hipError_t launch_rw_wave(const RwArgs &a, uint32_t wg, hipStream_t s) {
  switch (a.grid) {
    case 16: return wave_launch<16>(a, wg, s);
    case 32: return wave_launch<32>(a, wg, s);
    case 64: return wave_launch<64>(a, wg, s);
    case 128: return wave_launch<128>(a, wg, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_rw_simt(const RwArgs &a, bool one_lane, hipStream_t s) {
  switch (a.grid) {
    case 16: return simt_launch<16>(a, one_lane, s);
    case 32: return simt_launch<32>(a, one_lane, s);
    case 64: return simt_launch<64>(a, one_lane, s);
    case 128: return simt_launch<128>(a, one_lane, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace mrip
