// Neighbour-list construction from the cell list (Sec. 3.5: visit the cell
// of i and its 26 neighbours, keep the pairs closer than the list radius;
// GPU neighbour matrix W_{m,i} = m-th neighbour of i).
//
// The pair test is the exact FP64 minimum-image predicate
//   dx = xi - xj; dx > L/2 ? dx - L : (dx < -L/2 ? dx + L : dx)
//   d2 = (dx*dx + dy*dy) + dz*dz < r2
// with floating-point contraction off, on the caller's FP64 values, so the
// list is bit-identical to the all-pairs definition.
//
// The builder: one workgroup per brick (several for small systems) stages its
//    tile in LDS and tests the 27 tile cells of each particle's stencil (a
//    full list: each cell's particles of the lower half along x first, so
//    that a particle skips the half of the next or previous cell along x that
//    lies beyond the list radius, 5/6 of each stencil row); entries are
//    16-bit tile byte offsets, column-major, so the force pass reads one
//    coalesced word per four neighbours.  Large systems: a lane per particle,
//    distances on the matrix cores (lane_row); small or sparse ones and half
//    lists: a wave per home cell or less (scan_range, row_bits), and the
//    lists are the same, entry for entry.  A half list (each pair once,
//    Newton's third law) keeps j in the list of i only if j's tile index is
//    larger (tile.h): four of the nine stencil rows whole, and the row of i's
//    cell from i on.
#include <math.h>

#include <type_traits>

#include "device_util.h"
#include "internal.h"
#include "list_out.h"
#include "tile.h"

namespace mdpl {

// ------------------------------------------------------------------ LJ list
// One wave per home cell at a time.  The cell's particles (na <= 64 per
// pass) are spread over the 64 lanes as na x K (K = 64 / na): lane
// (a, k) tests particle a against candidates k, k+K, k+2K, ... of each
// stencil row (three consecutive tile cells, one contiguous index range),
// so all lanes walk the same 9 rows together and lanes with equal k read
// the same tile slot.  Accepted neighbours get their rank from a
// per-particle LDS counter and are stored as 16-bit halves of the list
// words; a final pass pads the last word and writes the counts.
//
// Exactness with an FP32 screen.  The tile holds FP32 positions relative to
// its corner with the periodic image already applied, X = fl32((x + s L) - o).
// Each coordinate is then within 2^-24 span of the exact image (span = tile
// extent), a difference within 2^-24 (2 span + 2 r_ext) of the exact one,
// and the FP32 squared distance d2f of any pair near the list radius
// within e = 2 sqrt(3) r_ext 2^-24 (2 span + 2 r_ext) + 3 2^-24 r^2 of the
// definition's d2 (whose own rounding is ~1e-14).  With the guard band
// g = 8 e, d2f < r^2 - g proves d2 < r^2 and d2f > r^2 + g proves d2 >= r^2;
// the rare pairs in between are decided by the definition itself (the
// conditional minimum image on the stored FP64 positions).  The list is
// therefore bit-identical to the all-pairs definition.
constexpr float kFarF = 1e30f;  // dummy slot: its d2f overflows to +inf
// Out of reach, and its square is finite: 2^50, so that the terms of two such
// particles cancel without rounding and leave the pair to the exact test.
constexpr float kFarLane = 1125899906842624.0f;
constexpr int kBuildWant = 512;  // workgroups of a build that shares its bricks
constexpr int kLaneThreads = 512;

struct RowScan {
  float xi, yi, zi;            // FP32 tile coordinates of the particle
  float r2lo, r2hi;            // r^2 -/+ g
  double xs, ys, zs;           // its stored FP64 position (exact test)
  const double *x, *y, *z;     // stored FP64 positions, sorted slots
  double r2, Lx, Ly, Lz, hx, hy, hz;
  int self, K, max_nb;
  int* cnt;                    // the particle's LDS counter
  uint16_t* base;              // its list: entry m at base[(m >> 2) * stride4 + (m & 3)]
  uint32_t stride4;
  uint32_t pitch;              // bytes per word row, 2 * stride4
};

// Candidates u = ub, ub + K, ... < ue (one contiguous range of tile
// indices), UNROLL at a time so that their LDS loads overlap; slots past the
// end read the far-away dummy.  One LDS atomic reserves the ranks of all
// accepted candidates of a step; each candidate's offset among them is
// known before it, so a store needs one comparison with the capacity.
// A24: the word-row pitch is below 2^24 bytes, so the byte offset of rank m
// (below 2^32, as m >> 2 < 2^8) comes from a 24-bit product.
// Candidate indices are carried as byte offsets into the 4-byte tile
// arrays (4 u), which saves a shift per candidate.
// COUNT: only the number of accepted candidates is returned, nothing is stored.
template <int UNROLL, int SHIFT, bool A24, bool COUNT, typename TS>
__device__ __forceinline__ int scan_range(const TS& t, int ub, int ue, const RowScan& q) {
  int found = 0;
  const int ue4 = 4 * ue, step4 = 4 * UNROLL * q.K, k4 = 4 * q.K, self4 = 4 * q.self;
  for (int u04 = 4 * ub; u04 < ue4; u04 += step4) {
    constexpr uint32_t kNone = 1u << 20;  // offset of a rejected candidate: past any list
    int uu4[UNROLL];
    uint32_t rank[UNROLL];  // offset among this step's accepted candidates, or kNone
    uint32_t na = 0;
#pragma unroll
    for (int j = 0; j < UNROLL; ++j) {
      const int u4 = u04 + j * k4;
      uu4[j] = u4 < ue4 ? u4 : 4 * TS::kDummy;
    }
#pragma unroll
    for (int j = 0; j < UNROLL; ++j) {
      const float dx = q.xi - *(const float*)((const char*)t.x + uu4[j]);
      const float dy = q.yi - *(const float*)((const char*)t.y + uu4[j]);
      const float dz = q.zi - *(const float*)((const char*)t.z + uu4[j]);
      const float d2f = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
      const bool other = uu4[j] != self4;
      bool acc = other && d2f < q.r2lo;
      if (other && !(d2f < q.r2lo) && d2f <= q.r2hi) {
        // inside the guard band: the definition decides
        const int u = uu4[j] >> 2;
        const int c = t.cell[u];
        const int sj = t.src[c] + (u - t.prefix[c]);
        acc = exact_d2(q.xs, q.ys, q.zs, q.x[sj], q.y[sj], q.z[sj], q.Lx, q.Ly, q.Lz, q.hx, q.hy,
                       q.hz) < q.r2;
      }
      rank[j] = acc ? na : kNone;
      na += acc ? 1u : 0u;
    }
    if constexpr (COUNT) {
      found += (int)na;
    } else if (na) {
      const uint32_t m = (uint32_t)atomicAdd(q.cnt, (int)na);
#pragma unroll
      for (int j = 0; j < UNROLL; ++j) {
        const uint32_t mj = m + rank[j];
        if (mj < (uint32_t)q.max_nb) {
          if constexpr (A24)
            *(uint16_t*)((char*)q.base + (__umul24(mj >> 2, q.pitch) + ((mj & 3u) << 1))) =
                (uint16_t)(uu4[j] << (SHIFT - 2));
          else
            q.base[(uint64_t)(mj >> 2) * q.stride4 + (mj & 3u)] = (uint16_t)(uu4[j] << (SHIFT - 2));
        }
      }
    }
  }
  return found;
}

// One stencil row of up to 128 candidates against one particle per lane, the
// decisions kept as a bit per candidate, so that a second pass over the
// accepted ones can store them without testing again.  The same screen and
// exact test as scan_range.  Candidates past the row (within the tile's
// arrays or just behind them in LDS) are masked out.
constexpr int kRowWords = 4;
struct RowBits {
  uint32_t w[kRowWords];
};
template <typename TS>
__device__ __forceinline__ int row_bits(const TS& t, int ub, int n, const RowScan& q, float r2,
                                        float guard, RowBits& bits) {
  int found = 0;
#pragma unroll
  for (int c = 0; c < kRowWords; ++c) {
    uint32_t word = 0;
    const int left = n - 32 * c, u0 = ub + 32 * c;
    if (__any(left > 0)) {
      const int u = left > 0 ? u0 : 0;
      const float *px = t.x + u, *py = t.y + u, *pz = t.z + u;
      float near = 3e38f;
#pragma unroll
      for (int b = 31; b >= 0; --b) {
        const float dx = q.xi - px[b], dy = q.yi - py[b], dz = q.zi - pz[b];
        const float e =
            __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, __builtin_fmaf(dx, dx, -r2)));
        near = fminf(near, __builtin_fabsf(e));
        word = (word << 1) | (e < 0.0f ? 1u : 0u);
        if (b % 8 == 0) __builtin_amdgcn_sched_barrier(0);
      }
      if (near <= guard) {  // the definition decides those inside the guard band
        for (int b = 0; b < 32 && b < left; ++b) {
          const float dx = q.xi - px[b], dy = q.yi - py[b], dz = q.zi - pz[b];
          const float e =
              __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, __builtin_fmaf(dx, dx, -r2)));
          if (!(__builtin_fabsf(e) <= guard)) continue;
          const int cell = t.cell[u0 + b];
          const int sj = t.src[cell] + (u0 + b - t.prefix[cell]);
          const bool in = exact_d2(q.xs, q.ys, q.zs, q.x[sj], q.y[sj], q.z[sj], q.Lx, q.Ly, q.Lz,
                                   q.hx, q.hy, q.hz) < q.r2;
          word = (word & ~(1u << b)) | (in ? 1u << b : 0u);
        }
      }
      word &= left >= 32 ? ~0u : (left > 0 ? (1u << left) - 1u : 0u);
      const int self = q.self - u0;
      word &= self >= 0 && self < 32 ? ~(1u << self) : ~0u;
    }
    bits.w[c] = word;
    found += __popc(word);
  }
  return found;
}

// Stores the accepted candidates of a row as entries m, m + 1, ... of the
// particle's list, in the order of scan_range with K = 1 (ascending) or K = 2
// lanes per particle (of every eight the even ones first).
__device__ __forceinline__ void row_store(const RowBits& bits, int ub, uint32_t m,
                                          const RowScan& q) {
#pragma unroll
  for (int c = 0; c < kRowWords; ++c) {
    uint32_t w = bits.w[c];
    if (q.K == 2) {  // even bits of each byte to its low half, odd bits to its high half
      uint32_t x = (w ^ (w >> 1)) & 0x22222222u;
      w ^= x ^ (x << 1);
      x = (w ^ (w >> 2)) & 0x0c0c0c0cu;
      w ^= x ^ (x << 2);
    }
    for (; w && m < (uint32_t)q.max_nb; w &= w - 1, ++m) {
      int b = __builtin_ctz(w);
      if (q.K == 2) b = (b & ~7) | ((b & 3) << 1) | ((b >> 2) & 1);
      *(uint16_t*)((char*)q.base + (__umul24(m >> 2, q.pitch) + ((m & 3u) << 1))) =
          (uint16_t)((ub + 32 * c + b) << kFullShift);
    }
  }
}

// A lane per particle (large systems).  What bounds it is vector issue and
// the latency of the screen's chain from table to decision, about 6500 vector
// instructions for the ~420 candidates and 80 entries of 64 particles: the
// screen costs 2.6 of them per candidate (four rank-1 products on the matrix
// cores, against 12 in scan_range), and the entries are appended four
// positions at a time without a loop (a loop over the set bits of each word,
// whose trips follow the fullest of 64 lanes, took half of the time).
// N = 10^6 408 -> 280 us, 262144 135 -> 101 us, 125000 (list radius 3.3)
// 133 -> 83 us against one wave per home cell.
//
// A list is in the order in which the
// cell kernel's lanes find its entries: of each row's candidates i = 0, 1, ...
// in blocks of 4 K, K = 64 / (particles of the cell), first those with
// i % K = 0 of a block, then those with i % K = 1, and so on.  The tables give
// for K <= kLaneK the candidate at position p of that order, as list entry
// and, for every fourth position, as byte offset into the 4-byte tile arrays
// (the three that follow lie K apart each), and the positions that exist in
// an incomplete last block of `rem` candidates.
constexpr int kLaneK = 8, kLaneRow = 256;  // largest K; positions of a row
static_assert(kListRow == kLaneRow - 4 * kLaneK, "an incomplete last block reaches past the row");
struct LaneTables {
  uint16_t pos[kLaneK][kLaneRow];
  uint16_t group[kLaneK][kLaneRow / 4];
  uint32_t valid[kLaneK][4 * kLaneK];
  int32_t over[kLaneK], over4[kLaneK];  // div_small's multipliers for K and 4 K
};
constexpr LaneTables lane_tables() {
  LaneTables t{};
  for (int K = 1; K <= kLaneK; ++K) {
    for (int p = 0; p < kLaneRow; ++p) {
      const int i = p / (4 * K) * (4 * K) + p % 4 * K + p / 4 % K;
      t.pos[K - 1][p] = (uint16_t)(i << kFullShift);
      if (p % 4 == 0) t.group[K - 1][p / 4] = (uint16_t)(4 * i);
    }
    t.over[K - 1] = 65536 / K + 1;
    t.over4[K - 1] = 65536 / (4 * K) + 1;
    for (int rem = 0; rem < 4 * K; ++rem)
      for (int p = 0; p < 4 * K; ++p)
        if (p % 4 * K + p / 4 < rem) t.valid[K - 1][rem] |= 1u << p;
  }
  return t;
}
__device__ const LaneTables kLaneTables = lane_tables();

__device__ __forceinline__ int wave_max_i32(int v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const int o = __shfl_xor(v, off, 64);
    v = o > v ? o : v;
  }
  return v;
}

// a / b for 0 <= a <= 2 kLaneRow, 1 <= b <= 4 kLaneK from m = 65536 / b + 1
__device__ __forceinline__ int div_small(int a, int m) { return (int)(__umul24(a, m) >> 16); }

__device__ const Compress kCompress = compress_table();

// The particle of a lane for the matrix cores: e = |x_i - x_j|^2 - r^2 of four
// particles and four candidates is (|x_i|^2 - r^2) + 1 |x_j|^2 - 2 x_i x_j -
// 2 y_i y_j - 2 z_i z_j, a start value and four rank-1 products.  In
// v_mfma_f32_4x4x1 every quad of lanes forms such a 4 x 4 block: lane l of
// the quad holds candidate l of the left operand and particle l of the right
// one and receives its own particle's four results.
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
struct LanePoint {
  float ax, ay, az;  // -2 x_i
  f32x4 c;           // |x_i|^2 - r^2, four times
  int self, slot, K;
};
// The definition's test of slot i and the particle at tile index u.
template <typename TS>
__device__ __forceinline__ bool exact_pair(const TS& t, const Grid& g, const double* __restrict__ x,
                                        const double* __restrict__ y,
                                        const double* __restrict__ z, int i, int u, double r2) {
  const int cell = t.cell[u];
  const int j = t.src[cell] + (u - t.prefix[cell]);
  return exact_d2(x[i], y[i], z[i], x[j], y[j], z[j], g.box[0], g.box[1], g.box[2],
                  0.5 * g.box[0], 0.5 * g.box[1], 0.5 * g.box[2]) < r2;
}

// One stencil row of n candidates from tile index ub on against the lane's
// particle, appended to its list (live: 0 in lanes that only hold candidates
// for their quad).  The lanes of a quad have particles of one cell, and of
// one half of it, so that ub, n and K agree.  K4 = 4 K, m4K and mK: the
// divisors of div_small for 4 K and K; selfrow: the row holds the particle
// itself.  The decisions of 32 positions are formed first, a bit each, then
// the accepted ones are appended.  The exact test decides inside the guard
// band, as in scan_range; the band is wider (build_tile_nlist).  Positions
// past the row read the tile's arrays (or what follows them in LDS) and are
// masked out.
template <typename TS, typename OFF>
__device__ __forceinline__ void lane_row(const TS& t, const LaneTables& tab, const Compress& pack,
                                         const Grid& g, const double* __restrict__ x,
                                         const double* __restrict__ y,
                                         const double* __restrict__ z, double r2, int ub, int n,
                                         const LanePoint& pt, float guard, int mK, int m4K,
                                         bool selfrow, uint32_t live, ListOut<OFF>& out) {
  const int K = pt.K, k4 = 4 * K;
  const int nfull = div_small(n, m4K) * k4, rem = n - nfull;
  const uint32_t part = tab.valid[K - 1][rem];
  const int end = nfull + 4 * (rem < K ? rem : K);  // positions to look at
  int pself = -1;
  if (selfrow) {
    const int i = pt.self - ub, b = div_small(i, mK);  // i = b K + k
    pself = (b >> 2) * k4 + 4 * (i - b * K) + (b & 3);
  }
  const uint16_t* const pos = tab.pos[K - 1];
  const uint32_t mine = 4 * ub + (threadIdx.x & 3) * k4;  // the lane's candidate of a group
  for (int c0 = 0; __any(c0 < end); c0 += 32) {
    const uint4 grp = *(const uint4*)&tab.group[K - 1][c0 / 4];
    const uint32_t gw[4] = {grp.x, grp.y, grp.z, grp.w};
    uint32_t word = 0;
    float near[4];
    // 16 positions at a time, so that loads and products overlap
#pragma unroll
    for (int h = 1; h >= 0; --h) {
      near[2 * h] = near[2 * h + 1] = 3e38f;
      if (h == 0 || __any(c0 + 16 < end)) {
        float x[4], y[4], z[4], sq[4];
        f32x4 e[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const uint32_t w = gw[2 * h + b / 2], off = mine + (b & 1 ? w >> 16 : w & 0xffffu);
          x[b] = *(const float*)((const char*)t.x + off);
          y[b] = *(const float*)((const char*)t.y + off);
          z[b] = *(const float*)((const char*)t.z + off);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          sq[b] = __builtin_fmaf(z[b], z[b], __builtin_fmaf(y[b], y[b], x[b] * x[b]));
          e[b] = __builtin_amdgcn_mfma_f32_4x4x1f32(x[b], pt.ax, pt.c, 0, 0, 0);
        }
#pragma unroll
        for (int b = 0; b < 4; ++b) e[b] = __builtin_amdgcn_mfma_f32_4x4x1f32(y[b], pt.ay, e[b], 0, 0, 0);
#pragma unroll
        for (int b = 0; b < 4; ++b) e[b] = __builtin_amdgcn_mfma_f32_4x4x1f32(z[b], pt.az, e[b], 0, 0, 0);
#pragma unroll
        for (int b = 0; b < 4; ++b) e[b] = __builtin_amdgcn_mfma_f32_4x4x1f32(sq[b], 1.0f, e[b], 0, 0, 0);
#pragma unroll
        for (int b = 3; b >= 0; --b) {
#pragma unroll
          for (int j = 3; j >= 0; --j)
            word = __builtin_amdgcn_alignbit(word, __float_as_uint(e[b][j]), 31);
          float& n = near[2 * h + b / 2];
          n = fminf(fminf(n, __builtin_fabsf(e[b][0])), __builtin_fabsf(e[b][1]));
          n = fminf(fminf(n, __builtin_fabsf(e[b][2])), __builtin_fabsf(e[b][3]));
        }
      }
    }
    const int d = nfull - c0;  // positions of whole blocks in this word
    uint32_t valid = ~0u;
    if (d < 32) valid = d >= 0 ? ((1u << d) - 1u) | part << d : (d > -32 ? part >> -d : 0u);
    valid &= live;
    if (fminf(fminf(near[0], near[1]), fminf(near[2], near[3])) <= guard) {
      // the definition decides those inside the guard band
      uint32_t v = 0;
#pragma unroll
      for (int h = 0; h < 4; ++h) v |= near[h] <= guard ? 0xffu << (8 * h) : 0u;
      for (v &= valid; v; v &= v - 1) {
        const int b = __builtin_ctz(v);
        const int u = ub + (pos[c0 + b] >> kFullShift);
        const float dx = t.x[pt.self] - t.x[u], dy = t.y[pt.self] - t.y[u],
                    dz = t.z[pt.self] - t.z[u];
        const float e = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, __builtin_fmaf(dx, dx, -(float)r2)));
        if (!(__builtin_fabsf(e) <= guard + guard)) continue;
        const bool in = exact_pair(t, g, x, y, z, pt.slot, u, r2);
        word = (word & ~(1u << b)) | (in ? 1u << b : 0u);
      }
    }
    word &= valid;
    const int ps = pself - c0;
    if (ps >= 0 && ps < 32) word &= ~(1u << ps);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (!__any(word & (0xffffu << (16 * h)))) continue;
      uint32_t nib[4];
      uint2 sel[4];
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        nib[b] = (word >> (16 * h + 4 * b)) & 15u;
        sel[b] = pack.sel[nib[b]];
      }
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        // entries are byte offsets into the tile arrays, as the table's
        const uint32_t w = gw[2 * h + b / 2], off = 4 * ub + (b & 1 ? w >> 16 : w & 0xffffu);
        const uint32_t two = off << 16 | off;
        out.push4(nib[b], sel[b], two + ((uint32_t)k4 << 16), two + ((uint32_t)(3 * k4) << 16 | 2 * k4));
      }
    }
  }
}

// One wave per home cell (up to 16 per workgroup); at most 64 VGPRs so that
// two 1024-thread workgroups share a CU.  TS: the tile (full or half list).
//
// LANES: a lane per particle (lane_row) in every brick whose cells and rows
// the tables cover, else as without; blockIdx.y as for RW > 1.
//
// RW > 1 (small systems, full lists): blockIdx.y is the workgroup's part of
// the brick, `cells` home cells, and RW waves share a cell, each taking 9/RW
// of its stencil rows.  The waves first count what their rows accept, so
// that each knows where its rows' entries start in the list, and then scan
// again and store; the lists are the same, entry for entry, as those of one
// wave.  One wave's scan of all nine rows, a serial chain, is what such
// builds wait for: N = 1000 118 -> 22 us, N = 4096 73 -> 18 us, N = 32768
// 82 -> 42 us.
template <typename TS, bool HALF, bool A24, int RW, bool LANES>
__global__ __launch_bounds__(LANES ? kLaneThreads : 1024)
__attribute__((amdgpu_waves_per_eu(RW == 9 ? 4 : (LANES ? 6 : 8)))) void
k_build_tile_nlist(
    const double* __restrict__ x, const double* __restrict__ y, const double* __restrict__ z,
    const int32_t* __restrict__ cs, Grid g, double r2,
    float guard, TileList tl, uint32_t* __restrict__ flags, int32_t* __restrict__ maxcount,
    int cells) {
  __shared__ TS t;
  __shared__ int acnt[kBrickMax];
  __shared__ int rcnt[RW > 1 ? RW : 1][RW > 1 ? kBrickMax : 1];  // per row group
  __shared__ int tlow[kTileCells];  // per tile cell, its particles in the lower x half
  const int brick = brick_of_block(g);
  if (brick >= g.nbricks) return;
  // the workgroup's home cells (local indices within the brick) and slots
  constexpr bool kParts = RW > 1 || LANES;
  const int lc0 = kParts ? (int)blockIdx.y * cells : 0;
  const int lc1 = kParts && lc0 + cells < g.V ? lc0 + cells : g.V;
  const int s0 = cs[brick * g.V], s1 = cs[(brick + 1) * g.V];
  const int p0 = kParts ? cs[brick * g.V + lc0] : s0, p1 = kParts ? cs[brick * g.V + lc1] : s1;
  if (kParts && blockIdx.y && p0 == p1) return;  // part 0 leaves the tables
  const bool xh = !HALF && tl.xlow != nullptr;
  const int total = tile_cells(g, brick, cs, t, HALF, tl.xlow, xh ? tlow : nullptr);
  if (!HALF && tl.tab && blockIdx.y == 0)
    tile_tables_store(g, t, tl.tab + (int64_t)brick * kTabInts);
  const int nbrick = s1 - s0;
  if (threadIdx.x == 0 && (total > TS::kCap || nbrick > kBrickMax))
    atomicOr(flags, MDPL_FLAG_NL_OVERFLOW);
  for (int a = threadIdx.x; a < kBrickMax; a += blockDim.x) {
    acnt[a] = 0;
    if (RW > 1)
      for (int r = 0; r < RW; ++r) rcnt[r][a] = 0;
  }
  const double Lx = g.box[0], Ly = g.box[1], Lz = g.box[2];
  const int TX = g.B[0] + 2, TXY = TX * (g.B[1] + 2);
  const int ntc = TXY * (g.B[2] + 2);
  int bx, by, bz;
  brick_coords(g, brick, bx, by, bz);
  // the tile corner (one cell below the brick) and FP32 relative image positions
  const double ox = (double)(bx * g.B[0] - 1) * (Lx / g.nc[0]);
  const double oy = (double)(by * g.B[1] - 1) * (Ly / g.nc[1]);
  const double oz = (double)(bz * g.B[2] - 1) * (Lz / g.nc[2]);
  // with a lane per particle the tile's centre: the screen forms |x|^2
  const double half_tile = LANES ? 0.5 : 0.0;
  const double tx = ox + half_tile * ((g.B[0] + 2) * (Lx / g.nc[0]));
  const double ty = oy + half_tile * ((g.B[1] + 2) * (Ly / g.nc[1]));
  const double tz = oz + half_tile * ((g.B[2] + 2) * (Lz / g.nc[2]));
  auto near_tile = [](double v) {  // and finite, or far from everything
    const float f = (float)v;
    return !LANES || __builtin_fabsf(f) < kFarLane ? f : kFarLane;
  };
  tile_slot_cells(ntc, total, t);
  {
    const int nt = total < TS::kCap ? total : TS::kCap;
    if (threadIdx.x == 0) {
      t.x[TS::kDummy] = kFarF;
      t.y[TS::kDummy] = kFarF;
      t.z[TS::kDummy] = kFarF;
    }
    // (several slots per thread in flight where the workgroups are small)
#pragma unroll RW == 9 || LANES ? 4 : 1
    for (int u = threadIdx.x; u < nt; u += blockDim.x) {
      const int c = t.cell[u];
      const int src = t.src[c] + (u - t.prefix[c]);
      const int code = t.code[c];
      t.x[u] = near_tile((x[src] + (double)((code & 3) - 1) * Lx) - tx);
      t.y[u] = near_tile((y[src] + (double)(((code >> 2) & 3) - 1) * Ly) - ty);
      t.z[u] = near_tile((z[src] + (double)(((code >> 4) & 3) - 1) * Lz) - tz);
    }
    __syncthreads();
  }
  const int max_nb = tl.max_nb;
  uint16_t* __restrict__ half = (uint16_t*)tl.nbr;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6;
  const float r2lo = (float)(r2 - (double)guard), r2hi = (float)(r2 + (double)guard);
  // the scan of the rows [r0, r1) of cell lc's particles; counters: per particle of the brick
  auto scan_cell = [&](int lc, int r0, int r1, int* counters, auto count) {
    constexpr bool kCount = decltype(count)::value;
    const int lx = lc % g.B[0], ly = (lc / g.B[0]) % g.B[1], lz = lc / (g.B[0] * g.B[1]);
    // the last brick along an axis may be partial: its missing cells would
    // alias periodic images of another brick's cells
    if (bx * g.B[0] + lx >= g.nc[0] || by * g.B[1] + ly >= g.nc[1] || bz * g.B[2] + lz >= g.nc[2])
      return;
    const int tc0 = ((lz + 1) * (g.B[1] + 2) + (ly + 1)) * TX + (lx + 1);
    const int ncell = t.prefix[tc0 + 1] - t.prefix[tc0];
    const int slot0 = t.src[tc0];
    for (int a0 = 0; a0 < ncell; a0 += 64) {
      const int na = ncell - a0 < 64 ? ncell - a0 : 64;
      const int K = 64 / na;
      const int a = a0 + lane % na, k = lane / na;
      const bool active = k < K;
      const int self = t.prefix[tc0] + a;
      const int s = slot0 + a;          // sorted slot of particle a
      const int la = s - s0;            // its index within the brick
      const bool ok = active && self < TS::kCap && la >= 0 && la < kBrickMax && s < s1;
      RowScan q;
      q.xi = ok ? t.x[self] : 0.0f;
      q.yi = ok ? t.y[self] : 0.0f;
      q.zi = ok ? t.z[self] : 0.0f;
      q.r2lo = r2lo;
      q.r2hi = r2hi;
      q.xs = ok ? x[s] : 0.0;
      q.ys = ok ? y[s] : 0.0;
      q.zs = ok ? z[s] : 0.0;
      q.x = x;
      q.y = y;
      q.z = z;
      q.r2 = r2;
      q.Lx = Lx;
      q.Ly = Ly;
      q.Lz = Lz;
      q.hx = 0.5 * Lx;
      q.hy = 0.5 * Ly;
      q.hz = 0.5 * Lz;
      q.self = self;
      q.K = K;
      q.max_nb = max_nb;
      q.cnt = &counters[ok ? la : 0];
      q.base = half + (int64_t)(ok ? s : 0) * 4;
      q.stride4 = (uint32_t)(tl.stride * 4);
      q.pitch = (uint32_t)(tl.stride * 8);
      // a particle in the lower x half of its cell skips the upper half of
      // the next cell along x, one in the upper half the lower half of the
      // previous cell: more than a cell width, which exceeds the list
      // radius, away along x alone
      const bool lower = xh && a < tlow[tc0];
      const bool upper = xh && !lower;
      if (!ok) continue;
      int found = 0;
      for (int row = r0; row < r1; ++row) {
        // a stencil row: three consecutive tile cells, one contiguous index range
        const int roz = row / 3 - 1, roy = row % 3 - 1;
        const int tcl = tc0 + roz * TXY + roy * TX - 1;
        // half list: only tile indices past the particle's own (rows below it are empty)
        if (HALF && (roz < 0 || (roz == 0 && roy < 0))) continue;
        int ub = t.prefix[tcl] + (upper ? tlow[tcl] : 0);
        if (HALF && ub <= self) ub = self + 1;
        int ue = lower ? t.prefix[tcl + 2] + tlow[tcl + 2] : t.prefix[tcl + 3];
        ue = ue < TS::kCap ? ue : TS::kCap;
        found += scan_range<4, HALF ? kHalfShift : kFullShift, A24, kCount>(t, ub + k, ue, q);
      }
      if (kCount && found) atomicAdd(q.cnt, found);
    }
  };
  if constexpr (RW > 1) {
    const int lc = lc0 + wave / RW, r = wave % RW;  // one cell per RW waves (cells * RW waves)
    // A cell of 22 to 64 particles takes a lane each (K below is at most 2) and
    // a row's decisions fit registers, unless the row is very long
    RowScan q;
    RowBits bits;
    int row_ub = 0, row_la = -1;
    bool direct = false;
    if constexpr (RW == 9) {
      const int lx = lc % g.B[0], ly = (lc / g.B[0]) % g.B[1], lz = lc / (g.B[0] * g.B[1]);
      const int tc0 = ((lz + 1) * (g.B[1] + 2) + (ly + 1)) * TX + (lx + 1);
      const int na = lc < lc1 ? t.prefix[tc0 + 1] - t.prefix[tc0] : 0;
      if (na > 21 && na <= 64) {
        const int self = t.prefix[tc0] + lane, s = t.src[tc0] + lane;
        const bool ok = lane < na && self < TS::kCap && s - s0 >= 0 && s - s0 < kBrickMax && s < s1;
        const int tcl = tc0 + (r / 3 - 1) * TXY + (r % 3 - 1) * TX - 1;
        const bool lower = xh && lane < tlow[tc0], upper = xh && !lower;
        row_ub = t.prefix[tcl] + (upper ? tlow[tcl] : 0);
        int ue = lower ? t.prefix[tcl + 2] + tlow[tcl + 2] : t.prefix[tcl + 3];
        ue = ue < TS::kCap ? ue : TS::kCap;
        const int n = ok ? ue - row_ub : 0;
        direct = !__any(n > 32 * kRowWords);
        if (direct) {
          q.self = self;
          q.K = 64 / na;
          q.max_nb = max_nb;
          q.xi = ok ? t.x[self] : 0.0f;
          q.yi = ok ? t.y[self] : 0.0f;
          q.zi = ok ? t.z[self] : 0.0f;
          q.xs = ok ? x[s] : 0.0;
          q.ys = ok ? y[s] : 0.0;
          q.zs = ok ? z[s] : 0.0;
          q.x = x;
          q.y = y;
          q.z = z;
          q.r2 = r2;
          q.Lx = Lx;
          q.Ly = Ly;
          q.Lz = Lz;
          q.hx = 0.5 * Lx;
          q.hy = 0.5 * Ly;
          q.hz = 0.5 * Lz;
          q.base = half + (int64_t)(ok ? s : 0) * 4;
          q.pitch = (uint32_t)(tl.stride * 8);
          row_la = ok ? s - s0 : -1;
          const int found = row_bits(t, row_ub, n, q, (float)r2, guard, bits);
          if (ok) rcnt[r][row_la] = found;
        }
      }
    }
    if (!direct && lc < lc1)
      scan_cell(lc, 9 / RW * r, 9 / RW * (r + 1), rcnt[r], std::true_type());
    __syncthreads();
    // where each row group's entries start, and the particle's count
    for (int la = p0 - s0 + threadIdx.x; la < p1 - s0 && la < kBrickMax; la += blockDim.x) {
      int sum = 0;
      for (int q = 0; q < RW; ++q) {
        const int n = rcnt[q][la];
        rcnt[q][la] = sum;
        sum += n;
      }
      acnt[la] = sum;
    }
    __syncthreads();
    if (direct) {
      if (row_la >= 0) row_store(bits, row_ub, (uint32_t)rcnt[r][row_la], q);
    } else if (lc < lc1) {
      scan_cell(lc, 9 / RW * r, 9 / RW * (r + 1), rcnt[r], std::false_type());
    }
  } else {
    if constexpr (LANES) {
      // The particles of each cell's lower and upper half in quads of lanes
      // (acnt: tile cell, particle of the cell, and whether the lane only
      // fills its quad); every cell's K and rows must be within the tables.
      __shared__ __attribute__((aligned(16))) LaneTables tab;
      __shared__ Compress pack;
      __shared__ int quads[64], nlanes;
      if (threadIdx.x < 16) pack.sel[threadIdx.x] = kCompress.sel[threadIdx.x];
      for (int k = threadIdx.x; k < (int)(sizeof(LaneTables) / 16); k += blockDim.x)
        ((uint4*)&tab)[k] = ((const uint4*)&kLaneTables)[k];
      const int mB0 = 65536 / g.B[0] + 1, mB1 = 65536 / g.B[1] + 1;
      auto home_cell = [&](int lc) {  // tile cell, or -1 past the grid
        const int yz = div_small(lc, mB0), lz = div_small(yz, mB1);
        const int lx = lc - yz * g.B[0], ly = yz - lz * g.B[1];
        if (bx * g.B[0] + lx >= g.nc[0] || by * g.B[1] + ly >= g.nc[1] || bz * g.B[2] + lz >= g.nc[2])
          return -1;
        return ((lz + 1) * (g.B[1] + 2) + (ly + 1)) * TX + (lx + 1);
      };
      if (wave == 0) {
        const int tc = lane >= lc0 && lane < lc1 ? home_cell(lane) : -1;
        const int ncell = tc >= 0 ? t.prefix[tc + 1] - t.prefix[tc] : 0;
        const int low = xh && tc >= 0 ? tlow[tc] : 0;
        const int want = ((low + 3) & ~3) + ((ncell - low + 3) & ~3), upto = wave_scan_i32(want);
        quads[lane] = upto - want;
        if (lane == 63) nlanes = upto;
      }
      __syncthreads();
      const int T = nlanes;
      bool bad = nbrick > kBrickMax || total > TS::kCap || T > kBrickMax || g.V > 64;
      for (int lc = lc0 + wave; lc < lc1; lc += nwaves) {
        const int tc = home_cell(lc);
        if (tc < 0) continue;
        const int ncell = t.prefix[tc + 1] - t.prefix[tc];
        bad |= ncell > 64 || (ncell && ncell < (64 + kLaneK) / (kLaneK + 1));
        if (lane < 9 && ncell) {
          const int tcl = tc + (lane / 3 - 1) * TXY + (lane % 3 - 1) * TX - 1;
          bad |= t.prefix[tcl + 3] - t.prefix[tcl] > kListRow;
        }
        const int low = xh ? tlow[tc] : 0, plow = (low + 3) & ~3;
        for (int p = lane; p < plow + ((ncell - low + 3) & ~3); p += 64) {
          const int last = p < plow ? low - 1 : ncell - 1, a = p < plow ? p : low + p - plow;
          if (quads[lc] + p < kBrickMax)
            acnt[quads[lc] + p] = tc | (a < last ? a : last) << 8 | (a > last ? 1 : 0) << 24;
        }
      }
      if (!__syncthreads_or(bad)) {
        int most = 0;
        for (int l0 = 64 * wave; l0 < T; l0 += 64 * nwaves) {
          const bool has = l0 + lane < T;
          const int code = acnt[has ? l0 + lane : l0], tc0 = code & 255, a = (code >> 8) & 0xffff;
          const bool ok = has && !(code >> 24);
          const int first = t.prefix[tc0], na = t.prefix[tc0 + 1] - first;
          const int s = t.src[tc0] + a;
          LanePoint pt;
          // 64 / na: na is 8 to 64, and 64 / na at least 1 / 64 off the next integer
          pt.K = (int)(64.0f * __builtin_amdgcn_rcpf((float)na) + 0.001f);
          pt.self = first + a;
          pt.slot = s;
          const float px = t.x[pt.self], py = t.y[pt.self], pz = t.z[pt.self];
          pt.ax = -2.0f * px;
          pt.ay = -2.0f * py;
          pt.az = -2.0f * pz;
          const float c = (float)(((double)px * px + (double)py * py + (double)pz * pz) - r2);
          pt.c = f32x4{c, c, c, c};
          const bool lower = xh && a < tlow[tc0], upper = xh && !lower;
          const int mK = tab.over[pt.K - 1], m4K = tab.over4[pt.K - 1];
          typedef std::conditional_t<A24, uint32_t, uint64_t> Off;
          const Off pitch = (Off)tl.stride * 8;
          ListOut<Off> out{0, 0, (Off)s * 8, pitch, (Off)((max_nb + 3) >> 2) * pitch, (char*)half};
          for (int row = 0; row < 9; ++row) {
            const int tcl = tc0 + (row / 3 - 1) * TXY + (row % 3 - 1) * TX - 1;
            const int ub = t.prefix[tcl] + (upper ? tlow[tcl] : 0);
            const int ue = lower ? t.prefix[tcl + 2] + tlow[tcl + 2] : t.prefix[tcl + 3];
            lane_row(t, tab, pack, g, x, y, z, r2, ub, has ? ue - ub : 0, pt, guard, mK, m4K,
                     row == 4, ok ? ~0u : 0u, out);
          }
          if (ok) {
            const int m = out.finish((Off)s * 8, max_nb, (uint32_t)TS::kDummy << kFullShift);
            tl.cnt[s] = m < max_nb ? m : max_nb;
            if (m > max_nb) atomicOr(flags, MDPL_FLAG_NL_OVERFLOW);
            most = m > most ? m : most;
          }
        }
        most = wave_max_i32(most);
        if (lane == 0 && most > 0) atomicMax(maxcount, most);
        return;
      }
      for (int a = threadIdx.x; a < kBrickMax; a += blockDim.x) acnt[a] = 0;
      __syncthreads();
    }
    for (int lc = lc0 + wave; lc < lc1; lc += nwaves) scan_cell(lc, 0, 9, acnt, std::false_type());
  }
  __syncthreads();
  // every slot gets its count (zero past kBrickMax, flagged above)
  int most = 0;
  for (int s = p0 + threadIdx.x; s < p1; s += blockDim.x) {
    const int la = s - s0;
    const int count = la < kBrickMax ? acnt[la] : 0;
    const int kept = count < max_nb ? count : max_nb;
    for (int m = kept; m < ((kept + 3) & ~3); ++m)  // pad the last word
      half[((int64_t)(m >> 2) * tl.stride + s) * 4 + (m & 3)] =
          (uint16_t)(TS::kDummy << (HALF ? kHalfShift : kFullShift));
    tl.cnt[s] = kept;
    if (count > max_nb) atomicOr(flags, MDPL_FLAG_NL_OVERFLOW);
    most = count > most ? count : most;
  }
  most = wave_max_i32(most);
  if ((threadIdx.x & 63) == 0 && most > 0) atomicMax(maxcount, most);
}

hipError_t build_tile_nlist(const double* x, const double* y, const double* z,
                            const int32_t* cell_start, const Grid& g,
                            double r2, TileList tl, uint32_t* flags, int32_t* maxcount,
                            hipStream_t st) {
  const unsigned threads = g.V * 64 < 1024 ? (unsigned)g.V * 64 : 1024u;
  // guard band of the FP32 screen (see the derivation above k_build_tile_nlist)
  double span = 0.0;
  for (int k = 0; k < 3; ++k) {
    const double e = (double)(g.B[k] + 2) * (g.box[k] / g.nc[k]);
    span = e > span ? e : span;
  }
  const double u32 = 1.0 / 16777216.0;  // 2^-24
  const double rext = sqrt(r2);
  const double err = 2.0 * sqrt(3.0) * rext * u32 * (2.0 * span + 2.0 * rext) + 3.0 * u32 * r2;
  const float guard = (float)(8.0 * err);
  const dim3 grid(tile_grid(g));
  if (tl.half) {
    hipLaunchKernelGGL((k_build_tile_nlist<TileHalf32, true, false, 1, false>), grid, dim3(threads), 0, st,
                       x, y, z, cell_start, g, r2, guard, tl, flags, maxcount, g.V);
    return hipGetLastError();
  }
  // few bricks: the cells of a brick shared by several workgroups, the rows
  // of a cell by 9 or 3 waves (as many as a workgroup holds)
  int parts = brick_parts(g, kBuildWant, g.V);
  const int cells = (int)div_up(g.V, parts);
  parts = (int)div_up(g.V, cells);
  const int rw = cells * 9 <= 16 ? 9 : (cells * 3 <= 16 ? 3 : 1);
  const bool a24 = tl.stride * 8 < (int64_t)(1 << 24);
  // a lane per particle where cells hold enough of them, but not over 64
  // (those of a full brick; the stride is the padded number of all): waves
  // for its quads, but at most 8, so that two workgroups share a CU evenly
  // (N = 10^6: 5 waves 330 us, 7 316, 8 305, 9 353, 12 337).  Few bricks are
  // shared here too: whole builds with the sort, N = 64000 (128 bricks of 3^3
  // cells) 82 -> 68 us, but two parts of 208 such bricks 82 -> 90; N = 42875 at
  // list radius 3.3 (216 of 2^3) 104 -> 82 us in two parts, 113 with three
  // waves per cell, which stay ahead for 3^3 bricks (N = 32768 55 against 62).
  const int64_t full = tl.stride * g.V / ((int64_t)g.nc[0] * g.nc[1] * g.nc[2]);
  const bool small_bricks = g.V <= 8;
  unsigned lane_threads = 0;
  int lane_cells = g.V, lane_parts = 1;
  // (and lengths whose squares are far from those of kFarLane and of FP32's least)
  const bool lengths = span < 0x1p36 && rext > 0x1p-36;
  if (lengths && full >= 10 * (int64_t)g.V && full <= 48 * (int64_t)g.V) {
    lane_cells = (int)div_up(g.V, brick_parts(g, small_bricks ? kBuildWant : kBuildWant / 2, g.V));
    lane_parts = (int)div_up(g.V, lane_cells);
    lane_threads = (unsigned)div_up(full * 6 / 5 * lane_cells / g.V, 64) * 64;
    lane_threads = lane_threads < 256 ? 256 : (lane_threads > kLaneThreads ? kLaneThreads : lane_threads);
  }
  // its screen on the matrix cores: with coordinates up to span / 2 from the
  // tile's centre, |x|^2 <= 3 span^2 / 4, the squares are within 3 and 4 ulp
  // of it, and each of four accumulations of terms below 6 span^2 / 4 rounds
  // (2 ulp allowed): 17.3 span^2 2^-24 on top of err
  const float lane_guard = (float)(8.0 * err + 2.0 * 17.3 * span * span * u32);
  // A lane's offsets: 64 bits cost a build of 1.5 * 10^6 particles 458 -> 471 us,
  // numbering the words in 32 bits 468 (and one of 10^6 325 -> 332).
  if (a24 && parts > 1 && rw == 9)
    hipLaunchKernelGGL((k_build_tile_nlist<TileShared32, false, true, 9, false>), dim3(grid.x, parts),
                       dim3(cells * 9 * 64), 0, st, x, y, z, cell_start, g, r2, guard, tl,
                       flags, maxcount, cells);
  else if (a24 && parts > 1 && rw == 3 && !(lane_threads && small_bricks))
    hipLaunchKernelGGL((k_build_tile_nlist<TileShared32, false, true, 3, false>), dim3(grid.x, parts),
                       dim3(cells * 3 * 64), 0, st, x, y, z, cell_start, g, r2, guard, tl,
                       flags, maxcount, cells);
  else if (lane_threads && list_offsets_32(tl.stride * 8))
    hipLaunchKernelGGL((k_build_tile_nlist<TileShared32, false, true, 1, true>), dim3(grid.x, lane_parts),
                       dim3(lane_threads), 0, st, x, y, z, cell_start, g, r2, lane_guard, tl, flags,
                       maxcount, lane_cells);
  else if (lane_threads)
    hipLaunchKernelGGL((k_build_tile_nlist<TileShared32, false, false, 1, true>), dim3(grid.x, lane_parts),
                       dim3(lane_threads), 0, st, x, y, z, cell_start, g, r2, lane_guard, tl, flags,
                       maxcount, lane_cells);
  else if (a24)
    hipLaunchKernelGGL((k_build_tile_nlist<TileShared32, false, true, 1, false>), grid,
                       dim3(threads), 0, st, x, y, z, cell_start, g, r2, guard, tl, flags,
                       maxcount, g.V);
  else
    hipLaunchKernelGGL((k_build_tile_nlist<TileShared32, false, false, 1, false>), grid,
                       dim3(threads), 0, st, x, y, z, cell_start, g, r2, guard, tl, flags,
                       maxcount, g.V);
  return hipGetLastError();
}

// Directed pairs in the caller's indices: entry m of slot s goes to
// offsets[s] + m; the tile index is mapped back to its sorted slot.
__global__ __launch_bounds__(1024) void k_export_tile_pairs(
    TileList tl, const int32_t* __restrict__ cs, Grid g, const int32_t* __restrict__ perm,
    const int32_t* __restrict__ offsets, int32_t* __restrict__ i_out, int32_t* __restrict__ j_out,
    int64_t cap) {
  __shared__ TileCells t;
  const int brick = brick_of_block(g);
  if (brick >= g.nbricks) return;
  tile_cells(g, brick, cs, t, tl.half != 0);
  const int ntc = (g.B[0] + 2) * (g.B[1] + 2) * (g.B[2] + 2);
  const int s0 = cs[brick * g.V], s1 = cs[(brick + 1) * g.V];
  for (int s = s0 + (int)threadIdx.x; s < s1; s += blockDim.x) {
    const int c = tl.cnt[s];
    const int64_t o = offsets[s];
    const int32_t pi = perm[s];
    for (int m = 0; m < c; ++m) {
      if (o + m >= cap) break;
      const int u = (int)((tl.nbr[(int64_t)(m >> 2) * tl.stride + s] >> (16 * (m & 3))) & 0xffff) >>
                    (tl.half ? kHalfShift : kFullShift);
      const int lo = tile_cell_of(t, ntc, u);
      i_out[o + m] = pi;
      j_out[o + m] = perm[t.src[lo] + (u - t.prefix[lo])];
    }
  }
}

hipError_t export_tile_pairs(const TileList& tl, const int32_t* cell_start, const Grid& g,
                             const int32_t* perm, const int32_t* offsets, int32_t* i_out,
                             int32_t* j_out, int64_t cap, hipStream_t st) {
  hipLaunchKernelGGL(k_export_tile_pairs, dim3(tile_grid(g)), dim3(tl.threads), 0,
                     st, tl, cell_start, g, perm, offsets, i_out, j_out, cap);
  return hipGetLastError();
}

}  // namespace mdpl
