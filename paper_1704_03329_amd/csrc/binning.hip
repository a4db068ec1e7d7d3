// Cell binning (Sec. 3.5: every particle belongs to exactly one cell of side
// >= the list radius) by counting sort, and the moves of the particles into
// the sorted order.
//
// The particles of a cell are counted with one atomic per run of equal keys
// in a wave, placed behind their cell's start in order of arrival, and each
// then finds its final place by counting the smaller values in its cell (the
// lower half of the cell along x first where the list build wants that, then
// the caller's order), so that the result is deterministic and independent of
// the arrival.  Systems of up to kSmallN particles do all of it in one
// workgroup and one launch.  Grids with many more cells than particles use a
// stable LSD radix sort of the keys instead, whose cost does not grow with
// the cells.
#include <math.h>

#include "device_util.h"
#include "internal.h"

namespace mdpl {

mdpl_status make_grid(const double box[3], double r, const int brick[3], Grid* g) {
  g->nbricks = 1;
  g->order = nullptr;
  g->norder = 0;
  for (int k = 0; k < 3; ++k) {
    double side_min = r * (1.0 + 1e-10);
    double q = floor(box[k] / side_min);
    if (!(q >= 3.0)) return MDPL_EBOX;
    if (q > 4096.0) q = 4096.0;
    g->nc[k] = (int)q;
    g->inv_side[k] = q / box[k];
    g->side[k] = box[k] / q;
    g->box[k] = box[k];
    int b = brick[k] < 1 ? 1 : brick[k];
    if (b > g->nc[k]) b = g->nc[k];
    g->B[k] = b;
    g->nb[k] = (g->nc[k] + b - 1) / b;
    g->nbricks *= g->nb[k];
  }
  g->V = g->B[0] * g->B[1] * g->B[2];
  const long long nk = (long long)g->nbricks * g->V;
  if (nk > (1ll << 30)) return MDPL_EBOX;
  g->nkeys = (int)nk;
  return MDPL_OK;
}

size_t sort_bytes(int64_t n) {
  int64_t ntiles = div_up(n, kSortTile);
  int64_t hist = (int64_t)kRadixBins * ntiles + 1;
  int64_t bs = div_up(hist > n ? hist : n, 1024) + 2;
  return 4 * align256(4 * (size_t)n) + align256(4 * (size_t)hist) + align256(4 * (size_t)bs);
}

void sort_carve(char*& p, int64_t n, SortBufs* s) {
  int64_t ntiles = div_up(n, kSortTile);
  int64_t hist = (int64_t)kRadixBins * ntiles + 1;
  int64_t bs = div_up(hist > n ? hist : n, 1024) + 2;
  for (int b = 0; b < 2; ++b) {
    s->keys[b] = (int32_t*)p;
    p += align256(4 * (size_t)n);
    s->vals[b] = (int32_t*)p;
    p += align256(4 * (size_t)n);
  }
  s->hist = (int32_t*)p;
  p += align256(4 * (size_t)hist);
  s->blocksums = (int32_t*)p;
  p += align256(4 * (size_t)bs);
  s->n = n;
  s->ntiles = (int)ntiles;
}

// Cell index along one axis; a non-finite coordinate lands in cell 0.
__device__ __forceinline__ int cell_coord(double x, double L, double inv_side, int nc) {
  const double q = fold(x, L) * inv_side;
  if (q >= 0.0 && q < (double)nc) return (int)q;
  return q >= (double)nc ? nc - 1 : 0;
}

// Cell key of a particle; upper (xbit only): the upper half of its cell along
// x, decided on the quotient that gave the cell index.
__device__ __forceinline__ int cell_of(double x, double y, double z, const Grid& g, bool xbit,
                                       bool& upper) {
  const int cx = cell_coord(x, g.box[0], g.inv_side[0], g.nc[0]);
  upper = xbit && !(fold(x, g.box[0]) * g.inv_side[0] - (double)cx < 0.5);
  return cell_key(g, cx, cell_coord(y, g.box[1], g.inv_side[1], g.nc[1]),
                  cell_coord(z, g.box[2], g.inv_side[2], g.nc[2]));
}

// The particles of each cell in two runs, the lower half of the cell along x
// first (each run in sorted order, so the order stays deterministic), and
// the length of the first run.  The half comes with each sorted value (its
// top bit, set by k_cell_keys for the upper half).  A group of 16 lanes per
// cell, a particle per lane (16 at a time), four cells per wave.
constexpr int kPartLanes = 16;
__global__ __launch_bounds__(256) void k_xhalf_partition(const int32_t* __restrict__ cs, int nkeys,
                                                         const int32_t* __restrict__ vin,
                                                         int32_t* __restrict__ vout,
                                                         int32_t* __restrict__ xlow) {
  const int c = (int)((blockIdx.x * blockDim.x + threadIdx.x) / kPartLanes);
  if (c >= nkeys) return;
  const int lane = (int)threadIdx.x & 63, sub = lane % kPartLanes;
  const unsigned long long group = ((1ull << kPartLanes) - 1) << (lane - sub);
  const unsigned long long below = ((1ull << lane) - 1) & group;
  const int b = cs[c], e = cs[c + 1];
  int lo = 0;  // the cell's lower-half particles
  for (int s0 = b; s0 < e; s0 += kPartLanes) {
    const bool has = s0 + sub < e;
    lo += __popcll(__ballot(has && vin[has ? s0 + sub : b] >= 0) & group);
  }
  if (sub == 0) xlow[c] = lo;
  int nl = 0, nu = 0;  // placed so far
  for (int s0 = b; s0 < e; s0 += kPartLanes) {
    const bool has = s0 + sub < e;
    const int v = has ? vin[s0 + sub] : 0;
    const bool low = has && v >= 0;
    const unsigned long long ml = __ballot(low) & group, mu = __ballot(has && !low) & group;
    if (has)
      vout[low ? b + nl + __popcll(ml & below) : b + lo + nu + __popcll(mu & below)] =
          v & 0x7fffffff;
    nl += __popcll(ml);
    nu += __popcll(mu);
  }
}

__global__ void k_cell_keys(const double* __restrict__ x, const double* __restrict__ y,
                            const double* __restrict__ z, int64_t n, Grid g,
                            int32_t* __restrict__ keys, int32_t* __restrict__ vals, int xbit,
                            int32_t* __restrict__ clear) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (clear && i < 16) clear[i] = 0;
  if (i >= n) return;
  bool upper;
  keys[i] = cell_of(x[i], y[i], z[i], g, xbit != 0, upper);
  vals[i] = (int32_t)((uint32_t)i | (upper ? 0x80000000u : 0u));
}

__global__ __launch_bounds__(kSortThreads) void k_radix_hist(const int32_t* __restrict__ keys,
                                                             int64_t n, int shift, int ntiles,
                                                             int32_t* __restrict__ hist) {
  __shared__ int h[kRadixBins];
  const int tid = threadIdx.x;
  h[tid] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * kSortTile;
#pragma unroll
  for (int k = 0; k < kSortItems; ++k) {
    int64_t idx = base + k * kSortThreads + tid;
    if (idx < n) atomicAdd(&h[(keys[idx] >> shift) & (kRadixBins - 1)], 1);
  }
  __syncthreads();
  hist[(int64_t)tid * ntiles + blockIdx.x] = h[tid];
}

// offs: the histogram scanned within blocks of 1024 counters, sums: the
// exclusive prefix of those blocks (the two halves of an exclusive scan).
__global__ __launch_bounds__(kSortThreads) void k_radix_scatter(
    const int32_t* __restrict__ kin, const int32_t* __restrict__ vin, int64_t n, int shift,
    int ntiles, const int32_t* __restrict__ offs, const int32_t* __restrict__ sums,
    int32_t* __restrict__ kout, int32_t* __restrict__ vout) {
  constexpr int kWaves = kSortThreads / 64;
  __shared__ int run[kRadixBins];
  __shared__ int wc[kWaves][kRadixBins];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const unsigned long long below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  const int64_t hi = (int64_t)tid * ntiles + blockIdx.x;
  run[tid] = offs[hi] + sums[hi >> 10];
  const int64_t base = (int64_t)blockIdx.x * kSortTile;
  for (int r = 0; r < kSortItems; ++r) {
#pragma unroll
    for (int w = 0; w < kWaves; ++w) wc[w][tid] = 0;
    __syncthreads();
    const int64_t idx = base + r * kSortThreads + tid;
    const bool valid = idx < n;
    const int key = valid ? kin[idx] : 0;
    const int d = (key >> shift) & (kRadixBins - 1);
    unsigned long long peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < kRadixBits; ++b) {
      const bool bit = (d >> b) & 1;
      const unsigned long long m = __ballot(bit);
      peers &= bit ? m : ~m;
    }
    const int rank = __popcll(peers & below);
    if (valid && rank == 0) wc[wave][d] = __popcll(peers);
    __syncthreads();
    if (valid) {
      int pos = run[d] + rank;
      for (int w = 0; w < wave; ++w) pos += wc[w][d];
      kout[pos] = key;
      vout[pos] = vin[idx];
    }
    __syncthreads();
    int add = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) add += wc[w][tid];
    run[tid] += add;
  }
}

__global__ void k_cell_start(const int32_t* __restrict__ skeys, int64_t n, int ncells,
                             int32_t* __restrict__ cs) {
  int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n) return;
  const int k = skeys[s];
  const int prev = s > 0 ? skeys[s - 1] : -1;
  for (int c = prev + 1; c <= k; ++c) cs[c] = (int32_t)s;
  if (s == n - 1)
    for (int c = k + 1; c <= ncells; ++c) cs[c] = (int32_t)n;
}

// ----------------------------------------------------------------- scan
// Block of 256 threads scans 1024 consecutive values.
__global__ __launch_bounds__(256) void k_scan_blocks(const int32_t* in,
                                                     int32_t* out, int64_t n,
                                                     int32_t* __restrict__ sums) {
  __shared__ int wsum[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t base = (int64_t)blockIdx.x * 1024 + tid * 4;
  int v[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = (base + k < n) ? in[base + k] : 0;
  int t = v[0] + v[1] + v[2] + v[3];
  // inclusive wave scan of t
  int incl = t;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    int o = __shfl_up(incl, off, 64);
    if (lane >= off) incl += o;
  }
  if (lane == 63) wsum[wave] = incl;
  __syncthreads();
  int wbase = 0;
  for (int w = 0; w < wave; ++w) wbase += wsum[w];
  int run = wbase + incl - t;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (base + k < n) out[base + k] = run;
    run += v[k];
  }
  if (tid == 255) sums[blockIdx.x] = wbase + incl;
}

// One block: exclusive scan of the block sums in place (any length), total
// to sums[nb].
__global__ __launch_bounds__(1024) void k_scan_sums(int32_t* __restrict__ sums, int64_t nb) {
  __shared__ int wsum[16];
  __shared__ int carry;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid == 0) carry = 0;
  __syncthreads();
  for (int64_t base = 0; base < nb; base += 1024) {
    const int64_t i = base + tid;
    const int t = i < nb ? sums[i] : 0;
    int incl = t;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      int o = __shfl_up(incl, off, 64);
      if (lane >= off) incl += o;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int wbase = carry;
    for (int w = 0; w < wave; ++w) wbase += wsum[w];
    if (i < nb) sums[i] = wbase + incl - t;
    __syncthreads();
    if (tid == 1023) carry = wbase + incl;
    __syncthreads();
  }
  if (tid == 0) sums[nb] = carry;
}

// The whole exclusive scan of up to 16 C x 256 values, in place, by one
// workgroup: each wave holds its consecutive piece in registers, C loads of
// four values per lane in flight at once.  Against the three launches of the
// general scan 14 -> 7.6 us at 59,320 cells.
constexpr int kScanOneMost = 65536;
template <int C>
__global__ __launch_bounds__(1024) void k_scan_one(int32_t* __restrict__ a, int n) {
  __shared__ int wsum[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int base = wave * C * 256 + lane * 4;
  int4 v[C];
  int total = 0;
#pragma unroll
  for (int k = 0; k < C; ++k) {
    const int i = base + k * 256;
    if (i + 3 < n) {
      v[k] = *(const int4*)(a + i);
    } else {
      v[k].x = i < n ? a[i] : 0;
      v[k].y = i + 1 < n ? a[i + 1] : 0;
      v[k].z = i + 2 < n ? a[i + 2] : 0;
      v[k].w = 0;
    }
  }
#pragma unroll
  for (int k = 0; k < C; ++k) total += v[k].x + v[k].y + v[k].z + v[k].w;
  total = wave_sum_i32(total);
  if (lane == 0) wsum[wave] = total;
  __syncthreads();
  int run = 0;
  for (int w = 0; w < wave; ++w) run += wsum[w];
#pragma unroll
  for (int k = 0; k < C; ++k) {
    const int t = v[k].x + v[k].y + v[k].z + v[k].w;
    const int incl = wave_scan_i32(t);
    int4 o;
    o.x = run + incl - t;
    o.y = o.x + v[k].x;
    o.z = o.y + v[k].y;
    o.w = o.z + v[k].z;
    const int i = base + k * 256;
    if (i + 3 < n) {
      *(int4*)(a + i) = o;
    } else {
      if (i < n) a[i] = o.x;
      if (i + 1 < n) a[i + 1] = o.y;
      if (i + 2 < n) a[i + 2] = o.z;
    }
    run += __builtin_amdgcn_readlane(incl, 63);
  }
}

__global__ __launch_bounds__(256) void k_scan_add(int32_t* __restrict__ out, int64_t n,
                                                  const int32_t* __restrict__ sums,
                                                  int write_total) {
  const int64_t base = (int64_t)blockIdx.x * 1024 + threadIdx.x * 4;
  const int add = sums[blockIdx.x];
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (base + k < n) out[base + k] += add;
  if (write_total && blockIdx.x == 0 && threadIdx.x == 0) {
    const int64_t nb = (n + 1023) / 1024;
    out[n] = sums[nb];
  }
}

hipError_t exclusive_scan(const int32_t* in, int32_t* out, int64_t n, int32_t* blocksums,
                          bool write_total, hipStream_t st) {
  const int64_t nb = div_up(n, 1024);
  hipLaunchKernelGGL(k_scan_blocks, dim3((unsigned)nb), dim3(256), 0, st, in, out, n, blocksums);
  hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(1024), 0, st, blocksums, nb);
  hipLaunchKernelGGL(k_scan_add, dim3((unsigned)nb), dim3(256), 0, st, out, n, blocksums,
                     write_total ? 1 : 0);
  return hipGetLastError();
}

// The radix path (sparse grids).
static hipError_t radix_bin(const double* x, const double* y, const double* z, int64_t n,
                            const Grid& g, SortBufs& s, int32_t* cell_start, int32_t** keys_out,
                            int32_t** vals_out, hipStream_t st, int32_t* xlow, int32_t* clear) {
  const unsigned nb = (unsigned)div_up(n, 256);
  hipLaunchKernelGGL(k_cell_keys, dim3(nb), dim3(256), 0, st, x, y, z, n, g, s.keys[0], s.vals[0],
                     xlow ? 1 : 0, clear);
  int bits = 1;
  while ((1ll << bits) < (long long)g.nkeys) ++bits;
  const int passes = (bits + kRadixBits - 1) / kRadixBits;
  int cur = 0;
  const int64_t hn = (int64_t)kRadixBins * s.ntiles;
  for (int p = 0; p < passes; ++p) {
    const int shift = p * kRadixBits;
    hipLaunchKernelGGL(k_radix_hist, dim3(s.ntiles), dim3(kSortThreads), 0, st, s.keys[cur], n,
                       shift, s.ntiles, s.hist);
    // the scan's final add is left to the scatter (one launch fewer per pass)
    const int64_t nsb = div_up(hn, 1024);
    hipLaunchKernelGGL(k_scan_blocks, dim3((unsigned)nsb), dim3(256), 0, st, s.hist, s.hist, hn,
                       s.blocksums);
    hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(1024), 0, st, s.blocksums, nsb);
    hipLaunchKernelGGL(k_radix_scatter, dim3(s.ntiles), dim3(kSortThreads), 0, st, s.keys[cur],
                       s.vals[cur], n, shift, s.ntiles, s.hist, s.blocksums, s.keys[cur ^ 1],
                       s.vals[cur ^ 1]);
    cur ^= 1;
  }
  hipLaunchKernelGGL(k_cell_start, dim3(nb), dim3(256), 0, st, s.keys[cur], n, g.nkeys,
                     cell_start);
  *keys_out = s.keys[cur];
  *vals_out = s.vals[cur];
  if (xlow) {
    hipLaunchKernelGGL(k_xhalf_partition, dim3((unsigned)div_up((int64_t)g.nkeys * kPartLanes, 256)), dim3(256), 0, st,
                       cell_start, g.nkeys, s.vals[cur], s.vals[cur ^ 1], xlow);
    *vals_out = s.vals[cur ^ 1];
  }
  return hipGetLastError();
}

// ------------------------------------------------------- counting sort
// Squared displacement of particle i since the last list build (a
// non-finite one counts as 1e300).
__device__ __forceinline__ double moved2(const MoveCheck& c, int64_t i) {
  const double a = c.x[i] - c.xb[i], b = c.y[i] - c.yb[i], e = c.z[i] - c.zb[i];
  const double d = a * a + b * b + e * e;
  return d < 1e300 ? d : 1e300;
}
__device__ __forceinline__ void skin_result(const MoveCheck& c, double m2) {
  const double d = sqrt(m2);
  if (d > *c.max_disp) *c.max_disp = d;
  if (d >= c.half_skin) atomicOr(c.flags, MDPL_FLAG_SKIN);
}

__global__ __launch_bounds__(256) void k_zero_cells(int32_t* __restrict__ cs, int nkeys,
                                                    int32_t* __restrict__ xlow,
                                                    int32_t* __restrict__ clear) {
  const int i = (int)(blockIdx.x * 256 + threadIdx.x);
  if (clear && i < 16) clear[i] = 0;
  if (i > nkeys) return;
  cs[i] = 0;
  if (xlow) xlow[i] = 0;
}

// keys[i] = cell, ranks[i] = arrival rank in the cell (top bit: upper x
// half).  Runs of equal keys in a wave share one atomic: the particles of a
// run that continues arrive nearly sorted.
__global__ __launch_bounds__(256) void k_count_cells(const double* __restrict__ x,
                                                     const double* __restrict__ y,
                                                     const double* __restrict__ z, int64_t n,
                                                     Grid g, int xbit, int32_t* __restrict__ cs,
                                                     int32_t* __restrict__ keys,
                                                     uint32_t* __restrict__ ranks, MoveCheck mc) {
  __shared__ double sh[4];
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int lane = threadIdx.x & 63;
  const bool has = i < n;
  bool upper = false;
  const int key = has ? cell_of(x[i], y[i], z[i], g, xbit != 0, upper) : -1;
  const int before = __shfl_up(key, 1, 64);
  const uint64_t heads = __ballot(lane == 0 || key != before);
  const uint64_t upto = ~0ull >> (63 - lane);
  const int head = 63 - __builtin_clzll(heads & upto);
  const uint64_t after = heads & ~upto;
  int base = 0;
  if (has && lane == head)
    base = atomicAdd(&cs[key], (after ? __builtin_ctzll(after) : 64) - lane);
  base = __shfl(base, head, 64);
  if (has) {
    keys[i] = key;
    ranks[i] = (uint32_t)(base + lane - head) | (upper ? 0x80000000u : 0u);
  }
  if (mc.part) {
    const double m = block_max256(has ? moved2(mc, i) : 0.0, sh);
    if (threadIdx.x == 0) mc.part[blockIdx.x] = m;
  }
}

// Value (index, top bit: upper x half) and key of every particle to its
// cell, in order of arrival.
__global__ __launch_bounds__(256) void k_place_cells(const int32_t* __restrict__ cs,
                                                     const int32_t* __restrict__ keys,
                                                     const uint32_t* __restrict__ ranks, int64_t n,
                                                     uint32_t* __restrict__ tv,
                                                     int32_t* __restrict__ tk) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int key = keys[i];
  const uint32_t r = ranks[i];
  const int32_t s = cs[key] + (int32_t)(r & 0x7fffffffu);
  tv[s] = (uint32_t)i | (r & 0x80000000u);
  tk[s] = key;
}

// Number of values below v among p[b .. e), and of those in the upper half.
template <typename P>
__device__ __forceinline__ int place_in_cell(const P* p, int b, int e, uint32_t v, int& upper) {
  int r = 0, up = 0;
#pragma unroll 4
  for (int t = b; t < e; ++t) {
    const uint32_t w = p[t];
    r += w < v ? 1 : 0;
    up += (int)(w >> 31);
  }
  upper = up;
  return r;
}

// The values of a crowded cell in ascending order, by one workgroup: a stable
// radix sort of [b, e) between tv and tmp, whose part [b, e) only this cell
// uses.  bits: of the largest index; the upper-half bit counts as the next
// one.  Returns the array that holds the result.
constexpr int kOrderThreads = 256;
__device__ inline uint32_t* order_crowded(uint32_t* tv, uint32_t* tmp, int b, int e, int bits) {
  constexpr int kWaves = kOrderThreads / 64, kLoads = 4;
  __shared__ int run[kRadixBins];
  __shared__ int wc[kWaves][kRadixBins];
  static_assert(kRadixBins == kOrderThreads, "a thread per bin");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint64_t below = (1ull << lane) - 1;
  uint32_t *in = tv + b, *out = tmp + b;
  const int m = e - b;
  for (int shift = 0; shift <= bits; shift += kRadixBits) {
    auto digit = [&](uint32_t v) {
      return (int)(((v & 0x7fffffffu) | (v >> 31) << bits) >> shift) & (kRadixBins - 1);
    };
    run[tid] = 0;
    __syncthreads();
#pragma unroll 4
    for (int k = tid; k < m; k += kOrderThreads) atomicAdd(&run[digit(in[k])], 1);
    __syncthreads();
    // the bins' first places
    const int mine = run[tid], incl = wave_scan_i32(mine);
    if (lane == 63) wc[0][wave] = incl;
    __syncthreads();
    int first = incl - mine;
    for (int w = 0; w < wave; ++w) first += wc[0][w];
    __syncthreads();
    run[tid] = first;
    for (int k0 = 0; k0 < m; k0 += kLoads * kOrderThreads) {
      uint32_t v[kLoads];
#pragma unroll
      for (int j = 0; j < kLoads; ++j) {
        const int k = k0 + j * kOrderThreads + tid;
        v[j] = k < m ? in[k] : 0;
      }
#pragma unroll 1
      for (int j = k0; j < m && j < k0 + kLoads * kOrderThreads; j += kOrderThreads) {
#pragma unroll
        for (int w = 0; w < kWaves; ++w) wc[w][tid] = 0;
        __syncthreads();
        const bool has = j + tid < m;
        const uint32_t val = v[0];
#pragma unroll
        for (int q = 1; q < kLoads; ++q) v[q - 1] = v[q];
        const int d = digit(val);
        uint64_t peers = __ballot(has);
#pragma unroll 1
        for (int q = 0; q < kRadixBits; ++q) {
          const bool bit = (d >> q) & 1;
          const uint64_t set = __ballot(bit);
          peers &= bit ? set : ~set;
        }
        const int rank = __popcll(peers & below);
        if (has && rank == 0) wc[wave][d] = __popcll(peers);
        __syncthreads();
        if (has) {
          int at = run[d] + rank;
          for (int w = 0; w < wave; ++w) at += wc[w][d];
          out[at] = val;
        }
        __syncthreads();
        int add = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) add += wc[w][tid];
        run[tid] += add;
      }
    }
    __syncthreads();  // orders the workgroup's stores before its next loads
    uint32_t* const t = in;
    in = out;
    out = t;
  }
  return in - b;
}

// Final places, keys, values and the move of every particle.  A cell of more
// than kOrderMost particles (far beyond any tile), where counting smaller
// values would take too long, is sorted as a whole by the workgroup in whose
// 256 slots it begins: whole builds of 10^6 particles in one cell 28.6 ms, of
// 10^5 7.9 ms (11.0 and 6.3 in the order of arrival, which differs from run
// to run; one wave instead 61 and 10.8).
constexpr int kOrderMost = 4096;
template <typename Move>
__global__ __launch_bounds__(kOrderThreads) __attribute__((amdgpu_waves_per_eu(8)))
void k_order_cells(const int32_t* __restrict__ cs, uint32_t* tv, uint32_t* tmp,
                   const int32_t* __restrict__ tk, int64_t n, int bits,
                   int32_t* __restrict__ xlow, int32_t* __restrict__ keys_out, Move move,
                   MoveCheck mc, int nparts) {
  __shared__ double sh[4];
  if (mc.part && blockIdx.x == 0) {
    double v = 0.0;
    for (int k = threadIdx.x; k < nparts; k += kOrderThreads) v = mc.part[k] > v ? mc.part[k] : v;
    v = block_max256(v, sh);
    if (threadIdx.x == 0) skin_result(mc, v);
  }
  const int64_t s0 = (int64_t)blockIdx.x * kOrderThreads, s = s0 + threadIdx.x;
  if (s < n) {
    const uint32_t v = tv[s];
    const int key = tk[s];
    const int b = cs[key], e = cs[key + 1];
    if (e - b <= kOrderMost) {
      int upper;
      const int r = place_in_cell(tv, b, e, v, upper);
      if (xlow && r == 0) xlow[key] = e - b - upper;
      if (keys_out) keys_out[b + r] = key;
      move((int64_t)b + r, (int32_t)(v & 0x7fffffffu));
    }
  }
  // a crowded cell that begins here is the one of the last slot
  const int key = tk[s0 + kOrderThreads < n ? s0 + kOrderThreads - 1 : n - 1];
  const int b = cs[key], e = cs[key + 1];
  if (e - b <= kOrderMost || b < s0) return;
  const uint32_t* const sorted = order_crowded(tv, tmp, b, e, bits);
  for (int t = b + (int)threadIdx.x; t < e; t += kOrderThreads) {
    const uint32_t v = sorted[t];  // (before the move: tmp may be what it writes)
    if (xlow) {
      if (v >> 31 && (t == b || !(sorted[t - 1] >> 31))) xlow[key] = t - b;
      if (t == e - 1 && !(v >> 31)) xlow[key] = e - b;
    }
    if (keys_out) keys_out[t] = key;
    move((int64_t)t, (int32_t)(v & 0x7fffffffu));
  }
}

// The whole sort in one workgroup, and the move too unless vals_out is given
// (a few thousand particles' ten arrays are more than one CU moves in the
// time of another launch): at these sizes every launch of the general path
// takes its minimum of some 3 us.  N = 1000 45 -> 12 us, N = 4096 48 -> 20 us a
// rebuild (13 launches before).
constexpr int kSmallN = 8192, kSmallKeys = 8192, kSmallThreads = 1024, kSmallMove = 2048;
template <typename Move>
__global__ __launch_bounds__(kSmallThreads) void k_sort_small(
    const double* __restrict__ x, const double* __restrict__ y, const double* __restrict__ z,
    int n, Grid g, int32_t* __restrict__ cs, int32_t* __restrict__ xlow,
    int32_t* __restrict__ keys_out, int32_t* __restrict__ vals_out, int32_t* __restrict__ clear,
    Move move, MoveCheck mc) {
  constexpr int kItems = kSmallN / kSmallThreads, kKeys = kSmallKeys / kSmallThreads;
  __shared__ int cnt[kSmallKeys + 1];
  __shared__ uint32_t tv[kSmallN];
  __shared__ int wsum[kSmallThreads / 64];
  __shared__ double sh[kSmallThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (clear && tid < 16) clear[tid] = 0;
  for (int c = tid; c <= kSmallKeys; c += kSmallThreads) cnt[c] = 0;
  __syncthreads();
  int key[kItems];
  uint32_t rank[kItems];
  double m2 = 0.0;
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    const int i = tid + k * kSmallThreads;
    if (i >= n) continue;
    bool upper;
    key[k] = cell_of(x[i], y[i], z[i], g, xlow != nullptr, upper);
    rank[k] = (uint32_t)atomicAdd(&cnt[key[k]], 1) | (upper ? 0x80000000u : 0u);
    if (mc.part) {
      const double d = moved2(mc, i);
      m2 = d > m2 ? d : m2;
    }
  }
  if (mc.part) {
    m2 = wave_max_nonneg(m2);
    if (lane == 0) sh[wave] = m2;
  }
  __syncthreads();
  if (mc.part && tid == 0) {
    for (int w = 1; w < kSmallThreads / 64; ++w) m2 = sh[w] > m2 ? sh[w] : m2;
    skin_result(mc, m2);
  }
  // exclusive scan of the counts, kKeys consecutive ones per thread
  int c[kKeys], sum = 0;
#pragma unroll
  for (int k = 0; k < kKeys; ++k) {
    c[k] = cnt[tid * kKeys + k];
    sum += c[k];
  }
  int incl = sum;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int o = __shfl_up(incl, off, 64);
    if (lane >= off) incl += o;
  }
  if (lane == 63) wsum[wave] = incl;
  __syncthreads();
  int run = incl - sum;
  for (int w = 0; w < wave; ++w) run += wsum[w];
#pragma unroll
  for (int k = 0; k < kKeys; ++k) {
    const int cell = tid * kKeys + k;
    cnt[cell] = run;
    if (cell <= g.nkeys) cs[cell] = run;
    if (xlow && cell < g.nkeys && c[k] == 0) xlow[cell] = 0;
    run += c[k];
  }
  if (tid == kSmallThreads - 1) {
    cnt[kSmallKeys] = run;
    if (g.nkeys == kSmallKeys) cs[kSmallKeys] = run;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    const int i = tid + k * kSmallThreads;
    if (i < n) tv[cnt[key[k]] + (int)(rank[k] & 0x7fffffffu)] = (uint32_t)i | (rank[k] & 0x80000000u);
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    const int i = tid + k * kSmallThreads;
    if (i >= n) continue;
    const int b = cnt[key[k]], e = cnt[key[k] + 1];
    int upper;
    const int r = place_in_cell(tv, b, e, (uint32_t)i | (rank[k] & 0x80000000u), upper);
    if (xlow && r == 0) xlow[key[k]] = e - b - upper;
    if (keys_out) keys_out[b + r] = key[k];
    if (vals_out) vals_out[b + r] = i;
    else move((int64_t)b + r, i);
  }
}

template <typename Move>
__global__ __launch_bounds__(256) void k_move(const int32_t* idx, int64_t n,
                                              Move move) {
  const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (s < n) move(s, idx[s]);
}

// The displacement check alone (the radix path and the end of a run).
__global__ __launch_bounds__(256) void k_moved_max(int64_t n, MoveCheck mc) {
  __shared__ double sh[4];
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const double m = block_max256(i < n ? moved2(mc, i) : 0.0, sh);
  if (threadIdx.x == 0) mc.part[blockIdx.x] = m;
}
__global__ __launch_bounds__(256) void k_skin_check(MoveCheck mc, int nparts) {
  __shared__ double sh[4];
  double v = 0.0;
  for (int k = threadIdx.x; k < nparts; k += 256) v = mc.part[k] > v ? mc.part[k] : v;
  v = block_max256(v, sh);
  if (threadIdx.x == 0) skin_result(mc, v);
}

hipError_t skin_check(const MoveCheck& mc, int64_t n, hipStream_t st) {
  const unsigned nb = (unsigned)div_up(n, 256);
  hipLaunchKernelGGL(k_moved_max, dim3(nb), dim3(256), 0, st, n, mc);
  hipLaunchKernelGGL(k_skin_check, dim3(1), dim3(256), 0, st, mc, (int)nb);
  return hipGetLastError();
}

// Sorts the particles by cell and moves them: cell_start, xlow and clear as
// declared for sort_*; *keys_out (nullable): the sorted keys, in the sort
// buffers.
template <typename Move>
static hipError_t sort_and_move(const double* x, const double* y, const double* z, int64_t n,
                                const Grid& g, SortBufs& s, int32_t* cs, int32_t* xlow,
                                int32_t* clear, int32_t** keys_out, const Move& move,
                                const MoveCheck& mc, hipStream_t st) {
  const unsigned nb = (unsigned)div_up(n, 256);
  if (n <= kSmallN && g.nkeys <= kSmallKeys) {
    int32_t* keys = keys_out ? s.keys[0] : nullptr;
    int32_t* vals = n > kSmallMove ? s.vals[1] : nullptr;
    hipLaunchKernelGGL(k_sort_small<Move>, dim3(1), dim3(kSmallThreads), 0, st, x, y, z, (int)n, g,
                       cs, xlow, keys, vals, clear, move, mc);
    if (vals) hipLaunchKernelGGL(k_move<Move>, dim3(nb), dim3(256), 0, st, vals, n, move);
    if (keys_out) *keys_out = keys;
    return hipGetLastError();
  }
  // up to 8 cells per particle the scan over the cells is cheap (and its
  // block sums fit the radix path's histogram area)
  if ((int64_t)g.nkeys <= 8 * n) {
    uint32_t *ranks = (uint32_t*)s.vals[0], *tv = (uint32_t*)s.vals[1];
    int32_t* keys = keys_out ? s.keys[0] : nullptr;  // the unsorted keys are done with by then
    const int64_t nk1 = (int64_t)g.nkeys + 1;
    hipLaunchKernelGGL(k_zero_cells, dim3((unsigned)div_up(nk1, 256)), dim3(256), 0, st, cs,
                       g.nkeys, xlow, clear);
    hipLaunchKernelGGL(k_count_cells, dim3(nb), dim3(256), 0, st, x, y, z, n, g, xlow ? 1 : 0, cs,
                       s.keys[0], ranks, mc);
    if (nk1 <= kScanOneMost) {
      // (cs is 256-byte aligned: a piece of the workspace)
      if (nk1 <= kScanOneMost / 4)
        hipLaunchKernelGGL(k_scan_one<4>, dim3(1), dim3(1024), 0, st, cs, (int)nk1);
      else
        hipLaunchKernelGGL(k_scan_one<16>, dim3(1), dim3(1024), 0, st, cs, (int)nk1);
    } else {
      const hipError_t e = exclusive_scan(cs, cs, nk1, s.hist, false, st);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_place_cells, dim3(nb), dim3(256), 0, st, cs, s.keys[0], ranks, n, tv,
                       s.keys[1]);
    int bits = 1;
    while ((1ll << bits) < n) ++bits;
    // (the ranks are done with by then)
    hipLaunchKernelGGL(k_order_cells<Move>, dim3(nb), dim3(kOrderThreads), 0, st, cs, tv, ranks,
                       s.keys[1], n, bits, xlow, keys, move, mc, (int)nb);
    if (keys_out) *keys_out = keys;
    return hipGetLastError();
  }
  int32_t *keys, *vals;
  if (mc.part) {
    const hipError_t e = skin_check(mc, n, st);
    if (e != hipSuccess) return e;
  }
  const hipError_t e = radix_bin(x, y, z, n, g, s, cs, &keys, &vals, st, xlow, clear);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_move<Move>, dim3(nb), dim3(256), 0, st, vals, n, move);
  if (keys_out) *keys_out = keys;
  return hipGetLastError();
}

// ------------------------------------------------------- moves and gathers
// The build's move: folded positions and the caller's index of each slot.
struct MoveBuild {
  const double *x, *y, *z;
  double *ox, *oy, *oz;
  int32_t* perm;
  double L[3];
  __device__ __forceinline__ void operator()(int64_t s, int32_t j) const {
    perm[s] = j;
    ox[s] = fold(x[j], L[0]);
    oy[s] = fold(y[j], L[1]);
    oz[s] = fold(z[j], L[2]);
  }
};

hipError_t sort_build(const double* x, const double* y, const double* z, int64_t n, const Grid& g,
                      SortBufs& s, int32_t* cell_start, int32_t* xlow, int32_t** skeys,
                      int32_t* perm, double* ox, double* oy, double* oz, hipStream_t st) {
  const MoveBuild m{x, y, z, ox, oy, oz, perm, {g.box[0], g.box[1], g.box[2]}};
  return sort_and_move(x, y, z, n, g, s, cell_start, xlow, nullptr, skeys, m, MoveCheck{}, st);
}

// The analyses' move.
struct MoveAnalysis {
  const double *x, *y, *z;
  double *ox, *oy, *oz;
  float *px, *py, *pz;
  int32_t *perm, *outside;
  double L[3];
  double reach;  // see sort_analysis
  __device__ __forceinline__ void operator()(int64_t s, int32_t j) const {
    const double a = x[j], b = y[j], c = z[j];
    const double fa = fold(a, L[0]), fb = fold(b, L[1]), fc = fold(c, L[2]);
    perm[s] = j;
    ox[s] = a;
    oy[s] = b;
    oz[s] = c;
    const bool near = __builtin_fabs(a) <= reach * L[0] && __builtin_fabs(b) <= reach * L[1] &&
                      __builtin_fabs(c) <= reach * L[2];
    px[s] = near ? (float)fa : __builtin_nanf("");
    py[s] = (float)fb;
    pz[s] = (float)fc;
    if (!(within_reach(a, L[0]) && within_reach(b, L[1]) && within_reach(c, L[2]))) *outside = 1;
  }
};

hipError_t sort_analysis(const double* x, const double* y, const double* z, int64_t n,
                         const Grid& g, SortBufs& s, int32_t* cell_start, int32_t** skeys,
                         int32_t** perm, double* ox, double* oy, double* oz, float* px, float* py,
                         float* pz, int32_t* small, double rc, hipStream_t st) {
  // the values' second buffer: free again when the move writes it (the radix
  // path may have sorted the values into it: each slot reads its own first)
  *perm = s.vals[0];
  const MoveAnalysis m{x, y, z, ox, oy, oz, px, py, pz, *perm, small, {g.box[0], g.box[1], g.box[2]},
                       screen_fits(g, rc) ? 1048576.0 : -1.0};
  return sort_and_move(x, y, z, n, g, s, cell_start, nullptr, small, skeys, m, MoveCheck{}, st);
}

// A run's move: all ten arrays, positions folded; xb/yb/zb receive a copy of
// them, *bound becomes zero (a new list: nothing has moved since).
template <typename FT>
struct MoveState {
  StateArrays src, dst;
  double *xb, *yb, *zb, *bound;
  double L[3];
  __device__ __forceinline__ void operator()(int64_t s, int32_t j) const {
    if (s == 0) *bound = 0.0;
    const double a = fold(src.x[j], L[0]), b = fold(src.y[j], L[1]), c = fold(src.z[j], L[2]);
    dst.x[s] = a;
    dst.y[s] = b;
    dst.z[s] = c;
    xb[s] = a;
    yb[s] = b;
    zb[s] = c;
    dst.vx[s] = src.vx[j];
    dst.vy[s] = src.vy[j];
    dst.vz[s] = src.vz[j];
    ((FT*)dst.fx)[s] = ((const FT*)src.fx)[j];
    ((FT*)dst.fy)[s] = ((const FT*)src.fy)[j];
    ((FT*)dst.fz)[s] = ((const FT*)src.fz)[j];
    dst.ids[s] = src.ids[j];
  }
};

hipError_t sort_state(const StateArrays& src, const StateArrays& dst, int64_t n, int fbytes,
                      const Grid& g, SortBufs& s, int32_t* cell_start, int32_t* xlow, double* xb,
                      double* yb, double* zb, double* bound, const MoveCheck& mc,
                      hipStream_t st) {
  if (fbytes == 4) {
    const MoveState<float> m{src, dst, xb, yb, zb, bound, {g.box[0], g.box[1], g.box[2]}};
    return sort_and_move(src.x, src.y, src.z, n, g, s, cell_start, xlow, nullptr, nullptr, m, mc, st);
  }
  const MoveState<double> m{src, dst, xb, yb, zb, bound, {g.box[0], g.box[1], g.box[2]}};
  return sort_and_move(src.x, src.y, src.z, n, g, s, cell_start, xlow, nullptr, nullptr, m, mc, st);
}

// Positions of the last build's slots, each moved to the periodic image
// nearest the centre of the cell it was binned in (the images the tiles
// assume), whatever image the caller passes.
__global__ void k_gather_canonical(const double* __restrict__ x, const double* __restrict__ y,
                                   const double* __restrict__ z, const int32_t* __restrict__ idx,
                                   const int32_t* __restrict__ skeys, int64_t n, Grid g,
                                   double* __restrict__ ox, double* __restrict__ oy,
                                   double* __restrict__ oz) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n) return;
  const int key = skeys[s];
  const int brick = key / g.V, local = key - brick * g.V;
  const int bx = brick % g.nb[0], by = (brick / g.nb[0]) % g.nb[1], bz = brick / (g.nb[0] * g.nb[1]);
  const int cx = bx * g.B[0] + local % g.B[0];
  const int cy = by * g.B[1] + (local / g.B[0]) % g.B[1];
  const int cz = bz * g.B[2] + local / (g.B[0] * g.B[1]);
  const int32_t j = idx[s];
  const double p[3] = {x[j], y[j], z[j]};
  const int c[3] = {cx, cy, cz};
  double q[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double L = g.box[k];
    const double centre = ((double)c[k] + 0.5) / g.inv_side[k];
    q[k] = p[k] + L * rint((centre - p[k]) / L);
  }
  ox[s] = q[0];
  oy[s] = q[1];
  oz[s] = q[2];
}

hipError_t gather_canonical(const double* x, const double* y, const double* z, const int32_t* idx,
                            const int32_t* skeys, int64_t n, const Grid& g, double* ox, double* oy,
                            double* oz, hipStream_t st) {
  hipLaunchKernelGGL(k_gather_canonical, dim3((unsigned)div_up(n, 256)), dim3(256), 0, st, x, y, z,
                     idx, skeys, n, g, ox, oy, oz);
  return hipGetLastError();
}

// dst[a][s] = src[a][s] for every array a whose two pointers differ, one
// launch for all of them (the end of a run hands the state back).
template <typename FT>
__global__ void k_copy_state(StateArrays src, StateArrays dst, int64_t n) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n) return;
  if (src.x != dst.x) dst.x[s] = src.x[s];
  if (src.y != dst.y) dst.y[s] = src.y[s];
  if (src.z != dst.z) dst.z[s] = src.z[s];
  if (src.vx != dst.vx) dst.vx[s] = src.vx[s];
  if (src.vy != dst.vy) dst.vy[s] = src.vy[s];
  if (src.vz != dst.vz) dst.vz[s] = src.vz[s];
  if (src.fx != dst.fx) ((FT*)dst.fx)[s] = ((const FT*)src.fx)[s];
  if (src.fy != dst.fy) ((FT*)dst.fy)[s] = ((const FT*)src.fy)[s];
  if (src.fz != dst.fz) ((FT*)dst.fz)[s] = ((const FT*)src.fz)[s];
  if (src.ids != dst.ids) dst.ids[s] = src.ids[s];
}

hipError_t copy_state(const StateArrays& src, const StateArrays& dst, int64_t n, int fbytes,
                      hipStream_t st) {
  if (src.x == dst.x && src.y == dst.y && src.z == dst.z && src.vx == dst.vx && src.vy == dst.vy &&
      src.vz == dst.vz && src.fx == dst.fx && src.fy == dst.fy && src.fz == dst.fz &&
      src.ids == dst.ids)
    return hipSuccess;
  const unsigned nb = (unsigned)div_up(n, 256);
  if (fbytes == 4)
    hipLaunchKernelGGL(k_copy_state<float>, dim3(nb), dim3(256), 0, st, src, dst, n);
  else
    hipLaunchKernelGGL(k_copy_state<double>, dim3(nb), dim3(256), 0, st, src, dst, n);
  return hipGetLastError();
}

}  // namespace mdpl
