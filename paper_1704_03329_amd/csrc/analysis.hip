// Structure analysis pair loops (Sec. 4).
//
// Both analyses first find the bonds of a particle in two steps.  The screen
// (one lane per particle) walks the nine rows of three consecutive cells of
// its stencil on FP32 copies of the folded sorted positions and notes, in an
// LDS column of its own, every candidate that the FP32 distance cannot rule
// out.  The bonds proper are then decided by the exact FP64 predicate on the
// few noted candidates.  Only a sixth of the candidates are bonds, and in a
// loop over candidates some lane of a wave nearly always has one, so that
// anything done per bond inside that loop is paid for every candidate.
//
// Bond order (Sec. 4.1, Eqs. Qell and qellm, Algs. sph_I and sph_II): each
// lane accumulates the moments of Y_l^m over its noted bonds in registers;
// the particle loop of Alg. sph_II is fused at the end.  With
// Y_l^m = N_lm P~_l^m(z) (x + i y)^m and P~_l^m = d^m P_l/dz^m,
//   Q_l = sqrt( sum_m w_lm (A_lm^2 + B_lm^2) ) / nu,
//   w_l0 = 1, w_lm = 2 (l-m)!/(l+m)! (m >= 1),
// where A + iB = sum_j P~_l^m(z_j) (x_j + i y_j)^m (the -m terms have the
// same modulus and are folded into the factor 2).  Unit vectors from the
// FP64 separation, harmonics in FP32.
//
// Common-neighbour analysis (Sec. 4.2, Algs. cna_I to cna_III and
// max_cluster_size): the bonds among the neighbours of i (every two members
// of N(i), exact bond test) become one bit mask per member (bit a of adj[b]
// <=> neighbour a bonded to neighbour b).  For the bond (i, N(i)[b]): common
// neighbours C = adj[b], n_cn = |C|, n_b = half the degree sum inside C, and
// n_lcb = largest number of edges in a connected component of C, by mask
// flood fill where the edge and vertex counts leave it open.  All integer
// work, bit-exact.
#include <math.h>

#include "device_util.h"
#include "internal.h"
#include "bond_screen.h"

namespace mdpl {

// ---------------------------------------------------------------- screen
// A candidate noted by the screen is its sorted slot (n <= 2^26, checked by
// the caller), in an LDS column of the lane's own: row k at word 64 k + lane
// of the wave's queue, so that writes and reads of all lanes fall into
// different banks whatever their rows.
constexpr int kQPitch = 64;

// a[i + j] by a 32-bit byte offset (i + j < 2^30)
template <int J = 0, typename T>
__device__ __forceinline__ T at32(const T* __restrict__ a, uint32_t i) {
  return ((const T*)((const char*)a + i * (uint32_t)sizeof(T)))[J];
}

// The definition's minimum-image separation (of exact_d2) of candidates that
// rarely need the wrap: it is formed only where a lane of the wave does.
__device__ __forceinline__ double bond_sep(double xi, double yi, double zi, double xj, double yj,
                                           double zj, const Grid& g, double& dx, double& dy,
                                           double& dz) {
  const double Lx = g.box[0], Ly = g.box[1], Lz = g.box[2];
  const double hx = 0.5 * Lx, hy = 0.5 * Ly, hz = 0.5 * Lz;
  dx = xi - xj;
  dy = yi - yj;
  dz = zi - zj;
  if (__any((__builtin_fabs(dx) > hx) | (__builtin_fabs(dy) > hy) | (__builtin_fabs(dz) > hz))) {
    dx = dx > hx ? dx - Lx : (dx < -hx ? dx + Lx : dx);
    dy = dy > hy ? dy - Ly : (dy < -hy ? dy + Ly : dy);
    dz = dz > hz ? dz - Lz : (dz < -hz ? dz + Lz : dz);
  }
  return sq_sum(dx, dy, dz);
}

// The screen of one particle per lane over its nine stencil rows.  A row's
// three cells are consecutive in memory except across the box edge along x,
// where one of them is a second range.  run() notes candidates until all rows
// are done (returns true) or the next four might overrun a column of CAP
// entries (false; KEEP: never, cnt may pass CAP and the column is then not to
// be used); the lane's noted candidates are col[0 .. cnt).  Four candidates
// are loaded at once, past the end of a row too (up to another row's length,
// within the workspace: the FP32 copies are followed by larger arrays).
template <int CAP, bool KEEP>
struct Screen {
  const BondScan& q;
  const Grid& g;
  uint32_t* col;
  int s, cnt, r, rows, per, lo, hi, wc, cx, cy, cz, t, e;
  bool ok, edge;
  float x, y, z, xw, r2;

  __device__ __forceinline__ Screen(const BondScan& q_, const Grid& g_, int s_, bool ok_,
                                    float r2_, uint32_t* col_)
      : q(q_), g(g_), col(col_), s(s_), cnt(0), r(0), ok(ok_), r2(r2_) {
    const int n0 = g.nc[0], n1 = g.nc[1];
    const int key = ok ? q.skeys[s] : 0;
    cx = key % n0;
    cy = (key / n0) % n1;
    cz = key / (n0 * n1);
    x = ok ? q.px[s] : 0.0f;
    y = ok ? q.py[s] : 0.0f;
    z = ok ? q.pz[s] : 0.0f;
    lo = cx > 0 ? cx - 1 : 0;
    hi = cx < n0 - 1 ? cx + 1 : n0 - 1;
    edge = ok && (cx == 0 || cx == n0 - 1);
    per = __any(edge) ? 2 : 1;  // ranges per row: two only where a lane is at the edge
    rows = 9 * per;
    // the cell across the edge and the particle's image next to it
    wc = cx == 0 ? n0 - 1 : 0;
    xw = screen_image(x, g.box[0], cx == 0 ? -1 : 1);
    range();
  }
  // y and z images of the particle next to row r
  __device__ __forceinline__ void image(float& xs, float& ys, float& zs) const {
    const int row = per == 2 ? r >> 1 : r;
    const int z2 = cz + row / 3 - 1, y2 = cy + row % 3 - 1;
    xs = per == 2 && (r & 1) ? xw : x;
    ys = screen_image(y, g.box[1], y2 < 0 ? -1 : (y2 >= g.nc[1] ? 1 : 0));
    zs = screen_image(z, g.box[2], z2 < 0 ? -1 : (z2 >= g.nc[2] ? 1 : 0));
  }
  // candidates [t, e) of row r
  __device__ __forceinline__ void range() {
    const int n0 = g.nc[0], n1 = g.nc[1], n2 = g.nc[2];
    const int row = per == 2 ? r >> 1 : r;
    const bool wrap = per == 2 && (r & 1);
    int z2 = cz + row / 3 - 1, y2 = cy + row % 3 - 1;
    z2 += z2 < 0 ? n2 : (z2 >= n2 ? -n2 : 0);
    y2 += y2 < 0 ? n1 : (y2 >= n1 ? -n1 : 0);
    // (64-bit offsets: a grid may have 2^30 cells, and cs one entry more)
    const int32_t* const row0 = q.cs + (z2 * n1 + y2) * n0;
    t = e = 0;
    if (wrap ? edge : ok) {
      t = row0[wrap ? wc : lo];
      e = row0[(wrap ? wc : hi) + 1];
    }
  }
  __device__ __forceinline__ bool run() {
    while (r < rows) {
      float xs, ys, zs;
      image(xs, ys, zs);
      while (__any(t < e)) {
        if (!KEEP && __any(cnt > CAP - 4)) return false;
        float dx[4], dy[4], dz[4];
        const uint32_t u = (uint32_t)t;
        dx[0] = at32<0>(q.px, u); dx[1] = at32<1>(q.px, u); dx[2] = at32<2>(q.px, u); dx[3] = at32<3>(q.px, u);
        dy[0] = at32<0>(q.py, u); dy[1] = at32<1>(q.py, u); dy[2] = at32<2>(q.py, u); dy[3] = at32<3>(q.py, u);
        dz[0] = at32<0>(q.pz, u); dz[1] = at32<1>(q.pz, u); dz[2] = at32<2>(q.pz, u); dz[3] = at32<3>(q.pz, u);
        const int left = e - t, self = s - t;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float d2 = screen_d2(xs - dx[j], ys - dy[j], zs - dz[j]);
          // written whether noted or not: the next note overwrites it
          col[(KEEP && cnt >= CAP ? CAP - 1 : cnt) * kQPitch] = u + j;
          // (a copy that is NaN is noted: only the exact test can tell)
          cnt += (int)(!(d2 > r2) & (left > j) & (self != j));
        }
        t += 4;
      }
      if (++r < rows) range();
    }
    return true;
  }
};

// ------------------------------------------------------------ bond order
// 2 (l-m)!/(l+m)! for m >= 1 and 1 for m = 0.
constexpr double qweight(int l, int m) {
  if (m == 0) return 1.0;
  double r = 2.0;
  for (int k = l - m + 1; k <= l + m; ++k) r /= (double)k;
  return r;
}
// The moments below are those of P~_l^m / f, f the factor taken out of the
// polynomial; the weight of a squared moment is then w_lm f^2.
constexpr float qscale(int l, int m, double f) { return (float)(qweight(l, m) * f * f); }

constexpr int kBoaThreads = 256;
constexpr int kBoaQueue = 24;  // noted candidates per lane before they are worked off

// What bounds it: vector instructions, about 13 per candidate in the screen
// and 130 per bond, 3770 per wave of 64 particles.  4 * 10^6 atoms of a
// polycrystal: 1211 -> 563 us (one loop with the harmonics inside it before),
// 125,000 with Q5 82 -> 39 us.
template <bool Q5>
__global__ __launch_bounds__(kBoaThreads) void k_boa(BondScan q, int64_t n, Grid g, double rc2,
                                                     float r2s, float* __restrict__ q4,
                                                     float* __restrict__ q5,
                                                     float* __restrict__ q6,
                                                     int32_t* __restrict__ nnb) {
  __shared__ uint32_t queue[kBoaThreads / 64][kBoaQueue * kQPitch];
  const int64_t s = (int64_t)blockIdx.x * kBoaThreads + threadIdx.x;
  const bool ok = s < n;
  uint32_t* const col = queue[threadIdx.x >> 6] + (threadIdx.x & 63);
  // moments: A[l][m] (m = 0..l), B[l][m] (m = 1..l) for l = 4, 5, 6
  float A4[5] = {0}, B4[5] = {0}, A5[6] = {0}, B5[6] = {0}, A6[7] = {0}, B6[7] = {0};
  int nu = 0;
  const double xi = ok ? q.sx[s] : 0.0, yi = ok ? q.sy[s] : 0.0, zi = ok ? q.sz[s] : 0.0;
  Screen<kBoaQueue, false> screen(q, g, (int)s, ok, r2s, col);
  for (bool done = false; !done;) {
    done = screen.run();
    const int cnt = screen.cnt;
    for (int k = 0; k < cnt; ++k) {
      const uint32_t t = col[k * kQPitch];
      double dx, dy, dz;
      const double d2 =
          bond_sep(xi, yi, zi, at32(q.sx, t), at32(q.sy, t), at32(q.sz, t), g, dx, dy, dz);
      if (!(d2 < rc2)) continue;
      ++nu;
      const float ir = __builtin_amdgcn_rsqf((float)d2);  // the bond test above is FP64
      const float ux = (float)dx * ir, uy = (float)dy * ir, uz = (float)dz * ir;
      // (x + i y)^m, m = 1..6
      const float c2 = ux * ux - uy * uy, s2 = 2.0f * (ux * uy);
      const float c3 = c2 * ux - s2 * uy, s3 = c2 * uy + s2 * ux;
      const float c4 = c2 * c2 - s2 * s2, s4 = 2.0f * (c2 * s2);
      const float c5 = c4 * ux - s4 * uy, s5 = c4 * uy + s4 * ux;
      const float c6 = c3 * c3 - s3 * s3, s6 = 2.0f * (c3 * s3);
      const float z2 = uz * uz;
      // polynomials in z^2, highest coefficient first, by Horner's rule: each
      // rounding is one of a partial result near the final one.  RMS errors of
      // a polycrystal's Q4, Q5, Q6 2.20, 2.78, 4.79 10^-8 (sums of powers of z
      // 2.24, 2.95, 4.98; the recurrence in l 2.24, 2.87, 4.87)
      auto poly2 = [z2](float a, float b, float c) {
        return __builtin_fmaf(__builtin_fmaf(a, z2, b), z2, c);
      };
      // z (x + i y)^m of the odd orders
      const float zc1 = uz * ux, zs1 = uz * uy, zc3 = uz * c3, zs3 = uz * s3;
      // l = 4: (35 z^4 - 30 z^2 + 3), z (7 z^2 - 3), 7 z^2 - 1, z, 1
      const float p41 = 7.0f * z2 - 3.0f, p42 = 7.0f * z2 - 1.0f;
      A4[0] += poly2(35.0f, -30.0f, 3.0f);
      A4[1] += p41 * zc1;
      B4[1] += p41 * zs1;
      A4[2] += p42 * c2;
      B4[2] += p42 * s2;
      A4[3] += zc3;
      B4[3] += zs3;
      A4[4] += c4;
      B4[4] += s4;
      if (Q5) {
        // l = 5: z (63 z^4 - 70 z^2 + 15), 21 z^4 - 14 z^2 + 1, z (3 z^2 - 1), 9 z^2 - 1, z, 1
        const float p51 = poly2(21.0f, -14.0f, 1.0f), p52 = (3.0f * z2 - 1.0f) * uz;
        const float p53 = 9.0f * z2 - 1.0f;
        A5[0] += uz * poly2(63.0f, -70.0f, 15.0f);
        A5[1] += p51 * ux;
        B5[1] += p51 * uy;
        A5[2] += p52 * c2;
        B5[2] += p52 * s2;
        A5[3] += p53 * c3;
        B5[3] += p53 * s3;
        A5[4] += uz * c4;
        B5[4] += uz * s4;
        A5[5] += c5;
        B5[5] += s5;
      }
      // l = 6: 231 z^6 - 315 z^4 + 105 z^2 - 5, z (33 z^4 - 30 z^2 + 5),
      //        33 z^4 - 18 z^2 + 1, z (11 z^2 - 3), 11 z^2 - 1, z, 1
      const float p61 = poly2(33.0f, -30.0f, 5.0f), p62 = poly2(33.0f, -18.0f, 1.0f);
      const float p63 = 11.0f * z2 - 3.0f, p64 = 11.0f * z2 - 1.0f;
      A6[0] += __builtin_fmaf(poly2(231.0f, -315.0f, 105.0f), z2, -5.0f);
      A6[1] += p61 * zc1;
      B6[1] += p61 * zs1;
      A6[2] += p62 * c2;
      B6[2] += p62 * s2;
      A6[3] += p63 * zc3;
      B6[3] += p63 * zs3;
      A6[4] += p64 * c4;
      B6[4] += p64 * s4;
      A6[5] += uz * c5;
      B6[5] += uz * s5;
      A6[6] += c6;
      B6[6] += s6;
    }
    screen.cnt = 0;
  }
  if (!ok) return;
  // weights times the squares of the factors taken out: 1/8, 5/2, 15/2, 105,
  // 105; 1/8, 15/8, 105/2, 105/2, 945, 945; 1/16, 21/8, 105/8, 315/2, 945/2, 10395, 10395
  constexpr float w4[5] = {qscale(4, 0, 1.0 / 8), qscale(4, 1, 2.5), qscale(4, 2, 7.5),
                           qscale(4, 3, 105.0), qscale(4, 4, 105.0)};
  constexpr float w5[6] = {qscale(5, 0, 1.0 / 8), qscale(5, 1, 1.875), qscale(5, 2, 52.5),
                           qscale(5, 3, 52.5), qscale(5, 4, 945.0), qscale(5, 5, 945.0)};
  constexpr float w6[7] = {qscale(6, 0, 1.0 / 16), qscale(6, 1, 2.625), qscale(6, 2, 13.125),
                           qscale(6, 3, 157.5), qscale(6, 4, 472.5), qscale(6, 5, 10395.0),
                           qscale(6, 6, 10395.0)};
  float s4 = 0.0f, s5 = 0.0f, s6 = 0.0f;
#pragma unroll
  for (int m = 0; m <= 4; ++m) s4 += w4[m] * (A4[m] * A4[m] + B4[m] * B4[m]);
#pragma unroll
  for (int m = 0; m <= 5; ++m) s5 += w5[m] * (A5[m] * A5[m] + B5[m] * B5[m]);
#pragma unroll
  for (int m = 0; m <= 6; ++m) s6 += w6[m] * (A6[m] * A6[m] + B6[m] * B6[m]);
  const float inv = nu > 0 ? 1.0f / (float)nu : 0.0f;
  const int32_t o = q.perm[s];
  q4[o] = sqrtf(s4) * inv;
  if (Q5) q5[o] = sqrtf(s5) * inv;
  q6[o] = sqrtf(s6) * inv;
  nnb[o] = nu;
}

hipError_t boa_q(const BondScan& q, int64_t n, const Grid& g, double rc2, float* q4, float* q5,
                 float* q6, int32_t* nnb, hipStream_t st) {
  const dim3 grid((unsigned)div_up(n, kBoaThreads)), block(kBoaThreads);
  const float r2s = screen_r2(g.box, g.side, rc2);
  if (q5)
    hipLaunchKernelGGL(k_boa<true>, grid, block, 0, st, q, n, g, rc2, r2s, q4, q5, q6, nnb);
  else
    hipLaunchKernelGGL(k_boa<false>, grid, block, 0, st, q, n, g, rc2, r2s, q4, q5, q6, nnb);
  return hipGetLastError();
}

// ------------------------------------------------------------------- CNA
constexpr int kCnaQueue = 32;  // noted candidates per lane, at most kept in registers

__device__ __forceinline__ uint32_t pack_triplet(int ncn, int nb, int nlcb) {
  return ((uint32_t)ncn << 20) | ((uint32_t)nb << 10) | (uint32_t)nlcb;
}

struct CnaOut {
  uint32_t* trip;
  int32_t* nnb;
  uint8_t* label;
  int max_nb;  // list capacity and row length of trip
  int quads;   // 1: the rows of trip are 16-byte aligned
};

// Whether a position lies more than a quarter of the box outside it: two that
// do not are at most 1.5 edges apart, and the definition's one wrap finds the
// nearest image.
__device__ __forceinline__ bool far_image(const Grid& g, double x, double y, double z) {
  return !(within_reach(x, g.box[0]) && within_reach(y, g.box[1]) && within_reach(z, g.box[2]));
}

// All ones where bit m of v is set, else zero.
__device__ __forceinline__ uint32_t bit_mask(uint32_t v, int m) {
  return (uint32_t)((int32_t)(v << (31 - m)) >> 31);
}

// Ascending order by Batcher's odd-even merge network (N <= 32, padded with
// the largest value, whose exchanges fold away).
template <int N>
__device__ __forceinline__ void sort_network(uint32_t (&c)[N]) {
  uint32_t v[32];
#pragma unroll
  for (int i = 0; i < 32; ++i) v[i] = i < N ? c[i < N ? i : 0] : 0xffffffffu;
#pragma unroll
  for (int p = 1; p < 32; p *= 2)
#pragma unroll
    for (int k = p; k >= 1; k /= 2)
#pragma unroll
      for (int j = k % p; j + k < 32; j += 2 * k)
#pragma unroll
        for (int i = 0; i < k; ++i)
          if (i + j + k < 32 && (i + j) / (2 * p) == (i + j + k) / (2 * p)) {
            const uint32_t a = v[i + j], b = v[i + j + k];
            v[i + j] = a < b ? a : b;
            v[i + j + k] = a < b ? b : a;
          }
#pragma unroll
  for (int i = 0; i < N; ++i) c[i] = v[i];
}

// The signature of one particle per lane, up to N noted candidates each
// (col[0 .. c), N a constant so that separations and masks stay in
// registers); unfolded: some particle's stored position lies far outside the
// box (far_image).  Returns the bond count, or -1 where the exact test of a pair
// of neighbours is needed (nothing is written then, col stays as it was).
template <int N>
__device__ __forceinline__ int cna_lane(const BondScan& q, const Grid& g, double rc2, float band,
                                        int s, int c, uint32_t* __restrict__ col,
                                        const CnaOut& out, bool unfolded) {
  const double xi = q.sx[s], yi = q.sy[s], zi = q.sz[s];
  // N(i): the exact bond test of every noted candidate, four loaded at once
  // (more would only cost registers)
  float X[N], Y[N], Z[N];
  uint32_t bonds = 0;
  bool odd = false;
#pragma unroll
  for (int k0 = 0; k0 < N; k0 += 4) {
    double xt[4], yt[4], zt[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (k0 + j >= N) continue;
      const uint32_t t = k0 + j < c ? col[(k0 + j) * kQPitch] : (uint32_t)s;
      xt[j] = at32(q.sx, t);
      yt[j] = at32(q.sy, t);
      zt[j] = at32(q.sz, t);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int k = k0 + j;
      if (k >= N) continue;
      double dx, dy, dz;
      const double d2 = bond_sep(xi, yi, zi, xt[j], yt[j], zt[j], g, dx, dy, dz);
      const bool bond = (k < c) & (d2 < rc2);
      bonds |= bond ? 1u << k : 0u;
      if (unfolded) odd |= bond & far_image(g, xt[j], yt[j], zt[j]);
      X[k] = bond ? (float)dx : 1e18f;
      Y[k] = bond ? (float)dy : 1e18f;
      Z[k] = bond ? (float)dz : 1e18f;
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  // The members bonded to each other, from the FP32 separations (each
  // component within 2^-24 rc of the FP64 one, their difference within 3 2^-24
  // rc, so that a squared distance near rc^2 is within (6 sqrt(3) + 4) 2^-24
  // rc^2 < 9 10^-7 rc^2 of the exact one).  A pair within band = 2 10^-6 rc^2 of
  // the cutoff needs the exact test, as do positions far outside
  // the box (whose images the conditional wrap of the definition may miss).
  const float r2 = (float)rc2;
  // Every member takes the sign bits of its pairs one by one, partners in
  // descending order: first those above it, then those below it.  (A slot
  // without a bond is far from all bonds; its bits go below.)
  uint32_t adj[N];
#pragma unroll
  for (int k = 0; k < N; ++k) adj[k] = 0;
  float near = 3e38f;
#pragma unroll
  for (int a = N - 1; a >= 0; --a) {
#pragma unroll
    for (int b = N - 1; b > a; --b) {
      const float ax = X[a] - X[b], ay = Y[a] - Y[b], az = Z[a] - Z[b];
      const float e = __builtin_fmaf(az, az, __builtin_fmaf(ay, ay, __builtin_fmaf(ax, ax, -r2)));
      near = fminf(near, __builtin_fabsf(e));
      adj[a] = __builtin_amdgcn_alignbit(adj[a], __float_as_uint(e), 31);
      adj[b] = __builtin_amdgcn_alignbit(adj[b], __float_as_uint(e), 31);
      if ((b - a) % 4 == 1) __builtin_amdgcn_sched_barrier(0);  // few pairs in flight
    }
  }
  // (the masks are to be complete here: moved below the return, their inputs
  // would all have to live until then)
#pragma unroll
  for (int k = 0; k < N; ++k) asm volatile("" : "+v"(adj[k]));
  if (near <= band || odd) return -1;
  // the masks in the lane's column: row b is bond b's common neighbours until
  // its triplet replaces them
#pragma unroll
  for (int k = 0; k < N; ++k) {
    adj[k] += adj[k] & (uint32_t)(~0ull << k);  // room for the member's own bit
    adj[k] &= bonds;
    col[k * kQPitch] = adj[k];
  }
  const int ni = __popc(bonds);
  int b = 0;
  for (uint32_t rest = bonds; rest; rest &= rest - 1) {
    b = __builtin_ctz(rest);
    const uint32_t C = col[b * kQPitch];
    uint32_t ends = 0;  // members of C with a bond inside C
    int deg = 0;
#pragma unroll
    for (int m = 0; m < N; ++m) {
      const uint32_t in = adj[m] & C & bit_mask(C, m);
      deg += __popc(in);
      ends |= in;
    }
    const int nb = deg >> 1, v = __popc(ends);
    int best = nb == 2 && v == 4 ? 1 : nb;
    // three or more edges on up to four members are connected
    if (nb > 2 && v > 4) {
      uint32_t rem = ends;
      best = 0;
      while (rem) {
        uint32_t comp = rem & (~rem + 1), before;
        do {
          before = comp;
#pragma unroll
          for (int m = 0; m < N; ++m) comp |= adj[m] & C & bit_mask(comp, m);
        } while (comp != before);
        int e2 = deg;
        if (comp != ends) {
          e2 = 0;
#pragma unroll
          for (int m = 0; m < N; ++m) e2 += __popc(adj[m] & comp & bit_mask(comp, m));
        }
        best = (e2 >> 1) > best ? e2 >> 1 : best;
        rem &= ~comp;
      }
    }
    col[b * kQPitch] = pack_triplet(__popc(C), nb, best);
  }
  uint32_t code[N];
#pragma unroll
  for (int k = 0; k < N; ++k) code[k] = (bonds >> k) & 1 ? col[k * kQPitch] : 0xffffffffu;
  sort_network<N>(code);
  const int32_t o = q.perm[s];
  out.nnb[o] = ni;
  uint8_t lab = 0;
  if (ni <= out.max_nb) {  // else the list is incomplete: no triplets, no signature
    uint32_t* __restrict__ row = out.trip + (int64_t)o * out.max_nb;
#pragma unroll
    for (int k = 0; k < N; k += 4) {
      if (k + 4 <= N && out.quads && k + 4 <= ni) {
        *(uint4*)(row + k) = make_uint4(code[k], code[k + 1 < N ? k + 1 : k],
                                        code[k + 2 < N ? k + 2 : k], code[k + 3 < N ? k + 3 : k]);
      } else {
#pragma unroll
        for (int j = k; j < k + 4 && j < N; ++j)
          if (j < ni) row[j] = code[j];
      }
    }
    // the reference signatures, as sorted: 12 (4,2,1); 6 (4,2,1) and 6 (4,2,2);
    // 6 (4,4,4) and 8 (6,6,6)
    const uint32_t t421 = pack_triplet(4, 2, 1), t422 = pack_triplet(4, 2, 2);
    if constexpr (N >= 12) {
      if (ni == 12 && code[0] == t421 && code[11] == t421) lab = 1;
      if (ni == 12 && code[0] == t421 && code[5] == t421 && code[6] == t422 && code[11] == t422)
        lab = 2;
    }
    if constexpr (N >= 14)
      if (ni == 14 && code[0] == pack_triplet(4, 4, 4) && code[5] == pack_triplet(4, 4, 4) &&
          code[6] == pack_triplet(6, 6, 6) && code[13] == pack_triplet(6, 6, 6))
        lab = 3;
  }
  out.label[o] = lab;
  return ni;
}

// All bonds of slot s by the whole wave (exact test of every stencil
// candidate): their number, and the slots of the first 64 in list (LDS).
// The 27 cells' ranges are laid end to end over the lanes, so that a stencil
// takes one or two rounds of loads.
__device__ inline int bonds_of(const BondScan& q, const Grid& g, double rc2, int s,
                               uint32_t* __restrict__ list) {
  const int lane = (int)threadIdx.x & 63;
  const double xi = q.sx[s], yi = q.sy[s], zi = q.sz[s];
  const double Lx = g.box[0], Ly = g.box[1], Lz = g.box[2];
  const int n0 = g.nc[0], n1 = g.nc[1], n2 = g.nc[2];
  const int key = q.skeys[s];
  const int cx = key % n0, cy = (key / n0) % n1, cz = key / (n0 * n1);
  // lane c < 27: its cell's first slot and the candidates before it
  const int x2 = (cx + lane % 3 - 1 + n0) % n0, y2 = (cy + (lane / 3) % 3 - 1 + n1) % n1;
  const int z2 = (cz + (lane / 9) % 3 - 1 + n2) % n2;
  const int cell = (z2 * n1 + y2) * n0 + x2;
  const int start = q.cs[cell];
  int upto = lane < 27 ? q.cs[cell + 1] - start : 0;
#pragma unroll
  for (int off = 1; off < 32; off <<= 1) {
    const int o = __shfl_up(upto, off, 64);
    if (lane >= off) upto += o;
  }
  const int total = __shfl(upto, 26, 64);
  int found = 0;
  wave_lds_sync();
  for (int u0 = 0; u0 < total; u0 += 64) {
    const int u = u0 + lane;
    int c = 0;  // the cell of candidate u: the first with upto > u
#pragma unroll
    for (int step = 16; step; step >>= 1) {
      const int below = __shfl(upto, c + step - 1, 64);  // lanes past 26 hold the total
      c += below <= u ? step : 0;
    }
    c = c < 26 ? c : 26;
    const int before = __shfl(upto, c > 0 ? c - 1 : 0, 64), first = __shfl(start, c, 64);
    const int t = u < total ? first + u - (c > 0 ? before : 0) : s;
    const bool in = t != s && exact_d2(xi, yi, zi, q.sx[t], q.sy[t], q.sz[t], Lx, Ly, Lz,
                                       0.5 * Lx, 0.5 * Ly, 0.5 * Lz) < rc2;
    const uint64_t m = __ballot(in);
    const int at = found + __popcll(m & ((1ull << lane) - 1));
    if (in && at < 64) list[at] = (uint32_t)t;
    found += __popcll(m);
  }
  wave_lds_sync();
  return found;
}

// The bonds of slot s among its noted candidates (c of them, lane k's in
// row k of the column): their number, their slots in list.
__device__ inline int bonds_noted(const BondScan& q, const Grid& g, double rc2, int s, int c,
                                  const uint32_t* __restrict__ col, uint32_t* __restrict__ list) {
  const int lane = (int)threadIdx.x & 63;
  const double Lx = g.box[0], Ly = g.box[1], Lz = g.box[2];
  const uint32_t t = lane < c ? col[lane * kQPitch] : (uint32_t)s;
  const bool in = lane < c && exact_d2(q.sx[s], q.sy[s], q.sz[s], q.sx[t], q.sy[t], q.sz[t], Lx, Ly,
                                       Lz, 0.5 * Lx, 0.5 * Ly, 0.5 * Lz) < rc2;
  const uint64_t m = __ballot(in);
  wave_lds_sync();
  if (in) list[__popcll(m & ((1ull << lane) - 1))] = t;
  wave_lds_sync();
  return __popcll(m);
}

// Bit m of the 64-bit mask (lo, hi), all ones where it is set.
__device__ __forceinline__ uint32_t bit_mask64(uint32_t lo, uint32_t hi, int m) {
  return bit_mask(m < 32 ? lo : hi, m & 31);
}

// The signature of slot s by the whole wave, lane b its bond b (ni <= 64 of
// them, slots in list).  Members of the loops are the same for all lanes, so
// that their values come by v_readlane.  The pairs of neighbours as in
// cna_lane, all of them by the exact test where that leaves one open.
// Fcc of 108,000 atoms with 41 bonds each 2160 -> 1066 us, fluid with 55 2830
// -> 1370 (every value by a shuffle, every pair by the exact test).
__device__ inline void cna_wave(const BondScan& q, const Grid& g, double rc2, float band, int s,
                                int ni, const uint32_t* __restrict__ list, const CnaOut& out,
                                bool unfolded) {
  const int b = (int)threadIdx.x & 63;
  const bool bond = b < ni;
  const uint32_t t = bond ? list[b] : (uint32_t)s;
  const double xt = q.sx[t], yt = q.sy[t], zt = q.sz[t];
  double dx, dy, dz;
  (void)bond_sep(q.sx[s], q.sy[s], q.sz[s], xt, yt, zt, g, dx, dy, dz);
  const float X = bond ? (float)dx : 1e18f, Y = bond ? (float)dy : 1e18f;
  const float Z = bond ? (float)dz : 1e18f, r2 = (float)rc2;
  auto lane_f = [](float v, int m) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), m));
  };
  uint32_t lo = 0, hi = 0;  // bit m: bonded to member m
  float near = 3e38f;
  for (int m = ni - 1; m >= 0; --m) {
    const float ax = X - lane_f(X, m), ay = Y - lane_f(Y, m), az = Z - lane_f(Z, m);
    const float e = __builtin_fmaf(az, az, __builtin_fmaf(ay, ay, __builtin_fmaf(ax, ax, -r2)));
    near = fminf(near, __builtin_fabsf(e));  // (the member itself: r2)
    hi = __builtin_amdgcn_alignbit(hi, lo, 31);
    lo = __builtin_amdgcn_alignbit(lo, __float_as_uint(e), 31);
  }
  if (__any(bond & ((near <= band) | (unfolded && far_image(g, xt, yt, zt))))) {
    const double Lx = g.box[0], Ly = g.box[1], Lz = g.box[2];
    uint64_t adj = 0;
    for (int m = 0; m < ni; ++m) {
      const double x2 = __shfl(xt, m, 64), y2 = __shfl(yt, m, 64), z2 = __shfl(zt, m, 64);
      const bool in =
          exact_d2(x2, y2, z2, xt, yt, zt, Lx, Ly, Lz, 0.5 * Lx, 0.5 * Ly, 0.5 * Lz) < rc2;
      adj |= in ? 1ull << m : 0ull;
    }
    lo = (uint32_t)adj;
    hi = (uint32_t)(adj >> 32);
  }
  lo &= bond ? ~(b < 32 ? 1u << b : 0u) : 0u;
  hi &= bond ? ~(b >= 32 ? 1u << (b - 32) : 0u) : 0u;
  // over the members m of the mask (olo, ohi), with C the lane's common
  // neighbours: what m is bonded to in C, and the bonds counted from m's end
  auto sweep = [&](uint32_t& olo, uint32_t& ohi, uint32_t& rlo, uint32_t& rhi) {
    int deg = 0;
    for (int m = 0; m < ni; ++m) {
      const uint32_t of = bit_mask64(olo, ohi, m);
      const uint32_t ilo = (uint32_t)__builtin_amdgcn_readlane((int)lo, m) & lo & of;
      const uint32_t ihi = (uint32_t)__builtin_amdgcn_readlane((int)hi, m) & hi & of;
      deg += __popc(ilo) + __popc(ihi);
      rlo |= ilo;
      rhi |= ihi;
    }
    return deg;
  };
  uint32_t elo = 0, ehi = 0;  // members of C with a bond inside C
  const int deg = sweep(lo, hi, elo, ehi), nb = deg >> 1, v = __popc(elo) + __popc(ehi);
  int best = nb == 2 && v == 4 ? 1 : nb;
  // three or more edges on up to four members are connected
  const bool open = nb > 2 && v > 4;
  uint32_t remlo = open ? elo : 0u, remhi = open ? ehi : 0u;
  if (open) best = 0;
  while (__any((remlo | remhi) != 0)) {
    // the component of the lowest member left, grown within each sweep too
    uint32_t clo = remlo & (~remlo + 1), chi = remlo ? 0u : remhi & (~remhi + 1);
    bool grows = (clo | chi) != 0;
    while (__any(grows)) {
      const uint32_t before_lo = clo, before_hi = chi;
      (void)sweep(clo, chi, clo, chi);
      grows = (clo != before_lo || chi != before_hi) && (clo != remlo || chi != remhi);
    }
    const bool part = clo != elo || chi != ehi;
    int e2 = part ? 0 : deg;
    if (__any(part && (clo | chi))) {
      uint32_t unused_lo = 0, unused_hi = 0;
      const int some = sweep(clo, chi, unused_lo, unused_hi);
      e2 = part ? some : deg;
    }
    best = open && (e2 >> 1) > best ? e2 >> 1 : best;
    remlo &= ~clo;
    remhi &= ~chi;
  }
  const uint32_t code = pack_triplet(__popc(lo) + __popc(hi), nb, best);
  const uint32_t key = code << 6 | (uint32_t)b;  // (a count is at most 63: 26 bits and 6)
  int rank = 0;
  for (int m = 0; m < ni; ++m)
    rank += (uint32_t)__builtin_amdgcn_readlane((int)key, m) < key ? 1 : 0;
  const int c421 = __popcll(__ballot(bond && code == pack_triplet(4, 2, 1)));
  const int c422 = __popcll(__ballot(bond && code == pack_triplet(4, 2, 2)));
  const int c444 = __popcll(__ballot(bond && code == pack_triplet(4, 4, 4)));
  const int c666 = __popcll(__ballot(bond && code == pack_triplet(6, 6, 6)));
  const int32_t o = q.perm[s];
  if (bond) out.trip[(int64_t)o * out.max_nb + rank] = code;
  if (b == 0) {
    uint8_t lab = 0;
    if (ni == 12 && c421 == 12) lab = 1;
    else if (ni == 12 && c421 == 6 && c422 == 6) lab = 2;
    else if (ni == 14 && c666 == 8 && c444 == 6) lab = 3;
    out.label[o] = lab;
    out.nnb[o] = ni;
  }
}

// The bonds of the lane's particle, counted: the screen's candidates in turns
// of a column each.
__device__ inline int count_bonds(const BondScan& q, const Grid& g, double rc2, float r2s, int s,
                                  uint32_t* __restrict__ col) {
  const double xi = q.sx[s], yi = q.sy[s], zi = q.sz[s];
  Screen<kCnaQueue, false> screen(q, g, s, true, r2s, col);
  int found = 0;
  for (bool done = false; !done; screen.cnt = 0) {
    done = screen.run();
    for (int k = 0; k < screen.cnt; ++k) {
      const uint32_t t = col[k * kQPitch];
      double dx, dy, dz;
      found += bond_sep(xi, yi, zi, at32(q.sx, t), at32(q.sy, t), at32(q.sz, t), g, dx, dy, dz) < rc2;
    }
  }
  return found;
}

// A particle per lane: the screen, then the signatures with the wave's
// largest noted count as a constant (the pairs of neighbours grow with its
// square); particles with more candidates than a column holds, or with a pair
// of neighbours so close to the cutoff that only the exact test decides, are
// then taken one at a time by the whole wave.  What bounds it: vector
// instructions, 7750 per wave of 64 particles.  4 * 10^6 atoms of a
// polycrystal: 1029 us against 3492 us for a list in memory (1079) and one
// lane per particle with its masks in LDS (2413), whose loops over ragged
// lists and graphs kept most lanes waiting.
// Where many lanes have a full column and the capacity is no larger, nearly
// all of them have too many bonds for a signature: counted side by side first.
constexpr int kCountLanes = 16;  // a count costs about 13 particles' turns of the wave
constexpr int kCnaThreads = 256;
__global__ __launch_bounds__(kCnaThreads) __attribute__((amdgpu_waves_per_eu(3)))
void k_cna(BondScan q, int64_t n, int per, Grid g, double rc2, float r2s, float band, CnaOut out,
           const int32_t* __restrict__ outside, int32_t* __restrict__ maxcount) {
  __shared__ uint32_t queue[kCnaThreads / 64][kCnaQueue * kQPitch];
  __shared__ uint32_t lists[kCnaThreads / 64][64];
  const int lane = (int)threadIdx.x & 63;
  const int base = (int)(blockIdx.x * (kCnaThreads / 64) + (threadIdx.x >> 6)) * per;
  if (base >= n) return;
  const int s = base + lane;
  const bool ok = lane < per && s < n;
  uint32_t* const wq = queue[threadIdx.x >> 6];
  Screen<kCnaQueue, true> screen(q, g, s, ok, r2s, wq + lane);
  (void)screen.run();
  const int kept = screen.cnt;
  const bool mine = ok && kept < kCnaQueue;  // a full column has been written past its end
  const int c = mine ? kept : 0;
  const int cm = wave_max_nonneg(c);
  const bool unfolded = *outside != 0;
  int ni = -1;
  if (mine) {
    if (cm <= 12) ni = cna_lane<12>(q, g, rc2, band, s, c, wq + lane, out, unfolded);
    else if (cm <= 14) ni = cna_lane<14>(q, g, rc2, band, s, c, wq + lane, out, unfolded);
    else if (cm <= 18) ni = cna_lane<18>(q, g, rc2, band, s, c, wq + lane, out, unfolded);
    else if (cm <= 24) ni = cna_lane<24>(q, g, rc2, band, s, c, wq + lane, out, unfolded);
    else ni = cna_lane<kCnaQueue>(q, g, rc2, band, s, c, wq + lane, out, unfolded);
  }
  if (out.max_nb <= kCnaQueue && __popcll(__ballot(ok && !mine)) >= kCountLanes) {
    if (ok && !mine) {
      const int found = count_bonds(q, g, rc2, r2s, s, wq + lane);
      if (found > out.max_nb) {  // no triplets, no signature
        const int32_t o = q.perm[s];
        out.nnb[o] = ni = found;
        out.label[o] = 0;
      }
    }
  }
  int most = ni > 0 ? ni : 0;
  uint64_t todo = __ballot(ok && ni < 0);
  while (todo) {
    const int p = __builtin_ctzll(todo);
    todo &= todo - 1;
    const int cp = __shfl(kept, p, 64);
    uint32_t* const list = lists[threadIdx.x >> 6];
    const int nw = cp < kCnaQueue ? bonds_noted(q, g, rc2, base + p, cp, wq + p, list)
                                  : bonds_of(q, g, rc2, base + p, list);
    if (nw <= out.max_nb) {  // (of at most 64)
      cna_wave(q, g, rc2, band, base + p, nw, list, out, unfolded);
    } else if (lane == 0) {  // the list is incomplete: no triplets, no signature
      const int32_t o = q.perm[base + p];
      out.nnb[o] = nw;
      out.label[o] = 0;
    }
    most = nw > most ? nw : most;
  }
  most = wave_max_nonneg(most);
  if (lane == 0 && most > 0) atomicMax(maxcount, most);
}

hipError_t cna_signatures(const BondScan& q, int64_t n, const Grid& g, double rc2, int max_nb,
                          uint32_t* trip, int32_t* nnb, uint8_t* label, const int32_t* outside,
                          int32_t* maxcount, hipStream_t st) {
  const CnaOut out{trip, nnb, label, max_nb, max_nb % 4 == 0 && ((uintptr_t)trip & 15) == 0};
  // (what the FP32 pairs cannot decide is left to the exact test)
  const float band = screen_fits(g, sqrt(rc2)) ? 2e-6f * (float)rc2 : 3.4e38f;
  // Particles of a wave: fewer where waves of 64 would not fill the chip (four
  // SIMDs on each of 256 CUs) and most particles are expected to have a full
  // column, so that their turns one after another set the time (864 atoms with
  // 41 bonds 904 -> 163 us; with 19 bonds 64 lanes stay ahead, 79 against 121).
  const double sites = (double)n / (g.box[0] * g.box[1] * g.box[2]);
  const double expected = 4.19 * sites * rc2 * sqrt(rc2);
  int per = 64;
  while (expected > kCnaQueue && per > 8 && div_up(n, per) < 1024) per /= 2;
  const int64_t waves = div_up(n, per);
  hipLaunchKernelGGL(k_cna, dim3((unsigned)div_up(waves, kCnaThreads / 64)), dim3(kCnaThreads), 0,
                     st, q, n, per, g, rc2, screen_r2(g.box, g.side, rc2), band, out, outside,
                     maxcount);
  return hipGetLastError();
}

}  // namespace mdpl
