// Dense layers of the learned potential on the matrix cores (BF16 inputs,
// FP32 accumulation): y = w3 . silu(W2 silu(W1 g + b1) + b2) + b3 with the
// standardised features g = (G - mu) / sd zero-padded to 32, silu(z) = z
// sigmoid(z), and E = e_mean + e_sd y.
//
// One wave handles 16 atoms at a time.  v_mfma_f32_16x16x32_bf16 takes lane
// l's A row l%16 and B column l%16 with K = 8(l/16)..+7 and returns rows
// 4(l/16)..+3 of column l%16.  The weights lie in LDS, W2 and W1 also
// transposed for the input gradient (dh1 = dz2 W2 and dg = dz1 W1);
// activations change layout through BF16 LDS rows of 72 halfwords, whose
// 16-byte reads and 2-byte writes are free of bank conflicts.  Training also
// forms the loss L = sum (y - t)^2 / B over a batch of B atoms and the weight
// gradients, sums over the atoms: the workgroup's four waves leave the
// operands of their 64 atoms in LDS with the atoms along K, and each wave
// forms a quarter of every gradient.  Partials are written per workgroup and
// reduced in a fixed order.
#include <math.h>

#include "device_util.h"
#include "internal.h"
#include "mlp_args.h"

namespace mdpl {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned u32x4;
typedef __attribute__((__vector_size__(2 * sizeof(unsigned)))) unsigned u32x2;
// 16-byte loads of arrays that are only known to be aligned to their elements
struct __attribute__((packed, aligned(4))) f32x4_a4 { f32x4 v; };
struct __attribute__((packed, aligned(2))) u32x4_a2 { u32x4 v; };

constexpr int kMlpThreads = 256;
constexpr int kNIn = 24, kNPad = 32, kNH = 64;
// packed FP32 parameter vector: W1 [64][32] | b1 | W2 [64][64] | b2 | w3 | b3
constexpr int kOffW1 = 0, kOffB1 = 2048, kOffW2 = 2112, kOffB2 = 6208, kOffW3 = 6272, kOffB3 = 6336;
constexpr int kNParam = 6337;

__device__ __forceinline__ unsigned short f2bf(float f) {
  unsigned u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);  // round to nearest even (finite inputs)
  return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float bf2f(unsigned short h) { return __uint_as_float((unsigned)h << 16); }

// Two values to BF16, round to nearest even (v_cvt_pk_bf16_f32), a below b
__device__ __forceinline__ unsigned pack2(float a, float b) {
  return __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2{a, b}), bf16x2));
}
__device__ __forceinline__ u32x4 pack8(const float v[8]) {
  return u32x4{pack2(v[0], v[1]), pack2(v[2], v[3]), pack2(v[4], v[5]), pack2(v[6], v[7])};
}
__device__ __forceinline__ bf16x8 frag(const unsigned short* p) {  // 16-byte aligned LDS
  return __builtin_bit_cast(bf16x8, *(const u32x4*)p);
}

// sigmoid with the hardware reciprocal (about 1 ulp; the network's BF16
// operands dominate its error)
__device__ __forceinline__ float sigm(float z) { return __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }

// Sum over the 16 lanes of a DPP row (the lanes 16 g .. 16 g + 15): the
// quads by lane ^ 1 and lane ^ 2, then the row's four quad sums by
// rotations of 4 and 8 lanes.  Every lane receives the row sum; lanes of
// quads 0 and 2 and of quads 1 and 3 pair the quad sums differently, so the
// two groups can differ in the last bit.
__device__ __forceinline__ float row16_sum(float v) {
  v += dpp_move<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp_move<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp_move<0x124>(v);  // row_ror:4
  v += dpp_move<0x128>(v);  // row_ror:8
  return v;
}

// The raw features 8 grp .. 8 grp + 7 of row 16 tile + col (zero past the
// 24 features); ok: the row exists.
__device__ __forceinline__ void load_features(const MlpArgs& a, int64_t tile, int64_t ntiles,
                                              int col, int grp, float g[8], bool& ok) {
  const int64_t ra = tile * 16 + col;
  ok = tile < ntiles && ra < a.n;
  f32x4 lo = {0, 0, 0, 0}, hi = {0, 0, 0, 0};
  if (ok && grp < 3) {
    const int64_t ia = a.index ? (int64_t)a.index[ra] : ra;
    const f32x4_a4* p = (const f32x4_a4*)(a.G + ia * kNIn + 8 * grp);
    lo = p[0].v;
    hi = p[1].v;
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    g[k] = lo[k];
    g[4 + k] = hi[k];
  }
}

// Rows of 64 (or, W1, 32) BF16 in LDS
constexpr int kPitch = 72, kPitch1 = 40;

// The weights of a workgroup: rows n (outputs), and transposed rows k.
struct MlpLds {
  unsigned short w1[kNH][kPitch1], w2[kNH][kPitch];
  unsigned short w2t[kNH][kPitch], w1t[kNPad][kPitch];
  unsigned short rows[kMlpThreads / 64][16][kPitch];  // a wave's activations, row-major
};

// Thread t loads 16 bytes of row t % 64 at a time (transposed writes by
// consecutive lanes to consecutive halfwords).
template <bool W1T>
__device__ __forceinline__ void stage_weights(const MlpArgs& a, bool grad, MlpLds& m) {
  const int n = threadIdx.x & 63, q = threadIdx.x >> 6;
  const u32x4 v1 = ((const u32x4_a2*)(a.w1 + n * kNPad + 8 * q))->v;
  u32x4 v2[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) v2[h] = ((const u32x4_a2*)(a.w2 + n * kNH + 8 * (q + 4 * h)))->v;
  *(u32x4*)&m.w1[n][8 * q] = v1;
#pragma unroll
  for (int h = 0; h < 2; ++h) *(u32x4*)&m.w2[n][8 * (q + 4 * h)] = v2[h];
  if (grad) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (W1T) m.w1t[8 * q + i][n] = (unsigned short)(v1[i / 2] >> (16 * (i & 1)));
#pragma unroll
      for (int h = 0; h < 2; ++h)
        m.w2t[8 * (q + 4 * h) + i][n] = (unsigned short)(v2[h][i / 2] >> (16 * (i & 1)));
    }
  }
  __syncthreads();
}

// Accumulator tile nt of a wave (rows 4 grp + r of column nt*16 + col) to its
// BF16 rows; returns the four values packed in row order.
__device__ __forceinline__ u32x2 put_tile(unsigned short (*S)[kPitch], int nt, int col, int grp,
                                          const f32x4& v) {
  const u32x2 p = {pack2(v[0], v[1]), pack2(v[2], v[3])};
#pragma unroll
  for (int r = 0; r < 4; ++r)
    S[4 * grp + r][nt * 16 + col] = (unsigned short)(p[r >> 1] >> (16 * (r & 1)));
  return p;
}

// What a lane keeps of the parameters: columns nt*16 + col.
struct MlpCols {
  float b1[4], b2[4], w3[4], b3;
  float mu8[8], isd8[8];  // of its eight layer-1 inputs 8 grp + k
};
__device__ __forceinline__ MlpCols mlp_cols(const MlpArgs& a, int col, int grp) {
  MlpCols c;
#pragma unroll
  for (int nt = 0; nt < 4; ++nt) {
    c.b1[nt] = a.b1[nt * 16 + col];
    c.b2[nt] = a.b2[nt * 16 + col];
    c.w3[nt] = bf2f(a.w3[nt * 16 + col]);
  }
  c.b3 = a.b3[0];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int f = 8 * grp + k < kNIn ? 8 * grp + k : 0;
    c.mu8[k] = a.mu[f];
    c.isd8[k] = 1.0f / a.sd[f];
  }
  return c;
}

// Layer 1 from the standardised features A1: h1 and the derivative of its
// silu (d1), h1 to the wave's rows and, packed along the rows, to hp.
__device__ __forceinline__ void layer1(const MlpLds& m, unsigned short (*S)[kPitch],
                                       const MlpCols& c, int col, int grp, const u32x4& A1,
                                       f32x4 (&d1)[4], u32x2 (&hp)[4]) {
#pragma unroll
  for (int nt = 0; nt < 4; ++nt) {
    const f32x4 z = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
        __builtin_bit_cast(bf16x8, A1), frag(&m.w1[nt * 16 + col][8 * grp]), f32x4{0, 0, 0, 0}, 0, 0, 0);
    f32x4 h;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float zz = z[r] + c.b1[nt], sg = sigm(zz);
      h[r] = zz * sg;
      d1[nt][r] = sg * (1.0f + zz * (1.0f - sg));
    }
    hp[nt] = put_tile(S, nt, col, grp, h);
  }
}

// acc[nt] = rows of S times W^T (W: 64 rows of pitch kPitch), NT column tiles
template <int NT>
__device__ __forceinline__ void mul64(unsigned short (*S)[kPitch], const unsigned short (*W)[kPitch],
                                      int col, int grp, f32x4 (&acc)[NT]) {
  const bf16x8 A0 = frag(&S[col][8 * grp]), A1 = frag(&S[col][32 + 8 * grp]);
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A0, frag(&W[nt * 16 + col][8 * grp]),
                                                      f32x4{0, 0, 0, 0}, 0, 0, 0);
    acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A1, frag(&W[nt * 16 + col][32 + 8 * grp]),
                                                      acc[nt], 0, 0, 0);
  }
}

// Layer 2 and the output y of rows 4 grp + r: z2 and its sigmoid.
__device__ __forceinline__ void layer2(const MlpLds& m, unsigned short (*S)[kPitch],
                                       const MlpCols& c, int col, int grp, f32x4 (&z2)[4],
                                       f32x4 (&sg)[4], float (&y)[4]) {
  mul64(S, m.w2, col, grp, z2);
#pragma unroll
  for (int r = 0; r < 4; ++r) y[r] = 0.0f;
#pragma unroll
  for (int nt = 0; nt < 4; ++nt)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      z2[nt][r] += c.b2[nt];
      sg[nt][r] = sigm(z2[nt][r]);
      y[r] += c.w3[nt] * z2[nt][r] * sg[nt][r];
    }
  // sum over the 16 columns held by the lanes of this group
#pragma unroll
  for (int r = 0; r < 4; ++r) y[r] = row16_sum(y[r]) + c.b3;
}

// Energies and, with dEdG, the input gradients.  A tile costs about 600 vector
// instructions (64 of them exponentials and reciprocals) against 24 matrix
// ones, so that vector issue bounds it: N = 262144 40 -> 32 us against
// fragments of the transposed weights gathered from memory by 2-byte loads
// and held in registers, and roundings and layout changes done value by value
// in FP32; N = 4096, where the loads before the first tile counted, 10.3 ->
// 5.4 us.
__global__ __launch_bounds__(kMlpThreads) void k_mlp_eval(MlpArgs a) {
  __shared__ __attribute__((aligned(16))) MlpLds m;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int col = lane & 15, grp = lane >> 4;
  unsigned short(*S)[kPitch] = m.rows[wv];
  const bool want_grad = a.dEdG != nullptr;
  const int64_t ntiles = (a.n + 15) >> 4;
  const int64_t wave_id = (int64_t)blockIdx.x * (kMlpThreads / 64) + wv;
  const int64_t nwaves = (int64_t)gridDim.x * (kMlpThreads / 64);
  float gnext[8];
  bool oknext = false;
  load_features(a, wave_id, ntiles, col, grp, gnext, oknext);
  const MlpCols c = mlp_cols(a, col, grp);
  float sc[2];  // of the features col and 16 + col of the gradients
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int f = j * 16 + col;
    sc[j] = f < kNIn ? a.e_sd * (1.0f / a.sd[f]) : 0.0f;
  }
  stage_weights<true>(a, want_grad, m);
  for (int64_t tile = wave_id; tile < ntiles; tile += nwaves) {
    const int64_t r0 = tile * 16;
    // A fragment = standardised features of row r0 + col; the next tile's
    // raw ones are loaded while this one is computed
    float gv[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) gv[k] = oknext && grp < 3 ? (gnext[k] - c.mu8[k]) * c.isd8[k] : 0.0f;
    load_features(a, tile + nwaves, ntiles, col, grp, gnext, oknext);
    // keep those loads here, a tile ahead of their use
    asm volatile("" ::: "memory");
    f32x4 d1[4], z2[4], sg[4];
    u32x2 hp[4];
    float y[4];
    layer1(m, S, c, col, grp, pack8(gv), d1, hp);
    wave_lds_sync();
    layer2(m, S, c, col, grp, z2, sg, y);
    if (col == 0 && a.energy) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (r0 + 4 * grp + r < a.n) a.energy[r0 + 4 * grp + r] = a.e_mean + a.e_sd * y[r];
    }
    wave_lds_sync();
    if (!want_grad) continue;
    // dz2 = w3 silu'(z2), dh1 = dz2 W2, dz1 = dh1 silu'(z1), dg = dz1 W1
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
      f32x4 d;
#pragma unroll
      for (int r = 0; r < 4; ++r)
        d[r] = c.w3[nt] * sg[nt][r] * (1.0f + z2[nt][r] * (1.0f - sg[nt][r]));
      put_tile(S, nt, col, grp, d);
    }
    wave_lds_sync();
    f32x4 dz1[4];
    mul64(S, m.w2t, col, grp, dz1);
    wave_lds_sync();
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
#pragma unroll
      for (int r = 0; r < 4; ++r) dz1[nt][r] *= d1[nt][r];
      put_tile(S, nt, col, grp, dz1[nt]);
    }
    wave_lds_sync();
    f32x4 dg[2];
    mul64(S, m.w1t, col, grp, dg);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int f = j * 16 + col;
      if (f < kNIn) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int64_t row = r0 + 4 * grp + r;
          if (row < a.n) a.dEdG[row * kNIn + f] = dg[j][r] * sc[j];
        }
      }
    }
    wave_lds_sync();
  }
}

// The four rows 4 grp .. 4 grp + 3 that the lane's wave computes of column n
// of an operand, packed, to LDS rows along the atoms.
typedef unsigned short MlpCross[kPitch];
__device__ __forceinline__ void put_cross(MlpCross* X, int n, int wv, int grp, const u32x2& p) {
  *(u32x2*)&X[n][16 * wv + 4 * grp] = p;
}

// Loss and weight gradients of a batch.  At batch 4096 (64 workgroups, one
// tile per wave) latency bounds it: every load is issued before the first
// use, an atom's target is standardised by one lane of a quad, and a wave
// holds a quarter of the gradients (24 accumulators instead of 96 per lane,
// and no sum over the waves): 14.7 -> 8.1 us.
__global__ __launch_bounds__(kMlpThreads) void k_mlp_train(MlpArgs a) {
  __shared__ __attribute__((aligned(16))) MlpLds m;
  // operands of the weight gradients, column-major: 64 atoms along each row
  __shared__ __attribute__((aligned(16))) MlpCross xh1[kNH], xdz2[kNH], xdz1[kNH], xg[kNPad];
  constexpr int kWaves = kMlpThreads / 64, kVec = 3 * kNH + 2;
  __shared__ float vec[kWaves][kVec];  // bias and w3 gradients, db3, loss
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int col = lane & 15, grp = lane >> 4;
  unsigned short(*S)[kPitch] = m.rows[wv];
  const int64_t ntiles = (a.n + 15) >> 4;
  // a lane's features, and the target of row 4 grp + col % 4
  float gnext[8];
  bool oknext = false;
  double tnext = 0.0;
  auto load = [&](int64_t tile) {
    load_features(a, tile, ntiles, col, grp, gnext, oknext);
    const int64_t row = tile * 16 + 4 * grp + (col & 3);
    if (row < a.n) tnext = a.target[a.index ? (int64_t)a.index[row] : row];
  };
  load((int64_t)blockIdx.x * kWaves + wv);
  const MlpCols c = mlp_cols(a, col, grp);
  stage_weights<false>(a, true, m);

  f32x4 gW2[4], gW1[2];  // tile row wv of dW2 and dW1
  float gb1[4] = {0, 0, 0, 0}, gb2[4] = {0, 0, 0, 0}, gw3[4] = {0, 0, 0, 0};
  float gb3 = 0.0f, loss = 0.0f;
#pragma unroll
  for (int j = 0; j < 4; ++j) gW2[j] = f32x4{0, 0, 0, 0};
  gW1[0] = gW1[1] = f32x4{0, 0, 0, 0};

  for (int64_t base = (int64_t)blockIdx.x * kWaves; base < ntiles; base += (int64_t)gridDim.x * kWaves) {
    const int64_t r0 = (base + wv) * 16;
    float gv[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) gv[k] = oknext && grp < 3 ? (gnext[k] - c.mu8[k]) * c.isd8[k] : 0.0f;
    // the target: the atom's energy standardised with the network's e_mean, e_sd
    const float tq = (float)((tnext - (double)a.e_mean) / (double)a.e_sd);
    const float t[4] = {dpp_move<0x00>(tq), dpp_move<0x55>(tq), dpp_move<0xAA>(tq), dpp_move<0xFF>(tq)};
    load(base + wv + (int64_t)gridDim.x * kWaves);
    asm volatile("" ::: "memory");
    const u32x4 A1 = pack8(gv);
#pragma unroll
    for (int k = 0; k < 8; ++k)
      xg[8 * grp + k][16 * wv + col] = (unsigned short)(A1[k / 2] >> (16 * (k & 1)));
    f32x4 d1[4], z2[4], sg[4];
    u32x2 hp[4];
    float y[4], dy[4];
    layer1(m, S, c, col, grp, A1, d1, hp);
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) put_cross(xh1, nt * 16 + col, wv, grp, hp[nt]);
    wave_lds_sync();
    layer2(m, S, c, col, grp, z2, sg, y);
    wave_lds_sync();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float diff = r0 + 4 * grp + r < a.n ? y[r] - t[r] : 0.0f;
      dy[r] = 2.0f * diff * a.inv_batch;
      if (col == 0) loss += diff * diff * a.inv_batch;
    }
    // dz2 = dy w3 silu'(z2), dw3 = sum dy h2, db2 = sum dz2, db3 = sum dy
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
      f32x4 d;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float zz = z2[nt][r], s = sg[nt][r];
        d[r] = dy[r] * c.w3[nt] * s * (1.0f + zz * (1.0f - s));
        gb2[nt] += d[r];
        gw3[nt] += dy[r] * zz * s;
      }
      put_cross(xdz2, nt * 16 + col, wv, grp, put_tile(S, nt, col, grp, d));
    }
    if (col == 0) gb3 += dy[0] + dy[1] + dy[2] + dy[3];
    wave_lds_sync();
    // dz1 = (dz2 W2) silu'(z1), db1 = sum dz1
    f32x4 dz1[4];
    mul64(S, m.w2t, col, grp, dz1);
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        dz1[nt][r] *= d1[nt][r];
        gb1[nt] += dz1[nt][r];
      }
      put_cross(xdz1, nt * 16 + col, wv, grp,
                u32x2{pack2(dz1[nt][0], dz1[nt][1]), pack2(dz1[nt][2], dz1[nt][3])});
    }
    __syncthreads();
    // dW2 = dz2^T h1, dW1 = dz1^T g over the workgroup's 64 atoms
#pragma unroll
    for (int kc = 0; kc < 2; ++kc) {
      const int o = kc * 32 + 8 * grp;
      const bf16x8 A2 = frag(&xdz2[wv * 16 + col][o]), Ag = frag(&xdz1[wv * 16 + col][o]);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        gW2[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A2, frag(&xh1[j * 16 + col][o]), gW2[j], 0, 0, 0);
#pragma unroll
      for (int j = 0; j < 2; ++j)
        gW1[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Ag, frag(&xg[j * 16 + col][o]), gW1[j], 0, 0, 0);
    }
    __syncthreads();
  }

  float* __restrict__ out = a.partial + (int64_t)blockIdx.x * (kNParam + 1);
  // accumulator tile (wv, j): rows 4 grp + r of column j*16 + col
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int n = wv * 16 + 4 * grp + r;
#pragma unroll
    for (int j = 0; j < 4; ++j) out[kOffW2 + n * kNH + j * 16 + col] = gW2[j][r];
#pragma unroll
    for (int j = 0; j < 2; ++j) out[kOffW1 + n * kNPad + j * 16 + col] = gW1[j][r];
  }
  // column sums over the 4 lane groups, then the waves in order
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float v1 = gb1[i], v2 = gb2[i], v3 = gw3[i];
    v1 += __shfl_xor(v1, 16, 64);
    v1 += __shfl_xor(v1, 32, 64);
    v2 += __shfl_xor(v2, 16, 64);
    v2 += __shfl_xor(v2, 32, 64);
    v3 += __shfl_xor(v3, 16, 64);
    v3 += __shfl_xor(v3, 32, 64);
    if (grp == 0) {
      vec[wv][i * 16 + col] = v1;
      vec[wv][kNH + i * 16 + col] = v2;
      vec[wv][2 * kNH + i * 16 + col] = v3;
    }
  }
  // db3 and the loss lie in lanes 0, 16, 32 and 48
  gb3 += __shfl_xor(gb3, 16, 64);
  gb3 += __shfl_xor(gb3, 32, 64);
  loss += __shfl_xor(loss, 16, 64);
  loss += __shfl_xor(loss, 32, 64);
  if (lane == 0) {
    vec[wv][3 * kNH] = gb3;
    vec[wv][3 * kNH + 1] = loss;
  }
  __syncthreads();
  if (threadIdx.x < kVec) {
    const int k = threadIdx.x;
    float s = vec[0][k];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) s += vec[w][k];
    const int at = k < kNH ? kOffB1 + k
                           : (k < 2 * kNH ? kOffB2 + k - kNH
                                          : (k < 3 * kNH ? kOffW3 + k - 2 * kNH : kOffB3 + k - 3 * kNH));
    out[at] = s;
  }
}

hipError_t mlp_eval(const MlpArgs& a, hipStream_t st) {
  // two waves per SIMD that each take many tiles, so that the weights a
  // workgroup stages first serve ~32 tiles at N = 262144 (512 blocks 32 us,
  // 1024 with room for four waves per SIMD 34 us)
  int64_t tiles = (a.n + 15) >> 4;
  int64_t blocks = (tiles + 3) / 4;
  if (blocks > 512) blocks = 512;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_mlp_eval, dim3((unsigned)blocks), dim3(kMlpThreads), 0, st, a);
  return hipGetLastError();
}

int mlp_train_blocks(int64_t n) {
  int64_t tiles = (n + 15) >> 4;
  int64_t blocks = (tiles + 3) / 4;
  if (blocks > 256) blocks = 256;
  if (blocks < 1) blocks = 1;
  return (int)blocks;
}

int mlp_train_waves(int64_t n) { return mlp_train_blocks(n) * (kMlpThreads / 64); }

hipError_t mlp_train_grad(const MlpArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(k_mlp_train, dim3((unsigned)mlp_train_blocks(a.n)), dim3(kMlpThreads), 0, st,
                     a);
  return hipGetLastError();
}

// out[k] = sum over workgroups of partial[w][k], k < kNParam + 1, fixed
// order: four threads per k take consecutive quarters of the partials, their
// sums are added in order.  What bounds it is the latency of the loads: at
// batch 4096 (64 partials) every thread has its 16 loads in flight at once
// and 100 workgroups run, 57 -> 3.6 us against one thread per k adding one
// partial per wave (256) in a serial chain of loads.
constexpr int kSumCols = 64, kSumParts = 4;
__global__ __launch_bounds__(kSumCols* kSumParts) void k_sum_partials(
    const float* __restrict__ partial, int nparts, float* __restrict__ out) {
  __shared__ float sh[kSumParts][kSumCols];
  const int c = threadIdx.x % kSumCols, q = threadIdx.x / kSumCols;
  const int k = blockIdx.x * kSumCols + c;
  const int per = (nparts + kSumParts - 1) / kSumParts;
  const int w0 = q * per, w1 = w0 + per < nparts ? w0 + per : nparts;
  float s = 0.0f;
  if (k <= kNParam) {
#pragma unroll 16
    for (int w = w0; w < w1; ++w) s += partial[(int64_t)w * (kNParam + 1) + k];
  }
  sh[q][c] = s;
  __syncthreads();
  if (q == 0 && k <= kNParam) out[k] = (sh[0][c] + sh[1][c]) + (sh[2][c] + sh[3][c]);
}

hipError_t mlp_sum_partials(const float* partial, int nparts, float* out, hipStream_t st) {
  hipLaunchKernelGGL(k_sum_partials, dim3((kNParam + kSumCols) / kSumCols),
                     dim3(kSumCols * kSumParts), 0, st, partial, nparts, out);
  return hipGetLastError();
}

// Adam (bias-corrected) on the FP32 master vector, then the bf16 copies of
// the three weight matrices.  W1 columns >= 24 stay zero.
__global__ void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, float lr, float b1, float b2, float eps, float c1,
                       float c2, unsigned short* __restrict__ w1, unsigned short* __restrict__ w2,
                       unsigned short* __restrict__ w3) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= kNParam) return;
  float gk = g[k];
  if (k < kOffB1 && (k % kNPad) >= kNIn) gk = 0.0f;
  const float mk = b1 * m[k] + (1.0f - b1) * gk;
  const float vk = b2 * v[k] + (1.0f - b2) * gk * gk;
  m[k] = mk;
  v[k] = vk;
  float pk = p[k] - lr * (mk / c1) / (sqrtf(vk / c2) + eps);
  if (k < kOffB1 && (k % kNPad) >= kNIn) pk = 0.0f;
  p[k] = pk;
  if (k < kOffB1) w1[k] = f2bf(pk);
  else if (k >= kOffW2 && k < kOffB2) w2[k - kOffW2] = f2bf(pk);
  else if (k >= kOffW3 && k < kOffB3) w3[k - kOffW3] = f2bf(pk);
}

hipError_t adam_step(float* p, const float* g, float* m, float* v, float lr, float b1, float b2,
                     float eps, int t, unsigned short* w1, unsigned short* w2, unsigned short* w3,
                     hipStream_t st) {
  const float c1 = 1.0f - powf(b1, (float)t), c2 = 1.0f - powf(b2, (float)t);
  hipLaunchKernelGGL(k_adam, dim3((kNParam + 255) / 256), dim3(256), 0, st, p, g, m, v, lr, b1, b2,
                     eps, c1, c2, w1, w2, w3);
  return hipGetLastError();
}

// BF16 copies of the weight matrices from the packed FP32 parameters
// (round to nearest even, as after every Adam step).
__global__ void k_bf16_weights(const float* __restrict__ p, unsigned short* __restrict__ w1,
                               unsigned short* __restrict__ w2, unsigned short* __restrict__ w3) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= kNParam) return;
  const float pk = p[k];
  if (k < kOffB1) w1[k] = f2bf(pk);
  else if (k >= kOffW2 && k < kOffB2) w2[k - kOffW2] = f2bf(pk);
  else if (k >= kOffW3 && k < kOffB3) w3[k - kOffW3] = f2bf(pk);
}

hipError_t bf16_weights(const float* p, unsigned short* w1, unsigned short* w2, unsigned short* w3,
                        hipStream_t st) {
  hipLaunchKernelGGL(k_bf16_weights, dim3((kNParam + 255) / 256), dim3(256), 0, st, p, w1, w2, w3);
  return hipGetLastError();
}

// Standardisation statistics of the training set, FP64 in a fixed order:
// means, then the mean squared deviations from them (two passes, as the
// population standard deviation is defined).  Column c < 24 is feature c of
// G (n x 24 floats), column 24 the energy.  Pass 1 (ref null): per-block
// sums; pass 2 (ref = the means): per-block sums of squared deviations.
constexpr int kStdCols = kNIn + 1;
__global__ __launch_bounds__(256) void k_std_partials(const float* __restrict__ G,
                                                      const double* __restrict__ e, int64_t n,
                                                      const double* __restrict__ ref,
                                                      double* __restrict__ part) {
  __shared__ double sh[4];
  const int64_t per = (n + gridDim.x - 1) / gridDim.x;
  const int64_t r0 = (int64_t)blockIdx.x * per, r1 = r0 + per < n ? r0 + per : n;
  for (int c = 0; c < kStdCols; ++c) {
    const double m = ref ? ref[c] : 0.0;
    double acc = 0.0;
    for (int64_t r = r0 + threadIdx.x; r < r1; r += blockDim.x) {
      const double v = c < kNIn ? (double)G[r * kNIn + c] : e[r];
      acc += ref ? (v - m) * (v - m) : v;
    }
    const double t = block_sum256(acc, sh);
    if (threadIdx.x == 0) part[(int64_t)blockIdx.x * kStdCols + c] = t;
  }
}

// Sums the partials of every column in block order; out[c] = sum / n.  With
// fin: the feature spreads sqrt(.) + 1e-6 to sd (float), the means to mu,
// the energy's mean and spread sqrt(.) + 1e-12 to e_stats.
__global__ __launch_bounds__(64) void k_std_reduce(const double* __restrict__ part, int nb,
                                                   int64_t n, double* __restrict__ out, bool fin,
                                                   const double* __restrict__ mean, float* mu,
                                                   float* sd, double* e_stats) {
  const int c = threadIdx.x;
  if (c >= kStdCols) return;
  double s = 0.0;
  for (int b = 0; b < nb; ++b) s += part[(int64_t)b * kStdCols + c];
  const double v = s / (double)n;
  out[c] = v;
  if (!fin) return;
  if (c < kNIn) {
    mu[c] = (float)mean[c];
    sd[c] = (float)(sqrt(v) + 1e-6);
  } else {
    e_stats[0] = mean[c];
    e_stats[1] = sqrt(v) + 1e-12;
  }
}

hipError_t mlp_standardise(const float* G, const double* e, int64_t n, float* mu, float* sd,
                           double* e_stats, double* scratch, hipStream_t st) {
  const int nb = kStdBlocks;
  double* part = scratch;
  double* mean = scratch + (int64_t)nb * kStdCols;
  double* var = mean + kStdCols;
  hipLaunchKernelGGL(k_std_partials, dim3(nb), dim3(256), 0, st, G, e, n, nullptr, part);
  hipLaunchKernelGGL(k_std_reduce, dim3(1), dim3(64), 0, st, part, nb, n, mean, false, nullptr,
                     nullptr, nullptr, nullptr);
  hipLaunchKernelGGL(k_std_partials, dim3(nb), dim3(256), 0, st, G, e, n, mean, part);
  hipLaunchKernelGGL(k_std_reduce, dim3(1), dim3(64), 0, st, part, nb, n, var, true, mean, mu, sd,
                     e_stats);
  return hipGetLastError();
}

// ------------------------------------------------------------ reductions
// partials[b] = sum of v over block b (FP64, fixed order).
__global__ __launch_bounds__(256) void k_sum_f32(const float* __restrict__ v, int64_t n,
                                                 double* __restrict__ partials) {
  __shared__ double sh[4];
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const double t = block_sum256(i < n ? (double)v[i] : 0.0, sh);
  if (threadIdx.x == 0) partials[blockIdx.x] = t;
}

hipError_t sum_f32(const float* v, int64_t n, double* partials, hipStream_t st, int* nblocks_out) {
  const unsigned nb = (unsigned)div_up(n, 256);
  *nblocks_out = (int)nb;
  hipLaunchKernelGGL(k_sum_f32, dim3(nb), dim3(256), 0, st, v, n, partials);
  return hipGetLastError();
}

// partials[2b] = sum |f - g|^2, partials[2b+1] = sum |g|^2 over block b.
__global__ __launch_bounds__(256) void k_force_diff(const float* __restrict__ fx,
                                                    const float* __restrict__ fy,
                                                    const float* __restrict__ fz,
                                                    const double* __restrict__ gx,
                                                    const double* __restrict__ gy,
                                                    const double* __restrict__ gz, int64_t n,
                                                    double* __restrict__ partials) {
  __shared__ double sh[4];
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  double d = 0.0, r = 0.0;
  if (i < n) {
    const double a = (double)fx[i] - gx[i], b = (double)fy[i] - gy[i], c = (double)fz[i] - gz[i];
    d = a * a + b * b + c * c;
    r = gx[i] * gx[i] + gy[i] * gy[i] + gz[i] * gz[i];
  }
  const double td = block_sum256(d, sh);
  __syncthreads();
  const double tr = block_sum256(r, sh);
  if (threadIdx.x == 0) {
    partials[2 * blockIdx.x] = td;
    partials[2 * blockIdx.x + 1] = tr;
  }
}

hipError_t force_diff(const float* fx, const float* fy, const float* fz, const double* gx,
                      const double* gy, const double* gz, int64_t n, double* partials,
                      hipStream_t st, int* nblocks_out) {
  const unsigned nb = (unsigned)div_up(n, 256);
  *nblocks_out = (int)nb;
  hipLaunchKernelGGL(k_force_diff, dim3(nb), dim3(256), 0, st, fx, fy, fz, gx, gy, gz, n,
                     partials);
  return hipGetLastError();
}

}  // namespace mdpl
