// Learned warm start: per-primitive features, a 16-128-128-11 GELU network
// run on bfloat16 matrix cores with float32 accumulation, its training
// (backward products, bias and GELU gradients, Adam on float32 master weights),
// and the warm-start application with its fallback to the plain allocation.
//
// Products use v_mfma_f32_16x16x16_bf16 with operands rounded from float32
// (nearest even).  Operand tiles: lane l holds A[l % 16][4 (l / 16) + j] and
// B[4 (l / 16) + j][l % 16]; results D[4 (l / 16) + j][l % 16], j = 0..3.
// Sums over the batch (weight gradients) are split into 512-row partial sums
// that are added in a fixed order.
#include <algorithm>
#include <cmath>

#include "common.h"
#include "devmath.h"

namespace gve {
namespace {

typedef short short4v __attribute__((ext_vector_type(4)));
typedef float float4v __attribute__((ext_vector_type(4)));

__device__ inline unsigned short f2bf(float x) {
  uint32_t u = __float_as_uint(x);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (unsigned short)0x7fc0;  // NaN
  u += 0x7fffu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}

__device__ inline float gelu_f(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }

__device__ inline float gelu_grad_f(float z) {
  return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) +
         z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

// ---- network layout --------------------------------------------------------------
//
// Flat weights (float32 master copy): W1 [128][16], b1, W2 [128][128], b2,
// W3 [11][128], b3.
constexpr int kIn = kMlpIn, kHid = kMlpHid, kOut = kMlpOut;
constexpr int oW1 = 0, oB1 = oW1 + kHid * kIn, oW2 = oB1 + kHid, oB2 = oW2 + kHid * kHid,
              oW3 = oB2 + kHid, oB3 = oW3 + kOut * kHid;
static_assert(oB3 + kOut == GVE_MLP_NWEIGHT, "weight layout");
constexpr int kHT = kHid / 16;  // 16-wide tiles of a hidden layer

// Everything the matrix cores read is kept as whole operand tiles: 64 lanes x
// 4 bfloat16 (512 contiguous bytes), lane l holding entries
// (4 (l / 16) + j, l % 16), j = 0..3, of a 16 x 16 block.  That is the layout
// results come out in, and, read as [reduction index][other index], the layout
// of both operands, so a product of two stored results over their shared rows
// (the weight gradients, over the batch) needs neither a transpose nor LDS.
constexpr int kFrag = 256;  // bfloat16 per tile

// Weight tiles as B operands, [reduction index][output index]:
constexpr int fW1 = 0;                          // x  -> z1 : [nt]
constexpr int fW2 = fW1 + kHT * kFrag;          // h1 -> z2 : [nt][kt]
constexpr int fW2t = fW2 + kHT * kHT * kFrag;   // dz2 -> dh1 : [nt][kt]
constexpr int fW3 = fW2t + kHT * kHT * kFrag;   // h2 -> y : [kt], outputs padded to 16
constexpr int fW3t = fW3 + kHT * kFrag;         // dy -> dh2 : [nt], reduction padded to 16
static_assert(fW3t + kHT * kFrag == kMlpFragElems, "weight tiles");

__device__ inline int frag_at(int k, int n) { return (((k & 15) >> 2) * 16 + (n & 15)) * 4 + (k & 3); }

// bfloat16 copies of flat weight i in the tiles that hold it.
__device__ inline void store_weight_tiles(int i, float w, unsigned short* __restrict__ wf) {
  const unsigned short b = f2bf(w);
  if (i < oB1) {
    const int n = i / kIn, k = i % kIn;
    wf[fW1 + (n >> 4) * kFrag + frag_at(k, n)] = b;
  } else if (i >= oW2 && i < oB2) {
    const int r = (i - oW2) / kHid, c = (i - oW2) % kHid;
    wf[fW2 + ((r >> 4) * kHT + (c >> 4)) * kFrag + frag_at(c, r)] = b;
    wf[fW2t + ((c >> 4) * kHT + (r >> 4)) * kFrag + frag_at(r, c)] = b;
  } else if (i >= oW3 && i < oB3) {
    const int r = (i - oW3) / kHid, c = (i - oW3) % kHid;
    wf[fW3 + (c >> 4) * kFrag + frag_at(c, r)] = b;
    wf[fW3t + (c >> 4) * kFrag + frag_at(r, c)] = b;
  }
}

// Weight tiles from the float32 master copy (padding entries zero).
__global__ __launch_bounds__(256) void k_mlp_pack(const float* __restrict__ w,
                                                  unsigned short* __restrict__ wf) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < GVE_MLP_NWEIGHT) store_weight_tiles(i, w[i], wf);
  if (i < kHT * kFrag) {
    const int l = (i % kFrag) >> 2, j = i & 3;
    if ((l & 15) >= kOut) wf[fW3 + i] = 0;               // outputs 11 .. 15
    if (4 * (l >> 4) + j >= kOut) wf[fW3t + i] = 0;      // reduction over them
  }
}

__device__ inline short4v ld4(const unsigned short* p) {
  return *reinterpret_cast<const short4v*>(p);
}

__device__ inline float4v mfma16(short4v a, short4v b, float4v c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// Rows of the LDS activation tiles: 136 bfloat16 (272 bytes), so that the
// sixteen rows of an operand read fall four banks apart.
constexpr int kRowS = kHid + 8;
constexpr int kRowX = kIn + 4;

// A operand from an LDS tile: lane l reads entries (l % 16, k0 + 4 (l / 16) + j).
__device__ inline short4v lds_a(const unsigned short* t, int stride, int lane, int k0) {
  return ld4(t + (lane & 15) * stride + k0 + 4 * (lane >> 4));
}

// Input row `row`, feature c, standardised when stats are given.
template <bool STD>
__device__ inline float input_at(const float* __restrict__ X, int cols, int64_t src, int c,
                                 const float* __restrict__ mean, const float* __restrict__ sd) {
  const float v = X[(size_t)src * cols + c];
  return STD ? (v - mean[c]) / sd[c] : v;
}

// ---- inference -------------------------------------------------------------------
//
// 64 rows per step and workgroup: wave w owns output columns 32 w .. 32 w + 31
// of both hidden layers for all four 16-row tiles (its weight tiles stay in
// registers over the workgroup's steps) and row tile w of the last layer; the
// activations pass between waves through LDS, so only X and Y touch memory.
// Bound by the exact erf of 256 activations a row (about 40 vector
// instructions each): the products are 0.04 MFLOP a row.  110,592 rows: 35 us
// (a kernel per layer with float32 activations in memory: 223 us).
template <bool STD>
__global__ __launch_bounds__(256) void k_mlp_infer(const float* __restrict__ X, int64_t n,
                                                   const float* __restrict__ stats,
                                                   const float* __restrict__ w,
                                                   const unsigned short* __restrict__ wf,
                                                   float* __restrict__ Y) {
  __shared__ __attribute__((aligned(16))) unsigned short xs[64 * kRowX];
  __shared__ __attribute__((aligned(16))) unsigned short h1[64 * kRowS], h2[64 * kRowS];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int col = lane & 15, g = lane >> 4;
  short4v w1[2], w2[2][kHT], w3[kHT];
  float b1[2], b2[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int nt = 2 * wv + u;
    w1[u] = ld4(wf + fW1 + nt * kFrag + 4 * lane);
#pragma unroll
    for (int kt = 0; kt < kHT; ++kt) w2[u][kt] = ld4(wf + fW2 + (nt * kHT + kt) * kFrag + 4 * lane);
    b1[u] = w[oB1 + 16 * nt + col];
    b2[u] = w[oB2 + 16 * nt + col];
  }
#pragma unroll
  for (int kt = 0; kt < kHT; ++kt) w3[kt] = ld4(wf + fW3 + kt * kFrag + 4 * lane);
  const float b3 = col < kOut ? w[oB3 + col] : 0.0f;
  const int64_t steps = (n + 63) / 64;
  for (int64_t st = blockIdx.x; st < steps; st += gridDim.x) {
    const int64_t row0 = st * 64;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int r = 16 * u + (t >> 4), c = t & 15;
      const float v = row0 + r < n ? input_at<STD>(X, kIn, row0 + r, c, stats, stats + kIn) : 0.0f;
      xs[r * kRowX + c] = f2bf(v);
    }
    __syncthreads();
#pragma unroll
    for (int rt = 0; rt < 4; ++rt) {
      const short4v a = lds_a(xs + 16 * rt * kRowX, kRowX, lane, 0);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const float4v z = mfma16(a, w1[u], float4v{0.f, 0.f, 0.f, 0.f});
#pragma unroll
        for (int j = 0; j < 4; ++j)
          h1[(16 * rt + 4 * g + j) * kRowS + 16 * (2 * wv + u) + col] = f2bf(gelu_f(z[j] + b1[u]));
      }
    }
    __syncthreads();
#pragma unroll
    for (int rt = 0; rt < 4; ++rt) {
      float4v z[2] = {float4v{0.f, 0.f, 0.f, 0.f}, float4v{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int kt = 0; kt < kHT; ++kt) {
        const short4v a = lds_a(h1 + 16 * rt * kRowS, kRowS, lane, 16 * kt);
        z[0] = mfma16(a, w2[0][kt], z[0]);
        z[1] = mfma16(a, w2[1][kt], z[1]);
      }
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          h2[(16 * rt + 4 * g + j) * kRowS + 16 * (2 * wv + u) + col] =
              f2bf(gelu_f(z[u][j] + b2[u]));
    }
    __syncthreads();
    float4v y = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kt = 0; kt < kHT; ++kt)
      y = mfma16(lds_a(h2 + 16 * wv * kRowS, kRowS, lane, 16 * kt), w3[kt], y);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t row = row0 + 16 * wv + 4 * g + j;
      if (col < kOut && row < n) Y[row * kOut + col] = y[j] + b3;
    }
    // the next step writes xs (read before the first barrier above) and, after
    // its own first barrier, h1: every wave is past its reads of both by then
  }
}

// ---- training ---------------------------------------------------------------------
//
// One optimiser step is three launches: forward and backward of every row tile
// (k_mlp_fb), the weight gradients and bias sums over the batch (k_mlp_wgrad),
// and the sums over the batch's splits with Adam (k_mlp_adam).  Results that a
// later kernel multiplies are stored as bfloat16 operand tiles, the bias
// gradients' terms in float32.  At 4,096 rows a step takes 39 us (15 + 19 + 5);
// with a product kernel per layer and direction, separate activation, loss and
// standardisation passes and a bias sum of one thread per column reading global
// memory row by row (725 us each, three a step) it took 2.46 ms in 21 launches.

struct MlpTiles {
  // [row tile][8] tiles of bfloat16 (x and dy: one per row tile)
  unsigned short *x, *h1, *h2, *dy, *dz1, *dz2;
  // the same blocks in float32 (float4 per lane) for the bias sums
  float4v *dy32, *dz132, *dz232;
  double* loss;  // [row tile] sum of (y - t)^2
};

__device__ inline void put_tile(unsigned short* tiles, int64_t tile, int lane, const float v[4]) {
  short4v b;
#pragma unroll
  for (int j = 0; j < 4; ++j) b[j] = (short)f2bf(v[j]);
  *reinterpret_cast<short4v*>(tiles + tile * kFrag + 4 * lane) = b;
}

// Sixteen rows per workgroup, so that a batch of 4,096 fills the 256 CUs; wave
// w owns hidden columns 32 w .. 32 w + 31 and keeps their z1 and z2 in
// registers from the forward to the backward pass.  The last layer (one
// 16-wide tile) is wave 0's.  Latency-bound: five short products with a
// barrier between each; the weight tiles are loaded before the first.  LOSS: the
// forward pass and o.loss alone, nothing else is stored.
template <bool STD, bool LOSS>
__global__ __launch_bounds__(256) void k_mlp_fb(const float* __restrict__ X,
                                                const float* __restrict__ T,
                                                const uint32_t* __restrict__ perm, int rows,
                                                const float* __restrict__ stats,
                                                const float* __restrict__ w,
                                                const unsigned short* __restrict__ wf, float scale,
                                                MlpTiles o) {
  __shared__ __attribute__((aligned(16))) unsigned short xs[16 * kRowX], dys[16 * kRowX];
  __shared__ __attribute__((aligned(16))) unsigned short hs[2][16 * kRowS];
  __shared__ float ts[16 * kOut];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int col = lane & 15, g = lane >> 4;
  const int64_t rt = blockIdx.x;
  const int row0 = blockIdx.x * 16;
  // weight tiles of this wave's columns
  short4v w1[2], w2[2][kHT], w2t[2][kHT], w3t[2];
  float b1[2], b2[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int nt = 2 * wv + u;
    w1[u] = ld4(wf + fW1 + nt * kFrag + 4 * lane);
    if (!LOSS) w3t[u] = ld4(wf + fW3t + nt * kFrag + 4 * lane);
#pragma unroll
    for (int kt = 0; kt < kHT; ++kt) {
      w2[u][kt] = ld4(wf + fW2 + (nt * kHT + kt) * kFrag + 4 * lane);
      if (!LOSS) w2t[u][kt] = ld4(wf + fW2t + (nt * kHT + kt) * kFrag + 4 * lane);
    }
    b1[u] = w[oB1 + 16 * nt + col];
    b2[u] = w[oB2 + 16 * nt + col];
  }
  {
    const int r = t >> 4, c = t & 15;
    float v = 0.0f;
    if (row0 + r < rows)
      v = input_at<STD>(X, kIn, perm ? (int64_t)perm[row0 + r] : row0 + r, c, stats, stats + kIn);
    xs[r * kRowX + c] = f2bf(v);
    if (t < 16 * kOut) {
      const int rr = t / kOut, cc = t % kOut;
      float q = 0.0f;
      if (row0 + rr < rows)
        q = input_at<STD>(T, kOut, perm ? (int64_t)perm[row0 + rr] : row0 + rr, cc,
                          stats + 2 * kIn, stats + 2 * kIn + kOut);
      ts[t] = q;
    }
  }
  __syncthreads();
  bool in[4];  // rows 4 g + j of the tile belong to the batch
#pragma unroll
  for (int j = 0; j < 4; ++j) in[j] = row0 + 4 * g + j < rows;
  if (!LOSS && wv == 3) {  // x as the right operand of the first weight gradient
    short4v b;
#pragma unroll
    for (int j = 0; j < 4; ++j) b[j] = (short)xs[(4 * g + j) * kRowX + col];
    *reinterpret_cast<short4v*>(o.x + rt * kFrag + 4 * lane) = b;
  }
  // forward; activations of rows past the batch are stored as zero
  float z1[2][4], z2[2][4];
  const short4v xa = lds_a(xs, kRowX, lane, 0);
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int nt = 2 * wv + u;
    const float4v z = mfma16(xa, w1[u], float4v{0.f, 0.f, 0.f, 0.f});
    float h[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      z1[u][j] = z[j] + b1[u];
      const float a = gelu_f(z1[u][j]);
      h[j] = in[j] ? a : 0.0f;
      hs[0][(4 * g + j) * kRowS + 16 * nt + col] = f2bf(h[j]);
    }
    if (!LOSS) put_tile(o.h1, rt * kHT + nt, lane, h);
  }
  __syncthreads();
  {
    float4v z[2] = {float4v{0.f, 0.f, 0.f, 0.f}, float4v{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int kt = 0; kt < kHT; ++kt) {
      const short4v a = lds_a(hs[0], kRowS, lane, 16 * kt);
      z[0] = mfma16(a, w2[0][kt], z[0]);
      z[1] = mfma16(a, w2[1][kt], z[1]);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int nt = 2 * wv + u;
      float h[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        z2[u][j] = z[u][j] + b2[u];
        const float a = gelu_f(z2[u][j]);
        h[j] = in[j] ? a : 0.0f;
        hs[1][(4 * g + j) * kRowS + 16 * nt + col] = f2bf(h[j]);
      }
      if (!LOSS) put_tile(o.h2, rt * kHT + nt, lane, h);
    }
  }
  __syncthreads();
  if (wv == 0) {
    float4v y = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kt = 0; kt < kHT; ++kt)
      y = mfma16(lds_a(hs[1], kRowS, lane, 16 * kt), ld4(wf + fW3 + kt * kFrag + 4 * lane), y);
    const float b3 = col < kOut ? w[oB3 + col] : 0.0f;
    double s = 0.0;
    float d[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      d[j] = 0.0f;
      if (col < kOut && in[j]) {
        const float yv = y[j] + b3;
        const float r = yv - ts[(4 * g + j) * kOut + col];
        s += (double)r * r;
        d[j] = 2.0f * r * scale;
      }
      dys[(4 * g + j) * kRowX + col] = f2bf(d[j]);
    }
    if (!LOSS) {
      put_tile(o.dy, rt, lane, d);
      o.dy32[rt * 64 + lane] = float4v{d[0], d[1], d[2], d[3]};
    }
#pragma unroll
    for (int k = 32; k >= 1; k >>= 1) s += __shfl_xor(s, k, 64);
    if (lane == 0) o.loss[rt] = s;
  }
  if constexpr (LOSS) return;
  __syncthreads();
  // backward; hs[0] (h1, last read two barriers ago) takes dz2
  const short4v da = lds_a(dys, kRowX, lane, 0);
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int nt = 2 * wv + u;
    const float4v dh = mfma16(da, w3t[u], float4v{0.f, 0.f, 0.f, 0.f});
    float d[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float v = dh[j] * gelu_grad_f(z2[u][j]);
      d[j] = in[j] ? v : 0.0f;
      hs[0][(4 * g + j) * kRowS + 16 * nt + col] = f2bf(d[j]);
    }
    put_tile(o.dz2, rt * kHT + nt, lane, d);
    o.dz232[(rt * kHT + nt) * 64 + lane] = float4v{d[0], d[1], d[2], d[3]};
  }
  __syncthreads();
  float4v dh[2] = {float4v{0.f, 0.f, 0.f, 0.f}, float4v{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
  for (int kt = 0; kt < kHT; ++kt) {
    const short4v a = lds_a(hs[0], kRowS, lane, 16 * kt);
    dh[0] = mfma16(a, w2t[0][kt], dh[0]);
    dh[1] = mfma16(a, w2t[1][kt], dh[1]);
  }
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int nt = 2 * wv + u;
    float d[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float v = dh[u][j] * gelu_grad_f(z1[u][j]);
      d[j] = in[j] ? v : 0.0f;
    }
    put_tile(o.dz1, rt * kHT + nt, lane, d);
    o.dz132[(rt * kHT + nt) * 64 + lane] = float4v{d[0], d[1], d[2], d[3]};
  }
}

// Weight gradients over the row tiles [r0, r1) of one split (M x N tiles of
// 16 x 16 from operand tiles a[rt][sa] and b[rt][sb]), row tiles in order.
template <int M, int N>
__device__ inline void wgrad_tiles(const unsigned short* __restrict__ a, int sa,
                                   const unsigned short* __restrict__ b, int sb, int64_t r0,
                                   int64_t r1, int lane, float4v (&acc)[M][N]) {
#pragma unroll
  for (int m = 0; m < M; ++m)
#pragma unroll
    for (int n = 0; n < N; ++n) acc[m][n] = float4v{0.f, 0.f, 0.f, 0.f};
  constexpr int kAhead = 4;  // row tiles loaded together
  int64_t r = r0;
  for (; r + kAhead <= r1; r += kAhead) {
    short4v fa[kAhead][M], fb[kAhead][N];
#pragma unroll
    for (int q = 0; q < kAhead; ++q) {
#pragma unroll
      for (int m = 0; m < M; ++m) fa[q][m] = ld4(a + ((r + q) * sa + m) * kFrag + 4 * lane);
#pragma unroll
      for (int n = 0; n < N; ++n) fb[q][n] = ld4(b + ((r + q) * sb + n) * kFrag + 4 * lane);
    }
#pragma unroll
    for (int q = 0; q < kAhead; ++q)
#pragma unroll
      for (int m = 0; m < M; ++m)
#pragma unroll
        for (int n = 0; n < N; ++n) acc[m][n] = mfma16(fa[q][m], fb[q][n], acc[m][n]);
  }
  for (; r < r1; ++r)
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
      for (int n = 0; n < N; ++n)
        acc[m][n] = mfma16(ld4(a + (r * sa + m) * kFrag + 4 * lane),
                           ld4(b + (r * sb + n) * kFrag + 4 * lane), acc[m][n]);
}

// Bias gradient of sixteen columns: the float32 terms added row by row, in row
// order (a running sum, whose length is the kernel's: 19.3 us at 4,096 rows, 4.7 ns
// a row; 21.4 us before the reads of LDS were issued ahead of the additions).
// 32 row tiles at a time are staged in LDS by all four waves, the next ones
// while sixteen lanes of wave 0 add the current ones.
constexpr int kBiasTiles = 32;
constexpr int kBiasAhead = 8;
__device__ inline void bias_sum(const float4v* __restrict__ v, int stride, int64_t tiles,
                                float4v* buf, float* __restrict__ out, int nout) {
  const int t = threadIdx.x;
  constexpr int kPer = kBiasTiles * 64 / 256;
  float4v q[kPer];
  auto fetch = [&](int64_t r0) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int64_t r = r0 + 4 * u + (t >> 6);
      q[u] = r < tiles ? v[r * stride * 64 + (t & 63)] : float4v{0.f, 0.f, 0.f, 0.f};
    }
  };
  float s = 0.0f;
  fetch(0);
  int b = 0;
  for (int64_t r0 = 0; r0 < tiles; r0 += kBiasTiles, b ^= 1) {
    float4v* cur = buf + b * kBiasTiles * 64;
#pragma unroll
    for (int u = 0; u < kPer; ++u) cur[(4 * u + (t >> 6)) * 64 + (t & 63)] = q[u];
    __syncthreads();
    if (r0 + kBiasTiles < tiles) fetch(r0 + kBiasTiles);
    // the buffer written next was read before the barrier above
    if (t < 16) {
      // rows 4 k .. 4 k + 3 at a time; the next eight reads of LDS are issued
      // before the current eight are added
      const int lim = (int)min((int64_t)kBiasTiles, tiles - r0) * 4;
      const float4v* p = cur + t;
      float4v x[kBiasAhead], y[kBiasAhead];
      auto read = [&](float4v(&d)[kBiasAhead], int k) {
#pragma unroll
        for (int u = 0; u < kBiasAhead; ++u) d[u] = p[(k + u) * 16];
      };
      auto add = [&](const float4v(&d)[kBiasAhead]) {
#pragma unroll
        for (int u = 0; u < kBiasAhead; ++u) {
          s += d[u][0];
          s += d[u][1];
          s += d[u][2];
          s += d[u][3];
        }
      };
      int k = 0;
      if (lim == 4 * kBiasTiles) {
        read(x, 0);
#pragma unroll
        for (; k < 4 * kBiasTiles; k += 2 * kBiasAhead) {
          read(y, k + kBiasAhead);
          __builtin_amdgcn_sched_barrier(0);
          add(x);
          if (k + 2 * kBiasAhead < 4 * kBiasTiles) read(x, k + 2 * kBiasAhead);
          __builtin_amdgcn_sched_barrier(0);
          add(y);
        }
      }
      for (; k < lim; ++k) {
        const float4v z = p[k * 16];
        s += z[0];
        s += z[1];
        s += z[2];
        s += z[3];
      }
    }
  }
  if (t < nout) out[t] = s;
}

constexpr int kBiasBlocks = 2 * kHT + 1;
constexpr int kSplitBlocks = 5;  // workgroups of one split: 20 waves

// Blocks 0 .. 16: bias sums.  Then five workgroups per split of `per` row
// tiles: waves 0 .. 15 a 2 x 2 patch of W2's 8 x 8 tiles, 16 and 17 half of
// W3's row of tiles, 18 and 19 half of W1's column.  Split z writes its
// partial gradient to part[z] (flat weight layout).
__global__ __launch_bounds__(256) void k_mlp_wgrad(MlpTiles o, int64_t tiles, int64_t per,
                                                   float* __restrict__ part,
                                                   float* __restrict__ bias) {
  __shared__ __attribute__((aligned(16))) float4v buf[2 * kBiasTiles * 64];
  if (blockIdx.x < kBiasBlocks) {
    const int b = blockIdx.x;
    if (b < kHT) bias_sum(o.dz232 + b * 64, kHT, tiles, buf, bias + kHid + 16 * b, 16);
    else if (b < 2 * kHT) bias_sum(o.dz132 + (b - kHT) * 64, kHT, tiles, buf, bias + 16 * (b - kHT), 16);
    else bias_sum(o.dy32, 1, tiles, buf, bias + 2 * kHid, kOut);
    return;
  }
  const int z = (blockIdx.x - kBiasBlocks) / kSplitBlocks;
  const int job = ((blockIdx.x - kBiasBlocks) % kSplitBlocks) * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4;
  const int64_t r0 = z * per, r1 = min(tiles, r0 + per);
  float* out = part + (size_t)z * GVE_MLP_NWEIGHT;
  if (job < 16) {
    const int m0 = (job >> 2) * 2, n0 = (job & 3) * 2;
    float4v acc[2][2];
    wgrad_tiles<2, 2>(o.dz2 + m0 * kFrag, kHT, o.h1 + n0 * kFrag, kHT, r0, r1, lane, acc);
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          out[oW2 + (16 * (m0 + m) + 4 * g + j) * kHid + 16 * (n0 + n) + col] = acc[m][n][j];
  } else if (job < 18) {
    const int n0 = (job - 16) * 4;
    float4v acc[1][4];
    wgrad_tiles<1, 4>(o.dy, 1, o.h2 + n0 * kFrag, kHT, r0, r1, lane, acc);
#pragma unroll
    for (int n = 0; n < 4; ++n)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (4 * g + j < kOut) out[oW3 + (4 * g + j) * kHid + 16 * (n0 + n) + col] = acc[0][n][j];
  } else {
    const int m0 = (job - 18) * 4;
    float4v acc[4][1];
    wgrad_tiles<4, 1>(o.dz1 + m0 * kFrag, kHT, o.x, 1, r0, r1, lane, acc);
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        out[oW1 + (16 * (m0 + m) + 4 * g + j) * kIn + col] = acc[m][0][j];
  }
}

// Adds the batch's loss, scaled, to *loss (one block of 256 threads).
__device__ inline void add_loss(const double* __restrict__ tile_loss, int64_t tiles, double scale,
                                double* __restrict__ loss) {
  __shared__ double sh[256];
  double s = 0.0;
  for (int64_t k = threadIdx.x; k < tiles; k += 256) s += tile_loss[k];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if ((int)threadIdx.x < k) sh[threadIdx.x] += sh[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) *loss += sh[0] * scale;
}

__global__ __launch_bounds__(256) void k_mlp_loss(const double* __restrict__ tile_loss,
                                                  int64_t tiles, double scale,
                                                  double* __restrict__ loss) {
  add_loss(tile_loss, tiles, scale, loss);
}

// Sum over the splits, in order, then the gradient to grad_out (when given) or
// a bias-corrected Adam step on the float32 weights with their bfloat16 tiles.
// Block 0 also adds the batch's loss, scaled, to *loss.
__global__ __launch_bounds__(256) void k_mlp_adam(const float* __restrict__ part, int splits,
                                                  const float* __restrict__ bias,
                                                  const double* __restrict__ tile_loss,
                                                  int64_t tiles, double loss_scale,
                                                  double* __restrict__ loss,
                                                  float* __restrict__ grad_out,
                                                  float* __restrict__ w, float* __restrict__ m,
                                                  float* __restrict__ v,
                                                  unsigned short* __restrict__ wf, float lr,
                                                  float b1, float b2, float eps, float ibc1,
                                                  float ibc2) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < GVE_MLP_NWEIGHT) {
    float gi;
    if (i >= oB1 && i < oW2) gi = bias[i - oB1];
    else if (i >= oB2 && i < oW3) gi = bias[kHid + i - oB2];
    else if (i >= oB3) gi = bias[2 * kHid + i - oB3];
    else {
      gi = 0.0f;
#pragma unroll 8
      for (int z = 0; z < splits; ++z) gi += part[(size_t)z * GVE_MLP_NWEIGHT + i];
    }
    if (grad_out) {
      grad_out[i] = gi;
    } else {
      const float mm = b1 * m[i] + (1.0f - b1) * gi;
      const float vv = b2 * v[i] + (1.0f - b2) * gi * gi;
      m[i] = mm;
      v[i] = vv;
      const float x = w[i] - lr * (mm * ibc1) / (sqrtf(vv * ibc2) + eps);
      w[i] = x;
      store_weight_tiles(i, x, wf);
    }
  }
  if (blockIdx.x == 0) add_loss(tile_loss, tiles, loss_scale, loss);
}

// Per-column mean and standard deviation (double) of a [rows][cols] matrix
// (cols <= 16): each block sums its rows (whole rows per wave, so coalesced),
// then one block adds the block sums in order.
constexpr int kStatBlocks = 128;
__global__ __launch_bounds__(256) void k_colstats_part(const float* __restrict__ X, int64_t rows,
                                                       int cols, double* __restrict__ part) {
  __shared__ double s1[256], s2[256];
  const int c = threadIdx.x & 15, q = threadIdx.x >> 4;
  double a = 0.0, b = 0.0;
  if (c < cols)
#pragma unroll 4
    for (int64_t r = (int64_t)blockIdx.x * 16 + q; r < rows; r += kStatBlocks * 16) {
      const double x = X[(size_t)r * cols + c];
      a += x;
      b += x * x;
    }
  s1[threadIdx.x] = a;
  s2[threadIdx.x] = b;
  __syncthreads();
  for (int k = 128; k >= 16; k >>= 1) {
    if ((int)threadIdx.x < k) {
      s1[threadIdx.x] += s1[threadIdx.x + k];
      s2[threadIdx.x] += s2[threadIdx.x + k];
    }
    __syncthreads();
  }
  if (threadIdx.x < 16) {
    part[(blockIdx.x * 16 + threadIdx.x) * 2] = s1[threadIdx.x];
    part[(blockIdx.x * 16 + threadIdx.x) * 2 + 1] = s2[threadIdx.x];
  }
}

__global__ __launch_bounds__(64) void k_colstats_final(const double* __restrict__ part, int64_t rows,
                                                       int cols, float* __restrict__ mean,
                                                       float* __restrict__ stdv) {
  const int c = threadIdx.x;
  if (c >= cols) return;
  double a = 0.0, b = 0.0;
#pragma unroll 16
  for (int k = 0; k < kStatBlocks; ++k) {
    a += part[(k * 16 + c) * 2];
    b += part[(k * 16 + c) * 2 + 1];
  }
  const double mu = a / (double)rows;
  double var = b / (double)rows - mu * mu;
  if (var < 0.0) var = 0.0;
  const double sd = sqrt(var);
  mean[c] = (float)mu;
  stdv[c] = (float)(sd > 1e-6 ? sd : 1.0);
}

// Random 32-bit keys and identity values for an epoch's permutation.
__global__ void k_perm_keys(uint32_t* __restrict__ keys, uint32_t* __restrict__ vals, int64_t n,
                            uint64_t seed, uint64_t epoch) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  keys[i] = (uint32_t)(hash_bits(seed, epoch, (uint64_t)i) >> 32);
  vals[i] = (uint32_t)i;
}

// ---- features --------------------------------------------------------------

// Mean and variance of V over a primitive's box come from prefix sums of V and
// V^2, in one of two forms.  Block tables: within each block of 64 x 8 x 8 voxels
// the sums from the block's corner, which one wave forms in one pass over the
// volume without a carry from other blocks (20 bytes a voxel); a box adds up to
// eight entries of each block it touches, a lane per block.  Summed-area tables
// of the whole volume: three passes (84 bytes a voxel), then eight entries a box.
// The blocks that the set's boxes touch are counted on the device, and the
// kernels of the form not taken return at once.  Features, tables -> blocks:
// 64^3 x 2,048 of scales 1.5 - 4 106 -> 85 us; 256^3 x 65,536, 2 - 6 599 -> 311, 8
// - 12 589 -> 457; 384^3 x 110,592, 1 - 3 1,530 -> 646; 256^3 x 20,000, 20 - 30
// (about 2.5 touched blocks per voxel) 468 -> 430: tables past 2.  The block
// tables take 257 us at 384^3, 4.4 TB/s: the rate of a copy.
constexpr int kSatX = 64, kSatY = 8, kSatZ = 8;
constexpr uint64_t kBlocksPerVoxel = 2;
constexpr int64_t kSatLines = 8192;           // workgroups of the x pass
constexpr int64_t kSatBlocks = 1 << 20;       // and of the block tables

__device__ inline bool takes_blocks(const unsigned long long* __restrict__ touched, int64_t M) {
  return *touched <= kBlocksPerVoxel * (uint64_t)M;
}

// Inclusive prefix sums of V and V^2 along x, a (y, z) line at a time.
__global__ __launch_bounds__(256) void k_sat_x(const float* __restrict__ f, int64_t nx,
                                               int64_t lines,
                                               const unsigned long long* __restrict__ touched,
                                               double* __restrict__ s1, double* __restrict__ s2) {
  if (takes_blocks(touched, nx * lines)) return;
  __shared__ double c1[256], c2[256];
  for (int64_t line = blockIdx.x; line < lines; line += gridDim.x) {
    const size_t base = (size_t)line * nx;
    double carry1 = 0.0, carry2 = 0.0;
    for (int64_t x0 = 0; x0 < nx; x0 += 256) {
      const int64_t x = x0 + threadIdx.x;
      const double v = x < nx ? (double)f[base + x] : 0.0;
      c1[threadIdx.x] = v;
      c2[threadIdx.x] = v * v;
      __syncthreads();
      for (int d = 1; d < 256; d <<= 1) {
        const double a = threadIdx.x >= (unsigned)d ? c1[threadIdx.x - d] : 0.0;
        const double b = threadIdx.x >= (unsigned)d ? c2[threadIdx.x - d] : 0.0;
        __syncthreads();
        c1[threadIdx.x] += a;
        c2[threadIdx.x] += b;
        __syncthreads();
      }
      if (x < nx) {
        s1[base + x] = carry1 + c1[threadIdx.x];
        s2[base + x] = carry2 + c2[threadIdx.x];
      }
      carry1 += c1[255];
      carry2 += c2[255];
      __syncthreads();
    }
  }
}

// Running sums along an axis with element stride `stride` (line = thread).
__global__ void k_sat_axis(double* __restrict__ s1, double* __restrict__ s2, int64_t nlines,
                           int64_t inner, int64_t len, int64_t stride,
                           const unsigned long long* __restrict__ touched) {
  const int64_t l = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (l >= nlines || takes_blocks(touched, nlines * len)) return;
  const size_t base = (size_t)(l / inner) * (size_t)(inner * len) + (size_t)(l % inner);
  double a = 0.0, b = 0.0;
  for (int64_t k = 0; k < len; ++k) {
    const size_t o = base + (size_t)k * stride;
    a += s1[o];
    b += s2[o];
    s1[o] = a;
    s2[o] = b;
  }
}

__device__ inline double sat_at(const double* __restrict__ S, int64_t nx, int64_t ny, int64_t x,
                                int64_t y, int64_t z) {
  if (x < 0 || y < 0 || z < 0) return 0.0;
  return S[(size_t)x + (size_t)nx * ((size_t)y + (size_t)ny * (size_t)z)];
}

__device__ inline double box_sum(const double* __restrict__ S, int64_t nx, int64_t ny, int64_t xa,
                                 int64_t xb, int64_t ya, int64_t yb, int64_t za, int64_t zb) {
  return sat_at(S, nx, ny, xb, yb, zb) - sat_at(S, nx, ny, xa - 1, yb, zb) -
         sat_at(S, nx, ny, xb, ya - 1, zb) - sat_at(S, nx, ny, xb, yb, za - 1) +
         sat_at(S, nx, ny, xa - 1, ya - 1, zb) + sat_at(S, nx, ny, xa - 1, yb, za - 1) +
         sat_at(S, nx, ny, xb, ya - 1, za - 1) - sat_at(S, nx, ny, xa - 1, ya - 1, za - 1);
}

// A primitive's k-sigma box, voxel indices within the volume; empty if some
// hi < lo.
struct FeatBox {
  int lo[3], hi[3];
};
static_assert(sizeof(FeatBox) == 3 * sizeof(double), "a box takes three doubles of the workspace");

struct FeatArgs {
  const float* f;
  const float* theta;
  int64_t n, n_detail;
  gve_grid g;
  double g99;
  const double* s1;
  const double* s2;
  const double* J6;  // [n][6] structure tensors at the centres (k_feat_tensor)
  const FeatBox* box;
  const double* mom;  // [n][2] sums of V and V^2 over the boxes (k_box_sums)
  const unsigned long long* touched;
  float* X;  // [n][16]
};

// The voxel nearest primitive i's centre, clamped to the grid.
__device__ inline void centre_voxel(const float* __restrict__ theta, int64_t n, int64_t i,
                                    const gve_grid& g, int64_t c[3]) {
  const double mu[3] = {theta[0 * n + i], theta[1 * n + i], theta[2 * n + i]};
  const int64_t org[3] = {g.x0, g.y0, g.z0};
  const int64_t dim[3] = {g.nx, g.ny, g.nz};
  for (int ax = 0; ax < 3; ++ax) {
    int64_t v = (int64_t)floor(mu[ax] - (double)org[ax] + 0.5);
    c[ax] = v < 0 ? 0 : (v > dim[ax] - 1 ? dim[ax] - 1 : v);
  }
}

// One wave per primitive: the structure tensor at its centre voxel.
__global__ __launch_bounds__(256) void k_feat_tensor(const float* __restrict__ f,
                                                     const float* __restrict__ theta, int64_t n,
                                                     gve_grid g, double* __restrict__ J6) {
  const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= n) return;  // wave-uniform
  int64_t c[3];
  centre_voxel(theta, n, i, g, c);
  __shared__ float box[4][kTensorBox];
  wave_structure_tensor(f, Dims{g.nx, g.ny, g.nz}, c[0], c[1], c[2], box[threadIdx.x >> 6],
                        J6 + 6 * i);
}

// The boxes, and the blocks they touch added to *touched.
__global__ __launch_bounds__(256) void k_feat_box(const float* __restrict__ theta, int64_t n,
                                                  gve_grid g, float k, FeatBox* __restrict__ box,
                                                  unsigned long long* __restrict__ touched) {
  __shared__ unsigned long long tot[4];
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  unsigned long long t = 0;
  if (i < n) {
    const double mu[3] = {theta[0 * n + i], theta[1 * n + i], theta[2 * n + i]};
    const int64_t org[3] = {g.x0, g.y0, g.z0};
    const int64_t dim[3] = {g.nx, g.ny, g.nz};
    double qw = theta[3 * n + i], qx = theta[4 * n + i], qy = theta[5 * n + i],
           qz = theta[6 * n + i];
    const double qn = sqrt(qw * qw + qx * qx + qy * qy + qz * qz);
    if (qn >= 1e-12) { qw /= qn; qx /= qn; qy /= qn; qz /= qn; } else { qw = 1; qx = qy = qz = 0; }
    const double R[3][3] = {{1 - 2 * (qy * qy + qz * qz), 2 * (qx * qy - qw * qz), 2 * (qx * qz + qw * qy)},
                            {2 * (qx * qy + qw * qz), 1 - 2 * (qx * qx + qz * qz), 2 * (qy * qz - qw * qx)},
                            {2 * (qx * qz - qw * qy), 2 * (qy * qz + qw * qx), 1 - 2 * (qx * qx + qy * qy)}};
    const double s2v[3] = {exp(2.0 * (double)theta[7 * n + i]), exp(2.0 * (double)theta[8 * n + i]),
                           exp(2.0 * (double)theta[9 * n + i])};
    int64_t lo[3], hi[3];
    bool empty = false;
    for (int ax = 0; ax < 3; ++ax) {
      const double sd = R[ax][0] * R[ax][0] * s2v[0] + R[ax][1] * R[ax][1] * s2v[1] +
                        R[ax][2] * R[ax][2] * s2v[2];
      const double h = (double)k * sqrt(sd);
      double lf = ceil(mu[ax] - h - (double)org[ax]), hf = floor(mu[ax] + h - (double)org[ax]);
      lf = fmax(lf, 0.0);
      hf = fmin(hf, (double)(dim[ax] - 1));
      if (lf > hf) empty = true;
      lo[ax] = (int64_t)lf;
      hi[ax] = (int64_t)hf;
    }
    FeatBox b;
    for (int ax = 0; ax < 3; ++ax) {
      b.lo[ax] = empty ? 1 : (int)lo[ax];
      b.hi[ax] = empty ? 0 : (int)hi[ax];
    }
    box[i] = b;
    if (!empty)
      t = (unsigned long long)((hi[0] / kSatX - lo[0] / kSatX + 1) *
                               (hi[1] / kSatY - lo[1] / kSatY + 1) *
                               (hi[2] / kSatZ - lo[2] / kSatZ + 1));
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
  if ((threadIdx.x & 63) == 0) tot[threadIdx.x >> 6] = t;
  __syncthreads();
  if (threadIdx.x == 0) atomicAdd(touched, tot[0] + tot[1] + tot[2] + tot[3]);
}

// x + (x of the lane DPP names), in the lanes of the rows of MASK.
template <int CTRL, int MASK>
__device__ inline double dpp_plus(double x) {
  const uint64_t b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, MASK, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, MASK, 0xF, false);
  return x + __longlong_as_double(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

// Inclusive prefix sum over the lanes of a wave.
__device__ inline double wave_prefix(double x) {
  x = dpp_plus<0x111, 0xF>(x);  // row_shr:1, 2, 4, 8
  x = dpp_plus<0x112, 0xF>(x);
  x = dpp_plus<0x114, 0xF>(x);
  x = dpp_plus<0x118, 0xF>(x);
  x = dpp_plus<0x142, 0xA>(x);  // row_bcast:15 into rows 1 and 3
  x = dpp_plus<0x143, 0xC>(x);  // row_bcast:31 into rows 2 and 3
  return x;
}

// One wave per block of 64 x 8 x 8 voxels: its prefix sums, row after row, the
// rows of the plane before held in registers.
__global__ __launch_bounds__(64) void k_sat_blocks(const float* __restrict__ f, gve_grid g,
                                                   const unsigned long long* __restrict__ touched,
                                                   int64_t nbx, int64_t nby, int64_t nblocks,
                                                   double2* __restrict__ T) {
  if (!takes_blocks(touched, g.nx * g.ny * g.nz)) return;
  const int lane = threadIdx.x;
  for (int64_t b = blockIdx.x; b < nblocks; b += gridDim.x) {
    const int64_t x = (b % nbx) * kSatX + lane;
    const int64_t y0 = (b / nbx) % nby * kSatY, z0 = b / (nbx * nby) * kSatZ;
    const bool in = x < g.nx;
    double2 below[kSatY];
#pragma unroll
    for (int u = 0; u < kSatY; ++u) below[u] = make_double2(0.0, 0.0);
    for (int w = 0; w < kSatZ && z0 + w < g.nz; ++w) {
      const size_t o = (size_t)(in ? x : 0) + (size_t)g.nx * ((size_t)y0 + (size_t)g.ny * (size_t)(z0 + w));
      float v[kSatY];
#pragma unroll
      for (int u = 0; u < kSatY; ++u)
        v[u] = in && y0 + u < g.ny ? f[o + (size_t)g.nx * u] : 0.0f;
      double a = 0.0, c = 0.0;
#pragma unroll
      for (int u = 0; u < kSatY; ++u) {
        const double d = (double)v[u];
        a += wave_prefix(d);
        c += wave_prefix(d * d);
        below[u].x += a;
        below[u].y += c;
        if (in && y0 + u < g.ny) T[o + (size_t)g.nx * u] = below[u];
      }
    }
  }
}

// Sums of V and V^2 over the boxes, one wave per primitive, a lane per block
// that the box touches; added in a fixed order.
__global__ __launch_bounds__(256) void k_box_sums(const double2* __restrict__ T, int64_t n,
                                                  gve_grid g, const FeatBox* __restrict__ box,
                                                  const unsigned long long* __restrict__ touched,
                                                  double* __restrict__ mom) {
  if (!takes_blocks(touched, g.nx * g.ny * g.nz)) return;
  const int64_t i = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (i >= n) return;  // wave-uniform
  const FeatBox b = box[i];
  if (b.hi[0] < b.lo[0]) return;  // empty: its sums are not read
  const int bx0 = b.lo[0] / kSatX, by0 = b.lo[1] / kSatY, bz0 = b.lo[2] / kSatZ;
  const uint32_t cx = b.hi[0] / kSatX - bx0 + 1, cy = b.hi[1] / kSatY - by0 + 1,
                 cz = b.hi[2] / kSatZ - bz0 + 1;
  double t1 = 0.0, t2 = 0.0;
  for (uint32_t j = threadIdx.x & 63; j < cx * cy * cz; j += 64) {
    const uint32_t q = j / cx;
    const int x0 = (bx0 + (int)(j - q * cx)) * kSatX, y0 = (by0 + (int)(q % cy)) * kSatY,
              z0 = (bz0 + (int)(q / cy)) * kSatZ;
    const int xa = max(b.lo[0], x0), xb = min(b.hi[0], x0 + kSatX - 1);
    const int ya = max(b.lo[1], y0), yb = min(b.hi[1], y0 + kSatY - 1);
    const int za = max(b.lo[2], z0), zb = min(b.hi[2], z0 + kSatZ - 1);
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      // a lower face on the block's own face adds nothing
      if (((c & 1) && xa == x0) || ((c & 2) && ya == y0) || ((c & 4) && za == z0)) continue;
      const size_t o = (size_t)((c & 1) ? xa - 1 : xb) +
                       (size_t)g.nx * ((size_t)((c & 2) ? ya - 1 : yb) +
                                       (size_t)g.ny * (size_t)((c & 4) ? za - 1 : zb));
      const double2 v = T[o];
      const bool minus = __builtin_popcount(c) & 1;
      t1 += minus ? -v.x : v.x;
      t2 += minus ? -v.y : v.y;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    t1 += __shfl_xor(t1, o, 64);
    t2 += __shfl_xor(t2, o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    mom[2 * i] = t1;
    mom[2 * i + 1] = t2;
  }
}

__global__ __launch_bounds__(128) void k_features(FeatArgs a) {
  const int64_t i = (int64_t)blockIdx.x * 128 + threadIdx.x;
  if (i >= a.n) return;
  const int64_t n = a.n;
  const Dims d{a.g.nx, a.g.ny, a.g.nz};
  const double mu[3] = {a.theta[0 * n + i], a.theta[1 * n + i], a.theta[2 * n + i]};
  const int64_t org[3] = {a.g.x0, a.g.y0, a.g.z0};
  const int64_t dim[3] = {a.g.nx, a.g.ny, a.g.nz};
  int64_t c[3];
  centre_voxel(a.theta, n, i, a.g, c);
  // structure tensor at the seed voxel, from k_feat_tensor
  const double* t = a.J6 + 6 * i;
  double J[3][3] = {{t[0], t[1], t[2]}, {t[1], t[3], t[4]}, {t[2], t[4], t[5]}};
  double lam[3] = {0, 0, 0};
  double E[3][3] = {{0, 0, 1}, {0, 1, 0}, {1, 0, 0}};  // rows: e1, e2, e3
  if (J[0][0] + J[1][1] + J[2][2] >= 1e-12) {
    double Am[3][3], V[3][3];
    for (int r = 0; r < 3; ++r)
      for (int q = 0; q < 3; ++q) Am[r][q] = J[r][q];
    jacobi3(Am, V);
    double w[3] = {Am[0][0], Am[1][1], Am[2][2]};
    int idx[3] = {0, 1, 2};  // descending
    for (int p = 0; p < 3; ++p)
      for (int q = p + 1; q < 3; ++q)
        if (w[idx[q]] > w[idx[p]]) { int t = idx[p]; idx[p] = idx[q]; idx[q] = t; }
    for (int r = 0; r < 3; ++r) {
      const int e = idx[r];
      lam[r] = w[e];
      int am = 0;
      double best = fabs(V[0][e]);
      for (int q = 1; q < 3; ++q)
        if (fabs(V[q][e]) > best) { best = fabs(V[q][e]); am = q; }
      const double sg = V[am][e] < 0.0 ? -1.0 : 1.0;
      for (int q = 0; q < 3; ++q) E[r][q] = sg * V[q][e];
    }
  }
  float* out = a.X + (size_t)i * 16;
  const double gg = a.g99 > 0.0 ? a.g99 * a.g99 : 1.0;
  for (int r = 0; r < 3; ++r) out[r] = (float)log1p(fmax(lam[r], 0.0) / gg);
  for (int r = 0; r < 3; ++r)
    for (int q = 0; q < 3; ++q) out[3 + 3 * r + q] = (float)E[r][q];
  const int64_t vox = c[0] + d.nx * (c[1] + d.ny * c[2]);
  out[12] = a.g99 > 0.0 ? (float)((double)grad_mag32(a.f, d, vox) / a.g99) : 0.0f;
  // mean and variance of V over the k-sigma box
  const FeatBox b = a.box[i];
  const bool empty = b.hi[0] < b.lo[0] || b.hi[1] < b.lo[1] || b.hi[2] < b.lo[2];
  if (!empty) {
    const double cnt = (double)((int64_t)(b.hi[0] - b.lo[0] + 1) * (b.hi[1] - b.lo[1] + 1) *
                                (b.hi[2] - b.lo[2] + 1));
    double t1, t2;
    if (takes_blocks(a.touched, dim[0] * dim[1] * dim[2])) {
      t1 = a.mom[2 * i];
      t2 = a.mom[2 * i + 1];
    } else {
      t1 = box_sum(a.s1, d.nx, d.ny, b.lo[0], b.hi[0], b.lo[1], b.hi[1], b.lo[2], b.hi[2]);
      t2 = box_sum(a.s2, d.nx, d.ny, b.lo[0], b.hi[0], b.lo[1], b.hi[1], b.lo[2], b.hi[2]);
    }
    const double m1 = t1 / cnt, m2 = t2 / cnt;
    out[13] = (float)m1;
    out[14] = (float)fmax(m2 - m1 * m1, 0.0);
  } else {
    out[13] = 0.0f;
    out[14] = 0.0f;
  }
  out[15] = i < a.n_detail ? 1.0f : 0.0f;
}

// Targets: theta_ref - theta_alloc per primitive, refined q normalised and
// sign-aligned to the allocated q; [n][11].
__global__ void k_targets(const float* __restrict__ ta, const float* __restrict__ tr, int64_t n,
                          float* __restrict__ T) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double q[4], qa[4];
  double nn = 0.0, dot = 0.0;
  for (int c = 0; c < 4; ++c) {
    q[c] = tr[(3 + c) * n + i];
    qa[c] = ta[(3 + c) * n + i];
    nn += q[c] * q[c];
  }
  nn = sqrt(nn);
  if (nn < 1e-30) nn = 1e-30;
  for (int c = 0; c < 4; ++c) {
    q[c] /= nn;
    dot += q[c] * qa[c];
  }
  const double sg = dot < 0.0 ? -1.0 : 1.0;
  float* out = T + (size_t)i * 11;
  for (int c = 0; c < 11; ++c) {
    const double r = (c >= 3 && c <= 6) ? sg * q[c - 3] : (double)tr[c * n + i];
    out[c] = (float)(r - (double)ta[c * n + i]);
  }
}

// theta += alpha * (Y * tstd + tmean)   (Y: standardised network output [n][11])
__global__ void k_apply_delta(float* __restrict__ theta, const float* __restrict__ base,
                              const float* __restrict__ Y, int64_t n, const float* __restrict__ tmean,
                              const float* __restrict__ tstd, float alpha) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  for (int c = 0; c < 11; ++c) {
    const float dlt = Y[(size_t)i * 11 + c] * tstd[c] + tmean[c];
    theta[c * n + i] = base[c * n + i] + alpha * dlt;
  }
}

}  // namespace

// ---------------------------------------------------------------------------
// Host-side helpers.

namespace {

int64_t row_tiles(int64_t rows) { return (rows + 15) / 16; }

// Splits of the batch for the weight gradients: 512 rows each once a batch has
// more than 1,024 rows, else one (fewer rows a split would only lengthen the
// sums that follow, one split of 4,096 rows leaves the chip to 20 waves).
int64_t split_tiles(int64_t rows) { return rows > 1024 ? 32 : std::max<int64_t>(row_tiles(rows), 1); }

}  // namespace

// Workspace of mlp_step for up to `rows` rows (bytes, 256-byte aligned parts).
size_t mlp_step_bytes(int64_t rows) {
  const size_t t = (size_t)row_tiles(rows);
  const size_t splits = rows > 1024 ? (t + 31) / 32 : 1;
  return t * (2 + 4 * kHT) * kFrag * 2 + t * (1 + 2 * kHT) * 1024 + t * 8 +
         splits * GVE_MLP_NWEIGHT * 4 + 4096 + 16 * 256;
}

size_t mlp_stat_tmp_doubles() { return kStatBlocks * 16 * 2; }

hipError_t mlp_pack(const float* w, unsigned short* wf, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_pack, dim3((GVE_MLP_NWEIGHT + 255) / 256), dim3(256), 0, s, w, wf);
  return hipGetLastError();
}

hipError_t mlp_infer(const float* X, int64_t n, const float* stats, const float* w,
                     const unsigned short* wf, float* Y, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  // four workgroups (of 37 KB LDS) fit a CU: 1,024 fill the chip
  const unsigned blocks = (unsigned)std::min<int64_t>((n + 63) / 64, 1024);
  if (stats)
    hipLaunchKernelGGL((k_mlp_infer<true>), dim3(blocks), dim3(256), 0, s, X, n, stats, w, wf, Y);
  else
    hipLaunchKernelGGL((k_mlp_infer<false>), dim3(blocks), dim3(256), 0, s, X, n, stats, w, wf, Y);
  return hipGetLastError();
}

hipError_t mlp_step(const float* X, const float* T, const uint32_t* perm, int rows,
                    const float* stats, float* w, float* m, float* v, unsigned short* wf,
                    void* work, double loss_scale, double* loss, float* grad_out, float lr,
                    int64_t t, hipStream_t s) {
  const int64_t tiles = row_tiles(rows);
  char* p = static_cast<char*>(work);
  auto take = [&](size_t bytes) {
    char* q = p;
    p += (bytes + 255) & ~(size_t)255;
    return q;
  };
  MlpTiles o;
  const size_t one = (size_t)tiles * kFrag * 2, hid = one * kHT;
  o.x = reinterpret_cast<unsigned short*>(take(one));
  o.dy = reinterpret_cast<unsigned short*>(take(one));
  o.h1 = reinterpret_cast<unsigned short*>(take(hid));
  o.h2 = reinterpret_cast<unsigned short*>(take(hid));
  o.dz1 = reinterpret_cast<unsigned short*>(take(hid));
  o.dz2 = reinterpret_cast<unsigned short*>(take(hid));
  o.dy32 = reinterpret_cast<float4v*>(take(2 * one));
  o.dz132 = reinterpret_cast<float4v*>(take(2 * hid));
  o.dz232 = reinterpret_cast<float4v*>(take(2 * hid));
  o.loss = reinterpret_cast<double*>(take((size_t)tiles * 8));
  const int64_t per = split_tiles(rows);
  const int splits = (int)((tiles + per - 1) / per);
  float* bias = reinterpret_cast<float*>(take(4096));
  float* part = reinterpret_cast<float*>(take((size_t)splits * GVE_MLP_NWEIGHT * 4));
  const double inv = 1.0 / ((double)rows * kOut);
  if (stats)
    hipLaunchKernelGGL((k_mlp_fb<true, false>), dim3((unsigned)tiles), dim3(256), 0, s, X, T, perm, rows,
                       stats, w, wf, (float)inv, o);
  else
    hipLaunchKernelGGL((k_mlp_fb<false, false>), dim3((unsigned)tiles), dim3(256), 0, s, X, T, perm, rows,
                       stats, w, wf, (float)inv, o);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_mlp_wgrad, dim3((unsigned)(kBiasBlocks + kSplitBlocks * splits)), dim3(256),
                     0, s, o, tiles, per, part, bias);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  const double tt = (double)std::max<int64_t>(t, 1);
  const float ibc1 = (float)(1.0 / (1.0 - pow((double)b1, tt)));
  const float ibc2 = (float)(1.0 / (1.0 - pow((double)b2, tt)));
  hipLaunchKernelGGL(k_mlp_adam, dim3((GVE_MLP_NWEIGHT + 255) / 256), dim3(256), 0, s, part, splits,
                     bias, o.loss, tiles, inv * loss_scale, loss, grad_out, w, m, v, wf, lr, b1, b2,
                     eps, ibc1, ibc2);
  return hipGetLastError();
}

int64_t mlp_loss_tiles(int64_t rows) { return row_tiles(rows); }

hipError_t mlp_loss(const float* X, const float* T, int rows, const float* w,
                    const unsigned short* wf, double* tile_loss, double* loss, hipStream_t s) {
  const int64_t tiles = row_tiles(rows);
  const double inv = 1.0 / ((double)rows * kOut);
  MlpTiles o{};
  o.loss = tile_loss;
  hipLaunchKernelGGL((k_mlp_fb<false, true>), dim3((unsigned)tiles), dim3(256), 0, s, X, T, nullptr,
                     rows, nullptr, w, wf, (float)inv, o);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_mlp_loss, dim3(1), dim3(256), 0, s, tile_loss, tiles, inv, loss);
  return hipGetLastError();
}

hipError_t mlp_colstats(const float* X, int64_t rows, int cols, float* mean, float* stdv,
                        double* tmp, hipStream_t s) {
  hipLaunchKernelGGL(k_colstats_part, dim3(kStatBlocks), dim3(256), 0, s, X, rows, cols, tmp);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_colstats_final, dim3(1), dim3(64), 0, s, tmp, rows, cols, mean, stdv);
  return hipGetLastError();
}

hipError_t mlp_perm_keys(uint32_t* keys, uint32_t* vals, int64_t n, uint64_t seed, uint64_t epoch,
                         hipStream_t s) {
  hipLaunchKernelGGL(k_perm_keys, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, keys, vals, n,
                     seed, epoch);
  return hipGetLastError();
}

size_t mlp_feature_doubles(int64_t M, int64_t n) { return 2 * (size_t)M + 11 * (size_t)n + 1; }

hipError_t mlp_features(const float* f, const float* theta, int64_t n, int64_t n_detail,
                        const gve_grid& g, double g99, float k, double* work, float* X,
                        hipStream_t s) {
  const int64_t M = g.nx * g.ny * g.nz;
  double *s1 = work, *s2 = s1 + M, *J6 = s2 + M, *mom = J6 + 6 * n;
  FeatBox* box = reinterpret_cast<FeatBox*>(mom + 2 * n);
  unsigned long long* touched = reinterpret_cast<unsigned long long*>(mom + 5 * n);
  hipError_t e = fill_u64(touched, 1, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_feat_box, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, theta, n, g, k,
                     box, touched);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t lines = g.ny * g.nz;
  hipLaunchKernelGGL(k_sat_x, dim3((unsigned)std::min<int64_t>(lines, kSatLines)), dim3(256), 0, s,
                     f, g.nx, lines, touched, s1, s2);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  // along y: lines (x, z), inner = nx, len = ny, stride nx
  const int64_t ly = g.nx * g.nz;
  hipLaunchKernelGGL(k_sat_axis, dim3((unsigned)((ly + 255) / 256)), dim3(256), 0, s, s1, s2, ly,
                     g.nx, g.ny, g.nx, touched);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  // along z: lines (x, y), inner = nx * ny, len = nz, stride nx * ny
  const int64_t lz = g.nx * g.ny;
  hipLaunchKernelGGL(k_sat_axis, dim3((unsigned)((lz + 255) / 256)), dim3(256), 0, s, s1, s2, lz,
                     g.nx * g.ny, g.nz, g.nx * g.ny, touched);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  double2* T = reinterpret_cast<double2*>(work);
  const int64_t nbx = (g.nx + kSatX - 1) / kSatX, nby = (g.ny + kSatY - 1) / kSatY,
                nblocks = nbx * nby * ((g.nz + kSatZ - 1) / kSatZ);
  hipLaunchKernelGGL(k_sat_blocks, dim3((unsigned)std::min<int64_t>(nblocks, kSatBlocks)), dim3(64),
                     0, s, f, g, touched, nbx, nby, nblocks, T);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_box_sums, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s, T, n, g, box, touched,
                     mom);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  FeatArgs a{f, theta, n, n_detail, g, g99, s1, s2, J6, box, mom, touched, X};
  hipLaunchKernelGGL(k_feat_tensor, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s, f, theta, n, g,
                     J6);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_features, dim3((unsigned)((n + 127) / 128)), dim3(128), 0, s, a);
  return hipGetLastError();
}

hipError_t mlp_targets(const float* ta, const float* tr, int64_t n, float* T, hipStream_t s) {
  hipLaunchKernelGGL(k_targets, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, ta, tr, n, T);
  return hipGetLastError();
}

hipError_t mlp_apply_delta(float* theta, const float* base, const float* Y, int64_t n,
                           const float* tmean, const float* tstd, float alpha, hipStream_t s) {
  hipLaunchKernelGGL(k_apply_delta, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, theta, base,
                     Y, n, tmean, tstd, alpha);
  return hipGetLastError();
}

}  // namespace gve
