// The paper's own training loop on the device (Sec. III-C eq:field, Sec. III-F,
// Table tab:training-config): the density-normalised kernel regression
//     Vt(p) = sum_i w_i a_i G_i(p) / max(sum_i w_i G_i(p), rho0)
// of 12-parameter primitives (mu, raw quaternion, log-scales, attribute a,
// weight logit b with w = sigmoid(b)), trained on a few thousand stratified,
// jittered sample points per iteration against a six-term objective.
//
// Few samples and many primitives: the samples (and a nearby partner of each
// for the smoothness term) are bucketed into a uniform grid of cells; every
// primitive visits the cells its k-sigma box overlaps and tests the points
// there (the paper buckets samples per radius bin and tests a 3^3-cell
// neighbourhood; one grid with a box-sized cell range covers every radius).
//   k_pclass_count : per 256-voxel block, voxels of the high (V > v_hi) and
//                    mid (v_occ < V <= v_hi) classes (ballot counts);
//   k_psample      : one wave per sample: class member j = floor(u n_class)
//                    found through the block prefix sums and a ballot rank
//                    inside the block, jitter, partner, trilinear value;
//   k_pbucket      : the points of an iteration in cell order (one workgroup
//                    per iteration; more points take k_pcell_keys, the radix
//                    sort and k_pgather);
//   k_pfwd         : per primitive, sum_i w a G and sum_i w G into the points'
//                    float64 accumulators (atomics), and the points it reached;
//   k_pcoef        : per point, the coefficients of d(w a G) and d(w G) in
//                    dL/dtheta (quotient rule; the density floor passes no
//                    gradient), and the samples' terms of the objective;
//   k_pbwd         : per primitive, the gradient from those points (no atomics:
//                    each primitive owns its sums), the regularisers with their
//                    terms, and either the gradient (test hook) or the Adam step.
// Sampling and bucketing depend on no parameter, so refinement does them for
// many iterations at once: an iteration is three launches.
#include <algorithm>
#include <cmath>

#include "common.h"
#include "devmath.h"

namespace gve {
namespace {

constexpr int kThreads = 256;
constexpr int kBlockVox = 256;
constexpr uint64_t kStreamPick = 20, kStreamJit = 21, kStreamPartner = 24;

// ---- primitive geometry ---------------------------------------------------------

struct PGeom {
  float mu[3];
  float P[6];      // precision xx, xy, xz, yy, yz, zz
  float half[3];   // k sqrt(Sigma_jj): the k-sigma box half-extent per axis
  float a, w;
};

__device__ inline PGeom pgeom(const float* __restrict__ th, int64_t n, int64_t i, float k) {
  PGeom g;
  g.mu[0] = th[0 * n + i];
  g.mu[1] = th[1 * n + i];
  g.mu[2] = th[2 * n + i];
  float qw = th[3 * n + i], qx = th[4 * n + i], qy = th[5 * n + i], qz = th[6 * n + i];
  const float qn = sqrtf(qw * qw + qx * qx + qy * qy + qz * qz);
  if (qn >= 1e-12f) {
    const float inv = 1.0f / qn;
    qw *= inv; qx *= inv; qy *= inv; qz *= inv;
  } else {
    qw = 1.f; qx = qy = qz = 0.f;
  }
  const float R[3][3] = {
      {1.f - 2.f * (qy * qy + qz * qz), 2.f * (qx * qy - qw * qz), 2.f * (qx * qz + qw * qy)},
      {2.f * (qx * qy + qw * qz), 1.f - 2.f * (qx * qx + qz * qz), 2.f * (qy * qz - qw * qx)},
      {2.f * (qx * qz - qw * qy), 2.f * (qy * qz + qw * qx), 1.f - 2.f * (qx * qx + qy * qy)}};
  float is2[3], s2[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const float l = th[(7 + j) * n + i];
    is2[j] = expf(-2.f * l);
    s2[j] = expf(2.f * l);
  }
  auto prec = [&](int a, int b) {
    return R[a][0] * R[b][0] * is2[0] + R[a][1] * R[b][1] * is2[1] + R[a][2] * R[b][2] * is2[2];
  };
  g.P[0] = prec(0, 0);
  g.P[1] = prec(0, 1);
  g.P[2] = prec(0, 2);
  g.P[3] = prec(1, 1);
  g.P[4] = prec(1, 2);
  g.P[5] = prec(2, 2);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float sig = R[a][0] * R[a][0] * s2[0] + R[a][1] * R[a][1] * s2[1] + R[a][2] * R[a][2] * s2[2];
    g.half[a] = k * sqrtf(sig) * (1.0f + 1e-5f) + 1e-3f;
  }
  g.a = th[10 * n + i];
  g.w = 1.0f / (1.0f + expf(-th[11 * n + i]));
  return g;
}

__device__ inline float mahal2(const PGeom& g, float dx, float dy, float dz) {
  return g.P[0] * dx * dx + g.P[3] * dy * dy + g.P[5] * dz * dz +
         2.0f * (g.P[1] * dx * dy + g.P[2] * dx * dz + g.P[4] * dy * dz);
}

__device__ inline int cell_coord(float x, float org, float h, int nc) {
  const float c = floorf((x - org) / h);
  if (!(c > 0.f)) return 0;  // also NaN
  return c >= (float)nc ? nc - 1 : (int)c;
}

// Trilinear interpolation of the float32 volume at a world point (clamped):
// the cell's lower corner, the fractions in it, and the weighted sum of its
// eight corners (x fastest).
struct TriCell {
  int64_t lo[3];
  double fr[3];
};

__device__ inline TriCell tri_cell(const gve_grid& g, double px, double py, double pz) {
  const double p[3] = {px - (double)g.x0, py - (double)g.y0, pz - (double)g.z0};
  const int64_t dim[3] = {g.nx, g.ny, g.nz};
  TriCell t;
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    double x = fmin(fmax(p[j], 0.0), (double)(dim[j] - 1));
    if (dim[j] > 1) {
      int64_t i0 = (int64_t)floor(x);
      if (i0 > dim[j] - 2) i0 = dim[j] - 2;
      t.lo[j] = i0;
      t.fr[j] = x - (double)i0;
    } else {
      t.lo[j] = 0;
      t.fr[j] = 0.0;
    }
  }
  return t;
}

__device__ inline void tri_corners(const float* __restrict__ f, const gve_grid& g,
                                   const TriCell& t, float v[8]) {
  const int64_t sx = t.lo[0] + 1 < g.nx ? 1 : 0, sy = t.lo[1] + 1 < g.ny ? g.nx : 0,
                sz = t.lo[2] + 1 < g.nz ? g.nx * g.ny : 0;
  const float* p = f + (t.lo[0] + g.nx * (t.lo[1] + g.ny * t.lo[2]));
#pragma unroll
  for (int c = 0; c < 8; ++c)
    v[c] = p[(c & 1 ? sx : 0) + (c & 2 ? sy : 0) + (c & 4 ? sz : 0)];
}

__device__ inline double tri_sum(const TriCell& t, const float v[8]) {
  double acc = 0.0;
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const double wgt = (c & 1 ? t.fr[0] : 1.0 - t.fr[0]) * (c & 2 ? t.fr[1] : 1.0 - t.fr[1]) *
                       (c & 4 ? t.fr[2] : 1.0 - t.fr[2]);
    acc += wgt * (double)v[c];
  }
  return acc;
}

__device__ inline double trilinear(const float* __restrict__ f, const gve_grid& g, double px,
                                   double py, double pz) {
  const TriCell t = tri_cell(g, px, py, pz);
  float v[8];
  tri_corners(f, g, t, v);
  return tri_sum(t, v);
}

template <typename T>
__device__ inline T wave_sum(T v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
  return v;
}

// Block sum of up to three doubles, one atomic per block per value.
__device__ inline void block_add3(double a, double b, double c, double* __restrict__ out) {
  __shared__ double sh[kThreads / 64][3];
  a = wave_sum(a);
  b = wave_sum(b);
  c = wave_sum(c);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) {
    sh[wave][0] = a;
    sh[wave][1] = b;
    sh[wave][2] = c;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    double t = 0.0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += sh[w][threadIdx.x];
    if (t != 0.0) atomicAdd(&out[threadIdx.x], t);
  }
}

// ---- sampling -----------------------------------------------------------------------

__global__ __launch_bounds__(kThreads) void k_pclass_count(const float* __restrict__ f, int64_t M,
                                                           float v_hi, float v_occ,
                                                           uint32_t* __restrict__ cnt_hi,
                                                           uint32_t* __restrict__ cnt_mid,
                                                           int64_t nblocks) {
  const int64_t b = ((int64_t)blockIdx.x * kThreads + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (b >= nblocks) return;
  uint32_t h = 0, m = 0;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t v = b * kBlockVox + 4 * lane + r;
    if (v < M) {
      const float x = f[v];
      h += x > v_hi ? 1u : 0u;
      m += (x > v_occ && x <= v_hi) ? 1u : 0u;
    }
  }
  h = wave_sum(h);
  m = wave_sum(m);
  if (lane == 0) {
    cnt_hi[b] = h;
    cnt_mid[b] = m;
  }
}

__device__ inline bool in_class(float x, int cls, float v_hi, float v_occ) {
  return cls == 0 ? x > v_hi : (x > v_occ && x <= v_hi);
}

struct SampleCfg {
  gve_grid g;
  int64_t M, nblocks;
  int S, n_hi, n_mid, batch;
  uint64_t seed, it;
  float v_hi, v_occ;
};

// One wave per sample of `batch` consecutive iterations.  An iteration's points
// are stored as [2S][3] (sample s at row s, its smoothness partner at row
// S + s) and its S values follow in `vals`.
__global__ __launch_bounds__(kThreads) void k_psample(const float* __restrict__ f,
                                                      const uint32_t* __restrict__ off_hi,
                                                      const uint32_t* __restrict__ off_mid,
                                                      SampleCfg c, float* __restrict__ pts,
                                                      float* __restrict__ vals) {
  const int64_t wv = ((int64_t)blockIdx.x * kThreads + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (wv >= (int64_t)c.S * c.batch) return;
  const int s = (int)(wv % c.S);
  const int64_t bi = wv / c.S;
  pts += bi * 6 * c.S;
  vals += bi * c.S;
  const uint64_t idx = (c.it + (uint64_t)bi) * (uint64_t)c.S + (uint64_t)s;
  const double u = uniform01(c.seed, kStreamPick, idx);
  int64_t vox;
  if (s < c.n_hi + c.n_mid) {
    const int cls = s < c.n_hi ? 0 : 1;
    const uint32_t* off = cls == 0 ? off_hi : off_mid;
    const uint64_t total = off[c.nblocks];
    uint64_t j = (uint64_t)floor(u * (double)total);
    if (j >= total) j = total - 1;
    // block b: the last with off[b] <= j (off[lo] <= j throughout), the range
    // cut to a 64th by one probe per lane
    int64_t lo = 0, len = c.nblocks;
    while (len > 1) {
      const int64_t step = (len + 63) / 64, p = lane * step;
      const uint64_t le =
          __builtin_amdgcn_ballot_w64(p < len && (uint64_t)off[lo + p] <= j);
      const int64_t last = 63 - __builtin_clzll(le);
      lo += last * step;
      len = min(step, len - last * step);
    }
    const uint32_t r = (uint32_t)(j - off[lo]);
    // rank inside the block: lane L holds voxels 4L .. 4L+3 (ascending)
    uint32_t mine = 0;
    bool hit[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t v = lo * kBlockVox + 4 * lane + q;
      hit[q] = v < c.M && in_class(f[v], cls, c.v_hi, c.v_occ);
      mine += hit[q] ? 1u : 0u;
    }
    uint32_t incl = mine;  // inclusive prefix over lanes
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(incl, d, 64);
      if (lane >= d) incl += y;
    }
    const uint32_t excl = incl - mine;
    const bool owner = r >= excl && r < incl;
    int64_t found = 0;
    if (owner) {
      uint32_t k = r - excl;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (hit[q]) {
          if (k == 0) {
            found = lo * kBlockVox + 4 * lane + q;
            break;
          }
          --k;
        }
      }
    }
    const uint64_t ob = __builtin_amdgcn_ballot_w64(owner);
    const int src = ob ? __builtin_ffsll((long long)ob) - 1 : 0;
    vox = __shfl(found, src, 64);
  } else {
    vox = (int64_t)floor(u * (double)c.M);
    if (vox >= c.M) vox = c.M - 1;
  }
  if (lane == 0) {
    const int64_t ix = vox % c.g.nx, iy = (vox / c.g.nx) % c.g.ny, iz = vox / (c.g.nx * c.g.ny);
    const double base[3] = {(double)(c.g.x0 + ix), (double)(c.g.y0 + iy), (double)(c.g.z0 + iz)};
    double p[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      p[j] = base[j] + uniform01(c.seed, kStreamJit + j, idx) - 0.5;
      pts[3 * s + j] = (float)p[j];
      pts[3 * ((int64_t)c.S + s) + j] =
          (float)(p[j] + uniform01(c.seed, kStreamPartner + j, idx) - 0.5);
    }
    vals[s] = (float)trilinear(f, c.g, p[0], p[1], p[2]);
  }
}

__global__ __launch_bounds__(kThreads) void k_pcell_keys(const float* __restrict__ pts, int64_t np,
                                                         CellGrid cg, uint32_t* __restrict__ keys,
                                                         uint32_t* __restrict__ idx) {
  const int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (j >= np) return;
  const int cx = cell_coord(pts[3 * j + 0], cg.x0, cg.h, cg.ncx);
  const int cy = cell_coord(pts[3 * j + 1], cg.y0, cg.h, cg.ncy);
  const int cz = cell_coord(pts[3 * j + 2], cg.z0, cg.h, cg.ncz);
  keys[j] = (uint32_t)(cx + cg.ncx * (cy + cg.ncy * cz));
  idx[j] = (uint32_t)j;
}

// Points in cell order as (x, y, z, index): what the primitives' passes read.
__global__ __launch_bounds__(kThreads) void k_pgather(const float* __restrict__ pts, int64_t np,
                                                      const uint32_t* __restrict__ sorted,
                                                      float4* __restrict__ p4) {
  const int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (j >= np) return;
  const uint32_t i = sorted[j];
  p4[j] = make_float4(pts[3 * (size_t)i], pts[3 * (size_t)i + 1], pts[3 * (size_t)i + 2],
                      __uint_as_float(i));
}

// The same for one iteration's points in one workgroup: a stable radix sort of
// the cell keys in LDS (8 bits a pass; a wave ranks its own PER * 64 items in
// index order by ballots, so the rounds need no barrier), the points written in
// cell order and the cells' ranges found by binary search.  A dozen short
// launches otherwise; here the launch covers a whole batch of iterations, one
// workgroup each.
constexpr int kBucketThreads = 1024;
constexpr int kBucketWaves = kBucketThreads / 64;
template <int PER>
__global__ __launch_bounds__(kBucketThreads) void k_pbucket(const float* __restrict__ pts, int np,
                                                            CellGrid cg, int bits,
                                                            float4* __restrict__ p4,
                                                            uint32_t* __restrict__ start) {
  constexpr int kCap = PER * kBucketThreads;
  __shared__ uint32_t keys[kCap];
  __shared__ uint16_t ids[kCap];
  __shared__ uint32_t cnt[kBucketWaves][256];
  __shared__ uint32_t wsum[4];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int ncells = cg.ncx * cg.ncy * cg.ncz;
  pts += (size_t)blockIdx.x * 3 * np;
  p4 += (size_t)blockIdx.x * np;
  start += (size_t)blockIdx.x * (ncells + 1);
  uint32_t key[PER];
  uint32_t id[PER];
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    const int i = (wave * PER + r) * 64 + lane;
    id[r] = (uint32_t)i;
    key[r] = 0xFFFFFFFFu;  // past the points: after every cell
    if (i < np) {
      const int cx = cell_coord(pts[3 * i + 0], cg.x0, cg.h, cg.ncx);
      const int cy = cell_coord(pts[3 * i + 1], cg.y0, cg.h, cg.ncy);
      const int cz = cell_coord(pts[3 * i + 2], cg.z0, cg.h, cg.ncz);
      key[r] = (uint32_t)(cx + cg.ncx * (cy + cg.ncy * cz));
    }
  }
  for (int shift = 0; shift < bits; shift += 8) {
    if (shift > 0) {
#pragma unroll
      for (int r = 0; r < PER; ++r) {
        const int i = (wave * PER + r) * 64 + lane;
        key[r] = keys[i];
        id[r] = ids[i];
      }
    }
    volatile uint32_t* mine = cnt[wave];
    for (int d = lane; d < 256; d += 64) mine[d] = 0;
    uint32_t rank[PER];
#pragma unroll
    for (int r = 0; r < PER; ++r) {
      const uint32_t d = (key[r] >> shift) & 255u;
      uint64_t same = ~0ull;
#pragma unroll
      for (int bit = 0; bit < 8; ++bit) {
        const bool on = (d >> bit) & 1u;
        const uint64_t b = __builtin_amdgcn_ballot_w64(on);
        same &= on ? b : ~b;
      }
      // a wave's LDS operations complete in order: every lane reads the count
      // before the group's first lane raises it
      const uint32_t base = mine[d];
      const uint32_t below = (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
      rank[r] = base + below;
      if (below == 0) mine[d] = base + (uint32_t)__popcll(same);
    }
    __syncthreads();
    // digit bases (threads 0 .. 255, one digit each) and each wave's start
    uint32_t total = 0;
    if (t < 256)
      for (int w = 0; w < kBucketWaves; ++w) total += cnt[w][t];
    uint32_t inc = total;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(inc, d, 64);
      if (lane >= d) inc += y;
    }
    if (t < 256 && lane == 63) wsum[wave] = inc;
    __syncthreads();
    if (t < 256) {
      uint32_t run = inc - total;
      for (int w = 0; w < wave; ++w) run += wsum[w];
      for (int w = 0; w < kBucketWaves; ++w) {
        const uint32_t c = cnt[w][t];
        cnt[w][t] = run;
        run += c;
      }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < PER; ++r) {
      const uint32_t pos = cnt[wave][(key[r] >> shift) & 255u] + rank[r];
      keys[pos] = key[r];
      ids[pos] = (uint16_t)id[r];
    }
    __syncthreads();
  }
  if (bits <= 0) {  // one cell
    for (int j = t; j < np; j += kBucketThreads) {
      keys[j] = 0u;
      ids[j] = (uint16_t)j;
    }
    __syncthreads();
  }
  for (int j = t; j < np; j += kBucketThreads) {
    const int i = ids[j];
    p4[j] = make_float4(pts[3 * i], pts[3 * i + 1], pts[3 * i + 2], __uint_as_float((uint32_t)i));
  }
  for (int c = t; c <= ncells; c += kBucketThreads) {
    int lo = 0, hi = np;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (keys[mid] < (uint32_t)c) lo = mid + 1; else hi = mid;
    }
    start[c] = (uint32_t)lo;
  }
}

// ---- forward / backward over the cells a primitive's box overlaps -------------------

struct PairCfg {
  CellGrid cg;
  float k2;
  int64_t S;  // points [0, S) are samples (get the numerator), [S, np) partners
};

// Cells a primitive's box overlaps.  The cells of one row (fixed y and z) are
// consecutive, so a row is one range of points.
struct BoxCells {
  int x0, x1, y0, y1, z0, z1;
};

__device__ inline BoxCells box_cells(const PGeom& g, const CellGrid& cg) {
  BoxCells b;
  b.x0 = cell_coord(g.mu[0] - g.half[0], cg.x0, cg.h, cg.ncx);
  b.x1 = cell_coord(g.mu[0] + g.half[0], cg.x0, cg.h, cg.ncx);
  b.y0 = cell_coord(g.mu[1] - g.half[1], cg.y0, cg.h, cg.ncy);
  b.y1 = cell_coord(g.mu[1] + g.half[1], cg.y0, cg.h, cg.ncy);
  b.z0 = cell_coord(g.mu[2] - g.half[2], cg.z0, cg.h, cg.ncz);
  b.z1 = cell_coord(g.mu[2] + g.half[2], cg.z0, cg.h, cg.ncz);
  return b;
}

// fn(j, d, G) for every point (position j in cell order) inside the support.
template <typename F>
__device__ inline void for_points(const PGeom& g, const PairCfg& c, const float4* __restrict__ p4,
                                  const uint32_t* __restrict__ start, F&& fn) {
  const BoxCells b = box_cells(g, c.cg);
  for (int cz = b.z0; cz <= b.z1; ++cz)
    for (int cy = b.y0; cy <= b.y1; ++cy) {
      const uint32_t row = (uint32_t)(c.cg.ncx * (cy + c.cg.ncy * cz));
      const uint32_t e = start[row + b.x1 + 1];
      for (uint32_t j = start[row + b.x0]; j < e; ++j) {
        const float4 q = p4[j];
        const float dx = q.x - g.mu[0];
        const float dy = q.y - g.mu[1];
        const float dz = q.z - g.mu[2];
        const float m2 = mahal2(g, dx, dy, dz);
        if (m2 < c.k2) fn(j, dx, dy, dz, expf(-0.5f * m2));
      }
    }
}

// Forward pass, one wave per 64 primitives.  The rows of a primitive's box hold
// a handful of points each, unevenly: with a lane per primitive a wave takes as
// many steps as its busiest lane (some fifty, nine of them useful on average).
// So the lanes only collect their candidate points, four a lane and round, into
// a list in LDS that is then tested 64 at a time.
//
// Points a primitive reached are kept for the backward pass: the wave's lists,
// primitive after primitive, in its 64 kPaperHits entries of hit_list, and
// hit_range [n] = first entry << 16 | number.  A wave that reached more keeps
// none (kAllPoints): the backward pass then searches again.
constexpr int kWavePrims = 64;
constexpr int kCandidates = 512;
constexpr int kWaveHits = kWavePrims * kPaperHits;
constexpr uint32_t kAllPoints = 0xFFFFu;

// Inclusive prefix sum over a wave by data-parallel moves (no LDS traffic): four
// shifts within the rows of sixteen lanes, then the rows' totals.
__device__ inline uint32_t wave_scan(uint32_t v) {
  int x = (int)v;
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);  // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);  // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);  // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31
  return (uint32_t)x;
}

__global__ __launch_bounds__(kWavePrims) void k_pfwd(const float* __restrict__ th, int64_t n,
                                                     PairCfg c, float k,
                                                     const float4* __restrict__ p4,
                                                     const uint32_t* __restrict__ start,
                                                     double* __restrict__ num,
                                                     double* __restrict__ den,
                                                     uint32_t* __restrict__ hit_range,
                                                     uint32_t* __restrict__ hit_list) {
  __shared__ uint32_t cand[kCandidates];     // candidate points
  __shared__ uint8_t cand_of[kCandidates];   // and their primitives
  __shared__ uint32_t hit[kWaveHits];
  __shared__ uint8_t hit_of[kWaveHits];
  __shared__ uint32_t nhit[kWavePrims];
  const int lane = threadIdx.x;
  const int64_t i = (int64_t)blockIdx.x * kWavePrims + lane;
  const uint64_t below = (1ull << lane) - 1ull;
  PGeom g{};
  BoxCells b{0, 0, 0, -1, 0, 0};
  if (i < n) {
    g = pgeom(th, n, i, k);
    b = box_cells(g, c.cg);
  }
  nhit[lane] = 0;
  uint32_t listed = 0, kept = 0;  // candidates waiting, points kept (uniform)
  int cy = b.y0 - 1, cz = b.z0;   // row walked last
  bool rows = i < n;
  // tests the listed candidates, 64 at a time; the next ones' points are loaded
  // meanwhile
  auto flush = [&]() {
    __syncthreads();
    uint32_t on = 0, cn = 0;
    float4 qn = make_float4(0.f, 0.f, 0.f, 0.f);
    if ((uint32_t)lane < listed) {
      on = cand_of[lane];
      cn = cand[lane];
      qn = p4[cn];
    }
    for (uint32_t t0 = 0; t0 < listed; t0 += 64) {
      const bool live = t0 + lane < listed;
      const uint32_t o = on, cj = cn;
      const float4 q = qn;
      if (t0 + 64 + lane < listed) {
        on = cand_of[t0 + 64 + lane];
        cn = cand[t0 + 64 + lane];
        qn = p4[cn];
      }
      // the primitive's geometry, from the lane that holds it
      PGeom go;
#pragma unroll
      for (int a = 0; a < 6; ++a) go.P[a] = __shfl(g.P[a], (int)o, 64);
      const float m2 = mahal2(go, q.x - __shfl(g.mu[0], (int)o, 64),
                              q.y - __shfl(g.mu[1], (int)o, 64),
                              q.z - __shfl(g.mu[2], (int)o, 64));
      const float ow = __shfl(g.w, (int)o, 64), oa = __shfl(g.a, (int)o, 64);
      const uint32_t pi = __float_as_uint(q.w);
      const bool in = live && m2 < c.k2;
      if (in) {
        const float wg = ow * expf(-0.5f * m2);
        atomicAdd(&den[pi], (double)wg);
        if ((int64_t)pi < c.S) atomicAdd(&num[pi], (double)(wg * oa));
      }
      if (hit_range) {
        const uint64_t hm = __builtin_amdgcn_ballot_w64(in);
        const uint32_t pos = kept + (uint32_t)__popcll(hm & below);
        if (in && pos < (uint32_t)kWaveHits) {
          hit[pos] = cj;
          hit_of[pos] = (uint8_t)o;
          atomicAdd(&nhit[o], 1u);
        }
        kept += (uint32_t)__popcll(hm);
      }
    }
    listed = 0;
    __syncthreads();
  };
  while (__builtin_amdgcn_ballot_w64(rows) != 0ull) {
    // the lane's next rows, their ranges loaded together
    constexpr int kRows = 4;
    uint32_t j[kRows], e[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      j[r] = e[r] = 0;
      if (rows && ++cy > b.y1) {
        cy = b.y0;
        if (++cz > b.z1) rows = false;
      }
      if (rows) {
        const uint32_t row = (uint32_t)(c.cg.ncx * (cy + c.cg.ncy * cz));
        j[r] = start[row + b.x0];
        e[r] = start[row + b.x1 + 1];
      }
    }
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      // up to four points of every lane join the list, lane after lane
      while (__builtin_amdgcn_ballot_w64(j[r] < e[r]) != 0ull) {
        const uint32_t m = min(e[r] - j[r], 4u);
        const uint32_t inc = wave_scan(m);
        const uint32_t at = listed + inc - m;
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q)
          if (q < m) {
            cand[at + q] = j[r] + q;
            cand_of[at + q] = (uint8_t)lane;
          }
        j[r] += m;
        listed += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
        // room for one more round of 4 x 64
        if (listed > kCandidates - 4 * kWavePrims) flush();
      }
    }
  }
  flush();
  if (!hit_range) return;
  uint32_t* out = hit_list + (size_t)blockIdx.x * kWaveHits;
  if (kept > (uint32_t)kWaveHits) {
    if (i < n) hit_range[i] = kAllPoints;
    return;
  }
  // entries grouped by primitive, in order: first entry of each primitive, then
  // an entry's place among its primitive's (entries of one primitive in a
  // step are ranked by lane)
  const uint32_t mine = nhit[lane];
  const uint32_t inc = wave_scan(mine);
  __syncthreads();
  nhit[lane] = inc - mine;
  if (i < n) hit_range[i] = ((inc - mine) << 16) | mine;
  __syncthreads();
  for (uint32_t t0 = 0; t0 < kept; t0 += 64) {
    const uint32_t t = t0 + lane;
    const bool live = t < kept;
    const uint32_t o = live ? hit_of[t] : 255u;
    uint64_t left = __builtin_amdgcn_ballot_w64(live);
    uint32_t pos = 0;
    while (left) {
      const int l = __builtin_ctzll(left);
      const uint32_t ol = __shfl(o, l, 64);
      const uint64_t same = __builtin_amdgcn_ballot_w64(o == ol);
      if (o == ol) {
        const uint32_t base = nhit[ol];
        pos = base + (uint32_t)__popcll(same & below);
        // read by every lane of the group before its first lane raises it
        if ((same & below) == 0ull) nhit[ol] = base + (uint32_t)__popcll(same);
      }
      left &= ~same;
    }
    if (live) out[pos] = hit[t];
  }
}

struct CoefCfg {
  int64_t S;
  double rho0, lam_rho, lam_sm, v_occ;
  const double *num, *den;
  const float* vals;
};

// Coefficients of d(w a G) (samples only) and of d(w G) of the point at each
// position of the cell order, and the samples' terms of the objective.
__global__ __launch_bounds__(kThreads) void k_pcoef(CoefCfg c, const float4* __restrict__ p4,
                                                    float2* __restrict__ coef,
                                                    double* __restrict__ loss) {
  const int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  double lv = 0.0, lr = 0.0, ls = 0.0;
  if (j < 2 * c.S) {
    const int64_t pi = (int64_t)__float_as_uint(p4[j].w);
    const int64_t s = pi < c.S ? pi : pi - c.S;
    const double d1 = c.den[s], d2 = c.den[c.S + s];
    float2 o;
    if (pi >= c.S) {
      o.x = 0.0f;
      o.y = (float)(-2.0 * c.lam_sm * (d1 - d2));
    } else {
      const double D = fmax(d1, c.rho0);
      const double vt = c.num[s] / D;
      const double val = (double)c.vals[s];
      const bool occ = val > c.v_occ;
      const double u = occ ? 2.0 * (vt - val) : 0.0;
      const double v = (occ ? 2.0 * c.lam_rho * (d1 - 1.0) : 0.0) + 2.0 * c.lam_sm * (d1 - d2);
      o.x = (float)(u / D);
      o.y = (float)(v - (d1 > c.rho0 ? u * vt / D : 0.0));
      if (occ) {
        lv = (vt - val) * (vt - val);
        lr = (d1 - 1.0) * (d1 - 1.0);
      }
      ls = (d1 - d2) * (d1 - d2);
    }
    coef[j] = o;
  }
  block_add3(lv, lr, ls, loss + (blockIdx.x % kPaperSlots) * 6);
}

struct BwdCfg {
  float k, lam_anc, lam_aniso, lam_cap, log_aniso, ell_lo, ell_hi;
  float lr, b1, b2, eps, inv_bc1, inv_bc2;
  int mode;        // 0: write the gradient; 1: Adam step
  double* clear;   // the accumulators of the next iteration, zeroed here
  int64_t nclear;
};

// Gradient, regularisers and step of every primitive, and their terms of the
// objective into loss[slot][3 ..] (slot = block mod kPaperSlots, so that the
// blocks' atomics do not queue on one address).  With `corner`, the eight volume
// values around a centre are kept from iteration to iteration of one call
// ([9][n]: the cell's first voxel, then its corners): a centre moves by about the
// learning rate, so it rarely leaves its cell, and the eight values are read
// side by side instead of from four lines all over the volume (at 400,000
// primitives some 200 MB an iteration).  Bound by the parameters and moments it
// reads and writes (288 bytes a primitive).
__global__ __launch_bounds__(kThreads) void k_pbwd(float* __restrict__ th, float* __restrict__ m,
                                                   float* __restrict__ v, int64_t n, PairCfg c,
                                                   BwdCfg b, const float4* __restrict__ p4,
                                                   const uint32_t* __restrict__ start,
                                                   const float2* __restrict__ coef,
                                                   const uint32_t* __restrict__ hit_range,
                                                   const uint32_t* __restrict__ hit_list,
                                                   const float* __restrict__ field, gve_grid fg,
                                                   float* __restrict__ corner,
                                                   float* __restrict__ grad_out,
                                                   double* __restrict__ loss) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  // the next iteration's accumulators
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  for (int64_t j = i; j < b.nclear; j += stride) b.clear[j] = 0.0;
  double la = 0.0, lan = 0.0, lc = 0.0;
  if (i < n) {
    const uint32_t hr = hit_range[i];
    const uint32_t nh = hr & 0xFFFFu;
    float t[12], gr[12];
#pragma unroll
    for (int a = 0; a < 12; ++a) t[a] = th[a * n + i];
    const TriCell tc = tri_cell(fg, (double)t[0], (double)t[1], (double)t[2]);
    float cv[8];
    if (corner) {
      const uint32_t at = (uint32_t)(tc.lo[0] + fg.nx * (tc.lo[1] + fg.ny * tc.lo[2]));
#pragma unroll
      for (int q = 0; q < 8; ++q) cv[q] = corner[(1 + q) * n + i];
      if (__float_as_uint(corner[i]) != at) {
        tri_corners(field, fg, tc, cv);
        corner[i] = __uint_as_float(at);
#pragma unroll
        for (int q = 0; q < 8; ++q) corner[(1 + q) * n + i] = cv[q];
      }
    } else {
      tri_corners(field, fg, tc, cv);
    }
    const double aref = tri_sum(tc, cv);
    float sgd[3] = {0.f, 0.f, 0.f}, D[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float dA = 0.f, dB = 0.f;
    const float w = 1.0f / (1.0f + expf(-t[11]));
    if (nh > 0) {
      const PGeom g = pgeom(th, n, i, b.k);
      auto add = [&](uint32_t j, float dx, float dy, float dz, float G) {
        const float2 cj = coef[j];
        const float cA = cj.x, cB = cj.y;
        const float e = fmaf(cA, g.a, cB);  // coefficient of d(w G)
        const float gc = e * g.w * G;
        sgd[0] = fmaf(gc, dx, sgd[0]);
        sgd[1] = fmaf(gc, dy, sgd[1]);
        sgd[2] = fmaf(gc, dz, sgd[2]);
        D[0] = fmaf(gc * dx, dx, D[0]);
        D[1] = fmaf(gc * dx, dy, D[1]);
        D[2] = fmaf(gc * dx, dz, D[2]);
        D[3] = fmaf(gc * dy, dy, D[3]);
        D[4] = fmaf(gc * dy, dz, D[4]);
        D[5] = fmaf(gc * dz, dz, D[5]);
        dA = fmaf(cA * g.w, G, dA);
        dB = fmaf(e, G, dB);
      };
      if (nh != kAllPoints) {
        const uint32_t* mine = hit_list + (size_t)(i / kWavePrims) * kWaveHits + (hr >> 16);
        for (uint32_t h = 0; h < nh; ++h) {
          const uint32_t j = mine[h];
          const float4 q = p4[j];
          const float dx = q.x - g.mu[0];
          const float dy = q.y - g.mu[1];
          const float dz = q.z - g.mu[2];
          add(j, dx, dy, dz, expf(-0.5f * mahal2(g, dx, dy, dz)));
        }
      } else {
        for_points(g, c, p4, start, add);
      }
    }
    geometry_grad(&t[3], &t[7], sgd, D, gr);
    gr[10] = dA;
    gr[11] = dB * w * (1.0f - w);
    // regularisers
    const double da = (double)t[10] - aref;
    gr[10] += (float)(2.0 * b.lam_anc * da);
    la = da * da;
    int jmax = 0, jmin = 0;
#pragma unroll
    for (int j = 1; j < 3; ++j) {
      if (t[7 + j] > t[7 + jmax]) jmax = j;
      if (t[7 + j] < t[7 + jmin]) jmin = j;
    }
    const float spread = t[7 + jmax] - t[7 + jmin] - b.log_aniso;
    if (spread > 0.f) {
      gr[7 + jmax] += 2.f * b.lam_aniso * spread;
      gr[7 + jmin] -= 2.f * b.lam_aniso * spread;
      lan = (double)spread * spread;
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const float l = t[7 + j];
      if (l > b.ell_hi) {
        gr[7 + j] += 2.f * b.lam_cap * (l - b.ell_hi);
        lc += (double)(l - b.ell_hi) * (l - b.ell_hi);
      }
      if (l < b.ell_lo) {
        gr[7 + j] -= 2.f * b.lam_cap * (b.ell_lo - l);
        lc += (double)(b.ell_lo - l) * (b.ell_lo - l);
      }
    }
    if (b.mode == 0) {
#pragma unroll
      for (int a = 0; a < 12; ++a) grad_out[a * n + i] = gr[a];
    } else {
#pragma unroll
      for (int a = 0; a < 12; ++a) {
        float mm = m[a * n + i], vv = v[a * n + i];
        mm = b.b1 * mm + (1.0f - b.b1) * gr[a];
        vv = b.b2 * vv + (1.0f - b.b2) * gr[a] * gr[a];
        m[a * n + i] = mm;
        v[a * n + i] = vv;
        th[a * n + i] = t[a] - b.lr * (mm * b.inv_bc1) / (sqrtf(vv * b.inv_bc2) + b.eps);
      }
    }
  }
  block_add3(la, lan, lc, loss + (blockIdx.x % kPaperSlots) * 6 + 3);
}

// Marks every primitive's corner values as not read yet (no cell starts at
// voxel 2^32 - 1: volumes have fewer voxels).
__global__ __launch_bounds__(kThreads) void k_pcorner_reset(float* __restrict__ corner, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i < n) corner[i] = __uint_as_float(0xFFFFFFFFu);
}

__global__ __launch_bounds__(kThreads) void k_pfill_d(double* __restrict__ p, int64_t n) {
  for (int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x; j < n;
       j += (int64_t)gridDim.x * kThreads)
    p[j] = 0.0;
}

__global__ __launch_bounds__(kThreads) void k_pdensity(const double* __restrict__ num,
                                                       const double* __restrict__ den,
                                                       int64_t np, float rho0,
                                                       float* __restrict__ vt,
                                                       float* __restrict__ dn) {
  const int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (j >= np) return;
  const double d = den[j];
  if (vt) vt[j] = (float)(num[j] / fmax(d, (double)rho0));
  if (dn) dn[j] = (float)d;
}

unsigned blocks_for(int64_t n) { return (unsigned)((n + kThreads - 1) / kThreads); }

}  // namespace

CellGrid make_cells(const gve_grid& g, float h) {
  CellGrid cg;
  cg.x0 = (float)g.x0 - 0.5f;
  cg.y0 = (float)g.y0 - 0.5f;
  cg.z0 = (float)g.z0 - 0.5f;
  cg.h = h;
  cg.ncx = (int)std::max<int64_t>(1, (int64_t)std::ceil((double)g.nx / h));
  cg.ncy = (int)std::max<int64_t>(1, (int64_t)std::ceil((double)g.ny / h));
  cg.ncz = (int)std::max<int64_t>(1, (int64_t)std::ceil((double)g.nz / h));
  return cg;
}

int64_t paper_class_blocks(int64_t M) { return (M + kBlockVox - 1) / kBlockVox; }

hipError_t paper_class_counts(const float* f, int64_t M, float v_hi, float v_occ, uint32_t* cnt_hi,
                              uint32_t* cnt_mid, hipStream_t s) {
  const int64_t nb = paper_class_blocks(M);
  hipLaunchKernelGGL(k_pclass_count, dim3(blocks_for(nb * 64)), dim3(kThreads), 0, s, f, M, v_hi,
                     v_occ, cnt_hi, cnt_mid, nb);
  return hipGetLastError();
}

hipError_t paper_sample(const float* f, const gve_grid& g, const uint32_t* off_hi,
                        const uint32_t* off_mid, int S, int n_hi, int n_mid, uint64_t seed,
                        uint64_t it, int batch, float v_hi, float v_occ, float* pts, float* vals,
                        hipStream_t s) {
  SampleCfg c;
  c.g = g;
  c.M = g.nx * g.ny * g.nz;
  c.nblocks = paper_class_blocks(c.M);
  c.S = S;
  c.n_hi = n_hi;
  c.n_mid = n_mid;
  c.batch = batch;
  c.seed = seed;
  c.it = it;
  c.v_hi = v_hi;
  c.v_occ = v_occ;
  hipLaunchKernelGGL(k_psample, dim3(blocks_for((int64_t)S * 64 * batch)), dim3(kThreads), 0, s, f,
                     off_hi, off_mid, c, pts, vals);
  return hipGetLastError();
}

// A workgroup's LDS holds 16,384 points (114 KB); the positions are 16 bits.  One
// workgroup also finds every cell's range of a set, about 1 ns a cell, beside
// those of the other sets, while the radix sort and the chip-wide ranges take some
// 45 us a set: an iteration of 3,072 samples in batches, 4,096 cells 26 us
// (sorted: 76), 262,144 33 (94), 636,056 52 (98), 2.1 million 307 (108), 12.6
// million 10,660 (171); one evaluation at 6,144 points, 4,096 cells 33 us (53),
// 32,768 57 (54), 79,507 103 (68); at 16,384 points, 4,096 cells 59 (57).
bool paper_buckets_in_lds(int64_t np, int64_t ncells, int batch) {
  return np <= 16 * kBucketThreads &&
         ncells <= (int64_t)32768 * (np <= 8 * kBucketThreads ? batch : batch - 1);
}

hipError_t paper_bucket(const float* pts, int np, const CellGrid& cg, int bits, int batch,
                        float4* p4, uint32_t* start, hipStream_t s) {
  if (np <= 8 * kBucketThreads)
    hipLaunchKernelGGL((k_pbucket<8>), dim3((unsigned)batch), dim3(kBucketThreads), 0, s, pts, np,
                       cg, bits, p4, start);
  else
    hipLaunchKernelGGL((k_pbucket<16>), dim3((unsigned)batch), dim3(kBucketThreads), 0, s, pts, np,
                       cg, bits, p4, start);
  return hipGetLastError();
}

hipError_t paper_gather(const float* pts, int64_t np, const uint32_t* sorted, float4* p4,
                        hipStream_t s) {
  hipLaunchKernelGGL(k_pgather, dim3(blocks_for(np)), dim3(kThreads), 0, s, pts, np, sorted, p4);
  return hipGetLastError();
}

hipError_t paper_cell_keys(const float* pts, int64_t np, const CellGrid& cg, uint32_t* keys,
                           uint32_t* idx, hipStream_t s) {
  hipLaunchKernelGGL(k_pcell_keys, dim3(blocks_for(np)), dim3(kThreads), 0, s, pts, np, cg, keys,
                     idx);
  return hipGetLastError();
}

hipError_t paper_zero(double* p, int64_t n, hipStream_t s) {
  const int64_t blocks = std::min<int64_t>((n + kThreads - 1) / kThreads, 4096);
  if (blocks <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_pfill_d, dim3((unsigned)blocks), dim3(kThreads), 0, s, p, n);
  return hipGetLastError();
}

size_t paper_hit_words(int64_t n) {
  return (size_t)n + (size_t)((n + kWavePrims - 1) / kWavePrims) * kWaveHits;
}

hipError_t paper_forward(const float* th, int64_t n, const CellGrid& cg, float k, int64_t S,
                         const float4* p4, const uint32_t* start, double* num, double* den,
                         uint32_t* hits, hipStream_t s) {
  PairCfg c;
  c.cg = cg;
  c.k2 = k * k;
  c.S = S;
  hipLaunchKernelGGL(k_pfwd, dim3((unsigned)((n + kWavePrims - 1) / kWavePrims)),
                     dim3(kWavePrims), 0, s, th, n, c, k, p4, start, num, den, hits,
                     hits ? hits + n : nullptr);
  return hipGetLastError();
}

hipError_t paper_density(const double* num, const double* den, int64_t np, float rho0, float* vt,
                         float* dn, hipStream_t s) {
  hipLaunchKernelGGL(k_pdensity, dim3(blocks_for(np)), dim3(kThreads), 0, s, num, den, np, rho0, vt,
                     dn);
  return hipGetLastError();
}

hipError_t paper_coef(int64_t S, const gve_paper_options& o, float lam_sm, const float4* p4,
                      const double* num, const double* den, const float* vals, float2* coef,
                      double* loss, hipStream_t s) {
  CoefCfg cc;
  cc.S = S;
  cc.rho0 = o.rho0;
  cc.lam_rho = o.lam_rho;
  cc.lam_sm = lam_sm;
  cc.v_occ = o.v_occ;
  cc.num = num;
  cc.den = den;
  cc.vals = vals;
  hipLaunchKernelGGL(k_pcoef, dim3(blocks_for(2 * S)), dim3(kThreads), 0, s, cc, p4, coef, loss);
  return hipGetLastError();
}

hipError_t paper_corner_reset(float* corner, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_pcorner_reset, dim3(blocks_for(n)), dim3(kThreads), 0, s, corner, n);
  return hipGetLastError();
}

hipError_t paper_backward(float* th, float* m, float* v, int64_t n, const CellGrid& cg,
                          const gve_paper_options& o, int mode, int64_t t, const float4* p4,
                          const uint32_t* start, const float2* coef, const uint32_t* hits,
                          const float* field, const gve_grid& fg, float* corner, float* grad_out,
                          double* loss, double* clear, int64_t nclear, hipStream_t s) {
  PairCfg c;
  c.cg = cg;
  c.k2 = o.k * o.k;
  c.S = 0;  // the coefficients already tell samples from partners
  BwdCfg b;
  b.clear = clear;
  b.nclear = nclear;
  b.k = o.k;
  b.lam_anc = o.lam_anc;
  b.lam_aniso = o.lam_aniso;
  b.lam_cap = o.lam_cap;
  b.log_aniso = logf(o.aniso_max);
  b.ell_lo = o.ell_lo;
  b.ell_hi = o.ell_hi;
  b.lr = o.lr;
  b.b1 = o.beta1;
  b.b2 = o.beta2;
  b.eps = o.eps;
  const double tt = (double)(t > 0 ? t : 1);
  b.inv_bc1 = (float)(1.0 / (1.0 - std::pow((double)o.beta1, tt)));
  b.inv_bc2 = (float)(1.0 / (1.0 - std::pow((double)o.beta2, tt)));
  b.mode = mode;
  hipLaunchKernelGGL(k_pbwd, dim3(blocks_for(n)), dim3(kThreads), 0, s, th, m, v, n, c, b,
                     p4, start, coef, hits, hits + n, field, fg, corner, grad_out, loss);
  return hipGetLastError();
}

}  // namespace gve
