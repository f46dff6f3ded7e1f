// Structure-aware fixed-budget allocation on the device (paper Sec. III-E;
// stages S1a-S1e of the stage table):
//
//   S1a  k_survey       : |grad V| per voxel (float32 central differences,
//                         one-sided at the faces; magnitude formed in double
//                         and rounded to float), occupied / eligible counts.
//   S1b  k_mark .. k_list_write : the N_det detail seeds (probability ~ |grad V|
//                         over V > 0.02, without replacement: exponential-clock
//                         keys -ln(u)/g, the N_det smallest) and the N_cov
//                         coverage seeds (uniform keys), ties to the lower voxel
//                         index; u from the SplitMix64 finaliser of the counter
//                         (seed, stream, voxel).
//   S1b  k_jitter       : off-grid centre c + u - 1/2 per axis.
//   S1c  k_nn / k_median: per group, the lower median over a strided subsample
//                         (<= 4096 seeds) of nearest-neighbour distances.
//   S1d/e k_assemble    : 7^3 structure tensor, Jacobi eigen
//                         frame R = [e3, e2, e1] (tangent = smallest
//                         eigenvalue), scales from the group spacing elongated
//                         along the tangent with the gradient, value V(c).
//   weights             : one truncated evaluation U = sum a_i G_i, then
//                         kappa = <U, V> / <U, U> scales every weight.
#include <algorithm>

#include "common.h"
#include "devmath.h"

namespace gve {
namespace {

constexpr int kThreads = 256;
constexpr int kBlockVox = 4096;             // voxels (or list entries) of one count
constexpr int kWords = kBlockVox / 64;      // mask words of a voxel block
constexpr float kOcc = 0.02f;

template <typename T>
__device__ inline T wave_reduce_add(T v) {
#pragma unroll
  for (int s = 32; s >= 1; s >>= 1) v += __shfl_xor(v, s, 64);
  return v;
}

__device__ inline uint32_t block_excl_scan(uint32_t v, uint32_t* wsum) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t inc = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    uint32_t u = __shfl_up(inc, d, 64);
    if (lane >= d) inc += u;
  }
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  uint32_t before = 0;
  for (int w = 0; w < wave; ++w) before += wsum[w];
  __syncthreads();
  return before + inc - v;
}

// ---- S1a / S1b: gradients, the two draws and the 99th percentile --------------
//
// Both draws keep the voxels with the N smallest 64-bit keys (ties to the
// lower index): detail (V > 0.02, g > 0) the bits of -ln(u) / g as a positive
// double, coverage (V > 0.02) the top 53 bits of a hash.  Evaluating a key in
// double costs a logarithm and a division, and only a sliver of the volume can
// be drawn, so the volume is read twice:
//   k_survey  gradient magnitudes, domain counts, and histograms of cheap keys:
//             for detail a float approximation of the key (its top 12 bits,
//             eight bins per octave), for coverage the key's own top 11 bits,
//             and of g's top 12 bits;
//   k_pick    the bin that holds the Nth key.  A float key is within 1e-4 of
//             the exact one and a bin is at least 6 % wide, so with c(b) keys
//             in bins <= b >= N, the Nth exact key lies below the top of bin
//             b + 1 by more than that: every drawn voxel is in bins <= b + 1;
//   k_mark    bit masks of those voxels (about 1.2 N) and their number per block;
//   k_gather  their exact keys and indices, in voxel order;
//   k_list_*  exact selection of the N smallest from that list.
// The 99th percentile of g is refined by two more histograms of 10 bits each
// (in k_mark and k_digit).  512^3 voxels, 262,144 seeds: 13.6 ms with a radix
// select that evaluated exact keys over the volume in 21 passes, 2.3 ms now.

constexpr int kDetBins = 2048, kCovBins = 2048, kGBins = 4096, kLowBins = 1024;
constexpr int kSurveyBins = kDetBins + kCovBins + kGBins;

// Device block of the draws (u64 words).
enum {
  kOccupied = 0, kEligible = 1,           // domain counts
  kDetBin = 2, kDetCount = 3,             // last candidate bin, candidates
  kCovBin = 4, kCovCount = 5,
  kGBin = 6, kGRank = 7,                  // prefix of the percentile, rank left in it
  kHist = 16,                             // survey histograms
  kLowHist = kHist + kSurveyBins,         // two histograms of 10 bits
  kListState = kLowHist + 2 * kLowBins,   // (prefix, rank) of detail, coverage
  kListHist = kListState + 4,             // two histograms of 8 bits
  kSelectWords = kListHist + 512
};

// Counter hash of (seed, stream, index) with the (seed, stream) part done.
__device__ inline uint64_t hash_at(uint64_t stream_seed, uint64_t v) {
  return splitmix64(stream_seed ^ v);
}

// Key of a coverage voxel: 53 hash bits.
__device__ inline uint64_t cov_key(uint64_t cov_seed, uint64_t v) {
  return hash_at(cov_seed, v) >> 11;
}

// Key of a detail voxel: -ln(u) / g, u = (top 53 bits + 1) 2^-53.
__device__ inline uint64_t det_key(uint64_t det_seed, uint64_t v, float g) {
  const double u = (double)((hash_at(det_seed, v) >> 11) + 1ull) * 0x1.0p-53;
  const double kd = -log(u) / (double)g;
  return (uint64_t)__double_as_longlong(kd);
}

// Bin of a float approximation of that key.  With d = 1 - u (exact as an
// integer), -ln(1 - d) is its series below 2^-8 and the hardware logarithm of
// u above: relative error below 1e-4.  u = 1 (key -0, the largest as bits)
// goes to the top.
__device__ inline uint32_t det_bin(uint64_t det_seed, uint64_t v, float g) {
  const uint64_t h = hash_at(det_seed, v);
  const uint64_t di = ~h >> 11;
  if (di == 0) return kDetBins - 1;
  const float d = (float)di * 0x1.0p-53f;
  const float u = (float)((h >> 11) + 1ull) * 0x1.0p-53f;
  const float l = d < 0x1.0p-8f ? d * fmaf(d, fmaf(d, 0.33333333f, 0.5f), 1.0f)
                                : -0.69314718f * __builtin_amdgcn_logf(u);
  // a tiny g's reciprocal may overflow, a huge one's is subnormal (taken as 0)
  const float a = g > 0x1.0p-100f && g < 0x1.0p100f ? l * __builtin_amdgcn_rcpf(g)
                                                    : (float)((double)l / (double)g);
  return __float_as_uint(a) >> 20;
}

// Coordinates of voxel base + off (off < 4096) of the block whose first voxel
// is (i0, j0, k0): n / d for n < 2^25 from the truncated reciprocal
// floor(2^32 / d), low by at most one.
struct Magic {
  uint32_t d, m;
};
__device__ inline void div_mod(uint32_t n, Magic g, uint32_t& q, uint32_t& r) {
  q = g.d == 1 ? n : __umulhi(n, g.m);
  r = n - q * g.d;
  if (r >= g.d) { r -= g.d; ++q; }
}

// Central difference along one axis (one-sided at the faces, 0 on an axis of
// one voxel), as half_diff.
__device__ inline float axis_diff(const float* __restrict__ p, bool lo, bool hi, int64_t stride) {
  const float a = p[hi ? stride : 0], b = p[lo ? -stride : 0];
  return (lo && hi ? 0.5f : 1.0f) * (a - b);
}

// Persistent blocks of 1024 threads (the 32 KB histogram is flushed once per
// block), each taking blocks of 4,096 voxels.
constexpr int kSurveyThreads = 1024;
__global__ __launch_bounds__(kSurveyThreads) void k_survey(
    const float* __restrict__ f, Dims d, int64_t M, Magic mx, Magic my, uint64_t det_seed,
    uint64_t cov_seed, float* __restrict__ g32, unsigned long long* __restrict__ w) {
  __shared__ uint32_t h[kSurveyBins];
  __shared__ uint32_t cnt[2][kSurveyThreads / 64];
  for (int i = threadIdx.x; i < kSurveyBins; i += kSurveyThreads) h[i] = 0;
  __syncthreads();
  const int64_t plane = d.nx * d.ny;
  uint32_t occ = 0, el = 0;
  for (int64_t base = (int64_t)blockIdx.x * kBlockVox; base < M;
       base += (int64_t)gridDim.x * kBlockVox) {
    const uint32_t i0 = (uint32_t)(base % d.nx), j0 = (uint32_t)((base / d.nx) % d.ny);
    const int64_t k0 = base / plane;
#pragma unroll
    for (int r = 0; r < kBlockVox / kSurveyThreads; ++r) {
      const uint32_t off = (uint32_t)(r * kSurveyThreads) + threadIdx.x;
      const int64_t v = base + off;
      if (v >= M) continue;
      uint32_t q, i, jq, j;
      div_mod(i0 + off, mx, q, i);
      div_mod(j0 + q, my, jq, j);
      const int64_t k = k0 + jq;
      const float* p = f + v;
      const float fv = *p;
      float gx = axis_diff(p, i > 0, (int64_t)i < d.nx - 1, 1);
      float gy = axis_diff(p, j > 0, (int64_t)j < d.ny - 1, d.nx);
      float gz = axis_diff(p, k > 0, k < d.nz - 1, plane);
      if (d.nx == 1) gx = 0.0f;
      if (d.ny == 1) gy = 0.0f;
      if (d.nz == 1) gz = 0.0f;
      const double x = gx, y = gy, z = gz;
      const float g = (float)sqrt((x * x + y * y) + z * z);
      g32[v] = g;
      if (!(fv > kOcc)) continue;
      ++occ;
      atomicAdd(&h[kDetBins + (uint32_t)(cov_key(cov_seed, (uint64_t)v) >> 42)], 1u);
      atomicAdd(&h[kDetBins + kCovBins + (__float_as_uint(g) >> 20)], 1u);
      if (g > 0.0f) {
        ++el;
        atomicAdd(&h[det_bin(det_seed, (uint64_t)v, g)], 1u);
      }
    }
  }
  occ = wave_reduce_add(occ);
  el = wave_reduce_add(el);
  if ((threadIdx.x & 63) == 0) {
    cnt[0][threadIdx.x >> 6] = occ;
    cnt[1][threadIdx.x >> 6] = el;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    unsigned long long t = 0;
    for (int k = 0; k < kSurveyThreads / 64; ++k) t += cnt[threadIdx.x][k];
    if (t) atomicAdd(&w[threadIdx.x], t);
  }
  for (int i = threadIdx.x; i < kSurveyBins; i += kSurveyThreads)
    if (h[i]) atomicAdd(&w[kHist + i], (unsigned long long)h[i]);
}

// Block-wide: the bin of `bins` counts that holds the k-th (1-based; k = 0: bin
// 0), the counts before it, and through the bin `ahead` further on.  1024 threads.
__device__ inline void pick_bin(const unsigned long long* __restrict__ hist, int bins,
                                unsigned long long k, int ahead, unsigned long long* sh,
                                uint32_t& bin, unsigned long long& before,
                                unsigned long long& through) {
  __shared__ uint32_t found;
  __shared__ unsigned long long res[2];
  const int t = threadIdx.x;
  const int per = (bins + 1023) / 1024;
  unsigned long long mine = 0;
  for (int i = 0; i < per; ++i) {
    const int b = t * per + i;
    if (b < bins) mine += hist[b];
  }
  sh[t] = mine;
  if (t == 0) { found = (uint32_t)bins - 1; res[0] = res[1] = 0; }
  __syncthreads();
  for (int d = 1; d < 1024; d <<= 1) {
    const unsigned long long y = t >= d ? sh[t - d] : 0;
    __syncthreads();
    sh[t] += y;
    __syncthreads();
  }
  unsigned long long cum = sh[t] - mine;
  // the first bin with cum + count >= k
  if (cum < k || t == 0) {
    for (int i = 0; i < per; ++i) {
      const int b = t * per + i;
      if (b >= bins) break;
      const unsigned long long c = hist[b];
      if (cum + c >= k && (cum < k || b == 0)) {
        found = (uint32_t)b;
        res[0] = cum;
        break;
      }
      cum += c;
    }
  }
  __syncthreads();
  const int last = min((int)found + ahead, bins - 1);
  if (t == last / per) {
    unsigned long long c = sh[t] - mine;
    for (int b = t * per; b <= last; ++b) c += hist[b];
    res[1] = c;
  }
  __syncthreads();
  bin = found;
  before = res[0];
  through = res[1];
  __syncthreads();
}

// Candidate bins of the draws and the percentile's first digit.
__global__ __launch_bounds__(1024) void k_pick(unsigned long long* __restrict__ w,
                                               unsigned long long n_det,
                                               unsigned long long n_cov) {
  __shared__ unsigned long long sh[1024];
  uint32_t bin;
  unsigned long long before, through;
  pick_bin(w + kHist, kDetBins, n_det, 1, sh, bin, before, through);
  if (threadIdx.x == 0) {
    w[kDetBin] = min(bin + 1, (uint32_t)kDetBins - 1);
    w[kDetCount] = through;
    w[kListState] = 0;
    w[kListState + 1] = n_det;
  }
  pick_bin(w + kHist + kDetBins, kCovBins, n_cov, 0, sh, bin, before, through);
  if (threadIdx.x == 0) {
    w[kCovBin] = bin;
    w[kCovCount] = through;
    w[kListState + 2] = 0;
    w[kListState + 3] = n_cov;
  }
  // rank of the 99th percentile among the occupied voxels, 1-based
  const unsigned long long occ = w[kOccupied];
  const unsigned long long r = (unsigned long long)floor(0.99 * (double)(long long)(occ - 1)) + 1;
  pick_bin(w + kHist + kDetBins + kCovBins, kGBins, r, 0, sh, bin, before, through);
  if (threadIdx.x == 0) {
    w[kGBin] = (unsigned long long)bin << 20;
    w[kGRank] = r - before;
  }
}

// The percentile's next 10-bit digit, from histogram `which` at bit `shift`.
__global__ __launch_bounds__(1024) void k_pick_low(unsigned long long* __restrict__ w, int which,
                                                   int shift) {
  __shared__ unsigned long long sh[1024];
  uint32_t bin;
  unsigned long long before, through;
  const unsigned long long k = w[kGRank];
  pick_bin(w + kLowHist + which * kLowBins, kLowBins, k, 0, sh, bin, before, through);
  if (threadIdx.x == 0) {
    w[kGBin] |= (unsigned long long)bin << shift;
    w[kGRank] = k - before;
  }
}

// Masks of the candidate voxels (bit l of word v / 64: voxel 64 (v / 64) + l)
// and their number per block of 4,096 voxels; histogram of the percentile's
// second digit.  Persistent blocks; wave q of a block takes words 16 q .. 16 q
// + 15 of each 4,096 voxels.
__global__ __launch_bounds__(kThreads) void k_mark(
    const float* __restrict__ f, const float* __restrict__ g32, int64_t M, uint64_t det_seed,
    uint64_t cov_seed, unsigned long long* __restrict__ w, uint64_t* __restrict__ det_mask,
    uint64_t* __restrict__ cov_mask, uint32_t* __restrict__ det_cnt,
    uint32_t* __restrict__ cov_cnt) {
  __shared__ uint32_t h[kLowBins];
  __shared__ uint32_t cnt[2][kThreads / 64];
  for (int i = threadIdx.x; i < kLowBins; i += kThreads) h[i] = 0;
  const uint32_t det_last = (uint32_t)w[kDetBin], cov_last = (uint32_t)w[kCovBin];
  const uint32_t gbin = (uint32_t)w[kGBin] >> 20;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t nb = (M + kBlockVox - 1) / kBlockVox;
  __syncthreads();
  for (int64_t b = blockIdx.x; b < nb; b += gridDim.x) {
    const int64_t base = b * kBlockVox + wave * 1024;
    uint64_t dm = 0, cm = 0;  // lane r keeps word r
    uint32_t nd = 0, nc = 0;
#pragma unroll 4
    for (int r = 0; r < 16; ++r) {
      const int64_t v = base + 64 * r + lane;
      bool det = false, cov = false;
      if (v < M && f[v] > kOcc) {
        const float g = g32[v];
        cov = (uint32_t)(cov_key(cov_seed, (uint64_t)v) >> 42) <= cov_last;
        det = g > 0.0f && det_bin(det_seed, (uint64_t)v, g) <= det_last;
        const uint32_t gb = __float_as_uint(g);
        if (gb >> 20 == gbin) atomicAdd(&h[(gb >> 10) & (kLowBins - 1)], 1u);
      }
      const uint64_t bd = __builtin_amdgcn_ballot_w64(det), bc = __builtin_amdgcn_ballot_w64(cov);
      nd += (uint32_t)__popcll(bd);
      nc += (uint32_t)__popcll(bc);
      dm = lane == r ? bd : dm;
      cm = lane == r ? bc : cm;
    }
    if (lane < 16) {
      det_mask[b * kWords + wave * 16 + lane] = dm;
      cov_mask[b * kWords + wave * 16 + lane] = cm;
    }
    if (lane == 0) {
      cnt[0][wave] = nd;
      cnt[1][wave] = nc;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
      uint32_t t = 0;
      for (int k = 0; k < kThreads / 64; ++k) t += cnt[threadIdx.x][k];
      (threadIdx.x == 0 ? det_cnt : cov_cnt)[b] = t;
    }
    __syncthreads();
  }
  for (int i = threadIdx.x; i < kLowBins; i += kThreads)
    if (h[i]) atomicAdd(&w[kLowHist + i], (unsigned long long)h[i]);
}

// Histogram of the percentile's last digit.
__global__ __launch_bounds__(kThreads) void k_digit(const float* __restrict__ f,
                                                    const float* __restrict__ g32, int64_t M,
                                                    unsigned long long* __restrict__ w) {
  __shared__ uint32_t h[kLowBins];
  for (int i = threadIdx.x; i < kLowBins; i += kThreads) h[i] = 0;
  __syncthreads();
  const uint32_t prefix = (uint32_t)w[kGBin] >> 10;
  const int64_t step = (int64_t)gridDim.x * kThreads;
#pragma unroll 4
  for (int64_t v = (int64_t)blockIdx.x * kThreads + threadIdx.x; v < M; v += step) {
    const uint32_t gb = __float_as_uint(g32[v]);
    if (f[v] > kOcc && gb >> 10 == prefix) atomicAdd(&h[gb & (kLowBins - 1)], 1u);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kLowBins; i += kThreads)
    if (h[i]) atomicAdd(&w[kLowHist + kLowBins + i], (unsigned long long)h[i]);
}

// Exact keys and voxel indices of the marked voxels in voxel order; blockIdx.y
// 0: detail, 1: coverage.  Block b of 4,096 voxels writes from off[b].
struct ListArgs {
  const uint64_t* mask[2];
  const uint32_t* off[2];
  uint64_t* key[2];
  int64_t* vox[2];
  int64_t n[2];         // entries
  uint32_t* less[2];    // per 4,096 entries: keys below the Nth, keys equal to it
  uint32_t* tie[2];
  uint32_t* tie_off[2];
  uint32_t* take[2];
  uint32_t* out_off[2];
  int64_t* out[2];
};

__global__ __launch_bounds__(kThreads) void k_gather(ListArgs a, const float* __restrict__ g32,
                                                     uint64_t det_seed, uint64_t cov_seed) {
  const int y = blockIdx.y;
  const int64_t b = blockIdx.x;
  const uint32_t o = a.off[y][b];
  if (a.off[y][b + 1] == o) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // lane l holds word l of the block and the candidates before it
  const uint64_t word = a.mask[y][b * kWords + lane];
  uint32_t inc = (uint32_t)__popcll(word);
  const uint32_t own = inc;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t u = __shfl_up(inc, d, 64);
    if (lane >= d) inc += u;
  }
  const uint32_t before = inc - own;
  for (int r = 16 * wave; r < 16 * wave + 16; ++r) {
    const uint64_t m = __shfl(word, r, 64);
    const uint32_t p0 = __shfl(before, r, 64);
    if ((m >> lane) & 1ull) {
      const uint32_t pos = o + p0 + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
      const int64_t v = b * kBlockVox + 64 * r + lane;
      a.key[y][pos] = y == 0 ? det_key(det_seed, (uint64_t)v, g32[v]) : cov_key(cov_seed, (uint64_t)v);
      a.vox[y][pos] = v;
    }
  }
}

// ---- exact selection of the rank smallest keys of both lists ------------------
//
// Select state per list: [0] prefix, [1] remaining rank (1-based count of the
// smallest keys still to take at or below the prefix).
__global__ __launch_bounds__(kThreads) void k_list_hist(ListArgs a, int shift,
                                                        unsigned long long* __restrict__ w) {
  __shared__ unsigned int h[256];
  const int y = blockIdx.y;
  h[threadIdx.x] = 0;
  __syncthreads();
  const uint64_t prefix = w[kListState + 2 * y];
  const uint64_t hi_mask = (shift + 8 >= 64) ? 0ull : (~0ull << (shift + 8));
  const uint64_t* __restrict__ key = a.key[y];
  const int64_t n = a.n[y], step = (int64_t)gridDim.x * kThreads;
#pragma unroll 4
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += step) {
    const uint64_t k = key[i];
    if ((k & hi_mask) == (prefix & hi_mask)) atomicAdd(&h[(k >> shift) & 255u], 1u);
  }
  __syncthreads();
  if (h[threadIdx.x])
    atomicAdd(&w[kListHist + 256 * y + threadIdx.x], (unsigned long long)h[threadIdx.x]);
}

// The next digit of both lists (one block of 256 threads each).
__global__ __launch_bounds__(256) void k_list_step(int shift, unsigned long long* __restrict__ w) {
  __shared__ unsigned long long sh[256];
  __shared__ unsigned long long res[2];
  const int t = threadIdx.x;
  unsigned long long* st = w + kListState + 2 * blockIdx.x;
  unsigned long long* hist = w + kListHist + 256 * blockIdx.x;
  const unsigned long long k = st[1], c = hist[t];
  sh[t] = c;
  if (t == 0) { res[0] = 255; res[1] = 0; }
  __syncthreads();
  for (int d = 1; d < 256; d <<= 1) {
    const unsigned long long y = t >= d ? sh[t - d] : 0;
    __syncthreads();
    sh[t] += y;
    __syncthreads();
  }
  const unsigned long long before = sh[t] - c;
  if (before + c >= k && (before < k || t == 0)) {
    res[0] = (unsigned long long)t;
    res[1] = before;
  }
  hist[t] = 0;
  __syncthreads();
  if (t == 0) {
    st[0] |= res[0] << shift;
    st[1] = k - res[1];
  }
}

// Per block of 4,096 entries: keys below and equal to the rank-th key.
__global__ __launch_bounds__(kThreads) void k_list_count(ListArgs a,
                                                         const unsigned long long* __restrict__ w) {
  __shared__ uint32_t sl[kThreads / 64], stt[kThreads / 64];
  const int y = blockIdx.y;
  const int64_t base = (int64_t)blockIdx.x * kBlockVox;
  if (base >= a.n[y]) return;
  const uint64_t K = w[kListState + 2 * y];
  uint32_t nl = 0, nt = 0;
#pragma unroll
  for (int j = 0; j < kBlockVox / kThreads; ++j) {
    const int64_t i = base + j * kThreads + threadIdx.x;
    if (i < a.n[y]) {
      const uint64_t k = a.key[y][i];
      nl += k < K;
      nt += k == K;
    }
  }
  nl = wave_reduce_add(nl);
  nt = wave_reduce_add(nt);
  if ((threadIdx.x & 63) == 0) {
    sl[threadIdx.x >> 6] = nl;
    stt[threadIdx.x >> 6] = nt;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t p = 0, q = 0;
    for (int k = 0; k < kThreads / 64; ++k) { p += sl[k]; q += stt[k]; }
    a.less[y][blockIdx.x] = p;
    a.tie[y][blockIdx.x] = q;
  }
}

__global__ void k_list_take(ListArgs a, const unsigned long long* __restrict__ w) {
  const int y = blockIdx.y;
  const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (b * kBlockVox >= a.n[y]) return;
  const int64_t krem = (int64_t)w[kListState + 2 * y + 1];
  int64_t t = krem - (int64_t)a.tie_off[y][b];
  if (t < 0) t = 0;
  if (t > a.tie[y][b]) t = a.tie[y][b];
  a.take[y][b] = a.less[y][b] + (uint32_t)t;
}

// Writes the selected voxel indices in increasing voxel order (thread t of a
// block takes 16 consecutive entries).
__global__ __launch_bounds__(kThreads) void k_list_write(ListArgs a,
                                                         const unsigned long long* __restrict__ w) {
  __shared__ uint32_t wsum[kThreads / 64];
  const int y = blockIdx.y;
  constexpr int kPer = kBlockVox / kThreads;
  const int64_t n = a.n[y];
  if ((int64_t)blockIdx.x * kBlockVox >= n) return;
  const uint64_t K = w[kListState + 2 * y];
  const int64_t krem = (int64_t)w[kListState + 2 * y + 1];
  const int64_t base = (int64_t)blockIdx.x * kBlockVox + (int64_t)threadIdx.x * kPer;
  uint32_t lessm = 0, tiem = 0;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    if (base + j < n) {
      const uint64_t k = a.key[y][base + j];
      if (k < K) lessm |= 1u << j;
      else if (k == K) tiem |= 1u << j;
    }
  }
  uint32_t tie_rank =
      block_excl_scan((uint32_t)__popc(tiem), wsum) + a.tie_off[y][blockIdx.x];
  uint32_t takem = lessm;
  for (int j = 0; j < kPer; ++j)
    if ((tiem >> j) & 1u) {
      if ((int64_t)tie_rank < krem) takem |= 1u << j;
      ++tie_rank;
    }
  uint32_t pos = block_excl_scan((uint32_t)__popc(takem), wsum) + a.out_off[y][blockIdx.x];
  for (int j = 0; j < kPer; ++j)
    if ((takem >> j) & 1u) a.out[y][pos++] = a.vox[y][base + j];
}

// S1c: nearest-neighbour squared distances of eight subsamples of a group per
// block (blockIdx.y: group), so that a pass over the group's centres, which come
// from L2, serves eight.  The distance is exact to a rounding in double, but
// formed only for the centres that a float estimate does not rule out: float
// differences of float centres and their squares are off by less than 4e-7
// relative, well inside the allowance of 1e-5.  262,144 seeds: one subsample a
// block in double 800 us, with the float estimate 673, eight a block 264.
struct NnArgs {
  const float *mx, *my, *mz;  // [n] centres
  int64_t first[2], ng[2], stride[2], m[2];
  double* best[2];
};

constexpr int kNnPer = 8;
__global__ __launch_bounds__(kThreads) void k_nn(NnArgs a) {
#pragma clang fp contract(off)
  __shared__ double sh[kNnPer][kThreads / 64];
  const int y = blockIdx.y;
  const int64_t q0 = (int64_t)blockIdx.x * kNnPer;
  if (q0 >= a.m[y]) return;
  const float* __restrict__ mx = a.mx + a.first[y];
  const float* __restrict__ my = a.my + a.first[y];
  const float* __restrict__ mz = a.mz + a.first[y];
  const int64_t ng = a.ng[y];
  float xf[kNnPer], yf[kNnPer], zf[kNnPer], lim[kNnPer];
  double b[kNnPer];
#pragma unroll
  for (int q = 0; q < kNnPer; ++q) {
    const int64_t i = min(q0 + q, a.m[y] - 1) * a.stride[y];
    xf[q] = mx[i];
    yf[q] = my[i];
    zf[q] = mz[i];
    // the group is in voxel order: seeds near in the list give a bound that few
    // others stay below
    const int64_t j = i - 32 + (int)(threadIdx.x & 63);
    b[q] = INFINITY;
    if (j >= 0 && j < ng && j != i) {
      const double dx = (double)mx[j] - (double)xf[q], dy = (double)my[j] - (double)yf[q],
                   dz = (double)mz[j] - (double)zf[q];
      const double xx = dx * dx, yy = dy * dy, zz = dz * dz;
      b[q] = (xx + yy) + zz;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) b[q] = fmin(b[q], __shfl_xor(b[q], d, 64));
    lim[q] = (float)b[q] * 1.00001f + 1e-30f;
  }
  // the next centre is loaded while one is tested (past the end: the last
  // again, a distance already counted)
  const uint32_t last = (uint32_t)ng - 1u;
  uint32_t j = min((uint32_t)threadIdx.x, last);
  float px = mx[j], py = my[j], pz = mz[j];
  for (uint32_t j0 = 0; j0 <= last; j0 += kThreads) {
    const uint32_t jn = min(j0 + kThreads + threadIdx.x, last);
    const float nx = mx[jn], ny = my[jn], nz = mz[jn];
#pragma unroll
    for (int q = 0; q < kNnPer; ++q) {
      const float ex = px - xf[q], ey = py - yf[q], ez = pz - zf[q];
      const float e2 = ex * ex + ey * ey + ez * ez;
      if (!(e2 > lim[q])) {
        if ((int64_t)j == min(q0 + q, a.m[y] - 1) * a.stride[y]) continue;  // the subsample itself
        const double dx = (double)px - (double)xf[q], dy = (double)py - (double)yf[q],
                     dz = (double)pz - (double)zf[q];
        const double xx = dx * dx, yy = dy * dy, zz = dz * dz;
        const double d2 = (xx + yy) + zz;
        b[q] = fmin(b[q], d2);
        lim[q] = (float)b[q] * 1.00001f + 1e-30f;
      }
    }
    j = jn;
    px = nx;
    py = ny;
    pz = nz;
  }
#pragma unroll
  for (int q = 0; q < kNnPer; ++q) {
    double v = b[q];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v = fmin(v, __shfl_xor(v, d, 64));
    if ((threadIdx.x & 63) == 0) sh[q][threadIdx.x >> 6] = v;
  }
  __syncthreads();
  if (threadIdx.x < kNnPer && q0 + threadIdx.x < a.m[y]) {
    double v = sh[threadIdx.x][0];
    for (int w = 1; w < kThreads / 64; ++w) v = fmin(v, sh[threadIdx.x][w]);
    a.best[y][q0 + threadIdx.x] = v;
  }
}

// Lower median of m <= 4096 values -> sqrt, by bitonic sort in LDS (one block
// per group); 1 for a group of fewer than two seeds.
__global__ __launch_bounds__(1024) void k_median(NnArgs a, double* __restrict__ out) {
  __shared__ double v[4096];
  const double* __restrict__ best = a.best[blockIdx.x];
  const int m = (int)a.m[blockIdx.x];
  for (int i = threadIdx.x; i < 4096; i += 1024) v[i] = (i < m) ? best[i] : INFINITY;
  __syncthreads();
  for (int size = 2; size <= 4096; size <<= 1)
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int i = threadIdx.x; i < 4096; i += 1024) {
        const int j = i ^ stride;
        if (j > i) {
          const bool up = (i & size) == 0;
          const double p = v[i], q = v[j];
          if ((p > q) == up) { v[i] = q; v[j] = p; }
        }
      }
      __syncthreads();
    }
  if (threadIdx.x == 0) out[blockIdx.x] = (m >= 1) ? sqrt(v[(m - 1) / 2]) : 1.0;
}

__device__ inline void quat_from_R(const double R[3][3], double q[4]) {
  const double t = R[0][0] + R[1][1] + R[2][2];
  if (t > 0.0) {
    const double s = sqrt(t + 1.0) * 2.0;
    q[0] = 0.25 * s; q[1] = (R[2][1] - R[1][2]) / s; q[2] = (R[0][2] - R[2][0]) / s;
    q[3] = (R[1][0] - R[0][1]) / s;
  } else if (R[0][0] > R[1][1] && R[0][0] > R[2][2]) {
    const double s = sqrt(1.0 + R[0][0] - R[1][1] - R[2][2]) * 2.0;
    q[0] = (R[2][1] - R[1][2]) / s; q[1] = 0.25 * s; q[2] = (R[0][1] + R[1][0]) / s;
    q[3] = (R[0][2] + R[2][0]) / s;
  } else if (R[1][1] > R[2][2]) {
    const double s = sqrt(1.0 + R[1][1] - R[0][0] - R[2][2]) * 2.0;
    q[0] = (R[0][2] - R[2][0]) / s; q[1] = (R[0][1] + R[1][0]) / s; q[2] = 0.25 * s;
    q[3] = (R[1][2] + R[2][1]) / s;
  } else {
    const double s = sqrt(1.0 + R[2][2] - R[0][0] - R[1][1]) * 2.0;
    q[0] = (R[1][0] - R[0][1]) / s; q[1] = (R[0][2] + R[2][0]) / s; q[2] = (R[1][2] + R[2][1]) / s;
    q[3] = 0.25 * s;
  }
  const double n = sqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
  const double sg = (q[0] < 0.0) ? -1.0 : 1.0;
  for (int a = 0; a < 4; ++a) q[a] = sg * q[a] / n;
}

struct AssembleArgs {
  const float* f;
  const float* g32;
  Dims d;
  int64_t x0, y0, z0;
  const int64_t* det;
  const int64_t* cov;
  int64_t n_det, n;
  const double* s_base;   // [2]
  const unsigned long long* g99_bits;  // select state of the percentile (prefix = bits)
  double s_cap;
  uint64_t seed;
  float* theta;           // [11][n]
  const double* J6;       // [n][6] structure tensors at the seeds (k_tensor)
};

// One wave per primitive: the structure tensor at its seed voxel (S1d).
__global__ __launch_bounds__(256) void k_tensor(const float* __restrict__ f, Dims d,
                                                const int64_t* __restrict__ det,
                                                const int64_t* __restrict__ cov, int64_t n_det,
                                                int64_t n, double* __restrict__ J6) {
  const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= n) return;  // wave-uniform
  const int64_t vox = i < n_det ? det[i] : cov[i - n_det];
  const int64_t ii = vox % d.nx, jj = (vox / d.nx) % d.ny, kk = vox / (d.nx * d.ny);
  __shared__ float box[4][kTensorBox];
  wave_structure_tensor(f, d, ii, jj, kk, box[threadIdx.x >> 6], J6 + 6 * i);
}

__global__ __launch_bounds__(128) void k_assemble(AssembleArgs a) {
  const int64_t i = (int64_t)blockIdx.x * 128 + threadIdx.x;
  if (i >= a.n) return;
  const int group = i < a.n_det ? 0 : 1;
  const int64_t vox = group == 0 ? a.det[i] : a.cov[i - a.n_det];
  const int64_t n = a.n;
  // structure tensor over the clipped 7^3 box (S1d), from k_tensor
  const double* t = a.J6 + 6 * i;
  double J[3][3] = {{t[0], t[1], t[2]}, {t[1], t[3], t[4]}, {t[2], t[4], t[5]}};
  double R[3][3] = {{1, 0, 0}, {0, 1, 0}, {0, 0, 1}};
  if (J[0][0] + J[1][1] + J[2][2] >= 1e-12) {
    double A[3][3], V[3][3];
    for (int r = 0; r < 3; ++r)
      for (int c = 0; c < 3; ++c) A[r][c] = J[r][c];
    jacobi3(A, V);
    double w[3] = {A[0][0], A[1][1], A[2][2]};
    int idx[3] = {0, 1, 2};  // ascending eigenvalues
    for (int p = 0; p < 3; ++p)
      for (int q = p + 1; q < 3; ++q)
        if (w[idx[q]] < w[idx[p]]) { int t = idx[p]; idx[p] = idx[q]; idx[q] = t; }
    // columns: e3 (smallest), e2, e1 (largest); largest-|.| component positive
    for (int col = 0; col < 3; ++col) {
      const int e = idx[col];
      int am = 0;
      double best = fabs(V[0][e]);
      for (int r = 1; r < 3; ++r)
        if (fabs(V[r][e]) > best) { best = fabs(V[r][e]); am = r; }
      const double sg = (V[am][e] < 0.0) ? -1.0 : 1.0;
      for (int r = 0; r < 3; ++r) R[r][col] = sg * V[r][e];
    }
    const double det = R[0][0] * (R[1][1] * R[2][2] - R[1][2] * R[2][1]) -
                       R[0][1] * (R[1][0] * R[2][2] - R[1][2] * R[2][0]) +
                       R[0][2] * (R[1][0] * R[2][1] - R[1][1] * R[2][0]);
    if (det < 0.0)
      for (int r = 0; r < 3; ++r) R[r][2] = -R[r][2];
  }
  // scales (S1e)
  const double sb = a.s_base[group];
  const float g99 = __uint_as_float((unsigned)a.g99_bits[0]);
  double gh = 0.0;
  if (g99 > 0.0f) gh = fmin(fmax((double)a.g32[vox] / (double)g99, 0.0), 1.0);
  const double st = fmin(sb * (1.0 + 2.0 * gh), 3.0 * sb);
  const double cap = fmax(a.s_cap, 0.25);
  const double s3[3] = {fmin(fmax(st, 0.25), cap), fmin(fmax(sb, 0.25), cap),
                        fmin(fmax(sb, 0.25), cap)};
  double q[4];
  quat_from_R(R, q);
  for (int c = 0; c < 4; ++c) a.theta[(3 + c) * n + i] = (float)q[c];
  for (int c = 0; c < 3; ++c) a.theta[(7 + c) * n + i] = (float)log(s3[c]);
  a.theta[10 * n + i] = a.f[vox];
}

// S1b jitter: centre = (voxel + u) - 1/2 per axis in double, rounded to float.
__global__ __launch_bounds__(256) void k_jitter(Dims d, int64_t x0, int64_t y0, int64_t z0,
                                                const int64_t* __restrict__ det,
                                                const int64_t* __restrict__ cov, int64_t n_det,
                                                int64_t n, uint64_t seed, float* __restrict__ theta) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int group = i < n_det ? 0 : 1;
  const int64_t vox = group == 0 ? det[i] : cov[i - n_det];
  const int64_t base[3] = {vox % d.nx + x0, (vox / d.nx) % d.ny + y0, vox / (d.nx * d.ny) + z0};
  for (int ax = 0; ax < 3; ++ax) {
    const double u = uniform01(seed, 3 + 3 * group + ax, (uint64_t)vox);
    theta[ax * n + i] = (float)(((double)base[ax] + u) - 0.5);
  }
}

// Dot products <U, V> and <U, U> in double (two-level, deterministic).
constexpr int kDotBlocks = 256;
__global__ __launch_bounds__(kThreads) void k_dot_partial(const double2* __restrict__ in,
                                                          int64_t n, double* __restrict__ part) {
  __shared__ double s1[kThreads], s2[kThreads];
  const int64_t per = (n + gridDim.x - 1) / gridDim.x;
  const int64_t a = (int64_t)blockIdx.x * per, e = min(n, a + per);
  double uv = 0.0, uu = 0.0;
  for (int64_t i = a + threadIdx.x; i < e; i += kThreads) {
    uv += in[i].x;
    uu += in[i].y;
  }
  s1[threadIdx.x] = uv;
  s2[threadIdx.x] = uu;
  __syncthreads();
  for (int w = kThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      s1[threadIdx.x] += s1[threadIdx.x + w];
      s2[threadIdx.x] += s2[threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = s1[0];
    part[2 * blockIdx.x + 1] = s2[0];
  }
}

__global__ __launch_bounds__(kThreads) void k_kappa(const double* __restrict__ part, int np,
                                                    double* __restrict__ kappa) {
  __shared__ double s1[kThreads], s2[kThreads];
  double uv = 0.0, uu = 0.0;
  for (int i = threadIdx.x; i < np; i += kThreads) {
    uv += part[2 * i];
    uu += part[2 * i + 1];
  }
  s1[threadIdx.x] = uv;
  s2[threadIdx.x] = uu;
  __syncthreads();
  for (int w = kThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      s1[threadIdx.x] += s1[threadIdx.x + w];
      s2[threadIdx.x] += s2[threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) kappa[0] = (s2[0] > 0.0) ? s1[0] / s2[0] : 0.0;
}

__global__ void k_scale_row(float* __restrict__ row, int64_t n, const double* __restrict__ kappa) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) row[i] = (float)((double)row[i] * kappa[0]);
}

// Min-max normalisation (Sec. III-B preprocessing).
__global__ __launch_bounds__(kThreads) void k_minmax(const float* __restrict__ f, int64_t M,
                                                     float* __restrict__ part) {
  __shared__ float lo[kThreads], hi[kThreads];
  float a = INFINITY, b = -INFINITY;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < M;
       i += (int64_t)gridDim.x * kThreads) {
    a = fminf(a, f[i]);
    b = fmaxf(b, f[i]);
  }
  lo[threadIdx.x] = a;
  hi[threadIdx.x] = b;
  __syncthreads();
  for (int w = kThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      lo[threadIdx.x] = fminf(lo[threadIdx.x], lo[threadIdx.x + w]);
      hi[threadIdx.x] = fmaxf(hi[threadIdx.x], hi[threadIdx.x + w]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = lo[0];
    part[2 * blockIdx.x + 1] = hi[0];
  }
}

__global__ __launch_bounds__(kThreads) void k_normalize(float* __restrict__ f, int64_t M,
                                                        const float* __restrict__ part, int np) {
  float a = INFINITY, b = -INFINITY;
  for (int i = 0; i < np; ++i) {
    a = fminf(a, part[2 * i]);
    b = fmaxf(b, part[2 * i + 1]);
  }
  const float span = b - a;
  const float inv = span > 0.0f ? 1.0f / span : 0.0f;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < M;
       i += (int64_t)gridDim.x * kThreads)
    f[i] = (f[i] - a) * inv;
}

unsigned grid_for(int64_t M) {
  int64_t b = (M + kThreads - 1) / kThreads;
  if (b > 8192) b = 8192;
  if (b < 1) b = 1;
  return (unsigned)b;
}

}  // namespace

// ---------------------------------------------------------------------------
// Host-side sequencing (called from the ABI layer with preallocated buffers).

size_t alloc_block_count(int64_t n) { return (size_t)((n + kBlockVox - 1) / kBlockVox); }
size_t alloc_mask_words(int64_t M) { return alloc_block_count(M) * kWords; }
size_t alloc_select_words() { return kSelectWords; }

namespace {

Magic magic(int64_t d) {
  return Magic{(uint32_t)d, d > 1 ? (uint32_t)(0x100000000ull / (uint64_t)d) : 0u};
}

uint64_t stream_seed(uint64_t seed, uint64_t stream) {
  return splitmix64(seed ^ (stream * 0xD1B54A32D192ED03ull));
}

}  // namespace

// Gradient magnitudes, domain counts, histograms and candidate bins (w:
// alloc_select_words() u64, zeroed here).
hipError_t alloc_survey(const float* f, const gve_grid& g, uint64_t seed, int64_t n_det,
                        int64_t n_cov, float* g32, unsigned long long* w, hipStream_t s) {
  const int64_t M = g.nx * g.ny * g.nz;
  hipError_t e = fill_u64(w, kSelectWords, s);
  if (e != hipSuccess) return e;
  // two blocks of 1024 threads fill a CU
  const unsigned blocks = (unsigned)std::min<int64_t>((int64_t)alloc_block_count(M), 512);
  hipLaunchKernelGGL(k_survey, dim3(blocks), dim3(kSurveyThreads), 0, s, f, Dims{g.nx, g.ny, g.nz},
                     M, magic(g.nx), magic(g.ny), stream_seed(seed, 1), stream_seed(seed, 2), g32,
                     w);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_pick, dim3(1), dim3(1024), 0, s, w, (unsigned long long)n_det,
                     (unsigned long long)n_cov);
  return hipGetLastError();
}

// The draws from the surveyed volume: voxel indices of the n_det detail and
// n_cov coverage seeds, and the bits of the 99th percentile of g in w[6].
hipError_t alloc_draw(const float* f, const float* g32, const gve_grid& g, uint64_t seed,
                      unsigned long long* w, const AllocLists& l, int64_t* det, int64_t* cov,
                      void* scan_tmp, hipStream_t s) {
  const int64_t M = g.nx * g.ny * g.nz;
  const int64_t nb = (int64_t)alloc_block_count(M);
  const uint64_t ds = stream_seed(seed, 1), cs = stream_seed(seed, 2);
  ListArgs a{};
  for (int y = 0; y < 2; ++y) {
    a.mask[y] = l.mask[y];
    a.off[y] = l.off[y];
    a.key[y] = l.key[y];
    a.vox[y] = l.vox[y];
    a.n[y] = l.n[y];
    a.less[y] = l.blk[y];
    const int64_t lb = (int64_t)alloc_block_count(l.n[y]) + 1;
    a.tie[y] = a.less[y] + lb;
    a.tie_off[y] = a.tie[y] + lb;
    a.take[y] = a.tie_off[y] + lb;
    a.out_off[y] = a.take[y] + lb;
    a.out[y] = y == 0 ? det : cov;
  }
  hipError_t e = hipSuccess;
  auto ok = [&]() { return (e = hipGetLastError()) == hipSuccess; };
  const unsigned blocks = (unsigned)std::min<int64_t>(nb, 2048);
  hipLaunchKernelGGL(k_mark, dim3(blocks), dim3(kThreads), 0, s, f, g32, M, ds, cs, w, l.mask[0],
                     l.mask[1], l.cnt[0], l.cnt[1]);
  if (!ok()) return e;
  for (int y = 0; y < 2; ++y) {
    e = scan_exclusive_u32(l.cnt[y], l.off[y], nb, scan_tmp, s);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_gather, dim3((unsigned)nb, 2), dim3(kThreads), 0, s, a, g32, ds, cs);
  if (!ok()) return e;
  hipLaunchKernelGGL(k_pick_low, dim3(1), dim3(1024), 0, s, w, 0, 10);
  if (!ok()) return e;
  hipLaunchKernelGGL(k_digit, dim3(grid_for(M)), dim3(kThreads), 0, s, f, g32, M, w);
  if (!ok()) return e;
  hipLaunchKernelGGL(k_pick_low, dim3(1), dim3(1024), 0, s, w, 1, 0);
  if (!ok()) return e;
  // the lists
  const int64_t nmax = std::max<int64_t>(std::max(l.n[0], l.n[1]), 1);
  const unsigned hb = (unsigned)std::min<int64_t>((nmax + 4 * kThreads - 1) / (4 * kThreads), 512);
  for (int shift = 56; shift >= 0; shift -= 8) {
    hipLaunchKernelGGL(k_list_hist, dim3(hb, 2), dim3(kThreads), 0, s, a, shift, w);
    if (!ok()) return e;
    hipLaunchKernelGGL(k_list_step, dim3(2), dim3(256), 0, s, shift, w);
    if (!ok()) return e;
  }
  const unsigned lb = (unsigned)alloc_block_count(nmax);
  hipLaunchKernelGGL(k_list_count, dim3(lb, 2), dim3(kThreads), 0, s, a, w);
  if (!ok()) return e;
  for (int y = 0; y < 2; ++y) {
    e = scan_exclusive_u32(a.tie[y], a.tie_off[y], (int64_t)alloc_block_count(l.n[y]), scan_tmp, s);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_list_take, dim3((lb + 255) / 256, 2), dim3(256), 0, s, a, w);
  if (!ok()) return e;
  for (int y = 0; y < 2; ++y) {
    e = scan_exclusive_u32(a.take[y], a.out_off[y], (int64_t)alloc_block_count(l.n[y]), scan_tmp, s);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_list_write, dim3(lb, 2), dim3(kThreads), 0, s, a, w);
  return hipGetLastError();
}

// Both groups' spacing: seeds [0, n_det) and [n_det, n); best: 2 x 4096.
hipError_t alloc_spacing(const float* theta, int64_t n, int64_t n_det, double* best,
                         double* s_base, hipStream_t s) {
  NnArgs a{};
  a.mx = theta;
  a.my = theta + n;
  a.mz = theta + 2 * n;
  for (int y = 0; y < 2; ++y) {
    a.first[y] = y == 0 ? 0 : n_det;
    a.ng[y] = y == 0 ? n_det : n - n_det;
    a.stride[y] = std::max<int64_t>((a.ng[y] + 4095) / 4096, 1);
    // a single seed has no neighbour: unit spacing
    a.m[y] = a.ng[y] < 2 ? 0 : (a.ng[y] + a.stride[y] - 1) / a.stride[y];
    a.best[y] = best + 4096 * y;
  }
  const unsigned blocks = (unsigned)((std::max(a.m[0], a.m[1]) + kNnPer - 1) / kNnPer);
  if (blocks > 0) {
    hipLaunchKernelGGL(k_nn, dim3(blocks, 2), dim3(kThreads), 0, s, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_median, dim3(2), dim3(1024), 0, s, a, s_base);
  return hipGetLastError();
}

hipError_t alloc_jitter(const gve_grid& g, const int64_t* det, const int64_t* cov, int64_t n_det,
                        int64_t n, uint64_t seed, float* theta, hipStream_t s) {
  hipLaunchKernelGGL(k_jitter, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                     Dims{g.nx, g.ny, g.nz}, g.x0, g.y0, g.z0, det, cov, n_det, n, seed, theta);
  return hipGetLastError();
}

hipError_t alloc_assemble(const float* f, const float* g32, const gve_grid& g, const int64_t* det,
                          const int64_t* cov, int64_t n_det, int64_t n, const double* s_base,
                          const unsigned long long* g99_state, uint64_t seed, float* theta,
                          double* J6, hipStream_t s) {
  AssembleArgs a;
  a.f = f;
  a.g32 = g32;
  a.d = Dims{g.nx, g.ny, g.nz};
  a.x0 = g.x0; a.y0 = g.y0; a.z0 = g.z0;
  a.det = det;
  a.cov = cov;
  a.n_det = n_det;
  a.n = n;
  a.s_base = s_base;
  a.g99_bits = g99_state;
  int64_t mx = g.nx > g.ny ? g.nx : g.ny;
  if (g.nz > mx) mx = g.nz;
  a.s_cap = (double)mx / 16.0;
  a.seed = seed;
  a.theta = theta;
  a.J6 = J6;
  hipLaunchKernelGGL(k_tensor, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s, f, a.d, det, cov,
                     n_det, n, J6);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_assemble, dim3((unsigned)((n + 127) / 128)), dim3(128), 0, s, a);
  return hipGetLastError();
}

size_t alloc_dot_tmp_doubles() { return 2 * kDotBlocks + 8; }

hipError_t alloc_weights(const double* part, int64_t pairs, float* c_row, int64_t n, double* tmp,
                         hipStream_t s) {
  hipLaunchKernelGGL(k_dot_partial, dim3(kDotBlocks), dim3(kThreads), 0, s,
                     reinterpret_cast<const double2*>(part), pairs, tmp + 8);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_kappa, dim3(1), dim3(kThreads), 0, s, tmp + 8, kDotBlocks, tmp);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_scale_row, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, c_row, n, tmp);
  return hipGetLastError();
}

size_t normalize_tmp_floats() { return 2 * 1024; }

hipError_t normalize_field(float* f, int64_t M, float* tmp, hipStream_t s) {
  hipLaunchKernelGGL(k_minmax, dim3(1024), dim3(kThreads), 0, s, f, M, tmp);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_normalize, dim3(grid_for(M)), dim3(kThreads), 0, s, f, M, tmp, 1024);
  return hipGetLastError();
}

}  // namespace gve
