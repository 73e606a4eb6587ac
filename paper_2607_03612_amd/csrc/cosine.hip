// DINO Top-K kernel, block-wise form (Sec. 4.1 and Sec. 4.3): per query block,
// the key blocks of every frame whose features are most similar to its own.
//
// The features are the caller's per-token vectors (the paper uses the last
// DINO block's patch features). Every token's feature is scaled to unit
// length and averaged over its block; the dot product of two block means is
// then the mean cosine similarity over the tile of token pairs, the same
// linearity argument as the query probe. All of it runs in float64:
//   1. cosine_pool: one workgroup per block writes the block's mean unit
//      feature, a row of [nb][D];
//   2. cosine_sim_mfma_kernel: the block similarity matrix [nb][nb], the
//      product of that matrix with its transpose on the fp64 matrix cores
//      (upper tiles only, mirrored);
//   3. cosine_topk_kernel: one workgroup per (per-frame count k, query
//      block), one lane per frame (a key block counts under the frame of its
//      first token): the frame's k best (similarity desc, index asc) pairs go
//      out ascending at an offset from a prefix sum over the frames, into
//      every head that keeps k per frame.
// The lists depend on the features only, so they are computed once per
// sequence and reused by every layer.
#include <algorithm>
#include <type_traits>

#include "saf3r_internal.h"

namespace saf3r {
namespace {

constexpr int kPoolThreads = 256;

template <typename T>
__device__ inline double feat_at(const T* f, int64_t i);
template <>
__device__ inline double feat_at<uint16_t>(const uint16_t* f, int64_t i) {
  return (double)__uint_as_float((uint32_t)f[i] << 16);
}
template <>
__device__ inline double feat_at<float>(const float* f, int64_t i) {
  return (double)f[i];
}

// Where the mean unit feature of block b at dimension d lies in fb: groups of
// 16 blocks (the last one fewer), in each runs of 8 dimensions (the last one
// fewer), in each the blocks in turn. So a 16-block operand of 8 dimensions is
// 1 KB in one piece, where rows of a power of two of bytes would all start on
// one memory channel; nothing is padded.
__device__ inline int64_t fb_at(int b, int d, int nb, int dim) {
  const int b0 = b & ~15, d0 = d & ~7;
  const int blocks = min(16, nb - b0), width = min(8, dim - d0);
  return (int64_t)b0 * dim + (int64_t)d0 * blocks + (b - b0) * width + (d - d0);
}

// Mean unit feature of block b: fb[b][d] = (1/n_b) sum_t f[t][d] / |f[t]|. The
// general form: any width, the block's features read twice.
// kVec: rows are whole 16-byte vectors (feat_dim * element size a multiple
// of 16, 16-byte aligned base), read 16 bytes per lane; otherwise one element
// per lane.
template <typename T, bool kVec>
__global__ __launch_bounds__(kPoolThreads) void cosine_pool_kernel(const T* __restrict__ f,
                                                                  double* __restrict__ fb,
                                                                  CosineArgs a) {
  constexpr int kPer = 16 / (int)sizeof(T);  // elements per 16-byte vector
  __shared__ double inv_norm[kBlock];
  const int b = blockIdx.x;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int64_t row0 = (int64_t)b * kBlock;
  const int rows = (int)min<int64_t>(kBlock, a.n - row0);
  const int vecs = a.dim / kPer;  // 16-byte vectors per row (kVec)
  // 1/|f_t| for the block's tokens: one wave per token
  for (int r = wave; r < rows; r += kPoolThreads / 64) {
    double ss = 0.0;
    if constexpr (kVec) {
      const uint4* row = reinterpret_cast<const uint4*>(f + (row0 + r) * a.dim);
      for (int c = lane; c < vecs; c += 64) {
        const uint4 u = row[c];
        const T* e = reinterpret_cast<const T*>(&u);
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
          const double x = feat_at(e, q);
          ss = fma(x, x, ss);
        }
      }
    } else {
      for (int d = lane; d < a.dim; d += 64) {
        const double x = feat_at(f, (row0 + r) * a.dim + d);
        ss = fma(x, x, ss);
      }
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) ss += __shfl_xor(ss, m);
    if (lane == 0) inv_norm[r] = 1.0 / sqrt(ss);
  }
  __syncthreads();
  if constexpr (kVec) {
    // thread t: dimensions [kPer c, kPer c + kPer) for c = t, t + 256, ...
    for (int c = t; c < vecs; c += kPoolThreads) {
      double acc[kPer];
#pragma unroll
      for (int q = 0; q < kPer; ++q) acc[q] = 0.0;
      const uint4* col = reinterpret_cast<const uint4*>(f + row0 * a.dim) + c;
      for (int r = 0; r < rows; ++r) {
        const uint4 u = col[(int64_t)r * vecs];
        const T* e = reinterpret_cast<const T*>(&u);
#pragma unroll
        for (int q = 0; q < kPer; ++q) acc[q] = fma(feat_at(e, q), inv_norm[r], acc[q]);
      }
#pragma unroll
      for (int q = 0; q < kPer; ++q) fb[fb_at(b, kPer * c + q, a.nb, a.dim)] = acc[q] / (double)rows;
    }
  } else {
    for (int d = t; d < a.dim; d += kPoolThreads) {
      double acc = 0.0;
      for (int r = 0; r < rows; ++r) acc = fma(feat_at(f, (row0 + r) * a.dim + d), inv_norm[r], acc);
      fb[fb_at(b, d, a.nb, a.dim)] = acc / (double)rows;
    }
  }
}

// The same for rows of whole 16-byte vectors, at most 64 * kVecs of them,
// reading the features once: a wave keeps four rows at a time in registers
// (16 bytes per lane, row and 64 vectors) through their norms and their share
// of the weighted sum, the next four loading meanwhile; the four waves' sums
// meet in LDS. HBM-bound: 281 MB of 1024-wide bf16 features (137400 tokens)
// take 131 us read twice (and the means written as columns), 71 us so.
constexpr int kPoolWaves = 4;
constexpr int kPoolRows = 4;

template <typename T, int kVecs>
__global__ __launch_bounds__(64 * kPoolWaves) void cosine_pool_once_kernel(const T* __restrict__ f,
                                                                          double* __restrict__ fb,
                                                                          CosineArgs a) {
  extern __shared__ __attribute__((aligned(16))) double2 part[];  // kPoolWaves * 64 * kVecs * kPer doubles
  constexpr int kPer = 16 / (int)sizeof(T);
  constexpr int kPairs = kPer / 2;
  const int b = blockIdx.x;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int64_t row0 = (int64_t)b * kBlock;
  const int rows = (int)min<int64_t>(kBlock, a.n - row0);
  const int vecs = a.dim / kPer;
  uint4 next[kPoolRows][kVecs];
  // rows past the last token load it, and weigh nothing below
  auto load = [&](int r0) {
#pragma unroll
    for (int r = 0; r < kPoolRows; ++r) {
      const uint4* row = reinterpret_cast<const uint4*>(f + (row0 + min(r0 + r, rows - 1)) * a.dim);
#pragma unroll
      for (int v = 0; v < kVecs; ++v)
        next[r][v] = 64 * v + lane < vecs ? row[64 * v + lane] : uint4{0u, 0u, 0u, 0u};
    }
  };
  double2 acc[kVecs][kPairs];
#pragma unroll
  for (int v = 0; v < kVecs; ++v)
#pragma unroll
    for (int q = 0; q < kPairs; ++q) acc[v][q] = double2{0.0, 0.0};
  load(kPoolRows * wave);
#pragma unroll 1
  for (int r0 = kPoolRows * wave; r0 < rows; r0 += kPoolRows * kPoolWaves) {
    uint4 u[kPoolRows][kVecs];
#pragma unroll
    for (int r = 0; r < kPoolRows; ++r)
#pragma unroll
      for (int v = 0; v < kVecs; ++v) u[r][v] = next[r][v];
    if (r0 + kPoolRows * kPoolWaves < rows) load(r0 + kPoolRows * kPoolWaves);
    double inv[kPoolRows];
#pragma unroll
    for (int r = 0; r < kPoolRows; ++r) {
      double ss = 0.0;
#pragma unroll
      for (int v = 0; v < kVecs; ++v)
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
          const double x = feat_at(reinterpret_cast<const T*>(&u[r][v]), q);
          ss = fma(x, x, ss);
        }
      inv[r] = ss;
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1)
#pragma unroll
      for (int r = 0; r < kPoolRows; ++r) inv[r] += __shfl_xor(inv[r], m);
#pragma unroll
    for (int r = 0; r < kPoolRows; ++r) inv[r] = r0 + r < rows ? 1.0 / sqrt(inv[r]) : 0.0;
    // the sum widens the features again (kept from the norms, they would take four times the registers)
#pragma unroll
    for (int r = 0; r < kPoolRows; ++r)
#pragma unroll
      for (int v = 0; v < kVecs; ++v) {
        asm volatile("" : "+v"(u[r][v].x), "+v"(u[r][v].y), "+v"(u[r][v].z), "+v"(u[r][v].w));
#pragma unroll
        for (int q = 0; q < kPairs; ++q) {
          acc[v][q].x = fma(feat_at(reinterpret_cast<const T*>(&u[r][v]), 2 * q), inv[r], acc[v][q].x);
          acc[v][q].y = fma(feat_at(reinterpret_cast<const T*>(&u[r][v]), 2 * q + 1), inv[r], acc[v][q].y);
        }
      }
  }
  // [wave][vector / 64][pair of its dimensions][vector % 64]: 16-byte accesses without bank conflicts
#pragma unroll
  for (int v = 0; v < kVecs; ++v)
#pragma unroll
    for (int q = 0; q < kPairs; ++q) part[((wave * kVecs + v) * kPairs + q) * 64 + lane] = acc[v][q];
  __syncthreads();
  for (int c = t; c < vecs * kPairs; c += 64 * kPoolWaves) {  // pair c % kPairs of vector c / kPairs
    const int vec = c / kPairs, q = c % kPairs;
    double2 sum = {0.0, 0.0};
#pragma unroll
    for (int w = 0; w < kPoolWaves; ++w) {
      const double2 x = part[((w * kVecs + (vec >> 6)) * kPairs + q) * 64 + (vec & 63)];
      sum.x += x.x;
      sum.y += x.y;
    }
    double* dst = fb + fb_at(b, 2 * c, a.nb, a.dim);
    dst[0] = sum.x / (double)rows;
    dst[1] = sum.y / (double)rows;
  }
}

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

// sim[i][j] = sum_d fb[i][d] fb[j][d] on the fp64 matrix cores. A workgroup
// takes a tile of 32 rows x 64 columns; wave (c, half) its 32x32 part c over
// half the dimensions, as 2x2 tiles of v_mfma_f64_16x16x4f64 (lane: block
// lane % 16, dimensions from lane / 16), and the two halves meet in LDS: with
// whole sums per wave, 2147 blocks would make 2.3 waves per SIMD and take the
// time of 3. A lane reads two neighbouring dimensions (kPairs: 16 bytes, the
// lanes of an operand 1 KB in a row), so instruction k takes dimensions
// 8g + 2 (lane / 16) + k. Only tiles reaching the diagonal or above are
// computed, each stored transposed as well. XCD x takes a contiguous run of
// tiles in bands of 8 tile columns, so what it reads at a time fits its L2.
// 2147 blocks, 1024 dimensions: 175 us with 64x64 tiles on a [D][nb] matrix
// and half of the grid empty, 108 us so (65 at the rate of a large fp64 product).
constexpr int kSimBand = 8;

template <bool kPairs>
__global__ __launch_bounds__(256) void cosine_sim_mfma_kernel(const double* __restrict__ fb,
                                                             double* __restrict__ sim,
                                                             CosineArgs a, int units) {
  __shared__ double sums[2][16][64];
  const int nb = a.nb, dim = a.dim;
  const int tiles = (nb + 63) / 64;
  // 32-row i x 64-column j, i <= 2j + 1, numbered by bands of columns, then rows
  int r = (int)(blockIdx.x & 7) * ((units + 7) / 8) + (int)(blockIdx.x >> 3);
  if (r >= min(units, ((int)(blockIdx.x & 7) + 1) * ((units + 7) / 8))) return;
  int j0 = 0, width = min(kSimBand, tiles);
  for (;;) {
    const int in_band = width * (2 * j0 + width + 1);  // sum of 2j + 2 over its columns
    if (r < in_band) break;
    r -= in_band;
    j0 += kSimBand;
    width = min(kSimBand, tiles - j0);
  }
  int i, j;
  const int full = (2 * j0 + 2) * width;  // rows that all of the band's columns reach
  if (r < full) {
    i = r / width;
    j = j0 + r - i * width;
  } else {
    r -= full;
    int first = 1;  // the columns of row pair `first` below: j0 + first ..
    while (r >= 2 * (width - first)) {
      r -= 2 * (width - first);
      ++first;
    }
    const int second = r >= width - first ? 1 : 0;
    i = 2 * (j0 + first) + second;
    j = j0 + first + r - second * (width - first);
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r0 = i * 32, c0 = j * 64 + 32 * (wave & 1);
  const int half = wave >> 1;
  const int sub = lane >> 4;
  // half 0 takes the first half of the whole runs of 8 dimensions, half 1 the rest
  const int d_mid = 8 * ((dim / 8 + 1) / 2);
  const int d_lo = half ? d_mid : 0;
  const int d_hi = half ? dim : d_mid;
  // the four 16-block operands (byte offsets into fb, below 2^30; blocks past
  // the last one load it, and are never stored)
  uint32_t at[4], step_bytes[4];
#pragma unroll
  for (int o = 0; o < 4; ++o) {
    const int b0 = min((o < 2 ? r0 : c0) + 16 * (o & 1), (nb - 1) & ~15);
    const int blocks = min(16, nb - b0);
    step_bytes[o] = (uint32_t)blocks * 8 * sizeof(double);  // of 8 dimensions
    at[o] = ((uint32_t)b0 * dim + d_lo * blocks + min(lane & 15, blocks - 1) * 8 + 2 * sub) * sizeof(double);
  }
  f64x4 acc[2][2];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) acc[x][y] = f64x4{0.0, 0.0, 0.0, 0.0};
  const char* const fbb = reinterpret_cast<const char*>(fb);
  auto load = [&](uint32_t off) -> f64x2 {
    const double* x = reinterpret_cast<const double*>(fbb + off);
    if constexpr (kPairs) return *reinterpret_cast<const f64x2*>(x);
    else return f64x2{x[0], x[1]};
  };
  auto product = [&](const f64x2 (&op)[4]) {
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
          acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(op[x][k], op[2 + y][k], acc[x][y], 0, 0, 0);
  };
  // runs of 8 dimensions, two loading while two multiply
  const int runs = (d_hi - d_lo) / 8;  // whole ones
  f64x2 nx[2][4];
  if (runs > 0) {
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int o = 0; o < 4; ++o) nx[g][o] = load(at[o] + (runs > g ? g : 0) * step_bytes[o]);
  }
  for (int run = 0; run < runs; run += 2) {
    const bool more0 = run + 2 < runs, more1 = run + 3 < runs;
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      if (g == 1 && run + 1 >= runs) break;
      f64x2 cur[4];
#pragma unroll
      for (int o = 0; o < 4; ++o) {
        cur[o] = nx[g][o];
        // past the last run: this one again, unused
        nx[g][o] = load(at[o] + (g ? (more1 ? 3 : 1) : (more0 ? 2 : 0)) * step_bytes[o]);
      }
      product(cur);
    }
#pragma unroll
    for (int o = 0; o < 4; ++o) at[o] += 2 * step_bytes[o];
  }
  if (half && (dim & 7)) {  // the last, shorter run
    const int d = dim & ~7, width = dim & 7;
    f64x2 cur[4];
#pragma unroll
    for (int o = 0; o < 4; ++o) {
      const int b0 = min((o < 2 ? r0 : c0) + 16 * (o & 1), (nb - 1) & ~15);
      const int blocks = min(16, nb - b0);
      const double* x = fb + (int64_t)b0 * dim + d * blocks + min(lane & 15, blocks - 1) * width + 2 * sub;
      cur[o] = f64x2{2 * sub < width ? x[0] : 0.0, 2 * sub + 1 < width ? x[1] : 0.0};
    }
    product(cur);
  }
  if (half) {
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int y = 0; y < 2; ++y)
#pragma unroll
        for (int e = 0; e < 4; ++e) sums[wave & 1][(2 * x + y) * 4 + e][lane] = acc[x][y][e];
  }
  __syncthreads();
  if (half) return;
  // element e of a lane: row (lane / 16) + 4e, column lane % 16 of the tile
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = r0 + 16 * x + sub + 4 * e;
        const int col = c0 + 16 * y + (lane & 15);
        // NaN (of a zero, infinite or NaN feature row) ranks last, so that the lists can order every pair
        const double v = fmax(acc[x][y][e] + sums[wave & 1][(2 * x + y) * 4 + e][lane], -__builtin_inf());
        if (row <= col && col < nb) {
          sim[(int64_t)row * nb + col] = v;
          sim[(int64_t)col * nb + row] = v;
        }
      }
}

// (value, index) order of the selection: higher value first, then lower index
__device__ inline bool ranks_before(double v, int j, double w, int k) {
  return v > w || (v == w && j < k);
}

// Inclusive prefix sum over the 64 lanes.
__device__ inline int lane_scan_incl(int v) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int o = __shfl_up(v, d);
    if ((threadIdx.x & 63) >= d) v += o;
  }
  return v;
}

// The kFew best (value desc, index asc) of row[j_lo, j_hi), best first; nb and
// -inf where there are fewer. Indices ascend, so an equal value never ranks
// before an earlier one and a pair moves up on a strictly larger value or into
// an empty place only (a value may be -inf).
template <int kFew>
__device__ __forceinline__ void best_few(const double* row, int j_lo, int j_hi, int nb, double (&bv)[kFew],
                                         int (&bj)[kFew]) {
#pragma unroll
  for (int p = 0; p < kFew; ++p) {
    bv[p] = -__builtin_inf();
    bj[p] = nb;
  }
  for (int j = j_lo; j < j_hi; ++j) {
    const double v = row[j];
    bool up[kFew];
#pragma unroll
    for (int p = 0; p < kFew; ++p) up[p] = v > bv[p] || bj[p] == nb;
#pragma unroll
    for (int p = kFew - 1; p >= 0; --p) {
      const bool shift = p > 0 && up[p > 0 ? p - 1 : 0];  // the pair before moves down to p
      bv[p] = shift ? bv[p > 0 ? p - 1 : 0] : up[p] ? v : bv[p];
      bj[p] = shift ? bj[p > 0 ? p - 1 : 0] : up[p] ? j : bj[p];
    }
  }
}

// One workgroup per (group of cosine heads with one per-frame count k, query
// block), one thread per frame (kTopkThreads frames per pass). The frame's
// min(k, blocks) best (similarity desc, index asc) pairs are kept: for k up to
// kTopkFew one scan of its blocks finds them; above that further scans find
// the k-th and one more those ranked before it. They go, ascending, to the
// frame's offset (a prefix sum over the frames) in the list in LDS, which then
// goes out coalesced into the row of every head of the group.
// kLds: the similarity row is first copied into LDS (rows up to kTopkLdsRow
// doubles). 2147 blocks, 100 frames, k = 2 for 16 heads: 71 us with one wave
// per row, two passes over the frames and k + 2 scans, 27 us so.
constexpr int kTopkLdsRow = 8192;
constexpr int kTopkThreads = 256;
constexpr int kTopkFew = 4;

// list entries kept in LDS: a row keeps at most nb blocks
__host__ __device__ inline int topk_list_len(const CosineArgs& a) { return a.cap < a.nb ? a.cap : a.nb; }

template <bool kLds>
__global__ __launch_bounds__(kTopkThreads) void cosine_topk_kernel(const double* __restrict__ sim,
                                                                  int32_t* __restrict__ idx,
                                                                  int32_t* __restrict__ cnt,
                                                                  CosineArgs a) {
  extern __shared__ double srow[];  // [nb] doubles when kLds, then [list_len] ints
  __shared__ int wave_kept[kTopkThreads / 64];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int g = blockIdx.x / a.nb;
  const int i = blockIdx.x - g * a.nb;
  const int k = a.group_k[g];
  const int q0 = a.group_start[g], q1 = a.group_start[g + 1];
  const double* grow = sim + (int64_t)i * a.nb;
  const int list_len = topk_list_len(a);
  int* llist = reinterpret_cast<int*>(srow + (kLds ? a.nb : 0));
  if constexpr (kLds) {
    for (int j = t; j < a.nb; j += kTopkThreads) srow[j] = grow[j];
    __syncthreads();
  }
  const double* row = kLds ? srow : grow;
  const int64_t T = a.tokens_per_frame;
  const int frames = (int)((a.n + T - 1) / T);
  int base = 0;
  for (int f0 = 0; f0 < frames; f0 += kTopkThreads) {
    // key blocks whose first token lies in frame f
    const int f = f0 + t;
    int j_lo = 0, j_hi = 0;
    if (f < frames) {
      j_lo = (int)(((int64_t)f * T + kBlock - 1) / kBlock);
      j_hi = (int)min<int64_t>(((int64_t)(f + 1) * T + kBlock - 1) / kBlock, a.nb);
    }
    const int kk = min(k, max(j_hi - j_lo, 0));
    const int incl = lane_scan_incl(kk);
    if (lane == 63) wave_kept[wave] = incl;
    __syncthreads();
    int pos = base + incl - kk;
    for (int w = 0; w < wave; ++w) pos += wave_kept[w];
    auto put = [&](int j) {
      if (pos < list_len) llist[pos] = j;
      ++pos;
    };
    if (kk > 0 && k == 1) {
      double bv[1];
      int bj[1];
      best_few<1>(row, j_lo, j_hi, a.nb, bv, bj);
      put(bj[0]);
    } else if (kk > 0 && k == 2) {
      double bv[2];
      int bj[2];
      best_few<2>(row, j_lo, j_hi, a.nb, bv, bj);
      put(min(bj[0], bj[1]));
      if (kk == 2) put(max(bj[0], bj[1]));
    } else if (kk > 0) {
      double bv[kTopkFew];
      int bj[kTopkFew];
      best_few<kTopkFew>(row, j_lo, j_hi, a.nb, bv, bj);
      double tv = bv[0];  // the kk-th pair
      int tj = bj[0];
#pragma unroll
      for (int p = 1; p < kTopkFew; ++p)
        if (p < kk) {
          tv = bv[p];
          tj = bj[p];
        }
      for (int p = kTopkFew; p < kk; ++p) {  // each scan takes the best pair ranked after the last
        double v1 = -__builtin_inf();
        int j1 = a.nb;
        for (int j = j_lo; j < j_hi; ++j) {
          const double v = row[j];
          if (ranks_before(tv, tj, v, j) && ranks_before(v, j, v1, j1)) {
            v1 = v;
            j1 = j;
          }
        }
        tv = v1;
        tj = j1;
      }
      const int end = pos + kk;
      for (int j = j_lo; j < j_hi && pos < end; ++j)
        if (!ranks_before(tv, tj, row[j], j)) put(j);
    }
#pragma unroll
    for (int w = 0; w < kTopkThreads / 64; ++w) base += wave_kept[w];
    __syncthreads();
  }
  for (int q = q0; q < q1; ++q) {
    const int h = a.head[q];
    int32_t* dst = idx + ((int64_t)h * a.nb + i) * a.cap;
    for (int p = t; p < a.cap; p += kTopkThreads) dst[p] = p < base ? llist[p] : -1;
    if (t == 0) cnt[(int64_t)h * a.nb + i] = base;
  }
}

}  // namespace

hipError_t launch_cosine(int dtype, const void* f, double* fb, double* sim, int32_t* idx,
                         int32_t* cnt, const CosineArgs& a, hipStream_t s) {
  if (a.n_groups == 0) return hipSuccess;
  const int esz = dtype == 1 ? 2 : 4;
  const bool vec = ((int64_t)a.dim * esz) % 16 == 0 && (reinterpret_cast<uintptr_t>(f) & 15) == 0;
  const dim3 grid((unsigned)a.nb);
  // features read once: rows of up to 64 * 4 vectors, whose partial sums take
  // 16 KB (bf16) or 8 KB (fp32) of LDS per 64 vectors: at most 64 KB
  const int row_vecs = vec ? (int)((int64_t)a.dim * esz / 16) : 0;
  auto part_bytes = [&](int vecs) { return (size_t)kPoolWaves * 64 * vecs * (16 / esz) * sizeof(double); };
  auto pool = [&](auto kern, int threads, size_t lds, auto* fp) -> hipError_t {
    if (lds > 0) {
      hipError_t e2 = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e2 != hipSuccess) return e2;
    }
    hipLaunchKernelGGL(kern, grid, dim3(threads), lds, s, fp, fb, a);
    return hipGetLastError();
  };
  auto pool_any = [&](auto* fp) -> hipError_t {
    using T = std::remove_cv_t<std::remove_pointer_t<decltype(fp)>>;
    if (row_vecs > 0 && row_vecs <= 64) return pool(cosine_pool_once_kernel<T, 1>, 64 * kPoolWaves, part_bytes(1), fp);
    if (row_vecs > 0 && row_vecs <= 128) return pool(cosine_pool_once_kernel<T, 2>, 64 * kPoolWaves, part_bytes(2), fp);
    if (row_vecs > 0 && row_vecs <= 256) return pool(cosine_pool_once_kernel<T, 4>, 64 * kPoolWaves, part_bytes(4), fp);
    if (vec) return pool(cosine_pool_kernel<T, true>, kPoolThreads, 0, fp);
    return pool(cosine_pool_kernel<T, false>, kPoolThreads, 0, fp);
  };
  hipError_t e = dtype == 1 ? pool_any(static_cast<const uint16_t*>(f)) : pool_any(static_cast<const float*>(f));
  if (e != hipSuccess) return e;
  const int tiles = (a.nb + 63) / 64;
  const int units = tiles * (tiles + 1);  // 32 x 64 tiles reaching the diagonal or above
  const dim3 sgrid((unsigned)(8 * ((units + 7) / 8)));
  if (a.dim % 2 == 0 && (reinterpret_cast<uintptr_t>(fb) & 15) == 0)
    hipLaunchKernelGGL(cosine_sim_mfma_kernel<true>, sgrid, dim3(256), 0, s, fb, sim, a, units);
  else
    hipLaunchKernelGGL(cosine_sim_mfma_kernel<false>, sgrid, dim3(256), 0, s, fb, sim, a, units);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  const bool lds_row = a.nb <= kTopkLdsRow;
  const size_t lds = (lds_row ? (size_t)a.nb * sizeof(double) : 0) + (size_t)topk_list_len(a) * sizeof(int);
  auto go = [&](auto kern) -> hipError_t {
    hipError_t e2 = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e2 != hipSuccess) return e2;
    hipLaunchKernelGGL(kern, dim3((unsigned)(a.n_groups * a.nb)), dim3(kTopkThreads), lds, s, sim, idx, cnt, a);
    return hipGetLastError();
  };
  return lds_row ? go(cosine_topk_kernel<true>) : go(cosine_topk_kernel<false>);
}

}  // namespace saf3r
