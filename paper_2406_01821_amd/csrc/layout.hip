// Dataset upload: validation, label grouping, feature-major transpose, tau.
//
// The resident layout stores the samples feature-major (x_fm[f][n_pad]) so
// that a wave reads one feature of 64..256 consecutive samples with one
// coalesced access.  Samples are stably grouped by label and every class
// region is padded to a multiple of AERL_TILE samples, so every tile holds a
// single label; fitness counts do not depend on the sample order (accuracy
// is a sum over samples, Section 1).
//
// Four launches, no host step between them: labels counted per group of
// rows, the counts scanned per class, one pass over x that validates it,
// writes it grouped and transposed and keeps per-column statistics, and the
// rest of the layout (tile table, padding, tau).  The pass over x reads and
// writes every value once, which bounds it: on 2^20 x 64 (268 MB each way) it
// takes 118 us (4.5 TB/s; a plain copy reaches 5.2) and the four launches 133
// us together; a separate validation, a fill of the whole layout, stores in
// row order and two passes over the layout for tau took 560 us.
#include "internal.h"

namespace aerl {

namespace {

__global__ void k_fill_i32(int32_t *__restrict__ p, int64_t n, int32_t v) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = v;
}

__global__ void k_copy16(uint4 *__restrict__ dst, const uint4 *__restrict__ src, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += stride) dst[i] = src[i];
}

// counts[c][g]: samples of class c among rows [g*R, (g+1)*R); c = nc: labels
// outside [0, nc).  R is a power of two, 32..256.
constexpr int kCountBlock = 256, kCountRows = 1024, kCountGroups = kCountRows / 32;
__global__ __launch_bounds__(kCountBlock) void k_count_labels(const int32_t *__restrict__ y,
                                                              int64_t n, int32_t nc, int32_t R,
                                                              int64_t n_groups,
                                                              int32_t *__restrict__ counts) {
  __shared__ int32_t hist[(AERL_MAX_CLASSES + 1) * kCountGroups];
  const int groups = kCountRows / R;
  for (int i = threadIdx.x; i < (nc + 1) * groups; i += kCountBlock) hist[i] = 0;
  __syncthreads();
  const int64_t i0 = (int64_t)blockIdx.x * kCountRows;
  for (int k = threadIdx.x; k < kCountRows; k += kCountBlock) {
    if (i0 + k >= n) break;
    const int32_t c = y[i0 + k];
    atomicAdd(&hist[(c < 0 || c >= nc ? nc : c) * groups + k / R], 1);
  }
  __syncthreads();
  const int64_t g0 = (int64_t)blockIdx.x * groups;
  for (int i = threadIdx.x; i < (nc + 1) * groups; i += kCountBlock) {
    const int64_t g = g0 + i % groups;
    if (g < n_groups) counts[(int64_t)(i / groups) * n_groups + g] = hist[i];
  }
}

// Block c turns counts[c] into its exclusive prefix sums and writes the
// class's total to head[c] (c = nc: the bad labels; it also clears the
// bad-feature flag head[nc + 1]).
constexpr int kScanBlock = 1024;
__global__ __launch_bounds__(kScanBlock) void k_scan_counts(int32_t *__restrict__ counts,
                                                            int64_t n_groups, int32_t nc,
                                                            int32_t *__restrict__ head) {
  __shared__ int32_t wave_sum[kScanBlock / 64];
  int32_t *row = counts + (int64_t)blockIdx.x * n_groups;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int32_t run = 0;
  for (int64_t g0 = 0; g0 < n_groups; g0 += kScanBlock) {
    const int64_t g = g0 + threadIdx.x;
    const int32_t v = g < n_groups ? row[g] : 0;
    int32_t s = v;
    for (int d = 1; d < 64; d <<= 1) {
      const int32_t u = __shfl_up(s, d);
      if (lane >= d) s += u;
    }
    if (lane == 63) wave_sum[w] = s;
    __syncthreads();
    int32_t before = run, total = run;
    for (int k = 0; k < kScanBlock / 64; ++k) {
      if (k < w) before += wave_sum[k];
      total += wave_sum[k];
    }
    if (g < n_groups) row[g] = before + s - v;
    run = total;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    head[blockIdx.x] = run;
    if ((int)blockIdx.x == nc) head[nc + 1] = 0;
  }
}

// First tile of every class region from the class totals, then the tile
// count: tile0[0..nc].  All threads of the block call it; ends with a barrier.
__device__ __forceinline__ void class_regions(const int32_t *__restrict__ head, int nc,
                                              int32_t *tile0) {
  if ((int)threadIdx.x <= nc) {
    int32_t t = 0;
    for (int c = 0; c < (int)threadIdx.x; ++c) t += (int32_t)(((int64_t)head[c] + AERL_TILE - 1) / AERL_TILE);
    tile0[threadIdx.x] = t;
  }
  __syncthreads();
}

// Count, mean and sum of squared deviations of a set of values, and the
// merge of two sets (Chan, Golub and LeVeque 1979).
struct Moments {
  double n, mean, m2;
};
__device__ __forceinline__ void merge(Moments &a, const Moments &b) {
  const double n = a.n + b.n;
  if (b.n == 0.0) return;
  const double d = b.mean - a.mean, w = b.n / n;
  a.m2 += b.m2 + d * d * (a.n * w);
  a.mean += d * w;
  a.n = n;
}

// Rows [g*R, (g+1)*R) at a time: staged into LDS with one coalesced read
// (row pitch an odd number of 16-byte words, so that a column of 16-byte
// words is read without bank conflicts), ordered by class through a table
// of the group's rows, and stored feature by feature: consecutive lanes
// store consecutive slots of a class, runs of about R/nc samples.  A block
// takes a contiguous range of groups, so the lines at the ends of its runs
// are completed in the same L2.  LDS of up to 70 KiB leaves two blocks per
// CU.  The rank of a sample in its class comes from wave ballots and the
// scanned group counts, so each class keeps the original order.  Thread t
// also keeps the moments of column t mod cols over its share of the rows.
constexpr int kRegroupBlock = 512;
constexpr int kRegroupWaves = kRegroupBlock / 64;
struct RegroupArgs {
  const float *x;
  const int32_t *y;
  int64_t n, n_groups;
  int32_t nf, nc, R, p4, cols;  // rows per group, LDS row pitch / 16 B, nf up to a power of two
  uint32_t magic;               // ceil(2^32 / words per row), 0 for one word: row of a staged word
  int32_t vec;                  // 16-byte loads
  const int32_t *prefix;        // [nc][n_groups]
  int32_t *head;
  float *x_fm;
  int32_t *y_pad, *perm;
  double *part;  // [nf][3][gridDim.x]
};
__global__ __launch_bounds__(kRegroupBlock) void k_regroup(const RegroupArgs a) {
  extern __shared__ __align__(16) float tile[];  // [R][4 * p4]
  __shared__ int32_t wave_count[4][AERL_MAX_CLASSES];
  __shared__ int32_t tile0[AERL_MAX_CLASSES + 1], start[AERL_MAX_CLASSES], slot0[AERL_MAX_CLASSES];
  __shared__ int32_t order[256], slot[256];
  __shared__ int32_t n_sorted;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  class_regions(a.head, a.nc, tile0);
  const int64_t n_pad = (int64_t)tile0[a.nc] * AERL_TILE;
  const int pitch = 4 * a.p4, f_words = (a.nf + 3) / 4;
  const int col = t & (a.cols - 1), col_part = t / a.cols, col_parts = kRegroupBlock / a.cols;
  Moments mom = {0.0, 0.0, 0.0};
  int bad = 0;
  const int64_t g0 = a.n_groups * blockIdx.x / gridDim.x, g1 = a.n_groups * (blockIdx.x + 1) / gridDim.x;
  for (int64_t g = g0; g < g1; ++g) {
    const int64_t i0 = g * a.R;
    const int rows = (int)min((int64_t)a.R, a.n - i0);
    // the rows, eight words per thread in flight
    constexpr int kFly = 8;
    if (a.vec) {
      typedef float f4v __attribute__((ext_vector_type(4)));
      const f4v *src = reinterpret_cast<const f4v *>(a.x + i0 * a.nf);
      const int q4 = a.nf / 4, words = rows * q4;
      for (int b = t; b < words; b += kFly * kRegroupBlock) {
        f4v v[kFly];
#pragma unroll
        for (int k = 0; k < kFly; ++k)
          v[k] = __builtin_nontemporal_load(src + min(b + k * kRegroupBlock, words - 1));
#pragma unroll
        for (int k = 0; k < kFly; ++k) {
          const int i = b + k * kRegroupBlock;
          if (i >= words) break;
          const int r = a.magic ? (int)__umulhi((uint32_t)i, a.magic) : i;
          reinterpret_cast<f4v *>(tile)[r * a.p4 + i - r * q4] = v[k];
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (!__builtin_isfinite(v[k][e])) bad = 1;
        }
      }
    } else {
      const float *src = a.x + i0 * a.nf;
      const int words = rows * a.nf;
      for (int b = t; b < words; b += kFly * kRegroupBlock) {
        float v[kFly];
#pragma unroll
        for (int k = 0; k < kFly; ++k) v[k] = src[min(b + k * kRegroupBlock, words - 1)];
#pragma unroll
        for (int k = 0; k < kFly; ++k) {
          const int i = b + k * kRegroupBlock;
          if (i >= words) break;
          const int r = a.magic ? (int)__umulhi((uint32_t)i, a.magic) : i;
          tile[r * pitch + i - r * a.nf] = v[k];
          if (!__builtin_isfinite(v[k])) bad = 1;
        }
      }
    }
    // the group's rows by class, in order
    int32_t c_me = -1, rank = 0;
    if (t < 256) {
      if (t < rows) c_me = a.y[i0 + t];
      if (c_me >= a.nc) c_me = -1;
      const uint64_t below = lane == 0 ? 0ull : ~0ull >> (64 - lane);
      for (int c = 0; c < a.nc; ++c) {
        const uint64_t m = __builtin_amdgcn_ballot_w64(c_me == c);
        if (c_me == c) rank = __builtin_popcountll(m & below);
        if (lane == 0) wave_count[w][c] = __builtin_popcountll(m);
      }
    }
    __syncthreads();
    if (t < a.nc) {
      int32_t s = 0;
      for (int c = 0; c < t; ++c)
        s += wave_count[0][c] + wave_count[1][c] + wave_count[2][c] + wave_count[3][c];
      start[t] = s;
      slot0[t] = tile0[t] * AERL_TILE + a.prefix[(int64_t)t * a.n_groups + g];
      if (t == a.nc - 1)
        n_sorted = s + wave_count[0][t] + wave_count[1][t] + wave_count[2][t] + wave_count[3][t];
    }
    __syncthreads();
    if (c_me >= 0) {
      for (int ww = 0; ww < w; ++ww) rank += wave_count[ww][c_me];
      order[start[c_me] + rank] = t;
      slot[start[c_me] + rank] = slot0[c_me] + rank;
    }
    __syncthreads();
    const int sorted = n_sorted, at = t & (a.R - 1), stride = kRegroupBlock / a.R;
    if (at < sorted) {
      const int r = order[at];
      const int64_t s = slot[at];
      for (int q = t / a.R; q < f_words; q += stride) {
        const float4 v = reinterpret_cast<const float4 *>(tile)[r * a.p4 + q];
        float *dst = a.x_fm + (int64_t)(4 * q) * n_pad + s;
        dst[0] = v.x;
        if (4 * q + 1 < a.nf) dst[n_pad] = v.y;
        if (4 * q + 2 < a.nf) dst[2 * n_pad] = v.z;
        if (4 * q + 3 < a.nf) dst[3 * n_pad] = v.w;
      }
      if (t < a.R) {
        int c = 0;
        while (c + 1 < a.nc && start[c + 1] <= at) ++c;
        a.y_pad[s] = c;
        a.perm[s] = (int32_t)(i0 + r);
      }
    }
    if (col < a.nf) {
      Moments m = {0.0, 0.0, 0.0};
      double s = 0.0;
      for (int r = col_part; r < rows; r += col_parts) s += (double)tile[r * pitch + col];
      m.n = (double)((rows - col_part + col_parts - 1) / col_parts);
      if (col_part < rows) {
        m.mean = s / m.n;
        for (int r = col_part; r < rows; r += col_parts) {
          const double d = (double)tile[r * pitch + col] - m.mean;
          m.m2 += d * d;
        }
        merge(mom, m);
      }
    }
    __syncthreads();
  }
  if (bad) atomicOr(&a.head[a.nc + 1], 1);
  // the block's moments of each column, its shares merged in order
  double *sh = reinterpret_cast<double *>(tile);
  sh[t] = mom.n;
  sh[kRegroupBlock + t] = mom.mean;
  sh[2 * kRegroupBlock + t] = mom.m2;
  __syncthreads();
  if (t < a.nf) {
    Moments m = {0.0, 0.0, 0.0};
    for (int k = 0; k < col_parts; ++k) {
      const int i = k * a.cols + t;
      merge(m, Moments{sh[i], sh[kRegroupBlock + i], sh[2 * kRegroupBlock + i]});
    }
    double *p = a.part + (int64_t)t * 3 * gridDim.x + blockIdx.x;
    p[0] = m.n;
    p[gridDim.x] = m.mean;
    p[2 * gridDim.x] = m.m2;
  }
}

// The rest of the layout.  Blocks [0, nf): tau[f] = 0.05 * population std
// over the real samples (1 if the std is 0), fp64, rounded to float, and
// 1/tau, from the column's partial moments, merged in a fixed order so that
// tau is the same from run to run.  Then one block per (class, feature row
// or y_pad or perm): the padding slots of the class's region.  The last
// blocks: the tile table.
constexpr int kTailBlock = 256, kTileBlocks = 64;
__global__ __launch_bounds__(kTailBlock) void k_layout_tail(
    const int32_t *__restrict__ head, int32_t nf, int32_t nc, int64_t n,
    const double *__restrict__ part, int32_t n_parts, float *__restrict__ x_fm,
    int32_t *__restrict__ y_pad, int32_t *__restrict__ perm, int32_t *__restrict__ tile_info,
    float *__restrict__ tau) {
  __shared__ int32_t tile0[AERL_MAX_CLASSES + 1];
  __shared__ Moments red[kTailBlock];
  const int t = threadIdx.x;
  int b = blockIdx.x;
  if (b < nf) {
    const double *p = part + (int64_t)b * 3 * n_parts;
    Moments m = {0.0, 0.0, 0.0};
    for (int k = t; k < n_parts; k += kTailBlock)
      merge(m, Moments{p[k], p[n_parts + k], p[2 * n_parts + k]});
    red[t] = m;
    __syncthreads();
    for (int h = kTailBlock / 2; h > 0; h >>= 1) {
      if (t < h) merge(red[t], red[t + h]);
      __syncthreads();
    }
    if (t == 0) {
      const double sd = n > 0 ? sqrt(red[0].m2 / (double)n) : 0.0;
      const float tf = sd > 0.0 ? (float)(0.05 * sd) : 1.0f;
      tau[b] = tf;
      tau[nf + b] = (float)(1.0 / (double)tf);  // 1/tau follows tau
    }
    return;
  }
  class_regions(head, nc, tile0);
  b -= nf;
  const int64_t n_pad = (int64_t)tile0[nc] * AERL_TILE;
  if (b < nc * (nf + 2)) {
    const int c = b % nc, row = b / nc;
    const int64_t s = (int64_t)tile0[c] * AERL_TILE + head[c] + t;
    if (s < (int64_t)tile0[c + 1] * AERL_TILE) {
      if (row < nf)
        x_fm[(int64_t)row * n_pad + s] = 0.0f;
      else
        (row == nf ? y_pad : perm)[s] = -1;
    }
    return;
  }
  b -= nc * (nf + 2);
  for (int64_t i = (int64_t)b * kTailBlock + t; i < tile0[nc]; i += kTileBlocks * kTailBlock) {
    int c = 0;
    while (c + 1 < nc && tile0[c + 1] <= i) ++c;
    const int64_t left = head[c] - (i - tile0[c]) * AERL_TILE;
    tile_info[i] = c | (int32_t)min((int64_t)AERL_TILE, left) << 8;
  }
}

}  // namespace

hipError_t launch_fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)blocks), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

hipError_t launch_copy16(void *dst, const void *src, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (((uintptr_t)dst | (uintptr_t)src) & 15) return hipErrorInvalidValue;
  const int64_t blocks = std::min<int64_t>((n + 255) / 256, 512);
  hipLaunchKernelGGL(k_copy16, dim3((unsigned)blocks), dim3(256), 0, s, static_cast<uint4 *>(dst),
                     static_cast<const uint4 *>(src), n);
  return hipGetLastError();
}

namespace {
// LDS row pitch of k_regroup in 16-byte words: odd.
int regroup_pitch4(int nf) { return ((nf + 3) / 4) | 1; }
}  // namespace

UploadShape upload_shape(int64_t n, int32_t nf) {
  UploadShape p;
  const int row = 16 * regroup_pitch4(nf);
  p.rows = 256;
  while (p.rows > 32 && p.rows * row > 70 * 1024) p.rows >>= 1;
  p.n_groups = (n + p.rows - 1) / p.rows;
  p.parts = (int32_t)std::max<int64_t>(1, std::min<int64_t>(p.n_groups, kUploadParts));
  return p;
}

hipError_t launch_upload(const UploadLaunch &u, hipStream_t s) {
  const UploadShape p = upload_shape(u.n, u.nf);
  if (p.n_groups > 0)
    hipLaunchKernelGGL(k_count_labels, dim3((unsigned)((u.n + kCountRows - 1) / kCountRows)),
                       dim3(kCountBlock), 0, s, u.y, u.n, u.nc, p.rows, p.n_groups, u.counts);
  hipLaunchKernelGGL(k_scan_counts, dim3((unsigned)u.nc + 1), dim3(kScanBlock), 0, s, u.counts,
                     p.n_groups, u.nc, u.head);
  RegroupArgs a{};
  a.x = u.x;
  a.y = u.y;
  a.n = u.n;
  a.n_groups = p.n_groups;
  a.nf = u.nf;
  a.nc = u.nc;
  a.R = p.rows;
  a.p4 = regroup_pitch4(u.nf);
  a.cols = 1;
  while (a.cols < u.nf) a.cols *= 2;
  a.vec = u.nf % 4 == 0 && ((uintptr_t)u.x & 15) == 0;
  const uint32_t per_row = (uint32_t)(a.vec ? u.nf / 4 : u.nf);
  a.magic = per_row > 1 ? (uint32_t)((((uint64_t)1 << 32) + per_row - 1) / per_row) : 0u;
  a.prefix = u.counts;
  a.head = u.head;
  a.x_fm = u.x_fm;
  a.y_pad = u.y_pad;
  a.perm = u.perm;
  a.part = u.part;
  const size_t lds = std::max((size_t)p.rows * a.p4 * 16, (size_t)3 * kRegroupBlock * sizeof(double));
  hipLaunchKernelGGL(k_regroup, dim3((unsigned)p.parts), dim3(kRegroupBlock), lds, s, a);
  hipLaunchKernelGGL(k_layout_tail, dim3((unsigned)(u.nf + u.nc * (u.nf + 2) + kTileBlocks)),
                     dim3(kTailBlock), 0, s, u.head, u.nf, u.nc, u.n, u.part, p.parts, u.x_fm, u.y_pad,
                     u.perm, u.tile_info, u.tau);
  return hipGetLastError();
}

}  // namespace aerl
