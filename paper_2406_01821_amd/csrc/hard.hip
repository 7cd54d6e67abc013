// Hard fitness (correct counts + confusion) and prediction kernels.
//
// Fitness of a rule set is its classification accuracy on the labeled
// dataset (Section 1), with rules read as a first-firing decision list of
// ANDed step-activated conditions (Section 3, Fig. 1).
//
// Work decomposition of k_hard: block (chunk, group) evaluates rule sets
// [chunk*Q, chunk*Q+Q) on the layout tiles of one tile group; a group lies
// inside one class region, so every sample of the block has the same label.
// The block stages one wave tile (64*S samples x F features, fp32) at a time
// into LDS with coalesced 16-byte loads; its waves then pull rule sets from
// an LDS counter and evaluate them against the staged tile.  Per-class
// prediction counts accumulate in LDS (one writer per rule set and tile) and
// are added to the global outputs once per block with integer atomics, so
// the result does not depend on the schedule.
#include "eval_core.h"
#include "hard_block.h"
#include "predict_block.h"
#include "internal.h"

namespace aerl {

namespace {

constexpr int kHardBlock = 1024;
constexpr int kPredictBlock = 1024;
constexpr int64_t kPredictWideRows = 1 << 18;
constexpr int kPredictWideFeatures = 32;

struct HardArgs {
  const float *x_fm;
  int64_t n_pad;
  int32_t nf, nc;
  const int32_t *tile_info;
  const int4 *sets;
  const uint4 *conds;
  const uint4 *heads;
  int32_t set_begin, set_count;
  int32_t *correct;
  int32_t *confusion;
  uint32_t *part;
  int32_t sets_per_chunk, tiles_per_group, n_chunks;
  int32_t region_tile0[AERL_MAX_CLASSES];
  int32_t region_tiles[AERL_MAX_CLASSES];
};

// CAT: the population has categorical conditions (their walk body is left
// out of the other instantiation, which keeps the common walk's code tight).
// C10: single-tile groups (10-bit LDS counters).
template <int S, bool CAT, bool C10>
__global__ __launch_bounds__(kHardBlock, 8) AERL_HARD_SGPR_CAP void k_hard(const HardArgs a) {
  extern __shared__ __align__(16) float smem[];
  __shared__ int32_t sh[2];
  // Which class region and which tiles this block covers (uniform loop).
  HardTask t;
  t.x_fm = a.x_fm;
  t.n_pad = a.n_pad;
  t.nf = a.nf;
  t.nc = a.nc;
  t.tile_info = a.tile_info;
  t.sets = a.sets + a.set_begin;
  t.conds = a.conds;
  t.heads = a.heads;
  t.correct = a.correct;
  t.confusion = a.confusion;
  t.part = nullptr;
  t.part_stride = 0;
  t.label = 0;
  t.tile_lo = t.tile_hi = 0;
  // one-dimensional grid, set chunk fastest: consecutive blocks share a tile
  // group, and (blocks being spread over the XCDs in turn) an XCD keeps
  // seeing the same chunk's records when the chunk count divides eight
  const int chunk = (int)(blockIdx.x % (unsigned)a.n_chunks);
  {
    int g = (int)(blockIdx.x / (unsigned)a.n_chunks);
    for (int c = 0; c < a.nc; ++c) {
      const int ng = (a.region_tiles[c] + a.tiles_per_group - 1) / a.tiles_per_group;
      if (g < ng) {
        t.label = c;
        t.tile_lo = a.region_tile0[c] + g * a.tiles_per_group;
        t.tile_hi = min(t.tile_lo + a.tiles_per_group, a.region_tile0[c] + a.region_tiles[c]);
        break;
      }
      g -= ng;
    }
  }
  t.q0 = chunk * a.sets_per_chunk;
  t.Q = min(a.sets_per_chunk, a.set_count - t.q0);
  if (C10 && a.part) {
    const int wpc = hard_part_chunk_words(a.sets_per_chunk, a.nc);
    t.part = a.part + (int64_t)chunk * wpc;
    t.part_stride = a.n_chunks * wpc;
  }
  hard_block<S, CAT, C10>(t, smem, sh);
}

// Sums the per-tile counter words of a hard-eval launch over the tiles of
// each class region.  A tile's row holds, chunk by chunk of Q rule sets,
// the 10-bit counters of classes 0..nc-2 among the tile's real samples,
// counter i = q*(nc-1) + c of the chunk's set q in bits 10*(i%3) of word
// i/3 (at most two words per set); class nc-1 gets the rest of them.
// Thread p of block (x, y) takes rule set 256x + p over the tiles of slice
// y (neighbouring threads read neighbouring words of a tile's row) and adds
// each class region's totals to the outputs.
constexpr int kReduceBlock = 256;
__global__ __launch_bounds__(kReduceBlock) void k_hard_reduce(
    const uint32_t *__restrict__ part, const int32_t *__restrict__ tile_info, int64_t n_tiles,
    int32_t n_sets, int32_t Q, int32_t nc, int32_t *__restrict__ correct,
    int32_t *__restrict__ confusion) {
  const int p = blockIdx.x * kReduceBlock + threadIdx.x;
  if (p >= n_sets) return;
  const int ncc = nc - 1;
  const int wpc = hard_part_chunk_words(Q, nc);
  const int64_t stride = (int64_t)((n_sets + Q - 1) / Q) * wpc;
  const int i = (p % Q) * ncc;
  const int64_t w = (int64_t)(p / Q) * wpc + i / 3;
  const int b = i % 3 * 10;
  // the word after w when the set's counters run into it, else w again (a
  // second read of the same word keeps the loop free of branches)
  const int w2 = i % 3 + ncc > 3 ? 1 : 0;
  const int64_t t0 = n_tiles * blockIdx.y / gridDim.y, t1 = n_tiles * (blockIdx.y + 1) / gridDim.y;
  int label = -1;
  int32_t c0 = 0, c1 = 0, c2 = 0, n = 0;
  auto emit = [&]() {
    if (label < 0) return;
    for (int c = 0; c < nc; ++c) {
      const int32_t v = c == nc - 1 ? n - c0 - c1 - c2 : c == 0 ? c0 : c == 1 ? c1 : c2;
      if (v == 0) continue;
      if (confusion) atomicAdd(&confusion[((int64_t)p * nc + label) * nc + c], v);
      if (c == label) atomicAdd(&correct[p], v);
    }
  };
  // tiles in order, the words of eight requested before they are used
  constexpr int kBatch = 8;
  for (int64_t tb = t0; tb < t1; tb += kBatch) {
    uint32_t lo[kBatch], hi[kBatch];
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      const int64_t t = min(tb + k, t1 - 1);  // past the slice: its last tile again, unused
      const uint32_t *row = part + t * stride + w;
      lo[k] = row[0];
      hi[k] = row[w2];
    }
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      if (tb + k >= t1) break;
      const int info = ldc(tile_info, tb + k);
      if ((info & 0xff) != label) {
        emit();
        label = info & 0xff;
        c0 = c1 = c2 = n = 0;
      }
      // the set's fields from bit 0 on, ten bits each (those past its ncc
      // are not used)
      const uint64_t v = ((uint64_t)hi[k] << 30 | lo[k]) >> b;
      c0 += (int32_t)(v & 1023u);
      if (ncc > 1) c1 += (int32_t)(v >> 10 & 1023u);
      if (ncc > 2) c2 += (int32_t)(v >> 20 & 1023u);
      n += info >> 8;
    }
  }
  emit();
}

struct HardTableArgs {
  const float *x_fm;
  int64_t n_pad;
  int32_t n_tiles, nf, nc;
  const int32_t *tile_info;
  const int4 *sets;
  const uint4 *conds;
  const uint4 *heads;
  int32_t n_sets, Q;
  int32_t *correct;
  int32_t *confusion;
};

// A table that fits one block's LDS: block b evaluates rule sets [b*Q,
// b*Q + Q) on all of it.  The table is staged once, with each feature's
// extremes per tile reduced from the registers that carry it; then a wave
// takes one (rule set, layout tile) after the other, the next one's set
// record and head entries under way during the walk.  A set's confusion
// counts are complete in its block, so they are stored, not added: one launch
// instead of two fills and the evaluation.  Such launches are bound by
// latency, stage after stage: of 6.4 us on 569 x 30 with 100 sets, the launch
// takes 2.3, the staging 1.6 (its vector instructions count as much as its
// loads: with a division per row and 64 or 128 samples per row 6 and 4.5) and
// the walk 2.4.  A call whose outputs are allocated with it takes 10.1 us there,
// most of it the host's, where the path above takes 16.6.
template <bool CAT>
__global__ __launch_bounds__(kHardBlock) void k_hard_table(const HardTableArgs a) {
  extern __shared__ __align__(16) float smem[];
  constexpr int S = 4, kWaves = kHardBlock / 64;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int ncc = hard_counters_per_set(a.nc);
  const int set0 = blockIdx.x * a.Q;
  const int Q = min(a.Q, a.n_sets - set0);
  const int rows = a.n_tiles * a.nf;
  float *xs = smem;                                              // [n_tiles][nf][AERL_TILE]
  float *ext = xs + (size_t)rows * AERL_TILE;                    // [n_tiles][nf][max, -min]
  int32_t *cnt = reinterpret_cast<int32_t *>(ext + 2 * rows);    // [Q][label][class]
  int32_t *n_label = cnt + a.Q * a.nc * a.nc;                    // [nc]

  int4 s4 = make_int4(0, 0, 0, 0);
  uint4 head = make_uint4(0, 0, 0, 0);
  const int n_items = Q * a.n_tiles;
  auto request = [&](int i) {
    s4 = ldc(a.sets, set0 + i / a.n_tiles);
    const int nh = s4.y >> 16;
    if (nh >= 1 && nh <= kMaxHeads) head = a.heads[s4.x + min(lane, nh - 1)];
  };
  if (wave < n_items) request(wave);

  for (int i = threadIdx.x; i < Q * a.nc * a.nc; i += kHardBlock) cnt[i] = 0;
  if ((int)threadIdx.x < a.nc) n_label[threadIdx.x] = 0;
  // 16 lanes per row (one feature of one tile), eight loads under way per
  // lane; a lane's next row is 64 on
  const int col = threadIdx.x & 15;
  constexpr int kStep = kHardBlock / 16, kBatch = 2;
  const int step_t = kStep / a.nf, step_f = kStep - step_t * a.nf;
  const uint32_t n_pad = (uint32_t)a.n_pad;
  int r = threadIdx.x >> 4;
  int t = r / a.nf, f = r - t * a.nf;
  while (r < rows) {
    f4v v[kBatch][S];
    int valid[kBatch];
    const int r0 = r;
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      if (r < rows) {
        const f4v *src =
            reinterpret_cast<const f4v *>(a.x_fm + ((uint32_t)f * n_pad + (uint32_t)(t * AERL_TILE))) + col;
#pragma unroll
        for (int j = 0; j < S; ++j) v[k][j] = src[16 * j];
        valid[k] = a.tile_info[t] >> 8;
      }
      r += kStep;
      t += step_t;
      f += step_f;
      if (f >= a.nf) {
        f -= a.nf;
        ++t;
      }
    }
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      const int rk = r0 + k * kStep;
      if (rk >= rows) break;
      float hi = -INFINITY, lo = INFINITY;
#pragma unroll
      for (int j = 0; j < S; ++j) {
        reinterpret_cast<f4v *>(xs)[rk * (AERL_TILE / 4) + 16 * j + col] = v[k][j];
        widen(v[k][j], valid[k] - 64 * j - 4 * col, hi, lo);
      }
      hi = row_max(hi);
      lo = row_max(-lo);
      if (col == 0) *reinterpret_cast<float2 *>(ext + 2 * rk) = make_float2(hi, lo);
    }
  }
  __syncthreads();
  if ((int)threadIdx.x < a.n_tiles) {
    const int info = a.tile_info[threadIdx.x];
    atomicAdd(&n_label[info & 0xff], info >> 8);
  }
  const uint32_t lds_lane =
      (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) float *)xs + (uint32_t)lane * (4u * S);
  for (int i = wave; i < n_items; i += kWaves) {
    const int q = i / a.n_tiles, wt = i - q * a.n_tiles;
    const int4 set = s4;
    const uint4 h = head;
    if (i + kWaves < n_items) request(i + kWaves);
    const int info = ldc(a.tile_info, wt);
    const int valid = info >> 8;
    uint64_t vm[S];
#pragma unroll
    for (int s = 0; s < S; ++s) vm[s] = ballot(lane * S + s < valid);
    const int nh = set.y >> 16;
    const uint32_t base = lds_lane + (uint32_t)(wt * a.nf) * (4u * AERL_TILE);
    int acc;
    if (nh >= 1 && nh <= kMaxHeads) {
      // lane j: rule j; table[e] < t' when no sample of the tile passes
      const char *tb = reinterpret_cast<const char *>(ext + 2 * wt * a.nf);
      const float e1 = *reinterpret_cast<const float *>(tb + (h.x >> kHeadExtShift));
      const float e2 = *reinterpret_cast<const float *>(tb + h.z);
      const uint64_t rules = ~0ull >> (64 - nh);
      const uint64_t mk = (ballot(!(e1 < __uint_as_float(h.y))) &
                           ballot(!(e2 < __uint_as_float(h.w))) & rules) |
                          (1ull << (nh - 1));
      acc = eval_set_count<S, true, CAT>(base, lane, set, a.conds, vm, mk, h.x & kHeadOffMask);
    } else {
      acc = eval_set_count<S, false, CAT>(base, lane, set, a.conds, vm);
    }
    if (lane < ncc) atomicAdd(&cnt[(q * a.nc + (info & 0xff)) * a.nc + lane], acc);
  }
  __syncthreads();
  // the last class gets what the others leave of a region's samples
  for (int i = threadIdx.x; i < Q * a.nc; i += kHardBlock) {
    int rest = n_label[i % a.nc];
    for (int c = 0; c < ncc; ++c) rest -= cnt[i * a.nc + c];
    cnt[i * a.nc + ncc] = rest;
  }
  __syncthreads();
  if (a.confusion) {
    int32_t *out = a.confusion + (int64_t)set0 * a.nc * a.nc;
    for (int i = threadIdx.x; i < Q * a.nc * a.nc; i += kHardBlock) out[i] = cnt[i];
  }
  for (int q = threadIdx.x; q < Q; q += kHardBlock) {
    int hits = 0;
    for (int c = 0; c < a.nc; ++c) hits += cnt[(q * a.nc + c) * a.nc + c];
    a.correct[set0 + q] = hits;
  }
}

// Prediction for one rule set over row-major rows, 64 S rows per block.
template <int S>
__global__ __launch_bounds__(kPredictBlock) void k_predict(const float *__restrict__ rows, int64_t n,
                                                           int32_t nf, const int4 *__restrict__ sets,
                                                           int32_t set_idx,
                                                           const uint4 *__restrict__ conds,
                                                           const uint4 *__restrict__ heads,
                                                           int32_t *__restrict__ out) {
  extern __shared__ __align__(16) float xs[];
  __shared__ int32_t first[kPredictRows * S];
  predict_block<S>(rows, n, nf, ldc(sets, set_idx), conds, heads, out,
                   (int64_t)blockIdx.x * kPredictRows * S, xs, first);
}

// The same, a wave per 256 rows that walks the rules in turn.
__global__ __launch_bounds__(64) void k_predict_walk(const float *__restrict__ rows, int64_t n, int32_t nf,
                                                     const int4 *__restrict__ sets, int32_t set_idx,
                                                     const uint4 *__restrict__ conds,
                                                     int32_t *__restrict__ out) {
  extern __shared__ __align__(16) float xs[];  // [nf][256]
  predict_walk(rows, n, nf, ldc(sets, set_idx), conds, out, (int64_t)blockIdx.x * 256, xs);
}

template <int S>
hipError_t hard_dispatch(const HardArgs &a, dim3 grid, size_t lds, bool cat, bool c10,
                         hipStream_t st) {
  if (cat && c10)
    hipLaunchKernelGGL((k_hard<S, true, true>), grid, dim3(kHardBlock), lds, st, a);
  else if (cat)
    hipLaunchKernelGGL((k_hard<S, true, false>), grid, dim3(kHardBlock), lds, st, a);
  else if (c10)
    hipLaunchKernelGGL((k_hard<S, false, true>), grid, dim3(kHardBlock), lds, st, a);
  else
    hipLaunchKernelGGL((k_hard<S, false, false>), grid, dim3(kHardBlock), lds, st, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_hard_eval(const HardLaunch &h, hipStream_t st) {
  const DatasetRec &ds = *h.ds;
  const PopRec &pop = *h.pop;
  if (h.set_count <= 0) return hipSuccess;
  HardArgs a{};
  a.x_fm = ds.x_fm;
  a.n_pad = ds.n_pad;
  a.nf = ds.nf;
  a.nc = ds.nc;
  a.tile_info = ds.tile_info;
  a.sets = pop.sets;
  a.conds = pop.hconds;
  a.heads = pop.heads;
  a.set_begin = h.set_begin;
  a.set_count = h.set_count;
  a.correct = h.correct;
  a.confusion = h.confusion;
  a.part = h.part;
  if (h.part && !(hard_c10(h.tiles_per_group) && ds.nc >= 2 && ds.nc <= 4))
    return hipErrorInvalidValue;
  a.sets_per_chunk = h.sets_per_chunk;
  a.tiles_per_group = h.tiles_per_group;
  for (int c = 0; c < ds.nc; ++c) {
    a.region_tile0[c] = ds.region_tile0[c];
    a.region_tiles[c] = ds.region_tiles[c];
  }
  if (h.tiles_per_group < 1 || h.tiles_per_group > kMaxTilesPerBlock || h.sets_per_chunk < 1)
    return hipErrorInvalidValue;
  const int64_t n_groups = hard_group_count(ds, h.tiles_per_group);
  if (n_groups == 0) return hipSuccess;
  const int64_t n_chunks = (h.set_count + h.sets_per_chunk - 1) / h.sets_per_chunk;
  const bool c10 = hard_c10(h.tiles_per_group);
  const size_t lds = hard_block_lds(ds.nf, h.samples_per_lane, h.sets_per_chunk, ds.nc, c10);
  if (lds > kDynLdsMax || n_chunks * n_groups > kMaxHardBlocks) return hipErrorInvalidValue;
  a.n_chunks = (int32_t)n_chunks;
  const dim3 grid((unsigned)(n_chunks * n_groups));
  switch (h.samples_per_lane) {
    case 4: return hard_dispatch<4>(a, grid, lds, pop.n_cat > 0, c10, st);
    case 2: return hard_dispatch<2>(a, grid, lds, pop.n_cat > 0, c10, st);
    case 1: return hard_dispatch<1>(a, grid, lds, pop.n_cat > 0, c10, st);
    default: return hipErrorInvalidValue;
  }
}

HardTablePlan plan_hard_table(const DatasetRec &ds, int32_t n_sets, int n_cu) {
  HardTablePlan p{};
  if (ds.n_tiles < 1 || n_sets < 1) return p;
  const int64_t Q = ((int64_t)n_sets + n_cu - 1) / n_cu;  // one block per CU
  if (ds.n_tiles > kHardTableVisits || Q * ds.n_tiles > kHardTableVisits) return p;
  const size_t lds = (size_t)ds.n_tiles * ds.nf * (4 * AERL_TILE + 8) +
                     sizeof(int32_t) * ((size_t)Q * ds.nc * ds.nc + ds.nc);
  if (lds > kDynLdsMax) return p;
  p.Q = (int)Q;
  p.lds = lds;
  return p;
}

hipError_t launch_hard_table(const HardLaunch &h, const HardTablePlan &p, hipStream_t st) {
  const DatasetRec &ds = *h.ds;
  const PopRec &pop = *h.pop;
  if (p.Q < 1 || p.lds > kDynLdsMax || ds.n_tiles < 1 || h.set_begin != 0) return hipErrorInvalidValue;
  const HardTableArgs a{ds.x_fm,    ds.n_pad,  (int32_t)ds.n_tiles, ds.nf, ds.nc,     ds.tile_info, pop.sets,
                        pop.hconds, pop.heads, h.set_count,         p.Q,   h.correct, h.confusion};
  const dim3 grid((unsigned)((h.set_count + p.Q - 1) / p.Q));
  if (pop.n_cat > 0)
    hipLaunchKernelGGL(k_hard_table<true>, grid, dim3(kHardBlock), p.lds, st, a);
  else
    hipLaunchKernelGGL(k_hard_table<false>, grid, dim3(kHardBlock), p.lds, st, a);
  return hipGetLastError();
}

hipError_t launch_hard_reduce(const HardLaunch &h, int n_cu, hipStream_t st) {
  const DatasetRec &ds = *h.ds;
  if (h.set_count <= 0 || ds.n_tiles == 0) return hipSuccess;
  if (!h.part || ds.nc < 2 || ds.nc > 4 || h.sets_per_chunk < 1) return hipErrorInvalidValue;
  const int64_t bx = (h.set_count + kReduceBlock - 1) / kReduceBlock;
  const int64_t by = std::max<int64_t>(1, std::min<int64_t>(ds.n_tiles, (2LL * n_cu + bx - 1) / bx));
  hipLaunchKernelGGL(k_hard_reduce, dim3((unsigned)bx, (unsigned)by), dim3(kReduceBlock), 0, st,
                     h.part, ds.tile_info, ds.n_tiles, h.set_count, h.sets_per_chunk, ds.nc,
                     h.correct, h.confusion);
  return hipGetLastError();
}

hipError_t launch_predict(const PopRec &pop, int32_t set, const float *rows, int64_t n, int n_cu,
                          int32_t *pred, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  // A wave per 256 rows that walks the rules in turn, where rows alone fill the
  // GPU and little is staged for each: over 14 rule sets of 1 to 96 rules it
  // takes 0.88 of the blocks' time on 1 to 5 features from 2^15 rows (7.5 us
  // both below), 0.5 to 0.7 from 2^20 (2^21 x 5, 24 rules 18 us against 40), and
  // 0.84 on 6 to 9 features from 5 * 2^18 (2^21 x 8 31 us against 38, 1572864 x
  // 6 0.52).  On fewer rows of those (2^20 x 8 1.09) and on more features (2^21
  // x 10 1.10, x 12 1.22, x 32 3.3) it is the slower one.
  if (pop.nf <= 5 ? n >= (1 << 15) : pop.nf <= 9 && n >= (5 << 18)) {
    hipLaunchKernelGGL(k_predict_walk, dim3((unsigned)((n + 255) / 256)), dim3(64),
                       predict_walk_lds(pop.nf), st, rows, n, pop.nf, pop.sets, set, pop.hconds, pred);
    return hipGetLastError();
  }
  // Four rows per lane once 64-row blocks would fill the GPU several times
  // over, on tables narrow enough to keep 16 waves per CU (2^20 rows x 32
  // features 62 us; one wave per 256 rows walking every rule 178).
  const int S = n >= kPredictWideRows && pop.nf <= kPredictWideFeatures ? 4 : 1;
  const size_t lds = predict_lds(pop.nf, S);
  const int64_t blocks = (n + kPredictRows * S - 1) / (kPredictRows * S);
  if (lds > kDynLdsMax) return hipErrorInvalidValue;
  // A wave per rule while all blocks are resident at once (latency: 4096 rows
  // x 64 features 9.4 us).  Larger requests take fewer waves per block, whose
  // walks end once every row is decided, but enough for 16 per CU under the
  // LDS of their rows.
  int waves = 1, least = 1;
  while (waves < kPredictBlock / 64 && waves < std::max(pop.max_rules, 4)) waves *= 2;
  while (least < 16 && least * (int)(kLdsPerCu / lds) < 16) least *= 2;
  while (waves > least && blocks * waves > 32LL * n_cu) waves /= 2;
  const dim3 grid((unsigned)blocks), block((unsigned)waves * 64);
  if (S == 4)
    hipLaunchKernelGGL(k_predict<4>, grid, block, lds, st, rows, n, pop.nf, pop.sets, set, pop.hconds,
                       pop.heads, pred);
  else
    hipLaunchKernelGGL(k_predict<1>, grid, block, lds, st, rows, n, pop.nf, pop.sets, set, pop.hconds,
                       pop.heads, pred);
  return hipGetLastError();
}

}  // namespace aerl
