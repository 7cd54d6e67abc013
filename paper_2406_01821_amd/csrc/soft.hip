// Soft (sigmoid-relaxed) forward pass and its adjoint.
//
// Section 3: a differentiable activation (a sigmoid) replaces the step so that
// rule coefficients and thresholds can be tuned by back-propagation.  The
// relaxation evaluated here (one sample, label y, rules k = 0..R-1):
//   z_j  = s_j * (coef_j * x[f_j] - rhs_j) / tau[f_j],  rhs = theta or coef2*x[g]
//   a_k  = sum_j log sigmoid(z_j)             (log of the rule's soft truth r_k)
//   b_k  = log(1 - r_k)
//   l_k  = a_k + sum_{m<k} b_m                (log P(rule k fires first))
//   log P_y = LSE({l_k : class_k = y} u {sum_m b_m if default = y})
//   L = min(-log P_y, 100),  loss = mean over samples.
// Everything is carried in log space in fp32 with accurate log1p / expm1 /
// log1mexp built from the hardware exp2/log2 (both within ~1 ulp, also near 1).
//
// Adjoint (derivation in the oracle): with V_k = P(class y | rules 0..k did not
// fire) = exp(U_k), U_{R-1} = [default = y] ? 0 : -inf,
// U_{k-1} = LSE([class_k = y] a_k, b_k + U_k):
//   dL/da_k = exp(l_k + U_k - log P_y)                      if class_k != y
//           = -exp(l_k - log P_y) * (1 - V_k)               if class_k == y
//   dL/dz_j = dL/da_k * sigmoid(-z_j),  formed as one exponent (bounded by 1).
// The backward kernel re-evaluates every condition: a forward sweep keeps only
// a_k and the survival prefix per rule and sample (in LDS), then a reverse
// sweep rebuilds U_k and recomputes each sigmoid to form its gradient.
//
// Work decomposition matches the hard path: block (chunk of rule sets, group
// of label-uniform tiles).  Per-(set, tile) wave sums go into LDS with one
// writer per entry; per-block partials go to the caller's workspace and a
// second kernel reduces them over groups in a fixed order, so every result is
// bit-identical from run to run.
#include "eval_core.h"
#include "internal.h"
#include "soft_core.h"
#include "soft_plan.h"

namespace aerl {

namespace {

struct SoftArgs {
  const float *x_fm;
  int64_t n_pad;
  int32_t nf, nc;
  const int32_t *tile_info;
  const float *inv_tau;
  const int4 *sets;   // hard set records (default class in .z)
  const int4 *ssets;  // {first rule, #rules, first condition, #conditions}
  const int4 *rules;  // {first condition, #conditions, class, 0}
  const uint32_t *sconds;
  const float *coef, *coef2, *theta;
  // per condition {sconds, coef, theta or coef2, +-log2(e)/tau_f}, gathered
  // once per launch so that a condition is one scalar load
  const uint4 *crec;
  int32_t n_sets;
  int32_t sets_per_chunk, tiles_per_group, n_groups;
  int32_t max_rules, max_set_conds;
  double *part_loss;  // [n_groups][n_sets]
  float *part_grad;   // [n_groups][n_conds][2]
  int32_t n_conds;
  int32_t classify;  // adjoints: tiles classify the conditions (classify below)
  int32_t region_tile0[AERL_MAX_CLASSES];
  int32_t region_tiles[AERL_MAX_CLASSES];
};

// Class region and tile range of block group g (uniform).
__device__ __forceinline__ void group_range(const SoftArgs &a, int g, int &label, int &lo, int &hi) {
  label = 0; lo = 0; hi = 0;
  for (int c = 0; c < a.nc; ++c) {
    const int ng = (a.region_tiles[c] + a.tiles_per_group - 1) / a.tiles_per_group;
    if (g < ng) {
      label = c;
      lo = a.region_tile0[c] + g * a.tiles_per_group;
      hi = min(lo + a.tiles_per_group, a.region_tile0[c] + a.region_tiles[c]);
      return;
    }
    g -= ng;
  }
}

// z2 = z*log2(e) of condition j for S values of x[f], with x[f] and the
// right-hand factor xg: x[g] for feature conditions, 1 for threshold ones (so
// dz*xg is their theta term).  Branch-free on the kind (the row of g is read
// for threshold conditions too; g is 0 there), which keeps every array in
// registers.
template <int S>
__device__ __forceinline__ void cond_z(const SoftArgs &a, const float *xs, int lane, int j,
                                       float (&z)[S], float (&xf)[S], float (&xg)[S], bool &ff) {
  const uint4 r = ldc(a.crec, j);
  const uint32_t sc = r.x;
  const uint32_t f = sc & 0xfffu, g = (sc >> 12) & 0xfffu;
  ff = (sc & kSoftFF) != 0;
  const float c = __uint_as_float(r.y), rv = __uint_as_float(r.z), sinv = __uint_as_float(r.w);
  load_row<S>(xs, f * 1024u, lane, xf);
  load_row<S>(xs, g * 1024u, lane, xg);
  if (sc & kSoftCat) {
#pragma unroll
    for (int s = 0; s < S; ++s) {
      z[s] = cat_z(xf[s], r.y, r.z);
      xg[s] = 1.0f;
    }
    return;
  }
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const float rhs = ff ? rv * xg[s] : rv;
    xg[s] = ff ? xg[s] : 1.0f;
    z[s] = fmaf(c, xf[s], -rhs) * sinv;
  }
}

// Threshold-only populations: z2 and x[f] (xg is 1).
template <int S>
__device__ __forceinline__ void cond_z_t(const SoftArgs &a, const float *xs, int lane, int j,
                                         float (&z)[S], float (&xf)[S], float (&xg)[S]) {
  const uint4 r = ldc(a.crec, j);
  const uint32_t f = r.x & 0xfffu;
  const float c = __uint_as_float(r.y), th = __uint_as_float(r.z), sinv = __uint_as_float(r.w);
  load_row<S>(xs, f * 1024u, lane, xf);
#pragma unroll
  for (int s = 0; s < S; ++s) {
    z[s] = fmaf(c, xf[s], -th) * sinv;
    xg[s] = 1.0f;
  }
}

// z2 only (forward pass): nothing but z leaves the branch on the kind.
template <int S>
__device__ __forceinline__ void cond_z_only(const SoftArgs &a, const float *xs, int lane, int j,
                                            float (&z)[S]) {
  const uint4 r = ldc(a.crec, j);
  const uint32_t sc = r.x;
  const uint32_t f = sc & 0xfffu, g = (sc >> 12) & 0xfffu;
  const float c = __uint_as_float(r.y), rv = __uint_as_float(r.z), sinv = __uint_as_float(r.w);
  float xf[S];
  load_row<S>(xs, f * 1024u, lane, xf);
  if (sc & kSoftFF) {
    float xg[S];
    load_row<S>(xs, g * 1024u, lane, xg);
#pragma unroll
    for (int s = 0; s < S; ++s) z[s] = fmaf(c, xf[s], -(rv * xg[s])) * sinv;
  } else if (sc & kSoftCat) {
#pragma unroll
    for (int s = 0; s < S; ++s) z[s] = cat_z(xf[s], r.y, r.z);
  } else {
#pragma unroll
    for (int s = 0; s < S; ++s) z[s] = fmaf(c, xf[s], -rv) * sinv;
  }
}

// z2 of the condition of record r, x[f] read already.  TONLY: threshold
// conditions only.
template <int S, bool TONLY>
__device__ __forceinline__ void record_z(uint4 r, const float *xs, int lane, const float (&xf)[S],
                                         float (&z)[S]) {
  const float c = __uint_as_float(r.y), rv = __uint_as_float(r.z), sinv = __uint_as_float(r.w);
  if (!TONLY && (r.x & kSoftFF)) {
    float xg[S];
    load_row<S>(xs, ((r.x >> 12) & 0xfffu) * 1024u, lane, xg);
#pragma unroll
    for (int s = 0; s < S; ++s) z[s] = fmaf(c, xf[s], -(rv * xg[s])) * sinv;
  } else if (!TONLY && (r.x & kSoftCat)) {
#pragma unroll
    for (int s = 0; s < S; ++s) z[s] = cat_z(xf[s], r.y, r.z);
  } else {
#pragma unroll
    for (int s = 0; s < S; ++s) z[s] = fmaf(c, xf[s], -rv) * sinv;
  }
}

// z2 of the conditions of N records recs[i[]], i < 64 (forward pass): the
// records and x[f] rows are requested together, so that their latencies
// overlap; the same arithmetic as cond_z_only.  The byte offsets from recs
// take 32 bits, recs itself the 64 bits that a population of 2^28 conditions
// and more needs.
template <int S, bool TONLY, int N>
__device__ __forceinline__ void cond_zn(const uint4 *recs, const float *xs, int lane,
                                        const int (&i)[N], float (&z)[N][S]) {
  uint4 r[N];
  float xf[N][S];
#pragma unroll
  for (int k = 0; k < N; ++k) r[k] = ldc_at(recs, (uint32_t)i[k] * 16u);
#pragma unroll
  for (int k = 0; k < N; ++k) load_row<S>(xs, (r[k].x & 0xfffu) * 1024u, lane, xf[k]);
#pragma unroll
  for (int k = 0; k < N; ++k) record_z<S, TONLY>(r[k], xs, lane, xf[k], z[k]);
}

// z2 of four consecutive conditions j .. j+3: their records in one 64-byte
// scalar load; the same arithmetic as cond_z_only.
template <int S, bool TONLY>
__device__ __forceinline__ void cond_z4(const SoftArgs &a, const float *xs, int lane, int j,
                                        float (&z)[4][S]) {
  typedef uint32_t v16u __attribute__((ext_vector_type(16)));
  typedef const __attribute__((address_space(4))) v16u *cptr;
  const v16u r = *(cptr)(a.crec + j);
  float xf[4][S];
#pragma unroll
  for (int k = 0; k < 4; ++k) load_row<S>(xs, (r[4 * k] & 0xfffu) * 1024u, lane, xf[k]);
#pragma unroll
  for (int k = 0; k < 4; ++k)
    record_z<S, TONLY>(make_uint4(r[4 * k], r[4 * k + 1], r[4 * k + 2], r[4 * k + 3]), xs, lane, xf[k], z[k]);
}

// Adds all of a rule's conditions to ra, four at a time (the sweep of tables
// that do not classify).
template <int S, class Acc, bool TONLY>
__device__ __forceinline__ void add_all(const SoftArgs &a, const float *xs, int lane, int4 r,
                                        Acc (&ra)[S]) {
  int j = r.x;
  const int je = r.x + r.y;
  for (; j + 4 <= je; j += 4) {
    float z[4][S];
    cond_z4<S, TONLY>(a, xs, lane, j, z);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
#pragma unroll
      for (int s = 0; s < S; ++s) (void)ra[s].add(z[c][s]);
    }
  }
  for (; j < je; ++j) {
    float z[S];
    cond_z_only<S>(a, xs, lane, j, z);
#pragma unroll
    for (int s = 0; s < S; ++s) (void)ra[s].add(z[s]);
  }
}

__device__ __forceinline__ int pop_bit(uint64_t &m) {
  const int i = __builtin_ctzll(m);
  m &= m - 1;
  return i;
}

// Adds the conditions of recs[set bits of act], in order, to ra.
template <int S, class Acc, bool TONLY, int N>
__device__ __forceinline__ void add_n(const uint4 *recs, const float *xs, int lane, uint64_t &act,
                                      Acc (&ra)[S]) {
  int i[N];
#pragma unroll
  for (int k = 0; k < N; ++k) i[k] = pop_bit(act);
  float z[N][S];
  cond_zn<S, TONLY, N>(recs, xs, lane, i, z);
#pragma unroll
  for (int k = 0; k < N; ++k) {
#pragma unroll
    for (int s = 0; s < S; ++s) (void)ra[s].add(z[k][s]);
  }
}
template <int S, class Acc, bool TONLY>
__device__ __forceinline__ void add_conds(const uint4 *recs, const float *xs, int lane,
                                          uint64_t act, Acc (&ra)[S]) {
  int n = __builtin_popcountll(act);
  for (; n >= 4; n -= 4) add_n<S, Acc, TONLY, 4>(recs, xs, lane, act, ra);
  if (n & 2) add_n<S, Acc, TONLY, 2>(recs, xs, lane, act, ra);
  if (n & 1) add_n<S, Acc, TONLY, 1>(recs, xs, lane, act, ra);
}

// Largest and smallest value of every feature over a staged tile's `valid`
// real samples, into ext[f]: 16 threads per feature.  Ends with a barrier.
template <int TS>
__device__ __forceinline__ void tile_extremes(const float *xs, int nf, int valid, float2 *ext) {
  const int part = threadIdx.x & 15;
  for (int f0 = 0; f0 < nf; f0 += (int)blockDim.x >> 4) {
    const int f = f0 + ((int)threadIdx.x >> 4);
    float hi = kNegInf, lo = -kNegInf;
    if (f < nf) {
      for (int i = part; i < valid; i += 16) {
        const float v = xs[f * TS + i];
        hi = fmaxf(hi, v);
        lo = fminf(lo, v);
      }
    }
    for (int d = 1; d < 16; d <<= 1) {
      hi = fmaxf(hi, __shfl_xor(hi, d));
      lo = fminf(lo, __shfl_xor(lo, d));
    }
    if (f < nf && part == 0) ext[f] = make_float2(hi, lo);
  }
  __syncthreads();
}

// What a staged tile decides about up to 64 conditions of a rule set before
// any sample is looked at, lane j taking condition base + j: `dead`, those
// with z2 < -t_dead for every sample of the tile, and `sat`, those with z2 >
// t_sat for every sample.  Rounding is monotone, so z2 over the tile lies
// between its values at the corners of the tile's feature extremes, formed
// with the same operations (the parameters are those of set_regular, which
// give no NaN).  Categorical conditions decide nothing.
//
// The thresholds are where the exponentials give exactly 0 (v_exp_f32
// flushes below 2^-126), so what is left out would have added nothing:
//  - a rule with a condition below kDeadLoss has log2(1 - r) = 0 and a route
//    below 2^-180 to its class, which no loss under the 100-nat cap (144.3
//    bits) can show; below kDeadProb its r is 0 as computed;
//  - adding a condition above Acc::kNoop changes nothing;
//  - in the first-firing adjoint a condition's term is 2^(pre - max(z2, 0))
//    / (1 + u) with pre <= 144.3 (samples past the cap have no gradient) and,
//    for a rule with a condition below -kDeadGrad, pre < 144.3 - kDeadGrad:
//    0 on either side; under the softmax head pre = log2 r <= 0.
// Thresholds drawn over a column's whole range lie, for most tiles, many tau
// from all of its samples: on the 262,144 x 32 table with 1024 rule sets of
// 16 rules x 4 conditions a forward pass is left with 42% of the rules and
// 32% of the conditions (6.47 -> 2.8 ms), the adjoint with 62% and 54%
// (17.2 -> 8.2 ms), the softmax head with 32% and 23%; results bit for bit
// the same.  Both kernels stay VALU-bound.
constexpr float kDeadLoss = 180.0f;
constexpr float kDeadProb = 128.0f;
constexpr float kDeadGrad = 274.0f;
constexpr float kSatProb = 128.0f;
constexpr float kExp2Zero = -127.0f;  // v_exp_f32 gives 0 below
struct Window {
  int base, end;  // conditions [base, end) are classified
  uint64_t dead, sat;
};
// Without classification: every condition decided neither way.
__device__ __forceinline__ Window first_window(bool on) { return {0, on ? 0 : INT32_MAX, 0, 0}; }

// Whether every parameter of a rule set's conditions (ss, its soft record) is
// one that z2 is not NaN for (record_odd).  Parameters arrive unchecked (an
// optimizer run that diverges), and what NaN reaches has to show: a set that
// fails this is swept in full, nothing of it left out as zero.  One scalar
// load of the mark on the set's first record; looking over the records here
// instead made the adjoints 1% longer on average and up to 18%.
__device__ __forceinline__ bool set_regular(const SoftArgs &a, int4 ss) {
  return !(ldc(a.crec, max(min(ss.z, a.n_conds - 1), 0)).x & kRecOdd);
}
template <bool TONLY>
__device__ __forceinline__ void classify(const SoftArgs &a, const float2 *ext, int lane, int base,
                                         int end, float t_dead, float t_sat, Window &w) {
  const int j = min(base + lane, end - 1);
  const uint4 r = a.crec[j];
  const float c = __uint_as_float(r.y), rv = __uint_as_float(r.z), sinv = __uint_as_float(r.w);
  const float2 ef = ext[r.x & 0xfffu];
  bool dead, sat;
  if (TONLY) {
    const float z0 = fmaf(c, ef.x, -rv) * sinv, z1 = fmaf(c, ef.y, -rv) * sinv;
    dead = z0 < -t_dead && z1 < -t_dead;
    sat = z0 > t_sat && z1 > t_sat;
  } else {
    float2 eg = ext[(r.x >> 12) & 0xfffu];
    if (!(r.x & kSoftFF)) eg = make_float2(1.0f, 1.0f);
    const float r0 = rv * eg.x, r1 = rv * eg.y;
    const float z0 = fmaf(c, ef.x, -r0) * sinv, z1 = fmaf(c, ef.y, -r0) * sinv;
    const float z2 = fmaf(c, ef.x, -r1) * sinv, z3 = fmaf(c, ef.y, -r1) * sinv;
    const bool ok = !(r.x & kSoftCat);
    dead = ok && z0 < -t_dead && z1 < -t_dead && z2 < -t_dead && z3 < -t_dead;
    sat = ok && z0 > t_sat && z1 > t_sat && z2 > t_sat && z3 > t_sat;
  }
  const bool in = base + lane < end;
  w.base = base;
  w.end = min(base + 64, end);
  w.dead = ballot(dead && in);
  w.sat = ballot(sat && in);
}

// First n bits.
__device__ __forceinline__ uint64_t low_bits(int n) { return n > 0 ? ~0ull >> (64 - n) : 0ull; }

// Forward sweep's view of the rule of record r: false when the tile decides
// that it is dead; else `act` holds its conditions that add something (bit
// i: condition r.x + i, the first 64 of a longer rule, whose conditions are
// all taken).  Classifies the next 64 conditions of the set, from this rule
// on, when they leave the window.
template <bool TONLY>
__device__ __forceinline__ bool rule_live(const SoftArgs &a, const float2 *ext, int lane, int4 r,
                                          int set_end, float t_dead, float t_sat, Window &w,
                                          uint64_t &act) {
  act = low_bits(min(r.y, 64));
  if (r.y == 0 || r.y > 64) return true;
  if (r.x < w.base || r.x + r.y > w.end)
    classify<TONLY>(a, ext, lane, r.x, set_end, t_dead, t_sat, w);
  const int sh = (r.x - w.base) & 63;
  const bool dead = ((w.dead >> sh) & act) != 0;
  act &= ~(w.sat >> sh);
  return !dead;
}
// Reverse sweep: the same, classifying the 64 conditions up to this rule's
// last one.
template <bool TONLY>
__device__ __forceinline__ bool rule_live_back(const SoftArgs &a, const float2 *ext, int lane,
                                               int4 r, int set_begin, int set_end, float t_dead,
                                               float t_sat, Window &w, uint64_t &act) {
  if (r.y > 0 && r.y <= 64 && (r.x < w.base || r.x + r.y > w.end))
    classify<TONLY>(a, ext, lane, max(set_begin, r.x + r.y - 64), set_end, t_dead, t_sat, w);
  return rule_live<TONLY>(a, ext, lane, r, set_end, t_dead, t_sat, w, act);
}

// Adds a live rule's conditions to ra: those of act, then the rest of a rule
// of more than 64.
template <int S, class Acc, bool TONLY>
__device__ __forceinline__ void add_rule(const SoftArgs &a, const float *xs, int lane, int4 r,
                                         uint64_t act, Acc (&ra)[S]) {
  for (int b = 0;;) {
    add_conds<S, Acc, TONLY>(a.crec + (r.x + b), xs, lane, act, ra);
    b += 64;
    if (b >= r.y) break;
    act = low_bits(min(r.y - b, 64));
  }
}

// Gathers the per-condition records read by the kernels above, a rule set per
// block, and marks the first one of a set with a record_odd.
constexpr int kPrepBlock = 256;
__global__ __launch_bounds__(kPrepBlock) void k_soft_prep(
    const int4 *__restrict__ ssets, const uint32_t *__restrict__ sconds,
    const float *__restrict__ inv_tau, const float *__restrict__ coef, const float *__restrict__ coef2,
    const float *__restrict__ theta, const uint2 *__restrict__ cmask, uint4 *__restrict__ crec) {
  const int4 ss = ldc(ssets, blockIdx.x);
  int odd = 0;
  for (int i = threadIdx.x; i < ss.w; i += blockDim.x) {
    const int64_t j = (int64_t)ss.z + i;
    const uint4 r = cond_record(sconds[j], inv_tau, coef, coef2, theta, cmask, j);
    crec[j] = r;
    odd |= record_odd(r);
  }
  if (__syncthreads_or(odd) && threadIdx.x == 0) crec[ss.z].x |= kRecOdd;
}

// Eight waves per SIMD need at most 80 SGPRs per wave (measured on gfx950):
// the classifying forward sweeps would take 106 and leave seven (forward and
// adjoint on 262,144 x 32, 1024 rule sets: 11.97 ms, capped 11.70 ms).
#define AERL_SOFT_SGPR_CAP __attribute__((amdgpu_num_sgpr(80)))

// ------------------------------------------------------------------ forward
// Bodies shared by the kernels that classify a tile's conditions (CLS) and
// those that take all of them (forward_classifies chooses).  The classifying
// ones are held to eight waves per SIMD, which their larger state would
// leave: 64 VGPRs and 80 SGPRs (rules of more than 60 conditions would take
// 88-109 VGPRs and four waves, the softmax head of 16 classes 91 and five).
// The others fit by themselves and spill nothing.
template <int S, class Acc, bool TONLY, bool CLS>
__device__ __forceinline__ void soft_fwd(const SoftArgs a) {
  constexpr int TS = 64 * S, WPT = AERL_TILE / TS;
  extern __shared__ __align__(16) float smem[];
  float *xs = smem;
  float2 *ext = reinterpret_cast<float2 *>(smem + (size_t)a.nf * TS);  // [nf] with CLS
  double *acc = reinterpret_cast<double *>(ext + (CLS ? a.nf : 0));    // [Q]
  __shared__ int32_t next_q;
  const int lane = threadIdx.x & 63;
  int label, tile_lo, tile_hi;
  group_range(a, blockIdx.y, label, tile_lo, tile_hi);
  const int q0 = blockIdx.x * a.sets_per_chunk;
  const int Q = min(a.sets_per_chunk, a.n_sets - q0);
  for (int i = threadIdx.x; i < Q; i += blockDim.x) acc[i] = 0.0;
  const int n4 = a.nf * (TS / 4);
  const float4 *src = reinterpret_cast<const float4 *>(a.x_fm);
  float4 *dst = reinterpret_cast<float4 *>(xs);
  const int64_t row4 = a.n_pad / 4;
  for (int64_t wt = (int64_t)tile_lo * WPT; wt < (int64_t)tile_hi * WPT; ++wt) {
    __syncthreads();
    const int64_t base4 = wt * (TS / 4);
    for (int i = threadIdx.x; i < n4; i += blockDim.x) {
      const int f = i / (TS / 4), k = i % (TS / 4);
      dst[i] = src[(int64_t)f * row4 + base4 + k];
    }
    if (threadIdx.x == 0) next_q = 0;
    __syncthreads();
    const int info = ldc(a.tile_info, wt / WPT);
    const int valid = min(max((info >> 8) - (int)(wt % WPT) * TS, 0), TS);
    if (S < 4 && valid == 0) continue;  // an empty wave tile (S < 4 at a region's end)
    if constexpr (CLS) tile_extremes<TS>(xs, a.nf, valid, ext);
    bool live[S];
#pragma unroll
    for (int s = 0; s < S; ++s) live[s] = lane * S + s < valid;
    for (;;) {
      const int q = next_item(&next_q);
      if (q >= Q) break;
      const int4 ss = ldc(a.ssets, q0 + q);
      const int dflt = ldc(a.sets, q0 + q).z;
      const int set_end = ss.z + ss.w;
      Window win;
      if constexpr (CLS) win = first_window(set_regular(a, ss));
      float logpy[S], surv[S];
#pragma unroll
      for (int s = 0; s < S; ++s) { logpy[s] = kNegInf; surv[s] = 0.0f; }
      // each rule's record is requested one rule ahead (the last one twice)
      int4 r_next = ldc(a.rules, ss.x);
      for (int k = 0; k < ss.y; ++k) {
        const int4 r = r_next;
        r_next = ldc(a.rules, ss.x + min(k + 1, ss.y - 1));
        Acc ra[S];
        if constexpr (CLS) {
          uint64_t act;
          if (!rule_live<TONLY>(a, ext, lane, r, set_end, kDeadLoss, Acc::kNoop, win, act)) continue;
          add_rule<S, Acc, TONLY>(a, xs, lane, r, act, ra);
        } else {
          add_all<S, Acc, TONLY>(a, xs, lane, r, ra);
        }
        const bool hit = r.z == label;
#pragma unroll
        for (int s = 0; s < S; ++s) {
          float a2, b2;
          acc_finish(ra[s], a2, b2);
          if (hit) logpy[s] = lse(logpy[s], a2 + surv[s]);
          surv[s] += b2;
        }
      }
      float part = 0.0f;
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const float lp = dflt == label ? lse(logpy[s], surv[s]) : logpy[s];
        part += live[s] ? sample_loss(lp) : 0.0f;
      }
      part = wave_sum(part);
      if (lane == 0) acc[q] += (double)part;
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < Q; i += blockDim.x)
    a.part_loss[(int64_t)blockIdx.y * a.n_sets + q0 + i] = acc[i];
}

template <int S, class Acc, bool TONLY>
__global__ __launch_bounds__(kSoftBlock, 8) AERL_SOFT_SGPR_CAP void k_soft_fwd_cls(const SoftArgs a) {
  soft_fwd<S, Acc, TONLY, true>(a);
}
template <int S, class Acc, bool TONLY>
__global__ __launch_bounds__(kSoftBlock) void k_soft_fwd(const SoftArgs a) {
  soft_fwd<S, Acc, TONLY, false>(a);
}

// Mean loss per rule set from the per-group partial sums: block b takes
// sets 64b .. 64b+63 (lane: set, so a wave reads 512 contiguous bytes per
// group), wave w the groups w, w+16, ...; the 16 wave sums are then added
// in wave order (a fixed order: the result does not depend on timing).
constexpr int kFwdFinalWaves = 16;
__global__ __launch_bounds__(kFwdFinalWaves * 64) void k_soft_fwd_final(
    const double *__restrict__ part, int32_t n_groups, int32_t n_sets, int64_t n,
    float *__restrict__ loss) {
  __shared__ double acc[kFwdFinalWaves][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int p = blockIdx.x * 64 + lane;
  double s = 0.0;
  if (p < n_sets)
    for (int g = w; g < n_groups; g += kFwdFinalWaves) s += part[(int64_t)g * n_sets + p];
  acc[w][lane] = s;
  __syncthreads();
  if (w == 0 && p < n_sets) {
    double t = 0.0;
    for (int k = 0; k < kFwdFinalWaves; ++k) t += acc[k][lane];
    loss[p] = n > 0 ? (float)(t / (double)n) : 0.0f;
  }
}

// ----------------------------------------------------------------- backward
__global__ __launch_bounds__(kBwdWaves * 64) void k_soft_bwd(const SoftArgs a) {
  constexpr int TS = 64, WPT = AERL_TILE / TS;
  extern __shared__ __align__(16) float smem[];
  float *xs = smem;                                     // [nf][64]
  float *acc = xs + (size_t)a.nf * TS;                  // [Q][max_set_conds][2]
  float *store = acc + (size_t)a.sets_per_chunk * a.max_set_conds * 2;  // [wave][R][2][64]
  __shared__ int32_t next_q;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float *my = store + (size_t)wave * a.max_rules * 128;
  int label, tile_lo, tile_hi;
  group_range(a, blockIdx.y, label, tile_lo, tile_hi);
  const int q0 = blockIdx.x * a.sets_per_chunk;
  const int Q = min(a.sets_per_chunk, a.n_sets - q0);
  for (int i = threadIdx.x; i < Q * a.max_set_conds * 2; i += blockDim.x) acc[i] = 0.0f;
  const int n4 = a.nf * (TS / 4);
  const float4 *src = reinterpret_cast<const float4 *>(a.x_fm);
  float4 *dst = reinterpret_cast<float4 *>(xs);
  const int64_t row4 = a.n_pad / 4;
  for (int64_t wt = (int64_t)tile_lo * WPT; wt < (int64_t)tile_hi * WPT; ++wt) {
    __syncthreads();
    const int64_t base4 = wt * (TS / 4);
    for (int i = threadIdx.x; i < n4; i += blockDim.x) {
      const int f = i / (TS / 4), k = i % (TS / 4);
      dst[i] = src[(int64_t)f * row4 + base4 + k];
    }
    if (threadIdx.x == 0) next_q = 0;
    __syncthreads();
    const int info = ldc(a.tile_info, wt / WPT);
    const int valid = min(max((info >> 8) - (int)(wt % WPT) * TS, 0), TS);
    const bool live = lane < valid;
    for (;;) {
      const int q = next_item(&next_q);
      if (q >= Q) break;
      const int4 ss = ldc(a.ssets, q0 + q);
      const int dflt = ldc(a.sets, q0 + q).z;
      // forward sweep: keep a_k and the survival prefix before rule k
      float logpy = kNegInf, surv = 0.0f;
      for (int k = 0; k < ss.y; ++k) {
        const int4 r = ldc(a.rules, ss.x + k);
        RuleAcc ra;
        for (int j = r.x; j < r.x + r.y; ++j) {
          float z[1];
          cond_z_only<1>(a, xs, lane, j, z);
          ra.add(z[0]);
        }
        my[k * 128 + lane] = ra.a;
        my[k * 128 + 64 + lane] = surv;
        if (r.z == label) logpy = lse(logpy, ra.a + surv);
        surv += rule_log_miss(ra);
      }
      if (dflt == label) logpy = lse(logpy, surv);
      // samples whose loss is clamped (or padding) get no gradient; their
      // log P_y is replaced by 0 so that every exponent below stays finite
      const bool on = live && -logpy * kLn2 <= kLossCap;
      const float gate = on ? 1.0f : 0.0f;
      const float lpy = on ? logpy : 0.0f;
      // reverse sweep
      float U = dflt == label ? 0.0f : kNegInf;
      for (int k = ss.y - 1; k >= 0; --k) {
        const int4 r = ldc(a.rules, ss.x + k);
        const float ak = my[k * 128 + lane];
        const float lk = ak + my[k * 128 + 64 + lane];
        const bool hit = r.z == label;
        float pre, mul;
        if (hit) {
          pre = lk - lpy;
          mul = -one_minus_exp2(U) * gate;
        } else {
          pre = lk + U - lpy;
          mul = gate;
        }
        RuleAcc ra;
        for (int j = r.x; j < r.x + r.y; ++j) {
          float z[1], xf[1], xg[1];
          bool ff;
          cond_z<1>(a, xs, lane, j, z, xf, xg, ff);
          const float lp = ra.add(z[0]);
          // dL/dz = dL/da_k * sigmoid(-z), one exponent in bits
          const float dz = mul * fexp2(pre - (fmaxf(z[0], 0.0f) + lp));
          const float g0 = wave_sum(dz * xg[0]);
          const float g1 = wave_sum(dz * xf[0]);
          if (lane == 0) {
            float *ap = acc + ((size_t)q * a.max_set_conds + (j - ss.z)) * 2;
            ap[0] += g0;
            ap[1] += g1;
          }
        }
        U = lse(hit ? ak : kNegInf, rule_log_miss(ra) + U);
      }
    }
  }
  __syncthreads();
  for (int q = 0; q < Q; ++q) {
    const int4 ss = ldc(a.ssets, q0 + q);
    for (int i = threadIdx.x; i < ss.w * 2; i += blockDim.x)
      a.part_grad[((int64_t)blockIdx.y * a.n_conds + ss.z) * 2 + i] =
          acc[(size_t)q * a.max_set_conds * 2 + i];
  }
}

// The reverse sweep over one rule's conditions, two at a time: their four
// sums over the wave in one reduction (wave_totals4), added (negated when
// neg) to the rule set's block accumulators accq by the lane that holds each
// (one writer per rule set and tile: the order of these adds is fixed).
// pre: log2 |dL/da_k| per slot (with MUL, log2 r_k, and mul holds
// dL/dr_k).  UPD: also adds every condition to ra, for the rule's log2 r
// afterwards.
// act: the rule's conditions to take, as rule_live gives them (the rest have
// terms of exactly 0).
template <int S, class Acc, bool TONLY, bool UPD, bool MUL = false>
__device__ __forceinline__ void bwd_rule_conds(const SoftArgs &a, const float *xs, int lane,
                                               int4 r, uint64_t act, int cz, float *accq,
                                               const float (&pre)[S], const float (&mul)[S],
                                               bool neg, Acc (&ra)[S]) {
  for (int base = r.x;;) {
    while (act != 0) {
      int jj[2];
      jj[0] = base + pop_bit(act);
      const bool two = act != 0;
      jj[1] = two ? base + pop_bit(act) : jj[0];
      // sums start at -0, so that the first term is added exactly as is
      float g0[2] = {-0.0f, -0.0f}, g1[2] = {-0.0f, -0.0f};
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        if (c == 1 && !two) break;
        const int j = jj[c];
        float z[S], xf[S], xg[S];
        if constexpr (TONLY) {
          cond_z_t<S>(a, xs, lane, j, z, xf, xg);
        } else {
          bool ff;
          cond_z<S>(a, xs, lane, j, z, xf, xg, ff);
        }
#pragma unroll
        for (int s = 0; s < S; ++s) {
          const float t = UPD ? ra[s].add(z[s]) : Acc::term(z[s]);
          // |dL/dz| = |dL/da_k| * sigmoid(-z), or dL/dz = dL/dr_k * r_k * sigmoid(-z)
          const float sg = acc_sig_neg(ra[s], pre[s], z[s], t);
          const float dz = MUL ? mul[s] * sg : sg;
          g0[c] = fmaf(dz, xg[s], g0[c]);
          g1[c] = fmaf(dz, xf[s], g1[c]);
        }
      }
      const float tot = wave_totals4(g0[0], g0[1], g1[0], g1[1]);
      const int row = lane >> 4, c = row >> 1;
      if ((lane & 15) == 15 && (c == 0 || two)) {
        float *ap = accq + ((c ? jj[1] : jj[0]) - cz) * 2 + (row & 1);
        *ap += neg ? -tot : tot;
      }
    }
    base += 64;
    if (base >= r.x + r.y) break;
    act = low_bits(min(r.x + r.y - base, 64));
  }
}

// Adjoint for rule sets of at most kRegRules rules with S samples per lane:
// the per-rule state kept between the two sweeps is l_k = a_k + (survival
// before k) and log2(1 - r_k), in per-lane private memory (scratch, served by
// the vector caches: only the rows of a set's own rules are touched; R, 32 or
// 64, bounds what is reserved).  The reverse sweep recomputes every
// condition once for its sigmoid(-z); only a rule of the label adds its
// conditions up again, for the a_k of the U recurrence (the other rules' step
// of it needs log2(1 - r_k) alone).  Per condition the S slots are summed in
// the lane; two conditions' sums go over the wave in one reduction
// (wave_totals4), and the lane that ends each adds it to the block's LDS
// accumulators (one writer per rule set and tile).  Eight waves per SIMD (two
// blocks per CU) at 64 VGPRs and 80 SGPRs: sets of up to 24 rules on 20,011 x
// 45 take 234 us (520 us with two samples per lane, 124 VGPRs and one block
// per CU), of 10-16 rules on 60,000 x 90 0.83 ms (1.39 ms likewise).
// TONLY: the population has threshold conditions only (no x[g] rows).
template <int S, class Acc, bool TONLY, int R>
__global__ __launch_bounds__(kBwdRegBlock, 8) AERL_SOFT_SGPR_CAP void k_soft_bwd_reg(
    const SoftArgs a) {
  constexpr int TS = 64 * S, WPT = AERL_TILE / TS;
  extern __shared__ __align__(16) float smem[];
  float *xs = smem;                                             // [nf][TS]
  float2 *ext = reinterpret_cast<float2 *>(xs + (size_t)a.nf * TS);  // [nf] when tiles classify
  float *acc = reinterpret_cast<float *>(ext + (a.classify ? a.nf : 0));  // [Q][max_set_conds][2]
  __shared__ int32_t next_q;
  const int lane = threadIdx.x & 63;
  int label, tile_lo, tile_hi;
  group_range(a, blockIdx.y, label, tile_lo, tile_hi);
  const int q0 = blockIdx.x * a.sets_per_chunk;
  const int Q = min(a.sets_per_chunk, a.n_sets - q0);
  for (int i = threadIdx.x; i < Q * a.max_set_conds * 2; i += blockDim.x) acc[i] = 0.0f;
  const int n4 = a.nf * (TS / 4);
  const float4 *src = reinterpret_cast<const float4 *>(a.x_fm);
  float4 *dst = reinterpret_cast<float4 *>(xs);
  const int64_t row4 = a.n_pad / 4;
  for (int64_t wt = (int64_t)tile_lo * WPT; wt < (int64_t)tile_hi * WPT; ++wt) {
    __syncthreads();
    const int64_t base4 = wt * (TS / 4);
    for (int i = threadIdx.x; i < n4; i += blockDim.x) {
      const int f = i / (TS / 4), k = i % (TS / 4);
      dst[i] = src[(int64_t)f * row4 + base4 + k];
    }
    if (threadIdx.x == 0) next_q = 0;
    __syncthreads();
    const int info = ldc(a.tile_info, wt / WPT);
    const int valid = min(max((info >> 8) - (int)(wt % WPT) * TS, 0), TS);
    if (valid == 0) continue;  // an empty wave tile (S < 4 at a region's end)
    if (a.classify) tile_extremes<TS>(xs, a.nf, valid, ext);
    bool live[S];
#pragma unroll
    for (int s = 0; s < S; ++s) live[s] = lane * S + s < valid;
    for (;;) {
      const int q = next_item(&next_q);
      if (q >= Q) break;
      const int4 ss = ldc(a.ssets, q0 + q);
      const int dflt = ldc(a.sets, q0 + q).z;
      const int set_end = ss.z + ss.w;
      const bool regular = set_regular(a, ss);
      Window win = first_window(a.classify && regular);
      RuleState<S, R> L, B;
      float logpy[S], surv[S];
#pragma unroll
      for (int s = 0; s < S; ++s) { logpy[s] = kNegInf; surv[s] = 0.0f; }
      // forward sweep
      for (int k = 0; k < ss.y; ++k) {
        const int4 r = ldc(a.rules, ss.x + k);
        uint64_t act;
        if (!rule_live<TONLY>(a, ext, lane, r, set_end, kDeadGrad, kDeadGrad, win, act)) continue;
        Acc ra[S];
        add_rule<S, Acc, TONLY>(a, xs, lane, r, act, ra);
        const bool hit = r.z == label;
        float lk[S], bk[S];
#pragma unroll
        for (int s = 0; s < S; ++s) {
          float a2, b2;
          acc_finish(ra[s], a2, b2);
          lk[s] = a2 + surv[s];
          bk[s] = b2;
          if (hit) logpy[s] = lse(logpy[s], lk[s]);
          surv[s] += b2;
        }
        L.set(k, lk);
        B.set(k, bk);
      }
      float gate[S], U[S];
#pragma unroll
      for (int s = 0; s < S; ++s) {
        if (dflt == label) logpy[s] = lse(logpy[s], surv[s]);
        // samples whose loss is clamped (or padding) get no gradient; their
        // log P_y is replaced by 0 so that every exponent below stays finite
        const bool on = live[s] && -logpy[s] * kLn2 <= kLossCap;
        gate[s] = on ? 1.0f : 0.0f;
        logpy[s] = on ? logpy[s] : 0.0f;
        U[s] = dflt == label ? 0.0f : kNegInf;
      }
      // reverse sweep
      for (int k = ss.y - 1; k >= 0; --k) {
        const int4 r = ldc(a.rules, ss.x + k);
        const bool hit = r.z == label;
        uint64_t act;
        if (!rule_live_back<TONLY>(a, ext, lane, r, ss.z, set_end, kDeadGrad, kDeadGrad, win, act))
          continue;
        // dL/da_k = -(1 - 2^U) 2^pre for a rule of the label, +2^pre for
        // another: log2 of its size goes into pre (-inf for a sample with no
        // gradient) and its sign, the same for the whole wave, onto the sums.
        // U, the log2 of a probability, can round to just above 0: 1 - 2^U
        // is then taken as 0.
        float lk[S], bk[S], pre[S];
        L.get(k, lk);
        B.get(k, bk);
        bool quiet = regular;  // every term of the rule is 0 as computed
#pragma unroll
        for (int s = 0; s < S; ++s) {
          const float lm = hit ? log1mexp2(fminf(U[s], 0.0f)) : U[s];
          pre[s] = gate[s] != 0.0f ? lk[s] + lm - logpy[s] : kNegInf;
          quiet = quiet && pre[s] < kExp2Zero;
        }
        const bool silent = ballot(!quiet) == 0;
        float *accq = acc + (size_t)q * a.max_set_conds * 2;
        Acc ra[S];
        if (hit) {
          // U takes the rule's own log2 r: the conditions are added again
          if (silent)
            add_rule<S, Acc, TONLY>(a, xs, lane, r, act, ra);
          else
            bwd_rule_conds<S, Acc, TONLY, true>(a, xs, lane, r, act, ss.z, accq, pre, pre, true, ra);
#pragma unroll
          for (int s = 0; s < S; ++s) U[s] = lse(acc_log_r(ra[s]), bk[s] + U[s]);
        } else {
          // U_k = log2(1 - r_k) + U_k+1, from the forward sweep's log2(1 - r_k)
          if (!silent)
            bwd_rule_conds<S, Acc, TONLY, false>(a, xs, lane, r, act, ss.z, accq, pre, pre, false, ra);
#pragma unroll
          for (int s = 0; s < S; ++s) U[s] = bk[s] + U[s];
        }
      }
    }
  }
  __syncthreads();
  for (int q = 0; q < Q; ++q) {
    const int4 ss = ldc(a.ssets, q0 + q);
    for (int i = threadIdx.x; i < ss.w * 2; i += blockDim.x)
      a.part_grad[((int64_t)blockIdx.y * a.n_conds + ss.z) * 2 + i] =
          acc[(size_t)q * a.max_set_conds * 2 + i];
  }
}

// One block per rule set: sums the group partials of its conditions in a
// fixed order and applies dz/dparam = +-x/tau, -+1/tau and dloss/N.
__global__ void k_soft_bwd_final(const float *__restrict__ part, int32_t n_groups,
                                 int32_t n_conds, const int4 *__restrict__ ssets,
                                 const uint32_t *__restrict__ sconds,
                                 const float *__restrict__ inv_tau,
                                 const float *__restrict__ dloss, int64_t n,
                                 float *__restrict__ dcoef, float *__restrict__ dcoef2,
                                 float *__restrict__ dtheta) {
  const int p = blockIdx.x;
  const int4 ss = ssets[p];
  const double scale = n > 0 ? (double)dloss[p] / (double)n : 0.0;
  for (int i = threadIdx.x; i < ss.w; i += blockDim.x) {
    const int j = ss.z + i;
    double g0, g1;
    sum_groups(part, n_groups, n_conds, j, g0, g1);
    const uint32_t sc = sconds[j];
    const bool ff = (sc & kSoftFF) != 0;
    float dc, dr;
    param_grads(sc, inv_tau, g0, g1, scale, dc, dr);
    dcoef[j] = dc;
    dcoef2[j] = ff ? dr : 0.0f;
    dtheta[j] = ff ? 0.0f : dr;
  }
}

void fill_args(SoftArgs &a, const SoftLaunch &l, const SoftPlan &p) {
  const DatasetRec &ds = *l.ds;
  const PopRec &pop = *l.pop;
  a = SoftArgs{};
  a.x_fm = ds.x_fm;
  a.n_pad = ds.n_pad;
  a.nf = ds.nf;
  a.nc = ds.nc;
  a.tile_info = ds.tile_info;
  a.inv_tau = ds.inv_tau;
  a.sets = pop.sets;
  a.ssets = pop.ssets;
  a.rules = pop.rules;
  a.sconds = pop.sconds;
  a.coef = l.coef;
  a.coef2 = l.coef2;
  a.theta = l.theta;
  a.n_sets = pop.n_sets;
  a.n_conds = pop.n_conds;
  a.sets_per_chunk = p.Q;
  a.tiles_per_group = p.TG;
  a.n_groups = p.n_groups;
  a.classify = p.cls;
  a.max_rules = std::max(pop.max_rules, 1);
  a.max_set_conds = std::max(pop.max_set_conds, 1);
  for (int c = 0; c < ds.nc; ++c) {
    a.region_tile0[c] = ds.region_tile0[c];
    a.region_tiles[c] = ds.region_tiles[c];
  }
}

template <int S, class Acc, bool TONLY>
void launch_fwd_s(const SoftPlan &p, dim3 grid, hipStream_t st, const SoftArgs &a) {
  if (p.cls)
    hipLaunchKernelGGL((k_soft_fwd_cls<S, Acc, TONLY>), grid, dim3(kSoftBlock), p.lds, st, a);
  else
    hipLaunchKernelGGL((k_soft_fwd<S, Acc, TONLY>), grid, dim3(kSoftBlock), p.lds, st, a);
}

template <class Acc, bool TONLY>
void launch_fwd(const SoftPlan &p, dim3 grid, hipStream_t st, const SoftArgs &a) {
  switch (p.S) {
    case 4: launch_fwd_s<4, Acc, TONLY>(p, grid, st, a); break;
    case 2: launch_fwd_s<2, Acc, TONLY>(p, grid, st, a); break;
    default: launch_fwd_s<1, Acc, TONLY>(p, grid, st, a); break;
  }
}

template <int S, class Acc, bool TONLY>
void launch_bwd_reg_s(const SoftPlan &p, dim3 grid, hipStream_t st, const SoftArgs &a) {
  if (a.max_rules <= kFewRules)
    hipLaunchKernelGGL((k_soft_bwd_reg<S, Acc, TONLY, kFewRules>), grid, dim3(kBwdRegBlock), p.lds, st, a);
  else
    hipLaunchKernelGGL((k_soft_bwd_reg<S, Acc, TONLY, kRegRules>), grid, dim3(kBwdRegBlock), p.lds, st, a);
}

template <class Acc, bool TONLY>
void launch_bwd_reg(const SoftPlan &p, dim3 grid, hipStream_t st, const SoftArgs &a) {
  switch (p.S) {
    case 4: launch_bwd_reg_s<4, Acc, TONLY>(p, grid, st, a); break;
    case 2: launch_bwd_reg_s<2, Acc, TONLY>(p, grid, st, a); break;
    default: launch_bwd_reg_s<1, Acc, TONLY>(p, grid, st, a); break;
  }
}

}  // namespace

// Sets past 32 rules are bounded by the LDS-state kernel's one-wave form,
// whichever kernel runs them.
bool soft_backward_supported(const DatasetRec &ds, const PopRec &pop) {
  return (pop.max_rules <= 32 || plan_lds_state(ds, pop, SoftPlan{}, 1).lds <= kDynLdsMax) &&
         plan_backward(ds, pop).lds <= kDynLdsMax;
}

namespace {

// Workspace: the partial sums, then (256-byte aligned) the condition records.
size_t soft_part_bytes(const DatasetRec &ds, const PopRec &pop, bool backward) {
  size_t b;
  if (backward) {
    const SoftPlan p = plan_backward(ds, pop);
    b = (size_t)p.n_groups * (size_t)std::max(pop.n_conds, 1) * 2 * sizeof(float);
  } else {
    const SoftPlan p = plan_forward(ds, pop);
    b = (size_t)p.n_groups * (size_t)std::max(pop.n_sets, 1) * sizeof(double);
  }
  return (b + 255) & ~size_t(255);
}

hipError_t launch_prep(const SoftLaunch &l, const SoftArgs &a, uint4 *crec, hipStream_t st) {
  if (l.pop->n_conds == 0) return hipSuccess;
  const dim3 block(l.pop->max_set_conds <= 64 ? 64 : kPrepBlock);
  hipLaunchKernelGGL(k_soft_prep, dim3((unsigned)l.pop->n_sets), block, 0, st, a.ssets, a.sconds,
                     a.inv_tau, a.coef, a.coef2, a.theta, l.pop->cmask, crec);
  return hipGetLastError();
}

}  // namespace

size_t soft_ws_bytes(const DatasetRec &ds, const PopRec &pop, bool backward) {
  return soft_part_bytes(ds, pop, backward) + (size_t)std::max(pop.n_conds, 1) * sizeof(uint4);
}

hipError_t launch_soft_forward(const SoftLaunch &l, hipStream_t st) {
  const PopRec &pop = *l.pop;
  if (pop.n_sets == 0) return hipSuccess;
  const SoftPlan p = plan_forward(*l.ds, pop);
  SoftArgs a;
  fill_args(a, l, p);
  a.part_loss = static_cast<double *>(l.ws);
  uint4 *crec = reinterpret_cast<uint4 *>(static_cast<char *>(l.ws) + soft_part_bytes(*l.ds, pop, false));
  a.crec = crec;
  hipError_t e0 = launch_prep(l, a, crec, st);
  if (e0 != hipSuccess) return e0;
  if (p.n_groups > 0) {
    const dim3 grid((unsigned)((pop.n_sets + p.Q - 1) / p.Q), (unsigned)p.n_groups);
    const bool prod = pop.max_rule_conds <= kProdMaxConds, tonly = pop.n_ff == 0 && pop.n_cat == 0;
    if (prod && tonly) {
      launch_fwd<RuleProd, true>(p, grid, st, a);
    } else if (prod) {
      launch_fwd<RuleProd, false>(p, grid, st, a);
    } else if (tonly) {
      launch_fwd<RuleAcc, true>(p, grid, st, a);
    } else {
      launch_fwd<RuleAcc, false>(p, grid, st, a);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_soft_fwd_final, dim3((unsigned)((pop.n_sets + 63) / 64)),
                     dim3(kFwdFinalWaves * 64), 0, st,
                     a.part_loss, p.n_groups, pop.n_sets, l.ds->n, l.loss);
  return hipGetLastError();
}

// ------------------------------------------------------------ softmax head
// Section 5: probabilistic outputs through a softmax.  Each rule votes for
// its class with its soft truth r_k, the default class takes the probability
// that no rule fires, D = prod_k (1 - r_k):
//   v_c = sum_{k: class_k = c} r_k + [c = default] D,  P = softmax(beta v),
// L = min(-log P_y, 100).  Adjoint: dL/dv_c = beta (P_c - [c = y]),
// dL/dr_k = dL/dv_{class_k} - dL/dv_default * prod_{i != k} (1 - r_i), the
// product being 2^(S_k + T_k) with the prefix S_k and suffix T_k sums of
// log2(1 - r_i); dL/dz = dL/dr_k * r_k * sigmoid(-z).  Classes are padded to
// NC (a power of two up to kSmaxMaxClasses) in registers; rule classes are
// wave-uniform, so a vote is NC selects.
namespace {

template <int NC>
__device__ __forceinline__ void add_vote(float (&v)[NC], int cls, float r) {
#pragma unroll
  for (int c = 0; c < NC; ++c) v[c] += (c == cls) ? r : 0.0f;
}

template <int NC>
__device__ __forceinline__ float pick(const float (&v)[NC], int cls) {
  float out = 0.0f;
#pragma unroll
  for (int c = 0; c < NC; ++c) out = (c == cls) ? v[c] : out;
  return out;
}

// log2 P_y from the votes, and P (every class) into p.  beta2 = beta*log2(e).
template <int NC>
__device__ __forceinline__ float smax_log2py(const float (&v)[NC], int nc, float beta2, int y,
                                             float (&p)[NC]) {
  float m = kNegInf;
#pragma unroll
  for (int c = 0; c < NC; ++c)
    if (c < nc) m = fmaxf(m, beta2 * v[c]);
  float sum = 0.0f;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    p[c] = c < nc ? fexp2(beta2 * v[c] - m) : 0.0f;
    sum += p[c];
  }
  const float inv = 1.0f / sum;
  float ty = 0.0f;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    ty = (c == y) ? beta2 * v[c] : ty;
    p[c] *= inv;
  }
  return ty - m - flog2(sum);
}

template <int S, int NC, class Acc, bool TONLY, bool CLS>
__device__ __forceinline__ void smax_fwd(const SoftArgs a, float beta2) {
  constexpr int TS = 64 * S, WPT = AERL_TILE / TS;
  extern __shared__ __align__(16) float smem[];
  float *xs = smem;
  float2 *ext = reinterpret_cast<float2 *>(smem + (size_t)a.nf * TS);  // [nf] with CLS
  double *acc = reinterpret_cast<double *>(ext + (CLS ? a.nf : 0));    // [Q]
  __shared__ int32_t next_q;
  const int lane = threadIdx.x & 63;
  int label, tile_lo, tile_hi;
  group_range(a, blockIdx.y, label, tile_lo, tile_hi);
  const int q0 = blockIdx.x * a.sets_per_chunk;
  const int Q = min(a.sets_per_chunk, a.n_sets - q0);
  for (int i = threadIdx.x; i < Q; i += blockDim.x) acc[i] = 0.0;
  const int n4 = a.nf * (TS / 4);
  const float4 *src = reinterpret_cast<const float4 *>(a.x_fm);
  float4 *dst = reinterpret_cast<float4 *>(xs);
  const int64_t row4 = a.n_pad / 4;
  for (int64_t wt = (int64_t)tile_lo * WPT; wt < (int64_t)tile_hi * WPT; ++wt) {
    __syncthreads();
    const int64_t base4 = wt * (TS / 4);
    for (int i = threadIdx.x; i < n4; i += blockDim.x) {
      const int f = i / (TS / 4), k = i % (TS / 4);
      dst[i] = src[(int64_t)f * row4 + base4 + k];
    }
    if (threadIdx.x == 0) next_q = 0;
    __syncthreads();
    const int info = ldc(a.tile_info, wt / WPT);
    const int valid = min(max((info >> 8) - (int)(wt % WPT) * TS, 0), TS);
    if (S < 4 && valid == 0) continue;  // an empty wave tile (S < 4 at a region's end)
    if constexpr (CLS) tile_extremes<TS>(xs, a.nf, valid, ext);
    for (;;) {
      const int q = next_item(&next_q);
      if (q >= Q) break;
      const int4 ss = ldc(a.ssets, q0 + q);
      const int dflt = ldc(a.sets, q0 + q).z;
      const int set_end = ss.z + ss.w;
      Window win;
      if constexpr (CLS) win = first_window(set_regular(a, ss));
      float v[S][NC], surv[S];
#pragma unroll
      for (int s = 0; s < S; ++s) {
        surv[s] = 0.0f;
#pragma unroll
        for (int c = 0; c < NC; ++c) v[s][c] = 0.0f;
      }
      for (int k = 0; k < ss.y; ++k) {
        const int4 r = ldc(a.rules, ss.x + k);
        Acc ra[S];
        if constexpr (CLS) {
          uint64_t act;
          if (!rule_live<TONLY>(a, ext, lane, r, set_end, kDeadProb, Acc::kNoop, win, act)) continue;
          add_rule<S, Acc, TONLY>(a, xs, lane, r, act, ra);
        } else {
          add_all<S, Acc, TONLY>(a, xs, lane, r, ra);
        }
#pragma unroll
        for (int s = 0; s < S; ++s) {
          float a2, b2;
          acc_finish(ra[s], a2, b2);
          add_vote(v[s], r.z, fexp2(a2));
          surv[s] += b2;
        }
      }
      float part = 0.0f;
#pragma unroll
      for (int s = 0; s < S; ++s) {
        add_vote(v[s], dflt, fexp2(surv[s]));
        float p[NC];
        const float l2 = smax_log2py(v[s], a.nc, beta2, label, p);
        part += lane * S + s < valid ? sample_loss(l2) : 0.0f;
      }
      part = wave_sum(part);
      if (lane == 0) acc[q] += (double)part;
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < Q; i += blockDim.x)
    a.part_loss[(int64_t)blockIdx.y * a.n_sets + q0 + i] = acc[i];
}

template <int S, int NC, class Acc, bool TONLY>
__global__ __launch_bounds__(kSoftBlock, 8) AERL_SOFT_SGPR_CAP void k_smax_fwd_cls(const SoftArgs a,
                                                                                 float beta2) {
  smax_fwd<S, NC, Acc, TONLY, true>(a, beta2);
}
template <int S, int NC, class Acc, bool TONLY>
__global__ __launch_bounds__(kSoftBlock) void k_smax_fwd(const SoftArgs a, float beta2) {
  smax_fwd<S, NC, Acc, TONLY, false>(a, beta2);
}

template <int NC, class Acc, bool TONLY>
__global__ __launch_bounds__(kSmaxBwdWaves * 64) void k_smax_bwd(const SoftArgs a, float beta,
                                                                 float beta2) {
  constexpr int TS = 64, WPT = AERL_TILE / TS;
  extern __shared__ __align__(16) float smem[];
  float *xs = smem;                                                     // [nf][64]
  float *acc = xs + (size_t)a.nf * TS;                                  // [Q][max_set_conds][2]
  float *store = acc + (size_t)a.sets_per_chunk * a.max_set_conds * 2;  // [wave][R][2][64]
  __shared__ int32_t next_q;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float *my = store + (size_t)wave * a.max_rules * 128;
  int label, tile_lo, tile_hi;
  group_range(a, blockIdx.y, label, tile_lo, tile_hi);
  const int q0 = blockIdx.x * a.sets_per_chunk;
  const int Q = min(a.sets_per_chunk, a.n_sets - q0);
  for (int i = threadIdx.x; i < Q * a.max_set_conds * 2; i += blockDim.x) acc[i] = 0.0f;
  const int n4 = a.nf * (TS / 4);
  const float4 *src = reinterpret_cast<const float4 *>(a.x_fm);
  float4 *dst = reinterpret_cast<float4 *>(xs);
  const int64_t row4 = a.n_pad / 4;
  for (int64_t wt = (int64_t)tile_lo * WPT; wt < (int64_t)tile_hi * WPT; ++wt) {
    __syncthreads();
    const int64_t base4 = wt * (TS / 4);
    for (int i = threadIdx.x; i < n4; i += blockDim.x) {
      const int f = i / (TS / 4), k = i % (TS / 4);
      dst[i] = src[(int64_t)f * row4 + base4 + k];
    }
    if (threadIdx.x == 0) next_q = 0;
    __syncthreads();
    const int info = ldc(a.tile_info, wt / WPT);
    const int valid = min(max((info >> 8) - (int)(wt % WPT) * TS, 0), TS);
    const bool live = lane < valid;
    for (;;) {
      const int q = next_item(&next_q);
      if (q >= Q) break;
      const int4 ss = ldc(a.ssets, q0 + q);
      const int dflt = ldc(a.sets, q0 + q).z;
      // forward sweep: log2 r_k and the prefix of log2(1 - r_i) before k
      float v[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) v[c] = 0.0f;
      float surv = 0.0f;
      for (int k = 0; k < ss.y; ++k) {
        const int4 r = ldc(a.rules, ss.x + k);
        Acc ra;
        for (int j = r.x; j < r.x + r.y; ++j) {
          float z[1];
          cond_z_only<1>(a, xs, lane, j, z);
          (void)ra.add(z[0]);
        }
        float a2, b2;
        acc_finish(ra, a2, b2);
        my[k * 128 + lane] = a2;
        my[k * 128 + 64 + lane] = surv;
        add_vote(v, r.z, fexp2(a2));
        surv += b2;
      }
      add_vote(v, dflt, fexp2(surv));
      float p[NC];
      const float l2 = smax_log2py(v, a.nc, beta2, label, p);
      // clamped samples (and padding) get no gradient
      const bool on = live && -l2 * kLn2 <= kLossCap;
      // dL/dv_c = beta (P_c - [c = y]); for the label, -beta times the sum of
      // the other classes' probabilities (P_y - 1 would cancel when P_y ~ 1)
      float others = 0.0f;
#pragma unroll
      for (int c = 0; c < NC; ++c) others += c == label ? 0.0f : p[c];
      float gv[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) gv[c] = on ? beta * (c == label ? -others : p[c]) : 0.0f;
      const float gd = pick(gv, dflt);
      // reverse sweep with the suffix of log2(1 - r_i) after k
      float tail = 0.0f;
      const bool few = ss.w <= 64;
      int tot0 = 0, tot1 = 0;
      for (int k = ss.y - 1; k >= 0; --k) {
        const int4 r = ldc(a.rules, ss.x + k);
        const float a2k = my[k * 128 + lane];
        const float others = my[k * 128 + 64 + lane] + tail;  // log2 prod_{i != k} (1 - r_i)
        // a rule of the default class: g_d (1 - prod), with 1 - prod formed
        // directly (the difference of the two terms would cancel)
        const float drk = r.z == dflt ? gd * one_minus_exp2(others)
                                      : pick(gv, r.z) - gd * fexp2(others);
        Acc ra;
        for (int j = r.x; j < r.x + r.y; ++j) {
          float z[1], xf[1], xg[1];
          if constexpr (TONLY) {
            cond_z_t<1>(a, xs, lane, j, z, xf, xg);
          } else {
            bool ff;
            cond_z<1>(a, xs, lane, j, z, xf, xg, ff);
          }
          const float t = ra.add(z[0]);
          // dL/dz = dL/dr_k * r_k * sigmoid(-z)
          const float dz = drk * acc_sig_neg(ra, a2k, z[0], t);
          const float g0 = wave_total_last(dz * xg[0]);
          const float g1 = wave_total_last(dz * xf[0]);
          if (few) {
            // lane i keeps the walk's totals of condition i of the set
            const int v0 = __builtin_amdgcn_readlane(__float_as_int(g0), 63);
            const int v1 = __builtin_amdgcn_readlane(__float_as_int(g1), 63);
            const bool mine = lane == j - ss.z;
            tot0 = mine ? v0 : tot0;
            tot1 = mine ? v1 : tot1;
          } else if (lane == 63) {
            // one writer per (rule set, tile): the order of these adds is fixed
            float *ap = acc + ((size_t)q * a.max_set_conds + (j - ss.z)) * 2;
            ap[0] += g0;
            ap[1] += g1;
          }
        }
        float a2, b2;
        acc_finish(ra, a2, b2);
        tail += b2;
      }
      if (few && lane < ss.w) {
        float *ap = acc + ((size_t)q * a.max_set_conds + lane) * 2;
        ap[0] += __int_as_float(tot0);
        ap[1] += __int_as_float(tot1);
      }
    }
  }
  __syncthreads();
  for (int q = 0; q < Q; ++q) {
    const int4 ss = ldc(a.ssets, q0 + q);
    for (int i = threadIdx.x; i < ss.w * 2; i += blockDim.x)
      a.part_grad[((int64_t)blockIdx.y * a.n_conds + ss.z) * 2 + i] =
          acc[(size_t)q * a.max_set_conds * 2 + i];
  }
}

// Adjoint of the softmax head for rule sets of at most kRegRules rules, 16
// waves per block: the per-rule state between the two sweeps (log2 r_k, the
// prefix sum of log2(1 - r_i) before k and log2(1 - r_k), for each of the
// lane's samples) is in private memory as in the first-firing adjoint; the
// votes and their gradients take S x NC registers each, at most 16.  The
// reverse sweep needs each condition's sigmoid(-z) alone, so it adds no
// condition up again; the conditions' sums go over the wave and to LDS as in
// the first-firing adjoint.  Same formulas as k_smax_bwd, which takes 4-15
// times as long (sets of up to 24 rules on 20,011 x 45: 0.97 ms against
// 0.25).
template <int S, int NC, class Acc, bool TONLY, int R>
__global__ __launch_bounds__(kBwdRegBlock, 8) AERL_SOFT_SGPR_CAP void k_smax_bwd_reg(
    const SoftArgs a, float beta, float beta2) {
  constexpr int TS = 64 * S, WPT = AERL_TILE / TS;
  extern __shared__ __align__(16) float smem[];
  float *xs = smem;                                             // [nf][TS]
  float2 *ext = reinterpret_cast<float2 *>(xs + (size_t)a.nf * TS);  // [nf] when tiles classify
  float *acc = reinterpret_cast<float *>(ext + (a.classify ? a.nf : 0));  // [Q][max_set_conds][2]
  __shared__ int32_t next_q;
  const int lane = threadIdx.x & 63;
  int label, tile_lo, tile_hi;
  group_range(a, blockIdx.y, label, tile_lo, tile_hi);
  const int q0 = blockIdx.x * a.sets_per_chunk;
  const int Q = min(a.sets_per_chunk, a.n_sets - q0);
  for (int i = threadIdx.x; i < Q * a.max_set_conds * 2; i += blockDim.x) acc[i] = 0.0f;
  const int n4 = a.nf * (TS / 4);
  const float4 *src = reinterpret_cast<const float4 *>(a.x_fm);
  float4 *dst = reinterpret_cast<float4 *>(xs);
  const int64_t row4 = a.n_pad / 4;
  for (int64_t wt = (int64_t)tile_lo * WPT; wt < (int64_t)tile_hi * WPT; ++wt) {
    __syncthreads();
    const int64_t base4 = wt * (TS / 4);
    for (int i = threadIdx.x; i < n4; i += blockDim.x) {
      const int f = i / (TS / 4), k = i % (TS / 4);
      dst[i] = src[(int64_t)f * row4 + base4 + k];
    }
    if (threadIdx.x == 0) next_q = 0;
    __syncthreads();
    const int info = ldc(a.tile_info, wt / WPT);
    const int valid = min(max((info >> 8) - (int)(wt % WPT) * TS, 0), TS);
    if (valid == 0) continue;  // an empty wave tile (S < 4 at a region's end)
    if (a.classify) tile_extremes<TS>(xs, a.nf, valid, ext);
    for (;;) {
      const int q = next_item(&next_q);
      if (q >= Q) break;
      const int4 ss = ldc(a.ssets, q0 + q);
      const int dflt = ldc(a.sets, q0 + q).z;
      const int set_end = ss.z + ss.w;
      const bool regular = set_regular(a, ss);
      Window win = first_window(a.classify && regular);
      RuleState<S, R> LA, LP, LB;
      float v[S][NC], surv[S];
#pragma unroll
      for (int s = 0; s < S; ++s) {
        surv[s] = 0.0f;
#pragma unroll
        for (int c = 0; c < NC; ++c) v[s][c] = 0.0f;
      }
      // forward sweep: log2 r_k and the prefix of log2(1 - r_i) before k
      for (int k = 0; k < ss.y; ++k) {
        const int4 r = ldc(a.rules, ss.x + k);
        uint64_t act;
        if (!rule_live<TONLY>(a, ext, lane, r, set_end, kDeadProb, Acc::kNoop, win, act)) continue;
        Acc ra[S];
        add_rule<S, Acc, TONLY>(a, xs, lane, r, act, ra);
        float a2s[S], pre[S], b2s[S];
#pragma unroll
        for (int s = 0; s < S; ++s) {
          float a2, b2;
          acc_finish(ra[s], a2, b2);
          a2s[s] = a2;
          pre[s] = surv[s];
          b2s[s] = b2;
          add_vote(v[s], r.z, fexp2(a2));
          surv[s] += b2;
        }
        LA.set(k, a2s);
        LP.set(k, pre);
        LB.set(k, b2s);
      }
      // dL/dv per slot (clamped samples and padding get none); for the
      // label, -beta times the other classes' probabilities
      float gv[S][NC], gd[S], tail[S];
#pragma unroll
      for (int s = 0; s < S; ++s) {
        add_vote(v[s], dflt, fexp2(surv[s]));
        float p[NC];
        const float l2 = smax_log2py(v[s], a.nc, beta2, label, p);
        const bool on = lane * S + s < valid && -l2 * kLn2 <= kLossCap;
        float others = 0.0f;
#pragma unroll
        for (int c = 0; c < NC; ++c) others += c == label ? 0.0f : p[c];
#pragma unroll
        for (int c = 0; c < NC; ++c) gv[s][c] = on ? beta * (c == label ? -others : p[c]) : 0.0f;
        gd[s] = pick(gv[s], dflt);
        tail[s] = 0.0f;
      }
      // reverse sweep with the suffix of log2(1 - r_i) after k
      win = first_window(a.classify && regular);
      for (int k = ss.y - 1; k >= 0; --k) {
        const int4 r = ldc(a.rules, ss.x + k);
        uint64_t act;
        if (!rule_live_back<TONLY>(a, ext, lane, r, ss.z, set_end, kDeadProb, kSatProb, win, act))
          continue;
        float la[S], lp[S], drk[S];
        LA.get(k, la);
        LP.get(k, lp);
        bool quiet = regular;  // every term of the rule is 0 as computed
#pragma unroll
        for (int s = 0; s < S; ++s) {
          const float oth = lp[s] + tail[s];  // log2 prod_{i != k} (1 - r_i)
          drk[s] = r.z == dflt ? gd[s] * one_minus_exp2(oth)
                               : pick(gv[s], r.z) - gd[s] * fexp2(oth);
          quiet = quiet && (la[s] < kExp2Zero || drk[s] == 0.0f);
        }
        // the conditions' terms need no accumulator: log2(1 - r_k) comes
        // from the forward sweep
        if (ballot(!quiet) != 0) {
          Acc ra[S];
          bwd_rule_conds<S, Acc, TONLY, false, true>(a, xs, lane, r, act, ss.z,
                                                     acc + (size_t)q * a.max_set_conds * 2, la, drk,
                                                     false, ra);
        }
        float lb[S];
        LB.get(k, lb);
#pragma unroll
        for (int s = 0; s < S; ++s) tail[s] += lb[s];
      }
    }
  }
  __syncthreads();
  for (int q = 0; q < Q; ++q) {
    const int4 ss = ldc(a.ssets, q0 + q);
    for (int i = threadIdx.x; i < ss.w * 2; i += blockDim.x)
      a.part_grad[((int64_t)blockIdx.y * a.n_conds + ss.z) * 2 + i] =
          acc[(size_t)q * a.max_set_conds * 2 + i];
  }
}

// Class probabilities of one rule set for row-major rows, one row per
// thread (the gathered condition records give z).
template <int NC>
__global__ __launch_bounds__(256) void k_smax_proba(const float *__restrict__ rows, int64_t n,
                                                    int32_t nf, int32_t nc, int32_t set,
                                                    const int4 *__restrict__ sets,
                                                    const int4 *__restrict__ ssets,
                                                    const int4 *__restrict__ rules,
                                                    const uint4 *__restrict__ crec, float beta2,
                                                    float *__restrict__ probs) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int4 ss = ssets[set];
  const int32_t dflt = sets[set].z;
  const float *x = rows + i * nf;
  float v[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) v[c] = 0.0f;
  float surv = 0.0f;
  for (int k = 0; k < ss.y; ++k) {
    const int4 r = rules[ss.x + k];
    RuleAcc ra;
    for (int j = r.x; j < r.x + r.y; ++j) {
      const uint4 c4 = crec[j];
      const uint32_t sc = c4.x;
      const float xf = x[sc & 0xfffu];
      if (sc & kSoftCat) {
        (void)ra.add(cat_z(xf, c4.y, c4.z));
        continue;
      }
      const float rv = __uint_as_float(c4.z);
      const float rhs = (sc & kSoftFF) ? rv * x[(sc >> 12) & 0xfffu] : rv;
      (void)ra.add(fmaf(__uint_as_float(c4.y), xf, -rhs) * __uint_as_float(c4.w));
    }
    float a2, b2;
    acc_finish(ra, a2, b2);
    add_vote(v, r.z, fexp2(a2));
    surv += b2;
  }
  add_vote(v, dflt, fexp2(surv));
  float p[NC];
  (void)smax_log2py(v, nc, beta2, 0, p);
  for (int c = 0; c < nc; ++c) probs[i * nc + c] = p[c];
}

template <int S, int NC, class Acc, bool TONLY>
void launch_smax_fwd_t(const SoftPlan &p, dim3 grid, hipStream_t st, const SoftArgs &a, float beta2) {
  const dim3 b(kSoftBlock);
  if (p.cls)
    hipLaunchKernelGGL((k_smax_fwd_cls<S, NC, Acc, TONLY>), grid, b, p.lds, st, a, beta2);
  else
    hipLaunchKernelGGL((k_smax_fwd<S, NC, Acc, TONLY>), grid, b, p.lds, st, a, beta2);
}

template <int S, int NC>
void launch_smax_fwd_s(const SoftPlan &p, dim3 grid, hipStream_t st, const SoftArgs &a, bool prod,
                       bool tonly, float beta2) {
  if (prod && tonly)
    launch_smax_fwd_t<S, NC, RuleProd, true>(p, grid, st, a, beta2);
  else if (prod)
    launch_smax_fwd_t<S, NC, RuleProd, false>(p, grid, st, a, beta2);
  else if (tonly)
    launch_smax_fwd_t<S, NC, RuleAcc, true>(p, grid, st, a, beta2);
  else
    launch_smax_fwd_t<S, NC, RuleAcc, false>(p, grid, st, a, beta2);
}

template <int NC>
void launch_smax_fwd_nc(const SoftPlan &p, dim3 grid, hipStream_t st, const SoftArgs &a, bool prod,
                        bool tonly, float beta2) {
  if constexpr (NC <= 4) {
    if (p.S == 4) return launch_smax_fwd_s<4, NC>(p, grid, st, a, prod, tonly, beta2);
  }
  if (p.S == 2) return launch_smax_fwd_s<2, NC>(p, grid, st, a, prod, tonly, beta2);
  launch_smax_fwd_s<1, NC>(p, grid, st, a, prod, tonly, beta2);
}

template <int S, int NC, class Acc, bool TONLY>
void launch_smax_bwd_t(const SoftPlan &p, dim3 grid, hipStream_t st, const SoftArgs &a, float beta,
                       float beta2) {
  const dim3 b(kBwdRegBlock);
  if (a.max_rules <= kFewRules)
    hipLaunchKernelGGL((k_smax_bwd_reg<S, NC, Acc, TONLY, kFewRules>), grid, b, p.lds, st, a, beta, beta2);
  else
    hipLaunchKernelGGL((k_smax_bwd_reg<S, NC, Acc, TONLY, kRegRules>), grid, b, p.lds, st, a, beta, beta2);
}

template <int S, int NC>
void launch_smax_bwd_s(const SoftPlan &p, dim3 grid, hipStream_t st, const SoftArgs &a, bool prod,
                       bool tonly, float beta, float beta2) {
  if (prod && tonly)
    launch_smax_bwd_t<S, NC, RuleProd, true>(p, grid, st, a, beta, beta2);
  else if (prod)
    launch_smax_bwd_t<S, NC, RuleProd, false>(p, grid, st, a, beta, beta2);
  else if (tonly)
    launch_smax_bwd_t<S, NC, RuleAcc, true>(p, grid, st, a, beta, beta2);
  else
    launch_smax_bwd_t<S, NC, RuleAcc, false>(p, grid, st, a, beta, beta2);
}

template <int NC>
void launch_smax_bwd_nc(const SoftPlan &p, dim3 grid, hipStream_t st, const SoftArgs &a, bool prod,
                        bool tonly, float beta, float beta2) {
  if (!p.reg) {
    const dim3 b(p.waves * 64);
    // threshold rules alone spare a branch per condition (29,646 x 44, 111 rule
    // sets of 80 rules: 9.9 ms against 10.4)
    if (prod && tonly)
      hipLaunchKernelGGL((k_smax_bwd<NC, RuleProd, true>), grid, b, p.lds, st, a, beta, beta2);
    else if (prod)
      hipLaunchKernelGGL((k_smax_bwd<NC, RuleProd, false>), grid, b, p.lds, st, a, beta, beta2);
    else if (tonly)
      hipLaunchKernelGGL((k_smax_bwd<NC, RuleAcc, true>), grid, b, p.lds, st, a, beta, beta2);
    else
      hipLaunchKernelGGL((k_smax_bwd<NC, RuleAcc, false>), grid, b, p.lds, st, a, beta, beta2);
    return;
  }
  if constexpr (NC <= 4) {
    if (p.S == 4) return launch_smax_bwd_s<4, NC>(p, grid, st, a, prod, tonly, beta, beta2);
  }
  if constexpr (NC <= 8) {
    if (p.S == 2) return launch_smax_bwd_s<2, NC>(p, grid, st, a, prod, tonly, beta, beta2);
  }
  launch_smax_bwd_s<1, NC>(p, grid, st, a, prod, tonly, beta, beta2);
}

}  // namespace

// Tables wide enough that a forward tile of two samples per lane does not
// fit are refused, and sets past 16 rules (four classes, 64 features) are
// bounded by the LDS-state adjoint's one-wave form, whichever kernels run.
bool smax_supported(const DatasetRec &ds, const PopRec &pop) {
  const bool few = pop.max_rules <= 16 && smax_nc(ds.nc) <= 4 && ds.nf <= 64;
  return ds.nc <= kSmaxMaxClasses &&
         (few || plan_lds_state(ds, pop, SoftPlan{}, 1).lds <= kDynLdsMax) &&
         (size_t)ds.nf * 64 * 2 * 4 + (size_t)plan_forward(ds, pop).Q * 8 <= kDynLdsMax;
}

hipError_t launch_smax_forward(const SoftLaunch &l, float beta, hipStream_t st) {
  const PopRec &pop = *l.pop;
  if (pop.n_sets == 0) return hipSuccess;
  const SoftPlan p = plan_smax_forward(*l.ds, pop);
  SoftArgs a;
  fill_args(a, l, p);
  a.part_loss = static_cast<double *>(l.ws);
  uint4 *crec = reinterpret_cast<uint4 *>(static_cast<char *>(l.ws) + soft_part_bytes(*l.ds, pop, false));
  a.crec = crec;
  hipError_t e = launch_prep(l, a, crec, st);
  if (e != hipSuccess) return e;
  const float beta2 = beta * kLog2e;
  if (p.n_groups > 0) {
    const dim3 grid((unsigned)((pop.n_sets + p.Q - 1) / p.Q), (unsigned)p.n_groups);
    const bool prod = pop.max_rule_conds <= kProdMaxConds, tonly = pop.n_ff == 0 && pop.n_cat == 0;
    switch (smax_nc(l.ds->nc)) {
      case 2: launch_smax_fwd_nc<2>(p, grid, st, a, prod, tonly, beta2); break;
      case 4: launch_smax_fwd_nc<4>(p, grid, st, a, prod, tonly, beta2); break;
      case 8: launch_smax_fwd_nc<8>(p, grid, st, a, prod, tonly, beta2); break;
      default: launch_smax_fwd_nc<16>(p, grid, st, a, prod, tonly, beta2); break;
    }
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_soft_fwd_final, dim3((unsigned)((pop.n_sets + 63) / 64)),
                     dim3(kFwdFinalWaves * 64), 0, st,
                     a.part_loss, p.n_groups, pop.n_sets, l.ds->n, l.loss);
  return hipGetLastError();
}

hipError_t launch_smax_backward(const SoftLaunch &l, float beta, hipStream_t st) {
  const PopRec &pop = *l.pop;
  if (pop.n_sets == 0) return hipSuccess;
  const SoftPlan p = plan_smax_backward(*l.ds, pop);
  if (p.lds > kDynLdsMax) return hipErrorInvalidValue;
  SoftArgs a;
  fill_args(a, l, p);
  a.part_grad = static_cast<float *>(l.ws);
  uint4 *crec = reinterpret_cast<uint4 *>(static_cast<char *>(l.ws) + soft_part_bytes(*l.ds, pop, true));
  a.crec = crec;
  hipError_t e = launch_prep(l, a, crec, st);
  if (e != hipSuccess) return e;
  const float beta2 = beta * kLog2e;
  if (p.n_groups > 0) {
    const dim3 grid((unsigned)((pop.n_sets + p.Q - 1) / p.Q), (unsigned)p.n_groups);
    const bool prod = pop.max_rule_conds <= kProdMaxConds, tonly = pop.n_ff == 0 && pop.n_cat == 0;
    switch (smax_nc(l.ds->nc)) {
      case 2: launch_smax_bwd_nc<2>(p, grid, st, a, prod, tonly, beta, beta2); break;
      case 4: launch_smax_bwd_nc<4>(p, grid, st, a, prod, tonly, beta, beta2); break;
      case 8: launch_smax_bwd_nc<8>(p, grid, st, a, prod, tonly, beta, beta2); break;
      default: launch_smax_bwd_nc<16>(p, grid, st, a, prod, tonly, beta, beta2); break;
    }
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_soft_bwd_final, dim3((unsigned)pop.n_sets), dim3(64), 0, st, a.part_grad,
                     p.n_groups, pop.n_conds, pop.ssets, pop.sconds, l.ds->inv_tau, l.dloss,
                     l.ds->n, l.dcoef, l.dcoef2, l.dtheta);
  return hipGetLastError();
}

hipError_t launch_smax_proba(const SoftLaunch &l, int32_t set, float beta, const float *rows,
                             int64_t n, float *probs, hipStream_t st) {
  const PopRec &pop = *l.pop;
  if (n <= 0) return hipSuccess;
  SoftArgs a;
  fill_args(a, l, plan_forward(*l.ds, pop));
  uint4 *crec = reinterpret_cast<uint4 *>(static_cast<char *>(l.ws) + soft_part_bytes(*l.ds, pop, false));
  a.crec = crec;
  hipError_t e = launch_prep(l, a, crec, st);
  if (e != hipSuccess) return e;
  const float beta2 = beta * kLog2e;
  const dim3 grid((unsigned)((n + 255) / 256)), block(256);
  const int nc = l.ds->nc;
  switch (smax_nc(nc)) {
    case 2:
      hipLaunchKernelGGL(k_smax_proba<2>, grid, block, 0, st, rows, n, pop.nf, nc, set, pop.sets,
                         pop.ssets, pop.rules, crec, beta2, probs);
      break;
    case 4:
      hipLaunchKernelGGL(k_smax_proba<4>, grid, block, 0, st, rows, n, pop.nf, nc, set, pop.sets,
                         pop.ssets, pop.rules, crec, beta2, probs);
      break;
    case 8:
      hipLaunchKernelGGL(k_smax_proba<8>, grid, block, 0, st, rows, n, pop.nf, nc, set, pop.sets,
                         pop.ssets, pop.rules, crec, beta2, probs);
      break;
    default:
      hipLaunchKernelGGL(k_smax_proba<16>, grid, block, 0, st, rows, n, pop.nf, nc, set, pop.sets,
                         pop.ssets, pop.rules, crec, beta2, probs);
      break;
  }
  return hipGetLastError();
}

namespace {
// Scratch of the no-allocation soft forward: one copy per GPU, loaded with the
// code object.  On the host this name is only a stand-in for the symbol;
// kernels receive the device address hipGetSymbolAddress gives for it.
static __device__ __align__(256) unsigned char scratch[AERL_NOALLOC_SCRATCH_BYTES];
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t noalloc_scratch(int device, void **out) {
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  if (!g_scratch_ptr[device]) {
    void *ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[device] = ptr;
  }
  *out = g_scratch_ptr[device];
  return hipSuccess;
}

hipError_t launch_soft_adjoint(const SoftLaunch &l, bool gather, SoftParts *out, hipStream_t st) {
  const PopRec &pop = *l.pop;
  const SoftPlan p = plan_backward(*l.ds, pop);
  if (p.lds > kDynLdsMax) return hipErrorInvalidValue;
  SoftArgs a;
  fill_args(a, l, p);
  a.part_grad = static_cast<float *>(l.ws);
  uint4 *crec = reinterpret_cast<uint4 *>(static_cast<char *>(l.ws) + soft_part_bytes(*l.ds, pop, true));
  a.crec = crec;
  *out = SoftParts{a.part_grad, crec, p.n_groups};
  const hipError_t e0 = gather ? launch_prep(l, a, crec, st) : hipSuccess;
  if (e0 != hipSuccess) return e0;
  if (p.n_groups > 0) {
    const dim3 grid((unsigned)((pop.n_sets + p.Q - 1) / p.Q), (unsigned)p.n_groups);
    const bool prod = pop.max_rule_conds <= kProdMaxConds, tonly = pop.n_ff == 0 && pop.n_cat == 0;
    if (p.reg && prod && tonly) {
      launch_bwd_reg<RuleProd, true>(p, grid, st, a);
    } else if (p.reg && prod) {
      launch_bwd_reg<RuleProd, false>(p, grid, st, a);
    } else if (p.reg && tonly) {
      launch_bwd_reg<RuleAcc, true>(p, grid, st, a);
    } else if (p.reg) {
      launch_bwd_reg<RuleAcc, false>(p, grid, st, a);
    } else {
      hipLaunchKernelGGL(k_soft_bwd, grid, dim3(p.waves * 64), p.lds, st, a);
    }
  }
  return hipGetLastError();
}

hipError_t launch_soft_backward(const SoftLaunch &l, hipStream_t st) {
  const PopRec &pop = *l.pop;
  if (pop.n_sets == 0) return hipSuccess;
  SoftParts p;
  const hipError_t e = launch_soft_adjoint(l, true, &p, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_soft_bwd_final, dim3((unsigned)pop.n_sets), dim3(64), 0, st, p.grad, p.n_groups,
                     pop.n_conds, pop.ssets, pop.sconds, l.ds->inv_tau, l.dloss, l.ds->n, l.dcoef,
                     l.dcoef2, l.dtheta);
  return hipGetLastError();
}

}  // namespace aerl
