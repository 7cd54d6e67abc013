// On-device fine-tuning of a population's coefficients and thresholds.
//
// Section 3: back-propagation through the sigmoid relaxation adjusts the
// coefficients of every rule without changing its logical structure; the
// paper applies 50 epochs of gradient updates to each candidate rule set
// (Section 4.1, the fine-tuning example of Fig. 1).  Every rule set is its
// own model: the gradient of sum_s loss[s] with respect to a condition's
// parameters is the gradient of its own rule set's loss.  One epoch here is
// one full-batch step: the adjoint over the whole resident dataset, then a
// fused optimizer update of every parameter in place.  The parameters of a
// condition are its coefficient, plus its threshold (threshold condition)
// or its second coefficient (feature-vs-feature condition); the unused one
// of the two is never written, so the structure stays exactly as packed.
#include "internal.h"
#include "soft_core.h"

namespace aerl {

namespace {

// Optimizer of a launch: Adam (Kingma and Ba) or plain gradient descent.
struct Opt {
  int32_t kind;
  float lr, b1, b2, eps;
};

// One Adam step of parameter p with bias corrections c1 = 1/(1 - beta1^t),
// c2 = 1/(1 - beta2^t):
//   m = b1*m + (1-b1)*g;  v = b2*v + (1-b2)*g^2;
//   p -= lr * (m*c1) / (sqrt(v*c2) + eps)
__device__ __forceinline__ float adam(const Opt &o, float p, float g, float &m, float &v, float c1,
                                      float c2) {
  m = o.b1 * m + (1.0f - o.b1) * g;
  v = o.b2 * v + (1.0f - o.b2) * (g * g);
  return p - o.lr * (m * c1) / (sqrtf(v * c2) + o.eps);
}

// One epoch's end for tables the adjoint kernel runs on: a condition per
// thread sums its partial gradients (dloss = 1), updates (coef, rhs), rhs =
// theta or coef2 by kind, in place and writes the record the next epoch's
// adjoint reads, in one launch instead of three (sums 4.7, update 4.6,
// records 2-5 us; 50 epochs of 100 rule sets on 3000 x 60 3.45 -> 2.83 ms).
__global__ __launch_bounds__(64) void k_tune_update(
    const SoftParts p, const uint32_t *__restrict__ sconds, const float *__restrict__ inv_tau,
    const int4 *__restrict__ ssets, const int4 *__restrict__ rules, int32_t n_sets, int32_t n_rules,
    int32_t n_conds, int64_t n, float *__restrict__ coef, float *__restrict__ coef2,
    float *__restrict__ theta, float *__restrict__ m, float *__restrict__ v, const Opt o, float c1,
    float c2) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n_conds) return;
  const uint32_t sc = sconds[j];
  if (sc & kSoftCat) return;  // a code set: nothing to tune
  double g0, g1;
  sum_groups(p.grad, p.n_groups, n_conds, j, g0, g1);
  float dc, dr;
  param_grads(sc, inv_tau, g0, g1, n > 0 ? 1.0 / (double)n : 0.0, dc, dr);
  float *rhs = (sc & kSoftFF) ? coef2 : theta;
  float c = coef[j], r = rhs[j];
  if (o.kind == AERL_OPT_ADAM) {
    const int64_t k = moment_index(1, n_conds, j);
    c = adam(o, c, dc, m[j], v[j], c1, c2);
    r = adam(o, r, dr, m[k], v[k], c1, c2);
  } else {
    c -= o.lr * dc;
    r -= o.lr * dr;
  }
  coef[j] = c;
  rhs[j] = r;
  uint4 rec = p.crec[j];
  rec.y = __float_as_uint(c);
  rec.z = __float_as_uint(r);
  p.crec[j].y = rec.y;
  p.crec[j].z = rec.z;
  if (record_odd(rec)) {
    // mark the first record of the condition's rule set: its rule is the last
    // one whose conditions start at j or before, its set the last one whose
    // rules start there or before (x is written by these marks alone)
    int lo = 0, hi = n_rules - 1;
    while (lo < hi) {
      const int mid = lo + (hi - lo + 1) / 2;
      if (rules[mid].x <= j) lo = mid;
      else hi = mid - 1;
    }
    const int rule = lo;
    lo = 0, hi = n_sets - 1;
    while (lo < hi) {
      const int mid = lo + (hi - lo + 1) / 2;
      if (ssets[mid].x <= rule) lo = mid;
      else hi = mid - 1;
    }
    atomicOr(&p.crec[ssets[lo].z].x, kRecOdd);
  }
}

// Every epoch of a rule set in one block: rule sets are models of their own,
// so nothing crosses blocks.  A small table's epoch is a few microseconds of
// work behind four launches (records, adjoint, sums, update), and its adjoint
// a chain of scalar loads by one wave per (rule set, tile) spread over few
// blocks.  Here wave (set, tile) of the block takes one wave tile of its rule
// set through the forward and the reverse sweep, with the table (when it
// fits) and the set's records in LDS; the block then sums the tiles' partial
// gradients and updates the records in place, epoch after epoch.  The same
// arithmetic as the kernels for larger tables (wave totals in fp32, tiles in
// order in fp64).  Bound by the largest rule set: its VALU work on the one
// CU.  569 x 30, 100 rule sets of 1-8 rules x 1-4 conditions, 50 epochs:
// 0.71 ms against 2.30 ms.
struct TuneSetsArgs {
  const float *x_fm;
  int64_t n_pad;
  int32_t nf, n_wt;  // wave tiles of the table
  const int32_t *tile_info;
  const float *inv_tau;
  const int4 *sets, *ssets, *rules;
  const uint32_t *sconds;
  const uint2 *cmask;
  float *coef, *coef2, *theta;
  float *m, *v;       // [2][n_conds] moments, kept between launches
  float *loss_hist;   // [epochs + 1][n_sets] or null
  int32_t n_sets, n_conds;
  int64_t n;
  int32_t ep0, ep1, epochs;  // epochs [ep0, ep1) of all
  double b1t, b2t;           // beta^ep0
  Opt opt;
  int32_t spb, max_conds;    // rule sets per block, conditions per rule set
};
template <int S, class Acc, bool XLDS, int R>
__global__ __launch_bounds__(kTuneSetsWaves * 64) void k_tune_sets(const TuneSetsArgs a) {
  constexpr int TS = 64 * S, WPT = AERL_TILE / TS;
  extern __shared__ __align__(16) char lds[];
  const int waves = (int)blockDim.x >> 6, lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  float *xl = reinterpret_cast<float *>(lds);
  const size_t nx = XLDS ? (size_t)a.nf * a.n_pad : 0;
  double *loss_w = reinterpret_cast<double *>(xl + nx);                    // [waves]
  uint4 *recs = reinterpret_cast<uint4 *>(loss_w + (waves + 1) / 2 * 2);   // [spb][max_conds]
  float4 *mom = reinterpret_cast<float4 *>(recs + a.spb * a.max_conds);    // likewise
  float2 *part = reinterpret_cast<float2 *>(mom + a.spb * a.max_conds);    // [waves][max_conds]
  if (XLDS) {
    const float4 *src = reinterpret_cast<const float4 *>(a.x_fm);
    for (size_t i = threadIdx.x; i < nx / 4; i += blockDim.x) reinterpret_cast<float4 *>(xl)[i] = src[i];
  }
  const float *x = XLDS ? xl : a.x_fm;
  const int slot = w / a.n_wt, wt = w - slot * a.n_wt;
  const int q = (int)blockIdx.x * a.spb + slot;
  const bool active = slot < a.spb && q < a.n_sets;
  const int4 ss = active ? ldc(a.ssets, q) : make_int4(0, 0, 0, 0);
  const int dflt = active ? ldc(a.sets, q).z : 0;
  const int info = ldc(a.tile_info, wt / WPT);
  const int label = info & 0xff;
  const int valid = min(max((info >> 8) - wt % WPT * TS, 0), TS);
  bool live[S];
#pragma unroll
  for (int s = 0; s < S; ++s) live[s] = lane * S + s < valid;
  const int t = (int)threadIdx.x - slot * a.n_wt * 64, nt = a.n_wt * 64;  // thread of the set's waves
  uint4 *rec = recs + slot * a.max_conds;
  float4 *mv = mom + slot * a.max_conds;
  float2 *my = part + (size_t)w * a.max_conds;
  if (active) {
    for (int i = t; i < ss.w; i += nt) {
      const int64_t j = ss.z + i;
      rec[i] = cond_record(a.sconds[j], a.inv_tau, a.coef, a.coef2, a.theta, a.cmask, j);
      mv[i] = a.ep0 == 0 ? make_float4(0.0f, 0.0f, 0.0f, 0.0f)
                         : make_float4(a.m[j], a.m[a.n_conds + j], a.v[j], a.v[a.n_conds + j]);
    }
  }
  __syncthreads();
  // Condition i of the set: its record and rows, then z2 (xg is 1 for a
  // threshold).  Apart, so that two conditions' reads are under way at once.
  struct Cond {
    uint4 r;
    uint32_t sc;
    float xf[S], xg[S];
  };
  auto row = [&](uint32_t f, float(&v)[S]) {
    const float *p = x + (uint32_t)f * (uint32_t)a.n_pad + (uint32_t)(wt * TS + lane * S);
    if constexpr (S == 4) {
      const float4 u = *reinterpret_cast<const float4 *>(p);
      v[0] = u.x; v[1] = u.y; v[2] = u.z; v[3] = u.w;
    } else if constexpr (S == 2) {
      const float2 u = *reinterpret_cast<const float2 *>(p);
      v[0] = u.x; v[1] = u.y;
    } else {
      v[0] = *p;
    }
  };
  auto fetch = [&](Cond &c) {
    c.sc = __builtin_amdgcn_readfirstlane(c.r.x);
    row(c.sc & 0xfffu, c.xf);
#pragma unroll
    for (int s = 0; s < S; ++s) c.xg[s] = 1.0f;
    if (c.sc & kSoftFF) row((c.sc >> 12) & 0xfffu, c.xg);
  };
  auto value = [&](const Cond &c, float(&z)[S]) {
    const float co = __uint_as_float(c.r.y), rv = __uint_as_float(c.r.z), sinv = __uint_as_float(c.r.w);
    if (c.sc & kSoftCat) {
#pragma unroll
      for (int s = 0; s < S; ++s) z[s] = cat_z(c.xf[s], c.r.y, c.r.z);
    } else {
      // rv * 1 is rv for a threshold
#pragma unroll
      for (int s = 0; s < S; ++s) z[s] = fmaf(co, c.xf[s], -(rv * c.xg[s])) * sinv;
    }
  };
  auto add = [&](int4 r, Acc(&ra)[S]) {
    const int j1 = r.x - ss.z + r.y;
    int j = r.x - ss.z;
    float z[S];
    for (; j + 1 < j1; j += 2) {
      Cond c0, c1;
      c0.r = rec[j];
      c1.r = rec[j + 1];
      fetch(c0);
      fetch(c1);
      value(c0, z);
#pragma unroll
      for (int s = 0; s < S; ++s) (void)ra[s].add(z[s]);
      value(c1, z);
#pragma unroll
      for (int s = 0; s < S; ++s) (void)ra[s].add(z[s]);
    }
    if (j < j1) {
      Cond c0;
      c0.r = rec[j];
      fetch(c0);
      value(c0, z);
#pragma unroll
      for (int s = 0; s < S; ++s) (void)ra[s].add(z[s]);
    }
  };
  const double scale = a.n > 0 ? 1.0 / (double)a.n : 0.0;
  double b1t = a.b1t, b2t = a.b2t;
  const int last = a.loss_hist && a.ep1 == a.epochs ? a.ep1 : a.ep1 - 1;  // epoch `epochs`: loss only
  for (int ep = a.ep0; ep <= last; ++ep) {
    const bool step = ep < a.ep1;
    if (active) {
      RuleState<S, R> L, B;
      float logpy[S], surv[S];
#pragma unroll
      for (int s = 0; s < S; ++s) { logpy[s] = kNegInf; surv[s] = 0.0f; }
      // each rule's record is requested one rule ahead (the last one twice)
      int4 ahead = ldc(a.rules, ss.x);
      for (int k = 0; k < ss.y; ++k) {
        const int4 r = ahead;
        ahead = ldc(a.rules, ss.x + min(k + 1, ss.y - 1));
        Acc ra[S];
        add(r, ra);
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
      float gate[S], U[S], loss = 0.0f;
#pragma unroll
      for (int s = 0; s < S; ++s) {
        if (dflt == label) logpy[s] = lse(logpy[s], surv[s]);
        loss += live[s] ? sample_loss(logpy[s]) : 0.0f;
        // samples whose loss is clamped (or padding) get no gradient; their
        // log P_y is replaced by 0 so that every exponent below stays finite
        const bool on = live[s] && -logpy[s] * kLn2 <= kLossCap;
        gate[s] = on ? 1.0f : 0.0f;
        logpy[s] = on ? logpy[s] : 0.0f;
        U[s] = dflt == label ? 0.0f : kNegInf;
      }
      if (a.loss_hist) {
        loss = wave_sum(loss);
        if (lane == 0) loss_w[w] = (double)loss;
      }
      for (int k = step ? ss.y - 1 : -1; k >= 0; --k) {
        const int4 r = ahead;
        ahead = ldc(a.rules, ss.x + max(k - 1, 0));
        const bool hit = r.z == label;
        float lk[S], bk[S], pre[S];
        L.get(k, lk);
        B.get(k, bk);
#pragma unroll
        for (int s = 0; s < S; ++s) {
          const float lm = hit ? log1mexp2(fminf(U[s], 0.0f)) : U[s];
          pre[s] = gate[s] != 0.0f ? lk[s] + lm - logpy[s] : kNegInf;
        }
        Acc ra[S];
        for (int j = r.x - ss.z; j < r.x - ss.z + r.y; j += 2) {
          const bool two = j + 1 < r.x - ss.z + r.y;
          float g0[2] = {-0.0f, -0.0f}, g1[2] = {-0.0f, -0.0f};
          Cond cs[2];
          cs[0].r = rec[j];
          cs[1].r = rec[two ? j + 1 : j];
          fetch(cs[0]);
          fetch(cs[1]);
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            if (c == 1 && !two) break;
            float z[S];
            value(cs[c], z);
#pragma unroll
            for (int s = 0; s < S; ++s) {
              const float u = hit ? ra[s].add(z[s]) : Acc::term(z[s]);
              const float dz = acc_sig_neg(ra[s], pre[s], z[s], u);
              g0[c] = fmaf(dz, cs[c].xg[s], g0[c]);
              g1[c] = fmaf(dz, cs[c].xf[s], g1[c]);
            }
          }
          const float tot = wave_totals4(g0[0], g0[1], g1[0], g1[1]);
          const int half = lane >> 5;
          if ((lane & 15) == 15 && (half == 0 || two))
            reinterpret_cast<float *>(my + j + half)[lane >> 4 & 1] = hit ? -tot : tot;
        }
        if (hit) {
#pragma unroll
          for (int s = 0; s < S; ++s) U[s] = lse(acc_log_r(ra[s]), bk[s] + U[s]);
        } else {
#pragma unroll
          for (int s = 0; s < S; ++s) U[s] = bk[s] + U[s];
        }
      }
    }
    __syncthreads();
    if (active) {
      if (a.loss_hist && t == 0) {
        double l = 0.0;
        for (int i = 0; i < a.n_wt; ++i) l += loss_w[slot * a.n_wt + i];
        a.loss_hist[(int64_t)ep * a.n_sets + q] = a.n > 0 ? (float)(l / (double)a.n) : 0.0f;
      }
      if (step) {
        b1t *= (double)a.opt.b1;
        b2t *= (double)a.opt.b2;
        const float c1 = (float)(1.0 / (1.0 - b1t)), c2 = (float)(1.0 / (1.0 - b2t));
        for (int i = t; i < ss.w; i += nt) {
          uint4 r = rec[i];
          if (r.x & kSoftCat) continue;  // a code set: nothing to tune
          const float2 *pp = part + (size_t)slot * a.n_wt * a.max_conds + i;
          double g0 = 0.0, g1 = 0.0;
          for (int k = 0; k < a.n_wt; k += WPT) {
            // a tile's waves in fp32, the tiles in fp64
            float2 v = pp[(size_t)k * a.max_conds];
#pragma unroll
            for (int e = 1; e < WPT; ++e) {
              const float2 u = pp[(size_t)(k + e) * a.max_conds];
              v.x += u.x;
              v.y += u.y;
            }
            g0 += (double)v.x;
            g1 += (double)v.y;
          }
          float dc, dr, c = __uint_as_float(r.y), rv = __uint_as_float(r.z);
          param_grads(r.x, a.inv_tau, g0, g1, scale, dc, dr);
          if (a.opt.kind == AERL_OPT_ADAM) {
            float4 s = mv[i];
            c = adam(a.opt, c, dc, s.x, s.z, c1, c2);
            rv = adam(a.opt, rv, dr, s.y, s.w, c1, c2);
            mv[i] = s;
          } else {
            c -= a.opt.lr * dc;
            rv -= a.opt.lr * dr;
          }
          r.y = __float_as_uint(c);
          r.z = __float_as_uint(rv);
          rec[i] = r;
        }
      }
    }
    __syncthreads();
  }
  if (!active) return;
  for (int i = t; i < ss.w; i += nt) {
    const uint4 r = rec[i];
    const int64_t j = ss.z + i;
    if (r.x & kSoftCat) continue;
    a.coef[j] = __uint_as_float(r.y);
    ((r.x & kSoftFF) ? a.coef2 : a.theta)[j] = __uint_as_float(r.z);
    if (a.ep1 < a.epochs) {
      const float4 s = mv[i];
      a.m[j] = s.x;
      a.m[a.n_conds + j] = s.y;
      a.v[j] = s.z;
      a.v[a.n_conds + j] = s.w;
    }
  }
}

__global__ void k_fill_f32(float *__restrict__ p, int64_t n, float v) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

hipError_t fill_f32(float *p, int64_t n, float v, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = std::min<int64_t>((n + 255) / 256, 4096);
  hipLaunchKernelGGL(k_fill_f32, dim3((unsigned)blocks), dim3(256), 0, st, p, n, v);
  return hipGetLastError();
}

size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

}  // namespace

TuneLayout tune_layout(const DatasetRec &ds, const PopRec &pop) {
  TuneLayout L{};
  const size_t nc = (size_t)std::max(pop.n_conds, 1);
  size_t off = 0;
  L.soft_off = off;  off = align256(off + std::max(soft_ws_bytes(ds, pop, false), soft_ws_bytes(ds, pop, true)));
  L.mom_off = off;   off = align256(off + 4 * nc * sizeof(float));
  L.total = off;
  return L;
}

namespace {

template <int S, class Acc, bool XLDS>
void launch_tune_sets_t(const TuneSetsPlan &p, const TuneSetsArgs &a, int max_rules, hipStream_t st) {
  const dim3 grid((unsigned)((a.n_sets + p.spb - 1) / p.spb)), block((unsigned)(p.spb * p.n_wt * 64));
  if (max_rules <= kFewRules)
    hipLaunchKernelGGL((k_tune_sets<S, Acc, XLDS, kFewRules>), grid, block, p.lds, st, a);
  else
    hipLaunchKernelGGL((k_tune_sets<S, Acc, XLDS, kRegRules>), grid, block, p.lds, st, a);
}

template <int S>
void launch_tune_sets(const TuneSetsPlan &p, const TuneSetsArgs &a, const PopRec &pop, hipStream_t st) {
  const bool prod = pop.max_rule_conds <= kProdMaxConds;
  if (prod && p.x_lds)
    launch_tune_sets_t<S, RuleProd, true>(p, a, pop.max_rules, st);
  else if (prod)
    launch_tune_sets_t<S, RuleProd, false>(p, a, pop.max_rules, st);
  else if (p.x_lds)
    launch_tune_sets_t<S, RuleAcc, true>(p, a, pop.max_rules, st);
  else
    launch_tune_sets_t<S, RuleAcc, false>(p, a, pop.max_rules, st);
}

// Every epoch through k_tune_sets, kTuneEpochs per launch (a launch stays in
// the milliseconds; the moments go through the workspace between them).
constexpr int32_t kTuneEpochs = 256;
hipError_t run_tune_sets(const TuneLaunch &t, const TuneSetsPlan &p, float *mom, hipStream_t st) {
  const DatasetRec &ds = *t.ds;
  const PopRec &pop = *t.pop;
  TuneSetsArgs a{};
  a.x_fm = ds.x_fm;
  a.n_pad = ds.n_pad;
  a.nf = ds.nf;
  a.n_wt = p.n_wt;
  a.tile_info = ds.tile_info;
  a.inv_tau = ds.inv_tau;
  a.sets = pop.sets;
  a.ssets = pop.ssets;
  a.rules = pop.rules;
  a.sconds = pop.sconds;
  a.cmask = pop.cmask;
  a.coef = t.coef;
  a.coef2 = t.coef2;
  a.theta = t.theta;
  a.m = mom;
  a.v = mom + 2 * (int64_t)pop.n_conds;
  a.loss_hist = t.loss_hist;
  a.n_sets = pop.n_sets;
  a.n_conds = pop.n_conds;
  a.n = ds.n;
  a.epochs = t.epochs;
  a.opt = Opt{t.optimizer, t.lr, t.beta1, t.beta2, t.eps};
  a.spb = p.spb;
  a.max_conds = std::max(pop.max_set_conds, 1);
  a.b1t = a.b2t = 1.0;
  for (a.ep0 = 0; a.ep0 < std::max(t.epochs, 1); a.ep0 = a.ep1) {
    a.ep1 = std::min(a.ep0 + kTuneEpochs, t.epochs);
    switch (p.S) {
      case 4: launch_tune_sets<4>(p, a, pop, st); break;
      case 2: launch_tune_sets<2>(p, a, pop, st); break;
      default: launch_tune_sets<1>(p, a, pop, st); break;
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    for (int32_t k = a.ep0; k < a.ep1; ++k) {
      a.b1t *= (double)t.beta1;
      a.b2t *= (double)t.beta2;
    }
    if (t.epochs == 0) break;
  }
  return hipSuccess;
}

}  // namespace

hipError_t run_finetune(const TuneLaunch &t, hipStream_t st) {
  const DatasetRec &ds = *t.ds;
  const PopRec &pop = *t.pop;
  const TuneLayout L = tune_layout(ds, pop);
  char *w = static_cast<char *>(t.ws);
  float *mom = reinterpret_cast<float *>(w + L.mom_off);
  if (const TuneSetsPlan p = plan_tune_sets(ds, pop, t.n_cu); p.use)
    return run_tune_sets(t, p, mom, st);
  const int64_t nc = pop.n_conds;
  SoftLaunch s{};
  s.ds = &ds;
  s.pop = &pop;
  s.coef = t.coef;
  s.coef2 = t.coef2;
  s.theta = t.theta;
  s.ws = w + L.soft_off;
  s.ws_bytes = L.mom_off - L.soft_off;
  hipError_t e = fill_f32(mom, 4 * nc, 0.0f, st);
  const unsigned blocks = (unsigned)((nc + 63) / 64);
  const Opt opt{t.optimizer, t.lr, t.beta1, t.beta2, t.eps};
  double b1t = 1.0, b2t = 1.0;
  for (int32_t ep = 0; e == hipSuccess && ep <= t.epochs; ++ep) {
    if (t.loss_hist) {
      s.loss = t.loss_hist + (int64_t)ep * pop.n_sets;
      e = launch_soft_forward(s, st);
      if (e != hipSuccess) break;
    }
    if (ep == t.epochs || nc == 0) continue;
    // the records stay in the workspace from epoch to epoch, unless a forward
    // pass has used it
    SoftParts p;
    e = launch_soft_adjoint(s, ep == 0 || t.loss_hist != nullptr, &p, st);
    if (e != hipSuccess) break;
    b1t *= (double)t.beta1;
    b2t *= (double)t.beta2;
    const float c1 = (float)(1.0 / (1.0 - b1t)), c2 = (float)(1.0 / (1.0 - b2t));
    hipLaunchKernelGGL(k_tune_update, dim3(blocks), dim3(64), 0, st, p, pop.sconds, ds.inv_tau,
                       pop.ssets, pop.rules, pop.n_sets, pop.n_rules, (int32_t)nc, ds.n, t.coef, t.coef2, t.theta, mom, mom + 2 * nc, opt, c1, c2);
    e = hipGetLastError();
  }
  return e;
}

}  // namespace aerl
