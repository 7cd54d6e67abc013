// Arithmetic of the sigmoid relaxation shared by the soft kernels (soft.hip)
// and the fine-tuning kernel (tune.hip).
#pragma once

#include "eval_core.h"
#include "internal.h"
#include "soft_plan.h"

namespace aerl {

namespace {

// Log-domain quantities inside the kernels are in bits (base-2 logs): the
// hardware computes 2^x (v_exp_f32) and log2(x) (v_log_f32) directly, so the
// inner loops carry no scaling multiplies.  A condition value is evaluated as
// z2 = z * log2(e); the loss is converted back to nats at the end.
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kNegInf = -__builtin_huge_valf();
constexpr float kLossCap = 100.0f;  // nats

__device__ __forceinline__ float fexp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float flog2(float x) { return __builtin_amdgcn_logf(x); }
__device__ __forceinline__ float frcp(float x) { return __builtin_amdgcn_rcpf(x); }

// log2(1 + u) for u in [0, 1]: w = 1 + u is rounded; (w - 1) - u is that
// rounding error exactly, which corrects log2(w) to first order.
__device__ __forceinline__ float log2_1p_unit(float u) {
  const float w = 1.0f + u;
  return fmaf(-((w - 1.0f) - u), kLog2e, flog2(w));
}

// Per-rule accumulator of the soft truth: a = log2 r = sum_j log2 sigmoid(z_j),
// and us = sum_j 2^(kShift2 - |z2_j|).  When every condition holds strongly,
// a is so close to 0 that fp32 cannot carry -a (it underflows near 2^-126),
// yet log(1 - r) ~ log(sum_j e^-z_j) still matters down to the loss clamp
// (e^-100); the shifted sum keeps it (normal floats down to z ~ 150).  The
// shift is a power of two, so unscaling it is exact.
constexpr float kShift2 = 92.0f;
constexpr float kExp2NegShift = 0x1p-92f;
struct RuleAcc {
  // add() of a larger z2 changes nothing: kShift2 - z2 < -126, where
  // v_exp_f32 gives 0 (it flushes results below the normal range, measured)
  static constexpr float kNoop = 219.0f;
  float a = 0.0f, us = 0.0f;
  // Adds condition value z2; returns log2(1 + 2^-|z2|), from which
  // -log2 sigmoid(+-z) = max(-+z2, 0) + that.
  __device__ __forceinline__ float add(float z2) {
    const float e_s = fexp2(kShift2 - fabsf(z2));
    const float lp = log2_1p_unit(e_s * kExp2NegShift);
    a -= fmaxf(-z2, 0.0f) + lp;
    us += e_s;
    return lp;
  }
  // add's return value for z2, without adding the condition
  __device__ static __forceinline__ float term(float z2) {
    return log2_1p_unit(fexp2(kShift2 - fabsf(z2)) * kExp2NegShift);
  }
};

// 1 - 2^a for a <= 0 (bits).  Near 0 uses Kahan's form of expm1,
// 2^a - 1 = (u - 1) * a / log2(u) with u = 2^a, which cancels the rounding
// of u.
__device__ __forceinline__ float one_minus_exp2(float a) {
  const float u = fexp2(a);
  if (a > -1.0f) {
    const float lu = flog2(u);
    const float em1 = (u == 1.0f) ? a * kLn2 : (u - 1.0f) * (a * frcp(lu));
    return -em1;
  }
  return 1.0f - u;
}

// log2(1 - 2^a) for a <= 0 (a = 0 gives -inf).
__device__ __forceinline__ float log1mexp2(float a) { return flog2(one_minus_exp2(a)); }

// log2(1 - r) of a rule: from a while fp32 represents -a well, otherwise from
// the shifted sum (there 1 - r = sum_j e^-z_j to within a relative 1e-30).
__device__ __forceinline__ float rule_log_miss(const RuleAcc &r) {
  return r.a > -1e-30f ? flog2(r.us) - kShift2 : log1mexp2(r.a);
}

// log2(2^p + 2^q), -inf safe.
__device__ __forceinline__ float lse(float p, float q) {
  float m;  // fmaxf(p, q); p and q are never NaN, so no canonicalizing copies
  asm("v_max_f32 %0, %1, %2" : "=v"(m) : "v"(p), "v"(q));
  if (m == kNegInf) return kNegInf;
  return m + log2_1p_unit(fexp2(-fabsf(p - q)));
}

// Interface shared by the two accumulators below:
//   add(z2)                 adds a condition, returns a per-condition value t
//   sig_neg(pre, z2, t)     2^pre * sigmoid(-z) for that condition
//   finish(a2, b2)          a2 = log2 r, b2 = log2(1 - r) of the rule
__device__ __forceinline__ void acc_finish(const RuleAcc &r, float &a2, float &b2) {
  a2 = r.a;
  b2 = rule_log_miss(r);
}
__device__ __forceinline__ float acc_log_r(const RuleAcc &r) { return r.a; }
__device__ __forceinline__ float acc_sig_neg(const RuleAcc &, float pre, float z2, float lp) {
  return fexp2(pre - (fmaxf(z2, 0.0f) + lp));
}

// log2(1 + p) for any p >= 0 (first-order correction of the rounding of
// w = 1 + p, as in log2_1p_unit).
__device__ __forceinline__ float log2_1p(float p) {
  const float w = 1.0f + p;
  return fmaf(-((w - 1.0f) - p) * frcp(w), kLog2e, flog2(w));
}

// Product form of a rule's soft truth, for rules of at most kProdMaxConds
// conditions.  With u_j = e^-|z_j| and M = sum_j max(-z_j, 0),
//   r = e^-M / prod_j (1 + u_j),  p = prod_j (1 + u_j) - 1 >= 0,
//   log r = -M - log1p(p),  1 - r = (p + (1 - e^-M)) / (1 + p),
// and p is built by p <- p (1 + u) + u from non-negative terms (1 + u
// rounded once), so it keeps full relative accuracy (also when r is within
// e^-100 of 1) with one exponential per condition; the logarithms are taken
// once per rule.  p is
// kept scaled by 2^64 (pt), so that u down to 2^-190 stays a normal float;
// with at most 60 conditions pt < 2^124.
// min(v, 0) in one v_min_f32.  fminf on a value the compiler cannot prove
// canonical (here a product carried across the wave reductions' branches)
// gets a canonicalizing copy first; no signaling NaN reaches this point, so
// the copy changes nothing and is left out.
__device__ __forceinline__ float min0(float v) {
  float r;
  asm("v_min_f32 %0, 0, %1" : "=v"(r) : "v"(v));
  return r;
}

struct RuleProd {
  static constexpr float kNoop = 191.0f;  // 64 - z2 < -126: as RuleAcc's
  float m = 0.0f, pt = 0.0f;  // m = M in bits, pt = p * 2^64
  // returns 1 + u, rounded once
  __device__ __forceinline__ float add(float z2) {
    const float ut = fexp2(64.0f - fabsf(z2));  // u * 2^64
    const float w = fmaf(ut, 0x1p-64f, 1.0f);
    // p' = p (1 + u) + u: rounding 1 + u first moves the product by at most
    // one rounding of it (a term of p' that is at least p), so p' keeps the
    // accuracy of two roundings while sharing 1 + u with the sigmoid
    pt = fmaf(pt, w, ut);
    m -= min0(z2);  // m += max(-z2, 0), the same value bit for bit
    return w;
  }
  // add's return value for z2, without adding the condition
  __device__ static __forceinline__ float term(float z2) {
    return fmaf(fexp2(64.0f - fabsf(z2)), 0x1p-64f, 1.0f);
  }
};
// log2(x * 2^-64) for x >= 0, from the exact exponent and the mantissa, so
// that a result near -64 carries no rounding of 64.
__device__ __forceinline__ float log2_scaled64(float x) {
  const float mant = __builtin_amdgcn_frexp_mantf(x);  // [0.5, 1), or 0
  const int e = __builtin_amdgcn_frexp_expf(x);
  return flog2(mant) + (float)(e - 64);
}

// a2 = log2 r = -M - log2(1 + p) is accurate in every regime.  b2 = log2(1 - r)
// follows from a2 while r is not within 2^-60 of 1; closer than that, from
// 1 - r = (p + (1 - e^-M)) / (1 + p) with p kept scaled (p may be far below
// the normal range there).
__device__ __forceinline__ void acc_finish(const RuleProd &r, float &a2, float &b2) {
  const float l1p = log2_1p(r.pt * 0x1p-64f);
  a2 = -r.m - l1p;
  b2 = a2 > -0x1p-60f ? log2_scaled64(fmaf(one_minus_exp2(-r.m), 0x1p64f, r.pt)) - l1p
                       : log1mexp2(a2);
}
// a2 alone, the same value as acc_finish's
__device__ __forceinline__ float acc_log_r(const RuleProd &r) {
  return -r.m - log2_1p(r.pt * 0x1p-64f);
}
__device__ __forceinline__ float acc_sig_neg(const RuleProd &, float pre, float z2, float w) {
  return fexp2(pre - fmaxf(z2, 0.0f)) * frcp(w);
}

// Loss of one sample in nats from log2 P_y.
__device__ __forceinline__ float sample_loss(float logpy2) { return fminf(-logpy2 * kLn2, kLossCap); }

// Sum of v over the wave, left in lane 63: an inclusive scan inside each
// 16-lane row (row_shr 1, 2, 4, 8), then the row totals carried forward
// with row_bcast 15 and 31.  A fixed order, so bit-identical from run to run.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_add(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROW_MASK, 0xf, true));
}
__device__ __forceinline__ float wave_total_last(float v) {
  v = dpp_add<0x111, 0xf>(v);
  v = dpp_add<0x112, 0xf>(v);
  v = dpp_add<0x114, 0xf>(v);
  v = dpp_add<0x118, 0xf>(v);
  v = dpp_add<0x142, 0xa>(v);
  v = dpp_add<0x143, 0xc>(v);
  return v;
}

// Wave totals of four values at once, each ending in lane 15 of one row:
// row 0 the total of a0, row 1 of b0, row 2 of a1, row 3 of b1.  The
// half-wave swaps pair lane l with l + 32 (a0 with a1, b0 with b1 in the two
// halves), then rows with the row 16 lanes on; an inclusive scan in each
// row finishes.  A fixed order, so bit-identical from run to run.
__device__ __forceinline__ float wave_totals4(float a0, float a1, float b0, float b1) {
  const auto sa = __builtin_amdgcn_permlane32_swap(__float_as_uint(a0), __float_as_uint(a1), false, false);
  const auto sb = __builtin_amdgcn_permlane32_swap(__float_as_uint(b0), __float_as_uint(b1), false, false);
  // lanes 0-31: a0 (b0) over lanes l and l + 32; lanes 32-63: a1 (b1)
  const float pa = __uint_as_float(sa[0]) + __uint_as_float(sa[1]);
  const float pb = __uint_as_float(sb[0]) + __uint_as_float(sb[1]);
  const auto sr = __builtin_amdgcn_permlane16_swap(__float_as_uint(pa), __float_as_uint(pb), false, false);
  // rows 0 and 2: pa over a row and the next; rows 1 and 3: pb
  float v = __uint_as_float(sr[0]) + __uint_as_float(sr[1]);
  v = dpp_add<0x111, 0xf>(v);
  v = dpp_add<0x112, 0xf>(v);
  v = dpp_add<0x114, 0xf>(v);
  v = dpp_add<0x118, 0xf>(v);
  return v;
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
  return v;
}

// A categorical condition has no parameter to relax: its soft truth is its
// truth, z = +inf (x[f] is a code k in 0..63 with bit k of the mask {lo, hi}
// set) or -inf.
__device__ __forceinline__ float cat_z(float v, uint32_t lo, uint32_t hi) {
  const bool ok = v >= 0.0f && v <= 63.0f && v == truncf(v);  // NaN fails
  const int code = ok ? (int)v : 0;
  const uint32_t word = code < 32 ? lo : hi;
  const bool in = ok && ((word >> (code & 31)) & 1u) != 0u;
  return in ? __builtin_huge_valf() : -__builtin_huge_valf();
}

// Per-condition record {sconds, coef, theta or coef2, +-log2(e)/tau_f}: the
// operand of the right-hand side is theta for a threshold and coef2 for a
// feature-vs-feature condition, the scale's sign the direction's; a
// categorical condition's code set replaces the parameters.
__device__ __forceinline__ uint4 cond_record(uint32_t sc, const float *__restrict__ inv_tau,
                                             const float *__restrict__ coef,
                                             const float *__restrict__ coef2,
                                             const float *__restrict__ theta,
                                             const uint2 *__restrict__ cmask, int64_t j) {
  if (sc & kSoftCat) {
    const uint2 m = cmask[j];
    return make_uint4(sc, m.x, m.y, 0u);
  }
  const float inv = inv_tau[sc & 0xfffu] * kLog2e;
  const float sinv = ((sc >> 25) & 1u) ? inv : -inv;
  const float rv = (sc & kSoftFF) ? coef2[j] : theta[j];
  return make_uint4(sc, __float_as_uint(coef[j]), __float_as_uint(rv), __float_as_uint(sinv));
}

// A record whose z2 is NaN for some sample, or on the zeros of the padding: a
// parameter that is NaN, or but for a threshold infinite.  The first record of
// a rule set that holds one carries kRecOdd in x.
constexpr uint32_t kRecOdd = 1u << 31;
__device__ __forceinline__ bool record_odd(uint4 r) {
  if (r.x & kSoftCat) return false;
  const float c = __uint_as_float(r.y), rv = __uint_as_float(r.z), sinv = __uint_as_float(r.w);
  return !(__builtin_isfinite(c) && __builtin_isfinite(sinv) &&
           ((r.x & kSoftFF) ? __builtin_isfinite(rv) : rv == rv));
}

// Sums a condition's partial gradients [n_groups][n_conds][2] in group order,
// eight loads in flight at a time.
__device__ __forceinline__ void sum_groups(const float *__restrict__ part, int n_groups,
                                           int n_conds, int j, double &g0, double &g1) {
  g0 = g1 = 0.0;
  int g = 0;
  for (; g + 8 <= n_groups; g += 8) {
    float2 v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k)
      v[k] = *reinterpret_cast<const float2 *>(part + ((int64_t)(g + k) * n_conds + j) * 2);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      g0 += (double)v[k].x;
      g1 += (double)v[k].y;
    }
  }
  for (; g < n_groups; ++g) {
    const float *pp = part + ((int64_t)g * n_conds + j) * 2;
    g0 += (double)pp[0];
    g1 += (double)pp[1];
  }
}

// Gradients of one condition's coefficient and right-hand operand from its
// sums over the samples g0 = sum dL/dz x_g (1 for a threshold) and g1 =
// sum dL/dz x_f: dz/dparam = +-x/tau, -+1/tau, and dloss/N.
__device__ __forceinline__ void param_grads(uint32_t sc, const float *__restrict__ inv_tau, double g0,
                                            double g1, double scale, float &dcoef, float &drhs) {
  const double sinv = (((sc >> 25) & 1u) ? 1.0 : -1.0) * (double)inv_tau[sc & 0xfffu];
  dcoef = (float)(sinv * g1 * scale);
  drhs = (float)(-sinv * g0 * scale);
}

// Per-rule state of a lane's S samples for up to R rules, indexed by the rule:
// private memory, the address the same for the whole wave.  Rules run fastest,
// so that a rule's S values are S single accesses: one of 4 S bytes would need
// its registers in a row, which the adjoints at 64 VGPRs do not have.
template <int S, int R>
struct RuleState {
  float v[S][R];
  __device__ __forceinline__ void get(int k, float (&out)[S]) const {
#pragma unroll
    for (int s = 0; s < S; ++s) out[s] = v[s][k];
  }
  __device__ __forceinline__ void set(int k, const float (&in)[S]) {
#pragma unroll
    for (int s = 0; s < S; ++s) v[s][k] = in[s];
  }
};

}  // namespace

}  // namespace aerl
