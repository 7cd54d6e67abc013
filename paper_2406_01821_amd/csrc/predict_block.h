// One block's share of a prediction: 64 S consecutive rows of a row-major
// request, evaluated with one rule set (Section 3: step activation, AND of
// conditions, first firing rule, else the default class).  Shared by the
// single-request kernel and the batched one.
//
// A request is a few thousand rows at most, so its time is the latency of
// one block: staging and a chain of dependent record reads.  All waves stage
// the rows (coalesced, into rows of odd pitch, so that lane = row reads a
// feature without bank conflicts), then wave w takes rules w, w + waves, ...
// for the same rows, and the first firing rule of each row is the minimum
// over the waves.  S = 4 rows per lane share each record's reads where a
// request is large enough for throughput to count.  4096 rows x 64 features,
// a rule set of up to 32 rules: 9.4 us per call (launch-bound) against 47 us
// with one wave per 256 rows walking every rule in turn.
#pragma once

#include "eval_core.h"

namespace aerl {

constexpr int kPredictRows = 64;
// Row pitch of the staged rows in floats, and their LDS.
__host__ __device__ inline int predict_pitch(int nf) { return nf | 1; }
inline size_t predict_lds(int nf, int S = 1) { return (size_t)kPredictRows * S * predict_pitch(nf) * 4; }

// ok[s] &= the row at x + 64 s pitch passes a record (the forms of
// eval_core.h); false when none does.
template <int S>
__device__ __forceinline__ bool take_record(uint4 r, const float *x, int pitch, bool (&ok)[S]) {
  const float *xf = x + (r.x >> 10);
  const float y = __uint_as_float(r.y), z = __uint_as_float(r.z);
  const uint32_t w = r.w;
  float v[S];
#pragma unroll
  for (int s = 0; s < S; ++s) v[s] = xf[64 * s * pitch];
  auto each = [&](auto holds) {
    bool any = false;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      ok[s] = ok[s] && holds(s);
      any = any || ok[s];
    }
    return any;
  };
  if (w & kRecFF) {
    const float *xg = x + (w & kRecGMask);
    if (w & kRecGE) return each([&](int s) { return y * v[s] >= z * xg[64 * s * pitch]; });
    return each([&](int s) { return y * v[s] > z * xg[64 * s * pitch]; });
  }
  if (!(w & (kRecAlways | kRecMul | kRecCat))) {
    if (w & kRecLE) return each([&](int s) { return v[s] <= y; });
    return each([&](int s) { return v[s] >= y; });
  }
  if (w & kRecAlways) return each([&](int) { return true; });
  if (w & kRecMul) return each([&](int s) { return y * v[s] > z; });
  return each([&](int s) {
    if (!(v[s] >= 0.0f && v[s] <= 63.0f && v[s] == truncf(v[s]))) return false;
    const int code = (int)v[s];
    return ((code < 32 ? r.y : r.z) >> (code & 31) & 1u) != 0u;
  });
}

// Rows [base, base + 64 S) of the n rows, lane l taking rows l, l + 64, ...
// xs: predict_lds(nf, S) of LDS; first: 64 S words.  Called by a block of
// whole waves.
template <int S>
__device__ __forceinline__ void predict_block(const float *__restrict__ rows, int64_t n, int32_t nf,
                                              const int4 set, const uint4 *__restrict__ conds,
                                              const uint4 *__restrict__ heads,
                                              int32_t *__restrict__ out, int64_t base, float *xs,
                                              int32_t *first) {
  constexpr int32_t kNone = INT32_MAX;
  const int t = threadIdx.x, lane = t & 63, waves = (int)blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int pitch = predict_pitch(nf);
  const int m = (int)min((int64_t)kPredictRows * S, n - base);
  const float *src = rows + base * nf;
  // row of word i: i / nf, exact for i < 256 * 512 through the rounded-up
  // reciprocal (its excess times i stays below 2^32)
  const uint32_t magic = nf > 1 ? 0xffffffffu / (uint32_t)nf + 1u : 0u;
  for (int i = t; i < m * nf; i += (int)blockDim.x) {
    const int r = magic ? (int)__umulhi((uint32_t)i, magic) : i;
    xs[r * pitch + i - r * nf] = src[i];
  }
  for (int i = t; i < kPredictRows * S; i += (int)blockDim.x) first[i] = kNone;
  __syncthreads();
  const float *x = xs + lane * pitch;
  const int rules = (set.y >> 16) - 1;
  const uint4 *recs = conds + set.x;
  for (int k = wave; k < rules; k += waves) {
    // a row that an earlier rule is known to take is out, for later rules too
    // (others may still be in flight: the minimum decides)
    bool ok[S], any = false;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      ok[s] = lane + 64 * s < m && *(volatile int32_t *)&first[lane + 64 * s] > (k << 6);
      any = any || ok[s];
    }
    if (ballot(any) == 0) break;
    // the record after the current one is requested with it (the stream ends
    // with a spare record)
    uint32_t at = ldc(heads, set.x + k).x & kHeadOffMask;
    uint4 r, ahead = ldc_at(recs, at);
    do {
      r = ahead;
      at += 16u;
      ahead = ldc_at(recs, at);
      any = take_record<S>(r, x, pitch, ok);
    } while (!(r.w & kRecLast) && ballot(any) != 0);
    const int32_t key = k << 6 | (int32_t)(r.w >> kRecClsShift & 63u);  // rule, class
#pragma unroll
    for (int s = 0; s < S; ++s)
      if (ok[s]) atomicMin(&first[lane + 64 * s], key);
  }
  __syncthreads();
  for (int i = t; i < m; i += (int)blockDim.x)
    out[base + i] = first[i] == kNone ? set.z : first[i] & 63;
}

// The same for rows [base, base + 256), by one wave with four rows per lane and
// the counting path's walk (rules in turn until every row is decided): the
// least work per row, for requests whose rows alone fill the GPU.  Few features
// only: LDS holds a kilobyte of rows per feature and wave.  The row of a word
// comes from a multiplication (2^18 x 8 10.2 -> 8.2 us against a division).
// xs: predict_walk_lds(nf) of LDS.  Called by a 64-thread block.
inline size_t predict_walk_lds(int nf) { return (size_t)nf * 256 * 4; }
__device__ __forceinline__ void predict_walk(const float *__restrict__ rows, int64_t n, int32_t nf,
                                             const int4 set, const uint4 *__restrict__ conds,
                                             int32_t *__restrict__ out, int64_t base, float *xs) {
  constexpr int S = 4, TS = 64 * S;
  const int lane = threadIdx.x;
  const int m = (int)min((int64_t)TS, n - base);
  const float *src = rows + base * nf;
  const uint32_t magic = nf > 1 ? 0xffffffffu / (uint32_t)nf + 1u : 0u;  // as above
  for (int i = lane; i < TS * nf; i += 64) {
    const int r = magic ? (int)__umulhi((uint32_t)i, magic) : i;
    xs[(i - r * nf) * TS + r] = r < m ? src[i] : 0.0f;
  }
  __syncthreads();
  uint64_t vm[S];
  int pred[S];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    vm[s] = ballot(lane * S + s < m);
    pred[s] = set.z;
  }
  const uint32_t lds_lane =
      (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) float *)xs + (uint32_t)lane * (4u * S);
  eval_set_pred4(lds_lane, set, conds, vm, pred);
#pragma unroll
  for (int s = 0; s < S; ++s)
    if (lane * S + s < m) out[base + lane * S + s] = pred[s];
}

}  // namespace aerl
