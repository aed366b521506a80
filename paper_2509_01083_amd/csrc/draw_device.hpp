// Device routines of the draw shared by the per-sequence kernels and the
// vocabulary-shard kernels: the draw job, fp64 helpers of the latency-bound
// steps, the combine of chunk partials, the draw-weight passes over units of
// 2048 logits (residual max(0, p - q), p, bonus exponentials, bonus argmax),
// and the inverse-CDF search over what those passes left behind.
#pragma once

#include <float.h>
#include <math.h>

#include "common.hpp"
#include "lanes.hpp"
#include "row_io.hpp"

namespace dsde {
namespace {

// The draw job as read from memory, moved to scalar registers (it is the same
// in every lane), which frees vector registers for the draw stream's loads.
__device__ __forceinline__ float uniform_f(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}
__device__ __forceinline__ DrawJob uniform_job(const DrawJob &j) {
  DrawJob u;
  u.kind = __builtin_amdgcn_readfirstlane(j.kind);
  u.accepted = __builtin_amdgcn_readfirstlane(j.accepted);
  u.target_row = __builtin_amdgcn_readfirstlane(j.target_row);
  u.draft_row = __builtin_amdgcn_readfirstlane(j.draft_row);
  u.scale = uniform_f(j.scale);
  u.mt = uniform_f(j.mt);
  u.md = uniform_f(j.md);
  u.inv_sp = uniform_f(j.inv_sp);
  u.inv_sq = uniform_f(j.inv_sq);
  u.u = uniform_f(j.u);
  u.token = __builtin_amdgcn_readfirstlane(j.token);
  return u;
}

// 2^x in double for the latency-bound steps: x = n + r with n = rint(x) and
// |r| <= 1/2; e^(r ln 2) by its Taylor series to degree 10 (remainder below
// 0.35^11 / 11! * e^0.35 < 4e-13 relative), scaled by 2^n.
__device__ __forceinline__ double exp2_taylor(double x) {
  if (!(x >= -1100.0)) return x != x ? x : 0.0;  // NaN stays NaN; below 2^-1074 is 0
  if (x > 1100.0) return HUGE_VAL;
  const double n = rint(x);
  const double y = (x - n) * kLn2;
  double p = 1.0 / 3628800.0;
  p = fma(p, y, 1.0 / 362880.0);
  p = fma(p, y, 1.0 / 40320.0);
  p = fma(p, y, 1.0 / 5040.0);
  p = fma(p, y, 1.0 / 720.0);
  p = fma(p, y, 1.0 / 120.0);
  p = fma(p, y, 1.0 / 24.0);
  p = fma(p, y, 1.0 / 6.0);
  p = fma(p, y, 0.5);
  p = fma(p, y, 1.0);
  p = fma(p, y, 1.0);
  return ldexp(p, int(n));
}

// log2 of a positive row sum in double: s = m 2^e with m in [1/2, 1); the
// hardware log2 (v_log_f32) gives y0 = log2 m to about 1.5e-7, and one
// correction step finishes it: m 2^-y0 = 1 + d with |d| < 3e-7, and
// log2(1 + d) = (d - d^2 / 2) / ln 2 up to d^3 (below 1e-20).  Used for the
// KLD, the entropy and the log-normalisers; the acceptance test takes no
// logarithm.
__device__ __forceinline__ double log2_rowsum(double s) {
  int e;
  const double m = frexp(s, &e);
  const double y0 = double(__builtin_amdgcn_logf(float(m)));
  const double d = m * exp2_taylor(-y0) - 1.0;
  return double(e) + y0 + (d - 0.5 * d * d) * (1.0 / kLn2);
}

// 1 / s in double: the hardware estimate and two Newton steps.
__device__ __forceinline__ double rcp_newton(double s) {
  double r = __builtin_amdgcn_rcp(s);
  r = fma(fma(-s, r, 1.0), r, r);
  r = fma(fma(-s, r, 1.0), r, r);
  return r;
}

// reductions inside aligned groups of G lanes (G = 8, 16, 32 or 64)
template <int G>
__device__ __forceinline__ float group_max(float v) {
  return lanes::group_reduce<G>(v, lanes::Max{});
}
template <int G>
__device__ __forceinline__ double group_sum(double v) {
  return lanes::group_reduce<G>(v, lanes::Add{});
}

// Folds the statistics (mt, md, sp, sq, a, h) of one more part of a row pair
// (a chunk, or a vocabulary slice) into a running set: both are rescaled to
// the larger reference shifts; the KL and entropy accumulators take the shift
// of the log-ratio along (a = sum 2^at (at - ad) with at, ad relative to the
// references).
__device__ __forceinline__ void fold_pair_stats(float &lmt, float &lmd, double &lsp, double &lsq, double &la,
                                                double &lh, float qmt, float qmd, double qsp, double qsq, double qa,
                                                double qh) {
  const float nt = fmaxf(lmt, qmt), nd = fmaxf(lmd, qmd);
  const double d0t = double(lmt) - nt, d0d = double(lmd) - nd;
  const double d1t = double(qmt) - nt, d1d = double(qmd) - nd;
  const double f0t = exp2_taylor(d0t), f0d = exp2_taylor(d0d), f1t = exp2_taylor(d1t), f1d = exp2_taylor(d1d);
  la = f0t * (la + lsp * (d0t - d0d)) + f1t * (qa + qsp * (d1t - d1d));
  lh = f0d * (lh + lsq * d0d) + f1d * (qh + qsq * d1d);
  lsp = f0t * lsp + f1t * qsp;
  lsq = f0d * lsq + f1d * qsq;
  lmt = nt;
  lmd = nd;
}

// The statistics of one row pair from the sets folded by the lanes of a group
// of G (a lane without a part holds lmt = -inf): rescaled to the group's
// largest reference shifts and summed, in every lane of the group.
struct PairStats {
  float mt, md;
  double sp, sq, a, h;
};
template <int G>
__device__ __forceinline__ PairStats group_pair_stats(float lmt, float lmd, double lsp, double lsq, double la,
                                                      double lh) {
  PairStats r;
  r.mt = group_max<G>(lmt);
  r.md = group_max<G>(lmd);
  r.sp = r.sq = r.a = r.h = 0.0;
  if (lmt != -INFINITY) {
    const double dt = double(lmt) - double(r.mt), dd = double(lmd) - double(r.md);
    const double ft = exp2_taylor(dt), fd = exp2_taylor(dd);
    r.sp = lsp * ft;
    r.sq = lsq * fd;
    r.a = ft * (la + lsp * (dt - dd));
    r.h = fd * (lh + lsq * dd);
  }
  r.sp = group_sum<G>(r.sp);
  r.sq = group_sum<G>(r.sq);
  r.a = group_sum<G>(r.a);
  r.h = group_sum<G>(r.h);
  return r;
}

// Combines the chunk partials of every drafted pair of one sequence (stored
// under slots slot0 + j): groups of G lanes, one pair per group, lane g of a
// group folds chunks g, g + G, ...  Results go to LDS (st_*[j] for position j;
// st_zmax, when given, receives the greedy rows' largest raw target logit).
template <int G, int WAVES>
__device__ inline void combine_pairs(const PairChunk *__restrict__ part, int64_t slot0, int32_t s, int32_t nc,
                                     const PairChunk &q0, const ChunkArg *__restrict__ chunk_arg, ChunkArg arg0,
                                     float *st_mt, float *st_md, double *st_sp, double *st_sq, double *st_a,
                                     double *st_h, int *st_bad, int *st_arg, float *st_zmax = nullptr) {
  constexpr int P = 64 / G;  // pairs per wavefront
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane % G;
  for (int32_t base = 0; base < s; base += WAVES * P) {
    const int32_t j = base + wave * P + lane / G;
    float lmt = -INFINITY, lmd = -INFINITY;
    double lsp = 0.0, lsq = 0.0, la = 0.0, lh = 0.0;
    // greedy: the largest raw logit among this lane's chunks and its token
    float lz = -INFINITY;
    int32_t larg = 0x7fffffff;
    if (j < s) {
      for (int32_t ch = g; ch < nc; ch += G) {
        // the first chunk of the first round was fetched at kernel start
        const bool pre = base == 0 && ch == g;
        const PairChunk q = pre ? q0 : part[(slot0 + j) * nc + ch];
        if (chunk_arg) {
          const ChunkArg qa = pre ? arg0 : chunk_arg[(slot0 + j) * nc + ch];
          // chunks come in ascending order: on equal maxima the earlier wins
          if (larg == 0x7fffffff || qa.zmax > lz) {
            lz = qa.zmax;
            larg = qa.idx;
          }
        }
        if (lmt == -INFINITY) {
          lmt = q.mt;
          lmd = q.md;
          lsp = q.sp;
          lsq = q.sq;
          la = q.a;
          lh = q.h;
        } else {
          fold_pair_stats(lmt, lmd, lsp, lsq, la, lh, q.mt, q.md, q.sp, q.sq, q.a, q.h);
        }
      }
    }
    const PairStats r = group_pair_stats<G>(lmt, lmd, lsp, lsq, la, lh);
    int32_t arg = 0x7fffffff;
    float zm = -INFINITY;
    if (chunk_arg) {  // the row argmax: smallest token among the chunks holding the row maximum
      zm = group_max<G>(lz);
      arg = larg != 0x7fffffff && lz == zm ? larg : 0x7fffffff;
      arg = lanes::group_reduce<G>(arg, lanes::Min{});
    }
    if (j < s && g == 0) {
      st_mt[j] = r.mt;
      st_md[j] = r.md;
      st_sp[j] = r.sp;
      st_sq[j] = r.sq;
      st_a[j] = r.a;
      st_h[j] = r.h;
      st_bad[j] = !(isfinite(r.mt) && isfinite(r.md) && isfinite(r.sp) && isfinite(r.sq) && isfinite(r.a));
      st_arg[j] = arg;
      if (st_zmax) st_zmax[j] = zm;
    }
  }
}

// ---------------------------------------------------------------------------
// draw weights, one unit at a time
// ---------------------------------------------------------------------------
//
// The draw reads a row in units of kUnit = 2048 consecutive logits, one unit
// per wavefront and step, 32 logits per lane, and keeps for every unit the
// weight totals of its four sub-blocks of 512 logits.  A wavefront needs
// nothing from its neighbours to finish a unit (the chunk totals of a wider
// layout need a barrier or four times the logits per wavefront), so the units
// of one row can be dealt to any number of workgroups.  Lane l owns slots
// i = 0..31 of its unit:
//   bf16 rows        : logit 2048 u + 512 (i / 8) + 8 l + i % 8   (4 loads of 16 bytes)
//   fp32 rows        : logit 2048 u + 256 (i / 4) + 4 l + i % 4   (8 loads of 16 bytes)
//   rows below 16 B  : as bf16, 32 scalar loads
// Every wavefront load is contiguous, and slots 8 g .. 8 g + 7 lie in
// sub-block g in every layout.
constexpr int kUnitElts = kUnit / 64;
constexpr int kSubs = 4;
constexpr int kSubLen = kUnit / kSubs;

template <int DT, int ROW>
__device__ __forceinline__ int64_t unit_token(int64_t unit, int i, int lane) {
  if constexpr (ROW != kScalarRows && DT == DSDE_FP32) return unit * kUnit + (i / 4) * 256 + 4 * lane + (i % 4);
  return unit * kUnit + (i / 8) * 512 + 8 * lane + (i % 8);
}

// One row's logits of a unit.  issue() loads them from inside the row, so no
// load branches; place() puts the last load's logits in their places and pads
// past V.  Callers that read two rows issue both before they place either.
template <int DT, int ROW>
struct UnitRow {
  static constexpr bool kScalar = ROW == kScalarRows;
  static constexpr bool kBf16 = DT == DSDE_BF16;
  float z[kScalar ? kUnitElts : 1];
  u32x4_t h[!kScalar && kBf16 ? 4 : 1];
  f32x4_t f[!kScalar && !kBf16 ? 8 : 1];
  __device__ __forceinline__ void issue(const char *row, int64_t V, int32_t unit, int lane) {
    if constexpr (kScalar) {
#pragma unroll
      for (int i = 0; i < kUnitElts; ++i) {
        const int64_t v = unit_token<DT, ROW>(unit, i, lane);
        z[i] = load_logit(row, DT, v < V ? v : V - 1);
      }
    } else if constexpr (kBf16) {
#pragma unroll
      for (int g = 0; g < 4; ++g) h[g] = load_words<ROW>(row, uint32_t(V), uint32_t(unit) * 256u + 64u * g + lane);
    } else {
#pragma unroll
      for (int g = 0; g < 8; ++g) f[g] = load_quad<ROW>(row, uint32_t(V), uint32_t(unit) * 512u + 64u * g + lane);
    }
  }
  __device__ __forceinline__ void place(int64_t V, int32_t unit, int lane) {
    if constexpr (kScalar) {
#pragma unroll
      for (int i = 0; i < kUnitElts; ++i)
        if (unit_token<DT, ROW>(unit, i, lane) >= V) z[i] = kPadF32;
    } else if constexpr (kBf16) {
#pragma unroll
      for (int g = 0; g < 4; ++g) place_words<ROW>(h[g], uint32_t(V), uint32_t(unit) * 256u + 64u * g + lane);
    } else {
#pragma unroll
      for (int g = 0; g < 8; ++g) place_quad<ROW>(f[g], uint32_t(V), uint32_t(unit) * 512u + 64u * g + lane);
    }
  }
  __device__ __forceinline__ float at(int i) const {
    if constexpr (kScalar) return z[i];
    if constexpr (kBf16) {
      const uint32_t x = h[i >> 3][(i >> 1) & 3];
      return (i & 1) ? bf_hi(x) : bf_lo(x);
    }
    return f[i >> 2][i & 3];
  }
};

// What a unit's pass leaves behind, in two arrays per sequence: sub[4 u + g],
// the weight total of sub-block g, and ref[u].  Bonus rows: ref is the
// reference their exponentials are taken against, max(z) c of the unit, or,
// for a greedy row, its largest raw logit, with idx the smallest (row-local)
// token holding it; a NaN ref marks a NaN or infinite logit in the unit.
// Residual and p totals need no reference and leave ref unwritten.
struct UnitCells {
  float *sub;
  UnitRef *ref;
};

// The draw weights, each evaluated by one routine wherever it is needed (the
// unit totals and the final scan), with no contraction of the product into
// a neighbouring sum, so that both places see the same bits.
__device__ __forceinline__ float residual_weight(float zt, float zd, const DrawJob &job) {
#pragma clang fp contract(off)
  const float p = fast_exp2(fmaf(zt, job.scale, -job.mt)) * job.inv_sp;
  // p - q as one fused operation: p - 2^(z_d c - md) / S_q
  return fmaxf(fmaf(-fast_exp2(fmaf(zd, job.scale, -job.md)), job.inv_sq, p), 0.0f);  // padding: 0
}
__device__ __forceinline__ float target_p_weight(float zt, const DrawJob &job) {
#pragma clang fp contract(off)
  return fast_exp2(fmaf(zt, job.scale, -job.mt)) * job.inv_sp;
}
__device__ __forceinline__ float bonus_weight(float z, float scale, float ref) {
  return fast_exp2(fmaf(z, scale, -ref));
}

// Sums a lane's 32 weights f(i) into its four sub-block sums, and those over
// the wavefront: lane l receives the total of sub-block l % 4.
template <typename F>
__device__ __forceinline__ float unit_totals(F f) {
  float a[kSubs];
#pragma unroll
  for (int g = 0; g < kSubs; ++g) {
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) s += f(8 * g + e);
    a[g] = s;
  }
  return lanes::wave_sum4(a);
}
__device__ __forceinline__ void store_totals(float total, float *sub, int32_t unit) {
  const int lane = threadIdx.x & 63;
  if (lane < kSubs) sub[int64_t(unit) * kSubs + lane] = total;
}

// Residual weights max(0, p - q) of one unit of the rejected pair.
template <int DT, int ROW>
__device__ __forceinline__ void residual_unit(const char *trow, const char *drow, int64_t V, int32_t unit,
                                              const DrawJob &job, const UnitCells &c) {
  const int lane = threadIdx.x & 63;
  UnitRow<DT, ROW> t, d;
  t.issue(trow, V, unit, lane);
  d.issue(drow, V, unit, lane);
  t.place(V, unit, lane);
  d.place(V, unit, lane);
  store_totals(unit_totals([&](int i) { return residual_weight(t.at(i), d.at(i), job); }), c.sub, unit);
}

// p of one unit of the rejected pair's target row (the draw's fallback when
// the residual has no mass).
template <int DT, int ROW>
__device__ __forceinline__ void target_p_unit(const char *trow, int64_t V, int32_t unit, const DrawJob &job,
                                              const UnitCells &c) {
  const int lane = threadIdx.x & 63;
  UnitRow<DT, ROW> t;
  t.issue(trow, V, unit, lane);
  t.place(V, unit, lane);
  store_totals(unit_totals([&](int i) { return target_p_weight(t.at(i), job); }), c.sub, unit);
}

// The reference of a unit's exponentials: its largest z c.  Units that a
// vocabulary mask covers whole need care: the rounding of a mask's z c (512 at
// -1e10) is what the largest weight's exponent comes out as, so where it would
// be large the reference is rounded up instead, which can only take such a unit's
// weights to 0; and the type's lowest value times c can overflow.
__device__ __forceinline__ float unit_reference(float M, float scale) {
  const float ref = fmaxf(M * scale, -FLT_MAX);
  if (fmaf(M, scale, -ref) <= 64.0f) return ref;
  return __uint_as_float(__float_as_uint(ref) + (ref < 0.f ? -1 : 1));
}

// Bonus row, one unit: the exponentials 2^(z c - ref) against the unit's own
// reference.  +inf shows in the maximum, -inf in the minimum, NaN in the
// totals; padding is finite.  Where the row's last unit holds only logits below
// the padding, the padding's weights are taken out.
template <int DT, int ROW>
__device__ __forceinline__ void bonus_unit(const char *trow, int64_t V, int32_t unit, float scale,
                                           const UnitCells &c) {
  const int lane = threadIdx.x & 63;
  UnitRow<DT, ROW> t;
  t.issue(trow, V, unit, lane);
  t.place(V, unit, lane);
  float m = -INFINITY, lo = INFINITY;
#pragma unroll
  for (int i = 0; i < kUnitElts; ++i) {
    const float z = t.at(i);
    m = fmaxf(m, z);
    lo = fminf(lo, z);
  }
  const float M = lanes::wave_max(m);
  float ref = unit_reference(M, scale);
  float w = unit_totals([&](int i) { return bonus_weight(t.at(i), scale, ref); });
  if (M == kPadF32 && int64_t(unit) * kUnit + kUnit > V) {
    w *= 0.0f;  // NaN stays NaN
    ref = -FLT_MAX;
  }
  const bool bad = __ballot(m == INFINITY || lo == -INFINITY || !isfinite(w)) != 0 || ref == INFINITY;
  store_totals(w, c.sub, unit);
  if (lane == 0) c.ref[unit] = UnitRef{bad ? NAN : ref, 0};
}

// Greedy bonus row, one unit: the largest raw logit and the smallest token
// holding it.  A NaN shows in the sum (|z| <= 2^64 keeps finite sums finite).
template <int DT, int ROW>
__device__ __forceinline__ void bonus_argmax_unit(const char *trow, int64_t V, int32_t unit, const UnitCells &c) {
  const int lane = threadIdx.x & 63;
  UnitRow<DT, ROW> t;
  t.issue(trow, V, unit, lane);
  t.place(V, unit, lane);
  float m = -INFINITY, lo = INFINITY, sum = 0.f;
#pragma unroll
  for (int i = 0; i < kUnitElts; ++i) {
    const float z = t.at(i);
    m = fmaxf(m, z);
    lo = fminf(lo, z);
    sum += z;
  }
  const float M = lanes::wave_max(m);
  uint32_t best = 0xffffffffu;
  if (m == M) {  // a lane's slots ascend in token order: its first equal slot is its smallest token
#pragma unroll
    for (int i = kUnitElts - 1; i >= 0; --i)
      if (t.at(i) == M) best = uint32_t(unit_token<DT, ROW>(unit, i, lane));
  }
  best = lanes::wave_min(best);
  const bool bad = __ballot(m == INFINITY || lo == -INFINITY || sum != sum) != 0;
  if (lane == 0) c.ref[unit] = UnitRef{bad ? NAN : M, int32_t(best)};
}

// Every unit of a row that this wavefront takes: units first, first + step, ...
template <int DT, int ROW>
__device__ __forceinline__ void draw_units(const DrawJob &job, const char *target, const char *draft, int64_t V,
                                           int32_t nu, int32_t first, int32_t step, const UnitCells &c) {
  const size_t esz = DT == DSDE_BF16 ? 2 : 4;
  const char *trow = target + size_t(job.target_row) * size_t(V) * esz;
  if (job.kind == 0) {
    const char *drow = draft + size_t(job.draft_row) * size_t(V) * esz;
    for (int32_t u = first; u < nu; u += step) residual_unit<DT, ROW>(trow, drow, V, u, job, c);
  } else if (job.kind == 1) {
    for (int32_t u = first; u < nu; u += step) bonus_unit<DT, ROW>(trow, V, u, job.scale, c);
  } else if (job.kind == 3) {
    for (int32_t u = first; u < nu; u += step) bonus_argmax_unit<DT, ROW>(trow, V, u, c);
  }
}

// ---------------------------------------------------------------------------
// the search
// ---------------------------------------------------------------------------

// A unit's cell as one lane holds it.  The first 64 units of a row are kept in
// registers by the callers (lane u: unit u), which covers vocabularies up to
// 131,072; later units are read again where they are needed.
struct UnitCell {
  float4 s;
  UnitRef r;
};
__device__ __forceinline__ UnitCell load_cell(const UnitCells &c, int32_t unit, int32_t nu, bool with_ref) {
  UnitCell x;
  x.s = make_float4(0.f, 0.f, 0.f, 0.f);
  x.r = UnitRef{0.f, 0};
  if (unit < nu) {
    x.s = *reinterpret_cast<const float4 *>(c.sub + int64_t(unit) * kSubs);
    if (with_ref) x.r = c.ref[unit];
  }
  return x;
}
__device__ __forceinline__ double cell_sum(const UnitCell &x) {
  return (double(x.s.x) + double(x.s.y)) + (double(x.s.z) + double(x.s.w));
}
// The unit's weight in the row's scale (mode 2: the bonus exponentials, whose
// units carry a reference each; modes 0 and 1 share one scale).
__device__ __forceinline__ double cell_weight(const UnitCell &x, int mode, float row_ref) {
  const double w = cell_sum(x);
  return mode == 2 ? w * exp2_taylor(double(x.r.ref) - double(row_ref)) : w;
}

// Row total of the weights, in every lane, by one wavefront in a fixed order.
__device__ __forceinline__ double row_total(const UnitCells &c, int32_t nu, const UnitCell &cell0, int mode,
                                            float row_ref) {
  const int lane = threadIdx.x & 63;
  double part = lane < nu ? cell_weight(cell0, mode, row_ref) : 0.0;
  for (int32_t u = lane + 64; u < nu; u += 64) part += cell_weight(load_cell(c, u, nu, mode == 2), mode, row_ref);
  return lanes::wave_sum(part);
}

// Largest reference of a bonus row's units (sampled rows: the row's scale;
// greedy rows: the row maximum), and whether a unit is marked bad.
__device__ __forceinline__ float row_reference(const UnitCells &c, int32_t nu, const UnitCell &cell0, bool *bad) {
  const int lane = threadIdx.x & 63;
  float m = -INFINITY;
  bool b = false;
  for (int32_t u = lane; u < nu; u += 64) {
    const float r = u < 64 ? cell0.r.ref : c.ref[u].ref;
    b |= r != r;
    m = fmaxf(m, r);
  }
  *bad = __ballot(b) != 0;
  return lanes::wave_max(m);
}

// The smallest token of a greedy bonus row's maximum M: the first unit that
// reaches it.
__device__ __forceinline__ int32_t row_argmax(const UnitCells &c, int32_t nu, const UnitCell &cell0, float M) {
  const int lane = threadIdx.x & 63;
  int32_t best = 0x7fffffff;  // token ids ascend with the unit: the smallest id belongs to the first unit
  for (int32_t u = lane; u < nu; u += 64) {
    const UnitRef r = u < 64 ? cell0.r : c.ref[u];
    if (r.ref == M && r.idx < best) best = r.idx;
  }
  return lanes::wave_min(best);
}

// The inverse-CDF draw inside one row, by one wavefront, from the unit cells:
// target is the weight to pass, in [0, row total), in the row's scale.  The
// rule at every level (unit, sub-block, element) is the draw's: the last
// position with positive weight whose exclusive prefix is <= the target
// (prefixes tile exactly: each position's start is the previous one's end),
// which also covers rounding past the total.  Returns the row-local token id
// in every lane.
template <int DT, int ROW>
__device__ __forceinline__ int32_t draw_in_row(const UnitCells &c, int32_t nu, const UnitCell &cell0, float row_ref,
                                               double target, const char *trow, const char *drow, int64_t V, int mode,
                                               const DrawJob &job) {
  const int lane = threadIdx.x & 63;
  int32_t unit = 0;
  double unit_excl = 0.0, base = 0.0;
  float4 us = make_float4(0.f, 0.f, 0.f, 0.f);
  float uref = 0.f;
  for (int32_t u0 = 0; u0 < nu; u0 += 64) {
    const int32_t u = u0 + lane;
    const UnitCell x = u0 == 0 ? cell0 : load_cell(c, u, nu, mode == 2);
    const double w = u < nu ? cell_weight(x, mode, row_ref) : 0.0;
    const lanes::Scan<double> sc = lanes::wave_scan(w);
    const double incl = base + sc.incl;
    const double excl = lane == 0 ? base : base + sc.excl;
    const uint64_t cand = __ballot(u < nu && w > 0.0 && excl <= target);
    if (cand) {
      const int l = 63 - __builtin_clzll(cand);
      unit = u0 + l;
      unit_excl = lanes::readlane(excl, l);
      us = make_float4(lanes::readlane(x.s.x, l), lanes::readlane(x.s.y, l), lanes::readlane(x.s.z, l),
                       lanes::readlane(x.s.w, l));
      uref = lanes::readlane(x.r.ref, l);
    }
    base = lanes::readlane(incl, 63);
  }
  double rem = target - unit_excl;
  if (rem < 0.0) rem = 0.0;
  if (mode == 2) rem *= exp2_taylor(double(row_ref) - double(uref));  // into the unit's own scale

  // the sub-block: the four totals in order (uniform over the wavefront)
  const double b1 = double(us.x), b2 = b1 + double(us.y), b3 = b2 + double(us.z);
  int sb = 0;
  double sub_excl = 0.0;
  if (us.y > 0.f && b1 <= rem) sb = 1, sub_excl = b1;
  if (us.z > 0.f && b2 <= rem) sb = 2, sub_excl = b2;
  if (us.w > 0.f && b3 <= rem) sb = 3, sub_excl = b3;
  double rem2 = rem - sub_excl;
  if (rem2 < 0.0) rem2 = 0.0;

  // its 512 logits, 8 consecutive per lane, with the weights evaluated by the
  // routines of the totals; the lane holding the target walks its own eight
  const int64_t run0 = int64_t(unit) * kUnit + int64_t(sb) * kSubLen + 8 * lane;
  float w[8];
  {
    float zt[8];
    load_run8<DT, ROW>(trow, V, run0, zt);
    if (mode == 0) {
      float zd[8];
      load_run8<DT, ROW>(drow, V, run0, zd);
#pragma unroll
      for (int i = 0; i < 8; ++i) w[i] = residual_weight(zt[i], zd[i], job);
    } else if (mode == 1) {
#pragma unroll
      for (int i = 0; i < 8; ++i) w[i] = target_p_weight(zt[i], job);
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) w[i] = bonus_weight(zt[i], job.scale, uref);
    }
  }
  double run_total = 0.0;
  int last = -1;  // this lane's last positive weight
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    run_total += double(w[i]);
    if (w[i] > 0.0f) last = i;
  }
  const lanes::Scan<double> sr = lanes::wave_scan(run_total);
  const uint64_t cand = __ballot(last >= 0 && sr.excl <= rem2);
  const int winner = cand ? 63 - __builtin_clzll(cand) : 0;
  int pick = last >= 0 ? last : 0;
  double acc = sr.excl;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    acc += double(w[i]);
    if (acc > rem2) {
      pick = i;
      break;
    }
  }
  return lanes::readlane(int32_t(run0 + pick), winner);
}
}  // namespace
}  // namespace dsde
