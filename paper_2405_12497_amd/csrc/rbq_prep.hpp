// Device helpers of the per-pair quantisation (Sec. 3.3.1), shared by its kernels.
#pragma once
#include "rbq_internal.hpp"

namespace rbq {
namespace {

// <x_bar, q_bar> = k1 <x_b, q_u> + k2 popcount(x_b) + k0 with k1 = 2 Delta / sqrt(D),
// k2 = 2 v_l / sqrt(D) and k0 = -(Delta / sqrt(D)) sum(q_u) - sqrt(D) v_l
// (Sec. 3.3.1-3.3.2), in FP64; rd = sqrt(D) and ird = 1 / rd come from the host.
__device__ __forceinline__ void pair_coeffs(double vl, double delta, int sq, double rd, double ird,
                                            PairRec& r) {
  const double dr = delta * ird;
  r.k1 = (float)(2.0 * dr);
  r.k2 = (float)(2.0 * vl * ird);
  r.k0 = (float)(-dr * (double)sq - rd * vl);
}

// v_l = rmin / b and Delta = range / ((2^B_q - 1) b) of a pair, in FP64 (0 when b = 0).
__device__ __forceinline__ void pair_scalars(float rmin, float range, float b, int qmax, double& vl,
                                             double& delta) {
  vl = 0.0;
  delta = 0.0;
  if (b > 0.f) {
    const double ib = 1.0 / (double)b;
    vl = (double)rmin * ib;
    delta = (double)range * ib / (double)qmax;
  }
}

__device__ __forceinline__ PairRec pair_record(const SearchDev& s, float rmin, float range, float b, int sq, int list) {
  PairRec rec;
  double vl, delta;
  pair_scalars(rmin, range, b, s.qmax, vl, delta);
  pair_coeffs(vl, delta, sq, s.rd, s.ird, rec);
  rec.b = b;
  rec.vl = (float)vl;
  rec.delta = (float)delta;
  rec.sq = sq;
  rec.list = list;
  return rec;
}

// A probe slot past the query's nprobe.
__device__ __forceinline__ PairRec empty_record() {
  PairRec rec;
  rec.k1 = rec.k2 = rec.k0 = rec.b = rec.vl = rec.delta = 0.f;
  rec.sq = 0;
  rec.list = -1;
  return rec;
}

// ||q_r - c|| by one wave, given the rotated residual's norm b and the query's
// norm qn. Near a centroid the rotated residual is dominated by the rotation's
// rounding (~1e-6 (||q|| + ||c||)): b is taken from the raw vectors there, so
// that it is exactly 0 when the query coincides with the centroid.
__device__ __forceinline__ float pair_norm(const SearchDev& s, int64_t q, int list, float b, float qn) {
  const float scale_qc = uniform_f32(qn + sqrtf(s.cnorm[list]));
  if (b <= 1e-4f * scale_qc) {
    const float* qr = s.q + q * s.dim;
    const float* c = s.cent + (int64_t)list * s.dim;
    float acc = 0.f;
    for (int i = lane_id(); i < s.dim; i += kWave) {
      const float d = qr[i] - c[i];
      acc = fmaf(d, d, acc);
    }
    b = uniform_f32(sqrtf(wave_sum(acc)));
  }
  return b;
}

// Inner product: the pair's constant M_q - <q_r, c> from the raw vectors, by one wave.
__device__ __forceinline__ void pair_ip_term(const SearchDev& s, int64_t g, int64_t q, int list) {
  const float* qr = s.q + q * s.dim;
  const float* c = s.cent + (int64_t)list * s.dim;
  float acc = 0.f;
  for (int i = lane_id(); i < s.dim; i += kWave) acc = fmaf(qr[i], c[i], acc);
  const float gdot = wave_sum(acc);
  if (lane_id() == 0) s.pair_pt[g] = s.q_m[q] - gdot;
}

// k_prep_wide's randomised rounding of residual v: floor((v - rmin) scale + u), at
// most qmax, with u = f 2^-24, as a float. The sum is never negative, so truncation
// is the floor. One rounding of the product for words 2 j, one of the product and
// sum together for words 2 j + 1: written out, so that the compiler's choice of
// contraction cannot tell its instances apart (the popcount and the batched scan of
// one search must see the same quantised query). A pair that is not live has scale
// 0, so it quantises to 0, as does a NaN (the median with a NaN is the smaller of
// the other two).
__device__ __forceinline__ float round_even_word(float v, float rmin, float scale, uint32_t f, float qmax) {
#pragma clang fp contract(off)
  const float x = (v - rmin) * scale;
  return __builtin_amdgcn_fmed3f(truncf(__builtin_fmaf((float)f, 1.0f / 16777216.0f, x)), 0.f, qmax);
}
__device__ __forceinline__ float round_odd_word(float v, float rmin, float scale, uint32_t f, float qmax) {
#pragma clang fp contract(off)
  const float u = (float)f * (1.0f / 16777216.0f);
  return __builtin_amdgcn_fmed3f(truncf(__builtin_fmaf(v - rmin, scale, u)), 0.f, qmax);
}

}  // namespace
}  // namespace rbq
