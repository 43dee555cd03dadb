// Softmax statistics of 64-column chunks of logits rows, for the EB-Sampler's entropy
// (Sec. 2.2, eq. (eb_sampler)) straight from the LM head's epilogue (gemv.hip, gemm.hip):
// the logits then need not be stored and read back.  eb.hip merges the chunks of a row.
#pragma once

#include "sbd_device.h"

namespace sbd {

__device__ __forceinline__ double shfl_xor_d(double v, int m) {
  const int2 iv = *reinterpret_cast<int2*>(&v);
  int2 o;
  o.x = __shfl_xor(iv.x, m);
  o.y = __shfl_xor(iv.y, m);
  return *reinterpret_cast<double*>(&o);
}

// v of lane i (i uniform across the wave), in every lane
__device__ __forceinline__ double readlane_d(double v, int i) {
  const int2 iv = *reinterpret_cast<int2*>(&v);
  int2 o;
  o.x = __builtin_amdgcn_readlane(iv.x, i);
  o.y = __builtin_amdgcn_readlane(iv.y, i);
  return *reinterpret_cast<double*>(&o);
}

// 2^(j/32), j = 0 .. 31, rounded to float64 (the kernels stage it in LDS: one entry covers two
// of the 64 banks, so 64 lanes' reads of it never conflict).
static __constant__ const double kExp2Frac[32] = {
    0x1.0000000000000p+0, 0x1.059b0d3158574p+0, 0x1.0b5586cf9890fp+0, 0x1.11301d0125b51p+0,
    0x1.172b83c7d517bp+0, 0x1.1d4873168b9aap+0, 0x1.2387a6e756238p+0, 0x1.29e9df51fdee1p+0,
    0x1.306fe0a31b715p+0, 0x1.371a7373aa9cbp+0, 0x1.3dea64c123422p+0, 0x1.44e086061892dp+0,
    0x1.4bfdad5362a27p+0, 0x1.5342b569d4f82p+0, 0x1.5ab07dd485429p+0, 0x1.6247eb03a5585p+0,
    0x1.6a09e667f3bcdp+0, 0x1.71f75e8ec5f74p+0, 0x1.7a11473eb0187p+0, 0x1.82589994cce13p+0,
    0x1.8ace5422aa0dbp+0, 0x1.93737b0cdc5e5p+0, 0x1.9c49182a3f090p+0, 0x1.a5503b23e255dp+0,
    0x1.ae89f995ad3adp+0, 0x1.b7f76f2fb5e47p+0, 0x1.c199bdd85529cp+0, 0x1.cb720dcef9069p+0,
    0x1.d5818dcfba487p+0, 0x1.dfc97337b9b5fp+0, 0x1.ea4afa2a490dap+0, 0x1.f50765b6e4540p+0,
};
__device__ __forceinline__ void exp_table_stage(double* tab, int t) {
  if (t < 32) tab[t] = kExp2Frac[t];
}

// e^x in float64 for x in [kExpZero, 0], within about one unit in the last place.  With
// k = round(32 x / ln 2) and r = x - k ln 2 / 32 (|r| <= 0.0109, in two parts):
// e^x = 2^(k div 32) 2^((k mod 32) / 32) e^r, and e^r - 1 from its Taylor series to r^6 (the
// next term is below 4e-18).  14 float64 operations and no branch, where the library's exp is
// made for every argument.
constexpr double kExpZero = -800.0;  // e^-800 is zero: arguments below it may be raised to it
__device__ __forceinline__ double exp_neg(double x, const double* tab) {
  constexpr double kMagic = 6755399441055744.0;  // 1.5 * 2^52: adding it rounds to an integer
  const double kd = fma(x, 0x1.71547652b82fep+5, kMagic);  // 32 / ln 2
  const int k = __double2loint(kd);
  const double kf = kd - kMagic;
  // ln 2 / 32 as a high and a low part
  const double r = fma(kf, -0x1.abc9e3b39803fp-61, fma(kf, -0x1.62e42fefa39efp-6, x));
  double q = 1.0 / 720.0;
  q = fma(q, r, 1.0 / 120.0);
  q = fma(q, r, 1.0 / 24.0);
  q = fma(q, r, 1.0 / 6.0);
  q = fma(q, r, 0.5);
  const double p = fma(r * r, q, r);
  const double f = tab[k & 31];
  return ldexp(fma(f, p, f), k >> 5);
}

// Z = sum e^t and S = sum e^t t over a thread's N logits, t = l - mx in float64, in order; mx
// is at least every logit and above -inf.  A logit of -inf adds nothing (as one further than
// 800 below the maximum); a NaN logit or an infinite maximum makes both NaN.
template <int N>
__device__ __forceinline__ void exp_sums(const float (&v)[N], float mx, const double* tab, double& z, double& s) {
  const double md = (double)mx;
  bool nan = mx == INFINITY;
  z = 0.0;
  s = 0.0;
#pragma unroll
  for (int e = 0; e < N; ++e) {
    nan |= v[e] != v[e];
    const double x = fmax((double)v[e] - md, kExpZero);
    const double ex = exp_neg(x, tab);
    z += ex;
    s = fma(ex, x, s);
  }
  if (nan) z = s = __builtin_nan("");
}

// One 64-column chunk of one row held by LPC adjacent lanes (xor distances below LPC), each
// with VPL consecutive columns col0 .. col0 + VPL - 1 staged in LDS at p (fp32 products,
// times `scale` = the row's norm scale gives the logit exactly as stored).  The mask column
// is left out.  tab: the staged table of exp_neg.  Results, the same on the LPC lanes: the
// chunk maximum mx and the smallest column reaching it (INT32_MAX when no value is above
// -inf), then with t = l - mx in float64, Z = sum e^t and S = sum e^t t over the values above -inf (each lane in column
// order, then a fixed butterfly).  A NaN logit is never the maximum but makes Z and S NaN,
// an infinite maximum makes them NaN too (both as the EB partial kernel on stored logits).
template <int VPL, int LPC>
__device__ __forceinline__ void eb_seg_stats(const float* p, float scale, int col0, int mask_id, const double* tab,
                                             float& mx, int& arg, double& z, double& s) {
  float v[VPL];
#pragma unroll
  for (int e = 0; e < VPL; e += 4) {
    const f32x4 q = *reinterpret_cast<const f32x4*>(p + e);
#pragma unroll
    for (int u = 0; u < 4; ++u) v[e + u] = q[u] * scale;
  }
  mx = -INFINITY;
  arg = INT32_MAX;
#pragma unroll
  for (int e = 0; e < VPL; ++e) {
    if (col0 + e == mask_id) v[e] = -INFINITY;
    if (v[e] > mx) {  // columns ascend: the first of equal values is kept
      mx = v[e];
      arg = col0 + e;
    }
  }
#pragma unroll
  for (int o = 1; o < LPC; o <<= 1) {
    const float om = __shfl_xor(mx, o);
    const int oa = __shfl_xor(arg, o);
    if (om > mx || (om == mx && oa < arg)) {
      mx = om;
      arg = oa;
    }
  }
  z = 0.0;
  s = 0.0;
  if (mx != -INFINITY) exp_sums<VPL>(v, mx, tab, z, s);
#pragma unroll
  for (int o = 1; o < LPC; o <<= 1) {  // a + b = b + a: the LPC lanes end with the same bits
    z += shfl_xor_d(z, o);
    s += shfl_xor_d(s, o);
  }
}

// Store the statistics of chunk `chunk` of row m: part [rows][n_chunks][3] = (max, Z, S),
// part_arg [rows][n_chunks] = the argmax column or -1.
__device__ __forceinline__ void eb_chunk_store(double* part, int32_t* part_arg, int n_chunks, int64_t m, int chunk,
                                               float mx, int arg, double z, double s) {
  double* p = part + (m * n_chunks + chunk) * 3;
  p[0] = (double)mx;
  p[1] = z;
  p[2] = s;
  part_arg[m * n_chunks + chunk] = mx == -INFINITY ? -1 : arg;
}

}  // namespace sbd
