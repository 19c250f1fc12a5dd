// One site's CG residual update r -= alpha (A p), for the dslash launch that
// fuses it into its epilogue (FP32 and FP16 storage), and the whole vector
// update x += alpha p, r -= alpha (A p) of FP16-storage vectors for the
// separate kernel; each returns the site's contribution to <r, r> (of the
// values as stored). Also the store of a site of t = Q p with its squared
// norm, for the dslash launch that fuses <p, A p> = |t|^2 into its epilogue.
#pragma once

#include "fields.h"

namespace wd {

__device__ __forceinline__ double norm2(double2 a) { return fmar(a.x, a.x, a.y * a.y); }
__device__ __forceinline__ double norm2(float4 a) {
  const double x = a.x, y = a.y, z = a.z, w = a.w;
  return fmar(x, x, fmar(y, y, fmar(z, z, w * w)));
}

// Sum over the 64 lanes of a wave in a fixed order (every lane gets it), and
// over each 32 lanes of it.
__device__ __forceinline__ double half_wave_total(double v) {
#pragma unroll
  for (int off = 16; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
__device__ __forceinline__ double wave_total(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Share i of 256 of pp[0..np): pp[i + 256 j] added in order of j, with N loads in
// flight.
template <int N>
__device__ __forceinline__ double strided_sum256_by(const double* __restrict__ pp, int np, int i) {
  double s = 0.0;
  for (; i < np; i += N * 256) {
    double a[N];
#pragma unroll
    for (int j = 0; j < N; ++j) a[j] = i + 256 * j < np ? pp[i + 256 * j] : 0.0;
#pragma unroll
    for (int j = 0; j < N; ++j) s += a[j];
  }
  return s;
}
// ... in one round of memory latency for up to 3072 partial sums and two for 6144 (a
// lattice of 131072 sites has up to 5000). A round is latency ahead of a workgroup's
// first site: with eight loads in flight for all counts, a solve's iteration took 2 to
// 4 % longer on 65000 sites (20^3 x 16 and 19 x 7 x 20 x 23, FP32). Twelve take 8 to 16
// more registers in the small solves' kernels, a wave per SIMD in FP16 (-1 to -2 %
// on 18^4); sixteen took two. Every kernel that reduces partial sums adds these
// shares in waves of 64 and the four waves' sums in order, so that all of them get
// the same bits.
__device__ __forceinline__ double strided_sum256(const double* __restrict__ pp, int np, int i) {
  return np <= 8 * 256 ? strided_sum256_by<8>(pp, np, i) : strided_sum256_by<12>(pp, np, i);
}

// Squared norm of two components of a site. A site's norm adds its six pairs
// in order, so that it does not matter whether one lane or six hold them.
__device__ __forceinline__ double pair_norm2(cx<double> a, cx<double> b) {
  return fmar(a.re, a.re, a.im * a.im) + fmar(b.re, b.re, b.im * b.im);
}
__device__ __forceinline__ double pair_norm2(cx<float> a, cx<float> b) {
  return norm2(make_float4(a.re, a.im, b.re, b.im));
}
__device__ __forceinline__ double half_pair_norm2(h4 q, float m) {
  double n = 0.0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const double d = static_cast<float>(q[k]) * m;
    n = fmar(d, d, n);
  }
  return n;
}

__device__ __forceinline__ double site_norm2(const cx<float> (&v)[12]) {
  double s = 0.0;
#pragma unroll
  for (int c = 0; c < 12; ++c) {
    const double re = v[c].re, im = v[c].im;
    s = fmar(re, re, fmar(im, im, s));
  }
  return s;
}

__device__ __forceinline__ double half_site_norm2(const h8 (&q)[3], float m) {
  double n = 0.0;
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    n += half_pair_norm2(h4{q[j][0], q[j][1], q[j][2], q[j][3]}, m);
    n += half_pair_norm2(h4{q[j][4], q[j][5], q[j][6], q[j][7]}, m);
  }
  return n;
}

// Quantises and stores a site (cached stores: CG vectors are read again at
// once); returns the squared norm of the values as stored.
__device__ __forceinline__ double store_half_site(h8* __restrict__ p, long s, const cx<float> (&v)[12]) {
  h8 q[3];
  const float m = half_quantise(v, q);
#pragma unroll
  for (int j = 0; j < 3; ++j) p[half_unit(s, j)] = q[j];
  reinterpret_cast<float*>(p)[half_scale_index(s)] = m;
  return half_site_norm2(q, m);
}

// r -= alpha (A p) at one site; ap holds A p. FP32 vectors.
__device__ __forceinline__ double cg_site_update_r(float4* __restrict__ r, long V, long s,
                                                   const cx<float> (&ap)[12], double alpha) {
  const float a = static_cast<float>(alpha);
  double n = 0.0;
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    const long e = pidx(s, j, 6, V);
    float4 re = r[e];
    re.x = fmar(-a, ap[2 * j].re, re.x);
    re.y = fmar(-a, ap[2 * j].im, re.y);
    re.z = fmar(-a, ap[2 * j + 1].re, re.z);
    re.w = fmar(-a, ap[2 * j + 1].im, re.w);
    r[e] = re;
    n += norm2(re);
  }
  return n;
}

// The same for FP64 vectors.
__device__ __forceinline__ double cg_site_update_r(double2* __restrict__ r, long V, long s,
                                                   const cx<double> (&ap)[12], double alpha) {
  double n = 0.0;
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    cx<double> v[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const long i = pidx(s, 2 * j + e, 12, V);
      const double2 re = r[i];
      v[e] = {fmar(-alpha, ap[2 * j + e].re, re.x), fmar(-alpha, ap[2 * j + e].im, re.y)};
      r[i] = make_double2(v[e].re, v[e].im);
    }
    n += pair_norm2(v[0], v[1]);
  }
  return n;
}

// The same for FP16-storage vectors: r is requantised per site.
__device__ __forceinline__ double cg_site_update_r(h8* __restrict__ r, long V, long s,
                                                   const cx<float> (&ap)[12], double alpha) {
  const float a = static_cast<float>(alpha);
  cx<float> rv[12];
  load_spinor(r, V, static_cast<int>(s), rv);
#pragma unroll
  for (int c = 0; c < 12; ++c) rv[c] = {fmar(-a, ap[c].re, rv[c].re), fmar(-a, ap[c].im, rv[c].im)};
  return store_half_site(r, s, rv);
}

// x_lo += alpha p at one site, x_lo the FP32 accumulator (FP32 layout) and p
// in FP16 storage (pv: p at the site, dequantised).
__device__ __forceinline__ void cg_site_update_x(float4* __restrict__ x, long V, long s,
                                                 const cx<float> (&pv)[12], float a) {
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    const long e = pidx(s, j, 6, V);
    float4 xe = x[e];
    xe.x = fmar(a, pv[2 * j].re, xe.x);
    xe.y = fmar(a, pv[2 * j].im, xe.y);
    xe.z = fmar(a, pv[2 * j + 1].re, xe.z);
    xe.w = fmar(a, pv[2 * j + 1].im, xe.w);
    x[e] = xe;
  }
}

// x_lo += a0 p0, then += a1 p1, at one site (two updates of
// cg_site_update_x in turn, with one read and one write of x_lo).
__device__ __forceinline__ void cg_site_update_x2(float4* __restrict__ x, long V, long s,
                                                  const cx<float> (&p0)[12], float a0,
                                                  const cx<float> (&p1)[12], float a1) {
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    const long e = pidx(s, j, 6, V);
    float4 xe = x[e];
    xe.x = fmar(a0, p0[2 * j].re, xe.x);
    xe.y = fmar(a0, p0[2 * j].im, xe.y);
    xe.z = fmar(a0, p0[2 * j + 1].re, xe.z);
    xe.w = fmar(a0, p0[2 * j + 1].im, xe.w);
    xe.x = fmar(a1, p1[2 * j].re, xe.x);
    xe.y = fmar(a1, p1[2 * j].im, xe.y);
    xe.z = fmar(a1, p1[2 * j + 1].re, xe.z);
    xe.w = fmar(a1, p1[2 * j + 1].im, xe.w);
    x[e] = xe;
  }
}

// FP16-storage vectors: x is the FP32 accumulator x_lo (FP32 layout); r is
// requantised per site.
__device__ __forceinline__ double cg_site_update(float4* __restrict__ x, h8* __restrict__ r,
                                                 const h8* __restrict__ p, long V, long s,
                                                 const cx<float> (&ap)[12], double alpha) {
  const float a = static_cast<float>(alpha);
  cx<float> pv[12];
  load_spinor(p, V, static_cast<int>(s), pv);
  cg_site_update_x(x, V, s, pv, a);
  return cg_site_update_r(r, V, s, ap, alpha);
}

// Stores a site of t = Q p (streaming stores, as the plain operator) and
// returns its squared norm (of the values as stored).
__device__ __forceinline__ double store_site_norm(double2* __restrict__ p, long V, int s,
                                                  const cx<double> (&v)[12]) {
  store_spinor(p, V, s, v);
  double n = 0.0;
#pragma unroll
  for (int j = 0; j < 6; ++j) n += pair_norm2(v[2 * j], v[2 * j + 1]);
  return n;
}
__device__ __forceinline__ double store_site_norm(float4* __restrict__ p, long V, int s,
                                                  const cx<float> (&v)[12]) {
  store_spinor(p, V, s, v);
  double n = 0.0;
#pragma unroll
  for (int j = 0; j < 6; ++j) n += pair_norm2(v[2 * j], v[2 * j + 1]);
  return n;
}
__device__ __forceinline__ double store_site_norm(h8* __restrict__ p, long /*V*/, int s,
                                                  const cx<float> (&v)[12]) {
  h8 q[3];
  const float m = half_quantise(v, q);
#pragma unroll
  for (int j = 0; j < 3; ++j) __builtin_nontemporal_store(q[j], p + half_unit(s, j));
  __builtin_nontemporal_store(m, reinterpret_cast<float*>(p) + half_scale_index(s));
  return half_site_norm2(q, m);
}

// Stores components 2j, 2j + 1 of a site; returns their squared norm as stored.
// FP16 storage: m is the site's largest modulus; j = 0 also stores it.
__device__ __forceinline__ double store_pair(double2* __restrict__ p, long V, int s, int j,
                                             const cx<double> (&v)[2]) {
  p[pidx(s, 2 * j, 12, V)] = make_double2(v[0].re, v[0].im);
  p[pidx(s, 2 * j + 1, 12, V)] = make_double2(v[1].re, v[1].im);
  return pair_norm2(v[0], v[1]);
}
__device__ __forceinline__ double store_pair(float4* __restrict__ p, long V, int s, int j,
                                             const cx<float> (&v)[2]) {
  p[pidx(s, j, 6, V)] = make_float4(v[0].re, v[0].im, v[1].re, v[1].im);
  return pair_norm2(v[0], v[1]);
}
__device__ __forceinline__ double store_pair(h8* __restrict__ p, int s, int j, const cx<float> (&v)[2], float m) {
  const h4 q = half_quantise_pair(v, m);
  reinterpret_cast<h4*>(p)[2 * half_unit(s, j >> 1) + (j & 1)] = q;
  if (j == 0) reinterpret_cast<float*>(p)[half_scale_index(s)] = m;
  return half_pair_norm2(q, m);
}

// alpha = <r, r> / <p, A p> and its failure flag from <p, A p> = t.
__device__ __forceinline__ double cg_alpha(double t, double rr, bool* flag) {
  *flag = !isfinite(t);
  if (!(t > 0.0)) {
    if (rr > 0.0) *flag = true;
    return 0.0;
  }
  return rr / t;
}

}  // namespace wd
