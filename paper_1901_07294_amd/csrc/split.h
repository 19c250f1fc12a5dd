// The Wilson-Dirac operator, and the hops of an even-odd split one, with every
// site's hops spread over eight lanes.
//
// What bounds a small lattice is not bytes but latency: a lane that walks its
// site's eight hops one after the other waits for memory eight times or more,
// while most of the chip has nothing to do. Here a workgroup of four waves owns
// 32 consecutive sites; wave mu works on direction mu, its lower 32 lanes on the
// forward and its upper 32 on the backward hop, so all eight neighbour spinors
// and links of a site are in flight at once and an operator costs one round of
// memory latency. Each lane leaves its half spinor U h (or U^dag h) in LDS; then
// six groups of 32 lanes rebuild two of the twelve spin-colour components each,
// adding the hops in the order of the t-marching kernel (or, where that kernel
// does not apply, in the order x, y, z, t), so that both kernels give the same
// bits and the choice between them is one of speed alone.
//
// 32 sites rather than 64 per workgroup: 8^4 has 128 workgroups of them, and a
// CU's L1 has to pass 21 16-byte elements per hop, 86 KB for 32 FP64 sites.
//
// Measured on MI355X (one lane per site or a march of four slices -> this
// kernel): 8^4 FP32 in a solve 17.1 -> 5.7 us per launch (6.0 -> 2.8 ms per
// solve), 15 x 9 x 14 x 21 FP32 24.2 -> 7.6 us, 6 x 6 x 40 x 72 FP64 35.9 -> 19.2
// us, with four fields 174 -> 62 us. On larger lattices every neighbour spinor
// comes through L1, and the marches win (24^4 FP16 22 against 30 us).
#pragma once

#include <algorithm>

#include "cg_site.h"
#include "stencil.h"
#include "wd_internal.h"

namespace wd {

constexpr int kSplitSites = 32;     // sites per workgroup
constexpr int kSplitThreads = 256;  // (direction, sign, site)

// CG slices of small lattices: runs of kSplitSites consecutive sites, cut where a
// tile of the t-marching kernel begins (tiles are tile >= 64 consecutive sites; 0:
// no cuts), so that a workgroup of either kernel holds whole slices.
struct CgSlices {
  int tile;
  int both;  // the least common multiple of tile and kSplitSites
  // the slice of site s: one begins at every run and at every tile, not two where both do
  __host__ __device__ int of(int s) const { return s / kSplitSites + (tile == 0 ? 0 : s / tile - s / both); }
};

// The sites of a field, or (eo) of the output half field: rows of X sites, with
// the strides of y, z and t. eo: the outputs have parity `parity`, the inputs
// the other one; both half fields have the same half-site order.
struct SplitParams {
  int X, Y, Z, T;
  int sy, sz, st;
  int V;
  int eo, parity;
  int wide;    // eo_hop_kernel: CG slices of 256 sites instead of 32
  int ntiles;  // runs of kSplitSites sites
  int per;     // workgroups (a tile of one field each) per XCD; the last may have fewer
  int nrhs;
  int ny;      // y rows per tile of the t-marching kernel, 0 where it does not apply
  CgSlices cut;  // the sites' CG slices
  unsigned link_bytes;    // bytes of the packed links and of one packed spinor field
  unsigned spinor_bytes;  // (used when they are read through buffer resources)
};

// out = d * w + c * (sum of hops), per right-hand side, on field idx.
template <typename R>
struct SplitCoef {
  R d[kMaxMultiRhs];
  R c[kMaxMultiRhs];
  int idx[kMaxMultiRhs];
};

// h = psi_u + sg * A_mu psi_l with sg = -1 (forward hop) or +1 (backward): the
// additions of project<>, spelled as multiply-adds by +-1 (the same values).
template <int MU, typename R>
__device__ __forceinline__ void project_sg(const cx<R> (&p)[12], R sg, cx<R> (&h)[6]) {
  auto add = [&](cx<R> a, cx<R> b, R s) { return cx<R>{fmar(s, b.re, a.re), fmar(s, b.im, a.im)}; };
  auto addi_s = [&](cx<R> a, cx<R> b, R s) { return cx<R>{fmar(-s, b.im, a.re), fmar(s, b.re, a.im)}; };
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const cx<R> p0 = p[a], p1 = p[3 + a], p2 = p[6 + a], p3 = p[9 + a];
    if constexpr (MU == 0) {
      h[a] = addi_s(p0, p3, sg);
      h[3 + a] = addi_s(p1, p2, sg);
    } else if constexpr (MU == 1) {
      h[a] = add(p0, p3, -sg);
      h[3 + a] = add(p1, p2, sg);
    } else if constexpr (MU == 2) {
      h[a] = addi_s(p0, p2, sg);
      h[3 + a] = addi_s(p1, p3, -sg);
    } else {
      h[a] = add(p0, p2, sg);
      h[3 + a] = add(p1, p3, sg);
    }
  }
}

// u, or its conjugate transpose where dag.
template <typename R>
__device__ __forceinline__ void select_dagger(cx<R> (&u)[9], bool dag) {
  const R s = dag ? R(-1) : R(1);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    u[4 * a].im *= s;
#pragma unroll
    for (int b = a + 1; b < 3; ++b) {
      const cx<R> x = u[3 * a + b], y = u[3 * b + a];
      u[3 * a + b] = {dag ? y.re : x.re, s * (dag ? y.im : x.im)};
      u[3 * b + a] = {dag ? x.re : y.re, s * (dag ? x.im : y.im)};
    }
  }
}

// Hops of all sites of a workgroup, as left in LDS: [hop][half-spinor component][site].
template <typename R>
struct SplitHops {
  cx<R> g[8][6][kSplitSites];
};

// acc += the contribution of hop H (2 mu + backward) to component c = 2j or
// 2j + 1 of a spinor: lower says c >= 6, half which of the two half-spinor
// rows it belongs to, col its colour. The additions are reconstruct_add's.
template <int H, typename R>
__device__ __forceinline__ void add_hop(const SplitHops<R>& l, int site, bool lower, int half, int col,
                                        cx<R>& acc) {
  constexpr int mu = H / 2;
  constexpr R S = (H & 1) ? R(1) : R(-1);
  const int row = (mu < 2 && lower) ? 1 - half : half;
  const cx<R> g = l.g[H][3 * row + col][site];
  if constexpr (mu == 0 || mu == 2) {  // lower: S * (-i g), for mu = 2 with the sign flipped in row 1
    const R s = (mu == 2 && half == 1) ? -S : S;
    const R x = lower ? g.im : g.re, y = lower ? g.re : g.im;
    acc.re = fmar(lower ? s : R(1), x, acc.re);
    acc.im = fmar(lower ? -s : R(1), y, acc.im);
  } else {  // lower: S * g, for mu = 1 with the sign flipped in row 1
    const R s = !lower ? R(1) : (mu == 1 && half == 1) ? -S : S;
    acc.re = fmar(s, g.re, acc.re);
    acc.im = fmar(s, g.im, acc.im);
  }
}

// The neighbour of site s in direction mu, backward where up != 0 (periodic;
// extent 1 wraps onto the site itself).
__device__ __forceinline__ int split_neighbour(const SplitParams& p, int mu, int up, int s) {
  const unsigned u = static_cast<unsigned>(s);
  if (p.eo && mu == 0) {
    // x = 2 xh + o: x + 1 is the same half index for o = 0, the next one for
    // o = 1; x - 1 is the one before for o = 0, the same one for o = 1
    const unsigned r = u / static_cast<unsigned>(p.X);
    const int xh = s - static_cast<int>(r) * p.X;
    const unsigned y = r % static_cast<unsigned>(p.Y), zt = r / static_cast<unsigned>(p.Y);
    const unsigned z = zt % static_cast<unsigned>(p.Z), t = zt / static_cast<unsigned>(p.Z);
    const int o = static_cast<int>((y + z + t + static_cast<unsigned>(p.parity)) & 1u);
    if (o == up) return s;
    return up == 0 ? (xh + 1 == p.X ? s - (p.X - 1) : s + 1) : (xh == 0 ? s + (p.X - 1) : s - 1);
  }
  const int ext = mu == 0 ? p.X : mu == 1 ? p.Y : mu == 2 ? p.Z : p.T;
  const int st = mu == 0 ? 1 : mu == 1 ? p.sy : mu == 2 ? p.sz : p.st;
  const int c = static_cast<int>((u / static_cast<unsigned>(st)) % static_cast<unsigned>(ext));
  return up == 0 ? (c + 1 == ext ? s - (ext - 1) * st : s + st) : (c == 0 ? s + (ext - 1) * st : s - st);
}

// Workgroup -> run of sites (p.ntiles or more: nothing to do) and right-hand
// side. Every XCD gets one contiguous run of tiles (their halos meet in one L2),
// and the right-hand sides of a tile follow each other, so that its links come
// from HBM once: with the right-hand sides in the grid's second dimension four
// FP64 fields on an even-odd 24^4 took 443 us per application, now 284. The
// shares are of workgroups, not of tiles: 41 tiles of six fields are 31
// workgroups for each XCD's 32 CUs, where six tiles each were 36. One field skips the
// divisions, which stand before the first load (FP64 27 x 4 x 14 x 14 7.5 -> 7.1 us, the
// Schur operator on 12^4 12.9 -> 12.2).
// The kernels with CG work, whose first loads are the partial sums, lost 1 % by it (ONE).
template <bool ONE>
__device__ __forceinline__ int split_tile(const SplitParams& p, int* rhs) {
  const int b = blockIdx.x % kNumXcd * p.per + blockIdx.x / kNumXcd;
  if (ONE && p.nrhs == 1) {
    *rhs = 0;
    return b;
  }
  *rhs = b % p.nrhs;
  return b / p.nrhs;
}
// The grid for it: p.ntiles and p.nrhs given, p.per filled in.
inline unsigned split_grid(SplitParams& p) {
  p.per = (p.ntiles * p.nrhs + kNumXcd - 1) / kNumXcd;
  return static_cast<unsigned>(p.per) * kNumXcd;
}

// The CG direction p = r + beta p folded into the application of Q that follows
// it (a launch fewer per iteration): kFoldIn forms the input's neighbour spinors
// from the old p (in_all) and r as they are read, rounded as a stored p would be;
// kFoldOwn forms the site's own p (w_all is the old one), stores it into p_out
// and adds alpha times the old one to x. 8^4 FP32: 6.0 + 4.5 -> 7 us.
enum : int { kFoldNone = 0, kFoldIn = 1, kFoldOwn = 2, kFoldBoth = 3 };

__device__ __forceinline__ float pair_max(const cx<float> (&v)[2]) {
  return fmaxf(fmaxf(fabsf(v[0].re), fabsf(v[0].im)), fmaxf(fabsf(v[1].re), fabsf(v[1].im)));
}

// A spinor as its packed form holds it.
__device__ __forceinline__ void round_spinor(double, cx<double> (&)[12]) {}
__device__ __forceinline__ void round_spinor(float, cx<float> (&)[12]) {}
__device__ __forceinline__ void round_spinor(_Float16, cx<float> (&v)[12]) {
  h8 q[3];
  const float m = half_quantise(v, q);
#pragma unroll
  for (int j = 0; j < 3; ++j)
#pragma unroll
    for (int c = 0; c < 4; ++c)
      v[4 * j + c] = {fmar(static_cast<float>(q[j][2 * c]), m, 0.0f), fmar(static_cast<float>(q[j][2 * c + 1]), m, 0.0f)};
}

// x += a p on components 2j, 2j + 1 of a site (x FP64 for FP64 vectors, else the
// FP32 accumulator).
__device__ __forceinline__ void add_pair(void* x, long units, long k, int s, int j, const cx<double> (&p)[2], double a) {
  double2* const d = static_cast<double2*>(x) + k * units;
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    double2& v = d[pidx(s, 2 * j + e, 12, 0)];
    v = make_double2(fmar(a, p[e].re, v.x), fmar(a, p[e].im, v.y));
  }
}
__device__ __forceinline__ void add_pair(void* x, long units, long k, int s, int j, const cx<float> (&p)[2], float a) {
  float4& v = (static_cast<float4*>(x) + k * units)[pidx(s, j, 6, 0)];
  v = make_float4(fmar(a, p[0].re, v.x), fmar(a, p[0].im, v.y), fmar(a, p[1].re, v.z), fmar(a, p[1].im, v.w));
}

// lf: links of the forward hops (at the output site), lb: of the backward hops
// (at the neighbour); the same field unless eo. w_all may be null (no d * w).
template <typename T, bool C12, int CGM, bool BUF, int FOLD>
__global__ __launch_bounds__(kSplitThreads) void split_hop_kernel(
    const typename Packed<T>::S* __restrict__ in_all, const typename Packed<T>::S* __restrict__ w_all,
    typename Packed<T>::S* __restrict__ out_all, const typename Packed<T>::L* __restrict__ lf,
    const typename Packed<T>::L* __restrict__ lb, SplitCoef<typename Packed<T>::R> cf, long stride, int gamma5,
    SplitParams p, CgFuse cgf) {
  using R = typename Packed<T>::R;
  using GS = typename Packed<T>::S;
  __shared__ SplitHops<R> hops;
  __shared__ double red[CGM == kCgNone ? 1 : 6][kSplitSites];
  __shared__ float mx[sizeof(T) == 2 ? 6 : 1][kSplitSites];
  __shared__ float mp[sizeof(T) == 2 && (FOLD & kFoldOwn) != 0 ? 6 : 1][kSplitSites];
  __shared__ double aw[kSplitThreads / 64];

  int rhs;
  const int tile = split_tile<CGM == kCgNone>(p, &rhs);
  if (tile >= p.ntiles) return;
  const long k = cf.idx[rhs];
  const auto in = field_in<BUF>(in_all + k * stride, p.spinor_bytes);

  const int lane = threadIdx.x & 63;
  const int mu = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int site = lane & (kSplitSites - 1);
  const int up = lane / kSplitSites;  // 0: forward hop, 1: backward hop
  const int s0 = tile * kSplitSites + site;
  const bool valid = s0 < p.V;
  const int s = valid ? s0 : p.V - 1;
  const int nb = split_neighbour(p, mu, up, s);
  // the run's (first) CG slice, and the site at which a tile that begins inside the run cuts it in two
  int slice = tile, cut = kSplitSites;
  if (CGM != kCgNone && p.cut.tile != 0) {
    slice = p.cut.of(tile * kSplitSites);
    cut = (tile * kSplitSites / p.cut.tile + 1) * p.cut.tile - tile * kSplitSites;
  }

  cx<R> u[9], psi[12];
  if (lf == lb) {
    load_link<C12>(field_in<BUF>(lf, p.link_bytes), p.V, mu, up == 0 ? s : nb, u);
  } else if (up == 0) {
    load_link<C12>(field_in<BUF>(lf, p.link_bytes), p.V, mu, s, u);
  } else {
    load_link<C12>(field_in<BUF>(lb, p.link_bytes), p.V, mu, nb, u);
  }
  load_spinor(in, p.V, nb, psi);

  // what the second half needs: the site's own components 2j, 2j + 1
  const int j = 2 * mu + up;
  const bool mine = j < 6;
  cx<R> own[2] = {}, rv[2];
  if (mine && w_all != nullptr) load_pair(w_all + k * stride, p.V, s, j, own);
  constexpr bool kUsesR = CGM == kCgUpdate || FOLD != kFoldNone;
  GS* const r = kUsesR ? static_cast<GS*>(cgf.r) + k * stride : nullptr;
  double* const sc = kUsesR ? cgf.scal + k * kScalars : nullptr;
  if constexpr (FOLD != kFoldNone) {
    cx<R> rn[12];
    if constexpr ((FOLD & kFoldIn) != 0) load_spinor(field_in<BUF>(const_cast<const GS*>(r), p.spinor_bytes), p.V, nb, rn);
    if constexpr ((FOLD & kFoldOwn) != 0) {
      if (mine) load_pair(r, p.V, s, j, rv);
    }
    const double t = wave_total(strided_sum256(cgf.prr + k * cgf.nprr, cgf.nprr, threadIdx.x));
    if (lane == 0) aw[mu] = t;
    __syncthreads();
    double rr = 0.0;
    for (int w = 0; w < kSplitThreads / 64; ++w) rr += aw[w];
    const double old = sc[kRrPrev];
    const double beta = old > 0.0 ? rr / old : 0.0;
    const R b = static_cast<R>(beta);
    if constexpr ((FOLD & kFoldIn) != 0) {
#pragma unroll
      for (int c = 0; c < 12; ++c) psi[c] = {fmar(b, psi[c].re, rn[c].re), fmar(b, psi[c].im, rn[c].im)};
      round_spinor(T{}, psi);
    }
    if constexpr ((FOLD & kFoldOwn) != 0) {
      if (threadIdx.x == 0 && tile == 0) {  // only this workgroup writes the scalars, none reads these
        if (!isfinite(rr)) sc[kFlag] = 1.0;
        sc[kBeta] = beta;
        sc[kRr] = rr;
        if (rr > sc[kRrMax]) sc[kRrMax] = rr;
      }
      if (mine) {
        if (valid) add_pair(cgf.x, cgf.x_units, k, s, j, own, static_cast<R>(sc[kAlpha]));
#pragma unroll
        for (int e = 0; e < 2; ++e) own[e] = {fmar(b, own[e].re, rv[e].re), fmar(b, own[e].im, rv[e].im)};
        if constexpr (sizeof(T) == 2) mp[j][site] = pair_max(own);
      }
    }
  }
  if constexpr (CGM == kCgUpdate) {
    if (mine) load_pair(r, p.V, s, j, rv);
    const double t = wave_total(strided_sum256(cgf.pap + k * cgf.npap, cgf.npap, threadIdx.x));
    if (lane == 0) aw[mu] = t;
  }
  bool y_fwd_out = false, y_bwd_out = false;
  if (p.ny != 0 && p.ny != p.Y) {
    const unsigned y = (static_cast<unsigned>(s) / static_cast<unsigned>(p.X)) % static_cast<unsigned>(p.Y);
    const int yl = static_cast<int>(y % static_cast<unsigned>(p.ny));
    y_fwd_out = yl + 1 == p.ny;
    y_bwd_out = yl == 0;
  }

  {
    const R sg = up == 0 ? R(-1) : R(1);
    cx<R> h[6], g[6];
    if (mu == 0) project_sg<0>(psi, sg, h);
    else if (mu == 1) project_sg<1>(psi, sg, h);
    else if (mu == 2) project_sg<2>(psi, sg, h);
    else project_sg<3>(psi, sg, h);
    select_dagger(u, up != 0);
    su3_mul<false>(u, h, g);
#pragma unroll
    for (int a = 0; a < 6; ++a) hops.g[j][a][site] = g[a];
  }
  __syncthreads();

  if constexpr ((FOLD & kFoldOwn) != 0) {
    GS* const po = static_cast<GS*>(cgf.p_out) + k * stride;
    if constexpr (sizeof(T) == 2) {
      float m = 0.0f;
#pragma unroll
      for (int i = 0; i < 6; ++i) m = fmaxf(m, mp[i][site]);
      if (mine && valid) store_pair(po, s, j, own, m);
      half_pair(half_quantise_pair(own, m), m, own);
    } else {
      if (mine && valid) store_pair(po, p.V, s, j, own);
    }
  }

  cx<R> o[2];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int cc = mine ? 2 * j + e : 0;
    const bool lower = cc >= 6;
    const int c6 = lower ? cc - 6 : cc;
    const int half = c6 >= 3 ? 1 : 0;
    const int col = c6 - 3 * half;
    cx<R> acc = {R(0), R(0)};
    if (p.ny != 0) {
      add_hop<4>(hops, site, lower, half, col, acc);
      add_hop<5>(hops, site, lower, half, col, acc);
      if (y_fwd_out) add_hop<2>(hops, site, lower, half, col, acc);
      if (y_bwd_out) add_hop<3>(hops, site, lower, half, col, acc);
      add_hop<7>(hops, site, lower, half, col, acc);
      add_hop<6>(hops, site, lower, half, col, acc);
      add_hop<0>(hops, site, lower, half, col, acc);
      add_hop<1>(hops, site, lower, half, col, acc);
      if (!y_fwd_out) add_hop<2>(hops, site, lower, half, col, acc);
      if (!y_bwd_out) add_hop<3>(hops, site, lower, half, col, acc);
    } else {
      add_hop<0>(hops, site, lower, half, col, acc);
      add_hop<1>(hops, site, lower, half, col, acc);
      add_hop<2>(hops, site, lower, half, col, acc);
      add_hop<3>(hops, site, lower, half, col, acc);
      add_hop<4>(hops, site, lower, half, col, acc);
      add_hop<5>(hops, site, lower, half, col, acc);
      add_hop<6>(hops, site, lower, half, col, acc);
      add_hop<7>(hops, site, lower, half, col, acc);
    }
    const R d = cf.d[rhs], c = cf.c[rhs];
    if (w_all != nullptr) o[e] = {fmar(d, own[e].re, c * acc.re), fmar(d, own[e].im, c * acc.im)};
    else o[e] = {c * acc.re, c * acc.im};
    if (gamma5 && lower) o[e] = -o[e];
  }

  if constexpr (CGM == kCgUpdate) {  // r -= alpha A p, alpha as every workgroup finds it
    double t = 0.0;
    for (int w = 0; w < kSplitThreads / 64; ++w) t += aw[w];
    bool flag = false;
    const double alpha = cg_alpha(t, sc[kRr], &flag);
    if (threadIdx.x == 0 && tile == 0) {
      sc[kPap] = t;
      sc[kAlpha] = alpha;
      sc[kRrPrev] = sc[kRr];
      if (flag) sc[kFlag] = 1.0;
    }
    const R a = static_cast<R>(alpha);
#pragma unroll
    for (int e = 0; e < 2; ++e) o[e] = {fmar(-a, o[e].re, rv[e].re), fmar(-a, o[e].im, rv[e].im)};
  }

  // store, and with a CG mode the squared norm of the pair as stored
  GS* const dst = CGM == kCgUpdate ? r : out_all + k * stride;
  double n2 = 0.0;
  if constexpr (sizeof(T) == 2) {
    if (mine) mx[j][site] = pair_max(o);
    __syncthreads();
    float m = 0.0f;
#pragma unroll
    for (int i = 0; i < 6; ++i) m = fmaxf(m, mx[i][site]);
    if (mine && valid) n2 = store_pair(dst, s, j, o, m);
  } else {
    if (mine && valid) n2 = store_pair(dst, p.V, s, j, o);
  }
  if constexpr (CGM != kCgNone) {
    if (mine) red[j][site] = n2;
    __syncthreads();
    if (threadIdx.x < kSplitSites) {
      double v = red[0][site];
#pragma unroll
      for (int i = 1; i < 6; ++i) v += red[i][site];
      if (cut < kSplitSites && tile * kSplitSites + cut < p.V) {
        const double second = half_wave_total(site < cut ? 0.0 : v);
        if (site == 0) cgf.rr[k * cgf.nslices + slice + 1] = second;
        v = site < cut ? v : 0.0;
      }
      v = half_wave_total(v);
      if (site == 0) cgf.rr[k * cgf.nslices + slice] = v;
    }
  }
}

// Fields of ntiles tiles that fit one launch (HIP counts a launch's threads in 32
// bits; the grid is rounded up to the XCDs).
inline int split_fields_per_launch(int ntiles) {
  return static_cast<int>(std::min<long>(kMaxMultiRhs, (0xffffffffL / kSplitThreads - kNumXcd) / ntiles));
}

// Launches it; p's tiles are filled in here, link_bytes and spinor_bytes are 0
// where a field reaches 4 GiB (not with a fold, which small lattices use). A
// launch has fewer than 2^32 threads: eight per site and field pass that from
// 2^29 sites of all fields on (16 fields of 512 x 64 x 32 x 32), whose fields go
// in several launches then; three fields of the largest lattice fit one.
template <typename T, bool C12, int CGM, int FOLD = kFoldNone>
hipError_t launch_split_hop(const void* in, const void* w, void* out, const void* lf, const void* lb,
                            const SplitCoef<typename Packed<T>::R>& cf, long stride, int g5, SplitParams p,
                            const CgFuse& f, hipStream_t st) {
  using SV = typename Packed<T>::S;
  using LV = typename Packed<T>::L;
  p.ntiles = (p.V + kSplitSites - 1) / kSplitSites;
  const int nrhs = p.nrhs;
  const int most = split_fields_per_launch(p.ntiles);
  const auto run = [&](auto kernel) {
    for (int k0 = 0; k0 < nrhs; k0 += most) {
      SplitCoef<typename Packed<T>::R> part = cf;
      p.nrhs = nrhs - k0 < most ? nrhs - k0 : most;
      for (int k = 0; k < p.nrhs; ++k) {
        part.d[k] = cf.d[k0 + k];
        part.c[k] = cf.c[k0 + k];
        part.idx[k] = cf.idx[k0 + k];
      }
      const unsigned nb = split_grid(p);
      kernel<<<nb, kSplitThreads, 0, st>>>(static_cast<const SV*>(in), static_cast<const SV*>(w),
                                           static_cast<SV*>(out), static_cast<const LV*>(lf),
                                           static_cast<const LV*>(lb), part, stride, g5, p, f);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  };
  if (FOLD != kFoldNone && (f.r == nullptr || f.prr == nullptr || f.nprr < 1 || f.scal == nullptr))
    return hipErrorInvalidValue;
  if ((FOLD & kFoldOwn) != 0 && (f.p_out == nullptr || f.p_out == w || f.x == nullptr)) return hipErrorInvalidValue;
  if (p.link_bytes != 0 && p.spinor_bytes != 0) return run(&split_hop_kernel<T, C12, CGM, true, FOLD>);
  if constexpr (FOLD == kFoldNone) return run(&split_hop_kernel<T, C12, CGM, false, FOLD>);
  return hipErrorInvalidValue;
}

}  // namespace wd
