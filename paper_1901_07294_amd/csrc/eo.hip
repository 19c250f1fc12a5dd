// Hops between the two parities of an even-odd split lattice, for the Schur
// complement of the odd sites (eo.h), and gamma5 on FP64 fields.
//
// The eight neighbours of an output site all
// have the other parity: the x neighbours sit in the same half row at x
// half-index xh or xh +/- 1 (which one depends on the row's parity offset),
// the y, z and t neighbours at the same half index in the neighbouring half
// rows, planes and slices. The forward hop of direction mu uses the output
// site's own link (this parity's links), the backward hop the link of the
// neighbour it comes from (the other parity's links, at the neighbour's index).
// Over both parities every link is read once per application of H_{p,1-p},
// as in the full operator. HBM-bound on large lattices (8 links against 2 or 3
// spinors per output site), latency-bound on small ones.
#include "eo.h"
#include "split.h"
#include "stencil.h"

namespace wd {
namespace {

constexpr int kEoBlock = 256;

// Whether a launch takes the split kernel (eight lanes per output site) rather
// than one lane per site. In FP64 a lane that walks its hops keeps too few bytes
// in flight (one application of the Schur operator, one lane per site against
// split: 24^4 110 / 97 us, 24^3 x 48 235 / 201, 32^3 x 64 756 / 675, with two
// fields on 24^4 179 / 146); with FP32 arithmetic only while the launch is small
// (FP32: 16^4 16.4 / 14.0, with four fields 27.3 / 31.5; FP16: 12^4 13.9 / 12.1,
// 16^4 with two fields 14.8 / 17.3, 24^4 27.7 / 33.1). Between those, FP64 launches of
// up to 65536 half sites are one wave per SIMD of the other kernel, which then ends
// with its only round, and split ones three rounds of workgroups (16^4 with two
// fields 28.8 / 31.6, 12-real links 26.4 / 30.8; 16^3 x 32 37.1 / 37.3, 29.8 / 34.7; beyond
// it, 16^3 x 24 with two fields 56.0 / 43.9). 12-real links, a third less to read, move
// the lower end (8^2 x 12 x 16 with eight fields 20.6 / 22.3, else 22.6 / 21.3). Fused
// FP64 hops are always split (an iteration on 16^4 with two fields 93 / 89). Same bits
// either way.
bool use_split_eo(int prec, bool c12, long Vh, int nrhs) {
  const long w = Vh * nrhs;
  if (prec != WD_FP64) return w <= 48000;
  return w <= (c12 ? 48000 : 52000) || w > 65536;
}

// One lane per output half site, or (p.eo == 0) per site of a whole lattice.
// Workgroups of 256 half sites; the links and the
// input through buffer resources where they fit. Against plain pointers and a
// grid row per right-hand side (us per application of the Schur operator): FP16
// 24^4 36.3 -> 27.7, with four fields 97.6 -> 69.1; FP32 24^3 x 48 104 -> 98, with
// two fields 202 -> 164.
template <typename T, bool C12, int CGM, bool BUF>
__global__ __launch_bounds__(kEoBlock) void eo_hop_kernel(
    const typename Packed<T>::S* __restrict__ in_all, const typename Packed<T>::S* __restrict__ w_all,
    typename Packed<T>::S* __restrict__ out_all, const typename Packed<T>::L* __restrict__ lp,
    const typename Packed<T>::L* __restrict__ lq, SplitCoef<typename Packed<T>::R> cf, long stride, int gamma5,
    SplitParams p, CgFuse cgf) {
  using R = typename Packed<T>::R;
  using GS = typename Packed<T>::S;
  __shared__ double aw[kEoBlock / 64];
  int rhs;
  const int tile = split_tile<CGM == kCgNone>(p, &rhs);
  if (tile >= p.ntiles) return;
  const long k = cf.idx[rhs];
  const int h0 = tile * kEoBlock + static_cast<int>(threadIdx.x);
  const bool valid = h0 < p.V;
  const int h = valid ? h0 : p.V - 1;
  const long V = p.V;
  const auto in = field_in<BUF>(in_all + k * stride, p.spinor_bytes);
  const auto fp = field_in<BUF>(lp, p.link_bytes);
  const auto fq = field_in<BUF>(lq, p.link_bytes);

  GS* const r = CGM == kCgUpdate ? static_cast<GS*>(cgf.r) + k * stride : nullptr;
  double* const sc = CGM == kCgUpdate ? cgf.scal + k * kScalars : nullptr;
  if constexpr (CGM == kCgUpdate) {
    const double t = wave_total(strided_sum256(cgf.pap + k * cgf.npap, cgf.npap, threadIdx.x));
    if ((threadIdx.x & 63) == 0) aw[threadIdx.x / 64] = t;
    __syncthreads();
  }

  cx<R> acc[12];
#pragma unroll
  for (int c = 0; c < 12; ++c) acc[c] = {R(0), R(0)};
  // x + 1 is 2 xh + o + 1: half index xh when o = 0, xh + 1 (wrapping) when o = 1;
  // x - 1 is 2 xh + o - 1: xh - 1 (wrapping) when o = 0, xh when o = 1
  const int row = h / p.X, xh = h - row * p.X;
  const int y = row % p.Y, zt = row / p.Y, z = zt % p.Z, t = zt / p.Z;
  const int o = (y + z + t + p.parity) & 1;
  const int xp = !p.eo || o ? (xh + 1 == p.X ? h - (p.X - 1) : h + 1) : h;
  const int xm = p.eo && o ? h : (xh == 0 ? h + (p.X - 1) : h - 1);
  const int yp = y + 1 == p.Y ? h - (p.Y - 1) * p.sy : h + p.sy;
  const int ym = y == 0 ? h + (p.Y - 1) * p.sy : h - p.sy;
  const int zp = z + 1 == p.Z ? h - (p.Z - 1) * p.sz : h + p.sz;
  const int zm = z == 0 ? h + (p.Z - 1) * p.sz : h - p.sz;
  const int tp = t + 1 == p.T ? h - (p.T - 1) * p.st : h + p.st;
  const int tm = t == 0 ? h + (p.T - 1) * p.st : h - p.st;
  hop<0, -1, C12>(in, fp, V, xp, h, acc);
  hop<0, +1, C12>(in, fq, V, xm, xm, acc);
  hop<1, -1, C12>(in, fp, V, yp, h, acc);
  hop<1, +1, C12>(in, fq, V, ym, ym, acc);
  hop<2, -1, C12>(in, fp, V, zp, h, acc);
  hop<2, +1, C12>(in, fq, V, zm, zm, acc);
  hop<3, -1, C12>(in, fp, V, tp, h, acc);
  hop<3, +1, C12>(in, fq, V, tm, tm, acc);

  const R d = cf.d[rhs], c = cf.c[rhs];
  cx<R> res[12];
  if (w_all != nullptr) {
    cx<R> wv[12];
    load_spinor(w_all + k * stride, V, h, wv);
#pragma unroll
    for (int i = 0; i < 12; ++i) res[i] = {fmar(d, wv[i].re, c * acc[i].re), fmar(d, wv[i].im, c * acc[i].im)};
  } else {
#pragma unroll
    for (int i = 0; i < 12; ++i) res[i] = {c * acc[i].re, c * acc[i].im};
  }
  if (gamma5) {
#pragma unroll
    for (int i = 6; i < 12; ++i) res[i] = -res[i];
  }
  if constexpr (CGM == kCgNone) {
    if (valid) store_spinor(out_all + k * stride, V, h, res);
  } else {
    double n2 = 0.0;
    if constexpr (CGM == kCgNorm) {
      if (valid) n2 = store_site_norm(out_all + k * stride, V, h, res);
    } else {
      double pap = 0.0;
      for (int w = 0; w < kEoBlock / 64; ++w) pap += aw[w];
      bool flag = false;
      const double alpha = cg_alpha(pap, sc[kRr], &flag);
      if (h0 == 0) {
        sc[kPap] = pap;
        sc[kAlpha] = alpha;
        sc[kRrPrev] = sc[kRr];
        if (flag) sc[kFlag] = 1.0;
      }
      if (valid) n2 = cg_site_update_r(r, V, h, res, alpha);
    }
    // slices of 32 sites, as the split kernel's, or of the whole workgroup
    n2 = half_wave_total(n2);
    if (!p.wide) {
      const int slice = h0 / kSplitSites;
      if (threadIdx.x % kSplitSites == 0 && slice < cgf.nslices) cgf.rr[k * cgf.nslices + slice] = n2;
    } else {
      n2 += __shfl_xor(n2, 32, 64);
      __syncthreads();
      if ((threadIdx.x & 63) == 0) aw[threadIdx.x / 64] = n2;
      __syncthreads();
      if (threadIdx.x == 0) cgf.rr[k * cgf.nslices + tile] = ((aw[0] + aw[1]) + aw[2]) + aw[3];
    }
  }
}

// dst = gamma5 src on FP64 packed fields: plane 3 * spin + colour, spins 2
// and 3 negated.
__global__ __launch_bounds__(256) void gamma5_kernel(double2* __restrict__ dst, const double2* __restrict__ src,
                                                     long n, RhsSet set) {
  const long k = set.idx[blockIdx.y];
  for (long e = static_cast<long>(blockIdx.x) * 256 + threadIdx.x; e < n;
       e += static_cast<long>(gridDim.x) * 256) {
    const int plane = static_cast<int>((e / kLayoutBlock) % 12);
    double2 v = src[k * n + e];
    if (plane >= 6) v = make_double2(-v.x, -v.y);
    dst[k * n + e] = v;
  }
}

// CG slices of 256 sites, which only the one-lane-per-site kernel sums: on
// lattices where slices of 32 would leave more partial sums than every workgroup
// of the next kernel should read.
bool wide_slices(long Vh) { return Vh > 131072; }

template <typename T, bool C12, int CGM, int FOLD = kFoldNone>
hipError_t launch_hop_t(const wd_gauge* g, int p, const void* in, const void* w, void* out, const RhsSet& set,
                        const double* d, const double* c, int g5, const CgFuse& f, hipStream_t s) {
  using L = typename Packed<T>::L;
  using R = typename Packed<T>::R;
  const EoGeo geo = make_eo_geo(g->dims);
  SplitCoef<R> cf{};
  for (int i = 0; i < set.n; ++i) {
    cf.d[i] = static_cast<R>(d[i]);
    cf.c[i] = static_cast<R>(c[i]);
    cf.idx[i] = set.idx[i];
  }
  const size_t half = eo_gauge_half_bytes(geo.Vh, g->prec, g->c12);
  const char* links = static_cast<const char*>(g->links);
  const L* lp = reinterpret_cast<const L*>(links + p * half);        // this parity: forward hops
  const L* lq = reinterpret_cast<const L*>(links + (p ^ 1) * half);  // the other: backward hops
  const long stride = spinor_units<T>(geo.Vh);
  SplitParams sp{geo.Xh, geo.Y, geo.Z, geo.T, geo.Xh, geo.Xh * geo.Y, geo.Xh * geo.Y * geo.Z,
                 static_cast<int>(geo.Vh), 1, p, wide_slices(geo.Vh) ? 1 : 0};
  sp.nrhs = set.n;
  sp.link_bytes = half < (1ul << 32) ? static_cast<unsigned>(half) : 0u;
  sp.spinor_bytes = stride * 16 < (1l << 32) ? static_cast<unsigned>(stride * 16) : 0u;
  if constexpr (FOLD != kFoldNone || (sizeof(R) == 8 && CGM != kCgNone)) {
    return launch_split_hop<T, C12, CGM, FOLD>(in, w, out, lp, lq, cf, stride, g5, sp, f, s);
  } else {
    if (use_split_eo(g->prec, C12, geo.Vh, set.n) && !(CGM != kCgNone && wide_slices(geo.Vh)))
      return launch_split_hop<T, C12, CGM, FOLD>(in, w, out, lp, lq, cf, stride, g5, sp, f, s);
    sp.ntiles = (sp.V + kEoBlock - 1) / kEoBlock;
    const unsigned nb = split_grid(sp);
    const auto run = [&](auto kernel) {
      kernel<<<nb, kEoBlock, 0, s>>>(static_cast<const typename Packed<T>::S*>(in),
                                     static_cast<const typename Packed<T>::S*>(w),
                                     static_cast<typename Packed<T>::S*>(out), lp, lq, cf, stride, g5, sp, f);
      return hipGetLastError();
    };
    if (sp.link_bytes != 0 && sp.spinor_bytes != 0) return run(&eo_hop_kernel<T, C12, CGM, true>);
    return run(&eo_hop_kernel<T, C12, CGM, false>);
  }
}

template <typename T, bool C12>
hipError_t launch_hop_mode(const wd_gauge* g, int p, const void* in, const void* w, void* out, const RhsSet& set,
                           const double* d, const double* c, int g5, const CgFuse* f, hipStream_t s) {
  if (f == nullptr) return launch_hop_t<T, C12, kCgNone>(g, p, in, w, out, set, d, c, g5, CgFuse{}, s);
  // with a fold, the hop onto the even sites (no w) reads p, the one back owns it
  if (f->p_out != nullptr && w == nullptr)
    return launch_hop_t<T, C12, kCgNone, kFoldIn>(g, p, in, w, out, set, d, c, g5, *f, s);
  if (f->rr == nullptr || f->nslices < eo_fuse_slices(g->dims, g->prec) || f->nslices < 1)
    return hipErrorInvalidValue;
  if (f->mode == kCgNorm && f->p_out != nullptr)
    return launch_hop_t<T, C12, kCgNorm, kFoldOwn>(g, p, in, w, out, set, d, c, g5, *f, s);
  if (f->mode == kCgNorm) return launch_hop_t<T, C12, kCgNorm>(g, p, in, w, out, set, d, c, g5, *f, s);
  if (f->mode != kCgUpdate || f->r == nullptr || f->pap == nullptr || f->npap < 1 || f->scal == nullptr)
    return hipErrorInvalidValue;
  return launch_hop_t<T, C12, kCgUpdate>(g, p, in, w, out, set, d, c, g5, *f, s);
}

template <typename T>
hipError_t launch_hop_prec(const wd_gauge* g, int p, const void* in, const void* w, void* out,
                           const RhsSet& set, const double* d, const double* c, int g5, const CgFuse* f,
                           hipStream_t s) {
  return g->c12 ? launch_hop_mode<T, true>(g, p, in, w, out, set, d, c, g5, f, s)
                : launch_hop_mode<T, false>(g, p, in, w, out, set, d, c, g5, f, s);
}

hipError_t launch_hop(const wd_gauge* g, int parity, const void* in, const void* w, void* out, const RhsSet& set,
                      const double* d, const double* c, int g5, const CgFuse* f, hipStream_t s) {
  if (set.n < 1) return hipSuccess;
  if (set.n > kMaxRhs || !g->eo || (parity != 0 && parity != 1)) return hipErrorInvalidValue;
  switch (g->prec) {
    case WD_FP64: return launch_hop_prec<double>(g, parity, in, w, out, set, d, c, g5, f, s);
    case WD_FP32: return launch_hop_prec<float>(g, parity, in, w, out, set, d, c, g5, f, s);
    case WD_FP16: return launch_hop_prec<_Float16>(g, parity, in, w, out, set, d, c, g5, f, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_site_cg(const wd_gauge* g, const double* masses, int nrhs, const int* fields, const void* in,
                          void* out, const CgFuse& f, hipStream_t st) {
  const Geo geo = make_geo(g->dims);
  const long stride = spinor_units<_Float16>(geo.V);
  if (g->eo || g->prec != WD_FP16 || nrhs < 1 || nrhs > kMaxRhs || f.rr == nullptr ||
      f.nslices < (geo.V + kSplitSites - 1) / kSplitSites || g->link_bytes >= (1ul << 32) || stride * 16 >= (1l << 32))
    return hipErrorInvalidValue;
  if (f.mode == kCgUpdate && (f.r == nullptr || f.pap == nullptr || f.npap < 1 || f.scal == nullptr))
    return hipErrorInvalidValue;
  SplitCoef<float> cf{};
  for (int k = 0; k < nrhs; ++k) {
    cf.d[k] = static_cast<float>(4.0 + masses[k]);
    cf.c[k] = -0.5f;
    cf.idx[k] = fields ? fields[k] : k;
  }
  SplitParams p{geo.X, geo.Y, geo.Z, geo.T, geo.X, geo.XY, geo.XYZ, geo.V};
  p.nrhs = nrhs;
  p.link_bytes = static_cast<unsigned>(g->link_bytes);
  p.spinor_bytes = static_cast<unsigned>(stride * 16);
  p.ntiles = (p.V + kEoBlock - 1) / kEoBlock;
  const unsigned nb = split_grid(p);
  const auto run = [&](auto kernel) {
    const h2* links = static_cast<const h2*>(g->links);
    kernel<<<nb, kEoBlock, 0, st>>>(static_cast<const h8*>(in), static_cast<const h8*>(in), static_cast<h8*>(out),
                                    links, links, cf, stride, 1, p, f);
    return hipGetLastError();
  };
  if (f.mode == kCgNorm)
    return g->c12 ? run(&eo_hop_kernel<_Float16, true, kCgNorm, true>)
                  : run(&eo_hop_kernel<_Float16, false, kCgNorm, true>);
  if (f.mode == kCgUpdate)
    return g->c12 ? run(&eo_hop_kernel<_Float16, true, kCgUpdate, true>)
                  : run(&eo_hop_kernel<_Float16, false, kCgUpdate, true>);
  return hipErrorInvalidValue;
}

int eo_fuse_slices(const int32_t dims[4], int prec) {
  const long Vh = make_eo_geo(dims).Vh;
  if (!wide_slices(Vh)) return static_cast<int>((Vh + kSplitSites - 1) / kSplitSites);
  // Every workgroup of an update adds all partial sums of its field: reading that
  // grows with Vh^2, and with its share the gain (us per iteration unfused / fused:
  // FP16 64^4 7323 / 7172, 80^3 x 64 13990 / 14400; FP32 64^4 10570 / 9980, 80^3 x 64 20700 /
  // 20160, 80^3 x 68 21920 / 21360). The two meet at about these half volumes.
  constexpr long kLargest[] = {131072, 23000000, 11500000};  // FP64, FP32, FP16
  return Vh > kLargest[prec] ? 0 : static_cast<int>((Vh + kEoBlock - 1) / kEoBlock);
}

// Five launches per iteration become four; r is read by both hops. 8^4 FP64 35.9
// -> 33.5 us per iteration, FP16 41.4 -> 36.3; 12^4 with two fields FP64 43.6 ->
// 44.3 but FP16 42.3 -> 37.3; 16^4 FP32 47.0 -> 46.3, with four fields 97 -> 106;
// FP16 with two fields 60.8 -> 60.0, with four 79.6 -> 88.0.
bool eo_fold_p(const int32_t dims[4], int prec, int n) {
  const long Vh = make_eo_geo(dims).Vh;
  return !wide_slices(Vh) && Vh * n <= (prec == WD_FP64 ? 12000 : prec == WD_FP32 ? 32768 : 80000);
}

hipError_t launch_eo_hop(const wd_gauge* g, int parity, const void* in, const void* w, void* out,
                         const RhsSet& set, const double* d, const double* c, int g5, hipStream_t s) {
  return launch_hop(g, parity, in, w, out, set, d, c, g5, nullptr, s);
}

hipError_t launch_schur_q(const wd_gauge* g, const double* masses, const RhsSet& set, const void* in,
                          void* tmp, void* out, const CgFuse* f, hipStream_t s) {
  double d[kMaxRhs], c[kMaxRhs];
  for (int i = 0; i < set.n; ++i) {
    d[i] = 0.0;
    c[i] = -0.5;
  }
  const bool fold = f != nullptr && f->p_out != nullptr;
  hipError_t e = launch_hop(g, 0, in, nullptr, tmp, set, d, c, 0, fold ? f : nullptr, s);
  if (e != hipSuccess) return e;
  for (int i = 0; i < set.n; ++i) {
    const double a = 4.0 + masses[i];
    d[i] = a;
    c[i] = 1.0 / (2.0 * a);
  }
  return launch_hop(g, 1, tmp, in, out, set, d, c, 1, f, s);
}

hipError_t blas_gamma5(void* dst, const void* src, long n, const RhsSet& set, hipStream_t st) {
  if (set.n == 0) return hipSuccess;
  long nb = (n + 1023) / 1024;
  nb = nb < 1 ? 1 : (nb > 4096 ? 4096 : nb);
  gamma5_kernel<<<dim3(static_cast<unsigned>(nb), set.n), 256, 0, st>>>(
      static_cast<double2*>(dst), static_cast<const double2*>(src), n, set);
  return hipGetLastError();
}

}  // namespace wd
