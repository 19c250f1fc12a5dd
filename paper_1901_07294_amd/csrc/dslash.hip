// The Wilson-Dirac operator on gfx950: one lane per lattice site on large
// lattices (the t-marching kernel below), eight on small ones (split.h), and one
// in FP16 storage on larger ones that the march cannot tile.
//
//   out(x) = (4+m) psi(x) - 1/2 sum_mu [ (1-g_mu) U_mu(x) psi(x+mu)
//                                       + (1+g_mu) U_mu(x-mu)^dag psi(x-mu) ]
//
// (the hopping term of eq. (1), Sec. II-A, with the opposite sign of gamma_mu
// and the (4+m) normalisation), optionally multiplied by gamma5 = diag(1,1,-1,-1).
//
// The stencil is bound by HBM bandwidth (1320 flop against >= 960 compulsory
// bytes per site in FP64), so there is no matrix-core work here: every lane
// streams its site's links and spinor planes, coalesced across the wave.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <numeric>
#include <type_traits>

#include "blas.h"
#include "cg_site.h"
#include "split.h"
#include "stencil.h"
#include "wd_internal.h"

// Compile-time tuning knobs (the defaults are the measured best on MI355X).
#ifndef WD_SPLIT_SITES
#define WD_SPLIT_SITES 49152  // sites times fields up to which the split kernel is always taken
#endif
#ifndef WD_MARCH_THREADS
#define WD_MARCH_THREADS 256  // target sites per t-marching tile
#endif
#ifndef WD_UT_NT
#define WD_UT_NT 1            // non-temporal loads of the t links in the t-marching kernel
#endif
#ifndef WD_MARCH_BUF
#define WD_MARCH_BUF 1        // FP64/FP32 fields below 4 GiB through buffer resources
#endif
#ifndef WD_X_SHFL
#define WD_X_SHFL 1           // backward x links from the neighbour lane (x rows within a wave)
#endif

namespace wd {
namespace {

constexpr int kMarchMaxThreads = 256;       // lanes of a one-right-hand-side tile
constexpr int kMarchMultiThreads = 768;     // lanes of a several-right-hand-side workgroup
constexpr int kMarchTargetThreads = WD_MARCH_THREADS;
constexpr bool kUtNt = WD_UT_NT != 0;
constexpr bool kMarchBuf = WD_MARCH_BUF != 0;
constexpr bool kXShfl = WD_X_SHFL != 0;
constexpr int kNumCu = 256;
constexpr size_t kLdsBytes = 160 * 1024;  // LDS per CU on gfx950

// Workgroup -> tile. Consecutive workgroups are dispatched round-robin over the
// 8 XCDs, each with its own L2; with group > 0 the mapping gives every XCD runs
// of `group` consecutive tiles, so that neighbours in y and z, which sit a few
// tiles away, share an L2. A group of at least an eighth of the nb tiles gives
// each XCD one run; the grid then is 8 groups, and workgroups past the last tile
// (a result of nb or more) have nothing to do.
__device__ __forceinline__ int tile_of_block(int group, int nb) {
  const int b = blockIdx.x;
  if (group <= 0) return b;
  const int xcd = b % kNumXcd;
  const int l = b / kNumXcd;
  if (static_cast<long>(group) * kNumXcd >= nb) return xcd * group + l;
  if (nb % (kNumXcd * group) != 0) return b;
  return ((l / group) * kNumXcd + xcd) * group + (l % group);
}

// ---------------------------------------------------------------------------
// One lane per site, FP16 storage, on lattices without t-marching tiles (x rows
// longer than 256 sites, or fewer than 64 sites in the longest run of whole rows
// that divides y, as with a prime number of short rows).
//
// FP16 fields are few bytes and much conversion: with eight lanes per site every
// lane converts a spinor for one hop and, with 12-real links, rebuilds a third
// row, which is what bounds that kernel. Here a lane walks the eight hops, in the
// same order. What counts is that every CU gets work (workgroups of one wave) and
// that a wave keeps enough loads in flight: bound to four waves per SIMD the
// kernel takes 86 registers; left to itself the compiler stops at 66 and waits
// more often (300 x 4 x 4 x 20 10.4 -> 8.5 us). Eight lanes -> one lane, us: 24 x 17 x
// 20 x 60 43 -> 29, with 12-real links 43 -> 28 and with 12 fields of them 514 ->
// 311; 4^3 x 512 with 12 fields 31 -> 18.3, one field 6.1 -> 6.2.
// ---------------------------------------------------------------------------

constexpr int kSiteBlock = 64;
// Sites times fields from which it runs: below, one wave of eight lanes per site
// hides more latency (7 x 4 x 12 x 14 with three fields 5.3 / 5.8 us, 10 x 5 x 16 x 14
// with two 6.2 / 6.3 and with three 6.9 / 6.4).
constexpr long kSiteSites = 24576;
// ... and beyond which the fused CG work does, by the even-odd hop kernel (eo.hip),
// which sums the same slices. Eight lanes / one, us per iteration: 4^3 x 512 22.9 /
// 24.1, 10 x 5 x 16 x 14 with four fields 29.6 / 29.5, 33 x 17 x 11 x 7 with two 41.1 /
// 38.6 and with 16 182 / 127.
constexpr long kSiteCgSites = 45000;

template <bool C12, bool BUF>
__global__ __launch_bounds__(kSiteBlock) __attribute__((amdgpu_waves_per_eu(4, 4))) void dslash_site_kernel(
    const h8* __restrict__ in_all, h8* __restrict__ out_all, const h2* __restrict__ links, Diag<float> diags,
    long stride, int gamma5, SplitParams p) {
  int rhs;
  const int tile = split_tile<true>(p, &rhs);
  const int s = tile * kSiteBlock + static_cast<int>(threadIdx.x);
  if (tile >= p.ntiles || s >= p.V) return;
  const long V = p.V;
  const long k = diags.idx[rhs];
  const auto in = field_in<BUF>(in_all + k * stride, p.spinor_bytes);
  const auto lk = field_in<BUF>(links, p.link_bytes);
  const int xp = split_neighbour(p, 0, 0, s), xm = split_neighbour(p, 0, 1, s);
  const int yp = split_neighbour(p, 1, 0, s), ym = split_neighbour(p, 1, 1, s);
  const int zp = split_neighbour(p, 2, 0, s), zm = split_neighbour(p, 2, 1, s);
  const int tp = split_neighbour(p, 3, 0, s), tm = split_neighbour(p, 3, 1, s);
  cx<float> acc[12], psi[12], o[12];
#pragma unroll
  for (int c = 0; c < 12; ++c) acc[c] = {0.0f, 0.0f};
  hop<0, -1, C12>(in, lk, V, xp, s, acc);
  hop<0, +1, C12>(in, lk, V, xm, xm, acc);
  hop<1, -1, C12>(in, lk, V, yp, s, acc);
  hop<1, +1, C12>(in, lk, V, ym, ym, acc);
  hop<2, -1, C12>(in, lk, V, zp, s, acc);
  hop<2, +1, C12>(in, lk, V, zm, zm, acc);
  hop<3, -1, C12>(in, lk, V, tp, s, acc);
  hop<3, +1, C12>(in, lk, V, tm, tm, acc);
  load_spinor(in, V, s, psi);
  epilogue(psi, acc, diags.d[rhs], gamma5, o);
  store_spinor(field_out<BUF>(out_all + k * stride, p.spinor_bytes), V, s, o);
}

// ---------------------------------------------------------------------------
// t-marching kernel.
//
// A workgroup owns a tile of X x NY sites (whole x rows) at one z and walks
// t0 .. t1-1. The tile's spinors at the current t sit in LDS, so the x and
// in-tile y neighbours are read from LDS; the t neighbours come from the march
// itself: psi(t+1) is the workgroup's own next slice, and the backward t hop of
// step t+1, U_t(t)^dag P+ psi(t), is built from data of step t and carried. The
// z hops and the y hops that leave the tile need other workgroups' sites; in
// large FP64 tiles they are done one step early, while the workgroups that own
// those sites load the same slice, so their lines are still in L2. Which
// variant runs where: launch_march_b.
// ---------------------------------------------------------------------------

struct MarchParams {
  int ny;      // rows per tile (divides Y)
  int tb;      // t steps per workgroup
  int ytiles;  // Y / ny
  int group;   // XCD run length (workgroups), 0 = hardware order
  int nb;      // workgroups that have work
  int nrhs;    // right-hand sides of the launch
  int gw;      // lane groups per workgroup
  int rb;      // right-hand sides per lane (gw * rb divides nrhs)
  bool ahead;  // FP64: kOuterAhead
  CgSlices cut;  // SMALL: the sites' CG slices
  unsigned link_bytes;    // bytes of the packed links and of one packed spinor field (used
  unsigned spinor_bytes;  // when they are read through buffer resources, below 4 GiB)
};

// One hop for the RB right-hand sides of a lane: the link (direction MU at
// site ls) is loaded once and applied to each one's neighbour spinor at site
// nb. Each right-hand side sees exactly the operations of a one-field hop.
template <int MU, int S, bool C12, int RB, typename SA, typename LA, typename R>
__device__ __forceinline__ void hop_rb(const SA (&in)[RB], const LA& links, long V, int nb, int ls,
                                       cx<R> (&acc)[RB][12]) {
  cx<R> u[9];
  load_link<C12>(links, V, MU, ls, u);
#pragma unroll
  for (int r = 0; r < RB; ++r) {
    cx<R> psi[12];
    load_spinor(in[r], V, nb, psi);
    cx<R> h[6], g[6];
    project<MU, S>(psi, h);
    su3_mul<(S > 0)>(u, h, g);
    reconstruct_add<MU, S>(g, acc[r]);
  }
}

// The same with the neighbour spinors read from the LDS slices (slot li).
template <int MU, int S, bool C12, int RB, typename SL, typename LA, typename R>
__device__ __forceinline__ void lds_hop_rb(SL* const (&slice)[RB], int n, int li, const LA& links, long V,
                                           int ls, cx<R> (&acc)[RB][12]) {
  cx<R> u[9];
  load_link<C12>(links, V, MU, ls, u);
#pragma unroll
  for (int r = 0; r < RB; ++r) {
    cx<R> psi[12];
    lds_load_spinor(slice[r], n, li, psi);
    cx<R> h[6], g[6];
    project<MU, S>(psi, h);
    su3_mul<(S > 0)>(u, h, g);
    reconstruct_add<MU, S>(g, acc[r]);
  }
}

// The same with the link already in registers.
template <int MU, int S, int RB, typename SL, typename R>
__device__ __forceinline__ void lds_hop_u(SL* const (&slice)[RB], int n, int li, const cx<R> (&u)[9],
                                          cx<R> (&acc)[RB][12]) {
#pragma unroll
  for (int r = 0; r < RB; ++r) {
    cx<R> psi[12];
    lds_load_spinor(slice[r], n, li, psi);
    cx<R> h[6], g[6];
    project<MU, S>(psi, h);
    su3_mul<(S > 0)>(u, h, g);
    reconstruct_add<MU, S>(g, acc[r]);
  }
}

// Both x hops from LDS. The backward hop's link U_x(x - 1) is the forward
// hop's link of the lane holding x - 1; with xshfl (every x row lies within
// one wave: X divides 64) it is taken from that lane with a cross-lane
// shuffle (the same values, no memory access), otherwise loaded.
template <bool C12, int RB, typename SL, typename LA, typename R>
__device__ __forceinline__ void lds_x_hops(SL* const (&slice)[RB], int n, int lxp, int lxm, const LA& links,
                                           long V, int st, int dxm, bool xshfl, int src_lane,
                                           cx<R> (&acc)[RB][12]) {
  cx<R> u[9];
  load_link<C12>(links, V, 0, st, u);
  lds_hop_u<0, -1>(slice, n, lxp, u, acc);
  if (xshfl) {
#pragma unroll
    for (int k = 0; k < 9; ++k) u[k] = {__shfl(u[k].re, src_lane, 64), __shfl(u[k].im, src_lane, 64)};
  } else {
    load_link<C12>(links, V, 0, st + dxm, u);
  }
  lds_hop_u<0, +1>(slice, n, lxm, u, acc);
}

// Hops of time t that involve sites outside the tile: z forward and
// backward, and the y hops of the tile's edge rows.
template <bool C12, int RB, typename SA, typename LA, typename R>
__device__ __forceinline__ void outer_hops(const SA (&in)[RB], const LA& links, long V, int st, int dzp,
                                           int dzm, bool y_fwd_out, int dyp, bool y_bwd_out, int dym,
                                           cx<R> (&acc)[RB][12]) {
  hop_rb<2, -1, C12>(in, links, V, st + dzp, st, acc);
  hop_rb<2, +1, C12>(in, links, V, st + dzm, st + dzm, acc);
  if (y_fwd_out) hop_rb<1, -1, C12>(in, links, V, st + dyp, st, acc);
  if (y_bwd_out) hop_rb<1, +1, C12>(in, links, V, st + dym, st + dym, acc);
}

// Doubles of LDS per lane group and right-hand side that the fused CG work
// uses after the spinor slices: per-wave sums of two steps (tiles of at most
// 4 waves) and the four sums of <p, A p>. SMALL: the sites' norms of two steps
// follow them.
constexpr int kCgLds = 2 * 4 + 4;

// Variants of the march (KIND):
//  kOuterAhead  two LDS slices; the outer hops (z, and y out of the tile) of t+1
//               are done in step t, into a second accumulator.
//  kOuterNow    two LDS slices; the outer hops of t are done at the start of step
//               t, and only the backward t hop of t+1, before its reconstruction,
//               is carried: 48 registers fewer in FP64 per field, 24 in FP32.
//  kOneBuffer   kOuterNow with one LDS slice: psi(t+1) is loaded again when step t
//               is done with the slice, which costs a second barrier.
//  kOneSlice    marches of a single slice: nothing to carry, one LDS slice.
// Every site's hops are added in the same order in all of them.
constexpr int kOuterAhead = 0, kOuterNow = 1, kOneBuffer = 2, kOneSlice = 3;

// MAXT: launch bound. A workgroup holds p.gw groups of n = X * ny lanes of
// one tile; each lane carries RB right-hand sides (links loaded once for
// all), each with its own two LDS slices. The LDS slices hold spinors in the
// arithmetic precision (FP32 for FP16 storage).
// CGM (CG iterations, n a multiple of 64 unless SMALL): kCgNorm stores the output
// and leaves each tile slice's squared norm of it in cgf.rr; kCgUpdate does not
// store the output but applies r -= alpha A p of cgf to the field slots (x
// and p follow in a separate kernel).
// SMALL: the CG slices of small lattices (CgSlices) instead, and the sums of <p, A p>
// in the split kernel's order: the same bits as that kernel's, on tiles of any
// number of lanes.
// The fused modes with FP32 arithmetic and one right-hand side per lane are
// compiled for three waves per SIMD, the plain FP32-arithmetic kernel's
// occupancy; only their plain-pointer forms (fields or links of 4 GiB and more)
// spill for it, eight or nine registers in FP32 storage.
// kOneSlice (p.tb == 1): without a next slice there is one LDS slice and no
// accumulator or link column carried on, which brings FP16
// storage from 160 registers to 127 and, bound to five waves per SIMD, to 96
// without a spill (2 to 3 % faster than at four with several fields; six waves
// spill or serialise the loads: 3 to 7 % slower). Twice the waves outweigh that t
// neighbours' spinors and links are read from L2: the FP16 operator on 24^4 with
// one field 24.3 -> 22.0 us, 28 x 15 x 22 x 33 28.7 -> 24.7 us, 16^4 10.3 -> 6.9
// us; a solve with FP16 inner iterations on 16^3 x 32 7.9 -> 7.0 ms.
template <int CGM, typename T, int RB, int KIND>
constexpr int march_waves_per_eu() {
  if (KIND == kOneSlice) return sizeof(T) == 2 && CGM == kCgNone ? 5 : 1;
  return RB == 1 && sizeof(typename Packed<T>::R) == 4 && CGM != kCgNone ? 3 : 1;
}

template <typename T, bool C12, int MAXT, int RB, int CGM, bool BUF, int KIND, bool SMALL>
__global__ __launch_bounds__(MAXT)
__attribute__((amdgpu_waves_per_eu(march_waves_per_eu<CGM, T, RB, KIND>()))) void dslash_march_kernel(
    const typename Packed<T>::S* __restrict__ in, typename Packed<T>::S* __restrict__ out,
    const typename Packed<T>::L* __restrict__ links, Geo geo, Diag<typename Packed<T>::R> diags,
    long stride, int gamma5, MarchParams p, CgFuse cgf) {
  using R = typename Packed<T>::R;
  using SV = typename Packed<R>::S;
  using GS = typename Packed<T>::S;
  constexpr int kPlanes = sizeof(R) == 8 ? 12 : 6;
  extern __shared__ __align__(16) unsigned char smem[];
  const int n = geo.X * p.ny;  // sites per tile == lanes per lane group (SMALL: rounded up to whole waves)
  const int slot = SMALL ? 0 : static_cast<int>(threadIdx.x) / n;
  // slice (buffer f, right-hand side r) of this lane group
  constexpr bool ONE = KIND == kOneSlice;
  constexpr bool NOW = KIND == kOuterNow || KIND == kOneBuffer;
  constexpr bool RELOAD = KIND == kOneBuffer;
  constexpr int kSlices = ONE || RELOAD ? 1 : 2;
  cx<R> gb[RB][6];  // NOW: the carried backward t hop, before its reconstruction
  SV* const base = reinterpret_cast<SV*>(smem) + slot * kSlices * RB * kPlanes * n;
  const long V = geo.V;

  const int lane = static_cast<int>(threadIdx.x) - slot * n;
  const bool live = !SMALL || lane < n;
  const int tid = live ? lane : n - 1;  // lanes beyond the tile follow its last site and store nothing
  const int xl = tid % geo.X;
  const int yl = tid / geo.X;
  // The lane groups of a workgroup march in lock step (one barrier per
  // step), so a link line fetched for one of them is an L1/L2 hit for the
  // others. Further workgroups of the same tile are consecutive.
  const int groups = p.nrhs / (p.gw * RB);
  const int bb = tile_of_block(p.group, p.nb);
  if (bb >= p.nb) return;
  // (with BUF the host launches one lane group per workgroup, so slot is 0 and
  // the fields' bases derive from the block index alone: wave-uniform)
  const int rhs0 = ((bb % groups) * p.gw + (BUF ? 0 : slot)) * RB;
  const int b = bb / groups;
  // the fields: plain pointers, or buffer resources (BUF; the fused CG work
  // writes its outputs through plain pointers)
  constexpr bool kBufOut = BUF && CGM == kCgNone;
  decltype(field_in<BUF>(in, 0u)) inr[RB];
  decltype(field_out<kBufOut>(out, 0u)) outr[RB];
  const auto lk = field_in<BUF>(links, p.link_bytes);
  R diag[RB];
#pragma unroll
  for (int r = 0; r < RB; ++r) {
    inr[r] = field_in<BUF>(in + diags.idx[rhs0 + r] * stride, p.spinor_bytes);
    outr[r] = field_out<kBufOut>(out + diags.idx[rhs0 + r] * stride, p.spinor_bytes);
    diag[r] = diags.d[rhs0 + r];
  }
  const int yt = b % p.ytiles;
  const int z = (b / p.ytiles) % geo.Z;
  const int tblk = b / (p.ytiles * geo.Z);
  const int y = yt * p.ny + yl;
  const int t0 = tblk * p.tb;
  const int t1 = ONE ? t0 + 1 : min(t0 + p.tb, geo.T);

  const int s0 = xl + geo.X * (y + geo.Y * z);  // the site at t = 0
  // LDS slots of the in-tile x and y neighbours
  const int lxp = yl * geo.X + (xl + 1 == geo.X ? 0 : xl + 1);
  const int lxm = yl * geo.X + (xl == 0 ? geo.X - 1 : xl - 1);
  const bool whole_y = p.ny == geo.Y;
  const bool y_fwd_out = !whole_y && yl + 1 == p.ny;
  const bool y_bwd_out = !whole_y && yl == 0;
  const int lyp = (yl + 1 == p.ny ? 0 : yl + 1) * geo.X + xl;
  const int lym = (yl == 0 ? p.ny - 1 : yl - 1) * geo.X + xl;
  // site offsets of the periodic neighbours
  const int dxm = xl == 0 ? geo.X - 1 : -1;
  // the lane holding x - 1, for the shuffled backward x link (x rows within a wave)
  // (measured: FP32 storage 196 -> 192 us on 32^3x64; FP64 unchanged; with
  // FP16 storage the 18 shuffles cost more than the 9 small loads they replace)
  const bool xshfl = kXShfl && sizeof(T) == 4 && RB == 1 && CGM == kCgNone && 64 % geo.X == 0;
  const int src_lane = (static_cast<int>(threadIdx.x) & 63) + dxm;
  const int dyp = y + 1 == geo.Y ? -(geo.Y - 1) * geo.X : geo.X;
  const int dym = y == 0 ? (geo.Y - 1) * geo.X : -geo.X;
  const int dzp = z + 1 == geo.Z ? -(geo.Z - 1) * geo.XY : geo.XY;
  const int dzm = z == 0 ? (geo.Z - 1) * geo.XY : -geo.XY;

  cx<R> acc[RB][12];
#pragma unroll
  for (int r = 0; r < RB; ++r)
#pragma unroll
    for (int c = 0; c < 12; ++c) acc[r][c] = {R(0), R(0)};

  // fused CG work: per lane group and right-hand side, kCgLds doubles after
  // all spinor slices. For the update, alpha = <r,r> / <p,Ap>: every lane of
  // the tile sums a strided share of the <p,Ap> partial sums and each wave
  // its lanes (an order fixed by the tile size, which the lattice fixes);
  // after the prologue's barrier every lane adds the wave sums in order, so
  // all lanes of all workgroups get the same alpha
  double* cgs = reinterpret_cast<double*>(reinterpret_cast<SV*>(smem) + p.gw * kSlices * RB * kPlanes * n) +
                slot * RB * kCgLds;
  double alpha[RB];
#pragma unroll
  for (int r = 0; r < RB; ++r) alpha[r] = 0.0;
  if constexpr (CGM == kCgUpdate) {
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      const double* pp = cgf.pap + static_cast<long>(diags.idx[rhs0 + r]) * cgf.npap;
      if constexpr (SMALL) {  // the split kernel's order: 256 shares, in four waves' worth
        for (int g = lane >> 6; g < 4; g += (n + 63) / 64) {
          const double t = wave_total(strided_sum256(pp, cgf.npap, 64 * g + (lane & 63)));
          if ((lane & 63) == 0) cgs[r * kCgLds + 8 + g] = t;
        }
      } else {
        double t = 0.0;
        int i = tid;
        for (; i + 3 * n < cgf.npap; i += 4 * n) {  // four loads in flight, added in order
          const double a0 = pp[i], a1 = pp[i + n], a2 = pp[i + 2 * n], a3 = pp[i + 3 * n];
          t += a0;
          t += a1;
          t += a2;
          t += a3;
        }
        for (; i < cgf.npap; i += n) t += pp[i];
        t = wave_total(t);
        if ((tid & 63) == 0) cgs[r * kCgLds + 8 + (tid >> 6)] = t;
      }
    }
  }

  // prologue: the carried hops of t0 (in the loop's order: outer hops, then
  // the backward t hop, so every site rounds alike) and the first slice in LDS
  {
    const int tm = t0 == 0 ? geo.T - 1 : t0 - 1;
    const int st = s0 + t0 * geo.XYZ;
    if constexpr (NOW) {
      cx<R> u[9];
      load_link<C12>(lk, V, 3, s0 + tm * geo.XYZ, u);
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        cx<R> psi[12], h[6];
        load_spinor(inr[r], V, s0 + tm * geo.XYZ, psi);
        project<3, +1>(psi, h);
        su3_mul<true>(u, h, gb[r]);
      }
    } else {
      outer_hops<C12>(inr, lk, V, st, dzp, dzm, y_fwd_out, dyp, y_bwd_out, dym, acc);
      hop_rb<3, +1, C12>(inr, lk, V, s0 + tm * geo.XYZ, s0 + tm * geo.XYZ, acc);
    }
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      cx<R> psi[12];
      load_spinor(inr[r], V, st, psi);
      if (live) lds_store_spinor(base + (kSlices * r) * kPlanes * n, n, tid, psi);
    }
  }
  __syncthreads();
  if constexpr (CGM == kCgUpdate) {
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      double t = 0.0;
      for (int w = 0; w < (SMALL ? 4 : n / 64); ++w) t += cgs[r * kCgLds + 8 + w];
      const long k = diags.idx[rhs0 + r];
      double* sc = cgf.scal + k * kScalars;
      bool flag = false;
      alpha[r] = cg_alpha(t, sc[kRr], &flag);
      if (lane == 0 && b == 0) {  // the field's first tile: one workgroup per field
        sc[kPap] = t;
        sc[kAlpha] = alpha[r];
        sc[kRrPrev] = sc[kRr];
        if (flag) sc[kFlag] = 1.0;
      }
    }
  }

  for (int t = t0; t < (ONE ? t0 + 1 : t1); ++t) {
    const int f = ONE || RELOAD ? 0 : (t - t0) & 1;  // the buffer holding slice t
    SV* cur[RB];
    SV* nxt[RB];
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      cur[r] = base + (kSlices * r + f) * kPlanes * n;
      nxt[r] = base + (kSlices * r + (ONE || RELOAD ? 0 : f ^ 1)) * kPlanes * n;
    }
    const int st = s0 + t * geo.XYZ;
    const int sn = t + 1 == geo.T ? s0 : st + geo.XYZ;  // the site at t+1
    const bool more = !ONE && t + 1 < t1;

    // Slice t+1: this workgroup's own spinors (forward t hop, next LDS
    // slice) and, in the same window, the z and off-tile y hops of t+1,
    // whose spinors other workgroups are loading as their own slice now.
    // U_t(t) serves the forward t hop of t and, from registers, the backward
    // t hop of t+1: no other workgroup reads it
    if constexpr (NOW) {
#pragma unroll
      for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int c = 0; c < 12; ++c) acc[r][c] = {R(0), R(0)};
      outer_hops<C12>(inr, lk, V, st, dzp, dzm, y_fwd_out, dyp, y_bwd_out, dym, acc);
#pragma unroll
      for (int r = 0; r < RB; ++r) reconstruct_add<3, +1>(gb[r], acc[r]);
    }
    cx<R> ut[9];
    load_link<C12, kUtNt>(lk, V, 3, st, ut);
    cx<R> nacc[RB][12];
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
      for (int c = 0; c < 12; ++c) nacc[r][c] = {R(0), R(0)};
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      cx<R> psi[12];
      load_spinor(inr[r], V, sn, psi);
      if (!RELOAD && more) {
        if (live) lds_store_spinor(nxt[r], n, tid, psi);
        if (!NOW && r == 0) outer_hops<C12>(inr, lk, V, sn, dzp, dzm, y_fwd_out, dyp, y_bwd_out, dym, nacc);
      }
      cx<R> h[6], g[6];
      project<3, -1>(psi, h);
      su3_mul<false>(ut, h, g);
      reconstruct_add<3, -1>(g, acc[r]);
    }
    // x hops and in-tile y hops from LDS
    lds_x_hops<C12>(cur, n, lxp, lxm, lk, V, st, dxm, xshfl, src_lane, acc);
    if (!y_fwd_out) lds_hop_rb<1, -1, C12>(cur, n, lyp, lk, V, st, acc);
    if (!y_bwd_out) lds_hop_rb<1, +1, C12>(cur, n, lym, lk, V, st + dym, acc);
    // epilogue of t; the backward t hop of t+1 joins the next accumulator
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      cx<R> psi[12];
      lds_load_spinor(cur[r], n, tid, psi);
      cx<R> o[12];
      epilogue(psi, acc[r], diag[r], gamma5, o);
      if constexpr (SMALL) {
        double v = 0.0;
        if (live) {
          if constexpr (CGM == kCgUpdate)
            v = cg_site_update_r(static_cast<GS*>(cgf.r) + diags.idx[rhs0 + r] * stride, V, st, o, alpha[r]);
          else
            v = store_site_norm(outr[r], V, st, o);
          cgs[RB * kCgLds + n * (RB * ((t - t0) & 1) + r) + lane] = v;
        }
      } else if constexpr (CGM == kCgUpdate) {
        const long k = diags.idx[rhs0 + r];
        double v = cg_site_update_r(static_cast<GS*>(cgf.r) + k * stride, V, st, o, alpha[r]);
        v = wave_total(v);
        if ((tid & 63) == 0) cgs[r * kCgLds + 4 * ((t - t0) & 1) + (tid >> 6)] = v;
      } else if constexpr (CGM == kCgNorm) {
        double v = store_site_norm(outr[r], V, st, o);
        v = wave_total(v);
        if ((tid & 63) == 0) cgs[r * kCgLds + 4 * ((t - t0) & 1) + (tid >> 6)] = v;
      } else if constexpr (kBufOut && sizeof(R) == 8 && !C12) {
        // FP64 with full links stores with the default cache policy (measured
        // 360.4 -> 358.9 us on 32^3x64; with 12-real links and in FP32 the
        // non-temporal stores are faster)
        store_spinor<0>(outr[r], V, st, o);
      } else {
        store_spinor(outr[r], V, st, o);
      }
      if constexpr (NOW) {
        cx<R> h[6];
        project<3, +1>(psi, h);
        su3_mul<true>(ut, h, gb[r]);
      } else if (more) {
        cx<R> h[6], g[6];
        project<3, +1>(psi, h);
        su3_mul<true>(ut, h, g);
        reconstruct_add<3, +1>(g, nacc[r]);
      }
    }
    if constexpr (RELOAD) {
      if (more) {
        cx<R> psn[RB][12];
#pragma unroll
        for (int r = 0; r < RB; ++r) load_spinor(inr[r], V, sn, psn[r]);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < RB; ++r)
          if (live) lds_store_spinor(nxt[r], n, tid, psn[r]);
      }
    } else if constexpr (!NOW) {
#pragma unroll
      for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int c = 0; c < 12; ++c) acc[r][c] = nacc[r][c];
    }
    if (!ONE || CGM != kCgNone) __syncthreads();
    if constexpr (SMALL) {
      // the sums of the slices that the tile holds, 32 lanes each, every site on
      // the lane that it has in the split kernel (the next write to these words is
      // two steps on, behind the next barrier)
      const int first = n * ((t * geo.Z + z) * p.ytiles + yt);  // the tile's first site
      const int skip = first % kSplitSites;
      const int slices = (skip + n + kSplitSites - 1) / kSplitSites;
      for (int h = lane >> 5; (h & ~1) < slices; h += (n + 63) / 64 * 2) {
        const int l = kSplitSites * h + (lane & 31) - skip;
#pragma unroll
        for (int r = 0; r < RB; ++r) {
          const double v =
              half_wave_total(l >= 0 && l < n ? cgs[RB * kCgLds + n * (RB * ((t - t0) & 1) + r) + l] : 0.0);
          if ((lane & 31) == 0 && h < slices)
            cgf.rr[static_cast<long>(diags.idx[rhs0 + r]) * cgf.nslices + p.cut.of(first) + h] = v;
        }
      }
    } else if constexpr (CGM != kCgNone) {
      // the squared norm of this tile slice (Q p or r): its waves in order (the next write to these
      // words is two steps on, behind the next barrier)
      if (tid == 0) {
        const long ts = (static_cast<long>(t) * geo.Z + z) * p.ytiles + yt;
#pragma unroll
        for (int r = 0; r < RB; ++r) {
          double sum = 0.0;
          for (int w = 0; w < n / 64; ++w) sum += cgs[r * kCgLds + 4 * ((t - t0) & 1) + w];
          cgf.rr[static_cast<long>(diags.idx[rhs0 + r]) * cgf.nslices + ts] = sum;
        }
      }
    }
  }
}

template <int N>
constexpr std::integral_constant<int, N> kInt{};

// Whether two workgroups of n FP64 lanes, or of n FP32 lanes with two right-hand
// sides each, fit a CU's LDS with two slices per workgroup.
bool two_workgroups(int n) { return n <= 208; }

// Whether FP64 tiles of n lanes run kOuterAhead, for `work` sites times fields: where
// LDS holds one workgroup either way, and in the plain operator on tiles up to 128
// lanes while the fields stay in the caches. There the outer hops, done while their
// owners load the same lines, are worth more than the second wave per SIMD (now /
// ahead, us, each with its best t split: 16 x 8 x 20 x 30 with four fields 43.6 / 39.8,
// with eight 85.2 / 75.5, 10 x 10 x 20 x 40 with three 40.0 / 35.3; 33 x 9 x 20 x 30 with
// four 125 / 127, with six 180 / 201; 12 x 8 x 11 x 71 with 14 151 / 159). The fused CG
// work runs kOuterNow there (9 x 33 x 12 x 20 57 / 68 us per iteration).
bool outer_ahead(int n, long work, bool fused) {
  if (!two_workgroups(n)) return true;
  return !fused && n <= 128 && work <= (n % 64 == 0 ? 1000000 : 500000);
}

size_t march_lds_bytes(int threads, size_t real_bytes) {
  return 2 * 24 * real_bytes * static_cast<size_t>(threads);  // two spinor slices
}

size_t real_bytes_of(int prec) { return prec == WD_FP64 ? 8 : 4; }

// Cost model behind the default t split and right-hand sides per lane. A
// workgroup that marches tb slices costs tb + prologue slices (the prologue
// reads the outer hops, the backward t hop and the first slice). A CU works on
// `waves` waves' worth of workgroups at once; the busiest one, with
// ceil(workgroups / 256) of them, sets the time: a round for each full set, and for
// a last set that fills the share x of its places last + (1 - last) x of a round
// (1: as long as a full one, 0: in proportion). With FP16 storage, whose workgroups
// are short and uneven, the chip's rounds count as a whole, the last one as `tail`
// of one on average. rb2: the cost of a slice of two right-hand sides per lane in
// a launch of half the workgroups.
//
// All of these are fitted to times, `waves` too: it is the residency at which the
// model picks the fastest launches. Registers allow more in places (FP32 kernels
// of one field per lane hold three waves per SIMD, 12 per CU), or as much as that
// only in some modes (two FP32 fields per lane: 165 registers, three waves; with
// the fused CG work 171, two).
// Fitted on MI355X to every split of t and both rb timed on up to 20 lattices
// with 1 to 16 right-hand sides, from 16^4 to 32^3 x 64, among them 28 x 15 x 22 x 33, 9 x
// 33 x 12 x 20 and 21^4, in FP32 with 12-real links too. By how much the choice is
// slower than the best launch timed, on average (at most), in percent:
//   FP64  up to 208 lanes 0.9 (8); beyond, one workgroup per CU, 1.5
//   FP32  up to 208 lanes 0.9 (8), fused 1.5 (12); 256 lanes 1.2 (16), fused 0.6 (6);
//         between them 1.9 (5)
//   FP16  from 2^20 sites on 1.4 (5), fused 1.1 (5)
// where one resident round of workgroups whatever its last round leaves idle was
// 14 to 24 % slower (24^3 x 48 with 12 FP32 fields 757 -> 525 us), and whole rounds
// only, with the same weights for the fused modes, 2 to 4 % (us: FP32 16^4 with 12
// fields 56.5 -> 53, 32 x 16^2 x 32 with two 43.6 -> 40; per CG iteration 16^3 x 32
// with six 209 -> 199, 32 x 16^2 x 32 with two 151 -> 144, FP16 32^4 223 -> 217).
// Two right-hand sides per lane pay in FP32 (87 against 105 us for 4 fields on
// 24^4), not with FP16 storage, whose waves they halve; several lane groups per
// workgroup never were the fastest.
struct MarchCost {
  int waves, waves2;
  double prologue, prologue2, last, last2, rb2, tail;
};
MarchCost march_cost(int prec, int n, int nrhs, bool fused, bool ahead) {
  const bool two = two_workgroups(n);
  if (prec == WD_FP64) {
    if (!two) return {8, 0, 0.8, 0.0, 1.0, 0.0, 0.0, -1.0};
    if (ahead) return {4, 0, 0.8, 0.0, 1.0, 0.0, 0.0, -1.0};
    return {8, 0, n <= 128 ? 0.8 : 0.4, 0.0, n <= 128 ? 0.3 : 0.2, 0.0, 0.0, -1.0};
  }
  if (prec == WD_FP32 && two)
    return fused ? MarchCost{8, 8, 0.4, 0.7, 0.4, 1.0, 1.3, -1.0} : MarchCost{8, 12, 0.4, 0.4, 0.4, 1.0, 1.2, -1.0};
  if (prec == WD_FP32 && n == kMarchMaxThreads)
    return fused ? MarchCost{12, 8, 0.4, 0.7, 0.2, 1.0, 1.3, -1.0} : MarchCost{12, 8, 0.2, 0.4, 0.1, 0.6, 1.2, -1.0};
  if (prec == WD_FP32) return {8, 8, 0.4, 0.7, 1.0, 1.0, 1.2, -1.0};
  if (fused && nrhs > 1) return {12, 0, 1.1, 0.0, 0.0, 0.0, 0.0, 0.5};
  return {16, 0, 0.4, 0.0, 0.0, 0.0, 0.0, 0.3};
}

// Geometry of the t-marching kernel for a lattice, with the default launch
// choice, or ny = 0 if it does not apply (x rows longer than a workgroup, or
// too few sites per tile).
MarchParams march_params(const Geo& geo, int prec, int nrhs, bool fused = false, int most_rb = 2) {
  MarchParams p{0, 0, 0, 0, 0, nrhs, 1, 1, false, {}, 0u, 0u};
  const size_t real_bytes = real_bytes_of(prec);
  if (geo.X > kMarchMaxThreads) return p;
  int ny = 0;
  for (int d = 1; d <= geo.Y && geo.X * d <= kMarchTargetThreads; ++d)
    if (geo.Y % d == 0 && march_lds_bytes(geo.X * d, real_bytes) <= kLdsBytes) ny = d;
  if (ny == 0 || geo.X * ny < 64) return p;
  p.ny = ny;
  p.ytiles = geo.Y / ny;
  const int n = geo.X * ny;
  const int waves = (n + 63) / 64;
  p.ahead = prec == WD_FP64 && outer_ahead(n, static_cast<long>(geo.V) * nrhs, fused);
  const MarchCost mc = march_cost(prec, n, nrhs, fused, p.ahead);
  double best = 0.0;
  // among equals the shorter march; in FP32 the fused CG work on tiles up to 208
  // lanes also takes one that costs up to 4 % more (24^4 with three fields: 311 us
  // per iteration at 12 slices per workgroup, 287 at 6)
  // and the plain operator on tiles of 256 lanes, where the fields outgrow the caches,
  // a shorter march only if it costs 4 % less (32^3 x 64 190 us at 16 slices per
  // workgroup, 200 at 11, which the model puts 1 % lower; 64 x 32 x 16 x 24 72 at six, 78
  // at four; below, 16^2 x 24 x 48 with 12-real links 23.6 at the shorter, 27.1 at the longer)
  const bool large = static_cast<long>(geo.V) * nrhs >= 500000;
  double tie = 1.0;
  if (prec == WD_FP32 && fused && two_workgroups(n)) tie = 1.04;
  if (prec == WD_FP32 && !fused && n == kMarchMaxThreads && large) tie = 0.96;
  // FP16 storage: one slice per workgroup (its own kernel), unless the fields and
  // links outgrow the 256 MB cache that serves the t neighbours then (about 2^20
  // sites; us, one slice / best longer march: 24^3 x 48 37.5 / 41.2, 32^4 59.9 /
  // 56.8, 32^3 x 64 with four fields 398 / 397, with eight 838 / 767, with twelve
  // 1273 / 1152)
  const bool single = prec == WD_FP16 && geo.V < (1 << 20);
  if (single) p.tb = 1;
  for (int rb = 1; rb <= most_rb && !single; ++rb) {
    const size_t lds = march_lds_bytes(n, real_bytes) * (rb == 2 && two_workgroups(n) ? 2 : 1);  // one buffer per field
    if (rb == 2 && (mc.waves2 == 0 || nrhs % 2 != 0 || lds > kLdsBytes)) break;
    const int by_waves = (rb == 1 ? mc.waves : mc.waves2) / waves;
    const int by_lds = static_cast<int>(kLdsBytes / lds);
    const int per_cu = std::max(1, std::min(by_waves, by_lds));
    const double columns = static_cast<double>(p.ytiles) * geo.Z * (nrhs / rb);
    const double last = rb == 1 ? mc.last : mc.last2;
    // every distinct ceil(T / nt), largest first
    for (int tb = geo.T, nt = 1;;) {
      double rounds;
      if (mc.tail < 0.0) {
        const double busiest = std::ceil(columns * nt / kNumCu);
        rounds = std::floor(busiest / per_cu);
        const double share = busiest / per_cu - rounds;
        if (share > 0.0) rounds += last + (1.0 - last) * share;
      } else {
        rounds = std::max(1.0, columns * nt / (static_cast<double>(kNumCu) * per_cu) + mc.tail);
      }
      const double cost = rounds * (tb + (rb == 1 ? mc.prologue : mc.prologue2)) * (rb == 1 ? 1.0 : mc.rb2);
      if (p.tb == 0 || cost < best * std::min(tie, 1.0) || (cost <= best * tie && rb == p.rb)) {
        best = p.tb == 0 ? cost : std::min(best, cost);
        p.tb = tb;
        p.rb = rb;
      }
      if (tb == 1) break;
      nt = (geo.T + tb - 2) / (tb - 1);  // fewest workgroups along t with fewer steps each
      tb = (geo.T + nt - 1) / nt;
    }
  }
  const int nb = p.ytiles * geo.Z * (nrhs / p.rb) * ((geo.T + p.tb - 1) / p.tb);
  // every XCD gets one contiguous eighth of the workgroups: the right-hand
  // sides, y tiles and z planes that share links and halo slices meet in one L2
  p.group = (nb + kNumXcd - 1) / kNumXcd;
  return p;
}

template <typename T, bool C12, int MAXT, int RB, int CGM, bool BUF, int KIND, bool SMALL = false>
hipError_t launch_march_t(const void* in, void* out, const void* links, const Geo& geo,
                          const Diag<typename Packed<T>::R>& diag, long stride, int g5,
                          MarchParams p, const CgFuse& f, hipStream_t st) {
  using SV = typename Packed<T>::S;
  using LV = typename Packed<T>::L;
  using R = typename Packed<T>::R;
  const int n = geo.X * p.ny;
  size_t lds = static_cast<size_t>(p.gw) * RB * march_lds_bytes(n, sizeof(R)) / (KIND == kOuterAhead || KIND == kOuterNow ? 1 : 2);
  if (CGM != kCgNone) lds += static_cast<size_t>(p.gw) * RB * kCgLds * sizeof(double);
  if (SMALL) lds += 2 * static_cast<size_t>(RB) * n * sizeof(double);
  if (lds > kLdsBytes) return hipErrorInvalidValue;
  // raise the kernel's dynamic LDS limit once to the whole LDS of a CU
  static std::atomic<int> attr_set{0};
  if (!attr_set.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute(
        reinterpret_cast<const void*>(&dslash_march_kernel<T, C12, MAXT, RB, CGM, BUF, KIND, SMALL>),
        hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(kLdsBytes));
    if (e != hipSuccess) return e;
    attr_set.store(1, std::memory_order_release);
  }
  p.nb = (p.nrhs / (p.gw * RB)) * p.ytiles * geo.Z * ((geo.T + p.tb - 1) / p.tb);
  const int eighth = (p.nb + kNumXcd - 1) / kNumXcd;  // larger groups mean the same
  if (p.group > eighth) p.group = eighth;
  const unsigned grid = static_cast<unsigned>(p.group == eighth ? eighth * kNumXcd : p.nb);
  dslash_march_kernel<T, C12, MAXT, RB, CGM, BUF, KIND, SMALL><<<grid, SMALL ? (n + 63) / 64 * 64 : p.gw * n, lds, st>>>(
      static_cast<const SV*>(in), static_cast<SV*>(out), static_cast<const LV*>(links), geo, diag,
      stride, g5, p, f);
  return hipGetLastError();
}

// Which variant of the march runs. What decides is how many waves a CU holds;
// two LDS slices of two workgroups fit up to 208 lanes per tile (FP64, or FP32
// with two right-hand sides per lane; half that each with one).
//  - FP64: kOuterAhead needs 280 registers (one wave per SIMD), kOuterNow 204 to
//    238 (two). Up to 208 lanes kOuterNow is the faster one, but for the smaller
//    tiles of outer_ahead: 24^4 with four fields
//    235 -> 209 us, 28 x 15 x 22 x 33 71 -> 65 and with four 287 -> 222, with
//    12-real links 24^3 x 48 131 -> 108. Beyond, LDS holds one workgroup either
//    way and the outer hops must meet their owners' loads in L2: 32^3 x 64 357 us
//    ahead, 389 now, 16^3 x 32 26.0 and 27.9.
//  - FP32 arithmetic: kOuterNow (24^3 x 48 with three fields 174 -> 161 us, 28 x 15
//    x 22 x 33 43 -> 35, 32^4 97 -> 95). Two right-hand sides per lane beyond 208
//    lanes: kOneBuffer, which lets a second workgroup in (32^4 with two fields
//    176 -> 161 us, with four 316 -> 281, 16^3 x 32 with four 40.3 -> 36.4); the fused
//    CG modes take the same two variants there. The fused CG modes with one field per lane run kOuterAhead: their epilogue's loads
//    leave the outer hops to hide the next slice's (FP32 solves, ahead / now: 24^4
//    18.9 / 19.9 ms, 32^3 x 16 28.1 / 29.3, 24^4 with three fields 54.0 / 58.1).
template <typename T, bool C12, int CGM, bool BUF>
hipError_t launch_march_b(const void* in, void* out, const void* links, const Geo& geo,
                          const Diag<typename Packed<T>::R>& diag, long stride, int g5,
                          const MarchParams& p, const CgFuse& f, hipStream_t st) {
  const auto run = [&](auto maxt, auto rb, auto kind) {
    return launch_march_t<T, C12, decltype(maxt)::value, decltype(rb)::value, CGM, BUF, decltype(kind)::value>(
        in, out, links, geo, diag, stride, g5, p, f, st);
  };
  const bool two = two_workgroups(geo.X * p.ny);
  if constexpr (sizeof(typename Packed<T>::R) == 4) {
    if (p.rb == 2)  // two right-hand sides per lane: one lane group per workgroup
      return two ? run(kInt<kMarchMaxThreads>, kInt<2>, kInt<kOuterNow>)
                 : run(kInt<kMarchMaxThreads>, kInt<2>, kInt<kOneBuffer>);
    if (p.gw > 1) return run(kInt<kMarchMultiThreads>, kInt<1>, kInt<kOuterNow>);
    // FP64 keeps no kernel for single slices: it is bound by the loads that a
    // second slice saves (16^4 15.0 us with its best march, 15.4 with single ones)
    if constexpr (BUF) {
      if (p.tb == 1) return run(kInt<kMarchMaxThreads>, kInt<1>, kInt<kOneSlice>);
    }
    return run(kInt<kMarchMaxThreads>, kInt<1>, kInt<CGM != kCgNone ? kOuterAhead : kOuterNow>);
  } else {
    return p.ahead ? run(kInt<kMarchMaxThreads>, kInt<1>, kInt<kOuterAhead>)
                   : run(kInt<kMarchMaxThreads>, kInt<1>, kInt<kOuterNow>);
  }
}

// The operator reads its fields (and the plain operator also writes them)
// through buffer resources when every field is below 4 GiB and a workgroup
// holds one lane group (WD_MARCH_BUF 0 turns it off).
template <typename T, bool C12, int CGM>
hipError_t launch_march(const void* in, void* out, const void* links, const Geo& geo,
                        const Diag<typename Packed<T>::R>& diag, long stride, int g5,
                        const MarchParams& p, const CgFuse& f, hipStream_t st) {
  if (kMarchBuf && p.gw == 1 && p.link_bytes != 0 && p.spinor_bytes != 0)
    return launch_march_b<T, C12, CGM, true>(in, out, links, geo, diag, stride, g5, p, f, st);
  return launch_march_b<T, C12, CGM, false>(in, out, links, geo, diag, stride, g5, p, f, st);
}

bool small_march(const Geo& geo, const MarchParams& p, int prec);

// The CG slices of a small lattice. Runs are cut only where the march takes over
// for some number of fields: the cuts add up to a third to the partial sums that
// every workgroup reads (8 x 9 x 8 x 7 FP64 19.7 us per iteration with them, 19.0 without).
CgSlices cg_slices(const Geo& geo, MarchParams p, int prec) {
  const int tile = geo.X * p.ny;
  p.nrhs = kMaxMultiRhs;
  if (!small_march(geo, p, prec)) return {0, 0};
  return {tile % kSplitSites == 0 ? 0 : tile, tile == 0 ? 0 : std::lcm(tile, kSplitSites)};
}

// The march with the CG slices of small lattices, mode CGM of the launch: one
// field per lane, workgroups of whole waves.
template <typename T, bool C12, int CGM>
hipError_t launch_march_small(const void* in, void* out, const void* links, const Geo& geo,
                              const Diag<typename Packed<T>::R>& diag, long stride, int g5, const MarchParams& m,
                              const CgFuse& f, hipStream_t st) {
  const int prec = sizeof(T) == 8 ? WD_FP64 : sizeof(T) == 4 ? WD_FP32 : WD_FP16;
  MarchParams p = march_params(geo, prec, m.nrhs, true, 1);
  if (p.ny == 0 || m.link_bytes == 0 || m.spinor_bytes == 0) return hipErrorInvalidValue;
  p.link_bytes = m.link_bytes;
  p.spinor_bytes = m.spinor_bytes;
  p.cut = cg_slices(geo, p, prec);
  const auto run = [&](auto kind) {
    return launch_march_t<T, C12, kMarchMaxThreads, 1, CGM, true, decltype(kind)::value, true>(
        in, out, links, geo, diag, stride, g5, p, f, st);
  };
  if constexpr (sizeof(T) == 8) return p.ahead ? run(kInt<kOuterAhead>) : run(kInt<kOuterNow>);
  if constexpr (sizeof(T) == 4) return p.tb == 1 ? run(kInt<kOneSlice>) : run(kInt<kOuterAhead>);
  if constexpr (sizeof(T) == 2) return p.tb == 1 ? run(kInt<kOneSlice>) : hipErrorInvalidValue;
}

// The split kernel: mode CGM of the launch.
template <typename T, bool C12, int CGM, int FOLD = kFoldNone>
hipError_t launch_split(const void* in, void* out, const void* links, const Geo& geo,
                        const Diag<typename Packed<T>::R>& diag, long stride, int g5, const MarchParams& m,
                        const CgFuse& f, hipStream_t st) {
  using R = typename Packed<T>::R;
  SplitParams p{geo.X, geo.Y, geo.Z, geo.T, geo.X, geo.XY, geo.XYZ, geo.V};
  p.nrhs = m.nrhs;
  p.ny = m.ny;
  p.cut = cg_slices(geo, m, sizeof(T) == 8 ? WD_FP64 : sizeof(T) == 4 ? WD_FP32 : WD_FP16);
  p.link_bytes = m.link_bytes;
  p.spinor_bytes = m.spinor_bytes;
  SplitCoef<R> cf{};
  for (int k = 0; k < m.nrhs; ++k) {
    cf.d[k] = diag.d[k];
    cf.c[k] = R(-0.5);
    cf.idx[k] = diag.idx[k];
  }
  return launch_split_hop<T, C12, CGM, FOLD>(in, in, out, links, links, cf, stride, g5, p, f, st);
}

hipError_t launch_site(const wd_gauge* g, const void* in, void* out, const Geo& geo, const Diag<float>& diag,
                       long stride, int g5, const MarchParams& m, hipStream_t st) {
  SplitParams p{geo.X, geo.Y, geo.Z, geo.T, geo.X, geo.XY, geo.XYZ, geo.V};
  p.nrhs = m.nrhs;
  p.link_bytes = m.link_bytes;
  p.spinor_bytes = m.spinor_bytes;
  p.ntiles = (p.V + kSiteBlock - 1) / kSiteBlock;
  const unsigned nb = split_grid(p);
  const auto run = [&](auto kernel) {
    kernel<<<nb, kSiteBlock, 0, st>>>(static_cast<const h8*>(in), static_cast<h8*>(out),
                                      static_cast<const h2*>(g->links), diag, stride, g5, p);
    return hipGetLastError();
  };
  const bool buf = p.link_bytes != 0 && p.spinor_bytes != 0;
  if (g->c12) return buf ? run(&dslash_site_kernel<true, true>) : run(&dslash_site_kernel<true, false>);
  return buf ? run(&dslash_site_kernel<false, true>) : run(&dslash_site_kernel<false, false>);
}

// Whether the split kernel is the default for nrhs fields: where the t-marching
// one does not apply, in launches too small to fill the chip with marches, and
// in larger ones on lattices whose tiles leave lanes of their waves idle (X * ny
// not near a multiple of 64), up to the sites times fields at which the march
// overtook it on 22 lattices. Measured on MI355X, t-marching / split (us) on both
// sides of each line (lanes of the tile in brackets):
//   12^4 FP64 8.1 / 6.7; 16^4 (256 of 256) with one FP64 field 15.5 / 17.2, FP32 7.6 /
//   8.5, FP16 6.9 / 8.2;
//   FP16: 15 x 9 x 14 x 21 (135 of 192) 8.6 / 6.8, with two fields 9.4 / 9.0, with three
//   10.9 / 12.4; 65 x 5 x 20 x 40 (65 of 128) with three 59.9 / 69.5;
//   under six tenths: 65 x 5 x 12 x 20 with 12 FP64 fields 196 / 177, 11 x 6 x 30 x 60 (66
//   of 128) with eight 169 / 183, FP32 with six 60.9 / 59.6, with eight 76.4 / 80.9;
//   up to 128 lanes, FP64: 10 x 10 x 20 x 40 (100 of 128) with two fields 28.6 / 28.8,
//   with three 36.0 / 40.0; 14 x 8 x 31 x 16 (112) with three 31.3 / 31.3, with eight 66 /
//   79; FP32 with an even number: 18 x 6 x 12 x 31 (108) with two 6.9 / 7.6, with eight
//   23.0 / 28.1;
//   beyond: FP64 20^4 (200 of 256) with two 54.3 / 52.6, with three 67.9 / 77.6; 18^3 x 36
//   (162 of 192) with two 70.1 / 77.1; FP32 20^4 with two 30.3 / 28.7, with four 48.3 /
//   52.0; 12 x 12 x 24 x 36 (144 of 192) with three 37.1 / 31.3, with four 38.4 / 41.4.
bool use_split(const Geo& geo, const MarchParams& p, int prec) {
  if (p.ny == 0) return true;
  const long work = static_cast<long>(geo.V) * p.nrhs;
  if (work <= WD_SPLIT_SITES) return true;
  const int n = geo.X * p.ny;
  const int lanes = (n + 63) / 64 * 64;
  if (10 * n >= 9 * lanes) return false;  // at least nine tenths of the lanes at work
  if (prec == WD_FP16) return work <= 65536;
  if (10 * n < 6 * lanes) return work <= (prec == WD_FP64 ? 940000 : 750000);
  if (prec == WD_FP64) return work <= (n <= 128 && 10 * n >= 7 * lanes ? 200000 : 330000);
  return work <= (n <= 128 && p.nrhs % 2 == 0 ? 150000 : 450000);
}

// Whether a tuning line may name the split kernel: where it is the default, or has
// been, so that files saved then still load (it runs everywhere).
bool split_choice(const Geo& geo, const MarchParams& p, int prec) {
  const int n = geo.X * p.ny;
  const int lanes = (n + 63) / 64 * 64;
  const long most = 10 * n >= 9 * lanes ? 0 : 10 * n < 6 * lanes ? 800000 : prec == WD_FP16 ? 65536 : 450000;
  return use_split(geo, p, prec) || static_cast<long>(geo.V) * p.nrhs <= most;
}

// Whether the t-marching tiles are whole waves (what its fused CG work needs).
bool whole_waves(const Geo& geo, const MarchParams& p) { return p.ny > 0 && (geo.X * p.ny) % 64 == 0; }

// Whether the fused CG work sums slices of 32 sites (CgSlices), which the split
// kernel and the march (SMALL) both hold, so that a launch can take the faster
// one for its number of fields and a field keeps its bits: on small lattices, and,
// up to 131072 sites (some 5000 partial sums, which every workgroup of the kernel
// that follows reads), where the march's own slices need tiles of whole waves.
bool small_slices(const Geo& geo, const MarchParams& p) { return geo.V <= (whole_waves(geo, p) ? 16384 : 131072); }

// Which of the two runs: the march beyond these sites times fields, where it
// overtook the split kernel on 20 lattices (split / march, us per CG iteration):
// FP16 12^4 with three fields 35.9 / 38.5, with six 52.1 / 47.1, 16^2 x 8^2 with 16 79.1 /
// 58.0, 15 x 16^2 x 32 with eight 279 / 180; FP64 8^3 x 16 with six 40.9 / 41.2, with
// eight 48.3 / 46.2, 14^4 with three 80.0 / 85.0, 12^2 x 24 x 36 97.7 / 86.0, 65 x 5 x 12 x 20
// with four 208 / 196; FP32 18^4 with two 85.5 / 83.6, 12^4 with 16 109 / 125, 20^3 x 16
// with three 144 / 125, 15 x 16^2 x 32 54.5 / 48.6, with two 92.0 / 79.3, but 12 x 15 x 24 x
// 7 with four 49 / 56 (marches of seven slices).
bool small_march(const Geo& geo, const MarchParams& p, int prec) {
  if (p.ny == 0) return false;
  const long work = static_cast<long>(geo.V) * p.nrhs;
  if (prec == WD_FP16) return work > 80000;
  const int n = geo.X * p.ny;
  const int lanes = (n + 63) / 64 * 64;
  if (10 * n >= 9 * lanes) return work > (prec == WD_FP64 ? 60000 : 150000);
  if (10 * n >= 6 * lanes) return work > (prec == WD_FP64 ? 120000 : 350000);
  return prec == WD_FP64 && work > 300000;
}

// The tuning choice that stands for the split kernel.
constexpr MarchTuning kSplitTuning{0, 1, 0, 1};

// Applies a tuning choice to the default parameters.
MarchParams with_tuning(MarchParams p, const MarchTuning& t) {
  p.tb = t.tb;
  p.gw = t.gw;
  p.group = t.group;
  p.rb = t.rb;
  return p;
}

// cg: a CG iteration's fused work (cg->mode kCgNorm or kCgUpdate), or nullptr for a
// plain apply. On small lattices the split kernel or the march (small_march) does
// it, on others the march.
template <typename T, bool C12>
hipError_t launch_typed(const wd_gauge* g, const void* in, void* out, const Geo& geo,
                        const double* masses, int nrhs, const int* fields, int g5,
                        const MarchTuning* force, const CgFuse* cg, hipStream_t st) {
  using R = typename Packed<T>::R;
  Diag<R> diag{};
  for (int k = 0; k < nrhs; ++k) {
    diag.d[k] = static_cast<R>(4.0 + masses[k]);
    diag.idx[k] = fields ? fields[k] : k;
  }
  const long stride = spinor_units<T>(geo.V);  // 16-B elements per field
  MarchParams p = march_params(geo, g->prec, nrhs, cg != nullptr);
  // byte sizes for buffer-resource access, or 0 where a field reaches 4 GiB
  const unsigned long sbytes = static_cast<unsigned long>(stride) * 16;
  p.link_bytes = g->link_bytes < (1ul << 32) ? static_cast<unsigned>(g->link_bytes) : 0u;
  p.spinor_bytes = sbytes < (1ul << 32) ? static_cast<unsigned>(sbytes) : 0u;
  const long work = static_cast<long>(geo.V) * nrhs;
  MarchTuning t;
  bool split = use_split(geo, p, g->prec);
  if (p.ny > 0 && (force != nullptr || tuned_lookup(g->dims, g->prec, g->c12, nrhs, &t))) {
    if (force != nullptr) t = *force;
    split = t.tb == 0;
    if (!split) p = with_tuning(p, t);
  }
  if (cg != nullptr) {
    // a partial sum slot for every slice, and the inputs the update reads
    if (cg->rr == nullptr || cg->nslices < cg_fuse_slices(g->dims, g->prec)) return hipErrorInvalidValue;
    if (cg->mode == kCgUpdate && (cg->r == nullptr || cg->pap == nullptr || cg->npap < 1 || cg->scal == nullptr))
      return hipErrorInvalidValue;
    split = small_slices(geo, p);
    if (!split && !whole_waves(geo, p)) return hipErrorInvalidValue;
    if (split && small_march(geo, p, g->prec)) {
      if (cg->mode == kCgNorm && cg->p_out == nullptr)
        return launch_march_small<T, C12, kCgNorm>(in, out, g->links, geo, diag, stride, g5, p, *cg, st);
      if (cg->mode == kCgUpdate)
        return launch_march_small<T, C12, kCgUpdate>(in, nullptr, g->links, geo, diag, stride, g5, p, *cg, st);
      return hipErrorInvalidValue;
    }
    if (split && p.ny == 0 && g->prec == WD_FP16 && cg->p_out == nullptr && work > kSiteCgSites)
      return launch_site_cg(g, masses, nrhs, fields, in, out, *cg, st);
    if (cg->mode == kCgNorm && cg->p_out != nullptr)
      return split ? launch_split<T, C12, kCgNorm, kFoldBoth>(in, out, g->links, geo, diag, stride, g5, p, *cg, st)
                   : hipErrorInvalidValue;
    if (cg->mode == kCgNorm)
      return split ? launch_split<T, C12, kCgNorm>(in, out, g->links, geo, diag, stride, g5, p, *cg, st)
                   : launch_march<T, C12, kCgNorm>(in, out, g->links, geo, diag, stride, g5, p, *cg, st);
    if (cg->mode != kCgUpdate) return hipErrorInvalidValue;
    return split ? launch_split<T, C12, kCgUpdate>(in, nullptr, g->links, geo, diag, stride, g5, p, *cg, st)
                 : launch_march<T, C12, kCgUpdate>(in, nullptr, g->links, geo, diag, stride, g5, p, *cg, st);
  }
  if constexpr (sizeof(T) == 2) {
    if (p.ny == 0 && work >= kSiteSites) return launch_site(g, in, out, geo, diag, stride, g5, p, st);
  }
  return split ? launch_split<T, C12, kCgNone>(in, out, g->links, geo, diag, stride, g5, p, CgFuse{}, st)
               : launch_march<T, C12, kCgNone>(in, out, g->links, geo, diag, stride, g5, p, CgFuse{}, st);
}

template <typename T>
hipError_t launch_prec(const wd_gauge* g, const void* in, void* out, const Geo& geo,
                       const double* masses, int nrhs, const int* fields, int g5,
                       const MarchTuning* force, const CgFuse* cg, hipStream_t st) {
  return g->c12 ? launch_typed<T, true>(g, in, out, geo, masses, nrhs, fields, g5, force, cg, st)
                : launch_typed<T, false>(g, in, out, geo, masses, nrhs, fields, g5, force, cg, st);
}

hipError_t launch_any(const wd_gauge* g, const double* masses, int nrhs, const int* fields,
                      const void* in, void* out, int flags, const MarchTuning* force,
                      const CgFuse* cg, hipStream_t st) {
  if (nrhs < 1) return hipSuccess;
  if (nrhs > kMaxMultiRhs) return hipErrorInvalidValue;
  const Geo geo = make_geo(g->dims);
  const int g5 = (flags & WD_FLAG_GAMMA5) ? 1 : 0;
  switch (g->prec) {
    case WD_FP64: return launch_prec<double>(g, in, out, geo, masses, nrhs, fields, g5, force, cg, st);
    case WD_FP32: return launch_prec<float>(g, in, out, geo, masses, nrhs, fields, g5, force, cg, st);
    case WD_FP16:
      return launch_prec<_Float16>(g, in, out, geo, masses, nrhs, fields, g5, force, cg, st);
    default: return hipErrorInvalidValue;
  }
}


}  // namespace

hipError_t launch_dslash_multi(const wd_gauge* g, const double* masses, int nrhs, const int* fields,
                               const void* in, void* out, int flags, hipStream_t st) {
  return launch_any(g, masses, nrhs, fields, in, out, flags, nullptr, nullptr, st);
}

int cg_fuse_slices(const int32_t dims[4], int prec) {
  const Geo geo = make_geo(dims);
  const MarchParams p = march_params(geo, prec, 1);
  if (small_slices(geo, p)) return cg_slices(geo, p, prec).of(geo.V - 1) + 1;
  if (!whole_waves(geo, p)) return 0;
  const long n = static_cast<long>(geo.T) * geo.Z * p.ytiles;
  return n <= 0x7fffffffL ? static_cast<int>(n) : 0;
}

// FP64 vectors: the t-marching FP64 kernel holds one wave per SIMD, and the r
// update in its epilogue costs a little more than the separate update kernel's
// work, but saves a launch: 16^4 with one field 79 -> 51 us per iteration and
// 16^3 x 32 99 -> 88 (with the launch shapes of before: 24^4 277 -> 285).
bool cg_fuse_update(const int32_t dims[4], int prec) {
  return cg_fuse_slices(dims, prec) > 0 && (prec != WD_FP64 || make_geo(dims).V <= 131072);
}

// A launch per iteration saved against r read eight times over, with its
// rounding in FP16: 8^4 FP64 19.8 -> 17.2 us per iteration, FP32 19.4 -> 16.5,
// FP16 24.3 -> 17.9; 12^4 FP32 22.6 -> 21.2 but with two fields 28.1 -> 28.5, FP64
// 25.3 -> 26.0, FP16 with four fields 41.9 -> 40.4 and with eight 57.5 -> 60.8.
bool cg_fold_p(const int32_t dims[4], int prec, int n) {
  const Geo geo = make_geo(dims);
  const long most = prec == WD_FP64 ? 16384 : prec == WD_FP32 ? 32768 : 98304;
  const MarchParams p = march_params(geo, prec, n);
  return static_cast<long>(geo.V) * n <= most && small_slices(geo, p) && !small_march(geo, p, prec);
}

hipError_t launch_dslash_cg(const wd_gauge* g, const double* masses, int nrhs, const int* fields,
                            const void* in, void* out, const CgFuse& f, hipStream_t st) {
  return launch_any(g, masses, nrhs, fields, in, out, WD_FLAG_GAMMA5, nullptr, &f, st);
}

hipError_t launch_dslash(const wd_gauge* g, double mass, const void* in, void* out, int flags,
                         hipStream_t st) {
  return launch_dslash_multi(g, &mass, 1, nullptr, in, out, flags, st);
}

hipError_t launch_dslash_tuned(const wd_gauge* g, const double* masses, int nrhs, const void* in,
                               void* out, int flags, const MarchTuning& t, hipStream_t st) {
  return launch_any(g, masses, nrhs, nullptr, in, out, flags, &t, nullptr, st);
}

bool march_default(const int32_t dims[4], int prec, int nrhs, MarchTuning* t) {
  const Geo geo = make_geo(dims);
  const MarchParams p = march_params(geo, prec, nrhs);
  if (p.ny == 0) return false;
  *t = use_split(geo, p, prec) ? kSplitTuning : MarchTuning{p.tb, p.gw, p.group, p.rb};
  return true;
}

bool march_tuning_valid(const int32_t dims[4], int prec, int nrhs, const MarchTuning& t) {
  const Geo geo = make_geo(dims);
  const size_t real = real_bytes_of(prec);
  const MarchParams p = march_params(geo, prec, nrhs);
  if (p.ny == 0 || nrhs < 1 || nrhs > kMaxMultiRhs) return false;
  if (t.tb == 0)  // the split kernel
    return split_choice(geo, p, prec) && t.gw == kSplitTuning.gw && t.group == kSplitTuning.group && t.rb == kSplitTuning.rb;
  if (t.tb < 1 || t.tb > geo.T || t.group < 0) return false;
  if (t.rb != 1 && t.rb != 2) return false;
  if (t.gw < 1 || nrhs % (t.gw * t.rb) != 0) return false;
  const int n = geo.X * p.ny;
  if (t.gw > 1 || t.rb > 1) {  // several right-hand sides per workgroup: FP32 arithmetic only
    if (real != 4 || t.gw * n > kMarchMultiThreads) return false;
  }
  if (t.rb > 1 && t.gw != 1) return false;  // two per lane: one lane group per workgroup
  if (static_cast<size_t>(t.gw) * t.rb * march_lds_bytes(n, real) > kLdsBytes) return false;
  const long nb = static_cast<long>(nrhs / (t.gw * t.rb)) * p.ytiles * geo.Z * ((geo.T + t.tb - 1) / t.tb);
  return nb >= 1 && nb <= 0x7fffffffL;
}

void march_candidates(const int32_t dims[4], int prec, int nrhs, MarchTuning* out, int* n, int cap) {
  *n = 0;
  MarchTuning d;
  if (!march_default(dims, prec, nrhs, &d) || cap < 1) return;
  out[(*n)++] = d;
  const Geo geo = make_geo(dims);
  const MarchParams p = march_params(geo, prec, nrhs);
  // t steps per workgroup: the distinct ceil(T / nt) for nt workgroups along t
  int tbs[64];
  int ntb = 0;
  for (int nt = 1; nt <= geo.T && ntb < 64; ++nt) {
    const int tb = (geo.T + nt - 1) / nt;
    if (tb < 2 && nt > 1) break;
    if (ntb == 0 || tbs[ntb - 1] != tb) tbs[ntb++] = tb;
  }
  for (int rb = 1; rb <= 2; ++rb)
    for (int gw = 1; gw <= nrhs; ++gw) {
      if (nrhs % (gw * rb) != 0) continue;
      for (int i = 0; i < ntb; ++i) {
        const long nb =
            static_cast<long>(nrhs / (gw * rb)) * p.ytiles * geo.Z * ((geo.T + tbs[i] - 1) / tbs[i]);
        const int groups[2] = {0, static_cast<int>((nb + kNumXcd - 1) / kNumXcd)};
        for (int j = 0; j < 2; ++j) {
          const MarchTuning t{tbs[i], gw, groups[j], rb};
          if (!march_tuning_valid(dims, prec, nrhs, t)) continue;
          if (t.tb == d.tb && t.gw == d.gw && t.group == d.group && t.rb == d.rb) continue;
          if (*n < cap) out[(*n)++] = t;
        }
      }
    }
}

}  // namespace wd
