// Wilson-Dirac operator on the tiled site-major layout (FP64).
//
//   (M psi)(x) = psi(x) - kappa * sum_mu [ (1 - g_mu) U_mu(x) psi(x+mu)
//                                         + (1 + g_mu) U_mu(x-mu)^dag psi(x-mu) ]
//
// (the Wilson matrix of the paper's lattice tests, Section 2; conventions in
// include/deflan.h).  M^dag swaps the projector signs (gamma5 M gamma5 = M^dag)
// and gamma5 M flips the sign of spin components 2 and 3 of the result.
//
// Each (1 -/+ g_mu) has rank 2, so the neighbour spinor is first projected to
// a two-spin half spinor h (6 complex), multiplied by U or U^dag (two SU(3)
// mat-vecs instead of four), and the lower two spin rows are rebuilt from h.
// In the chiral basis, for the projector (1 + S g_mu), S = +-1:
//   mu=x: h0 = p0 + S i p3, h1 = p1 + S i p2;  rows 2,3 = -S i h1, -S i h0
//   mu=y: h0 = p0 - S p3,   h1 = p1 + S p2;    rows 2,3 =  S h1,   -S h0
//   mu=z: h0 = p0 + S i p2, h1 = p1 - S i p3;  rows 2,3 = -S i h0,  S i h1
//   mu=t: h0 = p0 + S p2,   h1 = p1 + S p3;    rows 2,3 =  S h0,    S h1
// One thread per site; loads of a component for 64 consecutive sites are one
// coalesced wavefront access; neighbour spinors and the backward links are
// re-read through L2 (blocks are mapped so that each XCD walks a contiguous
// slab of the lattice, keeping the +-z/+-t neighbours in its L2).
//
// The kernel is templated on the storage/arithmetic type (double: FP64,
// float: FP32 with FP32 accumulation) and applies the operator to a batch of
// right-hand sides: logical block b covers site block b / nrhs of right-hand
// side b % nrhs, so the nrhs blocks that read the same links are consecutive
// on one XCD and the links come from HBM once and from L2 for the others.
#include "internal.hpp"
#include "cplx.hpp"

#include <algorithm>
#include <map>
#include <mutex>

namespace dl {

// Element offsets are signed 32-bit ints (a field holds far fewer than 2^31
// elements), so component c of a site is base + off + c*64 and the c*64 part
// folds into the load's immediate offset.
__device__ __forceinline__ int sp_base(int site) { return (site >> 6) * (kSpin * kTile) + (site & 63); }
__device__ __forceinline__ int lk_base(int site, int mu) {
  return (site >> 6) * (kLinkC * kTile) + mu * 9 * kTile + (site & 63);
}

template <int MU, int S, class C>
__device__ __forceinline__ void project(const C p[12], C h[6]) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const C p0 = p[c], p1 = p[3 + c], p2 = p[6 + c], p3 = p[9 + c];
    if (MU == 0) {
      h[c] = S > 0 ? c_add(p0, c_i(p3)) : c_sub(p0, c_i(p3));
      h[3 + c] = S > 0 ? c_add(p1, c_i(p2)) : c_sub(p1, c_i(p2));
    } else if (MU == 1) {
      h[c] = S > 0 ? c_sub(p0, p3) : c_add(p0, p3);
      h[3 + c] = S > 0 ? c_add(p1, p2) : c_sub(p1, p2);
    } else if (MU == 2) {
      h[c] = S > 0 ? c_add(p0, c_i(p2)) : c_sub(p0, c_i(p2));
      h[3 + c] = S > 0 ? c_sub(p1, c_i(p3)) : c_add(p1, c_i(p3));
    } else {
      h[c] = S > 0 ? c_add(p0, p2) : c_sub(p0, p2);
      h[3 + c] = S > 0 ? c_add(p1, p3) : c_sub(p1, p3);
    }
  }
}

template <int MU, int S, class C>
__device__ __forceinline__ void reconstruct(C acc[12], const C g[6]) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const C g0 = g[c], g1 = g[3 + c];
    acc[c] = c_add(acc[c], g0);
    acc[3 + c] = c_add(acc[3 + c], g1);
    if (MU == 0) {
      acc[6 + c] = S > 0 ? c_sub(acc[6 + c], c_i(g1)) : c_add(acc[6 + c], c_i(g1));
      acc[9 + c] = S > 0 ? c_sub(acc[9 + c], c_i(g0)) : c_add(acc[9 + c], c_i(g0));
    } else if (MU == 1) {
      acc[6 + c] = S > 0 ? c_add(acc[6 + c], g1) : c_sub(acc[6 + c], g1);
      acc[9 + c] = S > 0 ? c_sub(acc[9 + c], g0) : c_add(acc[9 + c], g0);
    } else if (MU == 2) {
      acc[6 + c] = S > 0 ? c_sub(acc[6 + c], c_i(g0)) : c_add(acc[6 + c], c_i(g0));
      acc[9 + c] = S > 0 ? c_add(acc[9 + c], c_i(g1)) : c_sub(acc[9 + c], c_i(g1));
    } else {
      acc[6 + c] = S > 0 ? c_add(acc[6 + c], g0) : c_sub(acc[6 + c], g0);
      acc[9 + c] = S > 0 ? c_add(acc[9 + c], g1) : c_sub(acc[9 + c], g1);
    }
  }
}

template <int S, class C>
__device__ __forceinline__ void project_mu(int mu, const C p[12], C h[6]) {
  switch (mu) {
    case 0: project<0, S>(p, h); break;
    case 1: project<1, S>(p, h); break;
    case 2: project<2, S>(p, h); break;
    default: project<3, S>(p, h); break;
  }
}

template <int S, class C>
__device__ __forceinline__ void reconstruct_mu(int mu, C acc[12], const C g[6]) {
  switch (mu) {
    case 0: reconstruct<0, S>(acc, g); break;
    case 1: reconstruct<1, S>(acc, g); break;
    case 2: reconstruct<2, S>(acc, g); break;
    default: reconstruct<3, S>(acc, g); break;
  }
}

// g = U h (DAG false) or U^dag h (DAG true) on a half spinor (two colour vectors).
template <bool DAG, class C>
__device__ __forceinline__ void mul_half(const C u[9], const C h[6], C g[6]) {
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      C r = c_scale(h[s * 3], 0);
      if (!DAG) {
        r = c_fma(u[a * 3 + 0], h[s * 3 + 0], r);
        r = c_fma(u[a * 3 + 1], h[s * 3 + 1], r);
        r = c_fma(u[a * 3 + 2], h[s * 3 + 2], r);
      } else {
        r = c_fmac(u[0 * 3 + a], h[s * 3 + 0], r);
        r = c_fmac(u[1 * 3 + a], h[s * 3 + 1], r);
        r = c_fmac(u[2 * 3 + a], h[s * 3 + 2], r);
      }
      g[s * 3 + a] = r;
    }
}

// One hop in direction mu (runtime): load the neighbour spinor and the link (its 9
// components at up[e * ustride]), project, multiply by U (forward) or U^dag (backward,
// link taken at the neighbour), rebuild and accumulate.  Every load address depends on
// mu, so the loads of different directions cannot be hoisted ahead of each other.
template <int S, bool DAG, class C, class SV>
__device__ __forceinline__ void hop_at(const C* up, int ustride, const SV* in, int mu, int nb, C acc[12]) {
  C p[12], h[6], g[6], u[9];
  const SV* pp = in + sp_base(nb);
#pragma unroll
  for (int c = 0; c < 12; ++c) p[c] = sld(pp + c * kTile);
#pragma unroll
  for (int e = 0; e < 9; ++e) u[e] = up[e * ustride];
  project_mu<S>(mu, p, h);
  mul_half<DAG>(u, h, g);
  reconstruct_mu<S>(mu, acc, g);
}

template <int S, bool DAG, class C, class SV>
__device__ __forceinline__ void hop(const C* U, const SV* in, int mu, int nb, int lsite, C acc[12]) {
  hop_at<S, DAG>(U + lk_base(lsite, mu), kTile, in, mu, nb, acc);
}

// WHICH: 0 M, 1 M^dag, 2 gamma5 M.  RED: 0 none, 1 ||out||^2, 2 Re<in, out> (partials in FP64,
// column-major [nrhs][nbs]).  scale (optional, per rhs): out = scale * op(in).
// active (optional, per rhs): blocks of inactive right-hand sides return at once.
// Launch shape: NT threads per block, OCC the occupancy hint (waves per SIMD the
// register budget must allow); ORDER 0: rhs fastest, XCD-contiguous blocks; 1: sites
// fastest, XCD-contiguous; 2: rhs fastest, hardware block order.
// One site of the stencil for one field (zeroes padding sites); returns the fused
// reduction term (||out||^2 or Re<in, out>) of the site.
template <class R, class SV, int WHICH, int RED>
__device__ __forceinline__ double wilson_site(const typename CT<R>::type* __restrict__ U,
                                              const SV* __restrict__ in, SV* __restrict__ out, double kappa, int Lx, int Ly,
                                              int Lz, int Lt, long V, long Vpad, int site, R sc) {
  using C = typename CT<R>::type;
  double red = 0.0;
  if (site >= V && site < Vpad) {
    // padding sites of the last tile are kept at zero
    SV* op = out + sp_base(site);
#pragma unroll
    for (int c = 0; c < 12; ++c) sst(op + c * kTile, CT<R>::make(0, 0));
  }
  if (site < V) {
    const int x = site % Lx;
    const int y = (site / Lx) % Ly;
    const int z = (site / (Lx * Ly)) % Lz;
    const int t = site / (Lx * Ly * Lz);
    const int sy = Lx, sz = Lx * Ly, st = Lx * Ly * Lz;
    // neighbour offsets per direction
    const int fx = x == Lx - 1 ? 1 - Lx : 1, bx = x == 0 ? Lx - 1 : -1;
    const int fy = y == Ly - 1 ? (1 - Ly) * sy : sy, by = y == 0 ? (Ly - 1) * sy : -sy;
    const int fz = z == Lz - 1 ? (1 - Lz) * sz : sz, bz = z == 0 ? (Lz - 1) * sz : -sz;
    const int ft = t == Lt - 1 ? (1 - Lt) * st : st, bt = t == 0 ? (Lt - 1) * st : -st;
    C acc[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) acc[c] = CT<R>::make(0, 0);
    constexpr int SF = (WHICH == 1) ? 1 : -1;  // forward projector 1 + SF g_mu, backward 1 - SF g_mu
    // A runtime loop over the four directions (loads depend on mu) keeps the
    // compiler from hoisting all 168 neighbour/link loads ahead of the arithmetic.
#pragma unroll 1
    for (int mu = 0; mu < 4; ++mu) {
      const int df = mu == 0 ? fx : mu == 1 ? fy : mu == 2 ? fz : ft;
      const int db = mu == 0 ? bx : mu == 1 ? by : mu == 2 ? bz : bt;
      hop<SF, false>(U, in, mu, site + df, site, acc);
      hop<-SF, true>(U, in, mu, site + db, site + db, acc);
    }
    const R mk = (R)(-kappa);
    const SV* ip = in + sp_base(site);
    SV* op = out + sp_base(site);
    R sred = 0;  // this site's share of the reduction, summed in R
#pragma unroll
    for (int c = 0; c < 12; ++c) {
      const C p = sld(ip + c * kTile);
      C r = CT<R>::make(fma(mk, acc[c].x, p.x) * sc, fma(mk, acc[c].y, p.y) * sc);
      if (WHICH == 2 && c >= 6) r = CT<R>::make(-r.x, -r.y);
      sst(op + c * kTile, r);
      if (RED == 1) sred = fma(r.x, r.x, fma(r.y, r.y, sred));
      if (RED == 2) sred = fma(p.x, r.x, fma(p.y, r.y, sred));
    }
    if (RED == 1) red += (double)sred;
    if (RED == 2) red += (double)sred * sc;
  }
  return red;
}

template <class R, class SV, int WHICH, int RED, int NT, int OCC>
__global__ void __launch_bounds__(NT, OCC)
k_wilson(const typename CT<R>::type* __restrict__ U, const SV* __restrict__ in,
         SV* __restrict__ out, long fstride, int nrhs, double kappa, int Lx, int Ly, int Lz,
         int Lt, long V, long Vpad, int nbs, int order, const double* __restrict__ scale,
         const int* __restrict__ active, double* __restrict__ part) {
  const int lb = order == 2 ? (int)blockIdx.x : xcd_block(blockIdx.x, gridDim.x);
  const int rhs = order == 1 ? lb / nbs : lb % nrhs;
  const int sb = order == 1 ? lb % nbs : lb / nrhs;
  if (active && !active[rhs]) return;
  const int site = sb * NT + (int)threadIdx.x;
  const R sc = scale ? (R)scale[rhs] : (R)1;
  const double red = wilson_site<R, SV, WHICH, RED>(U, in + rhs * fstride, out + rhs * fstride, kappa, Lx, Ly, Lz, Lt,
                                                V, Vpad, site, sc);
  if (RED != 0) {
    __shared__ double lds[NT / 64];
    const double s = block_sum<NT>(red, lds);
    if (threadIdx.x == 0) part[(long)rhs * nbs + sb] = s;
  }
}

// Several lattices in one launch: a work list of items (lattice, links, kappa, range of
// right-hand sides).  Logical block b (XCD-contiguous) belongs to the item whose block
// range [block0, block0 + nbs * nrhs) holds it, and within the item to (site block, rhs)
// with the rhs fastest, so the blocks that read the same links are consecutive.  Field j
// starts at offs[j] (complex elements).  Partials: part[rhs * pstride + site block]; the
// first site block of each rhs zeroes the tail up to pstride, so every rhs reduces over
// pstride partials.
template <class R, class SV, int WHICH, int RED>
__global__ void __launch_bounds__(256, 2)
k_wilson_ml(const WilsonItem* __restrict__ items, int nitems, const SV* __restrict__ in,
            SV* __restrict__ out, const long* __restrict__ offs, int pstride,
            const double* __restrict__ scale, const int* __restrict__ active, double* __restrict__ part) {
  using C = typename CT<R>::type;
  const int b = xcd_block(blockIdx.x, gridDim.x);
  int it = 0;
  while (it + 1 < nitems && b >= items[it + 1].block0) ++it;
  const WilsonItem w = items[it];
  const int rl = (b - w.block0) % w.nrhs;
  const int sb = (b - w.block0) / w.nrhs;
  const int rhs = w.rhs0 + rl;
  if (active && !active[rhs]) return;
  const int site = sb * 256 + (int)threadIdx.x;
  const R sc = scale ? (R)scale[rhs] : (R)1;
  const long off = offs[rhs];
  const double red = wilson_site<R, SV, WHICH, RED>(static_cast<const C*>(w.U), in + off, out + off, w.kappa, w.L[0],
                                                w.L[1], w.L[2], w.L[3], w.V, w.Vpad, site, sc);
  if (RED != 0) {
    __shared__ double lds[256 / 64];
    const double s = block_sum<256>(red, lds);
    if (threadIdx.x == 0) part[(long)rhs * pstride + sb] = s;
    if (sb == 0)
      for (int q = w.nbs + (int)threadIdx.x; q < pstride; q += 256) part[(long)rhs * pstride + q] = 0.0;
  }
}

template <class R, class SV>
void wilson_multi(hipStream_t s, const WilsonItem* d_items, int nitems, int nblocks, int pstride, int which,
                  const SV* in, SV* out, const long* offs, int red, const double* scale, const int* active,
                  double* part) {
#define DL_ML(WH, RD)                                                                                          \
  hipLaunchKernelGGL((k_wilson_ml<R, SV, WH, RD>), dim3(nblocks), dim3(256), 0, s, d_items, nitems, in, out, offs, \
                     pstride, scale, active, part)
  if (which == 0) { if (red == 0) DL_ML(0, 0); else if (red == 1) DL_ML(0, 1); else DL_ML(0, 2); }
  else if (which == 1) { if (red == 0) DL_ML(1, 0); else if (red == 1) DL_ML(1, 1); else DL_ML(1, 2); }
  else { if (red == 0) DL_ML(2, 0); else if (red == 1) DL_ML(2, 1); else DL_ML(2, 2); }
#undef DL_ML
  DL_HIP(hipGetLastError());
}

template void wilson_multi<double, double2>(hipStream_t, const WilsonItem*, int, int, int, int, const double2*,
                                            double2*, const long*, int, const double*, const int*, double*);
template void wilson_multi<float, float2>(hipStream_t, const WilsonItem*, int, int, int, int, const float2*, float2*,
                                          const long*, int, const double*, const int*, double*);
template void wilson_multi<float, bf2>(hipStream_t, const WilsonItem*, int, int, int, int, const bf2*, bf2*,
                                       const long*, int, const double*, const int*, double*);

// t-marching form of the same operator.  A thread owns one (x, y, z) site and walks
// T consecutive time slices t0 .. t0+T-1 of it.  The forward-t neighbour psi(t+1)
// loaded at step t is the centre spinor of step t+1, and the backward-t hop of step
// t+1, U_t(t)^dag (1 + S g_t) psi(t), is formed at step t from the centre spinor and
// the forward link U_t(t) already in registers.  Every spinor and link is therefore
// read once along t; the x, y, z neighbours lie in the same time slice, which the
// blocks of one XCD walk together, so they come from L2.  A block is NT consecutive
// (x, y, z) sites of one time chunk of one right-hand side; logical block = (site block,
// rhs) with the same order options as k_wilson.  RES: out = add - op(in) (the residual
// b - M x, with its ||.||^2 under RED = 1), so M x is never written out.  LO = 1 / 2 (with RES):
// the residual is stored only rounded to FP32 / BF16 (through FP32) in lo, at the same element
// offsets, and RED = 1 sums the squares of the stored values.
template <class R, class SV, int WHICH, int RED, int NT, bool RES = false, int LO = 0>
__global__ void __launch_bounds__(NT)
k_wilson_tm(const typename CT<R>::type* __restrict__ U, const SV* __restrict__ in,
            SV* __restrict__ out, long fstride, int nrhs, double kappa, int Lx, int Ly, int Lz,
            int Lt, long V, long Vpad, int T, int nb3, int nbs, int order, const double* __restrict__ scale,
            const int* __restrict__ active, double* __restrict__ part, const SV* __restrict__ add,
            void* __restrict__ lo = nullptr) {
  using C = typename CT<R>::type;
  const int lb = order == 2 ? (int)blockIdx.x : xcd_block(blockIdx.x, gridDim.x);
  const int rhs = order == 1 ? lb / nbs : lb % nrhs;
  const int sb = order == 1 ? lb % nbs : lb / nrhs;
  if (active && !active[rhs]) {
    if (RES && RED != 0 && threadIdx.x == 0) part[(long)rhs * nbs + sb] = 0.0;  // an inactive rhs sums to 0
    return;
  }
  in += rhs * fstride;
  if (LO == 0) out += rhs * fstride;
  if (RES) add += rhs * fstride;
  float2* lo32 = LO == 1 ? static_cast<float2*>(lo) + rhs * fstride : nullptr;
  bf2* lo16 = LO == 2 ? static_cast<bf2*>(lo) + rhs * fstride : nullptr;
  const int b3 = sb % nb3, tc = sb / nb3;
  const int V3 = Lx * Ly * Lz;
  const int s3 = b3 * NT + (int)threadIdx.x;
  double red = 0.0;
  // (the low-precision residual's padding sites are zero already and stay so)
  if (LO == 0 && b3 == 0 && (tc + 1) * T >= Lt) {
    // padding sites of the last tile are kept at zero (written by the last chunk's first block)
    for (long sp = V + threadIdx.x; sp < Vpad; sp += NT) {
      SV* op = out + sp_base((int)sp);
#pragma unroll
      for (int c = 0; c < 12; ++c) sst(op + c * kTile, CT<R>::make(0, 0));
    }
  }
  if (s3 < V3) {
    const int x = s3 % Lx;
    const int y = (s3 / Lx) % Ly;
    const int z = s3 / (Lx * Ly);
    const int sy = Lx, sz = Lx * Ly;
    const int fx = x == Lx - 1 ? 1 - Lx : 1, bx = x == 0 ? Lx - 1 : -1;
    const int fy = y == Ly - 1 ? (1 - Ly) * sy : sy, by = y == 0 ? (Ly - 1) * sy : -sy;
    const int fz = z == Lz - 1 ? (1 - Lz) * sz : sz, bz = z == 0 ? (Lz - 1) * sz : -sz;
    constexpr int SF = (WHICH == 1) ? 1 : -1;  // forward projector 1 + SF g_mu, backward 1 - SF g_mu
    const int t0 = tc * T;
    const int t1 = t0 + T < Lt ? t0 + T : Lt;
    const R sc = scale ? (R)scale[rhs] : (R)1;
    const R mk = (R)(-kappa);
    // carried state: centre spinor of the current slice and the backward-t hop into it
    C cen[12], gb[6];
    {
      const int tp = t0 == 0 ? Lt - 1 : t0 - 1;
      const int sprev = tp * V3 + s3;
      C p[12], h[6], u[9];
      const SV* pp = in + sp_base(sprev);
#pragma unroll
      for (int c = 0; c < 12; ++c) p[c] = sld(pp + c * kTile);
      const C* up = U + lk_base(sprev, 3);
#pragma unroll
      for (int e = 0; e < 9; ++e) u[e] = up[e * kTile];
      project<3, -SF>(p, h);
      mul_half<true>(u, h, gb);
      const SV* cp = in + sp_base(t0 * V3 + s3);
#pragma unroll
      for (int c = 0; c < 12; ++c) cen[c] = sld(cp + c * kTile);
    }
#pragma unroll 1
    for (int t = t0; t < t1; ++t) {
      const int site = t * V3 + s3;
      C acc[12];
#pragma unroll
      for (int c = 0; c < 12; ++c) acc[c] = CT<R>::make(0, 0);
#pragma unroll 1
      for (int mu = 0; mu < 3; ++mu) {
        const int df = mu == 0 ? fx : mu == 1 ? fy : fz;
        const int db = mu == 0 ? bx : mu == 1 ? by : bz;
        hop<SF, false>(U, in, mu, site + df, site, acc);
        hop<-SF, true>(U, in, mu, site + db, site + db, acc);
      }
      // forward t: psi(t+1) is the next centre; U_t(t) also forms the next backward hop.
      // The hops are accumulated in k_wilson's order (x+, x-, y+, y-, z+, z-, t+, t-) with
      // the same arithmetic, so both kernels give the same result.
      const int snext = (t == Lt - 1 ? 0 : t + 1) * V3 + s3;
      C nx[12], u[9];
      {
        const SV* pp = in + sp_base(snext);
#pragma unroll
        for (int c = 0; c < 12; ++c) nx[c] = sld(pp + c * kTile);
        const C* up = U + lk_base(site, 3);
#pragma unroll
        for (int e = 0; e < 9; ++e) u[e] = up[e * kTile];
        C h[6], g[6];
        project<3, SF>(nx, h);
        mul_half<false>(u, h, g);
        reconstruct<3, SF>(acc, g);
        // backward t: the hop carried from the previous slice
        reconstruct<3, -SF>(acc, gb);
        project<3, -SF>(cen, h);
        mul_half<true>(u, h, gb);
      }
      SV* op = LO == 0 ? out + sp_base(site) : nullptr;  // (LO: out is not used)
      R sred = 0;  // this site's share of the reduction, summed in R
#pragma unroll
      for (int c = 0; c < 12; ++c) {
        const C p = cen[c];
        C r = CT<R>::make(fma(mk, acc[c].x, p.x) * sc, fma(mk, acc[c].y, p.y) * sc);
        if (WHICH == 2 && c >= 6) r = CT<R>::make(-r.x, -r.y);
        if (RES) {
          const C bv = sld(add + sp_base(site) + c * kTile);
          r = CT<R>::make(bv.x - r.x, bv.y - r.y);
        }
        if (LO != 0) {
          const float2 vf = make_float2((float)r.x, (float)r.y);
          float2 vs = vf;  // the stored value, as read back
          if (LO == 1) {
            lo32[sp_base(site) + c * kTile] = vf;
          } else {
            sst(lo16 + sp_base(site) + c * kTile, vf);
            vs = make_float2(__uint_as_float((unsigned)f2bf(vf.x) << 16), __uint_as_float((unsigned)f2bf(vf.y) << 16));
          }
          r = CT<R>::make((R)vs.x, (R)vs.y);
        } else {
          sst(op + c * kTile, r);
        }
        if (RED == 1) sred = fma(r.x, r.x, fma(r.y, r.y, sred));
        if (RED == 2) sred = fma(p.x, r.x, fma(p.y, r.y, sred));
      }
      if (RED == 1) red += (double)sred;
      if (RED == 2) red += (double)sred * sc;
#pragma unroll
      for (int c = 0; c < 12; ++c) cen[c] = nx[c];
    }
  }
  if (RED != 0) {
    __shared__ double lds[NT / 64];
    const double s = block_sum<NT>(red, lds);
    if (threadIdx.x == 0) part[(long)rhs * nbs + sb] = s;
  }
}

// Helpers of the slice-staged form: where hop h's neighbour comes from, and the loads of its
// spinor (raw storage values) and link, returned by value so they stay in registers.
struct HopSrc {
  bool near;    // the neighbour lies in the block's LDS slice
  unsigned li;  // its LDS index
  int d;        // site offset of the neighbour
};
template <class SV>
struct SpRaw {
  SV e[12];
};
template <class C>
struct Lk {
  C e[9];
};
template <int NT>
__device__ __forceinline__ HopSrc hop_src(int hh, int d, int s3, int base3, int V3) {
  const int mu = hh >> 1;
  const int nb3 = s3 + d;
  HopSrc r;
  r.d = d;
  r.li = (unsigned)(nb3 - base3);
  r.near = mu < 2 && r.li < (unsigned)NT && nb3 < V3;
  return r;
}
template <class SV>
__device__ __forceinline__ SpRaw<SV> fetch_sp(const SV* __restrict__ in, int site) {
  SpRaw<SV> r;
  const SV* pp = in + sp_base(site);
#pragma unroll
  for (int c = 0; c < 12; ++c) r.e[c] = pp[c * kTile];
  return r;
}
// link of hop hh: forward hops use U_mu(x), backward hops U_mu(x - mu)
template <class C>
__device__ __forceinline__ Lk<C> fetch_link(const C* __restrict__ U, int hh, const HopSrc& src, int site) {
  Lk<C> r;
  const C* up = U + lk_base((hh & 1) == 0 ? site : site + src.d, hh >> 1);
#pragma unroll
  for (int e = 0; e < 9; ++e) r.e[e] = up[e * kTile];
  return r;
}

// Time-marching form with the slice staged in LDS: a block is NT consecutive (x, y, z)
// sites of one time chunk of one rhs.  At each slice every thread writes its centre spinor
// to LDS; the x and y neighbours that fall inside the block's site range are then read from
// there instead of L2 (for a 16 x 16 plane per block that is all of them), the z neighbours
// and the links come from memory, and the t hops are carried along t as in k_wilson_tm.
// Same arithmetic and order as k_wilson.
template <class R, class SV, int WHICH, int RED, int NT, bool PF>
__global__ void __launch_bounds__(NT)
k_wilson_tmp(const typename CT<R>::type* __restrict__ U, const SV* __restrict__ in,
             SV* __restrict__ out, long fstride, int nrhs, double kappa, int Lx, int Ly, int Lz,
             int Lt, long V, long Vpad, int T, int nb3, int nbs, int order, const double* __restrict__ scale,
             const int* __restrict__ active, double* __restrict__ part) {
  using C = typename CT<R>::type;
  __shared__ C ps[12 * NT];  // centre spinors of the block's sites, component-major
  const int lb = order == 2 ? (int)blockIdx.x : xcd_block(blockIdx.x, gridDim.x);
  const int rhs = order == 1 ? lb / nbs : lb % nrhs;
  const int sb = order == 1 ? lb % nbs : lb / nrhs;
  if (active && !active[rhs]) return;
  in += rhs * fstride;
  out += rhs * fstride;
  const int b3 = sb % nb3, tc = sb / nb3;
  const int V3 = Lx * Ly * Lz;
  const int base3 = b3 * NT;
  const int tid = (int)threadIdx.x;
  const int s3 = base3 + tid;
  const bool valid = s3 < V3;
  double red = 0.0;
  if (b3 == 0 && (tc + 1) * T >= Lt) {
    for (long sp = V + tid; sp < Vpad; sp += NT) {
      SV* op = out + sp_base((int)sp);
#pragma unroll
      for (int c = 0; c < 12; ++c) sst(op + c * kTile, CT<R>::make(0, 0));
    }
  }
  int x = 0, y = 0, z = 0;
  if (valid) {
    x = s3 % Lx;
    y = (s3 / Lx) % Ly;
    z = s3 / (Lx * Ly);
  }
  const int sy = Lx, sz = Lx * Ly;
  const int fx = x == Lx - 1 ? 1 - Lx : 1, bx = x == 0 ? Lx - 1 : -1;
  const int fy = y == Ly - 1 ? (1 - Ly) * sy : sy, by = y == 0 ? (Ly - 1) * sy : -sy;
  const int fz = z == Lz - 1 ? (1 - Lz) * sz : sz, bz = z == 0 ? (Lz - 1) * sz : -sz;
  constexpr int SF = (WHICH == 1) ? 1 : -1;
  const int t0 = tc * T;
  const int t1 = t0 + T < Lt ? t0 + T : Lt;
  const R sc = scale ? (R)scale[rhs] : (R)1;
  const R mk = (R)(-kappa);
  C cen[12], gb[6];
  if (valid) {
    const int tp = t0 == 0 ? Lt - 1 : t0 - 1;
    const int sprev = tp * V3 + s3;
    C p[12], h[6], u[9];
    const SV* pp = in + sp_base(sprev);
#pragma unroll
    for (int c = 0; c < 12; ++c) p[c] = sld(pp + c * kTile);
    const C* up = U + lk_base(sprev, 3);
#pragma unroll
    for (int e = 0; e < 9; ++e) u[e] = up[e * kTile];
    project<3, -SF>(p, h);
    mul_half<true>(u, h, gb);
    const SV* cp = in + sp_base(t0 * V3 + s3);
#pragma unroll
    for (int c = 0; c < 12; ++c) cen[c] = sld(cp + c * kTile);
  }
#pragma unroll 1
  for (int t = t0; t < t1; ++t) {
    const int site = t * V3 + s3;
    __syncthreads();  // the previous slice is no longer read from LDS
    if (valid) {
#pragma unroll
      for (int c = 0; c < 12; ++c) ps[c * NT + tid] = cen[c];
    }
    __syncthreads();
    if (valid) {
      C acc[12];
#pragma unroll
      for (int c = 0; c < 12; ++c) acc[c] = CT<R>::make(0, 0);
      const int snext = (t == Lt - 1 ? 0 : t + 1) * V3 + s3;
      C nx[12];
      // Hop h (0..5: x+, x-, y+, y-, z+, z-) reads the neighbour's spinor from LDS (near) or
      // memory, and its link.  PF: the memory loads of hop h + 1 are issued before hop h is
      // computed, so two hops' loads are in flight at once.
      auto hop_d = [=](int hh) {
        return hh == 0 ? fx : hh == 1 ? bx : hh == 2 ? fy : hh == 3 ? by : hh == 4 ? fz : bz;
      };
      auto src_of = [=](int hh) { return hop_src<NT>(hh, hop_d(hh), s3, base3, V3); };
      HopSrc nsrc{};
      SpRaw<SV> nraw{};
      Lk<C> nu{};
      if (PF) {
        nsrc = src_of(0);
        if (!nsrc.near) nraw = fetch_sp(in, site + nsrc.d);
        nu = fetch_link(U, 0, nsrc, site);
      }
#pragma unroll 1
      for (int hop2 = 0; hop2 < 6; ++hop2) {
        const int mu = hop2 >> 1;
        const bool fwd = (hop2 & 1) == 0;
        C p[12], h[6], g[6], u[9];
        HopSrc src;
        SpRaw<SV> raw;
        Lk<C> lk;
        if (PF) {
          src = nsrc;
          raw = nraw;
          lk = nu;
          if (hop2 < 5) {
            nsrc = src_of(hop2 + 1);
            if (!nsrc.near) nraw = fetch_sp(in, site + nsrc.d);
            nu = fetch_link(U, hop2 + 1, nsrc, site);
          }
        } else {
          src = src_of(hop2);
          if (!src.near) raw = fetch_sp(in, site + src.d);
          lk = fetch_link(U, hop2, src, site);
        }
        if (src.near) {
#pragma unroll
          for (int c = 0; c < 12; ++c) p[c] = ps[c * NT + src.li];
        } else {
#pragma unroll
          for (int c = 0; c < 12; ++c) p[c] = sldv(raw.e[c]);
        }
#pragma unroll
        for (int e = 0; e < 9; ++e) u[e] = lk.e[e];
        if (fwd) {
          project_mu<SF>(mu, p, h);
          mul_half<false>(u, h, g);
          reconstruct_mu<SF>(mu, acc, g);
        } else {
          project_mu<-SF>(mu, p, h);
          mul_half<true>(u, h, g);
          reconstruct_mu<-SF>(mu, acc, g);
        }
      }
      C u[9];
      {
        {
          const SV* pp = in + sp_base(snext);
#pragma unroll
          for (int c = 0; c < 12; ++c) nx[c] = sld(pp + c * kTile);
        }
        const C* up = U + lk_base(site, 3);
#pragma unroll
        for (int e = 0; e < 9; ++e) u[e] = up[e * kTile];
        C h[6], g[6];
        project<3, SF>(nx, h);
        mul_half<false>(u, h, g);
        reconstruct<3, SF>(acc, g);
        reconstruct<3, -SF>(acc, gb);
        project<3, -SF>(cen, h);
        mul_half<true>(u, h, gb);
      }
      SV* op = out + sp_base(site);
      R sred = 0;  // this site's share of the reduction, summed in R
#pragma unroll
      for (int c = 0; c < 12; ++c) {
        const C p = cen[c];
        C r = CT<R>::make(fma(mk, acc[c].x, p.x) * sc, fma(mk, acc[c].y, p.y) * sc);
        if (WHICH == 2 && c >= 6) r = CT<R>::make(-r.x, -r.y);
        sst(op + c * kTile, r);
        if (RED == 1) sred = fma(r.x, r.x, fma(r.y, r.y, sred));
        if (RED == 2) sred = fma(p.x, r.x, fma(p.y, r.y, sred));
      }
      if (RED == 1) red += (double)sred;
      if (RED == 2) red += (double)sred * sc;
#pragma unroll
      for (int c = 0; c < 12; ++c) cen[c] = nx[c];
    }
  }
  if (RED != 0) {
    __shared__ double lds[NT / 64];
    const double s2 = block_sum<NT>(red, lds);
    if (threadIdx.x == 0) part[(long)rhs * nbs + sb] = s2;
  }
}

// Several right-hand sides per thread: a thread owns one site and RT consecutive rhs of a
// group; each hop's link is loaded once into registers and applied to the RT neighbour
// spinors, so links and neighbour offsets are read and computed once per site for the group
// (the one-rhs-per-block forms read each site's links once per rhs, from L2 at best) and the
// RT spinor loads of a hop are independent and in flight together.  Logical block = (site
// block, rhs group), order as k_wilson.  Same arithmetic and hop order as k_wilson per rhs.
template <class R, class SV, int WHICH, int RED, int NT, int RT>
__global__ void __launch_bounds__(NT)
k_wilson_mr(const typename CT<R>::type* __restrict__ U, const SV* __restrict__ in,
            SV* __restrict__ out, long fstride, int nrhs, double kappa, int Lx, int Ly, int Lz,
            int Lt, long V, long Vpad, int nbs, int ngroups, int order, const double* __restrict__ scale,
            const int* __restrict__ active, double* __restrict__ part) {
  using C = typename CT<R>::type;
  const int lb = order == 2 ? (int)blockIdx.x : xcd_block(blockIdx.x, gridDim.x);
  const int rg = order == 1 ? lb / nbs : lb % ngroups;
  const int sb = order == 1 ? lb % nbs : lb / ngroups;
  const int r0 = rg * RT;
  bool on[RT];
  bool any = false;
#pragma unroll
  for (int j = 0; j < RT; ++j) {
    on[j] = r0 + j < nrhs && (!active || active[r0 + j]);
    any |= on[j];
  }
  if (!any) return;
  const int site = sb * NT + (int)threadIdx.x;
  double red[RT];
#pragma unroll
  for (int j = 0; j < RT; ++j) red[j] = 0.0;
  if (site >= V && site < Vpad) {
#pragma unroll
    for (int j = 0; j < RT; ++j)
      if (on[j]) {
        SV* op = out + (r0 + j) * fstride + sp_base(site);
#pragma unroll
        for (int c = 0; c < 12; ++c) sst(op + c * kTile, CT<R>::make(0, 0));
      }
  }
  if (site < V) {
    const int x = site % Lx;
    const int y = (site / Lx) % Ly;
    const int z = (site / (Lx * Ly)) % Lz;
    const int t = site / (Lx * Ly * Lz);
    const int sy = Lx, sz = Lx * Ly, st = Lx * Ly * Lz;
    const int fx = x == Lx - 1 ? 1 - Lx : 1, bx = x == 0 ? Lx - 1 : -1;
    const int fy = y == Ly - 1 ? (1 - Ly) * sy : sy, by = y == 0 ? (Ly - 1) * sy : -sy;
    const int fz = z == Lz - 1 ? (1 - Lz) * sz : sz, bz = z == 0 ? (Lz - 1) * sz : -sz;
    const int ft = t == Lt - 1 ? (1 - Lt) * st : st, bt = t == 0 ? (Lt - 1) * st : -st;
    C acc[RT][12];
#pragma unroll
    for (int j = 0; j < RT; ++j)
#pragma unroll
      for (int c = 0; c < 12; ++c) acc[j][c] = CT<R>::make(0, 0);
    constexpr int SF = (WHICH == 1) ? 1 : -1;
#pragma unroll 1
    for (int hh = 0; hh < 8; ++hh) {
      const int mu = hh >> 1;
      const bool fwd = (hh & 1) == 0;
      const int d = fwd ? (mu == 0 ? fx : mu == 1 ? fy : mu == 2 ? fz : ft)
                        : (mu == 0 ? bx : mu == 1 ? by : mu == 2 ? bz : bt);
      const int nb = site + d;
      C u[9];
      const C* up = U + lk_base(fwd ? site : nb, mu);
#pragma unroll
      for (int e = 0; e < 9; ++e) u[e] = up[e * kTile];
      const SV* pb = in + sp_base(nb);
#pragma unroll
      for (int j = 0; j < RT; ++j) {
        if (!on[j]) continue;
        C p[12], h[6], g[6];
        const SV* pp = pb + (r0 + j) * fstride;
#pragma unroll
        for (int c = 0; c < 12; ++c) p[c] = sld(pp + c * kTile);
        if (fwd) {
          project_mu<SF>(mu, p, h);
          mul_half<false>(u, h, g);
          reconstruct_mu<SF>(mu, acc[j], g);
        } else {
          project_mu<-SF>(mu, p, h);
          mul_half<true>(u, h, g);
          reconstruct_mu<-SF>(mu, acc[j], g);
        }
      }
    }
    const R mk = (R)(-kappa);
#pragma unroll
    for (int j = 0; j < RT; ++j) {
      if (!on[j]) continue;
      const R sc = scale ? (R)scale[r0 + j] : (R)1;
      const SV* ip = in + (r0 + j) * fstride + sp_base(site);
      SV* op = out + (r0 + j) * fstride + sp_base(site);
      R sred = 0;
#pragma unroll
      for (int c = 0; c < 12; ++c) {
        const C p = sld(ip + c * kTile);
        C r = CT<R>::make(fma(mk, acc[j][c].x, p.x) * sc, fma(mk, acc[j][c].y, p.y) * sc);
        if (WHICH == 2 && c >= 6) r = CT<R>::make(-r.x, -r.y);
        sst(op + c * kTile, r);
        if (RED == 1) sred = fma(r.x, r.x, fma(r.y, r.y, sred));
        if (RED == 2) sred = fma(p.x, r.x, fma(p.y, r.y, sred));
      }
      if (RED == 1) red[j] = (double)sred;
      if (RED == 2) red[j] = (double)sred * sc;
    }
  }
  if (RED != 0) {
    __shared__ double lds[NT / 64];
#pragma unroll
    for (int j = 0; j < RT; ++j) {
      if (!on[j]) continue;  // uniform over the block
      const double s = block_sum<NT>(red[j], lds);
      if (threadIdx.x == 0) part[(long)(r0 + j) * nbs + sb] = s;
      __syncthreads();  // lds is reused by the next rhs's sum
    }
  }
}

// One hop per wave: a block is one 64-site tile of one rhs and eight waves; wave h forms the
// transported half spinor of hop h (x+, x-, y+, ...) for the tile's sites and leaves it in LDS, then
// the block adds the eight hops in k_wilson's order, 12 components x 64 sites over 512 threads.  What
// bounds a small lattice is the chain of memory latencies in a thread, not bytes: k_wilson walks four
// pairs of hops one after the other, here every load of a site is in flight at once, on eight times as
// many waves.  FP64, one field: 4^4 8.1 -> 5.0 us, 8^4 8.2 -> 5.1 us.  The tuner takes it for one FP64 field
// up to 16^3 x 32 (30.2 us, the box 31.2), in FP32 to 26^4, and for 12 fields to about 10^4 sites; with more
// sites in flight the LDS round trip costs more than it hides (24^3 x 48 168 us, the box 140).
template <int MU, int S, class C>
__device__ __forceinline__ void add_row(int spin, const C* g0, const C* g1, C& acc) {
  // row `spin` of the rebuilt spinor from the half spinor (g0, g1), as in reconstruct()
  if (spin == 0) acc = c_add(acc, *g0);
  else if (spin == 1) acc = c_add(acc, *g1);
  else if (spin == 2) {
    if (MU == 0) acc = S > 0 ? c_sub(acc, c_i(*g1)) : c_add(acc, c_i(*g1));
    if (MU == 1) acc = S > 0 ? c_add(acc, *g1) : c_sub(acc, *g1);
    if (MU == 2) acc = S > 0 ? c_sub(acc, c_i(*g0)) : c_add(acc, c_i(*g0));
    if (MU == 3) acc = S > 0 ? c_add(acc, *g0) : c_sub(acc, *g0);
  } else {
    if (MU == 0) acc = S > 0 ? c_sub(acc, c_i(*g0)) : c_add(acc, c_i(*g0));
    if (MU == 1) acc = S > 0 ? c_sub(acc, *g0) : c_add(acc, *g0);
    if (MU == 2) acc = S > 0 ? c_add(acc, c_i(*g1)) : c_sub(acc, c_i(*g1));
    if (MU == 3) acc = S > 0 ? c_add(acc, *g1) : c_sub(acc, *g1);
  }
}

template <class R, class SV, int WHICH, int RED>
__global__ void __launch_bounds__(512)
k_wilson_split(const typename CT<R>::type* __restrict__ U, const SV* __restrict__ in, SV* __restrict__ out,
               long fstride, int nrhs, double kappa, int Lx, int Ly, int Lz, int Lt, long V, long Vpad, int nbs,
               int order, const double* __restrict__ scale, const int* __restrict__ active,
               double* __restrict__ part) {
  using C = typename CT<R>::type;
  __shared__ C gs[8][6][kTile];
  const int lb = order == 2 ? (int)blockIdx.x : xcd_block(blockIdx.x, gridDim.x);
  const int rhs = order == 1 ? lb / nbs : lb % nrhs;
  const int sb = order == 1 ? lb % nbs : lb / nrhs;
  if (active && !active[rhs]) return;
  in += rhs * fstride;
  out += rhs * fstride;
  const int lane = threadIdx.x & 63, hop = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int site = sb * kTile + lane;
  constexpr int SF = (WHICH == 1) ? 1 : -1;
  if (site < V) {
    const int mu = hop >> 1;
    const bool fwd = (hop & 1) == 0;
    const int st = mu == 0 ? 1 : mu == 1 ? Lx : mu == 2 ? Lx * Ly : Lx * Ly * Lz;
    const int L = mu == 0 ? Lx : mu == 1 ? Ly : mu == 2 ? Lz : Lt;
    const int x = (site / st) % L;
    const int nb = fwd ? (x == L - 1 ? site - (L - 1) * st : site + st) : (x == 0 ? site + (L - 1) * st : site - st);
    C p[12], h[6], g[6], u[9];
    const SV* pp = in + sp_base(nb);
#pragma unroll
    for (int c = 0; c < 12; ++c) p[c] = sld(pp + c * kTile);
    const C* up = U + lk_base(fwd ? site : nb, mu);
#pragma unroll
    for (int e = 0; e < 9; ++e) u[e] = up[e * kTile];
    if (fwd) {
      project_mu<SF>(mu, p, h);
      mul_half<false>(u, h, g);
    } else {
      project_mu<-SF>(mu, p, h);
      mul_half<true>(u, h, g);
    }
#pragma unroll
    for (int c = 0; c < 6; ++c) gs[hop][c][lane] = g[c];
  }
  __syncthreads();
  const R sc = scale ? (R)scale[rhs] : (R)1;
  const R mk = (R)(-kappa);
  double red = 0.0;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int c = hop + 8 * k;  // component of this wave
    if (c >= 12) break;
    SV* op = out + sp_base(site) + c * kTile;
    if (site >= V) {
      if (site < Vpad) sst(op, CT<R>::make(0, 0));
      continue;
    }
    const int spin = c / 3, a = c % 3;
    C acc = CT<R>::make(0, 0);
#define DL_ROW(H, MU, S) add_row<MU, S>(spin, &gs[H][a][lane], &gs[H][3 + a][lane], acc)
    DL_ROW(0, 0, SF);
    DL_ROW(1, 0, -SF);
    DL_ROW(2, 1, SF);
    DL_ROW(3, 1, -SF);
    DL_ROW(4, 2, SF);
    DL_ROW(5, 2, -SF);
    DL_ROW(6, 3, SF);
    DL_ROW(7, 3, -SF);
#undef DL_ROW
    const C p = sld(in + sp_base(site) + c * kTile);
    C r = CT<R>::make(fma(mk, acc.x, p.x) * sc, fma(mk, acc.y, p.y) * sc);
    if (WHICH == 2 && c >= 6) r = CT<R>::make(-r.x, -r.y);
    sst(op, r);
    if (RED == 1) red += (double)fma(r.x, r.x, r.y * r.y);
    if (RED == 2) red += (double)fma(p.x, r.x, p.y * r.y) * sc;
  }
  if (RED != 0) {
    __shared__ double lds[8];
    const double s = block_sum<512>(red, lds);
    if (threadIdx.x == 0) part[(long)rhs * nbs + sb] = s;
  }
}

// Box form: a block is a box of by x bz whole x rows of a time slice (at most NT sites, spare threads
// idle) that marches through a time chunk for RT right-hand sides.  Each slice's centre spinors sit
// widened in LDS, so x neighbours (and y and z neighbours inside the box) are read from there, the
// others from memory; the t hops are carried along t as in k_wilson_tm.  Every hop is unrolled
// with its own projection, one link is loaded ahead of the hop before it, and serves the RT rhs.
// What bounds it: FP32 instruction issue (packed FP32 arithmetic is not used), 8 hops x 108 operations,
// the epilogue and the BF16 conversions, 1140 a site and rhs by the counters or 243 us for 64 rhs of
// 16^3 x 32 (0.69 of its time), and below that the latency of its loads: two rhs a thread halve the link loads
// and give two chains at two waves per SIMD.
// 16^3 x 32, 64 BF16 rhs: 436 -> 352 us alone (2.4 TB/s algorithmic; 458 -> 379 within D-CG); 16 FP32 rhs
// 178 -> 110 (187 -> 174 within D-CG, where its input comes from HBM); FP64, one field 35 -> 31, 64 rhs
// 1237 -> 971; 24^3 x 48 FP64, one field 168 -> 140 (4.6 TB/s).  Without the spinors one hop ahead 64 BF16
// rhs took 393 us.
// Registers: BF16 149 (one rhs, three waves per SIMD) and 210 (two), FP32 152 to 158 (one), none spilled.  FP32 with
// two rhs fills its 256 and spills 6 values a lane, 25 (48 B) with a fused reduction; FP64 253, with a reduction 4
// spilled (12 B); the FP64 residual stored whole (LO 0) 20 (76 B).
// nt: the result is stored non-temporally.  RES, LO: the residual forms of k_wilson_tm.
template <class R, class SV, int WHICH, int RED, int RT, int NT, bool RES = false, int LO = 0>
__global__ void __launch_bounds__(NT, RT == 1 && sizeof(R) == 4 ? 3 : 2)
k_wilson_box(const typename CT<R>::type* __restrict__ U, const SV* __restrict__ in, SV* __restrict__ out,
             long fstride, int nrhs, double kappa, int Lx, int Ly, int Lz, int Lt, long V, long Vpad, int T, int nb3,
             int nbs, int ngroups, int order, const double* __restrict__ scale, const int* __restrict__ active,
             double* __restrict__ part, int boy, int boz, int nt, const SV* __restrict__ add,
             void* __restrict__ lo) {
  using C = typename CT<R>::type;
  static_assert(!RES || RT == 1, "the residual is formed for one rhs a block");
  __shared__ C ps[RT][12 * NT];
  const int lb = order == 2 ? (int)blockIdx.x : xcd_block(blockIdx.x, gridDim.x);
  const int rg = order == 1 ? lb / nbs : lb % ngroups;
  const int sb = order == 1 ? lb % nbs : lb / ngroups;
  bool on[RT];
  bool any = false;
#pragma unroll
  for (int j = 0; j < RT; ++j) {
    const int r = rg * RT + j;
    on[j] = r < nrhs && (!active || active[r]);
    any |= on[j];
  }
  if (!any) {  // uniform over the block
    if (RES && RED != 0 && threadIdx.x == 0) part[(long)rg * nbs + sb] = 0.0;  // an inactive rhs sums to 0
    return;
  }
  in += (long)rg * RT * fstride;
  if (LO == 0) out += (long)rg * RT * fstride;
  if (RES) add += (long)rg * fstride;
  float2* lo32 = LO == 1 ? static_cast<float2*>(lo) + (long)rg * fstride : nullptr;
  bf2* lo16 = LO == 2 ? static_cast<bf2*>(lo) + (long)rg * fstride : nullptr;
  const int b3 = sb % nb3, tc = sb / nb3;
  const int V3 = Lx * Ly * Lz;
  const int tid = (int)threadIdx.x;
  const bool valid = tid < Lx * boy * boz;
  const int nby = Ly / boy;
  const int x = tid % Lx, ly = (tid / Lx) % boy, lz = tid / (Lx * boy);
  const int y = (b3 % nby) * boy + ly, z = (b3 / nby) * boz + lz;
  const int s3 = x + Lx * (y + Ly * z);
  const int t0 = tc * T;
  const int t1 = t0 + T < Lt ? t0 + T : Lt;
  double red[RT];
#pragma unroll
  for (int j = 0; j < RT; ++j) red[j] = 0.0;
  // (the low-precision residual's padding sites are zero already and stay so)
  if (LO == 0 && b3 == 0 && t1 == Lt) {
    for (long sp = V + tid; sp < Vpad; sp += NT)
#pragma unroll
      for (int j = 0; j < RT; ++j)
        if (on[j]) {
          SV* op = out + j * fstride + sp_base((int)sp);
#pragma unroll
          for (int c = 0; c < 12; ++c) sst(op + c * kTile, CT<R>::make(0, 0));
        }
  }
  // site offsets of the neighbours, and their LDS index (-1: outside the box)
  const int sy = Lx, sz = Lx * Ly;
  const int fx = x == Lx - 1 ? 1 - Lx : 1, bx = x == 0 ? Lx - 1 : -1;
  const int fy = y == Ly - 1 ? (1 - Ly) * sy : sy, by = y == 0 ? (Ly - 1) * sy : -sy;
  const int fz = z == Lz - 1 ? (1 - Lz) * sz : sz, bz = z == 0 ? (Lz - 1) * sz : -sz;
  const int ry = Lx, rz = Lx * boy;
  const int lfy = ly < boy - 1 ? tid + ry : boy == Ly ? tid - (boy - 1) * ry : -1;
  const int lby = ly > 0 ? tid - ry : boy == Ly ? tid + (boy - 1) * ry : -1;
  const int lfz = lz < boz - 1 ? tid + rz : boz == Lz ? tid - (boz - 1) * rz : -1;
  const int lbz = lz > 0 ? tid - rz : boz == Lz ? tid + (boz - 1) * rz : -1;
  constexpr int SF = (WHICH == 1) ? 1 : -1;
  constexpr bool PF = sizeof(R) == 4;  // spinors one hop ahead (FP64 has no registers left for them)
  const R mk = (R)(-kappa);
  R sc[RT];
#pragma unroll
  for (int j = 0; j < RT; ++j) sc[j] = scale && on[j] ? (R)scale[rg * RT + j] : (R)1;
  // Loads at a uniform base and a 32-bit byte offset of the site (links and fields are under 4 GB
  // here), with the components in the instruction's offset, counted from the middle one.
  auto link = [&](unsigned site, int mu) {
    Lk<C> l;
    const char* base = reinterpret_cast<const char*>(U + (mu * 9 + 4) * kTile);
    const unsigned o = (site >> 6) * (unsigned)(kLinkC * kTile * sizeof(C)) + (site & 63) * (unsigned)sizeof(C);
#pragma unroll
    for (int e = 0; e < 9; ++e)
      l.e[e] = *reinterpret_cast<const C*>(base + o + (e - 4) * (int)(kTile * sizeof(C)));
    return l;
  };
  auto soff = [](unsigned site) {
    return (site >> 6) * (unsigned)(kSpin * kTile * sizeof(SV)) + (site & 63) * (unsigned)sizeof(SV);
  };
  auto spinor = [&](int j, unsigned site) {
    SpRaw<SV> r;
    const char* base = reinterpret_cast<const char*>(in + j * fstride + 6 * kTile);
    const unsigned o = soff(site);
#pragma unroll
    for (int c = 0; c < 12; ++c)
      r.e[c] = *reinterpret_cast<const SV*>(base + o + (c - 6) * (int)(kTile * sizeof(SV)));
    return r;
  };
  SpRaw<SV> cur[RT];  // centre spinors of the slice, as stored
  Lk<C> u;            // link of the next hop
  C gb[RT][6];        // backward t hop into the slice
  if (valid) {
    const int sprev = (t0 == 0 ? Lt - 1 : t0 - 1) * V3 + s3;
    u = link(sprev, 3);
#pragma unroll
    for (int j = 0; j < RT; ++j) {
      if (!on[j]) continue;
      const SpRaw<SV> raw = spinor(j, sprev);
      cur[j] = spinor(j, t0 * V3 + s3);
      C p[12], h[6];
#pragma unroll
      for (int c = 0; c < 12; ++c) p[c] = sldv(raw.e[c]);
      project<3, -SF>(p, h);
      mul_half<true>(u.e, h, gb[j]);
    }
    u = link(t0 * V3 + s3, 0);
  }
#pragma unroll 1
  for (int t = t0; t < t1; ++t) {
    int site = t * V3 + s3;
    asm volatile("" : "+v"(site));  // keeps the compiler from carrying one pointer per hop around the loop
    __syncthreads();  // the previous slice is no longer read from LDS
    if (valid) {
#pragma unroll
      for (int j = 0; j < RT; ++j)
#pragma unroll
        for (int c = 0; c < 12; ++c) ps[j][c * NT + tid] = sldv(cur[j].e[c]);
    }
    __syncthreads();
    if (!valid) continue;
    C acc[RT][12];
    SpRaw<SV> raw[RT];
    // One hop: the next hop's link and, where they lie outside the box, its spinors are requested first
    // (nli, nnb: their LDS index and site), then this one's are taken from LDS (index li >= 0; x
    // neighbours always are) or from the registers that the hop before filled.
    auto hop = [&](auto MUc, auto Sc, auto DAGc, int li, int nb, auto FIRSTc, int next_site, int next_mu, int nli,
                   int nnb) {
      constexpr int MU = decltype(MUc)::value, S = decltype(Sc)::value;
      constexpr bool DAG = decltype(DAGc)::value, FIRST = decltype(FIRSTc)::value;
      // opaque here, so that the loads of later hops are not gathered ahead of this one's arithmetic
      asm volatile("" : "+v"(next_site), "+v"(nnb));
      const Lk<C> un = link(next_site, next_mu);
#pragma unroll
      for (int j = 0; j < RT; ++j) {
        if (!on[j]) continue;
        C p[12], h[6], g[6];
        if (MU == 0 || li >= 0) {
#pragma unroll
          for (int c = 0; c < 12; ++c) p[c] = ps[j][c * NT + li];
        } else {
          if (!PF) raw[j] = spinor(j, nb);
#pragma unroll
          for (int c = 0; c < 12; ++c) p[c] = sldv(raw[j].e[c]);
        }
        if (PF && !(MU == 0 && FIRST) && nli < 0) raw[j] = spinor(j, nnb);
        project<MU, S>(p, h);
        mul_half<DAG>(u.e, h, g);
        if (FIRST) {
#pragma unroll
          for (int c = 0; c < 12; ++c) acc[j][c] = CT<R>::make(0, 0);
        }
        reconstruct<MU, S>(acc[j], g);
        // the sums are wanted here: left to itself the compiler sinks a hop's arithmetic to the slice's
        // end, with every hop's operands held (256 registers)
#pragma unroll
        for (int c = 0; c < 12; ++c) asm volatile("" : "+v"(acc[j][c].x), "+v"(acc[j][c].y));
      }
      u = un;
      __builtin_amdgcn_sched_barrier(0);
    };
    constexpr std::integral_constant<int, SF> P{};
    constexpr std::integral_constant<int, -SF> N{};
    constexpr std::integral_constant<int, 0> X{};
    constexpr std::integral_constant<int, 1> Y{};
    constexpr std::integral_constant<int, 2> Z{};
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    const int snext = (t == Lt - 1 ? 0 : t + 1) * V3 + s3;
    if (!PF) u = link(site, 0);
    hop(X, P, no, tid + fx, site, yes, site + bx, 0, 0, site);
    hop(X, N, yes, tid + bx, site, no, site, 1, lfy, site + fy);
    hop(Y, P, no, lfy, site + fy, no, site + by, 1, lby, site + by);
    hop(Y, N, yes, lby, site + by, no, site, 2, lfz, site + fz);
    hop(Z, P, no, lfz, site + fz, no, site + bz, 2, lbz, site + bz);
    hop(Z, N, yes, lbz, site + bz, no, site, 3, -1, snext);
    Lk<C> ux{};
    if (PF) ux = link(snext, 0);  // the next slice's first link
#pragma unroll
    for (int j = 0; j < RT; ++j) {
      if (!on[j]) continue;
      cur[j] = PF ? raw[j] : spinor(j, snext);
      C p[12], h[6], g[6];
#pragma unroll
      for (int c = 0; c < 12; ++c) p[c] = sldv(cur[j].e[c]);
      project<3, SF>(p, h);
      mul_half<false>(u.e, h, g);
      reconstruct<3, SF>(acc[j], g);
      reconstruct<3, -SF>(acc[j], gb[j]);
#pragma unroll
      for (int c = 0; c < 12; ++c) p[c] = ps[j][c * NT + tid];
      project<3, -SF>(p, h);
      mul_half<true>(u.e, h, gb[j]);
      char* op = reinterpret_cast<char*>(out + j * fstride + 6 * kTile);
      const unsigned oo = soff(site);
      R sred = 0;  // this site's share of the reduction, summed in R
#pragma unroll
      for (int c = 0; c < 12; ++c) {
        const int co = (c - 6) * (int)(kTile * sizeof(SV));
        C r = CT<R>::make(fma(mk, acc[j][c].x, p[c].x) * sc[j], fma(mk, acc[j][c].y, p[c].y) * sc[j]);
        if (WHICH == 2 && c >= 6) r = CT<R>::make(-r.x, -r.y);
        if (RES) {
          const C bv = sldv(*reinterpret_cast<const SV*>(reinterpret_cast<const char*>(add + 6 * kTile) + oo + co));
          r = CT<R>::make(bv.x - r.x, bv.y - r.y);
        }
        if (LO != 0) {
          const float2 vf = make_float2((float)r.x, (float)r.y);
          float2 vs = vf;  // the stored value, as read back
          if (LO == 1) {
            sst_nt(lo32 + sp_base(site) + c * kTile, vf);
          } else {
            sst_nt(lo16 + sp_base(site) + c * kTile, vf);
            vs = make_float2(__uint_as_float((unsigned)f2bf(vf.x) << 16), __uint_as_float((unsigned)f2bf(vf.y) << 16));
          }
          r = CT<R>::make((R)vs.x, (R)vs.y);
        }
        acc[j][c] = r;
        if (RED == 1) sred = fma(r.x, r.x, fma(r.y, r.y, sred));
        if (RED == 2) sred = fma(p[c].x, r.x, fma(p[c].y, r.y, sred));
      }
      if (LO == 0) {
        char* o = op + oo - 6 * (int)(kTile * sizeof(SV));
        if (nt) {
#pragma unroll
          for (int c = 0; c < 12; ++c) sst_nt(reinterpret_cast<SV*>(o) + c * kTile, acc[j][c]);
        } else {
#pragma unroll
          for (int c = 0; c < 12; ++c) sst(reinterpret_cast<SV*>(o) + c * kTile, acc[j][c]);
        }
      }
      if (RED == 1) red[j] += (double)sred;
      if (RED == 2) red[j] += (double)sred * sc[j];
    }
    if (PF) u = ux;
  }
  if (RED != 0) {
    __shared__ double lds[NT / 64];
#pragma unroll
    for (int j = 0; j < RT; ++j) {
      if (!on[j]) continue;  // uniform over the block
      const double s = block_sum<NT>(red[j], lds);
      if (tid == 0) part[(long)(rg * RT + j) * nbs + sb] = s;
    }
  }
}

// Launch-shape variants.  0-3: k_wilson with (threads per block, occupancy hint)
// {(256,2), (128,2), (512,1), (256,1)}; 4-6: k_wilson_tm, 256 threads per block, time
// chunks of T = 4, 8, 16 slices; 12-14: k_wilson_tmp, T = 8, 16, 8 (14 with loads one hop ahead).
// 15-17: k_wilson_mr with (threads per block, rhs per thread) = (256, 2), (256, 4), (128, 2).
// 20: k_wilson_split, 64 sites per block.
// 21-26: k_wilson_box with (rhs per block, T) = (1, 4), (1, 8), (1, 16), (2, 4), (2, 8), (2, 16) (FP64: 24-26
// are 21-23); where no box fits a slice they launch variants 4 to 6.
// The numbers 7-11, 18 and 19 launch 12 or 13: their forms (links staged in LDS for several rhs or beside
// the spinors, an earlier box) were the fastest for 1 of 1143 keys (37 lattices from 4^3 x 8 to 34^3 x 8 and
// 16^3 x 64, three precisions, 1 to 64 rhs), by 1.2%, and took 29% of the tuning time.
static constexpr int kVariantNT[kWilsonVariants] = {256, 128, 512, 256, 256, 256, 256, 256, 256, 256, 256, 256, 256, 256,
                                                    256, 256, 256, 128, 256, 256, 64, 256, 256, 256, 256, 256, 256};
static constexpr int kVariantT[kWilsonVariants] = {0, 0, 0, 0, 4, 8, 16, 8, 16, 8, 8, 8, 8, 16, 8, 0, 0, 0, 8, 16, 0,
                                                   4, 8, 16, 4, 8, 16};
static constexpr int kVariantRT[kWilsonVariants] = {1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 2, 4, 2, 1, 1, 1,
                                                    1, 1, 1, 2, 2, 2};
constexpr int kFirstBox = 21, kBoxNT = 256;

static bool site_box(const Lattice& lat, int* by, int* bz);

// Blocks of a time slice.
static int tm_nb3(const Lattice& lat, int v) {
  if (v >= kFirstBox) {
    int by = 1, bz = 1;
    site_box(lat, &by, &bz);
    return (lat.L[1] / by) * (lat.L[2] / bz);
  }
  return (lat.L[0] * lat.L[1] * lat.L[2] + kVariantNT[v] - 1) / kVariantNT[v];
}
static int tm_chunks(const Lattice& lat, int v) { return (lat.L[3] + kVariantT[v] - 1) / kVariantT[v]; }

template <class R, class SV, int WHICH, int RED, int NT>
static void launch_tm(hipStream_t s, const Lattice& lat, const cplx_t<R>* U, double kappa, const SV* in,
                      SV* out, long fstride, int nrhs, int order, const double* scale, const int* active,
                      double* part, int nbs, int v) {
  const int* L = lat.L;
  hipLaunchKernelGGL((k_wilson_tm<R, SV, WHICH, RED, NT>), dim3(nbs * nrhs), dim3(NT), 0, s, U, in, out, fstride, nrhs,
                     kappa, L[0], L[1], L[2], L[3], lat.V, lat.ntiles * kTile, kVariantT[v], tm_nb3(lat, v), nbs,
                     order, scale, active, part, static_cast<const SV*>(nullptr), static_cast<void*>(nullptr));
}

template <class R, class SV, int WHICH, int RED, int NT, int OCC>
static void launch_one(hipStream_t s, const Lattice& lat, const cplx_t<R>* U, double kappa, const SV* in,
                       SV* out, long fstride, int nrhs, int order, const double* scale, const int* active,
                       double* part, int nbs) {
  const int* L = lat.L;
  hipLaunchKernelGGL((k_wilson<R, SV, WHICH, RED, NT, OCC>), dim3(nbs * nrhs), dim3(NT), 0, s, U, in, out, fstride, nrhs,
                     kappa, L[0], L[1], L[2], L[3], lat.V, lat.ntiles * kTile, nbs, order, scale, active, part);
}

// Box of k_wilson_box: by | Ly, bz | Lz, Lx by bz <= NT, for the least work per site: neighbour spinors from
// memory (2 / by and 2 / bz a site unless the box spans the lattice) on top of about five spinors'
// worth of arithmetic, over the share of threads with a site.  False if no box fills half a block.
static bool site_box(const Lattice& lat, int* by, int* bz) {
  const int* L = lat.L;
  double best = 1e300;
  for (int y = 1; y <= L[1] && L[0] * y <= kBoxNT; ++y) {
    if (L[1] % y != 0) continue;
    for (int z = 1; z <= L[2] && L[0] * y * z <= kBoxNT; ++z) {
      if (L[2] % z != 0 || 2 * L[0] * y * z < kBoxNT) continue;
      const double far = (y < L[1] ? 2.0 / y : 0.0) + (z < L[2] ? 2.0 / z : 0.0);
      const double cost = (5.0 + far) / (L[0] * y * z);
      if (cost < best) {
        best = cost;
        *by = y;
        *bz = z;
      }
    }
  }
  return best < 1e300;
}

// k_wilson_box needs a box, 32-bit byte offsets (the FP64 links under 4 GB) and no more blocks a field than the
// fused reductions take; FP64 has registers for one rhs a block only.
int wilson_shape(const Lattice& lat, int v, bool fp64) {
  int by, bz;
  if (wilson_retired(v)) return kVariantT[v] == 16 ? 13 : 12;
  if (v < kFirstBox) return v;
  if ((double)lat.ntiles * kTile * kLinkC * sizeof(double2) < 4294967296.0 && site_box(lat, &by, &bz) &&
      (long)(lat.L[1] / by) * (lat.L[2] / bz) * ((lat.L[3] + kVariantT[v] - 1) / kVariantT[v]) <= kMaxPartials)
    return fp64 ? kFirstBox + (v - kFirstBox) % 3 : v;
  return 4 + (v - kFirstBox) % 3;
}

// Every different launch once: no variant that runs as another one, no second chunk length that covers all of t,
// no site order where one group holds every rhs, and no grid wider than the fused reductions take.  Nine keys
// (three precisions; 1, 12 and 64 rhs) tuned in 181 -> 108 ms at 4^4, 3.23 -> 3.04 s at 16^3 x 32 and, where there is
// no box, 4.13 -> 2.49 s at 26^3 x 8.
std::vector<WilsonCfg> wilson_candidates(const Lattice& lat, bool fp64, int nrhs) {
  std::vector<WilsonCfg> out;
  for (int v = 0; v < kWilsonVariants; ++v) {
    if (wilson_shape(lat, v, fp64) != v || wilson_nbs(lat, WilsonCfg{v, 0}) > kMaxPartials) continue;
    // the family's shorter chunk is the variant before
    const bool longer = v == 5 || v == 6 || v == 13 || v == 22 || v == 23 || v == 25 || v == 26;
    if (longer && kVariantT[v - 1] >= lat.L[3]) continue;
    for (int o = 0; o < kWilsonOrders; ++o)
      if (o != 1 || nrhs > kVariantRT[v]) out.push_back(WilsonCfg{v, o});
  }
  return out;
}

// Inputs and results that together exceed the 256 MB Infinity Cache: storing the result past it leaves
// the inputs there (alone, 12 FP32 rhs of 16^3 x 32 108 -> 85 us, 64 BF16 rhs 352 -> 341 us); a smaller result is
// kept for the kernel that reads it next.
static int stream_out(long fstride, int nrhs, size_t elem) { return 2.0 * nrhs * fstride * elem > 256e6; }

template <class R, class SV, int WHICH, int RED, int RT>
static void launch_box(hipStream_t s, const Lattice& lat, const cplx_t<R>* U, double kappa, const SV* in, SV* out,
                       long fstride, int nrhs, int order, const double* scale, const int* active, double* part,
                       int nbs, int v) {
  const int* L = lat.L;
  int by = 1, bz = 1;
  site_box(lat, &by, &bz);
  const int ngroups = (nrhs + RT - 1) / RT;
  hipLaunchKernelGGL((k_wilson_box<R, SV, WHICH, RED, RT, kBoxNT>), dim3(nbs * ngroups), dim3(kBoxNT), 0, s, U, in, out,
                     fstride, nrhs, kappa, L[0], L[1], L[2], L[3], lat.V, lat.ntiles * kTile, kVariantT[v],
                     tm_nb3(lat, v), nbs, ngroups, order, scale, active, part, by, bz, stream_out(fstride, nrhs, sizeof(SV)),
                     static_cast<const SV*>(nullptr), static_cast<void*>(nullptr));
}

template <class R, class SV, int WHICH, int RED, int NT, bool PF>
static void launch_tmp(hipStream_t s, const Lattice& lat, const cplx_t<R>* U, double kappa, const SV* in,
                       SV* out, long fstride, int nrhs, int order, const double* scale, const int* active,
                       double* part, int nbs, int v) {
  const int* L = lat.L;
  hipLaunchKernelGGL((k_wilson_tmp<R, SV, WHICH, RED, NT, PF>), dim3(nbs * nrhs), dim3(NT), 0, s, U, in, out, fstride,
                     nrhs, kappa, L[0], L[1], L[2], L[3], lat.V, lat.ntiles * kTile, kVariantT[v], tm_nb3(lat, v), nbs,
                     order, scale, active, part);
}

template <class R, class SV, int WHICH, int RED, int NT, int RT>
static void launch_mr(hipStream_t s, const Lattice& lat, const cplx_t<R>* U, double kappa, const SV* in, SV* out,
                      long fstride, int nrhs, int order, const double* scale, const int* active, double* part,
                      int nbs) {
  const int* L = lat.L;
  const int ngroups = (nrhs + RT - 1) / RT;
  hipLaunchKernelGGL((k_wilson_mr<R, SV, WHICH, RED, NT, RT>), dim3(nbs * ngroups), dim3(NT), 0, s, U, in, out,
                     fstride, nrhs, kappa, L[0], L[1], L[2], L[3], lat.V, lat.ntiles * kTile, nbs, ngroups, order,
                     scale, active, part);
}

template <class R, class SV, int WHICH, int RED>
static void launch_split(hipStream_t s, const Lattice& lat, const cplx_t<R>* U, double kappa, const SV* in, SV* out,
                         long fstride, int nrhs, int order, const double* scale, const int* active, double* part,
                         int nbs) {
  const int* L = lat.L;
  hipLaunchKernelGGL((k_wilson_split<R, SV, WHICH, RED>), dim3(nbs * nrhs), dim3(512), 0, s, U, in, out, fstride, nrhs,
                     kappa, L[0], L[1], L[2], L[3], lat.V, lat.ntiles * kTile, nbs, order, scale, active, part);
}

template <class R, class SV, int WHICH, int RED>
static void launch_variant(int variant, hipStream_t s, const Lattice& lat, const cplx_t<R>* U, double kappa,
                           const SV* in, SV* out, long fstride, int nrhs, int order,
                           const double* scale, const int* active, double* part, int nbs) {
  switch (variant) {
    case 1: launch_one<R, SV, WHICH, RED, 128, 2>(s, lat, U, kappa, in, out, fstride, nrhs, order, scale, active, part, nbs); break;
    case 2: launch_one<R, SV, WHICH, RED, 512, 1>(s, lat, U, kappa, in, out, fstride, nrhs, order, scale, active, part, nbs); break;
    case 3: launch_one<R, SV, WHICH, RED, 256, 1>(s, lat, U, kappa, in, out, fstride, nrhs, order, scale, active, part, nbs); break;
    case 4: case 5: case 6:
      launch_tm<R, SV, WHICH, RED, 256>(s, lat, U, kappa, in, out, fstride, nrhs, order, scale, active, part, nbs, variant);
      break;
    case 12: case 13:
      launch_tmp<R, SV, WHICH, RED, 256, false>(s, lat, U, kappa, in, out, fstride, nrhs, order, scale, active, part,
                                                nbs, variant);
      break;
    case 14:
      launch_tmp<R, SV, WHICH, RED, 256, true>(s, lat, U, kappa, in, out, fstride, nrhs, order, scale, active, part,
                                               nbs, variant);
      break;
    case 15:
      launch_mr<R, SV, WHICH, RED, 256, 2>(s, lat, U, kappa, in, out, fstride, nrhs, order, scale, active, part, nbs);
      break;
    case 16:
      launch_mr<R, SV, WHICH, RED, 256, 4>(s, lat, U, kappa, in, out, fstride, nrhs, order, scale, active, part, nbs);
      break;
    case 17:
      launch_mr<R, SV, WHICH, RED, 128, 2>(s, lat, U, kappa, in, out, fstride, nrhs, order, scale, active, part, nbs);
      break;
    case 24: case 25: case 26:
      if constexpr (sizeof(R) == 4)
        launch_box<R, SV, WHICH, RED, 2>(s, lat, U, kappa, in, out, fstride, nrhs, order, scale, active, part, nbs, variant);
      break;
    case 21: case 22: case 23:
      launch_box<R, SV, WHICH, RED, 1>(s, lat, U, kappa, in, out, fstride, nrhs, order, scale, active, part, nbs, variant);
      break;
    case 20:
      launch_split<R, SV, WHICH, RED>(s, lat, U, kappa, in, out, fstride, nrhs, order, scale, active, part, nbs);
      break;
    default: launch_one<R, SV, WHICH, RED, 256, 2>(s, lat, U, kappa, in, out, fstride, nrhs, order, scale, active, part, nbs); break;
  }
}

// ---- even-odd (Schur complement) operator ---------------------------------------------
// Half fields hold the sites of one parity p(x) = (x + y + z + t) mod 2 in increasing full-site
// order; with every extent even the half index of a site is site / 2.  One thread per output
// half site; logical block = (site block, rhs), rhs fastest.

template <class C>
__device__ __forceinline__ C czero() {
  C z;
  z.x = 0;
  z.y = 0;
  return z;
}

// full coordinates of half site h of parity par
__device__ __forceinline__ void eo_coords(int h, int par, int Lx, int Ly, int Lz, int& x, int& y, int& z, int& t) {
  const int lxh = Lx >> 1;
  const int xh = h % lxh, r = h / lxh;
  y = r % Ly;
  z = (r / Ly) % Lz;
  t = r / (Ly * Lz);
  x = 2 * xh + ((par + y + z + t) & 1);
}

// acc = D_{par, 1-par} applied at half site h (input: half fields of the other parity, in storage SV)
// for RT right-hand sides.  As in k_wilson_box every hop is unrolled with its own projection, and the next hop's
// link and spinors are requested before this one's arithmetic (FP64: the link only).
template <int SF, int RT, class C, class SV>
__device__ __forceinline__ void eo_hops(const C* __restrict__ U, const SV* __restrict__ in, long fstride,
                                        const bool on[RT], int h, int par, int Lx, int Ly, int Lz, int Lt,
                                        C acc[RT][12]) {
  int x, y, z, t;
  eo_coords(h, par, Lx, Ly, Lz, x, y, z, t);
  const int sy = Lx, sz = Lx * Ly, st = Lx * Ly * Lz;
  const int site = x + sy * y + sz * z + st * t;
  const int fx = x == Lx - 1 ? 1 - Lx : 1, bx = x == 0 ? Lx - 1 : -1;
  const int fy = y == Ly - 1 ? (1 - Ly) * sy : sy, by = y == 0 ? (Ly - 1) * sy : -sy;
  const int fz = z == Lz - 1 ? (1 - Lz) * sz : sz, bz = z == 0 ? (Lz - 1) * sz : -sz;
  const int ft = t == Lt - 1 ? (1 - Lt) * st : st, bt = t == 0 ? (Lt - 1) * st : -st;
  constexpr bool PF = sizeof(C) == 8;
  auto link = [&](int s, int mu) {
    Lk<C> l;
    const C* up = U + lk_base(s, mu);
#pragma unroll
    for (int e = 0; e < 9; ++e) l.e[e] = up[e * kTile];
    return l;
  };
  auto spinor = [&](int j, int nb) {
    SpRaw<SV> r;
    const SV* pp = in + j * fstride + sp_base(nb >> 1);
#pragma unroll
    for (int c = 0; c < 12; ++c) r.e[c] = pp[c * kTile];
    return r;
  };
  Lk<C> u = link(site, 0);
  SpRaw<SV> raw[RT];
#pragma unroll
  for (int j = 0; j < RT; ++j) {
    if (PF && on[j]) raw[j] = spinor(j, site + fx);
#pragma unroll
    for (int c = 0; c < 12; ++c) acc[j][c] = czero<C>();
  }
  auto hop = [&](auto MUc, auto Sc, auto DAGc, int nb, auto LASTc, int next_site, int next_mu, int next_nb) {
    constexpr int MU = decltype(MUc)::value, S = decltype(Sc)::value;
    constexpr bool DAG = decltype(DAGc)::value, LAST = decltype(LASTc)::value;
    // opaque here, so that the loads of later hops are not gathered ahead of this one's arithmetic
    asm volatile("" : "+v"(next_site), "+v"(next_nb), "+v"(nb));
    Lk<C> un{};
    if (!LAST) un = link(next_site, next_mu);
#pragma unroll
    for (int j = 0; j < RT; ++j) {
      if (!on[j]) continue;
      C p[12], hs[6], g[6];
      if (!PF) raw[j] = spinor(j, nb);
#pragma unroll
      for (int c = 0; c < 12; ++c) p[c] = sldv(raw[j].e[c]);
      if (PF && !LAST) raw[j] = spinor(j, next_nb);
      project<MU, S>(p, hs);
      mul_half<DAG>(u.e, hs, g);
      reconstruct<MU, S>(acc[j], g);
#pragma unroll
      for (int c = 0; c < 12; ++c) asm volatile("" : "+v"(acc[j][c].x), "+v"(acc[j][c].y));
    }
    u = un;
    __builtin_amdgcn_sched_barrier(0);
  };
  constexpr std::integral_constant<int, SF> P{};
  constexpr std::integral_constant<int, -SF> N{};
  constexpr std::integral_constant<int, 0> X{};
  constexpr std::integral_constant<int, 1> Y{};
  constexpr std::integral_constant<int, 2> Z{};
  constexpr std::integral_constant<int, 3> T{};
  constexpr std::true_type yes{};
  constexpr std::false_type no{};
  hop(X, P, no, site + fx, no, site + bx, 0, site + bx);
  hop(X, N, yes, site + bx, no, site, 1, site + fy);
  hop(Y, P, no, site + fy, no, site + by, 1, site + by);
  hop(Y, N, yes, site + by, no, site, 2, site + fz);
  hop(Z, P, no, site + fz, no, site + bz, 2, site + bz);
  hop(Z, N, yes, site + bz, no, site, 3, site + ft);
  hop(T, P, no, site + ft, no, site + bt, 3, site + bt);
  hop(T, N, yes, site + bt, yes, site, 3, site);
}

// Which rhs of a group of RT the block works on; false if none.
template <int RT>
__device__ __forceinline__ bool eo_group(int rg, int nrhs, const int* __restrict__ active, bool on[RT]) {
  bool any = false;
#pragma unroll
  for (int j = 0; j < RT; ++j) {
    const int r = rg * RT + j;
    on[j] = r < nrhs && (!active || active[r]);
    any |= on[j];
  }
  return any;
}

// Both stages: bound by the latency of their loads (the links of one parity are every other site, so half
// of each line is not used).  Two rhs a thread share the link loads, each hop's loads are issued a hop ahead
// and a site block's rhs are neighbours on one XCD: 12 FP32 rhs of 16^3 x 32, stage 1 126 -> 78 us, stage 2
// 139 -> 83 us.  At three waves per SIMD (168 registers) two rhs spill in the FP32 stage 1 (3 or 19 values, 16 or
// 24 B a lane) and one value in stage 2 with a reduction.
// Stage 1: tmp (arithmetic precision) = D_{1-par0, par0} in for the rhs of the launch.
template <class R, class SV, int WHICH, int RT>
__global__ void __launch_bounds__(256, sizeof(R) == 4 ? 3 : 2)
k_eo_hop1(const typename CT<R>::type* __restrict__ U, const SV* __restrict__ in, typename CT<R>::type* __restrict__ tmp,
          long fstride, int nrhs, int ngroups, int Lx, int Ly, int Lz, int Lt, long V, long Vpad, int par,
          const int* __restrict__ active) {
  using C = typename CT<R>::type;
  const int lb = xcd_block(blockIdx.x, gridDim.x);
  const int rg = lb % ngroups, sb = lb / ngroups;
  bool on[RT];
  if (!eo_group<RT>(rg, nrhs, active, on)) return;
  const int h = sb * 256 + (int)threadIdx.x;
  C* op = tmp + rg * RT * fstride;
  if (h >= Vpad) return;
  C acc[RT][12];
  if (h >= V) {
#pragma unroll
    for (int j = 0; j < RT; ++j)
#pragma unroll
      for (int c = 0; c < 12; ++c) acc[j][c] = czero<C>();
  } else {
    constexpr int SF = (WHICH == 1) ? 1 : -1;
    eo_hops<SF, RT>(U, in + rg * RT * fstride, fstride, on, h, par, Lx, Ly, Lz, Lt, acc);
  }
#pragma unroll
  for (int j = 0; j < RT; ++j) {
    if (!on[j]) continue;
#pragma unroll
    for (int c = 0; c < 12; ++c) op[j * fstride + sp_base(h) + c * kTile] = acc[j][c];
  }
}

// Stage 2: out = scale * (in - kappa^2 D_{par, 1-par} tmp) (gamma5 on the result for WHICH 2), with
// the fused reduction of the result (RED 1: ||out||^2, RED 2: Re<in, out>) per block.
template <class R, class SV, int WHICH, int RED, int RT>
__global__ void __launch_bounds__(256, sizeof(R) == 4 ? 3 : 2)
k_eo_schur(const typename CT<R>::type* __restrict__ U, const typename CT<R>::type* __restrict__ tmp,
           const SV* __restrict__ in, SV* __restrict__ out, long fstride, int nrhs, int ngroups, double kappa2, int Lx,
           int Ly, int Lz, int Lt, long V, long Vpad, int par, int nbs, const double* __restrict__ scale,
           const int* __restrict__ active, double* __restrict__ part) {
  using C = typename CT<R>::type;
  const int lb = xcd_block(blockIdx.x, gridDim.x);
  const int rg = lb % ngroups, sb = lb / ngroups;
  bool on[RT];
  if (!eo_group<RT>(rg, nrhs, active, on)) return;
  const int h = sb * 256 + (int)threadIdx.x;
  double red[RT];
#pragma unroll
  for (int j = 0; j < RT; ++j) red[j] = 0.0;
  SV* op = out + rg * RT * fstride;
  if (h >= V && h < Vpad) {
#pragma unroll
    for (int j = 0; j < RT; ++j)
      if (on[j]) {
#pragma unroll
        for (int c = 0; c < 12; ++c) sst(op + j * fstride + sp_base(h) + c * kTile, CT<R>::make(0, 0));
      }
  }
  if (h < V) {
    constexpr int SF = (WHICH == 1) ? 1 : -1;
    C acc[RT][12];
    eo_hops<SF, RT>(U, tmp + rg * RT * fstride, fstride, on, h, par, Lx, Ly, Lz, Lt, acc);
    const R mk = (R)(-kappa2);
#pragma unroll
    for (int j = 0; j < RT; ++j) {
      if (!on[j]) continue;
      const R sc = scale ? (R)scale[rg * RT + j] : (R)1;
      const SV* ip = in + (rg * RT + j) * fstride + sp_base(h);
      R sred = 0;
#pragma unroll
      for (int c = 0; c < 12; ++c) {
        const C p = sld(ip + c * kTile);
        C r = CT<R>::make(fma(mk, acc[j][c].x, p.x) * sc, fma(mk, acc[j][c].y, p.y) * sc);
        if (WHICH == 2 && c >= 6) r = CT<R>::make(-r.x, -r.y);
        sst(op + j * fstride + sp_base(h) + c * kTile, r);
        if (RED == 1) sred = fma(r.x, r.x, fma(r.y, r.y, sred));
        if (RED == 2) sred = fma(p.x, r.x, fma(p.y, r.y, sred));
      }
      if (RED == 1) red[j] = (double)sred;
      if (RED == 2) red[j] = (double)sred * sc;
    }
  }
  if (RED != 0) {
    __shared__ double lds[256 / 64];
#pragma unroll
    for (int j = 0; j < RT; ++j) {
      if (!on[j]) continue;  // uniform over the block
      const double s = block_sum<256>(red[j], lds);
      if (threadIdx.x == 0) part[(long)(rg * RT + j) * nbs + sb] = s;
    }
  }
}

namespace {
std::mutex g_eo_mu;
std::map<hipStream_t, DBuf<char>> g_eo_scratch;
}  // namespace

void eo_reserve(hipStream_t s, size_t bytes) {
  std::lock_guard<std::mutex> lk(g_eo_mu);
  DBuf<char>& b = g_eo_scratch[s];
  if (b.n < bytes) b.alloc(bytes);
}

void eo_release(hipStream_t s) {
  std::lock_guard<std::mutex> lk(g_eo_mu);
  g_eo_scratch.erase(s);
}

static void* eo_buffer(hipStream_t s, size_t bytes) {
  eo_reserve(s, bytes);
  std::lock_guard<std::mutex> lk(g_eo_mu);
  return g_eo_scratch[s].get();
}

template <class R, class SV, int RT>
static void launch_eo(hipStream_t s, const Lattice& lat, const cplx_t<R>* U, double kappa, int which, const SV* in,
                      cplx_t<R>* tmp, SV* out, long fstride, int nrhs, int red, const double* scale, const int* active,
                      double* part, int nbs) {
  const int* L = lat.L;
  const long Vpad = lat.ntiles * kTile;
  const int ngroups = (nrhs + RT - 1) / RT;
  const dim3 grid((unsigned)((long)nbs * ngroups)), block(256);
  // stage 1: odd intermediate D_oe in (par 1 output); stage 2: even result
#define DL_EO1(WH) hipLaunchKernelGGL((k_eo_hop1<R, SV, WH, RT>), grid, block, 0, s, U, in, tmp, fstride, nrhs, \
                                      ngroups, L[0], L[1], L[2], L[3], lat.V, Vpad, 1, active)
#define DL_EO2(WH, RD) hipLaunchKernelGGL((k_eo_schur<R, SV, WH, RD, RT>), grid, block, 0, s, U, tmp, in, out, \
                                          fstride, nrhs, ngroups, kappa * kappa, L[0], L[1], L[2], L[3], lat.V, Vpad, \
                                          0, nbs, scale, active, part)
  if (which == 1) DL_EO1(1); else DL_EO1(0);
  if (which == 0) { if (red == 0) DL_EO2(0, 0); else if (red == 1) DL_EO2(0, 1); else DL_EO2(0, 2); }
  else if (which == 1) { if (red == 0) DL_EO2(1, 0); else if (red == 1) DL_EO2(1, 1); else DL_EO2(1, 2); }
  else { if (red == 0) DL_EO2(2, 0); else if (red == 1) DL_EO2(2, 1); else DL_EO2(2, 2); }
#undef DL_EO1
#undef DL_EO2
}

template <class R, class SV>
static int wilson_eo(hipStream_t s, const Lattice& lat, const cplx_t<R>* U, double kappa, int which, const SV* in,
                     SV* out, long fstride, int nrhs, int red, const double* scale, const int* active, double* part) {
  using C = cplx_t<R>;
  const int nbs = (int)((lat.V + 255) / 256);
  if (red && nbs > kMaxPartials) fail(DL_E_INVALID, "lattice too large for fused reduction");
  C* tmp = static_cast<C*>(eo_buffer(s, (size_t)nrhs * fstride * sizeof(C)));
  // two rhs a thread share the links; only where that still leaves two blocks for each of the 256 CUs
  if constexpr (sizeof(R) == 4) {
    if (nrhs > 1 && (long)nbs * ((nrhs + 1) / 2) >= 512) {
      launch_eo<R, SV, 2>(s, lat, U, kappa, which, in, tmp, out, fstride, nrhs, red, scale, active, part, nbs);
      DL_HIP(hipGetLastError());
      return red ? nbs : 0;
    }
  }
  launch_eo<R, SV, 1>(s, lat, U, kappa, which, in, tmp, out, fstride, nrhs, red, scale, active, part, nbs);
  DL_HIP(hipGetLastError());
  return red ? nbs : 0;
}

__global__ void k_eo_split(const double2* __restrict__ in, double2* __restrict__ half, long nc_full, long nc_half,
                           long Vh, int par, int Lx, int Ly, int Lz) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long f = blockIdx.y;
  if (i >= Vh * kSpin) return;
  const int h = (int)(i / kSpin), c = (int)(i % kSpin);
  int x, y, z, t;
  eo_coords(h, par, Lx, Ly, Lz, x, y, z, t);
  const int site = x + Lx * (y + Ly * (z + Lz * t));
  half[f * nc_half + sp_base(h) + c * kTile] = in[f * nc_full + sp_base(site) + c * kTile];
}

__global__ void k_eo_merge(const double2* __restrict__ half, double2* __restrict__ out, long nc_full, long nc_half,
                           long Vh, int par, int Lx, int Ly, int Lz) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long f = blockIdx.y;
  if (i >= Vh * kSpin) return;
  const int h = (int)(i / kSpin), c = (int)(i % kSpin);
  int x, y, z, t;
  eo_coords(h, par, Lx, Ly, Lz, x, y, z, t);
  const int site = x + Lx * (y + Ly * (z + Lz * t));
  out[f * nc_full + sp_base(site) + c * kTile] = half[f * nc_half + sp_base(h) + c * kTile];
}

// out = fac * D_{par, 1-par} in + add (FP64, one field)
__global__ void __launch_bounds__(256)
k_eo_hop_f64(const double2* __restrict__ U, const double2* __restrict__ in, const double2* __restrict__ add,
             double2* __restrict__ out, double fac, int Lx, int Ly, int Lz, int Lt, long V, long Vpad, int par) {
  const int h = (int)blockIdx.x * 256 + (int)threadIdx.x;
  if (h >= V && h < Vpad) {
#pragma unroll
    for (int c = 0; c < 12; ++c) out[sp_base(h) + c * kTile] = make_double2(0.0, 0.0);
  }
  if (h >= V) return;
  double2 accs[1][12];
  const bool on[1] = {true};
  eo_hops<-1, 1>(U, in, 0, on, h, par, Lx, Ly, Lz, Lt, accs);
  double2* acc = accs[0];
#pragma unroll
  for (int c = 0; c < 12; ++c) {
    const double2 a = add ? add[sp_base(h) + c * kTile] : make_double2(0.0, 0.0);
    out[sp_base(h) + c * kTile] = make_double2(fma(fac, acc[c].x, a.x), fma(fac, acc[c].y, a.y));
  }
}

void eo_split(hipStream_t s, const Lattice& full, const double2* in, double2* half, int par, int nfield) {
  if (nfield <= 0) return;
  const Lattice hl = make_lattice_eo(full.L);
  const long n = hl.V * kSpin;
  hipLaunchKernelGGL(k_eo_split, dim3((unsigned)((n + 255) / 256), nfield), dim3(256), 0, s, in, half, full.nc,
                     hl.nc, hl.V, par, full.L[0], full.L[1], full.L[2]);
  DL_HIP(hipGetLastError());
}

void eo_merge(hipStream_t s, const Lattice& full, const double2* half, double2* out, int par, int nfield) {
  if (nfield <= 0) return;
  const Lattice hl = make_lattice_eo(full.L);
  const long n = hl.V * kSpin;
  hipLaunchKernelGGL(k_eo_merge, dim3((unsigned)((n + 255) / 256), nfield), dim3(256), 0, s, half, out, full.nc,
                     hl.nc, hl.V, par, full.L[0], full.L[1], full.L[2]);
  DL_HIP(hipGetLastError());
}

void eo_hop_f64(hipStream_t s, const Lattice& lat, const double2* U, double fac, int par, const double2* in,
                const double2* add, double2* out) {
  const int* L = lat.L;
  hipLaunchKernelGGL(k_eo_hop_f64, dim3((unsigned)((lat.V + 255) / 256)), dim3(256), 0, s, U, in, add, out, fac, L[0],
                     L[1], L[2], L[3], lat.V, lat.ntiles * kTile, par);
  DL_HIP(hipGetLastError());
}

// The residual's shape: the tuned shape of the FP64 stencil if it is one of the two marching forms, which have a
// residual epilogue, else (small grids, where other forms win by the number of their blocks) the box or, without
// one, k_wilson_tm with the shortest chunks that the partials hold.  Fixed at chunks of 16, the box was slower than
// k_wilson_tm where few blocks are launched (8^4, 4 rhs 59 against 54 us, 22^4, 12 rhs 685 against 533) and the
// reverse on large batches (16^3 x 32, 64 rhs 1122 against 1283); by this rule 33, 531 and 1128.
int wilson_residual_shape(const Lattice& lat, const WilsonCfg& fp64) {
  int v = wilson_shape(lat, fp64.variant % kWilsonVariants, true);
  if (v >= kFirstBox || (v >= 4 && v <= 6)) return v;
  for (int i = 0; i < 3; ++i) {
    v = wilson_shape(lat, kFirstBox + i, true);
    if (wilson_nbs(lat, WilsonCfg{v, 0}) <= kMaxPartials) break;
  }
  return v;
}

int wilson_residual_f64(hipStream_t s, const Lattice& lat, const double2* U, double kappa, const double2* x,
                        const double2* b, double2* r, long fstride, int nrhs, const int* active, double* part,
                        const WilsonCfg& fp64, void* lo, int lo_prec) {
  if (lat.eo) fail(DL_E_INVALID, "the fused residual serves whole-lattice operators");
  if ((lo == nullptr) == (r == nullptr)) fail(DL_E_INVALID, "the fused residual goes to r or to lo");
  const int v = wilson_residual_shape(lat, fp64);  // in hardware block order
  const int nbs = tm_nb3(lat, v) * tm_chunks(lat, v);
  if (nbs > kMaxPartials) fail(DL_E_INVALID, "lattice too large for fused reduction");
  if ((long)nbs * nrhs > 2147483647L) fail(DL_E_INVALID, "grid too large");
  const int* L = lat.L;
  int by = 1, bz = 1;
  if (v >= kFirstBox) site_box(lat, &by, &bz);
#define DL_RES(LOP)                                                                                                 \
  if (v >= kFirstBox)                                                                                               \
    hipLaunchKernelGGL((k_wilson_box<double, double2, 0, 1, 1, kBoxNT, true, LOP>), dim3(nbs * nrhs), dim3(kBoxNT),  \
                       0, s, U, x, r, fstride, nrhs, kappa, L[0], L[1], L[2], L[3], lat.V, lat.ntiles * kTile,       \
                       kVariantT[v], tm_nb3(lat, v), nbs, nrhs, 2, static_cast<const double*>(nullptr), active,      \
                       part, by, bz, stream_out(fstride, nrhs, sizeof(double2)), b, lo);                             \
  else                                                                                                              \
    hipLaunchKernelGGL((k_wilson_tm<double, double2, 0, 1, 256, true, LOP>), dim3(nbs * nrhs), dim3(256), 0, s, U,   \
                       x, r, fstride, nrhs, kappa, L[0], L[1], L[2], L[3], lat.V, lat.ntiles * kTile, kVariantT[v],  \
                       tm_nb3(lat, v), nbs, 2, static_cast<const double*>(nullptr), active, part, b, lo)
  if (!lo) { DL_RES(0); }
  else if (lo_prec == DL_FP32) { DL_RES(1); }
  else if (lo_prec == DL_BF16) { DL_RES(2); }
  else fail(DL_E_INVALID, "lo_prec must be DL_FP32 or DL_BF16");
#undef DL_RES
  DL_HIP(hipGetLastError());
  return nbs;
}

int wilson_nbs(const Lattice& lat, const WilsonCfg& cfg) {
  if (lat.eo) return (int)((lat.V + 255) / 256);
  const int v = wilson_shape(lat, cfg.variant % kWilsonVariants, false);  // (FP64 runs the same blocks of sites)
  if (kVariantT[v] > 0) return tm_nb3(lat, v) * tm_chunks(lat, v);
  const int nt = kVariantNT[v];
  return (int)((lat.V + nt - 1) / nt);
}

long wilson_grid(const Lattice& lat, const WilsonCfg& cfg, bool fp64, int nrhs) {
  const int rt = kVariantRT[wilson_shape(lat, cfg.variant % kWilsonVariants, fp64)];
  return (long)wilson_nbs(lat, cfg) * ((nrhs + rt - 1) / rt);
}

int wilson_max_nbs(const Lattice& lat) {
  int m = 0;
  for (int v = 0; v < kWilsonVariants; ++v) {
    const int nbs = wilson_nbs(lat, WilsonCfg{v, 0});
    if (nbs <= kMaxPartials) m = std::max(m, nbs);
  }
  return m;
}

int wilson_red_stride(const Lattice& lat, const WilsonCfg& lo, const WilsonCfg& fp64) {
  return std::max(wilson_nbs(lat, lo), wilson_nbs(lat, WilsonCfg{wilson_residual_shape(lat, fp64), 0}));
}

template <class R, class SV>
int wilson_batched(hipStream_t s, const Lattice& lat, const cplx_t<R>* U, double kappa, int which,
                   const SV* in, SV* out, long fstride, int nrhs, int red, const double* scale,
                   const int* active, double* part, WilsonCfg cfg) {
  if (lat.eo) return wilson_eo<R, SV>(s, lat, U, kappa, which, in, out, fstride, nrhs, red, scale, active, part);
  const int v = wilson_shape(lat, cfg.variant % kWilsonVariants, sizeof(R) == 8);
  const int nbs = wilson_nbs(lat, cfg);
  if (red && nbs > kMaxPartials) fail(DL_E_INVALID, "lattice too large for fused reduction");
  if (wilson_grid(lat, cfg, sizeof(R) == 8, nrhs) > 2147483647L) fail(DL_E_INVALID, "grid too large");
  const int o = cfg.order;
#define DL_W(WH, RD) launch_variant<R, SV, WH, RD>(v, s, lat, U, kappa, in, out, fstride, nrhs, o, scale, active, part, nbs)
  if (which == 0) { if (red == 0) DL_W(0, 0); else if (red == 1) DL_W(0, 1); else DL_W(0, 2); }
  else if (which == 1) { if (red == 0) DL_W(1, 0); else if (red == 1) DL_W(1, 1); else DL_W(1, 2); }
  else { if (red == 0) DL_W(2, 0); else if (red == 1) DL_W(2, 1); else DL_W(2, 2); }
#undef DL_W
  DL_HIP(hipGetLastError());
  return red ? nbs : 0;
}

template int wilson_batched<double, double2>(hipStream_t, const Lattice&, const double2*, double, int, const double2*,
                                             double2*, long, int, int, const double*, const int*, double*, WilsonCfg);
template int wilson_batched<float, float2>(hipStream_t, const Lattice&, const float2*, double, int, const float2*,
                                           float2*, long, int, int, const double*, const int*, double*, WilsonCfg);
template int wilson_batched<float, bf2>(hipStream_t, const Lattice&, const float2*, double, int, const bf2*, bf2*,
                                        long, int, int, const double*, const int*, double*, WilsonCfg);

int wilson_f64(hipStream_t s, const Lattice& lat, const double2* U, double kappa, int which,
               const double2* in, double2* out, int red, double* part, WilsonCfg cfg) {
  return wilson_batched<double, double2>(s, lat, U, kappa, which, in, out, lat.nc, 1, red, nullptr, nullptr, part, cfg);
}

__global__ void k_gamma5_f64(const double2* __restrict__ in, double2* __restrict__ out, long nc) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nc) return;
  const int c = (int)((i >> 6) % kSpin);
  const double2 v = in[i];
  out[i] = c >= 6 ? make_double2(-v.x, -v.y) : v;
}

void gamma5_f64(hipStream_t s, const Lattice& lat, const double2* in, double2* out) {
  const long n = lat.nc;
  hipLaunchKernelGGL(k_gamma5_f64, dim3((n + 255) / 256), dim3(256), 0, s, in, out, n);
  DL_HIP(hipGetLastError());
}

}  // namespace dl
