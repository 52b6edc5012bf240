// Gauge-covariant parallel-transport convolution network (learned initial guess), FP32.
//
// Activations are colour triplets per site and channel in the tiled layout
//     elem(site, ch, col) = ((site / 64) * (C * 3) + ch * 3 + col) * 64 + site % 64
// (for C = 4 this is the spinor layout with spin as channel).  A layer computes
//     out[o](x) = sum_h sum_i W_h[o][i] (T_h in[i])(x)
// over the nine hops h = 0, +x, -x, +y, -y, +z, -z, +t, -t, with T_0 = 1,
// (T_{+mu} a)(x) = U_mu(x) a(x + mu) and (T_{-mu} a)(x) = U_mu(x - mu)^dag a(x - mu),
// optionally followed by f(z) = z / sqrt(1 + |z|^2) per site and channel (|z| the
// gauge-invariant colour norm).  Widths 4 -> 16 -> 16 -> 4; the input is scaled by
// 1/s with s the root-mean-square site norm of b over its nonzero sites and the output
// by s, so net(c b) = c net(b) and point and extended sources both enter at unit scale.
//
// Backward pass: the adjoint of T_h is T_{-h} and channel mixing commutes with the
// transport, so the data gradient is the forward kernel with W'_{-h} = W_h^H.  The
// weight gradient G_W[h][o][i] = sum_x sum_c G_out[o](x)_c conj((T_h in[i])(x)_c)
// is accumulated per 64-site chunk from LDS in FP64 (on the matrix cores) and reduced in a fixed order.
#include "ptc.hpp"
#include "small.hpp"
#include "tsk.hpp"
#include "cplx.hpp"

#include <algorithm>
#include <cmath>
#include <vector>

namespace dl {

namespace {

__device__ __forceinline__ long act_idx(int site, int C, int ch, int col) {
  return ((long)(site >> 6) * (C * 3) + ch * 3 + col) * kTile + (site & 63);
}
__device__ __forceinline__ long lnk_idx(int site, int mu, int e) {
  return ((long)(site >> 6) * kLinkC + mu * 9 + e) * kTile + (site & 63);
}

// Neighbour of `site` along hop h (1..8: +x, -x, +y, -y, +z, -z, +t, -t), the hop's direction
// and whether it is forward.  The link of a forward hop sits at `site`, of a backward hop at nb.
__device__ __forceinline__ void hop_geom(int h, int site, int Lx, int Ly, int Lz, int Lt, int& nb, int& mu,
                                         bool& fwd) {
  mu = (h - 1) >> 1;
  fwd = ((h - 1) & 1) == 0;
  const int st = mu == 0 ? 1 : mu == 1 ? Lx : mu == 2 ? Lx * Ly : Lx * Ly * Lz;
  const int L = mu == 0 ? Lx : mu == 1 ? Ly : mu == 2 ? Lz : Lt;
  const int c = (site / st) % L;
  if (fwd) nb = c == L - 1 ? site - (L - 1) * st : site + st;
  else nb = c == 0 ? site + (L - 1) * st : site - st;
}

// tr = U a (forward hop) or U^dag a (backward hop)
__device__ __forceinline__ void transport3(const float2 u[9], bool fwd, const float2 a[3], float2 tr[3]) {
  if (fwd) {
#pragma unroll
    for (int r = 0; r < 3; ++r) tr[r] = c_fma(u[r * 3 + 2], a[2], c_fma(u[r * 3 + 1], a[1], c_mul(u[r * 3], a[0])));
  } else {
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      float2 v = c_fmac(u[0 * 3 + r], a[0], make_float2(0.f, 0.f));
      v = c_fmac(u[1 * 3 + r], a[1], v);
      tr[r] = c_fmac(u[2 * 3 + r], a[2], v);
    }
  }
}

// One network layer over gridDim.x / nblk fields: thread = site.
// ACT 1: out = f(z), z saved to zsave if given;
// 2 (backward): out = the gradient G_z behind the non-linearity, from the sum G_f and z = zsave,
// G_z = g G_f + 2 g' Re<G_f, z> z with g(s) = (1 + s)^-1/2, s = |z|^2 (a pass over G of its own took
// 348 us for 16 channels of 8 fields of 16^3 x 32).
// The weights are the same for every lane, so they come through the scalar cache and are SGPR operands.
// Bound by the vector FMAs: 8 fields of 16^3 x 32 16 -> 16 1.16 -> 0.99 ms (0.96 of it issue), 4 -> 16 0.35 -> 0.33
// (0.27); the weights in LDS and each channel's loads waited for took the difference.
template <int CIN, int COUT, int ACT>
__global__ void __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(CIN == 4 ? 2 : 3, CIN == 4 ? 2 : 3)))
k_ptc_layer(const float2* __restrict__ U, const float2* __restrict__ in, float2* __restrict__ out,
            float2* __restrict__ zsave, const float2* __restrict__ W, int Lx, int Ly, int Lz, int Lt, int V,
            int Vpad, int nblk, long in_stride, long out_stride) {
  const int lb = xcd_block(blockIdx.x, gridDim.x);
  const int item = lb / nblk;
  in += item * in_stride;
  out += item * out_stride;
  if (zsave) zsave += item * out_stride;
  const int site = (lb - item * nblk) * blockDim.x + threadIdx.x;
  if (site >= Vpad) return;
  if (site >= V) {  // padding sites stay zero
    for (int o = 0; o < COUT; ++o)
      for (int c = 0; c < 3; ++c) {
        out[act_idx(site, COUT, o, c)] = make_float2(0.f, 0.f);
        if (ACT == 1 && zsave) zsave[act_idx(site, COUT, o, c)] = make_float2(0.f, 0.f);
      }
    return;
  }
  // CB channels at a time: transported, then the next CB channels' loads (and the next hop's link) are
  // issued and stay in flight while these are mixed into the COUT sums
  constexpr int CB = CIN == 4 ? 4 : 2, NB = CIN / CB;
  float2 acc[COUT][3];
#pragma unroll
  for (int o = 0; o < COUT; ++o)
#pragma unroll
    for (int c = 0; c < 3; ++c) acc[o][c] = make_float2(0.f, 0.f);
  int nb = site;
  float2 u[9], a[CB][3];
  auto load = [&](int ch0) {
#pragma unroll
    for (int i = 0; i < CB; ++i)
#pragma unroll
      for (int c = 0; c < 3; ++c) a[i][c] = in[act_idx(nb, CIN, ch0 + i, c)];
  };
  load(0);
#pragma unroll
  for (int e = 0; e < 9; ++e) u[e] = make_float2(0.f, 0.f);
#pragma unroll 1
  for (int st = 0; st < 9 * NB; ++st) {
    const int h = st / NB, k = st % NB;
    float2 tr[CB][3];
    if (h == 0) {
#pragma unroll
      for (int i = 0; i < CB; ++i)
#pragma unroll
        for (int c = 0; c < 3; ++c) tr[i][c] = a[i][c];
    } else {
#pragma unroll
      for (int i = 0; i < CB; ++i) transport3(u, (h & 1) != 0, a[i], tr[i]);
    }
    if (k + 1 < NB) {
      load((k + 1) * CB);
    } else if (h < 8) {
      int mu;
      bool f;
      hop_geom(h + 1, site, Lx, Ly, Lz, Lt, nb, mu, f);
      const int ls = f ? site : nb;
#pragma unroll
      for (int e = 0; e < 9; ++e) u[e] = U[lnk_idx(ls, mu, e)];
      load(0);
    }
    __builtin_amdgcn_sched_barrier(0);
    const float2* wh = W + h * COUT * CIN + k * CB;
#pragma unroll
    for (int i = 0; i < CB; ++i)
#pragma unroll
      for (int o = 0; o < COUT; ++o) {
        const float2 w = wh[o * CIN + i];
#pragma unroll
        for (int c = 0; c < 3; ++c) acc[o][c] = c_fma(w, tr[i][c], acc[o][c]);
      }
  }
#pragma unroll
  for (int o = 0; o < COUT; ++o) {
    if (ACT == 2) {
      float2 z[3];
      float n2 = 0.f, re = 0.f;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        z[c] = zsave[act_idx(site, COUT, o, c)];
        n2 += z[c].x * z[c].x + z[c].y * z[c].y;
        re += acc[o][c].x * z[c].x + acc[o][c].y * z[c].y;
      }
      const float gf = 1.f / sqrtf(1.f + n2);
      const float dgf = -0.5f * gf * gf * gf;
#pragma unroll
      for (int c = 0; c < 3; ++c)
        out[act_idx(site, COUT, o, c)] = c_axpy(2.f * dgf * re, z[c], c_scale(acc[o][c], gf));
    } else {
      float n2 = 0.f;
#pragma unroll
      for (int c = 0; c < 3; ++c) n2 += acc[o][c].x * acc[o][c].x + acc[o][c].y * acc[o][c].y;
      const float g = 1.f / sqrtf(1.f + n2);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        if (zsave) zsave[act_idx(site, COUT, o, c)] = acc[o][c];
        out[act_idx(site, COUT, o, c)] = c_scale(acc[o][c], g);
      }
    }
  }
}

// The 16 -> 4 layer: two waves per tile of 64 sites.  Each transports eight of the input channels, they
// meet in LDS, and each mixes them into two of the outputs (out = out_scale[item] * z; out_scale may be
// NULL), in the same order as one thread per site would.  Bound by what misses the L2: a site is read nine
// times, and with one site per thread an XCD's 32 CUs held 32 * 1024 sites of 384 B, three times its 4 MB,
// so that 90 % of the reads went past it.  Two waves per tile keep as many waves on fewer
// sites: 16 fields of 16^3 x 32 1158 -> 870 to 917 us, of which vector issue is 715 and where 44M of 71M requests
// still miss (one thread per site with its loads ahead 1018, one or two such waves per SIMD 1240 and 1018;
// four or five blocks a CU 1000 and 1040).
__global__ void __launch_bounds__(128)
k_ptc_layer16_4(const float2* __restrict__ U, const float2* __restrict__ in, float2* __restrict__ out,
                const float2* __restrict__ W, int Lx, int Ly, int Lz, int Lt, int V, int ntiles, long in_stride,
                long out_stride, const double* __restrict__ out_scale) {
  __shared__ float2 tl[48][64];  // [3 channel + colour][site]
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lb = xcd_block(blockIdx.x, gridDim.x);
  const int item = lb / ntiles, tile = lb - item * ntiles;
  in += item * in_stride;
  out += item * out_stride;
  const int site = min(tile * 64 + lane, V - 1);  // a padding site repeats the last one
  float2 acc[2][3];
#pragma unroll
  for (int o = 0; o < 2; ++o)
#pragma unroll
    for (int c = 0; c < 3; ++c) acc[o][c] = make_float2(0.f, 0.f);
  float2 u[9], a[8][3];
  auto load = [&](int h) {
    int nb = site;
    if (h > 0) {
      int mu;
      bool f;
      hop_geom(h, site, Lx, Ly, Lz, Lt, nb, mu, f);
      const int ls = f ? site : nb;
#pragma unroll
      for (int e = 0; e < 9; ++e) u[e] = U[lnk_idx(ls, mu, e)];
    }
    const float2* ap = in + act_idx(nb, 16, 8 * w, 0);
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int c = 0; c < 3; ++c) a[i][c] = ap[(3 * i + c) * kTile];
  };
#pragma unroll
  for (int e = 0; e < 9; ++e) u[e] = make_float2(0.f, 0.f);
  load(0);
#pragma unroll 1
  for (int h = 0; h < 9; ++h) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      float2 tr[3];
      if (h == 0) {
#pragma unroll
        for (int c = 0; c < 3; ++c) tr[c] = a[i][c];
      } else {
        transport3(u, (h & 1) != 0, a[i], tr);
      }
#pragma unroll
      for (int c = 0; c < 3; ++c) tl[3 * (8 * w + i) + c][lane] = tr[c];
    }
    if (h < 8) load(h + 1);  // in flight during the mixing
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
    const float2* wh = W + h * 64 + 32 * w;
#pragma unroll 8
    for (int i = 0; i < 16; ++i)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const float2 t = tl[3 * i + c][lane];
#pragma unroll
        for (int o = 0; o < 2; ++o) acc[o][c] = c_fma(wh[o * 16 + i], t, acc[o][c]);
      }
    __syncthreads();
  }
  const float sc = out_scale ? (float)out_scale[item] : 1.f;
  const bool ok = tile * 64 + lane < V;
#pragma unroll
  for (int o = 0; o < 2; ++o)
#pragma unroll
    for (int c = 0; c < 3; ++c)
      out[act_idx(tile * 64 + lane, 4, 2 * w + o, c)] = ok ? c_scale(acc[o][c], sc) : make_float2(0.f, 0.f);
}

// ---- 16 -> 16 layer with BF16 channel mixing on the matrix cores (inference) ------------------
//
// Two waves per tile of 64 sites.  For each hop each wave transports 8 of the input channels (FP32,
// one thread per site), rounds them to BF16 and stages them in LDS; the channel mixing is then
// the real form of a complex product: with K = (channel i, re/im) interleaved (32 per hop) and
// rows m < 16 the real parts, m >= 16 the imaginary parts of the 16 output channels,
//     A[o][2i] = Re W, A[o][2i+1] = -Im W, A[16+o][2i] = Im W, A[16+o][2i+1] = Re W,
// and out[m][(site, colour)] += sum_k A[m][k] T[k][(site, colour)] on v_mfma_f32_32x32x16_bf16:
// six 32-column tiles (3 colours x 2 halves of the tile's sites, one half a wave) and two K-steps per hop, FP32
// accumulation over all nine hops.  Lane l supplies row / column l % 32 and K-slice 8 * (l / 32)
// of both operands; the result register j of lane l is row 8 (j / 4) + 4 (l / 32) + j % 4, so a
// lane holds the real and imaginary parts of 8 output channels for the 3 colours of two sites,
// which is all the per-channel non-linearity needs.
// Bound by the latency of the loads and the vector work of the transport (16 fields of 16^3 x 32: 0.48 ms of
// issue; the products 0.05).  Two waves share a tile and the next hop's loads are in flight during the products:
// 1509 -> 917 to 953 us, 29M of 85M requests missing the L2.  One wave per tile with its loads ahead took 1041,
// with twice the misses.
typedef __bf16 bf16x8_n __attribute__((ext_vector_type(8)));
typedef float f32x16_n __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4_n __attribute__((ext_vector_type(4)));
typedef float f32x2_n __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_n __attribute__((ext_vector_type(2)));

// BF16 entries per (colour, site) row of the LDS stage; its four 16 B parts are swapped by bits 2-3 of the
// site against bank conflicts
constexpr int kMixRow = 32;

__device__ __forceinline__ unsigned pack_bf16x2(float a, float b) {
  const f32x2_n f = {a, b};
  return __builtin_bit_cast(unsigned, __builtin_convertvector(f, bf16x2_n));
}

// A fragments of a 16 -> 16 layer: frag[(h * 2 + ks) * 64 + lane] = 8 BF16 entries
// A[m = lane % 32][k = 16 ks + 8 (lane / 32) + j], j = 0..7.
__global__ void k_ptc_wfrag16(const float2* __restrict__ W, u32x4_n* __restrict__ frag) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= 9 * 2 * 64) return;
  const int lane = t % 64, hk = t / 64, h = hk / 2, ks = hk % 2;
  const int m = lane % 32, kb = 16 * ks + 8 * (lane / 32);
  float v[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int kk = kb + j, i = kk / 2, p = kk % 2;
    const int o = m % 16;
    const float2 w = W[(h * 16 + o) * 16 + i];
    v[j] = m < 16 ? (p == 0 ? w.x : -w.y) : (p == 0 ? w.y : w.x);
  }
  u32x4_n r;
#pragma unroll
  for (int q = 0; q < 4; ++q) r[q] = pack_bf16x2(v[2 * q], v[2 * q + 1]);
  frag[t] = r;
}

__global__ void __launch_bounds__(128)
k_ptc_layer16_mfma(const float2* __restrict__ U, const float2* __restrict__ in, float2* __restrict__ out,
                   const u32x4_n* __restrict__ frag, int Lx, int Ly, int Lz, int Lt, int V, int ntiles,
                   long in_stride, long out_stride) {
  __shared__ __align__(16) unsigned short stage[2][3 * 64 * kMixRow];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lb = xcd_block(blockIdx.x, gridDim.x);
  const int item = lb / ntiles, tile = lb - item * ntiles;
  in += item * in_stride;
  out += item * out_stride;
  const int site = min(tile * 64 + lane, V - 1);  // a padding site repeats the last one (columns do not mix)
  f32x16_n acc[3];
#pragma unroll
  for (int q = 0; q < 3; ++q)
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[q][j] = 0.f;
  const int g = lane >> 5, col = lane & 31;
  float2 u[9], a[8][3];
  auto load = [&](int h) {
    int nb = site;
    if (h > 0) {
      int mu;
      bool f;
      hop_geom(h, site, Lx, Ly, Lz, Lt, nb, mu, f);
      const int ls = f ? site : nb;
#pragma unroll
      for (int e = 0; e < 9; ++e) u[e] = U[lnk_idx(ls, mu, e)];
    }
    const float2* ap = in + act_idx(nb, 16, 8 * w, 0);
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int c = 0; c < 3; ++c) a[i][c] = ap[(3 * i + c) * kTile];
  };
#pragma unroll
  for (int e = 0; e < 9; ++e) u[e] = make_float2(0.f, 0.f);
  load(0);
#pragma unroll 1
  for (int h = 0; h < 9; ++h) {
    unsigned short* st = stage[h & 1];
    const u32x4_n af[2] = {frag[h * 128 + lane], frag[h * 128 + 64 + lane]};
    unsigned pk[3][8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      float2 tr[3];
      if (h == 0) {
#pragma unroll
        for (int c = 0; c < 3; ++c) tr[c] = a[i][c];
      } else {
        transport3(u, (h & 1) != 0, a[i], tr);
      }
#pragma unroll
      for (int c = 0; c < 3; ++c) pk[c][i] = pack_bf16x2(tr[c].x, tr[c].y);
    }
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int q = 0; q < 2; ++q)
        *reinterpret_cast<u32x4_n*>(st + (c * 64 + lane) * kMixRow + 8 * ((2 * w + q) ^ ((lane >> 2) & 3))) =
            u32x4_n{pk[c][4 * q], pk[c][4 * q + 1], pk[c][4 * q + 2], pk[c][4 * q + 3]};
    if (h < 8) load(h + 1);  // in flight during the products
    __syncthreads();         // one per hop: the other half of `stage` was read before the last one
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const u32x4_n bf = *reinterpret_cast<const u32x4_n*>(st + (c * 64 + w * 32 + col) * kMixRow +
                                                             8 * ((2 * ks + g) ^ ((col >> 2) & 3)));
        acc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_n, af[ks]),
                                                         __builtin_bit_cast(bf16x8_n, bf), acc[c], 0, 0, 0);
      }
  }
  // epilogue: lane holds rows 8q + 4g + r (q, r < 4) of the wave's three tiles: channel o = 8 (q % 2) + 4g + r,
  // real part for q < 2, imaginary part (row 16 + o) for q >= 2
  const int s2 = tile * 64 + w * 32 + col;
  const bool ok = s2 < V;
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int o = 8 * q + 4 * g + r;
      float2 z[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) z[c] = make_float2(acc[c][4 * q + r], acc[c][4 * (q + 2) + r]);
      float n2 = 0.f;
#pragma unroll
      for (int c = 0; c < 3; ++c) n2 += z[c].x * z[c].x + z[c].y * z[c].y;
      const float gsc = 1.f / sqrtf(1.f + n2);
#pragma unroll
      for (int c = 0; c < 3; ++c) out[act_idx(s2, 16, o, c)] = ok ? c_scale(z[c], gsc) : make_float2(0.f, 0.f);
    }
}

// Adjoint weights of a [9][cout][cin] layer: Wt[rev(h)][i][o] = conj(W[h][o][i]).
__global__ void k_ptc_adjoint_weights(const float2* __restrict__ W, float2* __restrict__ Wt, int cin, int cout) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= 9 * cout * cin) return;
  const int h = e / (cout * cin), o = (e / cin) % cout, i = e % cin;
  const int rh = h == 0 ? 0 : (((h - 1) & 1) == 0 ? h + 1 : h - 1);
  const float2 w = W[e];
  Wt[((long)rh * cin + i) * cout + o] = make_float2(w.x, -w.y);
}

// Weight-gradient partials: block (chunk group, hop h, item), four waves.  The block walks 64-site
// chunks blockIdx.x, blockIdx.x + gridDim.x, ... staging the transported inputs a and the output
// gradients g of a chunk in LDS (one wave per channel, lane = site: coalesced loads, the link read
// once per wave), and contracts them over (site, colour) on the FP64 matrix cores: rows are the real
// and imaginary parts of g's channels, columns those of a's, so a lane's one LDS read per operand gives
// a real and an imaginary row (column), and each wave takes a quarter of the 192 products.  Then
// G = sum g conj(a) is Re = <g_re, a_re> + <g_im, a_im>, Im = <g_im, a_re> - <g_re, a_im>.  Products of
// two FP32 numbers are exact in FP64 and summed in FP64.  Bound by the FP64 matrix rate
// and the vector instructions around it, which do not overlap with FP64 matrix products (16 -> 16, 8 fields of
// 16^3 x 32: 0.74 + 0.29 ms); with vector FMAs, a conversion per operand and gathered loads it took 3.69 ms,
// now 1.31 (16 -> 4: 2.05 -> 0.80, 4 -> 16: 1.67 -> 0.70).  The nine hops of a chunk range are neighbours on one
// XCD, where they read the same g and a through its L2, and the next chunk's loads are in flight during
// the products (1.82 ms without these two).
// part layout: part[((item * 9 + h) * COUT * CIN + p) * 2 * nblk + {blk (re), nblk + blk (im)}]
typedef double f64x4_n __attribute__((ext_vector_type(4)));

template <int CIN, int COUT>
__global__ void __launch_bounds__(256, 3)
k_ptc_wgrad(const float2* __restrict__ U, const float2* __restrict__ in, const float2* __restrict__ G, int Lx,
            int Ly, int Lz, int Lt, int V, int nchunks, int nblk, long in_stride, long g_stride,
            double* __restrict__ part) {
  constexpr int RI = CIN + 1, RO = COUT + 1;        // LDS rows, padded
  constexpr int CA = CIN / 4, CG = COUT / 4;        // channels a wave stages
  constexpr int NR = COUT == 16 ? 2 : 1;            // row tiles: re and im apart, or both in one
  constexpr int NC = CIN == 16 ? 2 : 1;             // column tiles
  __shared__ __align__(16) char smem[192 * (RI + RO) * sizeof(float2)];
  float2* tl = reinterpret_cast<float2*>(smem);     // [colour * 64 + site][channel]
  float2* gl = tl + 192 * RI;
  const int lb = xcd_block(blockIdx.x, gridDim.x);
  const int h = lb % 9, blk = (lb / 9) % nblk, item = lb / (9 * nblk);
  in += item * in_stride;
  G += item * g_stride;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int rc = lane & 15, kq = lane >> 4;         // row / column and k of this lane's operands
  f64x4_n acc[NR][NC];
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[r][c] = f64x4_n{0.0, 0.0, 0.0, 0.0};
  float2 u[9], a[CA][3], gr[CG][3];
  auto load = [&](int chunk) {
    const int site = min(chunk * 64 + lane, V - 1);
    int nb = site;
    if (h > 0) {
      int mu;
      bool f;
      hop_geom(h, site, Lx, Ly, Lz, Lt, nb, mu, f);
      const int ls = f ? site : nb;
#pragma unroll
      for (int e = 0; e < 9; ++e) u[e] = U[lnk_idx(ls, mu, e)];
    }
    const float2* ap = in + act_idx(nb, CIN, wid, 0);
    const float2* gp = G + act_idx(site, COUT, wid, 0);
#pragma unroll
    for (int k = 0; k < CA; ++k)
#pragma unroll
      for (int c = 0; c < 3; ++c) a[k][c] = ap[(12 * k + c) * kTile];
#pragma unroll
    for (int k = 0; k < CG; ++k)
#pragma unroll
      for (int c = 0; c < 3; ++c) gr[k][c] = gp[(12 * k + c) * kTile];
    if (chunk * 64 + 64 > V && chunk * 64 + lane >= V) {  // padding sites add nothing
#pragma unroll
      for (int k = 0; k < CA; ++k)
#pragma unroll
        for (int c = 0; c < 3; ++c) a[k][c] = make_float2(0.f, 0.f);
#pragma unroll
      for (int k = 0; k < CG; ++k)
#pragma unroll
        for (int c = 0; c < 3; ++c) gr[k][c] = make_float2(0.f, 0.f);
    }
  };
  // a lane's operands of k-step 0; with 4 channels rows (columns) 0..3 are real, 4..7 imaginary parts
  // and 8..15 repeat them (not read at the end)
  const float2* gq = reinterpret_cast<const float2*>(reinterpret_cast<const float*>(gl + kq * RO + (NR == 2 ? rc : rc & 3)) +
                                                     (NR == 2 ? 0 : (rc >> 2) & 1));
  const float2* aq = reinterpret_cast<const float2*>(reinterpret_cast<const float*>(tl + kq * RI + (NC == 2 ? rc : rc & 3)) +
                                                     (NC == 2 ? 0 : (rc >> 2) & 1));
  const int c1 = (int)((long)(blk + 1) * nchunks / nblk);
  int chunk = (int)((long)blk * nchunks / nblk);
#pragma unroll
  for (int e = 0; e < 9; ++e) u[e] = make_float2(0.f, 0.f);
  if (chunk < c1) load(chunk);
  for (; chunk < c1; ++chunk) {
#pragma unroll
    for (int k = 0; k < CA; ++k) {
      float2 tr[3];
      if (h > 0) {
        transport3(u, (h & 1) != 0, a[k], tr);
      } else {
#pragma unroll
        for (int c = 0; c < 3; ++c) tr[c] = a[k][c];
      }
#pragma unroll
      for (int c = 0; c < 3; ++c) tl[(c * 64 + lane) * RI + wid + 4 * k] = tr[c];
    }
#pragma unroll
    for (int k = 0; k < CG; ++k)
#pragma unroll
      for (int c = 0; c < 3; ++c) gl[(c * 64 + lane) * RO + wid + 4 * k] = gr[k][c];
    __syncthreads();
    if (chunk + 1 < c1) load(chunk + 1);
    __builtin_amdgcn_sched_barrier(0);  // keep these loads ahead of the products
#pragma unroll 4
    for (int s = 0; s < 12; ++s) {
      const int k = wid * 48 + 4 * s;
      double A[NR], B[NC];
      if (NR == 2) {
        const float2 v = gq[k * RO];
        A[0] = v.x;
        A[NR - 1] = v.y;
      } else {
        A[0] = reinterpret_cast<const float*>(gq)[2 * k * RO];
      }
      if (NC == 2) {
        const float2 v = aq[k * RI];
        B[0] = v.x;
        B[NC - 1] = v.y;
      } else {
        B[0] = reinterpret_cast<const float*>(aq)[2 * k * RI];
      }
#pragma unroll
      for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[r][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(A[r], B[c], acc[r][c], 0, 0, 0);
    }
    __syncthreads();
  }
  // add the four waves' tiles (register q of lane l is row 4 q + l / 16, column l % 16)
  double* red = reinterpret_cast<double*>(smem);
  static_assert(sizeof(smem) >= 4 * NR * NC * 256 * sizeof(double), "reduction buffer");
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int q = 0; q < 4; ++q) red[((wid * NR + r) * NC + c) * 256 + (4 * q + kq) * 16 + rc] = acc[r][c][q];
  __syncthreads();
  const int p = threadIdx.x;
  if (p < COUT * CIN) {
    const int o = p / CIN, i = p % CIN;
    auto at = [&](int gi, int ai) {  // <g part gi, a part ai> of the pair, 0 real, 1 imaginary
      const int rt = NR == 2 ? gi : 0, ct = NC == 2 ? ai : 0;
      const int row = NR == 2 ? o : o + 4 * gi, col = NC == 2 ? i : i + 4 * ai;
      double v = 0.0;
#pragma unroll
      for (int w = 0; w < 4; ++w) v += red[((w * NR + rt) * NC + ct) * 256 + row * 16 + col];
      return v;
    };
    const long base = (((long)item * 9 + h) * COUT * CIN + p) * 2 * nblk;
    part[base + blk] = at(0, 0) + at(1, 1);
    part[base + nblk + blk] = at(1, 0) - at(0, 1);
  }
}

// grad[e] = sum over items and blocks of the partials of entry e = (h, o, i), one wave per entry, fixed order.
__global__ void __launch_bounds__(256)
k_ptc_wgrad_reduce(const double* __restrict__ part, int nitems, int nentries, int nblk, float2* __restrict__ grad) {
  const int e = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (e >= nentries) return;
  double re = 0.0, im = 0.0;
  for (int it = 0; it < nitems; ++it) {
    const long base = ((long)it * nentries + e) * 2 * nblk;
    for (int c = lane; c < nblk; c += 64) {
      re += part[base + c];
      im += part[base + nblk + c];
    }
  }
  re = wave_sum(re);
  im = wave_sum(im);
  if (lane == 0) grad[e] = make_float2((float)re, (float)im);
}

// Adam with bias correction on each real component.
__global__ void k_adam(float* __restrict__ w, const float* __restrict__ g, float* __restrict__ m, float* __restrict__ v,
                       int n, float lr, float b1, float b2, float eps, float c1, float c2) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  w[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// Per item: ||b||^2 partials (part[item * gridDim.x + block]) and partial counts of the sites
// where b is nonzero (part[(nitems + item) * gridDim.x + block]); thread = site of the tiled field.
__global__ void __launch_bounds__(kBlock) k_site_stats(const double2* __restrict__ a, long nc, long Vpad,
                                                         int nitems, double* __restrict__ part) {
  const int item = blockIdx.y;
  a += item * nc;
  double acc = 0.0, cnt = 0.0;
  for (long site = (long)blockIdx.x * kBlock + threadIdx.x; site < Vpad; site += (long)gridDim.x * kBlock) {
    const long base = (site >> 6) * (kSpin * kTile) + (site & 63);
    double n2 = 0.0;
#pragma unroll
    for (int c = 0; c < kSpin; ++c) {
      const double2 v = a[base + c * kTile];
      n2 += v.x * v.x + v.y * v.y;
    }
    acc += n2;
    cnt += n2 > 0.0 ? 1.0 : 0.0;
  }
  __shared__ double lds[kBlock / 64];
  const double s = block_sum<kBlock>(acc, lds);
  __syncthreads();
  const double c = block_sum<kBlock>(cnt, lds);
  if (threadIdx.x == 0) {
    part[(long)item * gridDim.x + blockIdx.x] = s;
    part[(long)(nitems + item) * gridDim.x + blockIdx.x] = c;
  }
}
// per-item ||a||^2 partials of FP32 fields
__global__ void __launch_bounds__(kBlock) k_norm2_items_f32(const float2* __restrict__ a, long n,
                                                              double* __restrict__ part) {
  const int item = blockIdx.y;
  double acc = 0.0;
  for (long i = (long)blockIdx.x * kBlock + threadIdx.x; i < n; i += (long)gridDim.x * kBlock) {
    const float2 v = a[item * n + i];
    acc += (double)v.x * v.x + (double)v.y * v.y;
  }
  __shared__ double lds[kBlock / 64];
  const double s = block_sum<kBlock>(acc, lds);
  if (threadIdx.x == 0) part[(long)item * gridDim.x + blockIdx.x] = s;
}
// Input scale per item: the root-mean-square site norm over the sites where b is nonzero,
// s = sqrt(||b||^2 / n_nonzero), inv_s = 1/s (0 for b = 0), bn2 = ||b||^2; one thread per item.
__global__ void k_net_scales(const double* __restrict__ part, int nparts, int nitems, double* s, double* inv_s,
                             double* bn2) {
  const int it = blockIdx.x * blockDim.x + threadIdx.x;
  if (it >= nitems) return;
  double t = 0.0, c = 0.0;
  for (int g = 0; g < nparts; ++g) {
    t += part[(long)it * nparts + g];
    c += part[(long)(nitems + it) * nparts + g];
  }
  const double sv = c > 0.0 ? sqrt(t / c) : 0.0;
  s[it] = sv;
  inv_s[it] = sv > 0.0 ? 1.0 / sv : 0.0;
  bn2[it] = t;
}
// b32 = (float)(b64 * sc[item])
__global__ void k_to_f32_scaled(const double2* __restrict__ a, float2* __restrict__ b, long n,
                                const double* __restrict__ sc) {
  const int item = blockIdx.y;
  const double s = sc[item];
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    const double2 v = a[item * n + i];
    b[item * n + i] = make_float2((float)(v.x * s), (float)(v.y * s));
  }
}
__global__ void k_to_f64(const float2* __restrict__ a, double2* __restrict__ b, long n) {
  const int item = blockIdx.y;
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    b[item * n + i] = make_double2(a[item * n + i].x, a[item * n + i].y);
}
// d = y - x (FP32 minus FP64, rounded to FP32)
__global__ void k_sub_f32_f64(const float2* __restrict__ y, const double2* __restrict__ x, float2* __restrict__ d,
                              long n) {
  const int item = blockIdx.y;
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    const long k = item * n + i;
    d[k] = make_float2((float)((double)y[k].x - x[k].x), (float)((double)y[k].y - x[k].y));
  }
}
__global__ void k_scale_items_f32(float2* a, long n, const float* __restrict__ sc) {
  const int item = blockIdx.y;
  const float s = sc[item];
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    a[item * n + i] = c_scale(a[item * n + i], s);
}

constexpr int kStreamBlocks = 512;  // blocks per item of the streaming kernels here
constexpr int kStatBlocks = 128;    // blocks per item of the site statistics
constexpr int kWgradBlocks = 64;    // chunk groups of the weight-gradient kernel

long act_len(const Lattice& lat, int C) { return lat.ntiles * kTile * C * 3; }

void launch_layer(hipStream_t s, const Lattice& lat, const float2* U, const float2* in, float2* out, float2* zsave,
                  const float2* W, int cin, int cout, int act, int nitems, const double* out_scale) {
  const int Vpad = (int)(lat.ntiles * kTile), nblk = (Vpad + 255) / 256;
  const dim3 grid((unsigned)nblk * nitems), block(256);
  const int* L = lat.L;
  const long is = act_len(lat, cin), os = act_len(lat, cout);
  const int V = (int)lat.V;
#define DL_LAYER(CI, CO, NL)                                                                                  \
  hipLaunchKernelGGL((k_ptc_layer<CI, CO, NL>), grid, block, 0, s, U, in, out, zsave, W, L[0], L[1], L[2], L[3], \
                     V, Vpad, nblk, is, os)
  if (cin == 4 && cout == 16 && act == 1) DL_LAYER(4, 16, 1);
  else if (cin == 4 && cout == 16 && act == 2) DL_LAYER(4, 16, 2);
  else if (cin == 16 && cout == 16 && act == 1) DL_LAYER(16, 16, 1);
  else if (cin == 16 && cout == 16 && act == 2) DL_LAYER(16, 16, 2);
  else if (cin == 16 && cout == 4 && act == 0)
    hipLaunchKernelGGL(k_ptc_layer16_4, dim3((unsigned)lat.ntiles * nitems), dim3(128), 0, s, U, in, out, W, L[0], L[1],
                       L[2], L[3], V, (int)lat.ntiles, is, os, out_scale);
  else {
    fail(DL_E_INVALID, "unsupported layer width");
  }
#undef DL_LAYER
  DL_HIP(hipGetLastError());
}

// G (entries 9*cout*cin) = weight gradient of a layer with input `in` and output gradient `g`.
void layer_wgrad(hipStream_t s, const Lattice& lat, const float2* U, const float2* in, const float2* g, int cin,
                 int cout, int nitems, double* part, float2* G) {
  const int nblk = (int)std::min<long>(lat.ntiles, kWgradBlocks);
  const dim3 grid((unsigned)nblk * 9 * nitems), block(256);
  const int* L = lat.L;
  const long is = act_len(lat, cin), gs = act_len(lat, cout);
  const int V = (int)lat.V, nch = (int)lat.ntiles;
  if (cin == 4 && cout == 16)
    hipLaunchKernelGGL((k_ptc_wgrad<4, 16>), grid, block, 0, s, U, in, g, L[0], L[1], L[2], L[3], V, nch, nblk, is,
                       gs, part);
  else if (cin == 16 && cout == 16)
    hipLaunchKernelGGL((k_ptc_wgrad<16, 16>), grid, block, 0, s, U, in, g, L[0], L[1], L[2], L[3], V, nch, nblk, is,
                       gs, part);
  else
    hipLaunchKernelGGL((k_ptc_wgrad<16, 4>), grid, block, 0, s, U, in, g, L[0], L[1], L[2], L[3], V, nch, nblk, is,
                       gs, part);
  const int ne = 9 * cout * cin;
  hipLaunchKernelGGL(k_ptc_wgrad_reduce, dim3((ne + 3) / 4), dim3(256), 0, s, part, nitems, ne, nblk, G);
  DL_HIP(hipGetLastError());
}

// Forward pass; activations of layers 1, 2 (and pre-activations if keep) stay in net->acts.
void forward(dl_net* net, dl_op* op, int nitems, const double2* B, float2* Y, bool keep, bool bf16 = false) {
  hipStream_t s = net->ctx->stream;
  const Lattice& lat = op->lat;
  NetActs& a = net->acts;
  a.ensure(lat, nitems);
  const float2* U = op_links32_public(op);
  const long n = lat.nc;
  hipLaunchKernelGGL(k_site_stats, dim3(kStatBlocks, nitems), dim3(kBlock), 0, s, B, n, lat.ntiles * kTile, nitems,
                     a.part.get());
  hipLaunchKernelGGL(k_net_scales, dim3((nitems + 63) / 64), dim3(64), 0, s, a.part.get(), kStatBlocks, nitems,
                     a.s.get(), a.inv_s.get(), a.bn2.get());
  hipLaunchKernelGGL(k_to_f32_scaled, dim3(kStreamBlocks, nitems), dim3(256), 0, s, B, a.a0.get(), n,
                     (const double*)a.inv_s.get());
  DL_HIP(hipGetLastError());
  const float2* W = net->W.get();
  launch_layer(s, lat, U, a.a0.get(), a.a1.get(), keep ? a.z1.get() : nullptr, W + net_weight_offset(0), 4, 16, 1,
               nitems, nullptr);
  if (bf16 && !keep) {
    // inference: the 16 -> 16 layer's channel mixing in BF16 on the matrix cores
    if (net->frag16.n < (size_t)9 * 2 * 64 * 4) net->frag16.alloc((size_t)9 * 2 * 64 * 4);
    u32x4_n* fr = reinterpret_cast<u32x4_n*>(net->frag16.get());
    hipLaunchKernelGGL(k_ptc_wfrag16, dim3((9 * 2 * 64 + 255) / 256), dim3(256), 0, s, W + net_weight_offset(1), fr);
    const int* L = lat.L;
    const int ntiles = (int)lat.ntiles;
    hipLaunchKernelGGL(k_ptc_layer16_mfma, dim3((unsigned)ntiles * nitems), dim3(128), 0, s, U, a.a1.get(), a.a2.get(),
                       fr, L[0], L[1], L[2], L[3], (int)lat.V, ntiles, act_len(lat, 16), act_len(lat, 16));
    DL_HIP(hipGetLastError());
  } else {
    launch_layer(s, lat, U, a.a1.get(), a.a2.get(), keep ? a.z2.get() : nullptr, W + net_weight_offset(1), 16, 16,
                 1, nitems, nullptr);
  }
  launch_layer(s, lat, U, a.a2.get(), Y, nullptr, W + net_weight_offset(2), 16, 4, 0, nitems, a.s.get());
}

}  // namespace

int net_num_weights() {
  int n = 0;
  for (int l = 0; l < kNetLayers; ++l) n += 9 * kNetWidth[l + 1] * kNetWidth[l];
  return n;
}

long net_weight_offset(int layer) {
  long o = 0;
  for (int q = 0; q < layer; ++q) o += 9 * kNetWidth[q + 1] * kNetWidth[q];
  return o;
}

void NetActs::ensure(const Lattice& lat, int nitems) {
  if (items >= nitems && nc == lat.nc) return;
  items = nitems;
  nc = lat.nc;
  const size_t l4 = (size_t)act_len(lat, 4), l16 = (size_t)act_len(lat, 16);
  a0.alloc(nitems * l4);
  z1.alloc(nitems * l16);
  a1.alloc(nitems * l16);
  z2.alloc(nitems * l16);
  a2.alloc(nitems * l16);
  g16a.alloc(nitems * l16);
  g16b.alloc(nitems * l16);
  g4.alloc(nitems * l4);
  y.alloc(nitems * l4);
  r.alloc(nitems * l4);
  const size_t wg = (size_t)9 * 256 * 2 * kWgradBlocks;
  part.alloc((size_t)nitems * std::max<size_t>(wg, kStreamBlocks));
  s.alloc(nitems);
  inv_s.alloc(nitems);
  bn2.alloc(nitems);
  gsc.alloc(nitems);
}

const float2* net_guess(dl_net* net, dl_op* op, int nitems, const double2* B, bool bf16) {
  net->acts.ensure(op->lat, nitems);
  forward(net, op, nitems, B, net->acts.y.get(), false, bf16);
  return net->acts.y.get();
}

void net_apply(dl_net* net, dl_op* op, int nitems, const double2* B, double2* Y64, bool bf16) {
  net_guess(net, op, nitems, B, bf16);
  hipLaunchKernelGGL(k_to_f64, dim3(kStreamBlocks, nitems), dim3(256), 0, net->ctx->stream, net->acts.y.get(), Y64,
                     op->lat.nc);
  DL_HIP(hipGetLastError());
}

// d' = d - Y H^-1 Y^H (M^dag M d) for the error fields d (FP32, in acts.g4): the part of the
// guess's error that the D-CG start (net(b), then the Galerkin projection over Y) leaves.  The
// loss ||M d'||^2 then has gradient M^dag M d' with respect to d (the projection is orthogonal
// in the M^dag M inner product), so the backward pass below is unchanged.
__global__ void k_negate(long n, double2* a) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    a[i] = make_double2(-a[i].x, -a[i].y);
}

static void project_error(dl_net* net, dl_op* op, int nitems) {
  const dl_eig* e = net->proj;
  if (e->fingerprint != op->fingerprint || e->kind != op->kind)
    fail(DL_E_MISMATCH, "the training projection's eigenvectors belong to another operator");
  if (op->kind != DL_MDAGM) fail(DL_E_INVALID, "the projected training loss is the D-CG one (M^dag M operators)");
  hipStream_t s = net->ctx->stream;
  const Lattice& lat = op->lat;
  const long n = lat.nc, tot = (long)nitems * n;
  NetActs& a = net->acts;
  const float2* U = op_links32_public(op);
  const WilsonCfg cfg = wilson_cfg(op, DL_FP32, nitems);
  // A d (FP32 stencils) in a.g16a, widened; d widened
  wilson_batched<float>(s, lat, U, op->kappa, 0, a.g4.get(), a.r.get(), n, nitems, 0, nullptr, nullptr, nullptr, cfg);
  wilson_batched<float>(s, lat, U, op->kappa, 1, a.r.get(), a.g16a.get(), n, nitems, 0, nullptr, nullptr, nullptr,
                        cfg);
  DBuf<double2> ad((size_t)tot), d64((size_t)tot);
  widen_f64(s, tot, a.g16a.get(), ad.get());
  widen_f64(s, tot, a.g4.get(), d64.get());
  const int k = e->k;
  constexpr int kCols = 16, kRows = 64;
  DBuf<double> part((size_t)2 * kRows * kCols * tsk_multi_nblocks(n) + 64);
  DBuf<double2> cbuf(2 * (size_t)nitems * k);
  for (int c0 = 0; c0 < nitems; c0 += kCols) {
    const int nw = std::min(kCols, nitems - c0);
    for (int j0 = 0; j0 < k; j0 += kRows) {
      const int nv = std::min(kRows, k - j0);
      const int np = tsk_dots_multi(s, n, nv, e->Y.get() + (long)j0 * n, n, ad.get() + (long)c0 * n, n, nw, nullptr,
                                    part.get());
      for (int r = 0; r < nw; ++r)
        sum_partials(s, part.get() + (size_t)2 * r * nv * np, np, 2 * nv,
                     reinterpret_cast<double*>(cbuf.get() + (long)(c0 + r) * k + j0));
    }
  }
  double2* D = cbuf.get() + (long)nitems * k;
  proj_solve(s, k, nitems, e->Zr.get(), e->lamr.get(), cbuf.get(), D);
  hipLaunchKernelGGL(k_negate, dim3(64), dim3(256), 0, s, (long)nitems * k, D);
  for (int c0 = 0; c0 < nitems; c0 += kCols) {
    const int nw = std::min(kCols, nitems - c0);
    tsk_update_multi(s, n, k, e->Y.get(), n, D + (long)c0 * k, nw, nullptr, d64.get() + (long)c0 * n, n);
  }
  round_f32(s, tot, d64.get(), a.g4.get());
  DL_HIP(hipGetLastError());
}

double net_loss_grad(dl_net* net, dl_op* op, int nitems, const double2* B, const double2* X, bool grad) {
  hipStream_t s = net->ctx->stream;
  const Lattice& lat = op->lat;
  const long n = lat.nc;
  NetActs& a = net->acts;
  a.ensure(lat, nitems);
  const float2* U = op_links32_public(op);
  forward(net, op, nitems, B, a.y.get(), grad);
  // d = net(b) - x; r = M d; loss = mean ||r||^2 / ||b||^2
  hipLaunchKernelGGL(k_sub_f32_f64, dim3(kStreamBlocks, nitems), dim3(256), 0, s, a.y.get(), X, a.g4.get(), n);
  if (net->proj && net->proj->k > 0) project_error(net, op, nitems);
  wilson_batched<float>(s, lat, U, op->kappa, 0, a.g4.get(), a.r.get(), n, nitems, 0, nullptr, nullptr, nullptr,
                        wilson_cfg(op, DL_FP32, nitems));
  hipLaunchKernelGGL(k_norm2_items_f32, dim3(kStreamBlocks, nitems), dim3(kBlock), 0, s, a.r.get(), n, a.part.get());
  std::vector<double> hr((size_t)kStreamBlocks * nitems), hs(nitems), hb(nitems);
  DL_HIP(hipMemcpyAsync(hr.data(), a.part.get(), hr.size() * sizeof(double), hipMemcpyDeviceToHost, s));
  DL_HIP(hipMemcpyAsync(hs.data(), a.s.get(), nitems * sizeof(double), hipMemcpyDeviceToHost, s));
  DL_HIP(hipMemcpyAsync(hb.data(), a.bn2.get(), nitems * sizeof(double), hipMemcpyDeviceToHost, s));
  DL_HIP(hipStreamSynchronize(s));
  double L = 0.0;
  std::vector<float> gsc(nitems);
  for (int it = 0; it < nitems; ++it) {
    double rr = 0.0;
    for (int g = 0; g < kStreamBlocks; ++g) rr += hr[(size_t)it * kStreamBlocks + g];
    const double bn2 = hb[it];
    if (bn2 == 0.0) fail(DL_E_INVALID, "training pair with b = 0");
    L += rr / bn2 / nitems;
    // dL/dy = 2 M^dag r / (||b||^2 nitems) and y = s a3, so dL/da3 = s dL/dy
    gsc[it] = (float)(2.0 * hs[it] / bn2 / nitems);
  }
  if (!std::isfinite(L)) fail(DL_E_NONFINITE, "non-finite network loss");
  if (!grad) return L;
  DL_HIP(hipMemcpyAsync(a.gsc.get(), gsc.data(), nitems * sizeof(float), hipMemcpyHostToDevice, s));
  wilson_batched<float>(s, lat, U, op->kappa, 1, a.r.get(), a.g4.get(), n, nitems, 0, nullptr, nullptr, nullptr,
                        wilson_cfg(op, DL_FP32, nitems));
  hipLaunchKernelGGL(k_scale_items_f32, dim3(kStreamBlocks, nitems), dim3(256), 0, s, a.g4.get(), n,
                     (const float*)a.gsc.get());
  float2* W = net->W.get();
  float2* G = net->G.get();
  float2* Wt = net->Wt.get();
  // layer 3 (16 -> 4)
  layer_wgrad(s, lat, U, a.a2.get(), a.g4.get(), 16, 4, nitems, a.part.get(), G + net_weight_offset(2));
  hipLaunchKernelGGL(k_ptc_adjoint_weights, dim3((9 * 64 + 255) / 256), dim3(256), 0, s, W + net_weight_offset(2),
                     Wt + net_weight_offset(2), 16, 4);
  launch_layer(s, lat, U, a.g4.get(), a.g16a.get(), a.z2.get(), Wt + net_weight_offset(2), 4, 16, 2, nitems, nullptr);
  // layer 2 (16 -> 16)
  layer_wgrad(s, lat, U, a.a1.get(), a.g16a.get(), 16, 16, nitems, a.part.get(), G + net_weight_offset(1));
  hipLaunchKernelGGL(k_ptc_adjoint_weights, dim3((9 * 256 + 255) / 256), dim3(256), 0, s, W + net_weight_offset(1),
                     Wt + net_weight_offset(1), 16, 16);
  launch_layer(s, lat, U, a.g16a.get(), a.g16b.get(), a.z1.get(), Wt + net_weight_offset(1), 16, 16, 2, nitems,
               nullptr);
  // layer 1 (4 -> 16): weight gradient only
  layer_wgrad(s, lat, U, a.a0.get(), a.g16b.get(), 4, 16, nitems, a.part.get(), G + net_weight_offset(0));
  DL_HIP(hipGetLastError());
  return L;
}

void net_reset_adam(dl_net* net) {
  // m and v hold 2 * nw floats each = nw / 2 double2 (nw is even)
  const long nw = net_num_weights();
  zero(net->ctx->stream, nw / 2, reinterpret_cast<double2*>(net->m.get()));
  zero(net->ctx->stream, nw / 2, reinterpret_cast<double2*>(net->v.get()));
  net->step = 0;
}

void net_adam_step(dl_net* net, float lr) {
  net->step += 1;
  const int n = 2 * net_num_weights();
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  const float c1 = 1.f - std::pow(b1, (float)net->step), c2 = 1.f - std::pow(b2, (float)net->step);
  hipLaunchKernelGGL(k_adam, dim3((n + 255) / 256), dim3(256), 0, net->ctx->stream,
                     reinterpret_cast<float*>(net->W.get()), reinterpret_cast<const float*>(net->G.get()),
                     net->m.get(), net->v.get(), n, lr, b1, b2, eps, c1, c2);
  DL_HIP(hipGetLastError());
}

}  // namespace dl
