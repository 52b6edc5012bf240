// Layout conversion and BLAS-1 kernels with deterministic two-stage reductions.
//
// Reductions: each block of 256 threads reduces its grid-stride share with a
// wavefront shuffle tree and writes one partial per block; a second kernel sums
// the partials of each column in a fixed order.  The number of blocks depends
// only on the vector length, so results are bitwise reproducible.
#include "internal.hpp"
#include "cplx.hpp"

#include <algorithm>

namespace dl {

// ---- layout ----------------------------------------------------------------
// Caller's layout ([site][12] double2) <-> tiled fields in FP64, FP32 or BF16 storage (rounded through
// FP32).  One wave per 64-site tile: 12 coalesced accesses on each side, transposed in LDS (rows of
// 13 elements; each wave its own, so no block barrier), with the padding sites of the
// last tile written as zeros.  Bound by the copy's bytes.  Rounding here rather than in a pass of its
// own, and no zeroing pass before: for 12 fields of 16^3 x 32 to BF16 38 + 142 + 85 us became one
// 61 us launch (378 MB, 6.2 TB/s), and 64 + 111 us back became 54.  The caller's side is accessed
// non-temporally: it is touched once, and kept out of the Infinity Cache it leaves that to the tiled
// fields (100 us and 58 us without, and the stencil between them 99 instead of 85).
template <class SV>
__device__ __forceinline__ SV pack_cast(double2 v);
template <>
__device__ __forceinline__ double2 pack_cast<double2>(double2 v) { return v; }
template <>
__device__ __forceinline__ float2 pack_cast<float2>(double2 v) { return make_float2((float)v.x, (float)v.y); }
template <>
__device__ __forceinline__ bf2 pack_cast<bf2>(double2 v) {
  const unsigned w = bf_pack(make_float2((float)v.x, (float)v.y));
  return bf2{(unsigned short)(w & 0xffff), (unsigned short)(w >> 16)};
}
__device__ __forceinline__ double2 wide(double2 v) { return v; }
__device__ __forceinline__ double2 wide(float2 v) { return make_double2(v.x, v.y); }
__device__ __forceinline__ double2 wide(bf2 v) { return wide(sldv(v)); }

constexpr int kPackRow = kSpin + 1;

typedef double f64x2_nt __attribute__((ext_vector_type(2)));
__device__ __forceinline__ double2 ld_nt(const double2* p) {
  const f64x2_nt v = __builtin_nontemporal_load(reinterpret_cast<const f64x2_nt*>(p));
  return make_double2(v.x, v.y);
}
__device__ __forceinline__ void st_nt(double2* p, double2 v) {
  const f64x2_nt t = {v.x, v.y};
  __builtin_nontemporal_store(t, reinterpret_cast<f64x2_nt*>(p));
}

template <class SV>
__global__ void __launch_bounds__(256)
k_pack_spinor(const double2* __restrict__ in, SV* __restrict__ out, long V, long nc, long ntiles) {
  __shared__ SV stage[4][kTile * kPackRow];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const long tile = (long)blockIdx.x * 4 + wid;
  if (tile >= ntiles) return;  // whole waves
  const long f = blockIdx.y, e0 = tile * kTile * kSpin;
  const double2* src = in + f * V * kSpin + e0;
  const long left = V * kSpin - e0;  // elements of this tile and the ones after it
  SV* st = stage[wid];
  double2 v[kSpin];
#pragma unroll
  for (int k = 0; k < kSpin; ++k) {
    const int e = k * 64 + lane;
    v[k] = e < left ? ld_nt(src + e) : make_double2(0.0, 0.0);
  }
#pragma unroll
  for (int k = 0; k < kSpin; ++k) {
    const int e = k * 64 + lane;
    st[e / kSpin * kPackRow + e % kSpin] = pack_cast<SV>(v[k]);
  }
  wave_lds_exchange();
  SV* dst = out + f * nc + e0 + lane;
#pragma unroll
  for (int c = 0; c < kSpin; ++c) dst[c * kTile] = st[lane * kPackRow + c];
}

template <class SV>
__global__ void __launch_bounds__(256)
k_unpack_spinor(const SV* __restrict__ in, double2* __restrict__ out, long V, long nc, long ntiles) {
  __shared__ SV stage[4][kTile * kPackRow];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const long tile = (long)blockIdx.x * 4 + wid;
  if (tile >= ntiles) return;
  const long f = blockIdx.y, e0 = tile * kTile * kSpin;
  const SV* src = in + f * nc + e0 + lane;
  const long left = V * kSpin - e0;
  SV* st = stage[wid];
  SV v[kSpin];
#pragma unroll
  for (int c = 0; c < kSpin; ++c) v[c] = src[c * kTile];
#pragma unroll
  for (int c = 0; c < kSpin; ++c) st[lane * kPackRow + c] = v[c];
  wave_lds_exchange();
  double2* dst = out + f * V * kSpin + e0;
#pragma unroll
  for (int k = 0; k < kSpin; ++k) {
    const int e = k * 64 + lane;
    if (e < left) st_nt(dst + e, wide(st[e / kSpin * kPackRow + e % kSpin]));
  }
}

__global__ void k_pack_links(const double2* __restrict__ in, double2* __restrict__ out, long V) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= V * kLinkC) return;
  const long site = i / kLinkC;
  const int c = (int)(i % kLinkC);
  out[((site >> 6) * kLinkC + c) * kTile + (site & 63)] = in[i];
}

// fields of one launch: gridDim.y is at most 65535
constexpr int kMaxFieldsY = 65535;

template <class SV>
void pack_spinor(hipStream_t s, const Lattice& lat, const double2* in, SV* out, int nfield) {
  for (int f = 0; f < nfield; f += kMaxFieldsY)
    hipLaunchKernelGGL(k_pack_spinor<SV>, dim3((lat.ntiles + 3) / 4, std::min(nfield - f, kMaxFieldsY)), dim3(256), 0,
                       s, in + f * lat.V * kSpin, out + f * lat.nc, lat.V, lat.nc, lat.ntiles);
  DL_HIP(hipGetLastError());
}

template <class SV>
void unpack_spinor(hipStream_t s, const Lattice& lat, const SV* in, double2* out, int nfield) {
  for (int f = 0; f < nfield; f += kMaxFieldsY)
    hipLaunchKernelGGL(k_unpack_spinor<SV>, dim3((lat.ntiles + 3) / 4, std::min(nfield - f, kMaxFieldsY)), dim3(256), 0,
                       s, in + f * lat.nc, out + f * lat.V * kSpin, lat.V, lat.nc, lat.ntiles);
  DL_HIP(hipGetLastError());
}

#define DL_PACK(SV)                                                                                  \
  template void pack_spinor<SV>(hipStream_t, const Lattice&, const double2*, SV*, int);             \
  template void unpack_spinor<SV>(hipStream_t, const Lattice&, const SV*, double2*, int);
DL_PACK(double2)
DL_PACK(float2)
DL_PACK(bf2)
#undef DL_PACK

void pack_links(hipStream_t s, const Lattice& lat, const double2* in, double2* out) {
  const long n = lat.V * kLinkC;
  hipLaunchKernelGGL(k_pack_links, dim3((n + 255) / 256), dim3(256), 0, s, in, out, lat.V);
  DL_HIP(hipGetLastError());
}

// ---- streaming reductions -----------------------------------------------------
int nblocks_for(long n) {
  long nb = (n + 4 * kBlock - 1) / (4 * kBlock);
  if (nb < 1) nb = 1;
  if (nb > 1024) nb = 1024;
  return (int)nb;
}

__global__ void __launch_bounds__(kBlock)
k_norm2_partials(long n, const double2* __restrict__ a, double* __restrict__ part) {
  double acc = 0.0;
  for (long i = (long)blockIdx.x * kBlock + threadIdx.x; i < n; i += (long)gridDim.x * kBlock) {
    const double2 x = a[i];
    acc = fma(x.x, x.x, acc);
    acc = fma(x.y, x.y, acc);
  }
  __shared__ double lds[kBlock / 64];
  const double s = block_sum<kBlock>(acc, lds);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

int norm2_partials(hipStream_t s, long n, const double2* a, double* part) {
  const int nb = nblocks_for(n);
  hipLaunchKernelGGL(k_norm2_partials, dim3(nb), dim3(kBlock), 0, s, n, a, part);
  DL_HIP(hipGetLastError());
  return nb;
}

__global__ void __launch_bounds__(kBlock)
k_sum_partials(const double* __restrict__ part, int nparts, int width, double* __restrict__ out,
               double* __restrict__ last) {
  const int col = blockIdx.x;
  double acc = 0.0;
  const double* p = part + (long)col * nparts;
  for (int i = threadIdx.x; i < nparts; i += kBlock) acc += p[i];
  __shared__ double lds[kBlock / 64];
  const double s = block_sum<kBlock>(acc, lds);
  if (threadIdx.x == 0) *(col < width ? out + col : last) = s;
}

void sum_partials(hipStream_t s, const double* part, int nparts, int width, double* out, double* last) {
  hipLaunchKernelGGL(k_sum_partials, dim3(width + (last ? 1 : 0)), dim3(kBlock), 0, s, part, nparts, width, out, last);
  DL_HIP(hipGetLastError());
}

// ---- elementwise -------------------------------------------------------------
__global__ void k_copy(long n, const double2* __restrict__ a, double2* __restrict__ b) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) b[i] = a[i];
}
__global__ void k_zero(long n, double2* __restrict__ a) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) a[i] = make_double2(0.0, 0.0);
}

void copy(hipStream_t s, long n, const double2* a, double2* b) {
  hipLaunchKernelGGL(k_copy, dim3((n + 255) / 256), dim3(256), 0, s, n, a, b);
  DL_HIP(hipGetLastError());
}
void zero(hipStream_t s, long n, double2* a) {
  hipLaunchKernelGGL(k_zero, dim3((n + 255) / 256), dim3(256), 0, s, n, a);
  DL_HIP(hipGetLastError());
}

__global__ void k_round_f32(long n, const double2* __restrict__ a, float2* __restrict__ b) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    b[i] = make_float2((float)a[i].x, (float)a[i].y);
}
__global__ void k_widen_f64(long n, const float2* __restrict__ a, double2* __restrict__ b) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    b[i] = make_double2(a[i].x, a[i].y);
}

__global__ void k_round_bf16(long n, const double2* __restrict__ a, bf2* __restrict__ b) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    sst(b + i, make_float2((float)a[i].x, (float)a[i].y));
}
void round_bf16(hipStream_t s, long n, const double2* a, bf2* b) {
  hipLaunchKernelGGL(k_round_bf16, dim3(2048), dim3(256), 0, s, n, a, b);
  DL_HIP(hipGetLastError());
}

void round_f32(hipStream_t s, long n, const double2* a, float2* b) {
  hipLaunchKernelGGL(k_round_f32, dim3(2048), dim3(256), 0, s, n, a, b);
  DL_HIP(hipGetLastError());
}
void widen_f64(hipStream_t s, long n, const float2* a, double2* b) {
  hipLaunchKernelGGL(k_widen_f64, dim3(2048), dim3(256), 0, s, n, a, b);
  DL_HIP(hipGetLastError());
}

}  // namespace dl

namespace dl {

// splitmix64 finaliser (Steele, Lea and Flood, OOPSLA 2014) as the per-element mixer
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  return z ^ (z >> 31);
}

__global__ void __launch_bounds__(256) k_field_hash(long n, const double2* __restrict__ a, uint64_t* part) {
  uint64_t acc = 0;
  for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long)gridDim.x * 256) {
    const double2 v = a[i];
    const uint64_t re = (uint64_t)__double_as_longlong(v.x), im = (uint64_t)__double_as_longlong(v.y);
    acc += mix64(re ^ mix64(2 * (uint64_t)i + 1)) + mix64(im ^ mix64(2 * (uint64_t)i + 2));
  }
  __shared__ uint64_t lds[256];
  lds[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) lds[threadIdx.x] += lds[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = lds[0];
}

uint64_t field_hash(hipStream_t s, long n, const double2* a) {
  constexpr int kParts = 1024;
  DBuf<uint64_t> part(kParts);
  hipLaunchKernelGGL(k_field_hash, dim3(kParts), dim3(256), 0, s, n, a, part.get());
  DL_HIP(hipGetLastError());
  std::vector<uint64_t> h(kParts);
  DL_HIP(hipMemcpyAsync(h.data(), part.get(), kParts * sizeof(uint64_t), hipMemcpyDeviceToHost, s));
  DL_HIP(hipStreamSynchronize(s));
  uint64_t t = 0;
  for (uint64_t v : h) t += v;
  return t;
}

}  // namespace dl
