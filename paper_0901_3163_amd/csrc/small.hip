// Small dense FP64 problems of the restart and deflation steps (matrices of order m <= 512).
// They are chains of dependent steps, so what bounds them is the latency of one step: the
// serial parts (Jacobi rounds, Householder columns, Gram-Schmidt columns) run in one workgroup
// with their matrix in LDS (160 KB per CU), and what splits by rows or columns (eigenvectors,
// triangular solves, back substitutions) runs as one wave per row.
//
//  * jacobi -- cyclic Jacobi for real symmetric matrices with the
//    round-robin (circle) pairing: every round applies n/2 disjoint rotations
//    at once, so A <- J^T A J splits into independent 2x2 blocks and the round
//    needs two barriers.  Rotations are skipped when |a_pq| is below
//    eps * sqrt(|a_pp a_qq|) (relative accuracy for small eigenvalues); sweeps
//    stop when a sweep applies no rotation.
//  * landr_cycle -- end of a Lan-DR(m,k) cycle: Galerkin solve T_m d = c,
//    Ritz pairs of T_m, the k algebraically smallest kept, the arrowhead
//    projected matrix and right-hand side of the next cycle.
//  * minresdr_cycle -- end of a MinRes-DR(m,k) cycle: Householder QR of the
//    (m+1) x m matrix Tbar, least-squares d, the residual direction q spanning
//    range(Tbar)^perp, harmonic Ritz pairs from R^-T T_m R^-1 y = mu y
//    (Tbar^T Tbar = R^T R, theta = 1/mu), k smallest |theta| kept, the
//    orthonormal restart basis Q of [[G_k; 0], q], Q^T Tbar Q and Q^T s.
//  * proj_setup / k_proj_solve -- the Galerkin projection H d = c of
//    D-CG / D-MinRes with H = Y^H A Y complex Hermitian, solved through the
//    eigendecomposition of its real symmetric embedding [[Hr, -Hi], [Hi, Hr]].
//
// All projected matrices of the Hermitian Lanczos process are real: alpha_j
// and beta_j are real, and the restart matrices are real combinations.
#include "internal.hpp"
#include "cplx.hpp"
#include "rank.hpp"
#include "small.hpp"

namespace dl {

constexpr int kSmallThreads = 1024;

__device__ __forceinline__ double blk_reduce(double v, double* red, bool is_max) {
  // result broadcast to all threads
  for (int off = 32; off > 0; off >>= 1) {
    const double o = __shfl_xor(v, off, 64);
    v = is_max ? fmax(v, o) : v + o;
  }
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if (lane == 0) red[wid] = v;
  __syncthreads();
  double r = is_max ? -1.0 : 0.0;
  for (int w = 0; w < nw; ++w) r = is_max ? fmax(r, red[w]) : r + red[w];
  __syncthreads();
  return r;
}

// The general form, for orders that do not fit in LDS: matrices in global memory.
// Eigendecomposition of the symmetric n x n matrix A (destroyed; eigenvalues
// end on its diagonal), Z <- eigenvectors (columns).  rot: n/2+1 double4.
__device__ void jacobi_eigh(int n, double* A, int lda, double* Z, int ldz, double4* rot, double* red,
                            int* nrot) {
  const int tid = threadIdx.x, nt = blockDim.x;
  for (int e = tid; e < n * n; e += nt) {
    const int i = e / n, j = e % n;
    Z[(long)i * ldz + j] = (i == j) ? 1.0 : 0.0;
  }
  if (n <= 1) { __syncthreads(); return; }
  const int np = n + (n & 1), half = np / 2;
  for (int sweep = 0; sweep < 60; ++sweep) {
    double dm = 0.0;
    for (int i = tid; i < n; i += nt) dm = fmax(dm, fabs(A[(long)i * lda + i]));
    dm = blk_reduce(dm, red, true);
    double offmax = 0.0;
    for (int e = tid; e < n * n; e += nt) {
      const int i = e / n, j = e % n;
      if (i != j) offmax = fmax(offmax, fabs(A[(long)i * lda + j]));
    }
    offmax = blk_reduce(offmax, red, true);
    const double scale = fmax(dm, offmax);
    if (tid == 0) *nrot = 0;
    __syncthreads();
    for (int r = 0; r < np - 1; ++r) {
      for (int t = tid; t < half; t += nt) {
        int p, q;
        if (t == 0) { p = np - 1; q = r; }
        else { p = (r + t) % (np - 1); q = (r - t + np - 1) % (np - 1); }
        if (p > q) { const int tmp = p; p = q; q = tmp; }
        double c = 1.0, s = 0.0;
        if (q < n) {
          const double app = A[(long)p * lda + p], aqq = A[(long)q * lda + q], apq = A[(long)p * lda + q];
          const double aa = fabs(apq);
          if (aa > 2.220446049250313e-16 * sqrt(fabs(app * aqq)) && aa > 1e-18 * scale && aa > 1e-300) {
            const double tau = (aqq - app) / (2.0 * apq);
            const double tt = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
            c = 1.0 / sqrt(1.0 + tt * tt);
            s = tt * c;
            atomicAdd(nrot, 1);
          }
        }
        rot[t] = make_double4((double)p, (double)q, c, s);
      }
      __syncthreads();
      for (int e = tid; e < half * half; e += nt) {
        const int t1 = e / half, t2 = e % half;
        const double4 r1 = rot[t1], r2 = rot[t2];
        if (r1.w == 0.0 && r2.w == 0.0) continue;
        const int p1 = (int)r1.x, q1 = (int)r1.y, p2 = (int)r2.x, q2 = (int)r2.y;
        const bool q1ok = q1 < n, q2ok = q2 < n;
        const double c1 = r1.z, s1 = r1.w, c2 = r2.z, s2 = r2.w;
        const double a_pp = A[(long)p1 * lda + p2];
        const double a_pq = q2ok ? A[(long)p1 * lda + q2] : 0.0;
        const double a_qp = q1ok ? A[(long)q1 * lda + p2] : 0.0;
        const double a_qq = (q1ok && q2ok) ? A[(long)q1 * lda + q2] : 0.0;
        const double b_pp = c1 * a_pp - s1 * a_qp, b_pq = c1 * a_pq - s1 * a_qq;
        const double b_qp = s1 * a_pp + c1 * a_qp, b_qq = s1 * a_pq + c1 * a_qq;
        double n_pp = c2 * b_pp - s2 * b_pq, n_pq = s2 * b_pp + c2 * b_pq;
        double n_qp = c2 * b_qp - s2 * b_qq, n_qq = s2 * b_qp + c2 * b_qq;
        if (t1 == t2) { n_pq = 0.0; n_qp = 0.0; }
        A[(long)p1 * lda + p2] = n_pp;
        if (q2ok) A[(long)p1 * lda + q2] = n_pq;
        if (q1ok) A[(long)q1 * lda + p2] = n_qp;
        if (q1ok && q2ok) A[(long)q1 * lda + q2] = n_qq;
      }
      for (int e = tid; e < n * half; e += nt) {
        const int i = e / half, t = e % half;
        const double4 rr = rot[t];
        if (rr.w == 0.0) continue;
        const int p = (int)rr.x, q = (int)rr.y;
        const double zp = Z[(long)i * ldz + p], zq = Z[(long)i * ldz + q];
        Z[(long)i * ldz + p] = rr.z * zp - rr.w * zq;
        Z[(long)i * ldz + q] = rr.w * zp + rr.z * zq;
      }
      __syncthreads();
    }
    const int done = (*nrot == 0);
    __syncthreads();
    if (done) break;
  }
}

// ---- Jacobi with the matrix in LDS -----------------------------------------------------------
// A sits in LDS, so a round costs two barriers, LDS latency and the rotation's divisions instead of
// L2 round trips.  Measured, a whole cycle end: Lan-DR m = 60 1.97 -> 1.08 ms, MinRes-DR m = 120,
// k = 60 19.9 -> 4.2 ms (of them 2 x 1.37 ms here; the rest is the QR's, Gram-Schmidt's and
// eigenvectors' own chains below).
// The eigenvector update Z <- Z J is left out of that chain: the workgroup logs each round's
// rotations, and k_jacobi_vec applies the log to the rows of Z afterwards, one wave per row.
// Fits up to n = 142 (n^2 doubles plus the round's rotations in 160 KB).  Both triangles are kept and
// every block is updated by the rounded (c, s): then Lambda = Z^T T Z holds to rounding whatever
// the rotations' own errors, and the Galerkin solve Z Lambda^-1 Z^T c keeps its accuracy.  The
// packed triangle with the diagonal moved by t a_pq would halve the work, but the first solve's
// residual floor on a near-critical 4^4 field rose from 1e-12 to 1e-11 with it.

constexpr int kSweeps = 60;
constexpr size_t kLdsBytes = 163840;

__host__ __device__ inline int jac_half(int n) { return (n + (n & 1)) / 2; }
__host__ __device__ inline int jac_rounds(int n) { return n + (n & 1) - 1; }

static size_t jac_lds_bytes(int n) {
  return (size_t)n * n * sizeof(double) + (size_t)jac_half(n) * (sizeof(double2) + sizeof(int)) +
         (kSmallThreads / 64) * sizeof(double) + 4 * sizeof(int);
}
static bool jac_in_lds(int n) { return n >= 2 && jac_lds_bytes(n) <= kLdsBytes; }

// work of one eigendecomposition in doubles: the rotation log, its round numbers and their
// count, or (general form) the rotations of a round and a copy of A
static size_t jac_work(int n) {
  const size_t rounds = (size_t)kSweeps * jac_rounds(n);
  if (jac_in_lds(n)) return 2 * rounds * jac_half(n) + rounds / 2 + 4;
  return 4 * (size_t)(n / 2 + 1) + (size_t)n * n + 4;
}
// enough for every order up to n (the log of an order that fits in LDS outgrows the general form's)
static size_t jac_work_upto(int n) {
  int f = n;
  while (f > 1 && !jac_in_lds(f)) --f;
  return jac_work(n) > jac_work(f) ? jac_work(n) : jac_work(f);
}

// element (i >= j) of the symmetric input: 0 its lower triangle, 1 its upper, 2 the mean of both
__device__ __forceinline__ double sym_at(const double* A, int ld, int from, int i, int j) {
  if (from == 0) return A[(long)i * ld + j];
  if (from == 1) return A[(long)j * ld + i];
  return i == j ? A[(long)i * ld + i] : 0.5 * (A[(long)i * ld + j] + A[(long)j * ld + i]);
}

// pair t of round r (circle pairing of np = n + n % 2 players)
__device__ __forceinline__ void jac_pair(int r, int t, int np, int& p, int& q) {
  int a, b;
  if (t == 0) {
    a = np - 1;
    b = r;
  } else {
    a = r + t;
    if (a >= np - 1) a -= np - 1;
    b = r - t;
    if (b < 0) b += np - 1;
  }
  p = a < b ? a : b;
  q = a < b ? b : a;
}

// Eigenvalues of the symmetric matrix A (see sym_at) into ev (in the order the rotations leave
// them); log[round][t] = (c, s) of the rounds that rotated, rlist their numbers, meta[0] their
// count, meta[1] the rotations of the last sweep.  A thread keeps its pair t2 = tid % half and
// walks the pairs t1 = tid / half, + rows, ...
__global__ void __launch_bounds__(kSmallThreads)
k_jacobi_lds(int n, int rows, const double* __restrict__ A, int ld, int from, double* __restrict__ ev,
             double2* __restrict__ log, int* __restrict__ rlist, int* __restrict__ meta) {
  extern __shared__ __align__(16) double dyn[];
  const int half = jac_half(n), nrounds = jac_rounds(n), np = n + (n & 1);
  const int tid = threadIdx.x, nt = blockDim.x;
  double2* cs = reinterpret_cast<double2*>(dyn);           // the round's rotations
  double* red = dyn + 2 * half;                            // kSmallThreads / 64
  double* S = red + kSmallThreads / 64;                    // n x n
  int* pq = reinterpret_cast<int*>(S + n * n);
  int* flag = pq + half;                                   // [0, 1] a round rotated, [2] rotations of the sweep
  for (int e = tid; e < n * n; e += nt) {
    const int i = e / n, j = e % n;
    S[e] = i >= j ? sym_at(A, ld, from, i, j) : sym_at(A, ld, from, j, i);
  }
  const int t2 = tid % half, t1_0 = tid < rows * half ? tid / half : half;  // the last wave's spare lanes idle
  if (tid < 3) flag[tid] = 0;
  __syncthreads();
  int done_rounds = 0, g = 0, last = 0;
  for (int sweep = 0; sweep < kSweeps; ++sweep) {
    double mx = 0.0;
    for (int e = tid; e < n * n; e += nt) mx = fmax(mx, fabs(S[e]));
    const double scale = blk_reduce(mx, red, true);
    if (tid == 0) flag[2] = 0;
    __syncthreads();
    for (int r = 0; r < nrounds; ++r, ++g) {
      if (tid < half) {
        int p, q;
        jac_pair(r, tid, np, p, q);
        double c = 1.0, s = 0.0;
        if (q < n) {
          const double app = S[p * n + p], aqq = S[q * n + q], apq = S[p * n + q];
          const double aa = fabs(apq);
          if (aa > 2.220446049250313e-16 * sqrt(fabs(app * aqq)) && aa > 1e-18 * scale && aa > 1e-300) {
            const double tau = (aqq - app) / (2.0 * apq);
            const double tt = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
            c = 1.0 / sqrt(1.0 + tt * tt);
            s = tt * c;
          }
        }
        cs[tid] = make_double2(c, s);
        pq[tid] = p | (q << 16);
        const unsigned long long rotated = __ballot(s != 0.0);
        if (rotated && (tid & 63) == 0) {
          flag[g & 1] = 1;
          atomicAdd(&flag[2], __popcll(rotated));
        }
      }
      __syncthreads();
      if (flag[g & 1]) {
        if (tid < half) log[(long)done_rounds * half + tid] = cs[tid];
        if (tid == 0) rlist[done_rounds] = r;
        ++done_rounds;
        const double2 r2 = cs[t2];
        const int w2 = pq[t2], p2 = w2 & 0xffff, q2 = w2 >> 16;
        const bool q2ok = q2 < n;
        const double c2 = r2.x, s2 = r2.y;
#pragma unroll 2
        for (int t1 = t1_0; t1 < half; t1 += rows) {
          const double2 r1 = cs[t1];
          if (r1.y == 0.0 && r2.y == 0.0) continue;
          const int w1 = pq[t1], p1 = w1 & 0xffff, q1 = w1 >> 16;
          const bool q1ok = q1 < n;
          const double c1 = r1.x, s1 = r1.y;
          const double a_pp = S[p1 * n + p2];
          const double a_pq = q2ok ? S[p1 * n + q2] : 0.0;
          const double a_qp = q1ok ? S[q1 * n + p2] : 0.0;
          const double a_qq = (q1ok && q2ok) ? S[q1 * n + q2] : 0.0;
          const double b_pp = c1 * a_pp - s1 * a_qp, b_pq = c1 * a_pq - s1 * a_qq;
          const double b_qp = s1 * a_pp + c1 * a_qp, b_qq = s1 * a_pq + c1 * a_qq;
          double n_pp = c2 * b_pp - s2 * b_pq, n_pq = s2 * b_pp + c2 * b_pq;
          double n_qp = c2 * b_qp - s2 * b_qq, n_qq = s2 * b_qp + c2 * b_qq;
          if (t1 == t2) { n_pq = 0.0; n_qp = 0.0; }
          S[p1 * n + p2] = n_pp;
          if (q2ok) S[p1 * n + q2] = n_pq;
          if (q1ok) S[q1 * n + p2] = n_qp;
          if (q1ok && q2ok) S[q1 * n + q2] = n_qq;
        }
      }
      if (tid == 0) flag[(g + 1) & 1] = 0;
      __syncthreads();
    }
    last = flag[2];
    __syncthreads();
    if (last == 0) break;
  }
  for (int i = tid; i < n; i += nt) ev[i] = S[i * n + i];
  if (tid == 0) {
    meta[0] = done_rounds;
    meta[1] = last;
  }
}

// Rows of Z = I J_1 J_2 ...: one wave per row, the row in LDS, lane t rotating pairs t, t + 64.
// Only its own wave reads a row, so rounds need no block barrier; the log is read eight rounds ahead.
__global__ void __launch_bounds__(256)
k_jacobi_vec(int n, const double2* __restrict__ log, const int* __restrict__ rlist, const int* __restrict__ meta,
             double* __restrict__ Z) {
  extern __shared__ __align__(16) double dyn[];
  constexpr int kPer = 2, kAhead = 8;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int row = (int)blockIdx.x * 4 + wid;
  if (row >= n) return;  // whole waves; no barrier below
  double* z = dyn + (long)wid * (n + 2);
  const int half = jac_half(n), np = n + (n & 1);
  for (int j = lane; j <= n; j += 64) z[j] = j == row ? 1.0 : 0.0;
  wave_lds_exchange();
  const int nr = meta[0];
  for (int k0 = 0; k0 < nr; k0 += kAhead) {
    double2 c[kAhead][kPer];
    int rr[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int k = k0 + u < nr ? k0 + u : nr - 1;
      rr[u] = rlist[k];
#pragma unroll
      for (int h = 0; h < kPer; ++h) {
        const int t = lane + 64 * h;
        c[u][h] = t < half ? log[(long)k * half + t] : make_double2(1.0, 0.0);
      }
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      if (k0 + u >= nr) break;
#pragma unroll
      for (int h = 0; h < kPer; ++h) {
        const int t = lane + 64 * h;
        if (t < half && c[u][h].y != 0.0) {
          int p, q;
          jac_pair(rr[u], t, np, p, q);
          const double zp = z[p], zq = z[q];
          z[p] = c[u][h].x * zp - c[u][h].y * zq;
          z[q] = c[u][h].y * zp + c[u][h].x * zq;
        }
      }
      wave_lds_exchange();
    }
  }
  for (int j = lane; j < n; j += 64) Z[(long)row * n + j] = z[j];
}

// General form: copy of A in work, Jacobi on it.
__global__ void __launch_bounds__(kSmallThreads)
k_jacobi_global(int n, const double* A, int ld, int from, double* Z, double* ev, double* work) {
  __shared__ double red[kSmallThreads / 64];
  __shared__ int nrot;
  double4* rot = reinterpret_cast<double4*>(work);
  double* C = work + 4 * (n / 2 + 1);
  int* meta = reinterpret_cast<int*>(C + (long)n * n);
  for (int e = threadIdx.x; e < n * n; e += blockDim.x) {
    const int i = e / n, j = e % n;
    C[e] = i >= j ? sym_at(A, ld, from, i, j) : sym_at(A, ld, from, j, i);
  }
  __syncthreads();
  jacobi_eigh(n, C, n, Z, n, rot, red, &nrot);
  for (int i = threadIdx.x; i < n; i += blockDim.x) ev[i] = C[(long)i * n + i];
  if (threadIdx.x == 0) {
    meta[0] = 0;
    meta[1] = n > 1 ? nrot : 0;
  }
}

static int* jac_meta(int n, double* work) {
  if (!jac_in_lds(n)) return reinterpret_cast<int*>(work + 4 * (n / 2 + 1) + (size_t)n * n);
  const size_t rounds = (size_t)kSweeps * jac_rounds(n);
  return reinterpret_cast<int*>(work + 2 * rounds * jac_half(n) + rounds / 2);
}

// ev (unsorted) and Z (n x n, columns) of the symmetric matrix A; work: jac_work(n) doubles.  The
// block has about four 2x2 blocks a thread (fewer waves make the barriers cheaper), in whole rows
// of pairs and at least one thread a pair.
static void jacobi(hipStream_t s, int n, const double* A, int ld, int from, double* Z, double* ev, double* work) {
  if (!jac_in_lds(n)) {
    hipLaunchKernelGGL(k_jacobi_global, dim3(1), dim3(kSmallThreads), 0, s, n, A, ld, from, Z, ev, work);
    DL_HIP(hipGetLastError());
    return;
  }
  const int half = jac_half(n);
  const size_t rounds = (size_t)kSweeps * jac_rounds(n);
  double2* log = reinterpret_cast<double2*>(work);
  int* rlist = reinterpret_cast<int*>(work + 2 * rounds * half);
  int* meta = jac_meta(n, work);
  int rows = (half + 3) / 4;
  if (rows * half < 256) rows = (256 + half - 1) / half;
  while (rows > 1 && rows * half > kSmallThreads) --rows;
  hipLaunchKernelGGL(k_jacobi_lds, dim3(1), dim3((rows * half + 63) / 64 * 64), jac_lds_bytes(n), s, n, rows, A, ld,
                     from, ev, log, rlist, meta);
  hipLaunchKernelGGL(k_jacobi_vec, dim3((n + 3) / 4), dim3(256), 4 * (size_t)(n + 2) * sizeof(double), s, n, log,
                     rlist, meta, Z);
  DL_HIP(hipGetLastError());
}

// perm[rank] = i with ranks by (key ascending, NaN last, index ascending): every entry is set.
__device__ void rank_sort(int n, const double* key, int* perm) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) perm[key_rank(n, key, i)] = i;
  __syncthreads();
}

// ---------------------------------------------------------------------------
// Block j: eigenpair j of (key, Zt) to its place in ascending order.
__global__ void __launch_bounds__(256) k_eigh_sort(int n, const double* __restrict__ key,
                                                    const double* __restrict__ Zt, double* __restrict__ Z,
                                                    double* __restrict__ ev) {
  __shared__ int rank;
  const int j = blockIdx.x;
  if (threadIdx.x == 0) rank = 0;
  __syncthreads();
  const double kj = key[j];
  int r = 0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) r += key_before(key[i], i, kj, j);
  if (r) atomicAdd(&rank, r);
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += blockDim.x) Z[(long)i * n + rank] = Zt[(long)i * n + j];
  if (threadIdx.x == 0) ev[rank] = kj;
}

size_t small_eigh_work(int n) { return jac_work(n) + (size_t)n + (size_t)n * n + 8; }

void small_eigh(hipStream_t s, int n, double* A, double* Z, double* ev, double* work) {
  double* key = work + jac_work(n);
  double* Zt = key + n;
  jacobi(s, n, A, n, 1, Zt, key, work);
  hipLaunchKernelGGL(k_eigh_sort, dim3(n), dim3(256), 0, s, n, key, Zt, Z, ev);
  DL_HIP(hipGetLastError());
}

// ---------------------------------------------------------------------------
// Lan-DR cycle end.  Tb: (m+1) x m row-major (lower triangle valid), c: m+1.
// ev, Z: eigenpairs of T_m.  Outputs: d (m), Gk (m x k, ld k), info[0..]: see small.hpp.
__global__ void __launch_bounds__(kSmallThreads)
k_landr_end(int m, int ld, int k, double* Tb, double* c, const double* __restrict__ ev_, const double* __restrict__ Z,
            const int* __restrict__ meta, double* d, double* Gk, double* theta, double* rho, double* info) {
  extern __shared__ __align__(16) double dyn[];
  __shared__ double red[kSmallThreads / 64];
  __shared__ double sh_dm;
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wid = tid >> 6, nw = nt >> 6;
  double* ev = dyn;             // m
  double* y = ev + m;           // m
  double* part = y + m;         // nw x m
  int* perm = reinterpret_cast<int*>(part + (long)nw * m);  // m
  for (int i = tid; i < m; i += nt) ev[i] = ev_[i];
  double rs = 0.0;
  for (int i = wid; i < m; i += nw) {
    double s = 0.0;
    for (int j = lane; j < m; j += 64) s += fabs(i >= j ? Tb[(long)i * ld + j] : Tb[(long)j * ld + i]);
    rs = fmax(rs, wave_sum(s));
  }
  const double anorm = blk_reduce(rs, red, true);
  const double beta_m = Tb[(long)m * ld + (m - 1)];
  // d = Z diag(1/ev) Z^T c
  for (int i = lane; i < m; i += 64) {
    double s = 0.0;
    for (int j = wid; j < m; j += nw) s += Z[(long)j * m + i] * c[j];
    part[wid * m + i] = s;
  }
  __syncthreads();
  for (int i = tid; i < m; i += nt) {
    double s = 0.0;
    for (int w = 0; w < nw; ++w) s += part[w * m + i];
    y[i] = s / ev[i];
  }
  __syncthreads();
  for (int j = wid; j < m; j += nw) {
    double s = 0.0;
    for (int i = lane; i < m; i += 64) s += Z[(long)j * m + i] * y[i];
    s = wave_sum(s);
    if (lane == 0) {
      d[j] = s;
      if (j == m - 1) sh_dm = s;
    }
  }
  rank_sort(m, ev, perm);  // ends with a barrier
  for (int e = tid; e < m * k; e += nt) {
    const int j = e / k, l = e % k;
    Gk[e] = Z[(long)j * m + perm[l]];
  }
  for (int l = tid; l < k; l += nt) {
    theta[l] = ev[perm[l]];
    rho[l] = fabs(beta_m * Z[(long)(m - 1) * m + perm[l]]);
  }
  for (long e = tid; e < (long)(m + 1) * ld; e += nt) Tb[e] = 0.0;
  for (int i = tid; i <= m; i += nt) c[i] = 0.0;
  __syncthreads();
  for (int l = tid; l < k; l += nt) {
    Tb[(long)l * ld + l] = ev[perm[l]];
    Tb[(long)k * ld + l] = beta_m * Z[(long)(m - 1) * m + perm[l]];
  }
  if (tid == 0) {
    c[k] = -beta_m * sh_dm;
    info[0] = anorm;
    info[1] = beta_m;
    info[2] = fabs(beta_m * sh_dm);  // norm of the (normal-equation) FOM residual
    info[3] = (double)meta[1];
  }
}

size_t landr_work(int m) { return jac_work_upto(m) + (size_t)m * m + (size_t)m + 16; }

void landr_cycle(hipStream_t s, int m, int ld, int k, double* Tb, double* c, double* work, double* d, double* Gk,
                 double* theta, double* rho, double* info) {
  double* Z = work + jac_work(m);
  double* ev = Z + (size_t)m * m;
  jacobi(s, m, Tb, ld, 0, Z, ev, work);
  const size_t lds = ((size_t)2 * m + (size_t)(kSmallThreads / 64) * m) * sizeof(double) + (size_t)m * sizeof(int);
  hipLaunchKernelGGL(k_landr_end, dim3(1), dim3(kSmallThreads), lds, s, m, ld, k, Tb, c, ev, Z, jac_meta(m, work), d,
                     Gk, theta, rho, info);
  DL_HIP(hipGetLastError());
}

// ---------------------------------------------------------------------------
// MinRes-DR cycle end, in stages.  A lane holds rows lane, lane + 64, ... of a column (NR of them).

__device__ __forceinline__ double lane_at(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, l), hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Stage 1, one workgroup: Householder QR of Tbar with c as a last column (columns contiguous, in
// LDS when they fit, else in `cols`), one wave per trailing column and one barrier per
// reflector; d = R^-1 (Q^T c), q = Q e_m, s = c - Tbar d.  F: the full Tbar (row-major).
// Rr / Rc: R by rows and by columns.
template <bool LDS, int NR>
__global__ void __launch_bounds__(kSmallThreads)
k_mr_qr(int m, const double* __restrict__ Tb, const double* __restrict__ c, double* F, double* cols,
        double* __restrict__ Rr, double* __restrict__ Rc, double* __restrict__ d, double* __restrict__ q,
        double* __restrict__ s, double* __restrict__ info) {
  extern __shared__ __align__(16) double dyn[];
  __shared__ double red[kSmallThreads / 64];
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wid = tid >> 6, nw = nt >> 6;
  const int m1 = m + 1, lp = m1 | 1;
  double* al = dyn;       // m   diagonal of R
  double* tau = al + m;   // m
  double* vh = tau + m;   // m   head element of each reflector
  double* ev = vh + m;    // m1
  double* dv = ev + m1;   // m
  double* qv = dv + m;    // m1
  double* C = LDS ? qv + m1 : cols;  // m1 columns of lp
  double rs = 0.0;
  for (int i = wid; i <= m; i += nw) {
    double a = 0.0;
    for (int j = lane; j < m; j += 64) {
      const double v = (i >= j || i == m) ? Tb[(long)i * m + j] : Tb[(long)j * m + i];
      F[(long)i * m + j] = v;
      C[(long)j * lp + i] = v;
      a += fabs(v);
    }
    a = wave_sum(a);
    if (i < m) rs = fmax(rs, a);
  }
  for (int i = tid; i <= m; i += nt) C[(long)m * lp + i] = c[i];
  const double anorm = blk_reduce(rs, red, true);  // its barriers also publish the columns
  for (int j = 0; j < m; ++j) {
    // the reflector, formed by every wave: v = (v0, C[j][j+1..m])
    double v[NR];
    double ss = 0.0;
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      const int i = lane + 64 * k;
      v[k] = (i > j && i <= m) ? C[(long)j * lp + i] : 0.0;
      ss = fma(v[k], v[k], ss);
    }
    ss = wave_sum(ss);
    const double x0 = C[(long)j * lp + j];
    const double nrm = sqrt(ss + x0 * x0);
    double alpha = 0.0, tj = 0.0, v0 = 1.0;
    if (nrm != 0.0) {
      alpha = x0 >= 0.0 ? -nrm : nrm;
      v0 = x0 - alpha;
      tj = 2.0 / (v0 * v0 + ss);
    }
#pragma unroll
    for (int k = 0; k < NR; ++k)
      if (lane + 64 * k == j) v[k] = v0;
    for (int l = j + 1 + wid; l <= m; l += nw) {
      double* col = C + (long)l * lp;
      double x[NR], w = 0.0;
#pragma unroll
      for (int k = 0; k < NR; ++k) {
        const int i = lane + 64 * k;
        x[k] = (i >= j && i <= m) ? col[i] : 0.0;
        w = fma(v[k], x[k], w);
      }
      w = tj * wave_sum(w);
#pragma unroll
      for (int k = 0; k < NR; ++k) {
        const int i = lane + 64 * k;
        if (i >= j && i <= m) col[i] = x[k] - w * v[k];
      }
    }
    if (tid == 0) {
      al[j] = alpha;
      tau[j] = tj;
      vh[j] = v0;
    }
    __syncthreads();
  }
  if (wid == 0) {
    // d = R^-1 e, column-oriented, in one wave
    for (int i = lane; i <= m; i += 64) ev[i] = C[(long)m * lp + i];
    wave_lds_exchange();
    for (int j = m - 1; j >= 0; --j) {
      const double dj = ev[j] / al[j];
      if (lane == 0) dv[j] = dj;
      for (int i = lane; i < j; i += 64) ev[i] -= C[(long)j * lp + i] * dj;
      wave_lds_exchange();
    }
  } else if (wid == 1) {
    // q = H_0 ... H_{m-1} e_m
    double x[NR];
#pragma unroll
    for (int k = 0; k < NR; ++k) x[k] = lane + 64 * k == m ? 1.0 : 0.0;
    for (int j = m - 1; j >= 0; --j) {
      double v[NR], w = 0.0;
#pragma unroll
      for (int k = 0; k < NR; ++k) {
        const int i = lane + 64 * k;
        v[k] = i == j ? vh[j] : (i > j && i <= m) ? C[(long)j * lp + i] : 0.0;
        w = fma(v[k], x[k], w);
      }
      w = tau[j] * wave_sum(w);
#pragma unroll
      for (int k = 0; k < NR; ++k) x[k] -= w * v[k];
    }
#pragma unroll
    for (int k = 0; k < NR; ++k)
      if (lane + 64 * k <= m) q[lane + 64 * k] = x[k];
  }
  __syncthreads();
  double sn = 0.0;
  for (int i = wid; i <= m; i += nw) {
    double a = 0.0;
    for (int j = lane; j < m; j += 64) a = fma(F[(long)i * m + j], dv[j], a);
    a = c[i] - wave_sum(a);
    if (lane == 0) s[i] = a;
    sn += a * a;
  }
  if (lane != 0) sn = 0.0;
  sn = blk_reduce(sn, red, false);
  for (int j = wid; j < m; j += nw)
    for (int i = lane; i <= j; i += 64) {
      const double r = i == j ? al[j] : C[(long)j * lp + i];
      Rc[(long)j * m + i] = r;
      Rr[(long)i * m + j] = r;
    }
  for (int j = tid; j < m; j += nt) d[j] = dv[j];
  if (tid == 0) {
    info[0] = anorm;
    info[1] = Tb[(long)m * m + (m - 1)];
    info[2] = sqrt(sn);
  }
}

// x R = (row blockIdx.x of In), one wave per row; the result is stored as a column of Out.  Twice
// of this forms R^-T T R^-1: W^T from the rows of T, then its rows give the columns of A.
template <int NR>
__global__ void __launch_bounds__(64)
k_mr_trsm(int m, const double* __restrict__ In, const double* __restrict__ Rr, double* __restrict__ Out) {
  const int lane = threadIdx.x, row = blockIdx.x;
  double a[NR];
#pragma unroll
  for (int k = 0; k < NR; ++k) a[k] = lane + 64 * k < m ? In[(long)row * m + lane + 64 * k] : 0.0;
#pragma unroll
  for (int kk = 0; kk < NR; ++kk) {
#pragma unroll 4
    for (int lj = 0; lj < 64; ++lj) {
      const int j = 64 * kk + lj;
      if (j >= m) break;
      const double* r = Rr + (long)j * m;
      const double x = lane_at(a[kk], lj) / r[j];
#pragma unroll
      for (int k = kk; k < NR; ++k) {
        const int l = lane + 64 * k;
        if (l == j) a[k] = x;
        if (l > j && l < m) a[k] -= x * r[l];
      }
    }
  }
#pragma unroll
  for (int k = 0; k < NR; ++k)
    if (lane + 64 * k < m) Out[(long)(lane + 64 * k) * m + row] = a[k];
}

// Kept harmonic Ritz vector l = blockIdx.x (the l-th smallest |1/mu|, NaN last; ties: 1/mu ascending, then
// index): g_l = R^-1 y_l into row l of Q (m + 1 entries, the last zero); hth[l] = 1/mu.
template <int NR>
__global__ void __launch_bounds__(64)
k_mr_ritz(int m, const double* __restrict__ mu, const double* __restrict__ Z, const double* __restrict__ Rc,
          double* __restrict__ Q, double* __restrict__ hth) {
  __shared__ double key[512];
  __shared__ int scol;
  const int lane = threadIdx.x, l = blockIdx.x;
  for (int i = lane; i < m; i += 64) key[i] = mu[i] != 0.0 ? 1.0 / mu[i] : INFINITY;
  __syncthreads();
  for (int i = lane; i < m; i += 64)
    if (key_rank_abs(m, key, i) == l) scol = i;
  __syncthreads();
  const int col = scol;
  double a[NR];
#pragma unroll
  for (int k = 0; k < NR; ++k) a[k] = lane + 64 * k < m ? Z[(long)(lane + 64 * k) * m + col] : 0.0;
#pragma unroll
  for (int kk = NR - 1; kk >= 0; --kk) {
#pragma unroll 4
    for (int lj = 63; lj >= 0; --lj) {
      const int j = 64 * kk + lj;
      if (j >= m) continue;
      const double* r = Rc + (long)j * m;
      const double x = lane_at(a[kk], lj) / r[j];
#pragma unroll
      for (int k = 0; k <= kk; ++k) {
        const int i = lane + 64 * k;
        if (i == j) a[k] = x;
        if (i < j) a[k] -= x * r[i];
      }
    }
  }
  double* o = Q + (long)l * (m + 1);
#pragma unroll
  for (int k = 0; k < NR; ++k)
    if (lane + 64 * k <= m) o[lane + 64 * k] = lane + 64 * k < m ? a[k] : 0.0;
  if (lane == 0) hth[l] = key[col];
}

// Stage 3, one workgroup: the k + 1 rows of Qr (g_l, then q) orthonormalised by classical
// Gram-Schmidt applied twice, X = Tbar Q[:, :k], Tn = Q^T X ((k+1) x k), cn = Q^T s, H = sym(Tn[:k]).
// Q (m+1 x k+1) is the row-major copy.  Both work matrices in LDS when they fit, else in `big`.
template <bool LDS>
__global__ void __launch_bounds__(kSmallThreads)
k_mr_orth(int m, int k, const double* __restrict__ F, const double* __restrict__ Qr, const double* __restrict__ q,
          const double* __restrict__ s, double* big, double* __restrict__ Q, double* __restrict__ Tn,
          double* __restrict__ cn, double* __restrict__ H) {
  extern __shared__ __align__(16) double dyn[];
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wid = tid >> 6, nw = nt >> 6;
  const int m1 = m + 1, k1 = k + 1, lp = m1 | 1;
  double* h = dyn;                    // k1
  double* B = LDS ? h + k1 : big;     // k1 rows of lp: the basis
  double* X = B + (long)k1 * lp;      // k rows of lp
  for (int t = tid; t < k1 * m1; t += nt) {
    const int l = t / m1, i = t % m1;
    B[(long)l * lp + i] = l < k ? Qr[(long)l * m1 + i] : q[i];
  }
  __syncthreads();
  for (int j = 0; j <= k; ++j) {
    double* bj = B + (long)j * lp;
    for (int pass = 0; pass < 2; ++pass) {
      for (int i = wid; i < j; i += nw) {
        double a = 0.0;
        for (int r = lane; r <= m; r += 64) a = fma(B[(long)i * lp + r], bj[r], a);
        a = wave_sum(a);
        if (lane == 0) h[i] = a;
      }
      __syncthreads();
      for (int r = tid; r <= m; r += nt) {
        double a = bj[r];
        for (int i = 0; i < j; ++i) a -= h[i] * B[(long)i * lp + r];
        bj[r] = a;
      }
      __syncthreads();
    }
    double nn = 0.0;
    for (int r = lane; r <= m; r += 64) nn = fma(bj[r], bj[r], nn);
    nn = wave_sum(nn);
    const double inv = nn > 0.0 ? 1.0 / sqrt(nn) : 0.0;
    __syncthreads();
    for (int r = tid; r <= m; r += nt) bj[r] *= inv;
    __syncthreads();
  }
  for (int t = tid; t < m1 * k1; t += nt) Q[t] = B[(long)(t % k1) * lp + t / k1];
  for (int t = tid; t < m1 * k; t += nt) {
    const int i = t / k, l = t % k;
    double a = 0.0;
#pragma unroll 4
    for (int j = 0; j < m; ++j) a += F[(long)i * m + j] * B[(long)l * lp + j];
    X[(long)l * lp + i] = a;
  }
  __syncthreads();
  for (int t = tid; t < k1 * k; t += nt) {
    const int a_ = t / k, l = t % k;
    double a = 0.0;
    for (int i = 0; i <= m; ++i) a += B[(long)a_ * lp + i] * X[(long)l * lp + i];
    Tn[t] = a;
  }
  for (int a_ = wid; a_ <= k; a_ += nw) {
    double a = 0.0;
    for (int i = lane; i <= m; i += 64) a = fma(B[(long)a_ * lp + i], s[i], a);
    a = wave_sum(a);
    if (lane == 0) cn[a_] = a;
  }
  __syncthreads();  // Tn is read back by other threads of this workgroup
  for (int t = tid; t < k * k; t += nt) {
    const int i = t / k, j = t % k;
    H[t] = 0.5 * (Tn[(long)i * k + j] + Tn[(long)j * k + i]);
  }
}

// Stage 4: Rayleigh-Ritz in span V_k from H = Z diag(key) Z^T: S, lam ascending, rho = |Tn[k,:] S|; the
// next cycle's Tbar <- Tn and c <- cn.
__global__ void __launch_bounds__(kSmallThreads)
k_mr_end(int m, int k, const double* __restrict__ key_, const double* __restrict__ Z, const double* __restrict__ Tn,
         const double* __restrict__ cn, const int* __restrict__ meta, double* __restrict__ Tb, double* __restrict__ c,
         double* __restrict__ S, double* __restrict__ lam, double* __restrict__ rho, double* __restrict__ info) {
  __shared__ double key[512];
  __shared__ int perm[512];
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wid = tid >> 6, nw = nt >> 6;
  const int m1 = m + 1, k1 = k + 1;
  for (int i = tid; i < k; i += nt) key[i] = key_[i];
  for (long t = tid; t < (long)m1 * m; t += nt) {
    const int i = (int)(t / m), j = (int)(t % m);
    Tb[t] = i < k1 && j < k ? Tn[(long)i * k + j] : 0.0;
  }
  for (int i = tid; i <= m; i += nt) c[i] = i < k1 ? cn[i] : 0.0;
  __syncthreads();
  rank_sort(k, key, perm);
  for (int t = tid; t < k * k; t += nt) {
    const int i = t / k, l = t % k;
    S[t] = Z[(long)i * k + perm[l]];
  }
  for (int l = wid; l < k; l += nw) {
    double a = 0.0;
    for (int i = lane; i < k; i += 64) a = fma(Tn[(long)k * k + i], Z[(long)i * k + perm[l]], a);
    a = wave_sum(a);
    if (lane == 0) {
      lam[l] = key[perm[l]];
      rho[l] = fabs(a);
    }
  }
  if (tid == 0) info[3] = k > 0 ? (double)meta[1] : 0.0;
}

static size_t mr_qr_lds(int m, bool cols) {
  const int m1 = m + 1, lp = m1 | 1;
  return (4 * (size_t)m + 2 * (size_t)m1 + (cols ? (size_t)m1 * lp : 0)) * sizeof(double);
}
static size_t mr_orth_lds(int m, int k, bool mats) {
  const int m1 = m + 1, lp = m1 | 1;
  return ((size_t)(k + 1) + (mats ? (size_t)(2 * k + 1) * lp : 0)) * sizeof(double);
}
// static __shared__ of the stage kernels beside the dynamic part
constexpr size_t kStaticLds = 512;

// F, R by rows and by columns, W^T, A, Z (m x m) and the columns or work matrices that LDS cannot hold
size_t minresdr_work(int m) {
  const size_t m1 = m + 1, lp = m1 | 1;
  return m1 * m + 5 * (size_t)m * m + 2 * m1 * lp + m1 * m1 + 6 * m1 + jac_work_upto(m) + 64;
}

template <int NR>
static void mr_cycle(hipStream_t s, int m, int k, double* Tb, double* c, double* work, double* d, double* Q,
                     double* lam, double* S, double* rho, double* hth, double* info) {
  const size_t m1 = m + 1, lp = m1 | 1;
  double* F = work;                 // m1 x m
  double* Rr = F + m1 * m;          // m x m
  double* Rc = Rr + (size_t)m * m;  // m x m
  double* W = Rc + (size_t)m * m;   // m x m
  double* A = W + (size_t)m * m;    // m x m
  double* Z = A + (size_t)m * m;    // m x m
  double* big = Z + (size_t)m * m;  // 2 m1 lp
  double* Qr = big + 2 * m1 * lp;   // k1 x m1
  double* sv = Qr + m1 * m1;        // m1
  double* qv = sv + m1;             // m1
  double* cn = qv + m1;             // m1
  double* key = cn + m1;            // m
  double* jw = key + m1;            // jac_work_upto(m)
  // the QR's columns fit in LDS for every order of two rows a lane, for some of three and for none of eight
  const bool qr_lds = NR == 2 || (NR == 3 && mr_qr_lds(m, true) + kStaticLds <= kLdsBytes);
  const bool or_lds = mr_orth_lds(m, k, true) + kStaticLds <= kLdsBytes;
  const dim3 one(1), wide(kSmallThreads);
  if constexpr (NR <= 3) {
    if (qr_lds)
      hipLaunchKernelGGL((k_mr_qr<true, NR>), one, wide, mr_qr_lds(m, true), s, m, Tb, c, F, big, Rr, Rc, d, qv, sv,
                         info);
  }
  if constexpr (NR >= 3) {
    if (!qr_lds)
      hipLaunchKernelGGL((k_mr_qr<false, NR>), one, wide, mr_qr_lds(m, false), s, m, Tb, c, F, big, Rr, Rc, d, qv, sv,
                         info);
  }
  hipLaunchKernelGGL(k_mr_trsm<NR>, dim3(m), dim3(64), 0, s, m, F, Rr, W);   // W = W^T of T_m R^-1
  hipLaunchKernelGGL(k_mr_trsm<NR>, dim3(m), dim3(64), 0, s, m, W, Rr, A);
  jacobi(s, m, A, m, 2, Z, key, jw);
  if (k > 0)
    hipLaunchKernelGGL(k_mr_ritz<NR>, dim3(k), dim3(64), 0, s, m, key, Z, Rc, Qr, hth);
  double* Tn = W;                   // k1 x k
  double* H = A;                    // k x k
  if (or_lds)
    hipLaunchKernelGGL(k_mr_orth<true>, one, wide, mr_orth_lds(m, k, true), s, m, k, F, Qr, qv, sv, big, Q, Tn, cn, H);
  else
    hipLaunchKernelGGL(k_mr_orth<false>, one, wide, mr_orth_lds(m, k, false), s, m, k, F, Qr, qv, sv, big, Q, Tn, cn,
                       H);
  if (k > 0) jacobi(s, k, H, k, 1, Z, key, jw);
  hipLaunchKernelGGL(k_mr_end, one, wide, 0, s, m, k, key, Z, Tn, cn, jac_meta(k > 0 ? k : m, jw), Tb, c, S, lam, rho,
                     info);
  DL_HIP(hipGetLastError());
}

void minresdr_cycle(hipStream_t s, int m, int k, double* Tb, double* c, double* work, double* d, double* Q,
                    double* lam, double* S, double* rho, double* hth, double* info) {
  if (m + 1 <= 128) mr_cycle<2>(s, m, k, Tb, c, work, d, Q, lam, S, rho, hth, info);
  else if (m + 1 <= 192) mr_cycle<3>(s, m, k, Tb, c, work, d, Q, lam, S, rho, hth, info);
  else mr_cycle<8>(s, m, k, Tb, c, work, d, Q, lam, S, rho, hth, info);
}

// ---------------------------------------------------------------------------
// Projection matrix setup: Hc = complex k x k (interleaved, Hc[i*k+j] = <y_i, A y_j>)
// -> real embedding E (2k x 2k) -> Z (2k x 2k), lamr (2k).
__global__ void __launch_bounds__(256) k_proj_embed(int k, const double2* __restrict__ Hc, double* __restrict__ E) {
  const int n = 2 * k;
  for (int t = blockIdx.x * 256 + threadIdx.x; t < k * k; t += gridDim.x * 256) {
    const int i = t / k, j = t % k;
    const double2 a = Hc[(long)i * k + j], b = Hc[(long)j * k + i];
    const double hr = 0.5 * (a.x + b.x), hi = 0.5 * (a.y - b.y);  // Hermitian part
    E[(long)i * n + j] = hr;
    E[(long)(i + k) * n + (j + k)] = hr;
    E[(long)i * n + (j + k)] = -hi;
    E[(long)(i + k) * n + j] = hi;
  }
}

size_t proj_work(int k) { return jac_work(2 * k); }

void proj_setup(hipStream_t s, int k, const double2* Hc, double* E, double* Z, double* lamr, double* work) {
  hipLaunchKernelGGL(k_proj_embed, dim3((k * k + 255) / 256), dim3(256), 0, s, k, Hc, E);
  jacobi(s, 2 * k, E, 2 * k, 1, Z, lamr, work);
}

// d = H^-1 c for nrhs right-hand sides (c, d: [nrhs][k] complex); one block per rhs.
__global__ void __launch_bounds__(256)
k_proj_solve(int k, const double* Z, const double* lamr, const double2* c, double2* d) {
  extern __shared__ double sm[];
  const int n = 2 * k;
  const double2* cr = c + (long)blockIdx.x * k;
  double2* dr = d + (long)blockIdx.x * k;
  double* u = sm;  // n
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    double a = 0.0;
    for (int r = 0; r < n; ++r) {
      const double2 cv = cr[r % k];
      a += Z[(long)r * n + i] * (r < k ? cv.x : cv.y);
    }
    u[i] = a / lamr[i];
  }
  __syncthreads();
  for (int r = threadIdx.x; r < k; r += blockDim.x) {
    double re = 0.0, im = 0.0;
    for (int i = 0; i < n; ++i) {
      re += Z[(long)r * n + i] * u[i];
      im += Z[(long)(r + k) * n + i] * u[i];
    }
    dr[r] = make_double2(re, im);
  }
}

void proj_solve(hipStream_t s, int k, int nrhs, const double* Z, const double* lamr, const double2* c, double2* d) {
  if (k <= 0 || nrhs <= 0) return;
  hipLaunchKernelGGL(k_proj_solve, dim3(nrhs), dim3(256), 2 * k * sizeof(double), s, k, Z, lamr, c, d);
  DL_HIP(hipGetLastError());
}

}  // namespace dl
