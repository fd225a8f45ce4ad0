// libnsk: implicit time stepping with the six-stage fourth-order ESDIRK
// scheme named in Sec. 3.1 for the implicit runs (Kennedy and Carpenter's
// ARK4(3)6L[2]SA implicit tableau: gamma = 1/4, explicit first stage,
// stiffly accurate), with a Jacobian-free Newton-Krylov solver for the stage
// equations.
//
// One step from U_n:  K_1 = R(U_n); for stage i = 2..6 solve
//   G(X) = X - dt gamma R(X) - B_i = 0,   B_i = U_n + dt sum_{j<i} a_ij K_j,
// by Newton's method, each correction from one cycle of right-preconditioned
// GMRES with classical Gram-Schmidt (repeated when the projection cancels
// most of the vector) and the Jacobian-vector product (R(X + s z) - R(X))/s;
// then K_i = (X - B_i)/(dt gamma); U_{n+1} is the last stage's X.  Every
// right-hand side is nsk_rhs on the bound context; the vector work runs in
// the kernels below, with fixed-order reductions, so a run is bitwise
// reproducible.  The coefficients of a projection are formed on the device and
// the host reads the dot products of each Arnoldi step from pinned memory,
// while the kernel that uses them runs: only the two decisions (project again,
// converged) need the host.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>
#include <type_traits>
#include <vector>

#include "../../include/nsk.h"
#include "host_common.hpp"

using namespace nsk;

namespace {

constexpr int kVecThreads = 256;
constexpr int kDotBlocks = 1024;  // partial sums per dot product
constexpr int kLinTerms = 8;      // vectors per linear-combination launch

struct LinArgs {
  const double* x[kLinTerms];
  double a[kLinTerms];
};

// Calls f(std::integral_constant<int, K>{}) for the runtime count k in
// [0, kLinTerms]: the vector kernels take their vector count as a template
// parameter, so that all of an entry's loads issue together instead of one
// branch and wait per vector.
template <typename F>
void with_count(int k, F&& f) {
  switch (k) {
    case 0: f(std::integral_constant<int, 0>{}); break;
    case 1: f(std::integral_constant<int, 1>{}); break;
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 5: f(std::integral_constant<int, 5>{}); break;
    case 6: f(std::integral_constant<int, 6>{}); break;
    case 7: f(std::integral_constant<int, 7>{}); break;
    default: f(std::integral_constant<int, 8>{}); break;
  }
}
static_assert(kLinTerms == 8, "with_count covers counts up to 8");

// Every vector kernel here streams its operands once.  At 24x12x12 elements, N = 4
// (17 MB a vector, FP64 basis), a Krylov step of two vectors is: right-hand side
// 57 us, multidot_kernel with the product 16 us, dot_final_kernel 6 us,
// orth_kernel 12 us and, projected again, 6 + 17 us; a step of the
// scheme 6.06 ms, against 9.84 ms with the perturbed state, the product, each
// norm and the second products in passes of their own and the host waiting for
// every set of products before it launches what uses them.

// the block's sum of v in a fixed order into red[wave]; summed by block_total
__device__ __forceinline__ void wave_total(double v, double* red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
}

__device__ __forceinline__ double block_total(const double* red) {
  double t = 0.0;
  for (int k = 0; k < kVecThreads / 64; ++k) t += red[k];
  return t;
}

// part[j * kDotBlocks + b]: block b's sum over its contiguous chunk, row j
__device__ __forceinline__ void chunk_of(long long n, long long& beg, long long& end) {
  const long long chunk = (n + kDotBlocks - 1) / kDotBlocks;
  beg = (long long)blockIdx.x * chunk;
  end = beg + chunk < n ? beg + chunk : n;
}

// Start of a stage: K = (X - B) / (dt gamma) of the stage before (NEWK; else K is
// given), B = sum_{k < NK} a_k x_k + ak K, the predictor X = B + dt gamma K, and
// the chunk's sum of B^2 to row 0 of part.
template <int NK, bool NEWK>
__global__ void __launch_bounds__(kVecThreads) stage_start_kernel(LinArgs L, double ak, double dtg, double* K,
                                                                  double* B, double* X, long long n,
                                                                  double* __restrict__ part) {
  __shared__ double red[kVecThreads / 64];
  long long beg, end;
  chunk_of(n, beg, end);
  double bb = 0.0;
  const double ip = 1.0 / dtg;
  for (long long i = beg + threadIdx.x; i < end; i += kVecThreads) {
    double k;
    if constexpr (NEWK) {
      k = ip * X[i];
      k += -ip * B[i];
      K[i] = k;
    } else {
      k = K[i];
    }
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < NK; ++q) s += L.a[q] * L.x[q][i];
    s += ak * k;
    B[i] = s;
    X[i] = s + dtg * k;
    bb += s * s;
  }
  wave_total(bb, red);
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = block_total(red);
}

// r = B + dt gamma R(X) - X = -G(X); the chunk's sums of r^2 and X^2 to rows 0, 1
__global__ void __launch_bounds__(kVecThreads) residual_kernel(const double* __restrict__ B,
                                                               const double* __restrict__ RX,
                                                               const double* __restrict__ X, double dtg,
                                                               double* __restrict__ r, long long n,
                                                               double* __restrict__ part) {
  __shared__ double red[2][kVecThreads / 64];
  long long beg, end;
  chunk_of(n, beg, end);
  double rr = 0.0, xx = 0.0;
  for (long long i = beg + threadIdx.x; i < end; i += kVecThreads) {
    const double x = X[i], t = B[i] + dtg * RX[i], v = t - x;
    r[i] = v;
    rr += v * v;
    xx += x * x;
  }
  wave_total(rr, red[0]);
  wave_total(xx, red[1]);
  __syncthreads();
  if (threadIdx.x < 2) part[(long long)threadIdx.x * kDotBlocks + blockIdx.x] = block_total(red[threadIdx.x]);
}

// Node-local preconditioner of the relaxation source (model II): with
// a = dt gamma alpha / beta the stiff part of I - dt gamma dR/dU at a node is
// identity except the c row, (1 + a) c - a rho; its inverse maps v to v with
// c replaced by (v_c + a v_rho) / (1 + a).
struct Precond {
  int on;
  int ci;      // index of the c variable
  double a;
  long long S; // entries per variable
};

template <typename VT>
__device__ __forceinline__ double pinv(const VT* __restrict__ v, long long i, const Precond& p) {
  const long long c0 = (long long)p.ci * p.S;  // first entry of the c variable
  if (p.on && i >= c0 && i - c0 < p.S) {
    const long long o = i - c0;
    return (double(v[i]) + p.a * double(v[o])) / (1.0 + p.a);
  }
  return double(v[i]);
}

// The product of v with B = A - I, where A = (I - dt gamma dR/dU) P^{-1} is the
// GMRES operator:  w = (P^{-1} v - v) - c (Rp - RX), c = dt gamma / s.
// A and B span the same Krylov spaces and A's Hessenberg matrix is B's plus
// the identity; A is close to the identity, so projecting A v onto the basis
// would cancel most of it, while B v keeps only the part that is not v.
template <typename VT>
struct Jvp {
  const VT* v;
  const double *Rp, *RX;
  double c;
  Precond p;
};

// Rows j < NJ of part: the chunk's sums of w[i] * v_j[i], v_j = V + j * vstride;
// with self, row NJ: of w[i]^2.  V is the Krylov basis (FP64 or FP32); products
// and sums are FP64.  JVP: w is formed here from the two right-hand sides and
// stored, so that forming it costs no pass of its own (12.5 us a step at the
// size above); else it is read.
template <typename VT, int NJ, bool JVP>
__global__ void __launch_bounds__(kVecThreads) multidot_kernel(double* __restrict__ w, Jvp<VT> q,
                                                               const VT* __restrict__ V, long long vstride,
                                                               int self, long long n, double* __restrict__ part) {
  __shared__ double red[NJ + 1][kVecThreads / 64];
  long long beg, end;
  chunk_of(n, beg, end);
  double s[NJ + 1];
#pragma unroll
  for (int j = 0; j <= NJ; ++j) s[j] = 0.0;
  for (long long i = beg + threadIdx.x; i < end; i += kVecThreads) {
    double wi;
    if constexpr (JVP) {
      wi = (pinv(q.v, i, q.p) - double(q.v[i])) - q.c * (q.Rp[i] - q.RX[i]);
      w[i] = wi;
    } else {
      wi = w[i];
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) s[j] += wi * double(V[j * vstride + i]);
    s[NJ] += wi * wi;
  }
#pragma unroll
  for (int j = 0; j <= NJ; ++j) wave_total(s[j], red[j]);
  __syncthreads();
  const int outs = NJ + (self ? 1 : 0);
  if (threadIdx.x < outs) part[(long long)threadIdx.x * kDotBlocks + blockIdx.x] = block_total(red[threadIdx.x]);
}

constexpr int kFinalThreads = 1024;

// What a projection does with its dot products
enum { kSums = 0, kFirst = 1, kSecond = 2 };

// The sums of rows 0..nrow-1 of part in a fixed order (one wave a row), to the
// host; and for orth_kernel, coef[0] the factor of w, coef[1] whether the
// projection is to be repeated, coef[2 + j] the factors of the basis:
//   kSums    the factor 1/|r| of row 0, r the residual
//   kFirst   |w - sum h_j V_j|^2 by Pythagoras from rows 0..nrow-2 (the h_j) and
//            row nrow-1 (|w|^2); V_{k+1} = (w - sum h_j V_j) / its norm, or, where
//            that is <= reorth_tol |w|^2 (1/2: Kahan's criterion, more than
//            1/sqrt(2) of |w| cancelled), the FP64 w itself, to be projected again
//   kSecond  V_{k+1} after the second projection
// host[nrow] is the norm, host[nrow + 1] whether to repeat.
__global__ void __launch_bounds__(kFinalThreads) dot_final_kernel(const double* __restrict__ part, int nrow, int mode,
                                                                  double reorth_tol, double* __restrict__ coef,
                                                                  double* __restrict__ host) {
#pragma clang fp contract(off)
  __shared__ double h[NSK_GMRES_MAX + 2], sh[3];
  const int lane = threadIdx.x & 63;
  for (int j = threadIdx.x >> 6; j < nrow; j += kFinalThreads / 64) {
    const double* row = part + (long long)j * kDotBlocks;
    double t[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      t[q] = 0.0;
#pragma unroll
      for (int b = 0; b < kDotBlocks; b += 256) t[q] += row[b + q * 64 + lane];
    }
    double v = (t[0] + t[2]) + (t[1] + t[3]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off);
    if (lane == 0) h[j] = v;
  }
  __syncthreads();
  const int nj = nrow - 1;
  if (threadIdx.x == 0) {
    double norm, cw;
    bool again = false;
    if (mode == kSums) {
      norm = sqrt(h[0]);
      cw = 1.0 / norm;
    } else {
      const double ww = h[nj];
      double proj = 0.0;
      for (int j = 0; j < nj; ++j) proj += h[j] * h[j];
      norm = ww - proj > 0.0 ? sqrt(ww - proj) : 0.0;
      if (mode == kFirst) again = !(norm * norm > reorth_tol * ww) || !(norm > 0.0);
      cw = again ? 1.0 : (mode == kFirst || norm > 0.0 ? 1.0 / norm : 1.0);
    }
    sh[0] = norm;
    sh[1] = cw;
    sh[2] = again ? 1.0 : 0.0;
    coef[0] = cw;
    coef[1] = sh[2];
    host[nrow] = norm;
    host[nrow + 1] = sh[2];
  }
  __syncthreads();
  for (int j = threadIdx.x; j < nrow; j += kFinalThreads) {
    host[j] = h[j];
    if (mode != kSums && j < nj) coef[2 + j] = sh[2] != 0.0 ? -h[j] : (mode == kFirst ? -h[j] / sh[0] : -h[j] * sh[1]);
  }
  __threadfence_system();
}
static_assert(kDotBlocks == 1024, "four columns of 256 a row");

// w += ... of kLinTerms basis vectors, where a projection takes more than one launch
template <typename VT>
__global__ void __launch_bounds__(kVecThreads) accumulate_kernel(double* w, const double* __restrict__ coef, int j0,
                                                                 const VT* __restrict__ V, long long vstride,
                                                                 long long n) {
  const long long stride = (long long)gridDim.x * kVecThreads;
  const double cw = j0 == 0 ? coef[0] : 1.0;
  for (long long i = (long long)blockIdx.x * kVecThreads + threadIdx.x; i < n; i += stride) {
    double t = cw * w[i];
#pragma unroll
    for (int j = 0; j < kLinTerms; ++j) t += coef[2 + j0 + j] * double(V[j * vstride + i]);
    w[i] = t;
  }
}

// t = coef[0] w + sum_{j < NK} coef[2 + j0 + j] V_{j0 + j} (w as it stands for
// j0 > 0).  Where the projection is to be repeated, w = t, and with part, which
// is for j0 = 0, rows 0..NK of it are the next products, as of multidot_kernel
// (the basis is in registers here: 12 us and a gap less); else V_{k+1} = t and
// the state of the next Jacobian-vector product, Xp = X + s P^{-1} V_{k+1}, which
// would take a pass of 12 us by itself at the size above.  With the
// preconditioner a thread of a rho entry does the c entry as well.
template <typename VT, int NK>
__global__ void __launch_bounds__(kVecThreads) orth_kernel(double* w, const double* __restrict__ coef, int j0,
                                                           const VT* __restrict__ V, long long vstride,
                                                           VT* __restrict__ vnew, const double* __restrict__ X,
                                                           double s, Precond p, double* __restrict__ Xp, long long n,
                                                           double* __restrict__ part) {
  __shared__ double red[NK + 1][kVecThreads / 64];
  const long long stride = (long long)gridDim.x * kVecThreads;
  const long long i0 = (long long)blockIdx.x * kVecThreads + threadIdx.x;
  const double cw = j0 == 0 ? coef[0] : 1.0;
  double a[NK > 0 ? NK : 1];
#pragma unroll
  for (int j = 0; j < NK; ++j) a[j] = coef[2 + j0 + j];
  const auto comb = [&](long long i) {
    double t = cw * w[i];
#pragma unroll
    for (int j = 0; j < NK; ++j) t += a[j] * double(V[j * vstride + i]);
    return t;
  };
  if (coef[1] != 0.0) {
    if (!part) {
      for (long long i = i0; i < n; i += stride) w[i] = comb(i);
      return;
    }
    if (blockIdx.x >= kDotBlocks) return;
    long long beg, end;
    chunk_of(n, beg, end);
    double d[NK + 1];
#pragma unroll
    for (int j = 0; j <= NK; ++j) d[j] = 0.0;
    for (long long i = beg + threadIdx.x; i < end; i += kVecThreads) {
      double t = cw * w[i], v[NK > 0 ? NK : 1];
#pragma unroll
      for (int j = 0; j < NK; ++j) {
        v[j] = double(V[j * vstride + i]);
        t += a[j] * v[j];
      }
      w[i] = t;
#pragma unroll
      for (int j = 0; j < NK; ++j) d[j] += t * v[j];
      d[NK] += t * t;
    }
#pragma unroll
    for (int j = 0; j <= NK; ++j) wave_total(d[j], red[j]);
    __syncthreads();
    if (threadIdx.x <= NK) part[(long long)threadIdx.x * kDotBlocks + blockIdx.x] = block_total(red[threadIdx.x]);
    return;
  }
  const long long c0 = (long long)p.ci * p.S, nt = p.on ? c0 : n;
  for (long long i = i0; i < nt; i += stride) {
    const VT v = VT(comb(i));
    vnew[i] = v;
    Xp[i] = X[i] + s * double(v);
    if (p.on && i < p.S) {
      const VT vc = VT(comb(c0 + i));
      vnew[c0 + i] = vc;
      Xp[c0 + i] = X[c0 + i] + s * ((double(vc) + p.a * double(v)) / (1.0 + p.a));
    }
  }
}

// y = (y0 ? y0 : 0) + sum_{j < NK} a_j V_j; X += P^{-1} y, or with y1, y1 = y (a
// part of the sum; y0 and y1 may be the same vector)
struct BasisCoefs {
  double a[kLinTerms];
};
template <typename VT, int NK>
__global__ void __launch_bounds__(kVecThreads) correct_kernel(const double* y0, const VT* __restrict__ V,
                                                              long long vstride, BasisCoefs c, double* y1,
                                                              double* __restrict__ X, Precond p, long long n) {
  const long long stride = (long long)gridDim.x * kVecThreads;
  const auto comb = [&](long long i) {
    double t = y0 ? y0[i] : 0.0;
#pragma unroll
    for (int j = 0; j < NK; ++j) t += c.a[j] * double(V[j * vstride + i]);
    return t;
  };
  const long long c0 = (long long)p.ci * p.S, nt = !y1 && p.on ? c0 : n;
  for (long long i = (long long)blockIdx.x * kVecThreads + threadIdx.x; i < nt; i += stride) {
    const double y = comb(i);
    if (y1) {
      y1[i] = y;
      continue;
    }
    X[i] += y;
    if (p.on && i < p.S) X[c0 + i] += (comb(c0 + i) + p.a * y) / (1.0 + p.a);
  }
}

// ESDIRK4(6) implicit tableau (lower triangle with the diagonal gamma), gamma = 1/4.
constexpr double kGamma = 0.25;
const double kA[6][6] = {
    {0, 0, 0, 0, 0, 0},
    {1.0 / 4, 0.25, 0, 0, 0, 0},
    {8611.0 / 62500, -1743.0 / 31250, 0.25, 0, 0, 0},
    {5012029.0 / 34652500, -654441.0 / 2922500, 174375.0 / 388108, 0.25, 0, 0},
    {15267082809.0 / 155376265600, -71443401.0 / 120774400, 730878875.0 / 902184768, 2285395.0 / 8070912, 0.25,
     0},
    {82889.0 / 524892, 0.0, 15625.0 / 83664, 69875.0 / 102672, -2260.0 / 8211, 0.25},
};

// Workspace: FP64 vectors (each M doubles, padded to 256 bytes), then the
// Krylov basis V_0..V_m (FP64 or FP32), then the reduction scratch
enum { vK0 = 0, vB = 5, vX, vRX, vR, vXp, vRp, vY, vW, kNumVec };

struct Solver {
  nsk_ctx* c;
  char* base;
  long long M;       // doubles per state vector
  long long stride;  // doubles between workspace vectors
  int m;
  double* part;       // rows of kDotBlocks partial sums
  double* coef;       // a projection's coefficients (device)
  double* host;       // its dot products (pinned)
  hipEvent_t ready;   // host is written
  hipStream_t st;
  Precond pre;
  nsk_implicit_stats* stats;

  int f32;            // Krylov basis in FP32
  double reorth_tol;  // second projection when |w'|^2 <= reorth_tol |w|^2
  long long vstride;  // elements between basis vectors
  double* vec(int k) const { return reinterpret_cast<double*>(base) + (long long)k * stride; }
  template <typename VT>
  VT* V(int k) const {
    return reinterpret_cast<VT*>(reinterpret_cast<double*>(base) + (long long)kNumVec * stride) + (long long)k * vstride;
  }
  unsigned grid() const {
    const long long b = (M + kVecThreads - 1) / kVecThreads;
    return (unsigned)(b < 8192 ? b : 8192);
  }

  // sums of rows 0..nrow-1 and the coefficients of what follows; wait() when
  // the host needs them
  int finish(int nrow, int mode) {
    hipLaunchKernelGGL(dot_final_kernel, dim3(1), dim3(kFinalThreads), 0, st, part, nrow, mode, reorth_tol, coef, host);
    if (hipGetLastError() != hipSuccess) return NSK_EHIP;
    return hipEventRecord(ready, st) == hipSuccess ? NSK_OK : NSK_EHIP;
  }

  int wait() { return hipEventSynchronize(ready) == hipSuccess ? NSK_OK : NSK_EHIP; }

  // rows 0..nj-1: <w, V_j>, row nj: <w, w>; with q, w = q's product first
  template <typename VT>
  int dot_basis(double* w, const Jvp<VT>* q, int nj) {
    for (int j0 = 0; j0 < nj; j0 += kLinTerms) {
      const int nn = nj - j0 < kLinTerms ? nj - j0 : kLinTerms;
      const int self = j0 + nn >= nj;
      with_count(nn, [&](auto K) {
        constexpr int NJ = decltype(K)::value;
        if (q && j0 == 0)
          hipLaunchKernelGGL((multidot_kernel<VT, NJ, true>), dim3(kDotBlocks), dim3(kVecThreads), 0, st, w, *q,
                             V<VT>(0), vstride, self, M, part);
        else
          hipLaunchKernelGGL((multidot_kernel<VT, NJ, false>), dim3(kDotBlocks), dim3(kVecThreads), 0, st, w,
                             Jvp<VT>{}, V<VT>(j0), vstride, self, M, part + (long long)j0 * kDotBlocks);
      });
    }
    return hipGetLastError() == hipSuccess ? NSK_OK : NSK_EHIP;
  }

  // the basis vector V_nk (or w again, and for nk <= kLinTerms its products) from
  // w and V_0..V_{nk-1}, by the device's coefficients
  template <typename VT>
  int orth(double* w, int nk, double s) {
    int j0 = 0;
    for (; nk - j0 > kLinTerms; j0 += kLinTerms)
      hipLaunchKernelGGL(accumulate_kernel<VT>, dim3(grid()), dim3(kVecThreads), 0, st, w, coef, j0, V<VT>(j0), vstride,
                         M);
    with_count(nk - j0, [&](auto K) {
      const unsigned b = grid() > kDotBlocks ? grid() : kDotBlocks;
      hipLaunchKernelGGL((orth_kernel<VT, decltype(K)::value>), dim3(b), dim3(kVecThreads), 0, st, w, coef, j0,
                         V<VT>(j0), vstride, V<VT>(nk), vec(vX), s, pre, vec(vXp), M, j0 == 0 ? part : nullptr);
    });
    return hipGetLastError() == hipSuccess ? NSK_OK : NSK_EHIP;
  }

  // X += P^{-1} sum_{j < nk} a_j V_j; the partial sums of more than one launch are held in vY
  template <typename VT>
  int correct(int nk, const double* a) {
    for (int j0 = 0; j0 < nk; j0 += kLinTerms) {
      const int nn = nk - j0 < kLinTerms ? nk - j0 : kLinTerms;
      BasisCoefs cf;
      std::memset(&cf, 0, sizeof(cf));
      for (int j = 0; j < nn; ++j) cf.a[j] = a[j0 + j];
      with_count(nn, [&](auto K) {
        hipLaunchKernelGGL((correct_kernel<VT, decltype(K)::value>), dim3(grid()), dim3(kVecThreads), 0, st,
                           j0 ? vec(vY) : nullptr, V<VT>(j0), vstride, cf, j0 + nn < nk ? vec(vY) : nullptr, vec(vX),
                           pre, M);
      });
    }
    return hipGetLastError() == hipSuccess ? NSK_OK : NSK_EHIP;
  }

  int rhs(const double* X, double* R) {
    ++stats->rhs_evals;
    return nsk_rhs(c, X, R, 0.0);
  }

  int gmres(double dtg, double beta, double xnorm, double rtol, int* iters) {
    return f32 ? gmres_t<float>(dtg, beta, xnorm, rtol, iters) : gmres_t<double>(dtg, beta, xnorm, rtol, iters);
  }

  // One GMRES cycle for (I - dtg J) P^{-1} y = r, r in vR with norm beta (its
  // reciprocal is the device's coefficient); X += P^{-1} V y.
  template <typename VT>
  int gmres_t(double dtg, double beta, double xnorm, double rtol, int* iters) {
    int rc = NSK_OK;
    *iters = 0;
    if (!(beta > 0.0)) return NSK_OK;
    const double s = std::sqrt(2.2204460492503131e-16) * (1.0 + xnorm);
    if ((rc = orth<VT>(vec(vR), 0, s))) return rc;
    std::vector<double> H((size_t)(m + 1) * m, 0.0), cs(m), sn(m), g(m + 1, 0.0), h(m + 2), h2(m + 2);
    g[0] = beta;
    int kd = 0;
    for (int k = 0; k < m; ++k) {
      if ((rc = rhs(vec(vXp), vec(vRp)))) return rc;
      double* w = vec(vW);
      const Jvp<VT> q{V<VT>(k), vec(vRp), vec(vRX), dtg / s, pre};
      // classical Gram-Schmidt: one multi-dot gives <w, V_0..V_k> and |w|^2
      // together; the subtraction and the normalisation into V_{k+1} are one
      // combination, launched before the host has read the products
      if ((rc = dot_basis<VT>(w, &q, k + 1)) || (rc = finish(k + 2, kFirst)) || (rc = orth<VT>(w, k + 1, s)) ||
          (rc = wait()))
        return rc;
      double hk1 = host[k + 2];
      const bool again = host[k + 3] != 0.0;
      for (int j = 0; j <= k; ++j) { h[j] = host[j]; h2[j] = 0.0; }
      if (again) {
        if (k + 1 > kLinTerms && (rc = dot_basis<VT>(w, nullptr, k + 1))) return rc;
        if ((rc = finish(k + 2, kSecond)) || (rc = orth<VT>(w, k + 1, s)) || (rc = wait())) return rc;
        hk1 = host[k + 2];
        for (int j = 0; j <= k; ++j) h2[j] = host[j];
        ++stats->reorth;
      }
      for (int j = 0; j <= k; ++j) H[(size_t)j * m + k] = h[j] + h2[j];
      H[(size_t)k * m + k] += 1.0;  // A = I + B
      H[(size_t)(k + 1) * m + k] = hk1;
      // Givens rotations on the new column
      for (int j = 0; j < k; ++j) {
        const double t0 = H[(size_t)j * m + k], t1 = H[(size_t)(j + 1) * m + k];
        H[(size_t)j * m + k] = cs[j] * t0 + sn[j] * t1;
        H[(size_t)(j + 1) * m + k] = -sn[j] * t0 + cs[j] * t1;
      }
      const double a0 = H[(size_t)k * m + k], a1 = H[(size_t)(k + 1) * m + k];
      const double r = std::hypot(a0, a1);
      cs[k] = r > 0.0 ? a0 / r : 1.0;
      sn[k] = r > 0.0 ? a1 / r : 0.0;
      H[(size_t)k * m + k] = r;
      H[(size_t)(k + 1) * m + k] = 0.0;
      g[k + 1] = -sn[k] * g[k];
      g[k] = cs[k] * g[k];
      kd = k + 1;
      ++stats->gmres_iters;
      if (std::fabs(g[k + 1]) <= rtol * beta || !(hk1 > 0.0)) break;
    }
    // back substitution and the correction X += P^{-1} sum_j y_j V_j
    std::vector<double> y(kd);
    for (int i = kd - 1; i >= 0; --i) {
      double t = g[i];
      for (int j = i + 1; j < kd; ++j) t -= H[(size_t)i * m + j] * y[j];
      y[i] = t / H[(size_t)i * m + i];
    }
    *iters = kd;
    return correct<VT>(kd, y.data());
  }
};

size_t vec_stride(const nsk_ctx* c) {
  const size_t M = (size_t)c->nvar * c->S;
  return (M + 31) / 32 * 32;
}

// doubles taken by the Krylov basis of gmres_m + 1 vectors (either precision)
size_t basis_doubles(const nsk_ctx* c, int gmres_m) { return (size_t)(gmres_m + 1) * vec_stride(c); }

int check_opts(const nsk_implicit_opts* o) {
  if (!o) return NSK_EINVAL;
  if (!(o->newton_tol > 0.0) || !std::isfinite(o->newton_tol) || o->newton_max < 1 || o->newton_max > 1000)
    return NSK_EINVAL;
  if (!(o->gmres_rtol > 0.0) || !(o->gmres_rtol < 1.0) || o->gmres_m < 1 || o->gmres_m > NSK_GMRES_MAX)
    return NSK_EINVAL;
  if (o->precond != 0 && o->precond != 1) return NSK_EINVAL;
  if (o->basis_fp32 != 0 && o->basis_fp32 != 1) return NSK_EINVAL;
  if (!(o->reorth_tol >= 0.0 && o->reorth_tol < 1.0)) return NSK_EINVAL;
  return NSK_OK;
}

}  // namespace

extern "C" {

size_t nsk_implicit_workspace_bytes(const nsk_ctx* c, int gmres_m) {
  if (!c || gmres_m < 1 || gmres_m > NSK_GMRES_MAX) return 0;
  return sizeof(double) * ((size_t)kNumVec * vec_stride(c) + basis_doubles(c, gmres_m) +
                           (size_t)kDotBlocks * (gmres_m + 3) + 256);
}

int nsk_esdirk_step(nsk_ctx* c, void* d_iwork, double dt, int nsteps, const nsk_implicit_opts* opts,
                    nsk_implicit_stats* stats_out) {
  if (!c || !d_iwork || nsteps < 0 || !(dt > 0.0) || !std::isfinite(dt)) return NSK_EINVAL;
  int rc = check_opts(opts);
  if (rc) return rc;
  if ((reinterpret_cast<uintptr_t>(d_iwork) & 255) != 0) return NSK_EINVAL;
  // finite-difference Jacobian products need FP64 right-hand sides
  // FV sub-cell right-hand sides switch elements and limit slopes: not differentiable
  if (c->par.precision != 0 || c->par.closure != 0 || c->par.subcell != 0) return NSK_EUNSUPPORTED;
  if (opts->precond == 1 && c->par.model != 0) return NSK_EINVAL;  // the relaxation source is model II's
  if (!c->bound) return NSK_EUNBOUND;
  if (c->cur != 0) return NSK_EINVAL;

  nsk_implicit_stats stats;
  std::memset(&stats, 0, sizeof(stats));
  stats.converged = 1;
  Solver S;
  S.c = c;
  S.base = static_cast<char*>(d_iwork);
  S.M = (long long)c->nvar * c->S;
  S.stride = (long long)vec_stride(c);
  S.m = opts->gmres_m;
  S.f32 = opts->basis_fp32;
  S.reorth_tol = opts->reorth_tol;
  S.vstride = S.stride;  // elements of either precision (an FP32 basis fills half its region)
  S.part = reinterpret_cast<double*>(S.base) + (long long)kNumVec * S.stride + (long long)basis_doubles(c, S.m);
  S.coef = S.part + (long long)kDotBlocks * (S.m + 2);  // the last of m + 3 rows; sums take m + 1, or 2
  S.st = c->stream;
  if (!c->sync_host) {
    void* h = nullptr;
    if (hipHostMalloc(&h, sizeof(double) * (NSK_GMRES_MAX + 4), hipHostMallocMapped | hipHostMallocCoherent) !=
        hipSuccess)
      return NSK_EHIP;
    c->sync_host = static_cast<double*>(h);
  }
  if (!c->sync_event && hipEventCreateWithFlags(&c->sync_event, hipEventDisableTiming) != hipSuccess) {
    c->sync_event = nullptr;
    return NSK_EHIP;
  }
  S.host = c->sync_host;
  S.ready = c->sync_event;
  S.stats = &stats;
  const double dtg = dt * kGamma;
  S.pre.on = opts->precond;
  S.pre.ci = c->dim + 1;
  S.pre.a = dtg * c->par.alpha / c->par.beta;
  S.pre.S = c->S;

  double* U = c->U;
  for (int step = 0; step < nsteps && rc == NSK_OK; ++step) {
    if ((rc = S.rhs(U, S.vec(vK0)))) break;
    for (int i = 1; i < 6 && rc == NSK_OK; ++i) {
      // B = U + dt sum_{j<i} a_ij K_j, K_{i-1} = (X - B)/(dt gamma) for i > 1,
      // the predictor X = B + dt gamma K_{i-1}, and |B|^2
      LinArgs L;
      std::memset(&L, 0, sizeof(L));
      int nx = 0;
      L.x[nx] = U;
      L.a[nx++] = 1.0;
      for (int j = 0; j + 1 < i; ++j)
        if (kA[i][j] != 0.0) { L.x[nx] = S.vec(vK0 + j); L.a[nx++] = dt * kA[i][j]; }
      const double ak = dt * kA[i][i - 1];
      if (i == 1) {
        hipLaunchKernelGGL((stage_start_kernel<1, false>), dim3(kDotBlocks), dim3(kVecThreads), 0, S.st, L, ak, dtg,
                           S.vec(vK0), S.vec(vB), S.vec(vX), S.M, S.part);
      } else {
        with_count(nx, [&](auto K) {
          hipLaunchKernelGGL((stage_start_kernel<decltype(K)::value, true>), dim3(kDotBlocks), dim3(kVecThreads), 0,
                             S.st, L, ak, dtg, S.vec(vK0 + i - 1), S.vec(vB), S.vec(vX), S.M, S.part);
        });
      }
      if ((rc = S.finish(1, kSums)) || (rc = S.wait())) break;
      const double bnorm = std::sqrt(S.host[0]);
      bool conv = false;
      double res = 0.0;
      for (int it = 0; it <= opts->newton_max; ++it) {
        if ((rc = S.rhs(S.vec(vX), S.vec(vRX)))) break;
        hipLaunchKernelGGL(residual_kernel, dim3(kDotBlocks), dim3(kVecThreads), 0, S.st, S.vec(vB), S.vec(vRX),
                           S.vec(vX), dtg, S.vec(vR), S.M, S.part);
        if ((rc = S.finish(2, kSums)) || (rc = S.wait())) break;
        const double rn = std::sqrt(S.host[0]), xnorm = std::sqrt(S.host[1]);
        res = rn / (bnorm > 0.0 ? bnorm : 1.0);
        if (!std::isfinite(rn)) { rc = NSK_ENONPHYS; break; }
        if (res <= opts->newton_tol) { conv = true; break; }
        if (it == opts->newton_max) break;
        int gi = 0;
        if ((rc = S.gmres(dtg, rn, xnorm, opts->gmres_rtol, &gi))) break;
        ++stats.newton_iters;
      }
      if (rc) break;
      if (res > stats.max_residual) stats.max_residual = res;
      if (!conv) { stats.converged = 0; rc = NSK_ENOCONV; break; }
    }
    if (rc) break;
    // stiffly accurate: U_{n+1} is the last stage
    if (hipMemcpyAsync(U, S.vec(vX), sizeof(double) * S.M, hipMemcpyDeviceToDevice, S.st) != hipSuccess) {
      rc = NSK_EHIP;
      break;
    }
    ++stats.steps;
  }
  if (hipStreamSynchronize(S.st) != hipSuccess && rc == NSK_OK) rc = NSK_EHIP;
  if (stats_out) *stats_out = stats;
  return rc;
}

}  // extern "C"
