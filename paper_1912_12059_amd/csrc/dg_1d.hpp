// The stage kernels' work in 1D, included by dg_kernels.hpp.  A 1D element has
// one line and few nodes, and a launch is all latency: one thread per
// (element, node) and one per (element, face), so that no thread has more
// than one line's sums to form in turn.  (One lane per line, the form for 2D and
// 3D, took 10.3 us a stage against 8.1 here at N = 5 on 900 elements, 8.0 against
// 4.0 where the whole mesh is one workgroup.)  The operations on a value and their
// order are one in all 1D kernels, so that they give the same bits; unlike the line
// kernels in FP64, which start a line from its faces' terms, these add them last.
#pragma once

namespace nsk {

// One workgroup's elements: own[k] (-1: none) and the two neighbours.
template <int EPB>
struct Elems1D {
  int own[EPB], nb[EPB][2];
  double h2[EPB];
};

template <int EPB>
__device__ __forceinline__ void fill_elems(Elems1D<EPB>& x, const MeshArgs& m, int L, int tid,
                                           const int* __restrict__ skip) {
  if (tid < EPB) {
    const int pos = L * EPB + tid;
    int e = pos < m.E ? m.order[pos] : -1;
    // elements on FV sub-cells are updated by their own kernel: treat them as absent
    if (skip && e >= 0 && skip[e]) e = -1;
    x.own[tid] = e;
    if (e >= 0) {
      x.h2[tid] = m.h2[0][e];
      x.nb[tid][0] = e == 0 ? m.nel[0] - 1 : e - 1;
      x.nb[tid][1] = e == m.nel[0] - 1 ? 0 : e + 1;
    }
  }
}

// Lifting (see lift_block).
template <int NP, int EPB, typename R, typename GT, int MODEL>
__device__ __forceinline__ void lift_block_1d(int L, int tid, const double* __restrict__ U, GT* __restrict__ G,
                                              const BasisArgs& bas, const MeshArgs& msh, const PhysArgs& ph,
                                              double* __restrict__ lfpart) {
  constexpr int NV = MODEL == 1 ? 2 : 3, SI = MODEL == 1 ? 0 : 2, T = Tile<1, NP, EPB>::THREADS;
  __shared__ R sW[3][2][EPB * NP];  // primitives (v, s) of the element before, the own one and the one after
  __shared__ R sWs[2][2][EPB];      // central face values w*
  __shared__ R sD[NP][NP];
  __shared__ Elems1D<EPB> el;
  const long long S = msh.S;
  const auto& B = bas.of(R());
  if (tid < NP * NP) sD[tid / NP][tid % NP] = B.Dhat[tid / NP][tid % NP];
  fill_elems<EPB>(el, msh, L, tid, nullptr);
  __syncthreads();
  const int k = tid / NP, i = tid - k * NP;
  const int e = k < EPB ? el.own[k] : -1;
  double lfs = 0.0;
  if (e >= 0) {
    double u[3][NV];
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      const long long o = (long long)(s == 1 ? e : el.nb[k][s / 2]) * NP + i;
#pragma unroll
      for (int v = 0; v < NV; ++v) u[s][v] = U[v * S + o];
    }
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      const double irho = 1.0 / u[s][0];
      sW[s][0][tid] = R(u[s][1] * irho);
      sW[s][1][tid] = R(u[s][SI]);
    }
    if constexpr (MODEL == 1) lfs = lf_node_speed<1>(u[1], ph.T);
  }
  if constexpr (MODEL == 1) {
    __shared__ double sRed[(T + 63) / 64];
    if (lfpart) block_max_store<T>(lfs, sRed, lfpart + L, tid);
  }
  __syncthreads();
  if (tid < 2 * EPB && el.own[tid / 2] >= 0) {
    const int q = tid / 2, s = tid & 1;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      R wl = R(0), wr = R(0);
#pragma unroll
      for (int l = 0; l < NP; ++l) {
        wl += B.Lp[l] * sW[s][c][q * NP + l];
        wr += B.Lm[l] * sW[s + 1][c][q * NP + l];
      }
      sWs[s][c][q] = R(0.5) * (wl + wr);
    }
  }
  __syncthreads();
  if (e >= 0) {
    R qd[2];
    const R h2 = R(el.h2[k]);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      R vol = R(0);
#pragma unroll
      for (int l = 0; l < NP; ++l) vol += sD[i][l] * sW[1][c][k * NP + l];
      const R surf = (B.Lp[i] * sWs[1][c][k] - B.Lm[i] * sWs[0][c][k]) * B.invw[i];
      qd[c] = h2 * (surf - vol);
    }
    R div = R(0);
    div += qd[0];
    const R eps = R(ph.eps);
    R t = eps * (qd[0] + qd[0]);
    t -= eps * R(2.0 / 3.0) * div;
    const long long o = (long long)e * NP + i;
    G[o] = GT(t);
    G[S + o] = GT(qd[1]);
  }
}

// Second lifting of the original NSK path (see lap_block).
template <int NP, int EPB>
__device__ __forceinline__ void lap_block_1d(int L, int tid, const double* __restrict__ U, double* __restrict__ G,
                                             const BasisArgs& bas, const MeshArgs& msh, const PhysArgs& ph) {
  __shared__ double sg[3][EPB * NP];
  __shared__ double sgs[2][EPB];
  __shared__ double sD[NP][NP];
  __shared__ Elems1D<EPB> el;
  const long long S = msh.S;
  const auto& B = bas.d;
  if (tid < NP * NP) sD[tid / NP][tid % NP] = B.Dhat[tid / NP][tid % NP];
  fill_elems<EPB>(el, msh, L, tid, nullptr);
  __syncthreads();
  const int k = tid / NP, i = tid - k * NP;
  const int e = k < EPB ? el.own[k] : -1;
  double g = 0.0;
  if (e >= 0) {
#pragma unroll
    for (int s = 0; s < 3; ++s) sg[s][tid] = G[S + (long long)(s == 1 ? e : el.nb[k][s / 2]) * NP + i];
    g = sg[1][tid];
  }
  __syncthreads();
  if (tid < 2 * EPB && el.own[tid / 2] >= 0) {
    const int q = tid / 2, s = tid & 1;
    double a = 0.0, b = 0.0;
#pragma unroll
    for (int l = 0; l < NP; ++l) {
      a += B.Lp[l] * sg[s][q * NP + l];
      b += B.Lm[l] * sg[s + 1][q * NP + l];
    }
    sgs[s][q] = 0.5 * (a + b);
  }
  __syncthreads();
  if (e >= 0) {
    double vol = 0.0, lap = 0.0;
#pragma unroll
    for (int l = 0; l < NP; ++l) vol += sD[i][l] * sg[1][k * NP + l];
    const double surf = (B.Lp[i] * sgs[1][k] - B.Lm[i] * sgs[0][k]) * B.invw[i];
    lap += el.h2[k] * (surf - vol);
    const long long o = (long long)e * NP + i;
    const double iso = ph.kappa * (U[o] * lap + 0.5 * (g * g));
    double t = G[o] - ph.kappa * g * g;
    t += iso;
    G[o] = t;
  }
}

// Right-hand side and fused Runge-Kutta stage (see rhs_block).
template <int NP, int EPB, typename R, typename GT, int FLUX, int MODEL>
__device__ __forceinline__ void rhs_block_1d(int L, int tid, const double* __restrict__ U, const GT* __restrict__ G,
                                             double* __restrict__ Uout, double* __restrict__ dU, const BasisArgs& bas,
                                             const MeshArgs& msh, const PhysArgs& ph, const StageArgs& st) {
  constexpr int NV = MODEL == 1 ? 2 : 3;   // conserved variables
  constexpr int NVX = MODEL == 1 ? 1 : 2;  // viscous flux components: tau or Sigma, grad c
  constexpr bool MIXED = sizeof(R) != sizeof(double);
  __shared__ R sX[3][NV + NVX][EPB * NP];  // U and viscous components: before, own, after
  __shared__ double sRho64[MIXED ? 3 : 1][MIXED ? EPB * NP : 1];  // FP64 densities (mixed precision only)
  __shared__ R sF[NV][EPB * NP];           // nodal flux
  __shared__ R sFs[2][NV][EPB];            // numerical flux on the two faces
  __shared__ R sD[NP][NP];
  __shared__ Elems1D<EPB> el;
  const long long S = msh.S;
  const auto& B = bas.of(R());
  if (tid < NP * NP) sD[tid / NP][tid % NP] = B.Dhat[tid / NP][tid % NP];
  fill_elems<EPB>(el, msh, L, tid, st.skip);
  __syncthreads();
  const int k = tid / NP, i = tid - k * NP;
  const int e = k < EPB ? el.own[k] : -1;
  const long long o = (long long)(e >= 0 ? e : 0) * NP + i;
  const R kb = R(ph.kb);
  const R lam_g = FLUX == 2 ? R(*st.lf) : R(0);  // global Lax-Friedrichs speed
  double u64[NV], du_old[NV];
  R g[NVX];
#pragma unroll
  for (int v = 0; v < NV; ++v) du_old[v] = 0.0;
  if (e >= 0) {
    double x[3][NV];
    R y[3][NVX];
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      const long long on = (long long)(s == 1 ? e : el.nb[k][s / 2]) * NP + i;
#pragma unroll
      for (int v = 0; v < NV; ++v) x[s][v] = U[v * S + on];
#pragma unroll
      for (int c = 0; c < NVX; ++c) y[s][c] = R(G[c * S + on]);
    }
    if (st.mode == 1 && st.A != 0.0) {
#pragma unroll
      for (int v = 0; v < NV; ++v) du_old[v] = dU[v * S + o];
    }
#pragma unroll
    for (int s = 0; s < 3; ++s) {
#pragma unroll
      for (int v = 0; v < NV; ++v) sX[s][v][tid] = R(x[s][v]);
#pragma unroll
      for (int c = 0; c < NVX; ++c) sX[s][NV + c][tid] = y[s][c];
      if (MIXED) sRho64[MIXED ? s : 0][MIXED ? tid : 0] = x[s][0];
    }
    R u[NV], F[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      u64[v] = x[1][v];
      u[v] = R(u64[v]);
    }
#pragma unroll
    for (int c = 0; c < NVX; ++c) g[c] = y[1][c];
    conv_flux<1, R, NV>(0, u, R(1) / u[0], p_alpha_guarded<R>(u64[0], ph), F);
    F[1] -= g[0];
    if constexpr (MODEL == 0) F[2] -= kb * g[1];
#pragma unroll
    for (int v = 0; v < NV; ++v) sF[v][tid] = F[v];
  }
  __syncthreads();
  if (tid < 2 * EPB && el.own[tid / 2] >= 0) {
    const int q = tid / 2, s = tid & 1;
    R uL[NV], uR[NV], vL[NVX], vR[NVX], Fs[NV];
    double rL = 0.0, rR = 0.0;
#pragma unroll
    for (int v = 0; v < NV; ++v) uL[v] = uR[v] = R(0);
#pragma unroll
    for (int c = 0; c < NVX; ++c) vL[c] = vR[c] = R(0);
#pragma unroll
    for (int l = 0; l < NP; ++l) {
      const int a = q * NP + l;
      rL += bas.d.Lp[l] * (MIXED ? sRho64[MIXED ? s : 0][MIXED ? a : 0] : double(sX[s][0][a]));
      rR += bas.d.Lm[l] * (MIXED ? sRho64[MIXED ? s + 1 : 0][MIXED ? a : 0] : double(sX[s + 1][0][a]));
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        uL[v] += B.Lp[l] * sX[s][v][a];
        uR[v] += B.Lm[l] * sX[s + 1][v][a];
      }
#pragma unroll
      for (int c = 0; c < NVX; ++c) {
        vL[c] += B.Lp[l] * sX[s][NV + c][a];
        vR[c] += B.Lm[l] * sX[s + 1][NV + c][a];
      }
    }
#pragma unroll
    for (int c = 0; c < NVX; ++c) vL[c] += vR[c];
    face_flux<1, R, FLUX, MODEL, 0, NV, NVX>(uL, uR, vL, rL, rR, lam_g, kb, ph, Fs);
#pragma unroll
    for (int v = 0; v < NV; ++v) sFs[s][v][q] = Fs[v];
  }
  __syncthreads();
  if (e >= 0) {
    const R h2 = R(el.h2[k]);
    double Rv[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      R vol = R(0), acc = R(0);
#pragma unroll
      for (int l = 0; l < NP; ++l) vol += sD[i][l] * sF[v][k * NP + l];
      acc += h2 * (vol - (B.wp[i] * sFs[1][v][k] - B.wm[i] * sFs[0][v][k]));
      Rv[v] = double(acc);
    }
    if constexpr (MODEL == 0) {
      Rv[1] += ph.alpha * u64[0] * double(g[1]);
      Rv[2] += ph.ab * (u64[0] - u64[2]);
      if (st.closure) {
        Rv[1] += double(st.closure[o]);
        Rv[2] += double(st.closure[S + o]);
      }
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      if (st.mode == 0) {
        Uout[v * S + o] = Rv[v];
      } else {
        const double du = st.A * du_old[v] + st.dt * Rv[v];
        dU[v * S + o] = du;
        Uout[v * S + o] = u64[v] + st.B * du;
      }
    }
  }
}

// -------------------------------------------------------------------------
// Whole Runge-Kutta steps in one launch (model II).  A workgroup holds up to
// LE elements, a thread per node, and keeps their state and register in
// vector registers over the five stages of a step; LDS carries what
// neighbouring threads read.  An element's stage depends on the two elements
// on either side, so a mesh of more than LE elements is cut into ranges that
// overlap by kHalo1D = 10 elements at each end: the values at the ends of a
// workgroup's range are wrong, two elements deeper with every stage, and only
// the inner ones are written, one step a launch.  A mesh that fits runs all its
// steps in one launch, periodic inside the workgroup.
//
// The operations on a value and their order are those of the stage kernels,
// so the bits are the same.  What goes is the launches, two a stage, and the
// memory round trips: 64 elements, N = 3, FP64: 1.3 us a stage, 3.1 us with the
// stage kernels' work run in one workgroup through memory; 900 elements: 2.5
// us, 7.2 us as two launches a stage.  Bound by the chain of one stage: four
// barriers, and one lane's line sums between them.
// -------------------------------------------------------------------------
constexpr int kSteps1DThreads = 512;
constexpr int kHalo1D = 10;
template <int NP>
constexpr int kSteps1DElems = kSteps1DThreads / NP;

struct RkCoefs {
  double A[5], B[5];
};

// U1 <- nsteps steps from U0 (a single workgroup may have both the same: a
// thread reads and writes only its own node).  local: elements of a workgroup; halo: 0 (one
// workgroup, the whole mesh) or kHalo1D (nsteps = 1).
template <int NP, typename R, int FLUX>
__global__ void __launch_bounds__(kSteps1DThreads)
steps_kernel_1d(const double* U0, double* U1, double* dU, BasisArgs bas, MeshArgs msh, PhysArgs ph,
                RkCoefs rk, double dt, int nsteps, int local, int halo) {
  constexpr bool MIXED = sizeof(R) != sizeof(double);
  constexpr int T = kSteps1DThreads, LE = kSteps1DElems<NP>;
  __shared__ R sU[3][T], sW[2][T], sG[2][T], sF[3][T];
  __shared__ double sRho64[MIXED ? T : 1];
  __shared__ R sWs[2][LE + 1], sFs[3][LE + 1];  // face f: between local elements f - 1 and f
  __shared__ R sD[NP][NP], sL[5][NP];
  const auto& B = bas.of(R());
  const int tid = threadIdx.x, k = tid / NP, i = tid - k * NP;
  if (tid < NP * NP) sD[tid / NP][tid % NP] = B.Dhat[tid / NP][tid % NP];
  if (tid < NP) {
    sL[0][tid] = B.Lm[tid];
    sL[1][tid] = B.Lp[tid];
    sL[2][tid] = B.invw[tid];
    sL[3][tid] = B.wm[tid];
    sL[4][tid] = B.wp[tid];
  }
  const int E = msh.E, own = local - 2 * halo, first = (int)blockIdx.x * own;
  const bool node = k < local;
  int e = first + k - halo;
  if (e < 0) e += E;
  if (e >= E) e -= E;
  // the last range may reach round past its own start
  e = node ? e % E : 0;
  const long long S = msh.S, o = (long long)e * NP + i;
  double u[3] = {1.0, 0.0, 1.0}, du[3] = {0.0, 0.0, 0.0};
  R h2 = R(0);
  if (node) {
#pragma unroll
    for (int v = 0; v < 3; ++v) u[v] = U0[v * S + o];
    h2 = R(msh.h2[0][e]);
  }
  __syncthreads();
  R D[NP];
#pragma unroll
  for (int l = 0; l < NP; ++l) D[l] = sD[i][l];
  const R Lm = sL[0][i], Lp = sL[1][i], iw = sL[2][i], wm = sL[3][i], wp = sL[4][i];
  const R kb = R(ph.kb), eps = R(ph.eps);
  const bool face = tid < local;              // face tid, the left one of element tid
  const int le = tid == 0 ? local - 1 : tid - 1;  // the element before it
  const int fr = k + 1 < local ? k + 1 : 0;   // the element's right face
  const int line = k * NP;

  for (int step = 0; step < nsteps; ++step) {
    du[0] = du[1] = du[2] = 0.0;
#pragma nounroll
    for (int s = 0; s < 5; ++s) {
      if (node) {
        const double irho = 1.0 / u[0];
        sW[0][tid] = R(u[1] * irho);
        sW[1][tid] = R(u[2]);
#pragma unroll
        for (int v = 0; v < 3; ++v) sU[v][tid] = R(u[v]);
        if (MIXED) sRho64[MIXED ? tid : 0] = u[0];
      }
      __syncthreads();
      if (face) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          R wl = R(0), wr = R(0);
#pragma unroll
          for (int l = 0; l < NP; ++l) {
            wl += B.Lp[l] * sW[c][le * NP + l];
            wr += B.Lm[l] * sW[c][tid * NP + l];
          }
          sWs[c][tid] = R(0.5) * (wl + wr);
        }
      }
      __syncthreads();
      R gc = R(0);
      if (node) {
        R qd[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          R vol = R(0);
#pragma unroll
          for (int l = 0; l < NP; ++l) vol += D[l] * sW[c][line + l];
          const R surf = (Lp * sWs[c][fr] - Lm * sWs[c][k]) * iw;
          qd[c] = h2 * (surf - vol);
        }
        R div = R(0);
        div += qd[0];
        R t = eps * (qd[0] + qd[0]);
        t -= eps * R(2.0 / 3.0) * div;
        gc = qd[1];
        sG[0][tid] = t;
        sG[1][tid] = gc;
        R ur[3], Fn[3];
#pragma unroll
        for (int v = 0; v < 3; ++v) ur[v] = R(u[v]);
        conv_flux<1, R, 3>(0, ur, R(1) / ur[0], p_alpha_guarded<R>(u[0], ph), Fn);
        Fn[1] -= t;
        Fn[2] -= kb * gc;
#pragma unroll
        for (int v = 0; v < 3; ++v) sF[v][tid] = Fn[v];
      }
      __syncthreads();
      if (face) {
        R uL[3], uR[3], vL[2], vR[2], Fs[3];
        double rL = 0.0, rR = 0.0;
#pragma unroll
        for (int v = 0; v < 3; ++v) uL[v] = uR[v] = R(0);
#pragma unroll
        for (int c = 0; c < 2; ++c) vL[c] = vR[c] = R(0);
#pragma unroll
        for (int l = 0; l < NP; ++l) {
          const int a = le * NP + l, b = tid * NP + l;
          rL += bas.d.Lp[l] * (MIXED ? sRho64[MIXED ? a : 0] : double(sU[0][a]));
          rR += bas.d.Lm[l] * (MIXED ? sRho64[MIXED ? b : 0] : double(sU[0][b]));
#pragma unroll
          for (int v = 0; v < 3; ++v) {
            uL[v] += B.Lp[l] * sU[v][a];
            uR[v] += B.Lm[l] * sU[v][b];
          }
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            vL[c] += B.Lp[l] * sG[c][a];
            vR[c] += B.Lm[l] * sG[c][b];
          }
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) vL[c] += vR[c];
        face_flux<1, R, FLUX, 0, 0, 3, 2>(uL, uR, vL, rL, rR, R(0), kb, ph, Fs);
#pragma unroll
        for (int v = 0; v < 3; ++v) sFs[v][tid] = Fs[v];
      }
      __syncthreads();
      if (node) {
        double Rv[3];
#pragma unroll
        for (int v = 0; v < 3; ++v) {
          R vol = R(0), acc = R(0);
#pragma unroll
          for (int l = 0; l < NP; ++l) vol += D[l] * sF[v][line + l];
          acc += h2 * (vol - (wp * sFs[v][fr] - wm * sFs[v][k]));
          Rv[v] = double(acc);
        }
        Rv[1] += ph.alpha * u[0] * double(gc);
        Rv[2] += ph.ab * (u[0] - u[2]);
#pragma unroll
        for (int v = 0; v < 3; ++v) {
          du[v] = rk.A[s] * du[v] + dt * Rv[v];
          u[v] = u[v] + rk.B[s] * du[v];
        }
      }
    }
  }
  if (node && k >= halo && k < local - halo && first + k - halo < E) {
#pragma unroll
    for (int v = 0; v < 3; ++v) {
      U1[v * S + o] = u[v];
      dU[v * S + o] = du[v];
    }
  }
}

}  // namespace nsk
