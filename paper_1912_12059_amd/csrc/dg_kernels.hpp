// Device kernels of the DGSEM right-hand side for relaxation model II
// (Hitz, Keim, Munz, Rohde, Sec. 2.3 for the model, Sec. 3.1 for the scheme),
// written for gfx950 (64-wide wavefronts, 160 KB LDS per CU, 8 XCDs with a
// private 4 MB L2 each).
//
// One stage of the explicit scheme is two launches:
//   lift_kernel : state U -> G, where G holds per node the viscous stress
//                 tau (symmetric, dim(dim+1)/2 entries) and grad c, both built
//                 from the BR1-lifted gradients of the primitives (v, c)
//   rhs_kernel  : U, G -> volume integral + Rusanov/BR1 surface integral +
//                 pointwise source, then either R (dU/dt) or the fused
//                 low-storage Runge-Kutta stage update of U and the register.
//
// Work layout.  A workgroup owns EPB elements; its threads take node pairs and
// element lines in turn (see "Work of one workgroup" below; 1D has its own
// layout, dg_1d.hpp).  With Gauss-Legendre nodes the element ends are not
// nodes, so a face trace needs every node of the neighbour's line.  Each face
// value is computed identically by both elements sharing it (same operands,
// same order), so the scheme stays conservative bit for bit.
//
// Element order.  Which elements a workgroup owns comes from a host-built
// table.  The hardware hands consecutive workgroups to the XCDs in turn;
// renumbering the workgroups so that each XCD walks one contiguous range of
// that table, and building the table so that each range is a set of x-y tiles
// marched along z, keeps the neighbour re-reads inside the XCD's L2.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace nsk {

constexpr int kMaxNP = 7;  // N <= 6

template <int B, int E>
struct ipow { static constexpr int v = B * ipow<B, E - 1>::v; };
template <int B>
struct ipow<B, 0> { static constexpr int v = 1; };

__host__ __device__ constexpr int cmax(int a, int b) { return a > b ? a : b; }
__host__ __device__ constexpr int cmin(int a, int b) { return a < b ? a : b; }

// f(std::integral_constant<int, 0>), ..., f(std::integral_constant<int, K-1>)
template <int K, int I = 0, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < K) {
    f(std::integral_constant<int, I>{});
    static_for<K, I + 1>(f);
  }
}
constexpr int round64(int x) { return ((x + 63) / 64) * 64; }

template <int DIM, int NP>
struct Shape {
  static constexpr int NN = ipow<NP, DIM>::v;          // nodes per element
  static constexpr int NF = ipow<NP, DIM - 1>::v;      // nodes per face
  static constexpr int NVAR = DIM + 2;                 // rho, m, c
  static constexpr int NLIFT = DIM + 1;                // v, c
  static constexpr int NTAU = DIM * (DIM + 1) / 2;     // symmetric stress
  static constexpr int NG = NTAU + DIM;                // tau + grad c
};

// stride of Gauss index along direction d inside an element
template <int NP>
__host__ __device__ constexpr int dstride(int d) { return d == 0 ? 1 : (d == 1 ? NP : NP * NP); }

// Index of tau_{ij} (i, j < DIM) inside the packed symmetric storage:
// diagonal first, then (0,1), (0,2), (1,2).
template <int DIM>
__host__ __device__ constexpr int tau_index(int i, int j) {
  if (i == j) return i;
  int a = i < j ? i : j, b = i < j ? j : i;
  if (DIM == 2) return 2;
  return a == 0 ? (b == 1 ? 3 : 4) : 5;
}

// Constants of the 1D basis and the geometry, passed by value.
template <typename R>
struct BasisOf {
  R Dhat[kMaxNP][kMaxNP];  // weak-form derivative operator
  R Lm[kMaxNP], Lp[kMaxNP];  // Lagrange polynomials at xi = -1, +1
  R invw[kMaxNP];          // 1 / Gauss weight
  R wp[kMaxNP], wm[kMaxNP];  // Lp / weight, Lm / weight
};

struct BasisArgs {
  BasisOf<double> d;
  BasisOf<float> f;        // the same rounded to FP32
  __host__ __device__ const BasisOf<double>& of(double) const { return d; }
  __host__ __device__ const BasisOf<float>& of(float) const { return f; }
};

struct MeshArgs {
  const double* h2[3];  // 2 / h per element index along each direction
  const int* order;     // element of each position of the work order
  int nel[3];
  int E;                // number of elements
  long long S;          // E * NN, stride between variables
  int nxcd;             // XCDs sharing the work order in contiguous ranges
  int stream;           // kStreamState, kStreamG: arrays that pass the caches by
};

// Arrays that the next kernel will not find in the last-level cache (256 MB) are
// written without a place in it (and the old dU read so), which leaves the caches
// to the neighbours' lines.  The lines lie, by the bytes of the two states, dU and
// G together, where both sides are equal: ms a stage without / with, 3D N = 4 FP64
// 0.114 / 0.121 at 197 MB, 0.232 / 0.214 at 384 MB, N = 2 0.111 / 0.128 at 228 MB,
// mixed 0.181 / 0.174 at 312 MB, 2D N = 4 0.120 / 0.129 at 267 MB.  G in FP64 from a
// larger size on, as the next kernel reads it at once: 0.214 / 0.221 at 384 MB (state
// and dU streamed in both), 0.378 / 0.367 at 664 MB; in FP32 it is left alone.
constexpr int kStreamState = 1, kStreamG = 2;
constexpr double kStreamStateBytes = 288e6, kStreamGBytes = 512e6;
inline int stream_bits(double bytes) {
  return (bytes > kStreamStateBytes ? kStreamState : 0) | (bytes > kStreamGBytes ? kStreamG : 0);
}

struct PhysArgs {
  double T, eps, kappa, alpha, beta;
  double kb;         // kappa / beta
  double ab;         // alpha / beta
  int diss_c;        // numerical-flux dissipation on c
  int flux;          // 0: Rusanov, 1: HLLC, 2: global Lax-Friedrichs
  double rho_lo64, rho_hi64;  // mixed precision: FP64 EoS inside this band
};

struct StageArgs {
  double A, B, dt;   // low-storage coefficients of the stage and step size
  int mode;          // 0: write R; 1: Runge-Kutta stage update
  const float* closure = nullptr;  // learned closure source [dim+1][elem][node], or none
  const double* lf = nullptr;      // global Lax-Friedrichs speed (original NSK path)
  const int* skip = nullptr;       // elements left to the FV sub-cell kernel (flag per element)
};

// -------------------------------------------------------------------------
// Thermodynamics of the reduced Van-der-Waals fluid (Sec. 2.1)
//   p = 8 T rho / (3 - rho) - 3 rho^2,   p' = 24 T / (3 - rho)^2 - 6 rho
// Model II modified pressure p_alpha = p + alpha rho^2 / 2 and sound speed
// a = sqrt(p_alpha') = sqrt(p' + alpha rho) (Sec. 2.3).
// -------------------------------------------------------------------------
template <typename R>
__device__ __forceinline__ R p_alpha(R rho, R T, R alpha) {
  const R q = R(1) / (R(3) - rho);
  return R(8) * T * rho * q - R(3) * rho * rho + R(0.5) * alpha * rho * rho;
}

template <typename R>
__device__ __forceinline__ R sound_speed(R rho, R T, R alpha) {
  const R q = R(1) / (R(3) - rho);
  return sqrt(R(24) * T * q * q - R(6) * rho + alpha * rho);
}

// p_alpha and a together, sharing the reciprocal 1/(3 - rho)
template <typename R>
__device__ __forceinline__ void p_alpha_sound(R rho, R T, R alpha, R& pa, R& a) {
  const R q = R(1) / (R(3) - rho);
  pa = R(8) * T * rho * q - R(3) * rho * rho + R(0.5) * alpha * rho * rho;
  a = sqrt(R(24) * T * q * q - R(6) * rho + alpha * rho);
}

// EoS in the working precision R, except inside the spinodal band where the
// Van-der-Waals pressure is evaluated in FP64 (mixed-precision rule).
template <typename R>
__device__ __forceinline__ bool eos_in_fp64(double rho64, const PhysArgs& ph) {
  return sizeof(R) == sizeof(double) || (rho64 > ph.rho_lo64 && rho64 < ph.rho_hi64);
}

template <typename R>
__device__ __forceinline__ R p_alpha_guarded(double rho64, const PhysArgs& ph) {
  if (eos_in_fp64<R>(rho64, ph)) return R(p_alpha<double>(rho64, ph.T, ph.alpha));
  return p_alpha<R>(R(rho64), R(ph.T), R(ph.alpha));
}

template <typename R>
__device__ __forceinline__ void p_alpha_sound_guarded(double rho64, const PhysArgs& ph, R& pa, R& a) {
  if (eos_in_fp64<R>(rho64, ph)) {
    double p64, a64;
    p_alpha_sound<double>(rho64, ph.T, ph.alpha, p64, a64);
    pa = R(p64);
    a = R(a64);
  } else {
    p_alpha_sound<R>(R(rho64), R(ph.T), R(ph.alpha), pa, a);
  }
}

// Hardware hands consecutive workgroups to the XCDs in turn; renumber them
// so that XCD x works through one contiguous range of the work order.
__device__ __forceinline__ int remap_block(int b, int G, int nx) {
  if (nx <= 1) return b;
  const int q = G / nx, r = G - (G / nx) * nx;
  const int x = b % nx, i = b / nx;
  return x < r ? x * (q + 1) + i : r * (q + 1) + (x - r) * q + i;
}

// node with Gauss index 0 along d on the line of face node f
template <int NP>
__device__ __forceinline__ int face_base(int d, int f) {
  const int sd = dstride<NP>(d);
  return (f % sd) + sd * NP * (f / sd);
}

// face node of node n for direction d
template <int NP>
__device__ __forceinline__ int face_of(int d, int n) {
  const int sd = dstride<NP>(d);
  return (n % sd) + sd * (n / (sd * NP));
}

// Convective flux in direction d; irho = 1/rho; NV = DIM + 2 (model II, c
// not convected) or DIM + 1 (original NSK).
template <int DIM, typename R, int NV = DIM + 2>
__device__ __forceinline__ void conv_flux(int d, const R* u, R irho, R pa, R* F) {
  const R vd = u[1 + d] * irho;
  F[0] = u[1 + d];
#pragma unroll
  for (int j = 0; j < DIM; ++j) F[1 + j] = vd * u[1 + j] + (j == d ? pa : R(0));
  if constexpr (NV == DIM + 2) F[DIM + 1] = R(0);
}

// Original NSK path: the speed of the global Lax-Friedrichs flux at a node,
// max_d |v_d| + sqrt(max(p', 0)) (the sound speed is imaginary inside the
// spinodal interval).
template <int DIM>
__device__ __forceinline__ double lf_node_speed(const double* u, double T) {
  const double rho = u[0], q = 1.0 / (3.0 - rho);
  const double dp = 24.0 * T * q * q - 6.0 * rho;
  const double a = dp > 0.0 ? sqrt(dp) : 0.0;
  double m = 0.0;
#pragma unroll
  for (int d = 0; d < DIM; ++d) m = fmax(m, fabs(u[1 + d] / rho));
  return m + a;
}

// Maximum of v over the workgroup, written by thread 0 to *out (all threads
// call it).
template <int THREADS>
__device__ __forceinline__ void block_max_store(double v, double* red, double* out, int tid) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off));
  if ((tid & 63) == 0) red[tid >> 6] = v;
  __syncthreads();
  if (tid == 0) {
    double m = red[0];
    for (int w = 1; w < (THREADS + 63) / 64; ++w) m = fmax(m, red[w]);
    *out = m;
  }
}

// -------------------------------------------------------------------------
// Work of one workgroup (2D and 3D).  A workgroup owns EPB elements in two roles:
//   node role: a thread per pair of neighbouring nodes of an element: loads
//     the pair's values, puts them into LDS, and at the end combines the
//     directions' contributions and writes the pair's results;
//   line role: the waves are given to the directions in turn, and a lane
//     takes one (element, d-line): it forms the traces of the two neighbours'
//     d-lines, the face values of both ends of its line and the line's
//     contraction with the derivative matrix, all in registers (the matrix is
//     uniform, in scalar registers), and leaves NP values per component in LDS.
// All directions run at once, so a stage is three phases with two or three
// barriers, where one direction after the other takes seven; a contraction
// reads each value from LDS once instead of NP times; and only the element's
// own values stay in LDS, 16 a node in 3D instead of the 40 of staging whole
// neighbours beside them.  In 3D three waves serve two elements at N = 4.
// What bounds the 3D kernels at N = 4 now is the neighbours: without their loads
// the right-hand side runs at the rate of its streams (1.42 ms for 6.6 GB).  It is
// the L1's line requests that count: in the FP64 right-hand side at 96x48x48 elements
// 133 M lines of 128 bytes a launch at 69 in flight a CU and 560 cycles each, 44 % of
// the time stalled on pending lines; more waves a SIMD, or half as many load
// instructions for the same lines, change nothing.
//
// Measured, ms a launch, one direction after the other / this form with the fewer
// registers and the streamed stores of below (without those two the FP64 right-hand
// side took 2.04 and the lifting 1.11 ms, the mixed right-hand side 1.71):
//   3D N = 4, 96x48x48, FP64    lift 1.19 / 1.04   rhs 2.55 / 1.89
//   3D N = 4, 96x48x48, mixed   lift 0.85 / 0.76   rhs 1.82 / 1.66
//   a stage: 3D N = 2, 96x48x48, FP64 1.17 / 0.70; N = 5, 48x24x24, mixed 0.83 / 0.57;
//   2D N = 4, 96x96, FP64 0.0376 / 0.0245
// -------------------------------------------------------------------------
// LDS position of node n of an element: even for even n, so that a pair of
// values is one 16-byte access; the planes of lines of 2 or 4 nodes are padded
// by two, so that the lanes of a wave reading lines of any direction meet at
// most two to a bank.
template <int NP>
__host__ __device__ constexpr int lds_slot(int n) { return NP == 2 || NP == 4 ? n + 2 * (n / (NP * NP)) : n; }

// Distance in LDS between neighbouring nodes of a d-line.
template <int NP>
__device__ __forceinline__ constexpr int lds_step(int d) {
  return d == 2 && (NP == 2 || NP == 4) ? NP * NP + 2 : dstride<NP>(d);
}

// Forms of the line role: a lane a line, two lanes a line (LineEnd), or a lane a
// line with the neighbours staged through LDS (NbPairs).
constexpr int kLines = 0, kEnds = 1, kStaged = 2;

template <int DIM, int NP, int EPB, int FORM = kLines>
struct Tile {
  using Sh = Shape<DIM, NP>;
  static constexpr int LPE = (FORM == kEnds ? 2 : 1) * Sh::NF;  // lanes of an element in the line role
  static_assert(LPE <= 64, "a wave takes whole elements");
  static constexpr int EPW = cmin(EPB, 64 / LPE);          // elements of one wave in the line role
  static constexpr int WPD = (EPB + EPW - 1) / EPW;        // waves per direction in the line role
  static constexpr int NPC = (Sh::NN + 1) / 2;             // node pairs per element
  static constexpr int THREADS = cmax(round64(EPB * NPC), 64 * DIM * WPD);
  static constexpr int RPC = (EPW * NPC + 63) / 64;        // rounds in which a wave takes its elements' pairs
  // LDS values per element and component: even, and off the bank period
  static constexpr int PN = (lds_slot<NP>(Sh::NN - 1) + 2) / 2 * 2 +
                            (NP == 2 || NP == 3 || (DIM == 2 && (NP == 4 || NP == 5)) ? 2 : 0);
  static constexpr int SL = EPB * PN;
};

// In 1D a thread per node and one per face (dg_1d.hpp).
template <int NP, int EPB>
struct Tile<1, NP, EPB, kLines> {
  static constexpr int THREADS = round64(EPB * NP);
};

// Two neighbouring values of one component, 16 bytes a lane in FP64: the unit
// of whole-element loads and stores (the L1 takes 20 cycles for the 125
// values of an element this way, 35 with one value a lane).
template <typename T>
struct __attribute__((packed, aligned(sizeof(T)))) Pair {
  T a, b;
};

// Pair p of an element's NN values.  The last pair of an odd number holds
// the last value alone (in both places: it is loaded one value early).
template <int NN>
__host__ __device__ constexpr bool pair_solo(int p) { return NN % 2 != 0 && p == NN / 2; }
template <int NN, typename T>
__device__ __forceinline__ Pair<T> load_pair(const T* elem, int p) {
  const bool solo = pair_solo<NN>(p);
  Pair<T> x = *reinterpret_cast<const Pair<T>*>(elem + 2 * p - (solo ? 1 : 0));
  if (solo) x.a = x.b;
  return x;
}
template <int NN, typename T>
__device__ __forceinline__ void store_pair(T* elem, int p, T a, T b) {
  if (pair_solo<NN>(p))
    elem[2 * p] = a;
  else
    *reinterpret_cast<Pair<T>*>(elem + 2 * p) = Pair<T>{a, b};
}

// The same past the caches (nontemporal).
typedef double DoublePair __attribute__((ext_vector_type(2), aligned(8)));
template <int NN>
__device__ __forceinline__ Pair<double> load_pair_nt(const double* elem, int p) {
  const bool solo = pair_solo<NN>(p);
  const DoublePair x = __builtin_nontemporal_load(reinterpret_cast<const DoublePair*>(elem + 2 * p - (solo ? 1 : 0)));
  return Pair<double>{solo ? x.y : x.x, x.y};
}
template <int NN>
__device__ __forceinline__ void store_pair_nt(double* elem, int p, double a, double b) {
  if (pair_solo<NN>(p))
    __builtin_nontemporal_store(a, elem + 2 * p);
  else
    __builtin_nontemporal_store(DoublePair{a, b}, reinterpret_cast<DoublePair*>(elem + 2 * p));
}

// The same in LDS (even positions; the second value of a lone last one
// falls into the padding).
template <typename R>
struct alignas(2 * sizeof(R)) LdsPair {
  R a, b;
};
template <typename R>
__device__ __forceinline__ void lds_put(R* p, R a, R b) {
  *reinterpret_cast<LdsPair<R>*>(p) = LdsPair<R>{a, b};
}
template <typename R>
__device__ __forceinline__ LdsPair<R> lds_get(const R* p) {
  return *reinterpret_cast<const LdsPair<R>*>(p);
}

// Node role of a thread: element slot el of the workgroup and pair p of its
// nodes, at sl in LDS.
template <int DIM, int NP, int EPB>
struct NodeRole {
  using Tl = Tile<DIM, NP, EPB>;
  int el, p, sl;
  __device__ __forceinline__ explicit NodeRole(int tid) {
    el = tid / Tl::NPC;
    p = tid - el * Tl::NPC;
    sl = el * Tl::PN + lds_slot<NP>(2 * p);
  }
};

// LDS written by some lanes of a wave and read by others: the LDS operations
// of one wave execute in order, so only the compiler has to keep the order.
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// x, but unknown to the compiler: what is computed from it is not kept from
// an earlier use of x
__device__ __forceinline__ int opaque(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// coordinate of element e along d
template <int d>
__device__ __forceinline__ int elem_coord(const MeshArgs& m, int e) {
  const unsigned n0 = unsigned(m.nel[0]);
  if constexpr (d == 0) return int(unsigned(e) % n0);
  const unsigned q = unsigned(e) / n0;
  if constexpr (d == 1) return int(q % unsigned(m.nel[1]));
  return int(q / unsigned(m.nel[1]));
}

// Line role of a thread: the waves are given to the directions in turn, a
// lane takes one d-line: element slot el, element e (-1: none), its two
// d-neighbours, face node f, the line's first node and 2/h.
struct LineRole {
  int el = 0, e = -1, f = 0, base = 0;
  int end = 0;  // with kEnds the end of the line that the lane takes: 0 xi = -1, 1 xi = +1
  int nb[2] = {0, 0};
  double h2 = 0.0;
};

template <int DIM, int NP, int EPB, int d, int FORM = kLines>
__device__ __forceinline__ LineRole line_role(const MeshArgs& m, int L, int sub, int lane,
                                              const int* __restrict__ skip) {
  using Tl = Tile<DIM, NP, EPB, FORM>;
  constexpr int NF = Shape<DIM, NP>::NF;
  LineRole r;
  const int k = lane / Tl::LPE;
  r.f = lane - k * Tl::LPE;
  if constexpr (FORM == kEnds) {
    r.end = r.f >= NF ? 1 : 0;
    r.f -= r.end * NF;
  }
  r.el = sub * Tl::EPW + k;
  const int pos = L * EPB + r.el;
  if (k >= Tl::EPW || r.el >= EPB || pos >= m.E) return r;
  const int e = m.order[pos];
  if (skip && skip[e]) return r;
  r.e = e;
  const int c = elem_coord<d>(m, e);
  const int step = d == 0 ? 1 : (d == 1 ? m.nel[0] : m.nel[0] * m.nel[1]);
  r.nb[0] = c == 0 ? e + (m.nel[d] - 1) * step : e - step;
  r.nb[1] = c == m.nel[d] - 1 ? e - (m.nel[d] - 1) * step : e + step;
  r.base = face_base<NP>(d, r.f);
  r.h2 = m.h2[d][c];
  return r;
}

// How a wave gets its neighbours' lines.  Mostly its lanes read them straight
// from memory.  A line's values along x and y lie apart, which costs the L1 44
// cycles an element and component instead of the 20 of whole elements read a
// pair a lane; staging whole neighbours through LDS for that (kStaged, into rows that
// the own values take afterwards) needs one more barrier and twice the LDS
// traffic.  It wins where the lines are long, LDS values are four bytes and the mesh
// is large (Staged in host_common.hpp); it gains nothing at N = 3 (0.79 ms both) and
// loses at N = 2 (0.63 against 0.60) and in FP64 (N = 4 1.03 against 0.95, N = 2 0.83
// against 0.70).

// Places of a wave's neighbour pairs, round by round: the pair p and its
// position at in LDS (-1: none), and the two neighbours.
template <int DIM, int NP, int EPB>
struct NbPairs {
  using Tl = Tile<DIM, NP, EPB>;
  int p[Tl::RPC], at[Tl::RPC];
  int nb[2][Tl::RPC];
  __device__ __forceinline__ NbPairs(const LineRole& ln, int sub, int lane, int (*sNb)[2]) {
    constexpr int NF = Shape<DIM, NP>::NF;
    if (lane < NF * Tl::EPW && ln.f == 0 && ln.el < EPB) {
      sNb[ln.el][0] = ln.e >= 0 ? ln.nb[0] : -1;
      sNb[ln.el][1] = ln.nb[1];
    }
    wave_fence();
#pragma unroll
    for (int r = 0; r < Tl::RPC; ++r) {
      const int pc = lane + 64 * r, k = pc / Tl::NPC, pe = sub * Tl::EPW + k;
      p[r] = pc - k * Tl::NPC;
      nb[0][r] = sNb[cmin(pe, EPB - 1)][0];
      nb[1][r] = sNb[cmin(pe, EPB - 1)][1];
      at[r] = k < Tl::EPW && pe < EPB && nb[0][r] >= 0 ? pe * Tl::PN + lds_slot<NP>(2 * p[r]) : -1;
    }
  }
};

// Two lanes a line (kEnds).  One lane's chain, the loads of two neighbours' lines,
// two fluxes and a contraction with every row, is the time of a launch that leaves
// most of the chip idle (2D N = 6, 14x7 elements, FP64: lift 7.0 and rhs 10.5 us,
// with two lanes 5.5 and 7.8; one direction after the other, a thread a node, took 5.1
// and 8.1).  There each end of a line has a lane of its own, which
// loads that end's neighbour (every load issued at once: registers are free),
// forms that end's face values and, with the other end's by a shuffle, half of the
// rows of the contraction: in the middle row of an odd number both lanes get the
// same value.  The operations on a value and their order are those of one lane a
// line, so the bits are the same.
template <int NP>
struct LineEnd {
  static constexpr int H = (NP + 1) / 2;  // rows of a lane
  bool hi;                                // the end xi = +1
  int row0;                               // its first row
  __device__ __forceinline__ explicit LineEnd(int end) : hi(end != 0), row0(end ? NP - H : 0) {}
  // weights of the neighbour's and of the own trace at this end
  template <typename T>
  __device__ __forceinline__ T nb(const BasisOf<T>& B, int l) const { return hi ? B.Lm[l] : B.Lp[l]; }
  template <typename T>
  __device__ __forceinline__ T own(const BasisOf<T>& B, int l) const { return hi ? B.Lp[l] : B.Lm[l]; }
  // a value of both ends from the lanes' own
  template <int NF, typename T>
  __device__ __forceinline__ void both(T x, int lane, T& lo, T& up) const {
    const T y = __shfl(x, hi ? lane - NF : lane + NF, 64);
    lo = hi ? y : x;
    up = hi ? x : y;
  }
};

// What row i of a contraction takes, for lanes of different rows: the derivative
// matrix's row, then the K weights w_k[i] (in LDS: selecting between two scalar
// copies of them cost 130 spilled scalar registers at N = 6).
template <int NP, int K, bool ON, typename R>
struct RowTable {
  static constexpr int W = NP + K;
  R v[ON ? NP : 1][ON ? W : 1];
  __device__ __forceinline__ void fill(int tid, const BasisOf<R>& B, const R* const (&w)[K]) {
    if constexpr (ON) {
      if (tid < NP * NP) v[tid / NP][tid % NP] = B.Dhat[tid / NP][tid % NP];
      if (tid < NP) {
#pragma unroll
        for (int k = 0; k < K; ++k) v[tid][NP + k] = w[k][tid];
      }
    }
  }
};

// x[v][l] = p[v * S + l * ST]: NVAL lines of a d-neighbour
template <int NVAL, int NP, int ST, typename T>
__device__ __forceinline__ void load_lines(const T* __restrict__ p, long long S, T (&x)[NVAL][NP]) {
#pragma unroll
  for (int v = 0; v < NVAL; ++v)
#pragma unroll
    for (int l = 0; l < NP; ++l) x[v][l] = p[v * S + l * ST];
}

// -------------------------------------------------------------------------
// Lifting: G = (tau, grad s) from the BR1 gradients of (v, s), s = c for
// model II (MODEL 0) and s = rho for the original NSK path (MODEL 1):
//   q_d,i = (2/h_d) [ (L+_i w*_+ - L-_i w*_-) / omega_i - sum_l Dhat_il w_l ]
// along each d-line, w* = (w_left + w_right) / 2 on the faces.
// -------------------------------------------------------------------------
template <int DIM, int NP, int EPB, typename R, typename GT, int MODEL, int FORM>
__device__ __forceinline__ void lift_block_lines(int L, int tid, const double* __restrict__ U, GT* __restrict__ G,
                                                 const BasisArgs& bas, const MeshArgs& msh, const PhysArgs& ph,
                                                 double* __restrict__ lfpart) {
  using Sh = Shape<DIM, NP>;
  using Tl = Tile<DIM, NP, EPB, FORM>;
  constexpr int NN = Sh::NN, NL = Sh::NLIFT, SL = Tl::SL, PN = Tl::PN;
  constexpr int NV = MODEL == 1 ? DIM + 1 : DIM + 2;  // conserved variables
  constexpr int SI = MODEL == 1 ? 0 : DIM + 1;        // the lifted scalar: rho or c
  __shared__ __attribute__((aligned(16))) R sW[NL][SL];        // nodal primitives (v, s)
  __shared__ __attribute__((aligned(16))) R sX[DIM][NL][SL];   // per direction: gradients before the factor 2/h
  constexpr bool ENDS = FORM == kEnds, STAGE = FORM == kStaged;
  __shared__ double sH2[EPB][DIM];
  __shared__ int sNb[DIM][STAGE ? EPB : 1][2];
  __shared__ RowTable<NP, 3, ENDS, R> sT;

  const long long S = msh.S;
  const auto& B = bas.of(R());
  sT.fill(tid, B, {B.Lp, B.Lm, B.invw});
  const NodeRole<DIM, NP, EPB> nr(tid);
  const int pos = L * EPB + nr.el;
  const bool active = nr.el < EPB && pos < msh.E;
  const long long o = active ? (long long)msh.order[pos] * NN : 0;
  Pair<double> u[NV];
  if (active) {
#pragma unroll
    for (int v = 0; v < NV; ++v) u[v] = load_pair<NN>(U + v * S + o, nr.p);
  }

  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int dir = wv / Tl::WPD;
  const int sub = wv - dir * Tl::WPD, lane = tid & 63;
  // the neighbours' traces: the weights of xi = +1 before the element, of xi = -1 after it
  R wn[2][NL];  // with kEnds wn[0]: that of the lane's end
  double x1[ENDS ? NV : 1][NP];  // and its neighbour's line
  LineRole ln;
  static_for<DIM>([&](auto dc) {
    constexpr int d = decltype(dc)::value;
    if (dir != d) return;
    ln = line_role<DIM, NP, EPB, d, FORM>(msh, L, sub, lane, nullptr);
    if (ln.e >= 0 && ln.f == 0) sH2[ln.el][d] = ln.h2;
    if constexpr (STAGE) {
      const NbPairs<DIM, NP, EPB> np(ln, sub, lane, sNb[d]);
      const int b0 = ln.el * PN + lds_slot<NP>(ln.base);
      static_for<2>([&](auto sc) {
        constexpr int s = decltype(sc)::value;
        Pair<double> x[Tl::RPC][NV];
#pragma unroll
        for (int r = 0; r < Tl::RPC; ++r)
          if (np.at[r] >= 0) {
#pragma unroll
            for (int v = 0; v < NV; ++v) x[r][v] = load_pair<NN>(U + v * S + (long long)np.nb[s][r] * NN, np.p[r]);
          }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < Tl::RPC; ++r)
          if (np.at[r] >= 0) {
            const double ia = 1.0 / x[r][0].a, ib = 1.0 / x[r][0].b;
#pragma unroll
            for (int k = 0; k < DIM; ++k) lds_put(&sX[d][k][np.at[r]], R(x[r][1 + k].a * ia), R(x[r][1 + k].b * ib));
            lds_put(&sX[d][DIM][np.at[r]], R(x[r][SI].a), R(x[r][SI].b));
          }
        wave_fence();
        if (ln.e >= 0) {
#pragma unroll
          for (int k = 0; k < NL; ++k) {
            wn[s][k] = R(0);
#pragma unroll
            for (int l = 0; l < NP; ++l) wn[s][k] += (s ? B.Lm[l] : B.Lp[l]) * sX[d][k][b0 + l * lds_step<NP>(d)];
          }
        }
        wave_fence();
      });
      return;
    }
    if (ln.e < 0) return;
    if constexpr (ENDS) {
      load_lines<NV, NP, dstride<NP>(d)>(U + (long long)(ln.end ? ln.nb[1] : ln.nb[0]) * NN + ln.base, S, x1);
      __builtin_amdgcn_sched_barrier(0);
      return;
    }
    // every load of a line is issued before the first value is used
    static_for<2>([&](auto sc) {
      constexpr int s = decltype(sc)::value;
      double x[NV][NP];
      load_lines<NV, NP, dstride<NP>(d)>(U + (long long)ln.nb[s] * NN + ln.base, S, x);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 0; k < NL; ++k) wn[s][k] = R(0);
#pragma unroll
      for (int l = 0; l < NP; ++l) {
        const double irho = 1.0 / x[0][l];
        const R lw = s ? B.Lm[l] : B.Lp[l];
#pragma unroll
        for (int k = 0; k < DIM; ++k) wn[s][k] += lw * R(x[1 + k][l] * irho);
        wn[s][DIM] += lw * R(x[SI][l]);
      }
    });
  });

  double lfs = 0.0;  // global Lax-Friedrichs speed at this pair (MODEL 1)
  if (active) {
    const double ia = 1.0 / u[0].a, ib = 1.0 / u[0].b;
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      lds_put(&sW[d][nr.sl], R(u[1 + d].a * ia), R(u[1 + d].b * ib));
    }
    lds_put(&sW[DIM][nr.sl], R(u[SI].a), R(u[SI].b));
    if constexpr (MODEL == 1) {
      double ua[NV], ub[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) { ua[v] = u[v].a; ub[v] = u[v].b; }
      lfs = fmax(lf_node_speed<DIM>(ua, ph.T), lf_node_speed<DIM>(ub, ph.T));
    }
  }
  if constexpr (ENDS) {
    if (ln.e >= 0) {
      const LineEnd<NP> end(ln.end);
#pragma unroll
      for (int k = 0; k < NL; ++k) wn[0][k] = R(0);
#pragma unroll
      for (int l = 0; l < NP; ++l) {
        const double irho = 1.0 / x1[0][l];
        const R lw = end.nb(B, l);
#pragma unroll
        for (int k = 0; k < DIM; ++k) wn[0][k] += lw * R(x1[1 + k][l] * irho);
        wn[0][DIM] += lw * R(x1[SI][l]);
      }
    }
  }
  if constexpr (MODEL == 1) {
    __shared__ double sRed[(Tl::THREADS + 63) / 64];
    if (lfpart) block_max_store<Tl::THREADS>(lfs, sRed, lfpart + L, tid);
  }
  __syncthreads();

  static_for<DIM>([&](auto dc) {
    constexpr int d = decltype(dc)::value;
    if (dir != d || ln.e < 0) return;
    const int b0 = ln.el * PN + lds_slot<NP>(ln.base);
    if constexpr (ENDS) {
      const LineEnd<NP> end(ln.end);
#pragma unroll
      for (int k = 0; k < NL; ++k) {
        R w[NP], wo = R(0), wsm, wsp;
#pragma unroll
        for (int l = 0; l < NP; ++l) {
          w[l] = sW[k][b0 + l * lds_step<NP>(d)];
          wo += end.own(B, l) * w[l];
        }
        end.template both<Sh::NF>(R(0.5) * (wo + wn[0][k]), lane, wsm, wsp);
#pragma unroll
        for (int r = 0; r < end.H; ++r) {
          R vol = R(0);
#pragma unroll
          for (int l = 0; l < NP; ++l) vol += sT.v[end.row0 + r][l] * w[l];
          const R* const x = &sT.v[end.row0 + r][NP];
          const R surf = (x[0] * wsp - x[1] * wsm) * x[2];
          sX[d][k][b0 + (end.row0 + r) * lds_step<NP>(d)] = surf - vol;
        }
      }
      return;
    }
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      R w[NP], wl = R(0), wr = R(0);
#pragma unroll
      for (int l = 0; l < NP; ++l) {
        w[l] = sW[k][b0 + l * lds_step<NP>(d)];
        wl += B.Lp[l] * w[l];
        wr += B.Lm[l] * w[l];
      }
      const R wsm = R(0.5) * (wn[0][k] + wr), wsp = R(0.5) * (wl + wn[1][k]);
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        R vol = R(0);
#pragma unroll
        for (int l = 0; l < NP; ++l) vol += B.Dhat[i][l] * w[l];
        const R surf = (B.Lp[i] * wsp - B.Lm[i] * wsm) * B.invw[i];
        sX[d][k][b0 + i * lds_step<NP>(d)] = surf - vol;
      }
    }
  });
  __syncthreads();

  if (active) {
    R qd[2][DIM][NL], div[2];
    const R eps = R(ph.eps);
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      const R h2 = R(sH2[nr.el][d]);
#pragma unroll
      for (int k = 0; k < NL; ++k) {
        const LdsPair<R> x = lds_get(&sX[d][k][nr.sl]);
        qd[0][d][k] = h2 * x.a;
        qd[1][d][k] = h2 * x.b;
      }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      div[h] = R(0);
#pragma unroll
      for (int d = 0; d < DIM; ++d) div[h] += qd[h][d][d];
    }
    // each component is stored as it is formed: collecting them first changes
    // which products are fused, and so the FP32 roundings
    const bool past = sizeof(GT) == sizeof(double) && (msh.stream & kStreamG);
    auto store_g = [&](int k, GT a, GT b) {
      GT* const g = G + (long long)k * S + o;
      if constexpr (sizeof(GT) == sizeof(double)) {
        if (past) {
          store_pair_nt<NN>(g, nr.p, a, b);
          return;
        }
      }
      store_pair<NN>(g, nr.p, a, b);
    };
#pragma unroll
    for (int a = 0; a < DIM; ++a)
#pragma unroll
      for (int b = a; b < DIM; ++b) {
        R t[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          t[h] = eps * (qd[h][b][a] + qd[h][a][b]);
          if (a == b) t[h] -= eps * R(2.0 / 3.0) * div[h];
        }
        store_g(tau_index<DIM>(a, b), GT(t[0]), GT(t[1]));
      }
#pragma unroll
    for (int d = 0; d < DIM; ++d) store_g(Sh::NTAU + d, GT(qd[0][d][DIM]), GT(qd[1][d][DIM]));
  }
}

// -------------------------------------------------------------------------
// Original NSK path, second BR1 lifting (end of Sec. 3.1): with g = grad rho
// from the first lifting (G slots NTAU..NTAU+DIM-1),
//   lap_i = sum_d (2/h_d) [ (L+_i g*_+ - L-_i g*_-) / omega_i - sum_l Dhat_il g_d,l ],
// g* = (g_left + g_right) / 2 the central face values of g_d on the d-faces;
// then the viscous stress in G's tau slots becomes the full second-order
// stress Sigma = eps tau + kappa ((rho lap + |g|^2/2) I - g g^T) (the
// Korteweg stress of Sec. 2.2 in conservative form).  The gradient slots are
// only read, so neighbouring workgroups see the first lifting's values.
// -------------------------------------------------------------------------
template <int DIM, int NP, int EPB, int FORM>
__device__ __forceinline__ void lap_block_lines(int L, int tid, const double* __restrict__ U, double* __restrict__ G,
                                          const BasisArgs& bas, const MeshArgs& msh, const PhysArgs& ph) {
  using Sh = Shape<DIM, NP>;
  using Tl = Tile<DIM, NP, EPB, FORM>;
  constexpr int NN = Sh::NN, NT = Sh::NTAU, SL = Tl::SL, PN = Tl::PN;
  __shared__ __attribute__((aligned(16))) double sg[DIM][SL];   // own g_d; a d-line's lane overwrites it with the contribution to lap
  __shared__ double sH2[EPB][DIM];
  constexpr bool ENDS = FORM == kEnds;
  __shared__ RowTable<NP, 3, ENDS, double> sT;

  const long long S = msh.S;
  const auto& B = bas.of(double());
  sT.fill(tid, B, {B.Lp, B.Lm, B.invw});
  const NodeRole<DIM, NP, EPB> nr(tid);
  const int pos = L * EPB + nr.el;
  const bool active = nr.el < EPB && pos < msh.E;
  const long long o = active ? (long long)msh.order[pos] * NN : 0;
  Pair<double> g[DIM], tau[NT], rho{0.0, 0.0};
  if (active) {
#pragma unroll
    for (int d = 0; d < DIM; ++d) g[d] = load_pair<NN>(G + (long long)(NT + d) * S + o, nr.p);
#pragma unroll
    for (int k = 0; k < NT; ++k) tau[k] = load_pair<NN>(G + (long long)k * S + o, nr.p);
    rho = load_pair<NN>(U + o, nr.p);
  }

  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int dir = wv / Tl::WPD;
  const int sub = wv - dir * Tl::WPD, lane = tid & 63;
  double gn[2] = {0.0, 0.0};  // with kEnds gn[0]: that of the lane's end
  double x1[1][NP];           // and its neighbour's line
  LineRole ln;
  static_for<DIM>([&](auto dc) {
    constexpr int d = decltype(dc)::value;
    if (dir != d) return;
    ln = line_role<DIM, NP, EPB, d, FORM>(msh, L, sub, lane, nullptr);
    if (ln.e < 0) return;
    if (ln.f == 0) sH2[ln.el][d] = ln.h2;
    if constexpr (ENDS) {
      load_lines<1, NP, dstride<NP>(d)>(
          G + (long long)(NT + d) * S + (long long)(ln.end ? ln.nb[1] : ln.nb[0]) * NN + ln.base, S, x1);
      return;
    }
    double x[2][1][NP];
#pragma unroll
    for (int s = 0; s < 2; ++s)
      load_lines<1, NP, dstride<NP>(d)>(G + (long long)(NT + d) * S + (long long)ln.nb[s] * NN + ln.base, S, x[s]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int l = 0; l < NP; ++l) gn[s] += (s ? B.Lm[l] : B.Lp[l]) * x[s][0][l];
  });
  if (active) {
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      lds_put(&sg[d][nr.sl], g[d].a, g[d].b);
    }
  }
  if constexpr (ENDS) {
    if (ln.e >= 0) {
      const LineEnd<NP> end(ln.end);
#pragma unroll
      for (int l = 0; l < NP; ++l) gn[0] += end.nb(B, l) * x1[0][l];
    }
  }
  __syncthreads();

  static_for<DIM>([&](auto dc) {
    constexpr int d = decltype(dc)::value;
    if (dir != d || ln.e < 0) return;
    const int b0 = ln.el * PN + lds_slot<NP>(ln.base);
    if constexpr (ENDS) {
      const LineEnd<NP> end(ln.end);
      double w[NP], wo = 0.0, gm, gp;
#pragma unroll
      for (int l = 0; l < NP; ++l) {
        w[l] = sg[d][b0 + l * lds_step<NP>(d)];
        wo += end.own(B, l) * w[l];
      }
      end.template both<Sh::NF>(0.5 * (wo + gn[0]), lane, gm, gp);
      wave_fence();  // both lanes have read the line that they overwrite
#pragma unroll
      for (int r = 0; r < end.H; ++r) {
        double vol = 0.0;
#pragma unroll
        for (int l = 0; l < NP; ++l) vol += sT.v[end.row0 + r][l] * w[l];
        const double* const x = &sT.v[end.row0 + r][NP];
        const double surf = (x[0] * gp - x[1] * gm) * x[2];
        sg[d][b0 + (end.row0 + r) * lds_step<NP>(d)] = surf - vol;
      }
      return;
    }
    double w[NP], wl = 0.0, wr = 0.0;
#pragma unroll
    for (int l = 0; l < NP; ++l) {
      w[l] = sg[d][b0 + l * lds_step<NP>(d)];
      wl += B.Lp[l] * w[l];
      wr += B.Lm[l] * w[l];
    }
    const double gm = 0.5 * (wr + gn[0]), gp = 0.5 * (wl + gn[1]);
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      double vol = 0.0;
#pragma unroll
      for (int l = 0; l < NP; ++l) vol += B.Dhat[i][l] * w[l];
      const double surf = (B.Lp[i] * gp - B.Lm[i] * gm) * B.invw[i];
      sg[d][b0 + i * lds_step<NP>(d)] = surf - vol;
    }
  });
  __syncthreads();

  if (active) {
    double iso[2], lap[2] = {0.0, 0.0}, g2[2] = {0.0, 0.0};
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      const LdsPair<double> x = lds_get(&sg[d][nr.sl]);
      lap[0] += sH2[nr.el][d] * x.a;
      lap[1] += sH2[nr.el][d] * x.b;
      g2[0] += g[d].a * g[d].a;
      g2[1] += g[d].b * g[d].b;
    }
    iso[0] = ph.kappa * (rho.a * lap[0] + 0.5 * g2[0]);
    iso[1] = ph.kappa * (rho.b * lap[1] + 0.5 * g2[1]);
#pragma unroll
    for (int a = 0; a < DIM; ++a)
#pragma unroll
      for (int b = a; b < DIM; ++b) {
        const int k = tau_index<DIM>(a, b);
        double ta = tau[k].a - ph.kappa * g[a].a * g[b].a, tb = tau[k].b - ph.kappa * g[a].b * g[b].b;
        if (a == b) {
          ta += iso[0];
          tb += iso[1];
        }
        store_pair<NN>(G + (long long)k * S + o, nr.p, ta, tb);
      }
  }
}

// -------------------------------------------------------------------------
// Right-hand side and fused Runge-Kutta stage:
//   R_i = sum_d (2/h_d) [ sum_l Dhat_il F_d,l - (L+_i F*_+ - L-_i F*_-) / omega_i ] + S_i
// with F_d = Fc_d(U) - Fv_d(G), F* = Rusanov, HLLC or global LF (U-, U+)
// - (Fv(G-) + Fv(G+)) / 2 and S = (0, alpha rho grad c, (alpha/beta)(rho - c))
// (model II); the original NSK path (MODEL 1) has U = (rho, m), the
// second-order stress Sigma in G's tau slots and no source; then
//   dU <- A dU + dt R,  U <- U + B dU.
// -------------------------------------------------------------------------

// Numerical flux of direction d between the traces (uL, vL) and (uR, vR), rL
// and rR the FP64 traces of the density.
template <int DIM, typename R, int FLUX, int MODEL, int d, int NV, int NVX>
__device__ __forceinline__ void face_flux(const R* uL, const R* uR, const R* vLR, double rL, double rR,
                                          R lam_g, R kb, const PhysArgs& ph, R* Fs) {
  R paL, paR, aL = R(0), aR = R(0);
  if constexpr (FLUX == 2) {
    // the global Lax-Friedrichs flux needs no local sound speed
    paL = p_alpha_guarded<R>(rL, ph);
    paR = p_alpha_guarded<R>(rR, ph);
  } else {
    p_alpha_sound_guarded<R>(rL, ph, paL, aL);
    p_alpha_sound_guarded<R>(rR, ph, paR, aR);
  }
  const R irL = R(1) / uL[0], irR = R(1) / uR[0];
  R Fc[NV];
  if constexpr (FLUX == 2) {
    R FL[NV], FR[NV];
    conv_flux<DIM, R, NV>(d, uL, irL, paL, FL);
    conv_flux<DIM, R, NV>(d, uR, irR, paR, FR);
    // global Lax-Friedrichs: one dissipation speed for the whole grid
#pragma unroll
    for (int v = 0; v < NV; ++v) Fc[v] = R(0.5) * (FL[v] + FR[v]) - R(0.5) * lam_g * (uR[v] - uL[v]);
  } else if constexpr (FLUX == 0) {
    // Rusanov: central flux minus the larger wave speed times the jump
    const R vnL = uL[1 + d] * irL, vnR = uR[1 + d] * irR;
    const R sL = fabs(vnL) + aL, sR = fabs(vnR) + aR;
    const R lam = sL > sR ? sL : sR;
    __builtin_amdgcn_sched_barrier(0);
    Fc[0] = R(0.5) * (uL[1 + d] + uR[1 + d]) - R(0.5) * (lam * (uR[0] - uL[0]));
#pragma unroll
    for (int j = 0; j < DIM; ++j) {
      const R FL = vnL * uL[1 + j] + (j == d ? paL : R(0)), FR = vnR * uR[1 + j] + (j == d ? paR : R(0));
      Fc[1 + j] = R(0.5) * (FL + FR) - R(0.5) * (lam * (uR[1 + j] - uL[1 + j]));
    }
    const R dc = lam * (uR[NV - 1] - uL[NV - 1]);
    Fc[NV - 1] = R(0) - R(0.5) * (ph.diss_c ? dc : R(0));
  } else {
    // HLLC of the barotropic convective part: Davis speeds; HLL flux for
    // mass and normal momentum; tangential momenta carried by the mass
    // flux with the velocity of the upwind side of the contact
    // S* = F_hll[rho] / rho_hll; HLL dissipation alone on c
    const R vnL = uL[1 + d] * irL, vnR = uR[1 + d] * irR;
    // How the speeds are rounded is written out, SL from unrounded products and SR from
    // rounded ones: chosen by the compiler it changes with the code around it, and a
    // small v beside a large a then rounds differently in FP32 at one face in a
    // thousand (mixed precision, seven steps, 3D N = 5: 2e-8 of the state).
    const R SL = fmin(fma(uL[1 + d], irL, -aL), fma(uR[1 + d], irR, -aR));
    R SR;
    {
#pragma clang fp contract(off)
      SR = fmax(vnL + aL, vnR + aR);
    }
    // all three cases by selection, a component at a time: branches keep more
    // alive than 168 registers hold at N = 4
    const bool l = SL >= R(0), r = SR <= R(0);
    const R w = R(1) / (SR - SL);
    const R Fm = (SR * uL[1 + d] - SL * uR[1 + d] + SL * SR * (uR[0] - uL[0])) * w;
    const R rh = (SR * uR[0] - SL * uL[0] - (uR[1 + d] - uL[1 + d])) * w;
    __builtin_amdgcn_sched_barrier(0);
    const bool left = Fm / rh >= R(0);
    Fc[0] = l ? uL[1 + d] : (r ? uR[1 + d] : Fm);
#pragma unroll
    for (int j = 0; j < DIM; ++j) {
      const R FL = vnL * uL[1 + j] + (j == d ? paL : R(0)), FR = vnR * uR[1 + j] + (j == d ? paR : R(0));
      const R Fx = j == d ? (SR * FL - SL * FR + SL * SR * (uR[1 + j] - uL[1 + j])) * w
                          : Fm * (left ? uL[1 + j] * irL : uR[1 + j] * irR);
      Fc[1 + j] = l ? FL : (r ? FR : Fx);
    }
    Fc[NV - 1] = l || r || !ph.diss_c ? R(0) : SL * SR * (uR[NV - 1] - uL[NV - 1]) * w;
  }
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    Fs[v] = Fc[v];
    if (v >= 1 && v <= DIM) Fs[v] -= R(0.5) * vLR[v - 1];
    if constexpr (MODEL == 0) {
      if (v == NV - 1) Fs[v] -= R(0.5) * kb * vLR[DIM];
    }
  }
}

constexpr int kLineGroup = 3;

// In 3D at degree 4 in mixed precision the right-hand side has four waves per SIMD,
// five workgroups a CU instead of four: its registers are 131 with the own values
// kept, 99 (two lanes a line) and 103 without.  It counts where a launch has one to two
// rounds of workgroups (us for four steps, three waves / four: two lanes a line,
// 16x9x8 517 / 482; a lane a line, 14x14x14 821 / 796, 32x16x16 both 1674).
template <int DIM, int NP, typename R>
constexpr bool kFourWaves = DIM == 3 && NP == 5 && sizeof(R) == 4;

template <int DIM, int NP, int EPB, typename R, typename GT, int FLUX, int MODEL, int FORM>
__device__ __forceinline__ void rhs_block_lines(int L, int tid, const double* __restrict__ U, const GT* __restrict__ G,
                                          double* __restrict__ Uout, double* __restrict__ dU, const BasisArgs& bas,
                                          const MeshArgs& msh, const PhysArgs& ph, const StageArgs& st) {
  using Sh = Shape<DIM, NP>;
  using Tl = Tile<DIM, NP, EPB, FORM>;
  constexpr int NN = Sh::NN, NT = Sh::NTAU, SL = Tl::SL, PN = Tl::PN;
  constexpr int NV = MODEL == 1 ? DIM + 1 : DIM + 2;   // conserved variables
  constexpr int NG = MODEL == 1 ? NT : Sh::NG;         // G slots read: Sigma, or (tau, grad c)
  constexpr int NVX = MODEL == 1 ? DIM : DIM + 1;      // viscous flux components of one direction
  static_assert(MODEL == 0 || FLUX == 2, "the original NSK path uses the global Lax-Friedrichs flux");
  constexpr bool MIXED = sizeof(R) != sizeof(double);
  // own values: U, G, p_alpha, 1/rho; once every line is in registers the
  // same memory takes the directions' contributions
  constexpr int IP = NV + NG, II = IP + 1;
  constexpr int ROWS = cmax(NV + NG + 2, DIM * NV);
  constexpr bool ENDS = FORM == kEnds, STAGE = FORM == kStaged;
  // A pair's own values stay in registers to the end: 8 of the 81 components that
  // an element asks the L1 for, whose outstanding misses bound this kernel in 3D
  // (96x48x48 elements, N = 4: 2.02 -> 1.96 ms).  They are loaded again where the
  // registers matter more: with staged neighbours (1.80 against 1.74 ms there in mixed
  // precision), and with HLLC in FP64 at N = 1 in 3D (us for two steps, kept / again:
  // 46x23x23 519 / 511, 121x60x60 3764 / 3709, 182x91x91 12581 / 12335; in mixed
  // precision 10227 / 10399 there, in 2D 2394 / 2472 at 1414x707), and where it makes
  // room for a fourth wave (kFourWaves).
  constexpr bool AGAIN = STAGE || kFourWaves<DIM, NP, R> || (DIM == 3 && NP == 2 && FLUX == 1 && !MIXED);
  // With two lanes a line in 2D every load of the kernel is issued before the first
  // is waited for, unless that takes more registers than three waves a SIMD have
  // (N = 6 in FP64: 182; 3D: 204) or a fourth wave (MODEL 1: N = 4, 141x71, a stage
  // 33.2 -> 36.0 us).
  constexpr bool EARLY = ENDS && DIM == 2 && MODEL == 0 && (NP < 7 || MIXED);
  constexpr int RPD = ROWS / DIM;  // rows in which a direction's waves stage neighbours
  static_assert(!STAGE || (RPD >= NV && RPD >= NVX), "staging rows");
  __shared__ __attribute__((aligned(16))) R sIn[ROWS][SL];
  __shared__ __attribute__((aligned(16))) double sRho64[MIXED ? (STAGE ? DIM : 1) : 1][MIXED ? SL : 1];  // FP64 densities (mixed precision only)
  __shared__ int sNb[DIM][STAGE ? EPB : 1][2];
  __shared__ double sH2[EPB][DIM];
  __shared__ int sE[AGAIN ? EPB : 1];  // element of each slot, -1: none
  __shared__ RowTable<NP, 2, ENDS, R> sT;

  const long long S = msh.S;
  const auto& B = bas.of(R());
  sT.fill(tid, B, {B.wm, B.wp});
  const NodeRole<DIM, NP, EPB> nr(tid);
  const int pos = L * EPB + nr.el;
  int e = nr.el < EPB && pos < msh.E ? msh.order[pos] : -1;
  // elements on FV sub-cells are updated by their own kernel: treat them as absent
  if (st.skip && e >= 0 && st.skip[e]) e = -1;
  const R kb = R(ph.kb);
  const R lam_g = FLUX == 2 ? R(*st.lf) : R(0);  // global Lax-Friedrichs speed
  if (AGAIN && nr.el < EPB && nr.p == 0) sE[nr.el] = e;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int dir = wv / Tl::WPD;
  const int sub = wv - dir * Tl::WPD, lane = tid & 63;
  Pair<double> u0[NV];
  Pair<GT> g0[NG];
  auto load_own = [&]() {
    if (e < 0) return;
    const long long o = (long long)e * NN;
#pragma unroll
    for (int v = 0; v < NV; ++v) u0[v] = load_pair<NN>(U + v * S + o, nr.p);
#pragma unroll
    for (int k = 0; k < NG; ++k) g0[k] = load_pair<NN>(G + (long long)k * S + o, nr.p);
  };
  auto put_own = [&]() {
    if (e < 0) return;
#pragma unroll
    for (int v = 0; v < NV; ++v) lds_put(&sIn[v][nr.sl], R(u0[v].a), R(u0[v].b));
#pragma unroll
    for (int k = 0; k < NG; ++k) lds_put(&sIn[NV + k][nr.sl], R(g0[k].a), R(g0[k].b));
    lds_put(&sIn[IP][nr.sl], p_alpha_guarded<R>(u0[0].a, ph), p_alpha_guarded<R>(u0[0].b, ph));
    lds_put(&sIn[II][nr.sl], R(1) / R(u0[0].a), R(1) / R(u0[0].b));
    if (MIXED) lds_put(&sRho64[0][MIXED ? nr.sl : 0], u0[0].a, u0[0].b);
  };
  if constexpr (!STAGE) {
    load_own();
    if constexpr (!EARLY) put_own();
  }

  // line role: the neighbours' traces (with kEnds [0]: that of the lane's end)
  R un[2][NV], vn[2][NVX];
  double rn[2] = {0.0, 0.0};  // density traces in FP64 (EoS guard)
  LineRole ln;
  double xu1[ENDS ? NV : 1][NP];  // with kEnds the neighbour's line
  GT xg1[ENDS ? NVX : 1][NP];
  static_for<DIM>([&](auto dc) {
    constexpr int d = decltype(dc)::value;
    if (dir != d) return;
    ln = line_role<DIM, NP, EPB, d, FORM>(msh, L, sub, lane, st.skip);
    if (ln.e >= 0 && ln.f == 0) sH2[ln.el][d] = ln.h2;
    if constexpr (STAGE) {
      // U, then the viscous components, of each side, in the rows of the
      // direction; the loads run two batches ahead
      const NbPairs<DIM, NP, EPB> np(ln, sub, lane, sNb[d]);
      const int b0 = ln.el * PN + lds_slot<NP>(ln.base);
      Pair<double> xu[Tl::RPC][NV];
      Pair<GT> xg[Tl::RPC][NVX];
      auto load_u = [&](int s) {
#pragma unroll
        for (int r = 0; r < Tl::RPC; ++r)
          if (np.at[r] >= 0) {
#pragma unroll
            for (int v = 0; v < NV; ++v) xu[r][v] = load_pair<NN>(U + v * S + (long long)np.nb[s][r] * NN, np.p[r]);
          }
      };
      auto load_g = [&](int s) {
#pragma unroll
        for (int r = 0; r < Tl::RPC; ++r)
          if (np.at[r] >= 0) {
#pragma unroll
            for (int k = 0; k < NVX; ++k)
              xg[r][k] = load_pair<NN>(
                  G + (long long)(k < DIM ? tau_index<DIM>(k, d) : NT + d) * S + (long long)np.nb[s][r] * NN, np.p[r]);
          }
      };
      auto fold_u = [&](int s) {
#pragma unroll
        for (int r = 0; r < Tl::RPC; ++r)
          if (np.at[r] >= 0) {
#pragma unroll
            for (int v = 0; v < NV; ++v) lds_put(&sIn[d * RPD + v][np.at[r]], R(xu[r][v].a), R(xu[r][v].b));
            if constexpr (MIXED) lds_put(&sRho64[d][np.at[r]], xu[r][0].a, xu[r][0].b);
          }
        wave_fence();
        if (ln.e >= 0) {
#pragma unroll
          for (int v = 0; v < NV; ++v) {
            un[s][v] = R(0);
#pragma unroll
            for (int l = 0; l < NP; ++l)
              un[s][v] += (s ? B.Lm[l] : B.Lp[l]) * sIn[d * RPD + v][b0 + l * lds_step<NP>(d)];
          }
          if constexpr (MIXED) {
#pragma unroll
            for (int l = 0; l < NP; ++l)
              rn[s] += (s ? bas.d.Lm[l] : bas.d.Lp[l]) * sRho64[d][b0 + l * lds_step<NP>(d)];
          }
        }
        wave_fence();
      };
      auto fold_g = [&](int s) {
#pragma unroll
        for (int r = 0; r < Tl::RPC; ++r)
          if (np.at[r] >= 0) {
#pragma unroll
            for (int k = 0; k < NVX; ++k) lds_put(&sIn[d * RPD + k][np.at[r]], R(xg[r][k].a), R(xg[r][k].b));
          }
        wave_fence();
        if (ln.e >= 0) {
#pragma unroll
          for (int k = 0; k < NVX; ++k) {
            vn[s][k] = R(0);
#pragma unroll
            for (int l = 0; l < NP; ++l)
              vn[s][k] += (s ? B.Lm[l] : B.Lp[l]) * sIn[d * RPD + k][b0 + l * lds_step<NP>(d)];
          }
        }
        wave_fence();
      };
      load_u(0);
      load_g(0);
      __builtin_amdgcn_sched_barrier(0);
      fold_u(0);
      load_u(1);
      __builtin_amdgcn_sched_barrier(0);
      fold_g(0);
      load_g(1);
      __builtin_amdgcn_sched_barrier(0);
      fold_u(1);
      fold_g(1);
      return;
    }
    if (ln.e < 0) return;
    if constexpr (ENDS) {
      const long long on = (long long)(ln.end ? ln.nb[1] : ln.nb[0]) * NN + ln.base;
      load_lines<NV, NP, dstride<NP>(d)>(U + on, S, xu1);
#pragma unroll
      for (int k = 0; k < NVX; ++k)
#pragma unroll
        for (int l = 0; l < NP; ++l)
          xg1[k][l] = (G + (long long)(k < DIM ? tau_index<DIM>(k, d) : NT + d) * S + on)[l * dstride<NP>(d)];
      return;
    }
    // components in groups of kLineGroup, the loads of a group issued two
    // groups before their use
    constexpr int NC = NV + NVX, NGRP = (2 * NC + kLineGroup - 1) / kLineGroup;
    double xu[2 * kLineGroup][NP];
    GT xg[2 * kLineGroup][NP];
    static_for<NGRP + 2>([&](auto gc) {
      constexpr int g = decltype(gc)::value;
      static_for<kLineGroup>([&](auto jc) {
        constexpr int it = (g - 2) * kLineGroup + decltype(jc)::value;
        if constexpr (it >= 0 && it < 2 * NC) {
          constexpr int s = it / NC, k = it % NC, slot = it % (2 * kLineGroup);
          R a = R(0);
#pragma unroll
          for (int l = 0; l < NP; ++l) {
            if constexpr (k < NV) {
              a += (s ? B.Lm[l] : B.Lp[l]) * R(xu[slot][l]);
              if (MIXED && k == 0) rn[s] += (s ? bas.d.Lm[l] : bas.d.Lp[l]) * xu[slot][l];
            } else {
              a += (s ? B.Lm[l] : B.Lp[l]) * R(xg[slot][l]);
            }
          }
          if constexpr (k < NV) un[s][k] = a;
          else vn[s][k - NV] = a;
        }
      });
      static_for<kLineGroup>([&](auto jc) {
        constexpr int it = g * kLineGroup + decltype(jc)::value;
        if constexpr (it < 2 * NC) {
          constexpr int s = it / NC, k = it % NC, slot = it % (2 * kLineGroup);
          const long long on = (long long)ln.nb[s] * NN + ln.base;
          if constexpr (k < NV) {
#pragma unroll
            for (int l = 0; l < NP; ++l) xu[slot][l] = (U + k * S + on)[l * dstride<NP>(d)];
          } else {
            constexpr int gk = k - NV < DIM ? tau_index<DIM>(k - NV < DIM ? k - NV : 0, d) : NT + d;
#pragma unroll
            for (int l = 0; l < NP; ++l) xg[slot][l] = (G + (long long)gk * S + on)[l * dstride<NP>(d)];
          }
        }
      });
      __builtin_amdgcn_sched_barrier(0);
    });
  });
  Pair<double> du_old[NV];
  auto load_du = [&](long long o, int p) {
#pragma unroll
    for (int v = 0; v < NV; ++v) du_old[v] = Pair<double>{0.0, 0.0};
    if (e >= 0 && st.mode == 1 && st.A != 0.0) {
      if (msh.stream & kStreamState) {
#pragma unroll
        for (int v = 0; v < NV; ++v) du_old[v] = load_pair_nt<NN>(dU + v * S + o, p);
      } else {
#pragma unroll
        for (int v = 0; v < NV; ++v) du_old[v] = load_pair<NN>(dU + v * S + o, p);
      }
    }
  };
  if constexpr (EARLY) {
    load_du((long long)cmax(e, 0) * NN, nr.p);
    __builtin_amdgcn_sched_barrier(0);
    put_own();
  }
  if constexpr (ENDS) {
    __builtin_amdgcn_sched_barrier(0);
    if (ln.e >= 0) {
      const LineEnd<NP> end(ln.end);
#pragma unroll
      for (int v = 0; v < NV; ++v) un[0][v] = R(0);
#pragma unroll
      for (int k = 0; k < NVX; ++k) vn[0][k] = R(0);
#pragma unroll
      for (int l = 0; l < NP; ++l) {
        const R lw = end.nb(B, l);
#pragma unroll
        for (int v = 0; v < NV; ++v) un[0][v] += lw * R(xu1[v][l]);
        if (MIXED) rn[0] += end.nb(bas.d, l) * xu1[0][l];
#pragma unroll
        for (int k = 0; k < NVX; ++k) vn[0][k] += lw * R(xg1[k][l]);
      }
    }
  }
  if constexpr (STAGE) {
    load_own();
    __syncthreads();  // the neighbours are folded: their rows take the own values
    put_own();
  }
  __syncthreads();

  // line role: numerical fluxes at both ends, contraction of the nodal flux
  R t[ENDS ? (NP + 1) / 2 : NP][NV];
  static_for<DIM>([&](auto dc) {
    constexpr int d = decltype(dc)::value;
    if (dir != d || ln.e < 0) return;
    const int b0 = ln.el * PN + lds_slot<NP>(ln.base);
    if constexpr (ENDS) {
      const LineEnd<NP> end(ln.end);
      R uo[NV], uL[NV], uR[NV], Fe[NV], F0[NV], F1[NV];
      double ro = 0.0;
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        uo[v] = R(0);
#pragma unroll
        for (int l = 0; l < NP; ++l) uo[v] += end.own(B, l) * sIn[v][b0 + l * lds_step<NP>(d)];
        uL[v] = end.hi ? uo[v] : un[0][v];
        uR[v] = end.hi ? un[0][v] : uo[v];
      }
#pragma unroll
      for (int k = 0; k < NVX; ++k) {
        R vo = R(0);
#pragma unroll
        for (int l = 0; l < NP; ++l)
          vo += end.own(B, l) * sIn[NV + (k < DIM ? tau_index<DIM>(k, d) : NT + d)][b0 + l * lds_step<NP>(d)];
        vn[0][k] += vo;
      }
      if constexpr (MIXED) {
#pragma unroll
        for (int l = 0; l < NP; ++l) ro += end.own(bas.d, l) * sRho64[0][b0 + l * lds_step<NP>(d)];
      } else {
        ro = uo[0];
        rn[0] = un[0][0];
      }
      face_flux<DIM, R, FLUX, MODEL, d, NV, NVX>(uL, uR, vn[0], end.hi ? ro : rn[0], end.hi ? rn[0] : ro, lam_g, kb, ph,
                                                 Fe);
#pragma unroll
      for (int v = 0; v < NV; ++v) end.template both<Sh::NF>(Fe[v], lane, F0[v], F1[v]);
#pragma unroll
      for (int r = 0; r < end.H; ++r)
#pragma unroll
        for (int v = 0; v < NV; ++v)
          t[r][v] = MIXED ? R(0) : sT.v[end.row0 + r][NP] * F0[v] - sT.v[end.row0 + r][NP + 1] * F1[v];
#pragma unroll
      for (int l = 0; l < NP; ++l) {
        const int b = b0 + l * lds_step<NP>(d);
        R u[NV], F[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) u[v] = sIn[v][b];
        conv_flux<DIM, R, NV>(d, u, sIn[II][b], sIn[IP][b], F);
#pragma unroll
        for (int j = 0; j < DIM; ++j) F[1 + j] -= sIn[NV + tau_index<DIM>(j, d)][b];
        if constexpr (MODEL == 0) F[DIM + 1] -= kb * sIn[NV + NT + d][b];
#pragma unroll
        for (int r = 0; r < end.H; ++r)
#pragma unroll
          for (int v = 0; v < NV; ++v) t[r][v] += sT.v[end.row0 + r][l] * F[v];
      }
      if constexpr (MIXED) {
#pragma unroll
        for (int r = 0; r < end.H; ++r)
#pragma unroll
          for (int v = 0; v < NV; ++v)
            t[r][v] = t[r][v] - (sT.v[end.row0 + r][NP + 1] * F1[v] - sT.v[end.row0 + r][NP] * F0[v]);
      }
      return;
    }
    // own traces at both ends (0: xi = -1, 1: xi = +1), one pass over the line
    R uo[2][NV], Fs[2][NV];
    double ro[2] = {0.0, 0.0};
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      uo[0][v] = uo[1][v] = R(0);
#pragma unroll
      for (int l = 0; l < NP; ++l) {
        const R x = sIn[v][b0 + l * lds_step<NP>(d)];
        uo[0][v] += B.Lm[l] * x;
        uo[1][v] += B.Lp[l] * x;
      }
    }
#pragma unroll
    for (int k = 0; k < NVX; ++k) {
      R vo[2] = {R(0), R(0)};
#pragma unroll
      for (int l = 0; l < NP; ++l) {
        const R x = sIn[NV + (k < DIM ? tau_index<DIM>(k, d) : NT + d)][b0 + l * lds_step<NP>(d)];
        vo[0] += B.Lm[l] * x;
        vo[1] += B.Lp[l] * x;
      }
      vn[0][k] += vo[0];  // only the sum of the two traces is used
      vn[1][k] += vo[1];
    }
    if constexpr (MIXED) {
#pragma unroll
      for (int l = 0; l < NP; ++l) {
        const double x = sRho64[0][b0 + l * lds_step<NP>(d)];
        ro[0] += bas.d.Lm[l] * x;
        ro[1] += bas.d.Lp[l] * x;
      }
    } else {
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        ro[s] = uo[s][0];
        rn[s] = un[s][0];
      }
    }
    face_flux<DIM, R, FLUX, MODEL, d, NV, NVX>(un[0], uo[0], vn[0], rn[0], ro[0], lam_g, kb, ph, Fs[0]);
    __builtin_amdgcn_sched_barrier(0);
    face_flux<DIM, R, FLUX, MODEL, d, NV, NVX>(uo[1], un[1], vn[1], ro[1], rn[1], lam_g, kb, ph, Fs[1]);
    __builtin_amdgcn_sched_barrier(0);
    // the line is read again for the volume term rather than held in registers
    asm volatile("" ::: "memory");
#pragma unroll
    for (int i = 0; i < NP; ++i)
      // in FP64 the faces first, so that their fluxes take no registers any more
#pragma unroll
      for (int v = 0; v < NV; ++v) t[i][v] = MIXED ? R(0) : B.wm[i] * Fs[0][v] - B.wp[i] * Fs[1][v];
    if constexpr (!MIXED) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int l = 0; l < NP; ++l) {
      const int b = b0 + l * lds_step<NP>(d);
      R u[NV], F[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) u[v] = sIn[v][b];
      conv_flux<DIM, R, NV>(d, u, sIn[II][b], sIn[IP][b], F);
#pragma unroll
      for (int j = 0; j < DIM; ++j) F[1 + j] -= sIn[NV + tau_index<DIM>(j, d)][b];
      if constexpr (MODEL == 0) F[DIM + 1] -= kb * sIn[NV + NT + d][b];
#pragma unroll
      for (int i = 0; i < NP; ++i)
#pragma unroll
        for (int v = 0; v < NV; ++v) t[i][v] += B.Dhat[i][l] * F[v];
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (MIXED) {
#pragma unroll
      for (int i = 0; i < NP; ++i)
#pragma unroll
        for (int v = 0; v < NV; ++v) t[i][v] = t[i][v] - (B.wp[i] * Fs[1][v] - B.wm[i] * Fs[0][v]);
    }
  });
  __syncthreads();  // every line is read: sIn takes the contributions
  static_for<DIM>([&](auto dc) {
    constexpr int d = decltype(dc)::value;
    if (dir != d || ln.e < 0) return;
    const int b0 = ln.el * PN + lds_slot<NP>(ln.base);
    constexpr int ROWS_OF_LANE = ENDS ? (NP + 1) / 2 : NP;
    const int row0 = ENDS ? LineEnd<NP>(ln.end).row0 : 0;
#pragma unroll
    for (int i = 0; i < ROWS_OF_LANE; ++i)
#pragma unroll
      for (int v = 0; v < NV; ++v) sIn[d * NV + v][b0 + (row0 + i) * lds_step<NP>(d)] = t[i][v];
  });

  const NodeRole<DIM, NP, EPB> nu(AGAIN ? opaque(tid) : tid);
  if constexpr (AGAIN) e = nu.el < EPB ? sE[nu.el] : -1;
  const long long o = (long long)cmax(e, 0) * NN;
  Pair<double> ua[AGAIN ? NV : 1];
  Pair<GT> ga[AGAIN ? DIM : 1];
  Pair<double>* const u = AGAIN ? ua : u0;
  Pair<GT>* const gc = AGAIN ? ga : g0 + (MODEL == 0 ? NT : 0);
  if constexpr (AGAIN) {
    if (e >= 0) {
#pragma unroll
      for (int v = 0; v < NV; ++v) ua[v] = load_pair<NN>(U + v * S + o, nu.p);
#pragma unroll
      for (int d = 0; MODEL == 0 && d < DIM; ++d) ga[d] = load_pair<NN>(G + (long long)(NT + d) * S + o, nu.p);
    }
  }
  if constexpr (!EARLY) load_du(o, nu.p);
  __syncthreads();

  // source (FP64) and update
  if (e >= 0) {
    double Rv[2][NV];
    {
      R acc[2][NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) acc[0][v] = acc[1][v] = R(0);
#pragma unroll
      for (int d = 0; d < DIM; ++d) {
        const R h2 = R(sH2[nu.el][d]);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          const LdsPair<R> x = lds_get(&sIn[d * NV + v][nu.sl]);
          acc[0][v] += h2 * x.a;
          acc[1][v] += h2 * x.b;
        }
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        Rv[0][v] = double(acc[0][v]);
        Rv[1][v] = double(acc[1][v]);
      }
    }
    if constexpr (MODEL == 0) {
#pragma unroll
      for (int d = 0; d < DIM; ++d) {
        Rv[0][1 + d] += ph.alpha * u[0].a * double(R(gc[d].a));
        Rv[1][1 + d] += ph.alpha * u[0].b * double(R(gc[d].b));
      }
      Rv[0][DIM + 1] += ph.ab * (u[0].a - u[DIM + 1].a);
      Rv[1][DIM + 1] += ph.ab * (u[0].b - u[DIM + 1].b);
      if (st.closure) {
#pragma unroll
        for (int d = 0; d <= DIM; ++d) {
          const Pair<float> x = load_pair<NN>(st.closure + d * S + o, nu.p);
          Rv[0][1 + d] += double(x.a);
          Rv[1][1 + d] += double(x.b);
        }
      }
    }
    if (st.mode == 0) {
#pragma unroll
      for (int v = 0; v < NV; ++v) store_pair<NN>(Uout + v * S + o, nu.p, Rv[0][v], Rv[1][v]);
      return;
    }
    double da[NV], db[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      da[v] = st.A * du_old[v].a + st.dt * Rv[0][v];
      db[v] = st.A * du_old[v].b + st.dt * Rv[1][v];
    }
    if (msh.stream & kStreamState) {
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        store_pair_nt<NN>(dU + v * S + o, nu.p, da[v], db[v]);
        store_pair_nt<NN>(Uout + v * S + o, nu.p, u[v].a + st.B * da[v], u[v].b + st.B * db[v]);
      }
    } else {
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        store_pair<NN>(dU + v * S + o, nu.p, da[v], db[v]);
        store_pair<NN>(Uout + v * S + o, nu.p, u[v].a + st.B * da[v], u[v].b + st.B * db[v]);
      }
    }
  }
}

}  // namespace nsk

#include "dg_1d.hpp"

namespace nsk {

template <int DIM, int NP, int EPB, typename R, typename GT, int MODEL = 0, int FORM = kLines>
__device__ __forceinline__ void lift_block(int L, int tid, const double* __restrict__ U, GT* __restrict__ G,
                                           const BasisArgs& bas, const MeshArgs& msh, const PhysArgs& ph,
                                           double* __restrict__ lfpart = nullptr) {
  if constexpr (DIM == 1)
    lift_block_1d<NP, EPB, R, GT, MODEL>(L, tid, U, G, bas, msh, ph, lfpart);
  else
    lift_block_lines<DIM, NP, EPB, R, GT, MODEL, FORM>(L, tid, U, G, bas, msh, ph, lfpart);
}

template <int DIM, int NP, int EPB, int FORM>
__device__ __forceinline__ void lap_block(int L, int tid, const double* __restrict__ U, double* __restrict__ G,
                                          const BasisArgs& bas, const MeshArgs& msh, const PhysArgs& ph) {
  if constexpr (DIM == 1)
    lap_block_1d<NP, EPB>(L, tid, U, G, bas, msh, ph);
  else
    lap_block_lines<DIM, NP, EPB, FORM>(L, tid, U, G, bas, msh, ph);
}

template <int DIM, int NP, int EPB, typename R, typename GT, int FLUX = 0, int MODEL = 0, int FORM = kLines>
__device__ __forceinline__ void rhs_block(int L, int tid, const double* __restrict__ U, const GT* __restrict__ G,
                                          double* __restrict__ Uout, double* __restrict__ dU, const BasisArgs& bas,
                                          const MeshArgs& msh, const PhysArgs& ph, const StageArgs& st) {
  if constexpr (DIM == 1)
    rhs_block_1d<NP, EPB, R, GT, FLUX, MODEL>(L, tid, U, G, Uout, dU, bas, msh, ph, st);
  else
    rhs_block_lines<DIM, NP, EPB, R, GT, FLUX, MODEL, FORM>(L, tid, U, G, Uout, dU, bas, msh, ph, st);
}

// -------------------------------------------------------------------------
// One launch per stage kernel over a single mesh.
// -------------------------------------------------------------------------
template <int DIM, int NP, int EPB, typename R, typename GT, int FORM = kLines>
__global__ void __launch_bounds__((Tile<DIM, NP, EPB, FORM>::THREADS))
lift_kernel(const double* __restrict__ U, GT* __restrict__ G, BasisArgs bas, MeshArgs msh, PhysArgs ph) {
  lift_block<DIM, NP, EPB, R, GT, 0, FORM>(remap_block(blockIdx.x, gridDim.x, msh.nxcd), threadIdx.x, U, G, bas, msh,
                                           ph);
}

// The right-hand-side kernels are held to 3 waves per SIMD (168 VGPRs), where
// they need no scratch: each spilled register of a thread is written to memory
// (the degree 4 HLLC kernel with 38 spills: 10 % of a stage).  4 waves, with the LDS
// for a fifth workgroup, gained nothing (2.02 ms both, degree 4 in 3D FP64,
// 96x48x48 elements, before stores were streamed); 2 waves lose (2.41 against 2.14
// ms then; degree 5, 48x24x24, a stage: 0.86 against 0.73 ms).
constexpr int kRhsWaves = 3;
template <int DIM, int NP, typename R, int FORM>
constexpr int kRhsWavesOf = kFourWaves<DIM, NP, R> && FORM != kStaged ? 4 : kRhsWaves;
template <int DIM, int NP, int EPB, typename R, typename GT, int FLUX = 0, int MODEL = 0, int FORM = kLines>
__global__ void __launch_bounds__((Tile<DIM, NP, EPB, FORM>::THREADS))
    __attribute__((amdgpu_waves_per_eu((kRhsWavesOf<DIM, NP, R, FORM>))))
rhs_kernel(const double* __restrict__ U, const GT* __restrict__ G, double* __restrict__ Uout,
           double* __restrict__ dU, BasisArgs bas, MeshArgs msh, PhysArgs ph, StageArgs st) {
  rhs_block<DIM, NP, EPB, R, GT, FLUX, MODEL, FORM>(remap_block(blockIdx.x, gridDim.x, msh.nxcd), threadIdx.x, U, G,
                                                     Uout, dU, bas, msh, ph, st);
}

// Original NSK path: the first lifting, which also writes the workgroup's
// maximum of the global Lax-Friedrichs speed to lfpart[logical block] (when
// lfpart is set) ...
template <int DIM, int NP, int EPB, int FORM = kLines>
__global__ void __launch_bounds__((Tile<DIM, NP, EPB, FORM>::THREADS))
nsk_lift_kernel(const double* __restrict__ U, double* __restrict__ G, BasisArgs bas, MeshArgs msh, PhysArgs ph,
                double* __restrict__ lfpart) {
  lift_block<DIM, NP, EPB, double, double, 1, FORM>(remap_block(blockIdx.x, gridDim.x, msh.nxcd), threadIdx.x, U, G,
                                                     bas, msh, ph, lfpart);
}

// ... the second lifting ...
template <int DIM, int NP, int EPB, int FORM = kLines>
__global__ void __launch_bounds__((Tile<DIM, NP, EPB, FORM>::THREADS))
lap_kernel(const double* __restrict__ U, double* __restrict__ G, BasisArgs bas, MeshArgs msh, PhysArgs ph) {
  lap_block<DIM, NP, EPB, FORM>(remap_block(blockIdx.x, gridDim.x, msh.nxcd), threadIdx.x, U, G, bas, msh, ph);
}

// ... and the maximum of the partial speeds, in two launches: kMaxReduceBlocks
// workgroups each reduce a strided share into out[blockIdx.x], then one
// workgroup reduces those.
constexpr int kMaxReduceThreads = 256;
constexpr int kMaxReduceBlocks = 128;
template <int THREADS>
__global__ void __launch_bounds__(THREADS)
max_reduce_kernel(const double* __restrict__ part, int n, double* __restrict__ out) {
  __shared__ double red[THREADS / 64];
  const int tid = threadIdx.x;
  double m = 0.0;
  for (int i = blockIdx.x * THREADS + tid; i < n; i += gridDim.x * THREADS) m = fmax(m, part[i]);
  block_max_store<THREADS>(m, red, out + blockIdx.x, tid);
}

// -------------------------------------------------------------------------
// Persistent kernels over a batch of instances with the same degree.  The
// work list holds (instance, logical block) items; workgroup w takes the
// contiguous item range [w * chunk, (w + 1) * chunk), so that consecutive
// blocks of one instance's tiled work order stay on one XCD.
// -------------------------------------------------------------------------
struct BatchInst {
  const double* U;     // stage input state
  double* Uout;        // stage output state (or R)
  double* dU;          // Runge-Kutta register
  void* G;             // lifted gradients (tau, grad c)
  MeshArgs msh;        // mesh of the instance (nxcd unused)
};

constexpr int kBatchXcds = 8;  // XCDs the batched kernels spread rounds over

struct BatchItem {
  int inst;            // instance index
  int L;               // logical block of that instance
};

// Batched kernels: a group of instances of one degree shares a list of
// (instance, element block) items.  The one-item form gives every item its
// own workgroup; the persistent form runs a fixed grid that takes the list
// in rounds of gridDim.x consecutive items.  In both, each XCD takes a
// contiguous slice of the items in flight, so neighbouring elements meet in
// the same L2.
template <int DIM, int NP, int EPB, typename R, typename GT, int FORM>
__global__ void __launch_bounds__((Tile<DIM, NP, EPB, FORM>::THREADS))
lift_kernel_batch1(const BatchInst* __restrict__ inst, const BatchItem* __restrict__ items, BasisArgs bas,
                   PhysArgs ph) {
  const BatchItem w = items[remap_block(blockIdx.x, gridDim.x, kBatchXcds)];
  const BatchInst& I = inst[w.inst];
  lift_block<DIM, NP, EPB, R, GT, 0, FORM>(w.L, threadIdx.x, I.U, reinterpret_cast<GT*>(I.G), bas, I.msh, ph);
}

template <int DIM, int NP, int EPB, typename R, typename GT, int FORM>
__global__ void __launch_bounds__((Tile<DIM, NP, EPB, FORM>::THREADS)) __attribute__((amdgpu_waves_per_eu(kRhsWaves)))
rhs_kernel_batch1(const BatchInst* __restrict__ inst, const BatchItem* __restrict__ items, BasisArgs bas,
                  PhysArgs ph, StageArgs st) {
  const BatchItem w = items[remap_block(blockIdx.x, gridDim.x, kBatchXcds)];
  const BatchInst& I = inst[w.inst];
  rhs_block<DIM, NP, EPB, R, GT, 0, 0, FORM>(w.L, threadIdx.x, I.U, reinterpret_cast<const GT*>(I.G), I.Uout, I.dU, bas,
                                             I.msh, ph, st);
}

// The thread index handed to the block functions is opaque in every round:
// otherwise the compiler hoists the per-thread basis and index work out of the loop
// and holds it in registers across items, which lowers occupancy.
template <int DIM, int NP, int EPB, typename R, typename GT, int FORM>
__global__ void __launch_bounds__((Tile<DIM, NP, EPB, FORM>::THREADS))
lift_kernel_batch(const BatchInst* __restrict__ inst, const BatchItem* __restrict__ items, int nitems,
                  BasisArgs bas, PhysArgs ph) {
  const int slot = remap_block(blockIdx.x, gridDim.x, kBatchXcds);
  for (int base = 0; base < nitems; base += gridDim.x) {
    const int it = base + slot;
    if (it < nitems) {
      const BatchItem w = items[it];
      const BatchInst& I = inst[w.inst];
      lift_block<DIM, NP, EPB, R, GT, 0, FORM>(w.L, opaque(threadIdx.x), I.U, reinterpret_cast<GT*>(I.G), bas, I.msh,
                                               ph);
    }
    __syncthreads();  // LDS is reused by the next item
  }
}

template <int DIM, int NP, int EPB, typename R, typename GT, int FORM>
__global__ void __launch_bounds__((Tile<DIM, NP, EPB, FORM>::THREADS)) __attribute__((amdgpu_waves_per_eu(kRhsWaves)))
rhs_kernel_batch(const BatchInst* __restrict__ inst, const BatchItem* __restrict__ items, int nitems,
                 BasisArgs bas, PhysArgs ph, StageArgs st) {
  const int slot = remap_block(blockIdx.x, gridDim.x, kBatchXcds);
  for (int base = 0; base < nitems; base += gridDim.x) {
    const int it = base + slot;
    if (it < nitems) {
      const BatchItem w = items[it];
      const BatchInst& I = inst[w.inst];
      rhs_block<DIM, NP, EPB, R, GT, 0, 0, FORM>(w.L, opaque(threadIdx.x), I.U, reinterpret_cast<const GT*>(I.G),
                                                 I.Uout, I.dU, bas, I.msh, ph, st);
    }
    __syncthreads();
  }
}

// -------------------------------------------------------------------------
// Diagnostics: per-block partial sums, then one block reduces in a fixed
// order (deterministic).  Slots: 0..4 conserved integrals, 5 kinetic energy,
// 6 E^alpha, 7 (rho-c)^2, 8 rho min, 9 rho max, 10 max wave speed,
// 11 non-finite count, 12 max_e sum_d max(|v_d|+a)/h_d.
// -------------------------------------------------------------------------
constexpr int kDiagSlots = 13;

// index of element e in each direction (elements are numbered in 32 bits: the
// work order is a table of ints)
template <int DIM>
__device__ __forceinline__ void elem_index_diag(const MeshArgs& m, unsigned e, int (&c)[DIM]) {
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    if (d == DIM - 1) {
      c[d] = int(e);
    } else {
      const unsigned n = unsigned(m.nel[d]), q = e / n;
      c[d] = int(e - q * n);
      e = q;
    }
  }
}
constexpr int kDiagThreads = 256;

__device__ __forceinline__ double vdw_W(double rho, double T) {
  // W = rho R T ln(rho/(1 - b rho)) - a rho^2 with a = 3, b = 1/3, R = 8/3
  return rho * (8.0 / 3.0) * T * log(3.0 * rho / (3.0 - rho)) - 3.0 * rho * rho;
}

__device__ __forceinline__ double diag_combine(int k, double a, double b) {
  return k == 8 ? fmin(a, b) : ((k == 9 || k == 10 || k == 12) ? fmax(a, b) : a + b);
}

// the block's value of every slot, in a fixed order: lanes by shuffles, then the
// waves; red is free again when it returns (thread 0..kDiagSlots-1 hold a slot)
__device__ __forceinline__ double diag_block_reduce(double (&acc)[kDiagSlots], double (*red)[kDiagSlots]) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int k = 0; k < kDiagSlots; ++k)
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc[k] = diag_combine(k, acc[k], __shfl_down(acc[k], off));
  if ((tid & 63) == 0)
    for (int k = 0; k < kDiagSlots; ++k) red[tid >> 6][k] = acc[k];
  __syncthreads();
  double r = 0.0;
  if (tid < kDiagSlots) {
    r = red[0][tid];
    for (int w = 1; w < kDiagThreads / 64; ++w) r = diag_combine(tid, r, red[w][tid]);
  }
  return r;
}

// One thread per node for the pointwise terms; the lifted gradient of c (of rho
// in the original NSK path), which the energy needs, is formed here too, one
// thread per element line, so that the state is read once and no lifted
// gradients are written (a launch of the lifting kernel, then 72 bytes a node
// written and 24 read).  R: the precision of the lifting.  FULL false: only what
// the step size needs (slots 8..12), without gradient, integrals and logarithm.
// One reciprocal of rho and of the volume a node, element indexes in 32 bits and
// four workgroups a CU (the grid's 1024 are then resident at once): with the
// divisions of each term by itself, 64-bit indexes and three workgroups 144 us.
// Measured at 48x24x24, N = 4, FP64: 107 us, and 43 us without FULL (29 us to
// read the state at the rate of a large copy); a lifting launch and a kernel that
// took each element's maxima with one thread were 148 + 151 us for both.
template <int DIM, int NP, typename R, int MODEL, bool FULL>
__global__ void __launch_bounds__(kDiagThreads, 4)
diag_partial_kernel(const double* __restrict__ U, double* __restrict__ part, const double* __restrict__ wq1,
                    BasisArgs bas, MeshArgs msh, PhysArgs ph) {
  using Sh = Shape<DIM, NP>;
  constexpr int NN = Sh::NN, NF = Sh::NF;
  constexpr int NV = MODEL == 1 ? DIM + 1 : DIM + 2;
  constexpr int SI = MODEL == 1 ? 0 : DIM + 1;  // the lifted scalar
  constexpr int EPBD = (kDiagThreads / NN) > 0 ? kDiagThreads / NN : 1;  // whole elements per group
  constexpr int SLOTS = EPBD * NN, LINES = EPBD * NF;
  static_assert(SLOTS <= kDiagThreads, "one thread per node");
  __shared__ double red[kDiagThreads / 64][kDiagSlots];
  __shared__ double spd[DIM][kDiagThreads];  // per-node |v_d| + a
  __shared__ R sC[FULL ? SLOTS : 1], sX[DIM][FULL ? SLOTS : 1];
  const auto& B = bas.of(R());
  const int tid = threadIdx.x;
  double acc[kDiagSlots];
#pragma unroll
  for (int k = 0; k < kDiagSlots; ++k) acc[k] = 0.0;
  acc[8] = INFINITY;
  acc[9] = -INFINITY;
  const long long S = msh.S;
  const int el = tid / NN, n = tid - (tid / NN) * NN;
  double wn = 1.0;  // tensor-product quadrature weight of the node
  if constexpr (FULL) {
    int r = n;
#pragma unroll
    for (int d = 0; d < DIM; ++d) { wn *= wq1[r % NP]; r /= NP; }
  }
  // groups of whole elements, one thread per node (coalesced loads); the
  // per-element directional maxima of the wave speed go through LDS
  const long long ngroups = (msh.E + EPBD - 1) / EPBD;
  for (long long grp = blockIdx.x; grp < ngroups; grp += gridDim.x) {
    const long long e = grp * EPBD + el;
    const bool active = tid < SLOTS && e < msh.E;
    double u[NV];
    if (active) {
#pragma unroll
      for (int v = 0; v < NV; ++v) u[v] = U[v * S + e * NN + n];
    }
    if constexpr (FULL) {
      if (active) sC[tid] = R(u[SI]);
      // the two neighbours' traces of a line, then the line
      constexpr int ROUNDS = (DIM * LINES + kDiagThreads - 1) / kDiagThreads;
      R tr[ROUNDS][2];
      double h2l[ROUNDS];
#pragma unroll
      for (int q = 0; q < ROUNDS; ++q) {
        const int i = tid + q * kDiagThreads, d = i / LINES, le = (i - d * LINES) / NF, f = i % NF;
        const long long ee = grp * EPBD + le;
        tr[q][0] = tr[q][1] = R(0);
        h2l[q] = 0.0;
        if (d < DIM && ee < msh.E) {
          int ci[DIM];
          elem_index_diag<DIM>(msh, unsigned(ee), ci);
          int c = ci[0], step = 1, nd = msh.nel[0];
          const double* h2 = msh.h2[0];
#pragma unroll
          for (int k = 1; k < DIM; ++k)
            if (d == k) { c = ci[k]; step = k == 1 ? msh.nel[0] : msh.nel[0] * msh.nel[1]; nd = msh.nel[k]; h2 = msh.h2[k]; }
          const int sd = dstride<NP>(d), base = face_base<NP>(d, f);
          h2l[q] = h2[c];
          const long long nb[2] = {c == 0 ? ee + (long long)(nd - 1) * step : ee - step,
                                   c == nd - 1 ? ee - (long long)(nd - 1) * step : ee + step};
          double x[2][NP];
#pragma unroll
          for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int l = 0; l < NP; ++l) x[s][l] = U[SI * S + nb[s] * NN + base + l * sd];
#pragma unroll
          for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int l = 0; l < NP; ++l) tr[q][s] += (s ? B.Lm[l] : B.Lp[l]) * R(x[s][l]);
        }
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < ROUNDS; ++q) {
        const int i = tid + q * kDiagThreads, d = i / LINES, le = (i - d * LINES) / NF, f = i % NF;
        if (d < DIM && grp * EPBD + le < msh.E) {
          const int sd = dstride<NP>(d), b0 = le * NN + face_base<NP>(d, f);
          R w[NP], wl = R(0), wr = R(0);
#pragma unroll
          for (int l = 0; l < NP; ++l) {
            w[l] = sC[b0 + l * sd];
            wl += B.Lp[l] * w[l];
            wr += B.Lm[l] * w[l];
          }
          const R wsm = R(0.5) * (tr[q][0] + wr), wsp = R(0.5) * (wl + tr[q][1]), h2 = R(h2l[q]);
#pragma unroll
          for (int m = 0; m < NP; ++m) {
            R vol = R(0);
#pragma unroll
            for (int l = 0; l < NP; ++l) vol += B.Dhat[m][l] * w[l];
            const R surf = (B.Lp[m] * wsp - B.Lm[m] * wsm) * B.invw[m];
            sX[d][b0 + m * sd] = h2 * (surf - vol);
          }
        }
      }
      __syncthreads();
    }
#pragma unroll
    for (int d = 0; d < DIM; ++d) spd[d][tid] = 0.0;
    if (active) {
      bool finite = true;
#pragma unroll
      for (int v = 0; v < NV; ++v)
        if (!isfinite(u[v])) { acc[11] += 1.0; finite = false; }
      const double rho = u[0], ir = 1.0 / rho;
      if constexpr (FULL) {
        int ci[DIM];
        elem_index_diag<DIM>(msh, unsigned(e), ci);
        double hv = 1.0;
#pragma unroll
        for (int d = 0; d < DIM; ++d) hv *= msh.h2[d][ci[d]];
        const double wgt = wn / hv;  // J = prod of h/2
#pragma unroll
        for (int v = 0; v < NV; ++v) acc[v] += wgt * u[v];
        // model II: c and its lifted gradient; original NSK: the lifted
        // gradient of rho, no relaxation energy
        const double c = MODEL == 0 ? u[NV - 1] : rho;
        double m2 = 0.0, gc2 = 0.0;
#pragma unroll
        for (int d = 0; d < DIM; ++d) {
          m2 += u[1 + d] * u[1 + d];
          const double gcd = double(sX[d][tid]);
          gc2 += gcd * gcd;
        }
        const double ek = 0.5 * m2 * ir;
        acc[5] += wgt * ek;
        acc[6] += wgt * (ek + vdw_W(rho, ph.T) + 0.5 * ph.alpha * (rho - c) * (rho - c) + 0.5 * ph.kappa * gc2);
        acc[7] += wgt * (rho - c) * (rho - c);
      }
      if (finite) {
        acc[8] = fmin(acc[8], rho);
        acc[9] = fmax(acc[9], rho);
        double a;
        if constexpr (MODEL == 1) {
          const double q = 1.0 / (3.0 - rho), dp = 24.0 * ph.T * q * q - 6.0 * rho;
          a = dp > 0.0 ? sqrt(dp) : 0.0;
        } else {
          a = sound_speed<double>(rho, ph.T, ph.alpha);
        }
#pragma unroll
        for (int d = 0; d < DIM; ++d) {
          const double sp = fabs(u[1 + d] * ir) + a;
          acc[10] = fmax(acc[10], sp);
          spd[d][tid] = sp;
        }
      }
    }
    __syncthreads();
    // max over the element's nodes along each direction, 16 lanes an element;
    // the maximum does not depend on the order of its operands
    for (int q = tid / 16; q < EPBD; q += kDiagThreads / 16) {
      if (grp * EPBD + q >= msh.E) continue;
      int ci[DIM];
      elem_index_diag<DIM>(msh, unsigned(grp * EPBD + q), ci);
      double lam = 0.0;
#pragma unroll
      for (int d = 0; d < DIM; ++d) {
        double m = 0.0;
        for (int k = tid % 16; k < NN; k += 16) m = fmax(m, spd[d][q * NN + k]);
#pragma unroll
        for (int off = 8; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off, 16));
        lam += m * (0.5 * msh.h2[d][ci[d]]);
      }
      acc[12] = fmax(acc[12], lam);
    }
    __syncthreads();
  }
  const double r = diag_block_reduce(acc, red);
  if (tid < kDiagSlots) part[(long long)blockIdx.x * kDiagSlots + tid] = r;
}

// the blocks' partial values, in a fixed order
template <int SLOTS>
__global__ void __launch_bounds__(kDiagThreads) diag_final_kernel(const double* __restrict__ part, int nblocks,
                                                                  double* __restrict__ out) {
  __shared__ double red[kDiagThreads / 64][kDiagSlots];
  double acc[kDiagSlots];
#pragma unroll
  for (int k = 0; k < kDiagSlots; ++k) acc[k] = 0.0;
  acc[8] = INFINITY;
  acc[9] = -INFINITY;
  for (int b = threadIdx.x; b < nblocks; b += kDiagThreads)
#pragma unroll
    for (int k = 0; k < kDiagSlots; ++k) acc[k] = diag_combine(k, acc[k], part[(long long)b * kDiagSlots + k]);
  const double r = diag_block_reduce(acc, red);
  if (threadIdx.x < kDiagSlots) out[threadIdx.x] = r;
}

}  // namespace nsk
