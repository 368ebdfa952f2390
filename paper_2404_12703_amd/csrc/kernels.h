// kernels.h -- HIP kernels of the DGSEM time derivative and the low-storage
// RK update for gfx950 (CDNA4, wave64), as templates over the polynomial
// degree.  Each degree is instantiated in a translation unit of its own
// (kernels_n<N>.hip), so the degrees compile in parallel; kernels.hip holds
// the reductions and the dispatch over N.
//
// Paper (GALAEXI, arXiv 2404.12703) routines, Table tab:dg_routines and App. A:
//   ConsToPrim, ProlongToFace, FillFlux, VolInt, SurfInt, ApplyJac and the
//   Lift_* copies of BR1 (Sec. 2.2 "Second-Order Equations").
//
// Design: one workgroup slot per element, one thread per volume node.  Per
// RK stage with viscosity or shock capturing, two sweeps (BR1 needs every
// neighbour's lifted gradient before any viscous face flux can be formed):
//   k_volume : (shock capturing) the a-priori indicator value of the element;
//              BR1 lifting with g kept on chip; each own face node's viscous
//              normal flux; the whole volume integral.
//   k_surface: (shock capturing) the blending factor from the neighbours'
//              indicator values; the face fluxes (Riemann + BR1 viscous
//              mean) of the six faces, computed by both neighbours from the
//              same operands in the same order so both hold the same bits
//              and nothing is stored; the per-DOF SurfInt gather (one writer
//              per entry, as the paper's GPU SurfInt); ApplyJac; the LSERK
//              stage update; and the next stage's U traces (ProlongToFace).
//   k_blend  : (shock capturing) the same for the workgroups holding an
//              element with a positive blending factor, which k_surface lists
//              and skips, plus the FV subcell operator.
// On meshes of parallelepipeds every kernel reads one node's metrics, and the
// viscous standard form takes k_volume_affine for its volume sweep (FP64).
// Euler takes one sweep, k_rhs (with shock capturing then k_blend), unless the
// blending factors are smoothed over neighbours or the split form is chosen.
// Traces are ping-ponged between stages because the last sweep reads the
// neighbours' traces of the old state while writing those of the new one.
// Layouts are structure-of-arrays with one contiguous (N+1)^3 block per
// element and variable, so every global access of a workgroup is contiguous.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>

#include "dg_internal.h"
#include "physics.h"

namespace dg {

// loads and stores of single-use streams: non-temporal when NT (the working
// set exceeds the on-die caches), plain otherwise
template <bool NT, typename T>
__device__ __forceinline__ T ld(const T *p) {
  if constexpr (NT) return __builtin_nontemporal_load(p);
  else return *p;
}
template <bool NT, typename T>
__device__ __forceinline__ void st(T x, T *p) {
  if constexpr (NT) __builtin_nontemporal_store(x, p);
  else *p = x;
}

__device__ __forceinline__ int vnode(int n, int i, int j, int k) { return i + n * (j + n * k); }

template <int n>
__device__ __forceinline__ int lnode(int d, int l, int p, int q) {
  return d == 0 ? l + n * (p + n * q) : (d == 1 ? p + n * (l + n * q) : p + n * (q + n * l));
}

// Buffers that are read along face lines hold the volume nodes with padded
// strides: row (fixed j, k) n + 1 values, plane (fixed k) n (n + 1).  A wave
// prolongs one face; unpadded, the lanes of a xi face read n apart, which for
// n = 8 puts eight distinct doubles on each LDS bank pair.
template <int n>
struct Pad {
  static constexpr int row = n + 1, plane = n * (n + 1), size = n * n * (n + 1);
  static __device__ __forceinline__ int at(int i, int j, int k) { return i + row * j + plane * k; }
  // the line normal to face f through face node pq, in padded coordinates
  static __device__ __forceinline__ void face_line(int f, int pq, int &base, int &stride) {
    const int d = f >> 1, p = pq % n, q = pq / n;
    base = d == 0 ? row * p + plane * q : (d == 1 ? p + plane * q : p + row * q);
    stride = d == 0 ? 1 : (d == 1 ? row : plane);
  }
};

// a state value (FP64) in the arithmetic type; the mixed form's energy carries
// the background shift (rho e - p_ref/(gamma - 1))
template <typename real>
__device__ __forceinline__ real to_real(double u, int c, const View<real> &v) {
  if constexpr (sizeof(real) == 4) return (real)(c == 4 ? u - v.e_ref : u);
  else return u;
}

// ProlongToFace of the five conservative variables at one face node from a
// padded LDS copy of the element's state (rows of Pad<n>::size values).
// Explicit multiply-adds in a fixed order: an element that recomputes its own
// trace gets the bits its neighbours read from the stored one.
template <int n, typename real>
__device__ __forceinline__ void prolong_state(const real *rows, const real *lv, int base, int stride, real *out) {
  real s[5] = {0, 0, 0, 0, 0};
#pragma unroll
  for (int l = 0; l < n; ++l) {
    const real lw = lv[l];
#pragma unroll
    for (int c = 0; c < 5; ++c) s[c] = fma(lw, rows[c * Pad<n>::size + base + l * stride], s[c]);
  }
#pragma unroll
  for (int c = 0; c < 5; ++c) out[c] = s[c];
}

// The conservative state at one face node: with Gauss-Lobatto nodes the end
// node of the line (l(-1), l(+1) are unit vectors), else ProlongToFace.
template <int n, bool LGL, typename real>
__device__ __forceinline__ void face_state(const real *rows, const real *lv, int base, int stride, bool plus,
                                           real *out) {
  if constexpr (LGL) {
    const int at = base + (plus ? (n - 1) * stride : 0);
#pragma unroll
    for (int c = 0; c < 5; ++c) out[c] = rows[c * Pad<n>::size + at];
  } else {
    prolong_state<n>(rows, lv, base, stride, out);
  }
}

// which view and which element block this workgroup works on: a single
// solve (nreq = 0) takes its view from the kernel arguments; a batch of solves
// looks its request up in the block prefix sums and loads that request's view.
// One instantiation serves both, so a request computes the same bits alone and
// in any batch.
// The hardware hands consecutive workgroups to the eight XCDs in turn; with
// `remap` each XCD instead receives one contiguous range of element blocks, so
// face neighbours (adjacent element indices) share that XCD's L2.  A bijection
// of [0, gridDim.x).
__device__ __forceinline__ int xcd_block(int b, int nb) {
  const int q = nb >> 3, r = nb & 7, x = b & 7, idx = b >> 3;
  const int start = x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q;
  return start + idx;
}

// the descriptors of a batch hold byte offsets into the arena; rebuilding the
// pointers from the argument's arena pointer keeps every access a global-memory
// one (pointers read from memory would be addressed as generic pointers)
template <typename real>
__device__ __forceinline__ View<real> rebase(View<real> v, char *const base) {
  auto at = [base](auto p) { return (decltype(p))(base + (intptr_t)p); };
  auto at_or_null = [base](auto p) { return p ? (decltype(p))(base + (intptr_t)p) : p; };
  v.U = at(v.U);
  v.dU = at(v.dU);
  v.R = at_or_null(v.R);
  v.Ja = at(v.Ja);
  v.invJ = at(v.invJ);
  v.NS = at(v.NS);
  v.Utr0 = at(v.Utr0);
  v.Utr1 = at(v.Utr1);
  v.Hv = at_or_null(v.Hv);
  v.Vol = at_or_null(v.Vol);
  v.conn = at(v.conn);
  v.Xs = at_or_null(v.Xs);
  v.basis = at(v.basis);
  v.alpha = at(v.alpha);
  v.alpha_raw = at(v.alpha_raw);
  v.alpha_in = at_or_null(v.alpha_in);
  v.bcnt = at_or_null(v.bcnt);
  v.blist = at_or_null(v.blist);
  v.diag = at_or_null(v.diag);
  return v;
}

template <typename real>
__device__ __forceinline__ View<real> select_view(const View<real> *views, const int *blk_start, int nreq,
                                                  const View<real> &single, int &lblk) {
  if (nreq == 0) {
    lblk = single.remap ? xcd_block(blockIdx.x, gridDim.x) : blockIdx.x;
    return single;
  }
  const int b = blockIdx.x + blk_start[0];  // a launch may take a range of its group's requests
  int r = 0;
  while (r + 1 < nreq && b >= blk_start[r + 1]) ++r;
  lblk = b - blk_start[r];
  return rebase(views[r], single.base);
}

// whether the metrics of an element's first node stand for all (View::affine,
// which the mixed form never sets: its kernels do not ask)
template <typename real>
__device__ __forceinline__ bool one_node(const View<real> &v) {
  return sizeof(real) == sizeof(double) && v.affine;
}

template <int N, typename real>
struct Smem {
  using S = Sz<N>;
  real Dh[S::n * (S::n + 1)];  // rows padded to n + 1: lanes reading different rows hit different banks
  real lm[S::n], lp[S::n], lhm[S::n], lhp[S::n];
};

template <int N, typename real>
__device__ __forceinline__ void load_basis(Smem<N, real> &sb, const real *basis, int tid) {
  using S = Sz<N>;
  constexpr int n = S::n;
  BasisOffsets o(n);
  for (int t = tid; t < n * n; t += blockDim.x) sb.Dh[(t / n) * (n + 1) + t % n] = basis[o.Dhat + t];
  for (int t = tid; t < n; t += blockDim.x) {
    sb.lm[t] = basis[o.lm + t];
    sb.lp[t] = basis[o.lp + t];
    sb.lhm[t] = basis[o.lhm + t];
    sb.lhp[t] = basis[o.lhp + t];
  }
}

// ---------------------------------------------------------------------------
// ProlongToFace of the state into the current trace buffer
// ---------------------------------------------------------------------------
template <int N, typename real, bool LGL>
__global__ void __launch_bounds__(Sz<N>::threads) k_trace(const View<real> *views, const int *blk_start, int nreq,
                                                         View<real> single) {
  using S = Sz<N>;
  constexpr int n = S::n, n2 = S::n2, n3 = S::n3, nf = S::nf, epb = S::epb;
  int lblk;
  const View<real> v = select_view(views, blk_start, nreq, single, lblk);
  __shared__ Smem<N, real> sb;
  __shared__ real sU[epb][5 * Pad<n>::size];
  load_basis<N, real>(sb, v.basis, threadIdx.x);
  const int le = threadIdx.x / n3, a = threadIdx.x - le * n3;
  const int64_t e = (int64_t)lblk * epb + le;
  const bool active = le < epb && e < v.E;
  const int64_t Ev = v.E * n3, Ef = v.E * 6 * n2;
  const uint32_t vi = (uint32_t)(e * n3 + a), fb = (uint32_t)(e * 6 * n2);
  const int i = a % n, j = (a / n) % n, k = a / n2;
  real *const su = sU[le < epb ? le : 0];
  if (active) {
#pragma unroll
    for (int c = 0; c < 5; ++c) su[c * Pad<n>::size + Pad<n>::at(i, j, k)] = to_real((v.U + c * Ev)[vi], c, v);
  }
  __syncthreads();
  if (active) {
    real *tr = v.cur ? v.Utr1 : v.Utr0;
    for (int fn = a; fn < nf; fn += n3) {
      const int f = fn / n2, pq = fn - f * n2;
      int base, stride;
      Pad<n>::face_line(f, pq, base, stride);
      real t[5];
      face_state<n, LGL>(su, (f & 1) ? sb.lp : sb.lm, base, stride, f & 1, t);
#pragma unroll
      for (int c = 0; c < 5; ++c) (tr + c * Ef)[fb + fn] = t[c];
    }
  }
}

// ---------------------------------------------------------------------------
// a-priori indicator (Sec. 2.3): modal energy of eps = rho p.  m = (V^-1 (x)
// V^-1 (x) V^-1) eps by three line transforms through LDS rows r0..r2 (V^-1
// staged in vs), then fixed-order sums of the energies (no atomics, so the
// value is reproducible): within each wave by lane exchanges and over the
// waves of the element through r3..r6 where elements and waves align, else a
// tree through r3..r6.  The energy fractions of the top two shells (modes
// whose largest degree is N, and N - 1) are summed directly rather than formed
// as differences of nearly equal totals: the same quantity, but its rounding
// is relative to itself, which in FP32 keeps the logistic's steep part from
// amplifying the cancellation.  Every thread of the block must call it.
// Returns the clipped logistic value on thread a == 0 of each element.
// ---------------------------------------------------------------------------
template <int N, typename real>
__device__ __forceinline__ real indicator_raw(const View<real> &v, const real *Vinv, real *r0, real *r1, real *r2,
                                              real *r3, real *r4, real *r5, real *r6, real *vs, bool active, int a,
                                              real eps) {
  constexpr int n = N + 1, n2 = n * n, n3 = n2 * n;
  const int i = a % n, j = (a / n) % n, k = a / n2;
  if (active) {
    for (int t = a; t < n2; t += n3) vs[t] = Vinv[t];
    r0[a] = eps;
  }
  __syncthreads();
  if (active) {
    real t = real(0);
#pragma unroll
    for (int r = 0; r < n; ++r) t += vs[i * n + r] * r0[vnode(n, r, j, k)];
    r1[a] = t;
  }
  __syncthreads();
  if (active) {
    real t = real(0);
#pragma unroll
    for (int r = 0; r < n; ++r) t += vs[j * n + r] * r1[vnode(n, i, r, k)];
    r2[a] = t;
  }
  __syncthreads();
  // energies: all modes, largest degree <= N - 1, largest degree N, largest degree N - 1
  real e0 = real(0), e1 = real(0), h1 = real(0), h2 = real(0);
  if (active) {
    real m = real(0);
#pragma unroll
    for (int r = 0; r < n; ++r) m += vs[k * n + r] * r2[vnode(n, i, j, r)];
    e0 = m * m;
    const int top = max(i, max(j, k));
    e1 = top < N ? e0 : real(0);
    h1 = top == N ? e0 : real(0);
    h2 = top == N - 1 ? e0 : real(0);
  }
  // each element's nodes fill whole waves (or the element is alone in the
  // workgroup): reduce within waves, then over the element's waves
  constexpr bool wave_sums = (n3 % 64 == 0) || Sz<N>::epb == 1;
  real tot = real(0), c1 = real(0), t1 = real(0), t2 = real(0);
  if constexpr (wave_sums) {
    // every lane takes part; lanes without a node add zeros
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      e0 += __shfl_xor(e0, off, 64);
      e1 += __shfl_xor(e1, off, 64);
      h1 += __shfl_xor(h1, off, 64);
      h2 += __shfl_xor(h2, off, 64);
    }
    constexpr int W = (n3 + 63) / 64;
    if (active && (a & 63) == 0) {
      r3[a >> 6] = e0;
      r4[a >> 6] = e1;
      r5[a >> 6] = h1;
      r6[a >> 6] = h2;
    }
    __syncthreads();
    if (active && a == 0) {
#pragma unroll
      for (int w = 0; w < W; ++w) {
        tot += r3[w];
        c1 += r4[w];
        t1 += r5[w];
        t2 += r6[w];
      }
    }
  } else {
    if (active) {
      r3[a] = e0;
      r4[a] = e1;
      r5[a] = h1;
      r6[a] = h2;
    }
    __syncthreads();
    constexpr int P2 = n3 <= 8 ? 8 : (n3 <= 16 ? 16 : (n3 <= 32 ? 32 : (n3 <= 64 ? 64 : (n3 <= 128 ? 128 : (n3 <= 256 ? 256 : (n3 <= 512 ? 512 : 1024))))));
#pragma unroll
    for (int st = P2 / 2; st > 0; st >>= 1) {
      if (active && a < st && a + st < n3) {
        r3[a] += r3[a + st];
        r4[a] += r4[a + st];
        r5[a] += r5[a + st];
        r6[a] += r6[a + st];
      }
      __syncthreads();
    }
    if (active && a == 0) {
      tot = r3[0];
      c1 = r4[0];
      t1 = r5[0];
      t2 = r6[0];
    }
  }
  real alpha = real(0);
  if (active && a == 0) {
    const real E1 = tot > real(0) ? t1 / tot : real(0);
    const real E2 = c1 > real(0) ? t2 / c1 : real(0);
    const real Ev = fmax(E1, E2);
    const real T = v.ind_T;
    alpha = real(1) / (real(1) + exp(-(v.ind_s / T) * (Ev - T)));
    if (alpha < v.alpha_min) alpha = real(0);
    else if (alpha > real(1) - v.alpha_min) alpha = real(1);
    alpha = fmin(alpha, v.alpha_max);
  }
  return alpha;
}

// reconstruction helpers of the FV subcells
template <typename real>
__device__ __forceinline__ real minmod2(real a, real b) {
  if (a * b <= real(0)) return real(0);
  return (a > real(0) ? real(1) : real(-1)) * fmin(fabs(a), fabs(b));
}

template <typename real>
__device__ __forceinline__ void prim2cons(const real *q, real gamma, real *U) {
  U[0] = q[0];
  U[1] = q[0] * q[1];
  U[2] = q[0] * q[2];
  U[3] = q[0] * q[3];
  U[4] = q[4] / (gamma - real(1)) + real(0.5) * q[0] * (q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
}

// ---------------------------------------------------------------------------
// Euler, with or without shock capturing: one sweep per stage.  Nothing of
// the inviscid operator waits for a neighbour's result (the blending factor
// is local to the element unless it is smoothed), so the state, the metrics
// and the register cross HBM once: FillFlux (Riemann flux of both sides' U
// traces), VolInt of F_adv through LDS one direction at a time, the SurfInt
// gather, ApplyJac, the stage update and the next U traces.  mode 0: du = A du + dt R, U += B du; mode 1: write
// R only.  SHOCK: the element's indicator value comes first; a workgroup with
// a blended element is listed for k_blend and stops.
// Reading all metrics it is bound by HBM: 8 (30 + 13 f) bytes per node, f =
// 6/(N+1) face nodes per node, 4.7 TB/s (28^3 at N = 5: 350 us; as two sweeps 210
// + 319 us).  With one node's metrics, 320 us, no single unit bounds it: 263 bytes
// per node measured (3.9 TB/s), FP64 at 0.18 of its peak, the LDS index unit
// active in 0.62 of the CU-busy cycles, and four waves per SIMD that wait half
// of theirs at the barriers between the phases.  A second buffer of flux rows
// (two barriers fewer) measured the same at N = 5 and 3% slower at N = 4.
// ---------------------------------------------------------------------------
template <int N, typename real, bool SHOCK, bool LGL, bool NT, int RS>
__global__ void __launch_bounds__(Sz<N>::threads, Sz<N>::minw) k_rhs(const View<real> *views, const int *blk_start,
                                                                      int nreq, View<real> single, int mode) {
  using S = Sz<N>;
  constexpr int n = S::n, n2 = S::n2, n3 = S::n3, nf = S::nf, epb = S::epb;
  int lblk;
  const View<real> v = select_view(views, blk_start, nreq, single, lblk);
  __shared__ Smem<N, real> sb;
  // per element: the state in padded rows (this side's traces; then the flux
  // rows of one direction; at the end the new state) and the face fluxes
  // (before them the indicator's rows)
  constexpr int rows = 5 * Pad<n>::size, faces = 5 * nf;
  __shared__ real sA[epb][rows + faces];
  __shared__ real sAl[epb];
  load_basis<N, real>(sb, v.basis, threadIdx.x);
  if (SHOCK && lblk == 0 && threadIdx.x == 0) v.bcnt[1 - v.bpar] = 0;  // the next sweep's count
  const int le = threadIdx.x / n3, a = threadIdx.x - le * n3;
  const int64_t e = (int64_t)lblk * epb + le;
  const bool active = le < epb && e < v.E;
  real *const su = sA[le < epb ? le : 0];
  real *const sf = su + rows;
  const int64_t Ev = v.E * n3, Ef = v.E * 6 * n2;
  const uint32_t vi = (uint32_t)(e * n3 + a), fb = (uint32_t)(e * 6 * n2);
  const uint32_t gi = one_node(v) ? (uint32_t)(e * n3) : vi;  // where this node's metrics stand
  const real gam = v.gamma, rR = v.rRgas;
  const Bg<real> bg{v.bg_p, v.bg_H};
  const real *tr = v.cur ? v.Utr1 : v.Utr0;
  const int i = a % n, j = (a / n) % n, k = a / n2;
  constexpr bool plane_waves = n2 == 64 && epb == 1;  // a wave is one face of one element
  const int pa = Pad<n>::at(i, j, k);
  constexpr int upt = (nf + n3 - 1) / n3;  // face nodes per thread
  double Uold[5] = {0, 0, 0, 0, 0};
  constexpr bool fp64 = sizeof(real) == sizeof(double);
  // Two orders of the loads.  Late: the state, the metrics and the first face
  // operands where they are used, the register before the gather; it takes the
  // fewest registers (N = 8 mixed: 71 VGPRs and two workgroups per CU, early 85
  // and one, 1.19 times the time; N = 5: early spills 4, 1.10 times).  Early:
  // all of them beside the state.  It pays with shock capturing, whose
  // indicator runs meanwhile, and in FP64 at N = 7 (0.80 of the late time at
  // 1.6 million DOF), N = 3 on Gauss nodes (0.95), N = 1 on Lobatto nodes (0.93),
  // and at N = 2 to 4 where the working set streams (0.95 on boxes).
  constexpr bool early = SHOCK || (fp64 && (N == 7 || (N == 3 && !LGL) || (N == 1 && LGL) ||
                                            (NT && (N == 3 || N == 4 || (N == 2 && LGL)))));
  constexpr bool ahead = early && fp64;  // the mixed form's metrics and face operands always late
  // this side's trace: recomputed from the state in LDS (40 f bytes per node
  // less) where the working set streams from HBM and f is large (N <= 5: 0.90 of
  // the time with stored ones at N = 1 and 3; N = 6: 1.06), else read with the
  // neighbour's; of a state in LDS for the indicator anyway, the end node's
  constexpr bool stored = !(SHOCK || (NT && N <= 5) || (fp64 && N == 1 && LGL));
  // streaming hints cost 2 to 15% at N <= 2, and 3 to 11% in FP64 at N = 8 and 9
  // from 4 to 8 million nodes on; else they are worth 1 to 11%
  constexpr bool hint = NT && (SHOCK || (N > 2 && !(fp64 && N >= 8)));
  // both sides' operands fetched in the order that the Riemann solver takes
  // them (by address), not ordered after the loads: 1 to 4% except at N = 1
  constexpr bool ordered = stored && !(fp64 && N == 1);
  constexpr bool rows_first = !stored || SHOCK;  // the face phase or the indicator reads the state's rows
  real Uo[5], Un[5], ns[3];
  bool prim = false;
  real Ja[9];
  // the neighbour's trace and the normal at face node fn
  auto fetch = [&](int fn) {
    int f = fn / n2;
    if constexpr (plane_waves) f = __builtin_amdgcn_readfirstlane(f);
    const int pq = fn - f * n2;
    const int2 c = v.conn[e * 6 + f];
    prim = (c.y >> 3) & 1;
    int pp, qq;
    orient_map(c.y & 7, pq % n, pq / n, N, pp, qq);
    const uint32_t in = (uint32_t)c.x * n2 + pp + n * qq;
#pragma unroll
    for (int s = 0; s < 5; ++s) {
      if constexpr (stored) Uo[s] = (tr + s * Ef)[ordered && !prim ? in : fb + fn];
      Un[s] = (tr + s * Ef)[ordered && !prim ? fb + fn : in];
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) ns[d] = (v.NS + d * Ef)[fb + (one_node(v) ? f * n2 : fn)];
  };
  if (active) {
    if constexpr (early || rows_first) {
#pragma unroll
      for (int c = 0; c < 5; ++c) Uold[c] = ld<hint>(v.U + c * Ev + vi);
    }
    // the first face node's operands beside the state; with more than one per
    // thread (N <= 4) the others' where they are used: held from here they
    // spilled at N = 4
    if (ahead && a < nf) fetch(a);
    if constexpr (ahead) {
#pragma unroll
      for (int c = 0; c < 9; ++c) Ja[c] = ld<hint>(v.Ja + c * Ev + gi);
    }
    if constexpr (rows_first) {
#pragma unroll
      for (int c = 0; c < 5; ++c) su[c * Pad<n>::size + pa] = to_real(Uold[c], c, v);
    }
  }
  if constexpr (SHOCK) {
    real eps = real(0);  // rho p
    if (active) {
      real U[5], P[6];
#pragma unroll
      for (int c = 0; c < 5; ++c) U[c] = to_real(Uold[c], c, v);
      cons2prim(U, gam, rR, P, bg);
      eps = P[0] * full_p(P[4], bg);
    }
    // the indicator's rows in the face area: V^-1, three line transforms, and
    // the energies (over the dead first two rows where they need whole rows)
    constexpr bool waves = (n3 % 64 == 0) || epb == 1;
    constexpr int en = waves ? (n3 + 63) / 64 : n3;
    static_assert(n2 + 3 * n3 + (waves ? 4 : 2) * en <= faces, "the indicator's rows must fit the face area");
    const BasisOffsets o(n);
    real *const r = sf + n2;
    real al;
    if constexpr (waves)
      al = indicator_raw<N, real>(v, v.basis + o.Vinv, r, r + n3, r + 2 * n3, r + 3 * n3, r + 3 * n3 + en,
                                  r + 3 * n3 + 2 * en, r + 3 * n3 + 3 * en, sf, active, a, eps);
    else
      al = indicator_raw<N, real>(v, v.basis + o.Vinv, r, r + n3, r + 2 * n3, r, r + n3, r + 3 * n3, r + 4 * n3, sf,
                                  active, a, eps);
    if (le < epb && a == 0) {
      if (active) {
        v.alpha_raw[e] = al;
        if (v.alpha_in) al = v.alpha_in[e];
        v.alpha[e] = al;
      }
      sAl[le] = active ? al : real(0);
    }
  }
  if constexpr (rows_first) __syncthreads();
  if constexpr (SHOCK) {
    bool any = false;
#pragma unroll
    for (int q = 0; q < epb; ++q) any = any || sAl[q] > real(0);
    if (any) {  // left to the blend pass
      if (threadIdx.x == 0) v.blist[atomicAdd(v.bcnt + v.bpar, 1)] = lblk;
      return;
    }
  }
  if (active) {
    // FillFlux for the six faces of this element
#pragma unroll (ahead ? upt : 1)
    for (int r = 0; r < upt; ++r) {
      const int fn = a + r * n3;
      if (fn < nf) {
        if (!ahead || r > 0) fetch(fn);
        int f = fn / n2;
        if constexpr (plane_waves) f = __builtin_amdgcn_readfirstlane(f);
        const int pq = fn - f * n2;
        if constexpr (!stored) {
          int base, stride;
          Pad<n>::face_line(f, pq, base, stride);
          face_state<n, LGL>(su, (f & 1) ? sb.lp : sb.lm, base, stride, f & 1, Uo);
        }
        const bool primary = prim;
        real Um[5], Us[5], Pm[6], Ps[6];
#pragma unroll
        for (int s = 0; s < 5; ++s) {
          Um[s] = ordered || primary ? Uo[s] : Un[s];
          Us[s] = ordered || primary ? Un[s] : Uo[s];
        }
        cons2prim(Um, gam, rR, Pm, bg);
        cons2prim(Us, gam, rR, Ps, bg);
        real nsv[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) nsv[d] = primary ? ns[d] : -ns[d];
        const real sh = sqrt(nsv[0] * nsv[0] + nsv[1] * nsv[1] + nsv[2] * nsv[2]);
        const real ish = real(1) / sh;
        const real nv[3] = {nsv[0] * ish, nsv[1] * ish, nsv[2] * ish};
        real Fs[5];
        riemann<RS>(v.riemann, Um, Pm, Us, Ps, nv, gam, Fs, bg);
#pragma unroll
        for (int s = 0; s < 5; ++s) sf[s * nf + fn] = primary ? Fs[s] * sh : -(Fs[s] * sh);
      }
    }
  }
  // 1/J and the RK register: early before the volume integral, late before the
  // gather; their latency overlaps it, and the register's loads precede its stores
  real iJ = real(0);
  double dUo[5] = {0, 0, 0, 0, 0};
  auto load_register = [&]() {
    iJ = v.invJ[gi];
#pragma unroll
    for (int c = 0; c < 5; ++c) dUo[c] = (mode == 0 && v.rkA != 0.0) ? ld<hint>(v.dU + c * Ev + vi) : 0.0;
  };
  real Fx[5], Fy[5], Fz[5];
  if (active) {
    // the FP64 copy in LDS is exact: read back rather than held through the
    // face phase (those registers spilled at N = 3 to 5)
    if constexpr (!early && !rows_first) {
#pragma unroll
      for (int c = 0; c < 5; ++c) Uold[c] = ld<hint>(v.U + c * Ev + vi);
    } else if constexpr (rows_first && fp64) {
#pragma unroll
      for (int c = 0; c < 5; ++c) Uold[c] = su[c * Pad<n>::size + pa];
    }
    real U[5], P[6];
#pragma unroll
    for (int c = 0; c < 5; ++c) U[c] = to_real(Uold[c], c, v);
    cons2prim(U, gam, rR, P, bg);
    if constexpr (!ahead) {
#pragma unroll
      for (int c = 0; c < 9; ++c) Ja[c] = ld<hint>(v.Ja + c * Ev + gi);
    }
    if constexpr (early) load_register();
    flux_adv<0>(U, P, Fx, bg);
    flux_adv<1>(U, P, Fy, bg);
    flux_adv<2>(U, P, Fz, bg);
  }
  if constexpr (rows_first) __syncthreads();  // the state rows are read above; flux rows cover them
  // VolInt: one computational direction at a time
  real V[5] = {0, 0, 0, 0, 0};
#pragma unroll
  for (int ci = 0; ci < 3; ++ci) {
    if (active) {
#pragma unroll
      for (int c = 0; c < 5; ++c) su[c * n3 + a] = Ja[3 * ci + 0] * Fx[c] + Ja[3 * ci + 1] * Fy[c] + Ja[3 * ci + 2] * Fz[c];
    }
    __syncthreads();
    if (active) {
      const int idx = ci == 0 ? i : (ci == 1 ? j : k);
#pragma unroll
      for (int alp = 0; alp < n; ++alp) {
        const int src = ci == 0 ? vnode(n, alp, j, k) : (ci == 1 ? vnode(n, i, alp, k) : vnode(n, i, j, alp));
        const real dh = sb.Dh[idx * (n + 1) + alp];
#pragma unroll
        for (int c = 0; c < 5; ++c) V[c] += dh * su[c * n3 + src];
      }
    }
    __syncthreads();
  }
  double Unew[5] = {0, 0, 0, 0, 0};
  if (active) {
    if constexpr (!early) load_register();
    // SurfInt gather (one writer per entry) and ApplyJac
    const int pqf[3] = {j + n * k, i + n * k, i + n * j};
    const int lf[3] = {i, j, k};
#pragma unroll
    for (int f = 0; f < 6; ++f) {
      const int d = f >> 1;
      const real lh = (f & 1) ? sb.lhp[lf[d]] : sb.lhm[lf[d]];
#pragma unroll
      for (int c = 0; c < 5; ++c) V[c] += sf[c * nf + f * n2 + pqf[d]] * lh;
    }
    double R[5];
#pragma unroll
    for (int c = 0; c < 5; ++c) R[c] = (double)(-(V[c] * iJ));
    if (v.source == 1) {
      const double x = v.Xs[vi], y = (v.Xs + Ev)[vi], z = (v.Xs + 2 * Ev)[vi];
      const double cs = 0.1 * M_PI * cos(M_PI * (x + y + z - v.t));
      const double gg = (double)gam;
      R[0] += 2.0 * cs;
      R[1] += 3.0 * cs;
      R[2] += 3.0 * cs;
      R[3] += 3.0 * cs;
      R[4] += 2.0 * (3.0 * gg - 2.0) / (gg - 1.0) * cs;
    }
    if (mode == 1) {
#pragma unroll
      for (int c = 0; c < 5; ++c) (v.R + c * Ev)[vi] = R[c];
    } else {
#pragma unroll
      for (int c = 0; c < 5; ++c) {
        // the first stage (A = 0) does not read the register: whatever it
        // holds (a restored state, an aborted step) cannot leak into the step
        const double du = (v.rkA != 0.0 ? v.rkA * dUo[c] : 0.0) + v.dt * R[c];
        st<hint>(du, v.dU + c * Ev + vi);
        Unew[c] = Uold[c] + v.rkB * du;
        st<hint>(Unew[c], v.U + c * Ev + vi);
      }
    }
  }
  if (mode == 0) {
    // ProlongToFace of the updated state for the next stage (the last barrier
    // of the volume integral precedes these writes)
    if (active) {
#pragma unroll
      for (int c = 0; c < 5; ++c) su[c * Pad<n>::size + pa] = to_real(Unew[c], c, v);
    }
    __syncthreads();
    if (active) {
      real *trn = v.cur ? v.Utr0 : v.Utr1;
      for (int fn = a; fn < nf; fn += n3) {
        int f = fn / n2;
        if constexpr (plane_waves) f = __builtin_amdgcn_readfirstlane(f);
        const int pq = fn - f * n2;
        int base, stride;
        Pad<n>::face_line(f, pq, base, stride);
        real t[5];
        face_state<n, LGL>(su, (f & 1) ? sb.lp : sb.lm, base, stride, f & 1, t);
#pragma unroll
        for (int c = 0; c < 5; ++c) st<hint>(t[c], trn + c * Ef + fb + fn);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// FV subcell volume term of one element (Sec. 2.3).  Subcells sit on the
// Lobatto nodes with interfaces at the cumulative weights; the interface
// metric accumulates w_m (D Ja)_m along each line from the element face;
// primitives are reconstructed with minmod slopes (zero in the two boundary
// subcells) and joined by the LLF flux.  `rows` are 16 LDS rows of n3 values
// of this element: 0-4 primitives, 5-7 the metric of one direction, 8-10
// w_l (D Ja)_l, 11-15 interface fluxes.  sFV holds SubOps.  Every
// thread of the workgroup calls it: it holds barriers.  Adds the subcell
// term at this node to Vfv (the sign convention of the DG volume integral).
// ---------------------------------------------------------------------------
// the 1-D operators of the subcells in LDS: D, w, 1/w, the distances from a
// node down and up to its interfaces, 1/(distance to the next node)
template <int n>
struct SubOps {
  static constexpr int D = 0, w = n * n, rw = w + n, lo = rw + n, hi = lo + n, rdx = hi + n, size = rdx + n;
};

template <int N, typename real>
__device__ __forceinline__ void fv_subcells(real *rows, const real *sFV, bool active, int a, int i, int j, int k,
                                            const real *P, const real *Ja, real gam, real rR, Bg<real> bg,
                                            real *Vfv) {
  constexpr int n = N + 1, n3 = n * n * n;
  using Q = SubOps<n>;
  const real *Dm = sFV + Q::D, *wq = sFV + Q::w, *rw = sFV + Q::rw, *rdx = sFV + Q::rdx;
  if (active) {
#pragma unroll
    for (int c = 0; c < 5; ++c) rows[c * n3 + a] = P[c];
  }
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const int l = d == 0 ? i : (d == 1 ? j : k);
    const int pp = d == 0 ? j : i, qq = d == 2 ? j : k;
    if (active) {
#pragma unroll
      for (int c = 0; c < 3; ++c) rows[(5 + c) * n3 + a] = Ja[3 * d + c];
    }
    __syncthreads();
    if (active) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        real s = real(0);
#pragma unroll
        for (int m = 0; m < n; ++m) s += Dm[l * n + m] * rows[(5 + c) * n3 + lnode<n>(d, m, pp, qq)];
        rows[(8 + c) * n3 + a] = wq[l] * s;
      }
    }
    __syncthreads();
    if (active && l < N) {
      real Jh[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        real acc = rows[(5 + c) * n3 + lnode<n>(d, 0, pp, qq)];
        for (int m = 0; m <= l; ++m) acc += rows[(8 + c) * n3 + lnode<n>(d, m, pp, qq)];
        Jh[c] = acc;
      }
      const real sh = sqrt(Jh[0] * Jh[0] + Jh[1] * Jh[1] + Jh[2] * Jh[2]);
      const real ish = real(1) / sh;
      const real nv[3] = {Jh[0] * ish, Jh[1] * ish, Jh[2] * ish};
      const real rd = rdx[l], rdm = rdx[l >= 1 ? l - 1 : 0], rdp = rdx[l + 1], up = sFV[Q::hi + l], dn = sFV[Q::lo + l + 1];
      real qL[5], qR[5];
#pragma unroll
      for (int c = 0; c < 5; ++c) {
        const real q0 = rows[c * n3 + lnode<n>(d, l, pp, qq)];
        const real q1 = rows[c * n3 + lnode<n>(d, l + 1, pp, qq)];
        real s0 = real(0), s1 = real(0);
        if (l >= 1) {
          const real qm = rows[c * n3 + lnode<n>(d, l - 1, pp, qq)];
          s0 = minmod2((q0 - qm) * rdm, (q1 - q0) * rd);
        }
        if (l + 1 <= N - 1) {
          const real q2 = rows[c * n3 + lnode<n>(d, l + 2, pp, qq)];
          s1 = minmod2((q1 - q0) * rd, (q2 - q1) * rdp);
        }
        qL[c] = q0 + s0 * up;
        qR[c] = q1 - s1 * dn;
      }
      real UL[5], UR[5], PL[6], PR[6], F[5];
      prim2cons(qL, gam, UL);
      prim2cons(qR, gam, UR);
      cons2prim(UL, gam, rR, PL, bg);
      cons2prim(UR, gam, rR, PR, bg);
      riemann_llf(UL, PL, UR, PR, nv, gam, F, bg);
#pragma unroll
      for (int c = 0; c < 5; ++c) rows[(11 + c) * n3 + a] = F[c] * sh;
    }
    __syncthreads();
    if (active) {
#pragma unroll
      for (int c = 0; c < 5; ++c) {
        real r = real(0);
        if (l < N) r += rows[(11 + c) * n3 + a];
        if (l > 0) r -= rows[(11 + c) * n3 + lnode<n>(d, l - 1, pp, qq)];
        Vfv[c] += r * rw[l];
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// The xi and eta contractions with D-hat of one row of node values, at N = 7
// in FP64, on the 4x4x4 four-block matrix instruction.  Its operands sit at
// A[m][k]: lane 16k + 4b + m, B[k][n]: lane 16k + 4b + n, and its result at
// D[m][n]: lane 16m + 4b + n.  A wave holds one k-plane with node (i, j) on
// lane i + 8j, so taking i = n + 4 (b & 1) and j = (b >> 1) + 2m as the output
// indices puts every result in the lane that owns the node.  xi: A = values
// (row j, source l), B = D-hat^T; eta: A = D-hat (row j), B = values (column i,
// source l); sources in two halves of four.  Each lane reads each value it
// feeds once, where the per-lane sums read it eight times.
// ---------------------------------------------------------------------------
struct PlaneMfma {
  int lk, ix, jx;
  double bx[2], ay[2];
  __device__ __forceinline__ explicit PlaneMfma(const double *Dh) {
    const int lane = threadIdx.x & 63;
    lk = lane >> 4;
    ix = lane & 7;
    jx = ((lane >> 3) & 1) + 2 * (lane & 3);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      bx[h] = Dh[ix * 9 + 4 * h + lk];
      ay[h] = Dh[jx * 9 + 4 * h + lk];
    }
  }
  __device__ __forceinline__ double xi(const double *plane, double acc) const {
#pragma unroll
    for (int h = 0; h < 2; ++h)
      acc = __builtin_amdgcn_mfma_f64_4x4x4f64(plane[vnode(8, 4 * h + lk, jx, 0)], bx[h], acc, 0, 0, 0);
    return acc;
  }
  __device__ __forceinline__ double eta(const double *plane, double acc) const {
#pragma unroll
    for (int h = 0; h < 2; ++h)
      acc = __builtin_amdgcn_mfma_f64_4x4x4f64(ay[h], plane[vnode(8, ix, 4 * h + lk, 0)], acc, 0, 0, 0);
    return acc;
  }
};

// Face work unit t of an element: the direction d and first side s0 of its
// face nodes and their face index pq.  fpu = 2: both sides of line pq; fpu = 1:
// face node t.  With plane waves each wave's units share one face direction.
template <int n, int fpu, bool plane_waves>
__device__ __forceinline__ void face_unit(int t, int &d, int &s0, int &pq) {
  constexpr int n2 = n * n;
  int g = t / n2;  // d (fpu = 2) or the face (fpu = 1)
  if constexpr (plane_waves) g = __builtin_amdgcn_readfirstlane(g);
  pq = t - g * n2;
  d = fpu == 2 ? g : g >> 1;
  s0 = fpu == 2 ? 0 : g & 1;
}

template <int N, typename real, bool SHOCK, bool SPLIT>
struct VolLds {
  using S = Sz<N>;
  static constexpr int n3 = S::n3, nf = S::nf;
  // per-element offsets.  Lifting: primitives u, v, w, T (4 rows of n3), the
  // nine metric rows Ja^i_d (9 x n3), with the split form the density (1 x
  // n3), BR1 face averages (4 x nf) and own outward n shat (3 x nf).  g (12
  // padded rows) then covers the first blocks, and the 15 rows of
  // contravariant fluxes the whole area.
  static constexpr int V = 0, J = 4 * n3, Rho = 13 * n3, Avg = (SPLIT ? 14 : 13) * n3, Ns = Avg + 4 * nf, G = 0,
                       F = 0;
  static constexpr int gsz = Pad<S::n>::size;  // one padded row of g
  static constexpr int rows = (Ns + 3 * nf) > 15 * n3 ? (Ns + 3 * nf) : 15 * n3;
  // Face work units: with fpu = 2 a thread takes the two face nodes at the
  // ends of one line of nodes, so the line of g is read once for both; with
  // fpu = 1 one face node.  Two per unit halves the LDS reads of
  // Lift_ProlongToFace but also the threads that share them.  Measured per
  // degree on ~7M-DOF meshes, one per unit is faster at N = 6, and at N = 5
  // in FP64; two elsewhere (8% less volume-sweep time at N = 3, 3% at N = 7).
  // The FP64 sweeps at N = 9 and with shock capturing or the split form at
  // N = 7 take one: two would spill registers.
  static constexpr bool f64 = sizeof(real) == 8;
  static constexpr int fpu = (N == 6 || (f64 && (N == 5 || N >= 9 || (N == 7 && (SHOCK || SPLIT))))) ? 1 : 2;
  // Nodes per thread: at N = 7 (and N = 5 in the mixed form; one element
  // per workgroup, even n) a thread of the standard form without shock
  // capturing takes the two nodes k and k + n/2 of one column.  They share
  // the reads along zeta, the D-hat rows along xi and eta and the zeta faces
  // of Lift_SurfInt; the workgroup has half the threads, each with twice the
  // registers.  That took 7% off the mixed sweep at both degrees and 2 to 3%
  // off the FP64 sweep at N = 7, where the lifting contraction is unrolled by
  // 2 instead of n: fully unrolled, its loads in flight spilled past 256 VGPRs
  // (by 4: 216 VGPRs and slower than by 2, 176 VGPRs; not unrolled: slower
  // again).
  static constexpr bool plane_waves = S::n2 == 64 && S::epb == 1;
  static constexpr int npt = ((N == 7 && !SHOCK && !SPLIT) || (N == 5 && !SHOCK && !SPLIT && !f64)) ? 2 : 1;
  // The split form's loop also carries the two-point flux: not unrolled, it
  // fits the register budget of two 512-thread workgroups per CU at N = 7
  // (128 VGPRs, one spill; unrolled by 2 it needed 148, which left one
  // workgroup per CU and took 1.04 ms instead of 0.68 ms on the 24^3
  // supersonic TGV; 0.79 against 0.68 ms at N = 5).
  static constexpr int lift_unroll = SPLIT ? 1 : ((npt == 2 && f64) ? 2 : S::n);
  static constexpr int tpe = n3 / npt;  // threads per element
  static constexpr int threads = npt == 1 ? S::threads : tpe;
  static constexpr int minw = npt == 1 ? S::minw : 2;
  // FP64 at N = 7 (a wave is one k-plane): the xi and eta contractions of the
  // volume integral on the matrix cores (4x4x4, four blocks), results in the
  // lanes that own them (see k_volume)
  static constexpr bool mfma = f64 && N == 7;
  static constexpr int units = nf / fpu;
  static constexpr int upt = (units + tpe - 1) / tpe;  // units per thread
  static_assert(12 * gsz <= Ns, "g must not cover n shat");
  static_assert(npt == 1 || (S::n % 2 == 0 && S::epb == 1), "column pairs need an even n and one element");
};

// ---------------------------------------------------------------------------
// Volume sweep.  From the lifted gradient, which never leaves the chip, it
// forms (a) at each own face node this side's viscous normal flux
// H = F_v(prim, g).n shat, with n in the primary side's orientation, and (b) the
// complete volume integral of F_adv - F_v.  Writes H (4 values per face node:
// the mass component is zero) and the volume integral (5 per node); with
// shock capturing also the element's indicator value; with DIAG the
// element's dissipation sums (View::diag).  SUTH: Sutherland's law for the
// viscosity (a template flag: its divisions would cost the constant-viscosity
// sweeps registers).
// Split form (SPLIT, Gauss-Lobatto nodes; Sec. 2.2 "Nonlinear Stability"):
// the advective part of the volume integral becomes
//   sum_alpha (D + D-hat)_{i alpha} F#(U_ijk, U_alpha jk; mean Ja^1) + ...
// with Pirozzoli's two-point flux F#.  On Gauss-Lobatto nodes D + D-hat =
// 2 D - W^-1 B (summation by parts), so this is the strong split form with
// the boundary values of its surface correction folded in, and the weak
// form's surface integral of f* completes it.  The two-point fluxes take
// their operands from the rows the lifting contraction reads anyway (the
// metric rows, u, v, w, T) plus one density row; pressure and enthalpy
// follow from them: p = rho R T, H = gamma R T/(gamma - 1) + |u|^2/2.
// The viscous part keeps the weak form.
// ---------------------------------------------------------------------------
template <int N, typename real, bool SHOCK, bool LGL, bool SPLIT, bool SUTH, bool DIAG = false, bool NT = false>
__global__ void __launch_bounds__((VolLds<N, real, SHOCK, SPLIT>::threads), (VolLds<N, real, SHOCK, SPLIT>::minw))
    k_volume(const View<real> *views, const int *blk_start, int nreq, View<real> single) {
  using S = Sz<N>;
  using L = VolLds<N, real, SHOCK, SPLIT>;
  constexpr int n = S::n, n2 = S::n2, n3 = S::n3, nf = S::nf, epb = S::epb;
  constexpr int npt = L::npt, tpe = L::tpe, kstep = n / npt;
  static_assert(!SPLIT || LGL, "the split form needs Gauss-Lobatto nodes");
  int lblk;
  const View<real> v = select_view(views, blk_start, nreq, single, lblk);
  __shared__ Smem<N, real> sb;
  __shared__ __align__(16) real sA[epb][L::rows];
  // (D + D-hat)/16, rows padded to n + 1: the weights of the two-point sums
  // (two_point_kep_sums), exact scaling by a power of two
  __shared__ real sDs[SPLIT ? n * (n + 1) : 1];
  load_basis<N, real>(sb, v.basis, threadIdx.x);
  if constexpr (SPLIT) {
    const BasisOffsets o(n);
    for (int t = threadIdx.x; t < n * n; t += blockDim.x)
      sDs[(t / n) * (n + 1) + t % n] = (v.basis[o.D + t] + v.basis[o.Dhat + t]) * real(0.0625);
  }
  // thread a of an element holds its nodes a + m tpe, m < npt: the same i and
  // j, and k = k0 + m kstep
  const int le = threadIdx.x / tpe, a = threadIdx.x - le * tpe;
  const int64_t e = (int64_t)lblk * epb + le;
  const bool active = le < epb && e < v.E;
  real *const sm = sA[le < epb ? le : 0];
  // row strides of the volume and face arrays; per-lane indices are 32-bit
  // (the host keeps every row below 2^31 entries)
  const int64_t Ev = v.E * n3, Ef = v.E * 6 * n2;
  const uint32_t vi = (uint32_t)(e * n3 + a), fb = (uint32_t)(e * 6 * n2);
  const uint32_t gi = one_node(v) ? (uint32_t)(e * n3) : vi, gstep = one_node(v) ? 0 : tpe;  // where the metrics stand
  const real gam = v.gamma, rR = v.rRgas, mu = v.mu, lam = v.lambda;
  const Bg<real> bg{v.bg_p, v.bg_H};
  const bool visc = v.viscous != 0;  // the same for the whole grid
  constexpr bool suth = SUTH;
  const real *tr = v.cur ? v.Utr1 : v.Utr0;
  const int i = a % n, j = (a / n) % n, k0 = a / n2;
  // when a wave is one k-plane of one element (n^2 = 64), the k rows of D-hat
  // and the face of a face node are the same on every lane: scalar loads
  // instead of LDS reads
  constexpr bool plane_waves = L::plane_waves;
  real dk[npt][n];
  if constexpr (plane_waves) {
    const int ku = __builtin_amdgcn_readfirstlane(k0);
    const BasisOffsets o(n);
#pragma unroll
    for (int m = 0; m < npt; ++m)
#pragma unroll
      for (int al = 0; al < n; ++al) dk[m][al] = v.basis[o.Dhat + (ku + m * kstep) * n + al];
  }
  real U[npt][5];
  real pf[L::upt][L::fpu][4];  // own face velocity and viscosity at this thread's face nodes
  real mun[npt];               // viscosity at this thread's nodes (Sutherland: mu(T), computed early,
                               // where few registers are live)
  if (active) {
#pragma unroll
    for (int m = 0; m < npt; ++m)
#pragma unroll
      for (int c = 0; c < 5; ++c) U[m][c] = to_real(ld<NT>(v.U + c * Ev + vi + m * tpe), c, v);
  }
  // 1/J at this thread's nodes, fetched beside the state: its first use comes
  // after the lifting sums, and a load issued there would stall the wave
  real iJe[npt];
  if (active && visc) {
#pragma unroll
    for (int m = 0; m < npt; ++m) iJe[m] = v.invJ[gi + m * gstep];
  }
  // Lift_FillFlux operands: both sides' U traces and this side's n shat at
  // the thread's face nodes.  With one node per thread they are fetched here,
  // beside the state, which hides their latency behind the metric loads (the
  // split-form sweep 3.9% faster at N = 7); the column-pair sweep fetches
  // them where it uses them (1% faster so).
  real tUo[L::upt][L::fpu][5], tUn[L::upt][L::fpu][5], tNs[L::upt][L::fpu][3];
  bool prim[L::upt][L::fpu];  // this side is the face's primary side (read with the traces)
  auto fetch_face = [&](int r, int u, int f, int fn, int pq) {
    const int2 c = v.conn[e * 6 + f];
    prim[r][u] = (c.y >> 3) & 1;
    int pp, qq;
    orient_map(c.y & 7, pq % n, pq / n, N, pp, qq);
    const uint32_t io = fb + fn, in = (uint32_t)c.x * n2 + pp + n * qq;
#pragma unroll
    for (int s = 0; s < 5; ++s) {
      tUo[r][u][s] = (tr + s * Ef)[io];
      tUn[r][u][s] = (tr + s * Ef)[in];
    }
#pragma unroll
    for (int dd = 0; dd < 3; ++dd) tNs[r][u][dd] = (v.NS + dd * Ef)[one_node(v) ? fb + f * n2 : io];
  };
  if (npt == 1 && active && visc) {
#pragma unroll
    for (int r = 0; r < L::upt; ++r) {
      const int t = a + r * tpe;
      if (t < L::units) {
        int d, s0, pq;
        face_unit<n, L::fpu, plane_waves>(t, d, s0, pq);
#pragma unroll
        for (int u = 0; u < L::fpu; ++u) fetch_face(r, u, 2 * d + s0 + u, (2 * d + s0 + u) * n2 + pq, pq);
      }
    }
  }
  if constexpr (SHOCK) {
    static_assert(npt == 1, "the indicator takes one node per thread");
    // a-priori indicator of this element (Sec. 2.3) on epsilon = rho p, in the
    // metric rows before they are filled
    real eps = real(0);
    if (active) {
      real P[6];
      cons2prim(U[0], gam, rR, P, bg);
      eps = P[0] * full_p(P[4], bg);
    }
    const BasisOffsets o(n);
    real *r = sm + L::J;
    const real al = indicator_raw<N, real>(v, v.basis + o.Vinv, r, r + n3, r + 2 * n3, r + 3 * n3, r + 4 * n3,
                                           r + 5 * n3, r + 6 * n3, r + 7 * n3, active, a, eps);
    if (active && a == 0) v.alpha_raw[e] = al;
    __syncthreads();
  }
  if (active) {
#pragma unroll
    for (int m = 0; m < npt; ++m) {
      const int am = a + m * tpe;
#pragma unroll
      for (int c = 0; c < 9; ++c) sm[L::J + c * n3 + am] = ld<NT>(v.Ja + c * Ev + gi + m * gstep);
      real P[6];
      cons2prim(U[m], gam, rR, P, bg);
      sm[L::V + 0 * n3 + am] = P[1];
      sm[L::V + 1 * n3 + am] = P[2];
      sm[L::V + 2 * n3 + am] = P[3];
      sm[L::V + 3 * n3 + am] = P[5];
      if constexpr (SPLIT) sm[L::Rho + am] = P[0];
      mun[m] = suth ? sutherland(P[5], mu, v.rTref) : mu;
    }
  }
  if (active && visc) {
    // Lift_FillFlux: the BR1 average of both sides' traces, and this side's
    // outward n shat, face velocity and temperature for its viscous flux later on
#pragma unroll
    for (int r = 0; r < L::upt; ++r) {
      const int t = a + r * tpe;
      if (t < L::units) {
        int d, s0, pq;
        face_unit<n, L::fpu, plane_waves>(t, d, s0, pq);
#pragma unroll
        for (int u = 0; u < L::fpu; ++u) {
          const int f = 2 * d + s0 + u, fn = f * n2 + pq;
          if constexpr (npt != 1) fetch_face(r, u, f, fn, pq);
          real Po[6], Pn[6];
          cons2prim(tUo[r][u], gam, rR, Po, bg);
          cons2prim(tUn[r][u], gam, rR, Pn, bg);
          const real vo[4] = {Po[1], Po[2], Po[3], Po[5]}, vn[4] = {Pn[1], Pn[2], Pn[3], Pn[5]};
#pragma unroll
          for (int s = 0; s < 4; ++s) sm[L::Avg + s * nf + fn] = real(0.5) * (vo[s] + vn[s]);
#pragma unroll
          for (int dd = 0; dd < 3; ++dd) {
            sm[L::Ns + dd * nf + fn] = tNs[r][u][dd];
            pf[r][u][dd] = Po[1 + dd];
          }
          pf[r][u][3] = suth ? sutherland(Po[5], mu, v.rTref) : mu;
        }
      }
    }
  }
  __syncthreads();
  real Fc[npt][15];  // contravariant fluxes Ja^i . (F_adv - F_v), i = 0..2 (split form: -F_v only)
  real g[npt][12];
  real Vs[npt][5];   // split form: the advective volume integral of the two-point fluxes
#pragma unroll
  for (int m = 0; m < npt; ++m) {
#pragma unroll
    for (int c = 0; c < 12; ++c) g[m][c] = real(0);
#pragma unroll
    for (int c = 0; c < 5; ++c) Vs[m][c] = real(0);
  }
  if (active && (visc || SPLIT)) {
    // Lift_VolInt along the three computational directions.  Along xi and eta
    // a thread's nodes share the D-hat row; along zeta they share the line.
    // The split form's two-point fluxes ride on the same reads.
    real JG[npt][12];
#pragma unroll
    for (int m = 0; m < npt; ++m)
#pragma unroll
      for (int c = 0; c < 12; ++c) JG[m][c] = real(0);
    // own operands of the two-point flux (split form): rho, u, v, w, 4 p and 2 H
    real orho[npt], ou[npt], ov[npt], ow[npt], op4[npt], oH2[npt];
    const real R4 = v.Rgas4, cp2R = v.cpR2;
    if constexpr (SPLIT) {
#pragma unroll
      for (int m = 0; m < npt; ++m) {
        const int am = a + m * tpe;
        orho[m] = sm[L::Rho + am];
        ou[m] = sm[L::V + am];
        ov[m] = sm[L::V + n3 + am];
        ow[m] = sm[L::V + 2 * n3 + am];
        const real T = sm[L::V + 3 * n3 + am];
        op4[m] = orho[m] * (R4 * T);
        oH2[m] = cp2R * T + (ou[m] * ou[m] + ov[m] * ov[m] + ow[m] * ow[m]);
      }
    }
#pragma unroll
    for (int ci = 0; ci < 3; ++ci) {
      const real *Jr = sm + L::J + 3 * ci * n3;
      real oJ[npt][3];  // own metric vector Ja^ci (split form)
      if constexpr (SPLIT) {
#pragma unroll
        for (int m = 0; m < npt; ++m)
#pragma unroll
          for (int d = 0; d < 3; ++d) oJ[m][d] = Jr[d * n3 + a + m * tpe];
      }
      if constexpr (!SPLIT) {
#pragma unroll L::lift_unroll
      for (int al = 0; al < n; ++al) {
        if (ci < 2) {
          const real dh = sb.Dh[(ci == 0 ? i : j) * (n + 1) + al];
#pragma unroll
          for (int m = 0; m < npt; ++m) {
            const int km = k0 + m * kstep;
            const int src = ci == 0 ? vnode(n, al, j, km) : vnode(n, i, al, km);
            const real dj[3] = {dh * Jr[src], dh * Jr[n3 + src], dh * Jr[2 * n3 + src]};
            const real vv[4] = {sm[L::V + src], sm[L::V + n3 + src], sm[L::V + 2 * n3 + src],
                                sm[L::V + 3 * n3 + src]};
#pragma unroll
            for (int d = 0; d < 3; ++d)
#pragma unroll
              for (int s = 0; s < 4; ++s) JG[m][d * 4 + s] += dj[d] * vv[s];
          }
        } else {
          const int src = vnode(n, i, j, al);
          const real jr[3] = {Jr[src], Jr[n3 + src], Jr[2 * n3 + src]};
          const real vv[4] = {sm[L::V + src], sm[L::V + n3 + src], sm[L::V + 2 * n3 + src], sm[L::V + 3 * n3 + src]};
#pragma unroll
          for (int m = 0; m < npt; ++m) {
            const real dh = plane_waves ? dk[m][al] : sb.Dh[(k0 + m * kstep) * (n + 1) + al];
            const real dj[3] = {dh * jr[0], dh * jr[1], dh * jr[2]};
#pragma unroll
            for (int d = 0; d < 3; ++d)
#pragma unroll
              for (int s = 0; s < 4; ++s) JG[m][d * 4 + s] += dj[d] * vv[s];
          }
        }
      }
      } else {
      // one source node of node m's line: lifting sums and the split form's two-point flux
      auto take = [&](int m, int idx, int al, int src, const real *jr, const real *vv, real dh) {
        if (visc) {
          // D-hat times the metric first: 3 products and 12 multiply-adds per source node
          const real dj[3] = {dh * jr[0], dh * jr[1], dh * jr[2]};
#pragma unroll
          for (int d = 0; d < 3; ++d)
#pragma unroll
            for (int s = 0; s < 4; ++s) JG[m][d * 4 + s] += dj[d] * vv[s];
        }
        if constexpr (SPLIT) {
          const real rs = sm[L::Rho + src];
          const real ps4 = rs * (R4 * vv[3]);
          const real Hs2 = cp2R * vv[3] + (vv[0] * vv[0] + vv[1] * vv[1] + vv[2] * vv[2]);
          real G[5];
          two_point_kep_sums(orho[m] + rs, ou[m] + vv[0], ov[m] + vv[1], ow[m] + vv[2], op4[m] + ps4, oH2[m] + Hs2,
                             oJ[m][0] + jr[0], oJ[m][1] + jr[1], oJ[m][2] + jr[2], G);
          const real ds = sDs[idx * (n + 1) + al];  // (D + D-hat)/16
#pragma unroll
          for (int c = 0; c < 5; ++c) Vs[m][c] += ds * G[c];
        }
      };
#pragma unroll L::lift_unroll
      for (int al = 0; al < n; ++al) {
        if (ci < 2) {
          const real dh = sb.Dh[(ci == 0 ? i : j) * (n + 1) + al];
#pragma unroll
          for (int m = 0; m < npt; ++m) {
            const int km = k0 + m * kstep;
            const int src = ci == 0 ? vnode(n, al, j, km) : vnode(n, i, al, km);
            const real jr[3] = {Jr[src], Jr[n3 + src], Jr[2 * n3 + src]};
            const real vv[4] = {sm[L::V + src], sm[L::V + n3 + src], sm[L::V + 2 * n3 + src],
                                sm[L::V + 3 * n3 + src]};
            take(m, ci == 0 ? i : j, al, src, jr, vv, dh);
          }
        } else {
          const int src = vnode(n, i, j, al);
          const real jr[3] = {Jr[src], Jr[n3 + src], Jr[2 * n3 + src]};
          const real vv[4] = {sm[L::V + src], sm[L::V + n3 + src], sm[L::V + 2 * n3 + src], sm[L::V + 3 * n3 + src]};
#pragma unroll
          for (int m = 0; m < npt; ++m) {
            const int km = k0 + m * kstep;
            const real dh = plane_waves ? dk[m][al] : sb.Dh[km * (n + 1) + al];
            take(m, km, al, src, jr, vv, dh);
          }
        }
      }
      }
    }
    if (visc) {
      // Lift_SurfInt: the face average times n shat, through l-hat
#pragma unroll
      for (int f = 0; f < 6; ++f) {
        const int d = f >> 1;
        const int end = (f & 1) ? n - 1 : 0;  // the only node with nonzero l-hat at Gauss-Lobatto nodes
        if (d < 2) {
          if (LGL && (d == 0 ? i : j) != end) continue;
          const real lh = (f & 1) ? sb.lhp[d == 0 ? i : j] : sb.lhm[d == 0 ? i : j];
#pragma unroll
          for (int m = 0; m < npt; ++m) {
            const int km = k0 + m * kstep;
            const int fn = f * n2 + (d == 0 ? j : i) + n * km;
            const real av[4] = {sm[L::Avg + fn], sm[L::Avg + nf + fn], sm[L::Avg + 2 * nf + fn],
                                sm[L::Avg + 3 * nf + fn]};
#pragma unroll
            for (int dd = 0; dd < 3; ++dd) {
              const real nl = sm[L::Ns + dd * nf + fn] * lh;
#pragma unroll
              for (int s = 0; s < 4; ++s) JG[m][dd * 4 + s] += av[s] * nl;
            }
          }
        } else {
          const int fn = f * n2 + i + n * j;
          const real av[4] = {sm[L::Avg + fn], sm[L::Avg + nf + fn], sm[L::Avg + 2 * nf + fn], sm[L::Avg + 3 * nf + fn]};
          const real ns[3] = {sm[L::Ns + fn], sm[L::Ns + nf + fn], sm[L::Ns + 2 * nf + fn]};
#pragma unroll
          for (int m = 0; m < npt; ++m) {
            const int km = k0 + m * kstep;
            if (LGL && km != end) continue;
            const real lh = (f & 1) ? sb.lhp[km] : sb.lhm[km];
#pragma unroll
            for (int dd = 0; dd < 3; ++dd) {
              const real nl = ns[dd] * lh;
#pragma unroll
              for (int s = 0; s < 4; ++s) JG[m][dd * 4 + s] += av[s] * nl;
            }
          }
        }
      }
#pragma unroll
      for (int m = 0; m < npt; ++m) {
#pragma unroll
        for (int c = 0; c < 12; ++c) {
          g[m][c] = JG[m][c] * iJe[m];
          // formed here: sunk into the branch of the dissipation sums, their
          // arithmetic left every loaded operand live (418 spilled registers at N = 9)
          if constexpr (DIAG) asm volatile("" : "+v"(g[m][c]));
        }
      }
    }
  }
  // dissipation sums of Sec. 5.2 at this thread's nodes: w J mu |curl u|^2 and w J mu (div u)^2
  if constexpr (DIAG) {
    double dS = 0.0, dD = 0.0, dW = 0.0;
    if (active && visc) {
      const BasisOffsets o(n);
      const real *wq = v.basis + o.w;
#pragma unroll
      for (int m = 0; m < npt; ++m) {
        const real *gm = g[m];
        const double T = (double)sm[L::V + 3 * n3 + a + m * tpe];
        const double mud = v.visc_law ? sutherland<double>(T, (double)mu, (double)v.rTref) : (double)mu;
        const double wJ = (double)wq[i] * (double)wq[j] * (double)wq[k0 + m * kstep] / (double)v.invJ[gi + m * gstep];
        const double wx = (double)gm[1 * 4 + 2] - (double)gm[2 * 4 + 1];
        const double wy = (double)gm[2 * 4 + 0] - (double)gm[0 * 4 + 2];
        const double wz = (double)gm[0 * 4 + 1] - (double)gm[1 * 4 + 0];
        const double dv = (double)gm[0] + (double)gm[5] + (double)gm[10];
        dS += wJ * mud * (wx * wx + wy * wy + wz * wz);
        dD += wJ * mud * dv * dv;
        dW += wJ;
      }
    }
    // the element's sums in a fixed order (reproducible, no atomics): sixteen
    // threads each take every sixteenth node, then one adds their sums.  A
    // dissipation sweep needs nothing past the gradients, so it ends here (the
    // call on 24^3 at N = 7, 90 us of traces included: 677 us with one thread
    // adding all nodes and the face fluxes and volume integral written too, 422
    // us now)
    __syncthreads();  // the rows read above are covered below
    constexpr int parts = tpe < 16 ? tpe : 16;
    // 3 (tpe + 16) doubles per element fit its rows at every degree and precision
    static_assert(epb * L::rows * sizeof(real) >= epb * 3 * (tpe + 16) * sizeof(double), "sums in LDS");
    double *sd = (double *)&sA[0][0] + (le < epb ? le : 0) * 3 * (tpe + 16);
    if (active) {
      sd[a] = dS;
      sd[tpe + a] = dD;
      sd[2 * tpe + a] = dW;
    }
    __syncthreads();
    if (active && a < parts) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        double s = 0.0;
        for (int t = a; t < tpe; t += parts) s += sd[c * tpe + t];
        sd[3 * tpe + c * 16 + a] = s;
      }
    }
    __syncthreads();
    if (active && a < 3) {
      double s = 0.0;
#pragma unroll
      for (int t = 0; t < parts; ++t) s += sd[3 * tpe + a * 16 + t];
      v.diag[3 * e + a] = s;
    }
    return;
  }
  if (active) {
    // volume fluxes at each node, projected on the three contravariant directions
#pragma unroll
    for (int m = 0; m < npt; ++m) {
      const int am = a + m * tpe;
      real P[6];
      cons2prim(U[m], gam, rR, P, bg);
      real Fx[5], Fy[5], Fz[5];
      if constexpr (SPLIT) {
#pragma unroll
        for (int c = 0; c < 5; ++c) Fx[c] = Fy[c] = Fz[c] = real(0);
      } else {
        flux_adv<0>(U[m], P, Fx, bg);
        flux_adv<1>(U[m], P, Fy, bg);
        flux_adv<2>(U[m], P, Fz, bg);
      }
      if (visc) {
        const real lamn = suth ? mun[m] * v.kappa : lam;
        real Vx[5], Vy[5], Vz[5];
        flux_visc<0>(P, g[m], mun[m], lamn, Vx);
        flux_visc<1>(P, g[m], mun[m], lamn, Vy);
        flux_visc<2>(P, g[m], mun[m], lamn, Vz);
#pragma unroll
        for (int c = 0; c < 5; ++c) {
          Fx[c] -= Vx[c];
          Fy[c] -= Vy[c];
          Fz[c] -= Vz[c];
        }
      }
#pragma unroll
      for (int ci = 0; ci < 3; ++ci) {
        const real j0 = sm[L::J + (3 * ci) * n3 + am], j1 = sm[L::J + (3 * ci + 1) * n3 + am],
                   j2 = sm[L::J + (3 * ci + 2) * n3 + am];
#pragma unroll
        for (int c = 0; c < 5; ++c) Fc[m][5 * ci + c] = j0 * Fx[c] + j1 * Fy[c] + j2 * Fz[c];
      }
    }
  }
  __syncthreads();  // the rows read above are covered by g below
  if (active && visc) {
#pragma unroll
    for (int m = 0; m < npt; ++m) {
      const int pa = Pad<n>::at(i, j, k0 + m * kstep);
#pragma unroll
      for (int c = 0; c < 12; ++c) sm[L::G + c * L::gsz + pa] = g[m][c];
    }
  }
  __syncthreads();
  if (active && visc) {
    // Lift_ProlongToFace of g, then this side's viscous normal flux
#pragma unroll
    for (int r = 0; r < L::upt; ++r) {
      const int t = a + r * tpe;
      if (t < L::units) {
        int d, s0, pq;
        face_unit<n, L::fpu, plane_waves>(t, d, s0, pq);
        int base, stride;
        Pad<n>::face_line(2 * d, pq, base, stride);
        // l(-1) and l(+1) weights: scalar loads where the face is the same on
        // every lane
        const BasisOffsets o(n);
        const real *lw[L::fpu];
#pragma unroll
        for (int u = 0; u < L::fpu; ++u) {
          const bool plus = (s0 + u) != 0;
          lw[u] = plane_waves ? v.basis + (plus ? o.lp : o.lm) : (plus ? sb.lp : sb.lm);
        }
        real gt[L::fpu][12];
#pragma unroll
        for (int u = 0; u < L::fpu; ++u)
#pragma unroll
          for (int s = 0; s < 12; ++s) gt[u][s] = real(0);
        if constexpr (LGL) {
          // Gauss-Lobatto: the trace is the end node of the line
#pragma unroll
          for (int u = 0; u < L::fpu; ++u) {
            const real *row = sm + L::G + base + ((s0 + u) != 0 ? (n - 1) * stride : 0);
#pragma unroll
            for (int s = 0; s < 12; ++s) gt[u][s] = row[s * L::gsz];
          }
        } else {
#pragma unroll
          for (int l = 0; l < n; ++l) {
            real w[L::fpu];
#pragma unroll
            for (int u = 0; u < L::fpu; ++u) w[u] = lw[u][l];
            const real *row = sm + L::G + base + l * stride;
#pragma unroll
            for (int s = 0; s < 12; ++s) {
              const real gv = row[s * L::gsz];
#pragma unroll
              for (int u = 0; u < L::fpu; ++u) gt[u][s] += w[u] * gv;
            }
          }
        }
#pragma unroll
        for (int u = 0; u < L::fpu; ++u) {
          const int f = 2 * d + s0 + u, fn = f * n2 + pq;
          const bool primary = prim[r][u];
          real nsv[3];
#pragma unroll
          for (int dd = 0; dd < 3; ++dd) {
            const real ns = sm[L::Ns + dd * nf + fn];
            nsv[dd] = primary ? ns : -ns;
          }
          const real muf = pf[r][u][3];
          const real lamf = suth ? muf * v.kappa : lam;
          real H[5];
          flux_visc_face(pf[r][u], gt[u], muf, lamf, nsv, H);
#pragma unroll
          for (int s = 1; s < 5; ++s) st<NT>(H[s], v.Hv + (s - 1) * Ef + fb + fn);
        }
      }
    }
  }
  __syncthreads();  // g and n shat are read above; the flux rows below cover them
  // VolInt: the fluxes of all three directions at once (split form: the
  // viscous fluxes; without viscosity there is nothing left to contract)
  const bool contract = !SPLIT || visc;
  // the viscous fluxes have no mass component: the split form contracts four
  constexpr int c0 = SPLIT ? 1 : 0;
  if (active && contract) {
#pragma unroll
    for (int m = 0; m < npt; ++m)
#pragma unroll
      for (int c = 0; c < 15; ++c)
        if (c % 5 >= c0) sm[L::F + c * n3 + a + m * tpe] = Fc[m][c];
  }
  __syncthreads();
  if (active) {
    real Vi[npt][5];
#pragma unroll
    for (int m = 0; m < npt; ++m)
#pragma unroll
      for (int c = 0; c < 5; ++c) Vi[m][c] = real(0);
    if constexpr (L::mfma) {
      if (contract) {
        const PlaneMfma M(sb.Dh);
#pragma unroll
        for (int m = 0; m < npt; ++m) {
          const int km = k0 + m * kstep;
#pragma unroll
          for (int c = c0; c < 5; ++c) {
            Vi[m][c] = M.xi(sm + L::F + c * n3 + n2 * km, 0.0);
            Vi[m][c] = M.eta(sm + L::F + (5 + c) * n3 + n2 * km, Vi[m][c]);
          }
        }
        // zeta along the thread's own column
#pragma unroll
        for (int alp = 0; alp < n; ++alp) {
          const int src = vnode(n, i, j, alp);
          real fz[5];
#pragma unroll
          for (int c = c0; c < 5; ++c) fz[c] = sm[L::F + (10 + c) * n3 + src];
#pragma unroll
          for (int m = 0; m < npt; ++m) {
            const real dh = plane_waves ? dk[m][alp] : sb.Dh[(k0 + m * kstep) * (n + 1) + alp];
#pragma unroll
            for (int c = c0; c < 5; ++c) Vi[m][c] += dh * fz[c];
          }
        }
      }
    } else if (contract) {
#pragma unroll
      for (int ci = 0; ci < 3; ++ci) {
#pragma unroll
        for (int alp = 0; alp < n; ++alp) {
          if (ci < 2) {
            const real dh = sb.Dh[(ci == 0 ? i : j) * (n + 1) + alp];
#pragma unroll
            for (int m = 0; m < npt; ++m) {
              const int km = k0 + m * kstep;
              const int src = ci == 0 ? vnode(n, alp, j, km) : vnode(n, i, alp, km);
#pragma unroll
              for (int c = c0; c < 5; ++c) Vi[m][c] += dh * sm[L::F + (5 * ci + c) * n3 + src];
            }
          } else {
            const int src = vnode(n, i, j, alp);
            real fz[5];
#pragma unroll
            for (int c = c0; c < 5; ++c) fz[c] = sm[L::F + (10 + c) * n3 + src];
#pragma unroll
            for (int m = 0; m < npt; ++m) {
              const real dh = plane_waves ? dk[m][alp] : sb.Dh[(k0 + m * kstep) * (n + 1) + alp];
#pragma unroll
              for (int c = c0; c < 5; ++c) Vi[m][c] += dh * fz[c];
            }
          }
        }
      }
    }
    if constexpr (SPLIT) {
      // the two-point sums carry 8 F_0, 16 F_1..3 and 32 F_4 against weights /16
#pragma unroll
      for (int m = 0; m < npt; ++m) {
        Vs[m][0] *= real(2);
        Vs[m][4] *= real(0.5);
      }
    }
#pragma unroll
    for (int m = 0; m < npt; ++m)
#pragma unroll
      for (int c = 0; c < 5; ++c)
        st<NT>(SPLIT ? Vs[m][c] + Vi[m][c] : Vi[m][c], v.Vol + c * Ev + vi + m * tpe);
  }
}

template <int N, typename real>
struct AffLds {
  using S = Sz<N>;
  static constexpr int n3 = S::n3, nf = S::nf;
  // lifting: u, v, w, T (4 rows of n3) and the BR1 face averages (4 x nf);
  // then g (12 padded rows), then the 15 rows of contravariant fluxes
  static constexpr int V = 0, Avg = 4 * n3, G = 0, F = 0, gsz = Pad<S::n>::size;
  static constexpr int m1 = 4 * n3 + 4 * nf, m2 = 12 * gsz, m3 = 15 * n3;
  static constexpr int rows = m1 > m2 ? (m1 > m3 ? m1 : m3) : (m2 > m3 ? m2 : m3);
  static constexpr bool plane_waves = S::n2 == 64 && S::epb == 1;
  static constexpr bool mfma = sizeof(real) == 8 && N == 7;
  static constexpr int minw = N == 1 ? 3 : S::minw;  // N = 1 spills 30 registers at 128
  static constexpr int fpu = VolLds<N, real, false, false>::fpu;  // face nodes per work unit
  static constexpr int units = nf / fpu, upt = (units + n3 - 1) / n3;
};

// ---------------------------------------------------------------------------
// Volume sweep of the viscous standard form without shock capturing on a mesh
// of parallelepipeds (View::affine): the same result as k_volume up to
// round-off.  The metrics are nine numbers per element, so they come out of
// the contractions: the lifting differentiates u, v, w, T along each
// direction (12 sums per source node instead of 36 products and 36 sums) and
// applies the metrics once per node, and the nine metric rows and the face
// normals take neither HBM traffic (98 of 262 bytes per node at N = 7) nor
// LDS.  16^3 at N = 7: 139 -> 104 us.  Bound by LDS: its index unit is active in
// 0.66 of the CU-busy cycles, 0.17 of them bank conflicts, with FP64 at 0.26 of its
// peak and 148 bytes per node measured (3.0 TB/s).
// The contravariant fluxes formed after the face phase instead of held
// through it (116 against 124 VGPRs) measured 2% slower; one face node per work
// unit 4% slower at N = 7 and 16% at N = 3, two 27% slower at N = 6 and 7% at
// N = 9.
// ---------------------------------------------------------------------------
template <int N, typename real, bool LGL, bool SUTH, bool NT>
__global__ void __launch_bounds__(Sz<N>::threads, (AffLds<N, real>::minw)) k_volume_affine(const View<real> *views,
                                                                                const int *blk_start, int nreq,
                                                                                View<real> single) {
  using S = Sz<N>;
  using L = AffLds<N, real>;
  constexpr int n = S::n, n2 = S::n2, n3 = S::n3, nf = S::nf, epb = S::epb;
  int lblk;
  const View<real> v = select_view(views, blk_start, nreq, single, lblk);
  __shared__ Smem<N, real> sb;
  __shared__ __align__(16) real sA[epb][L::rows];
  load_basis<N, real>(sb, v.basis, threadIdx.x);
  const int le = threadIdx.x / n3, a = threadIdx.x - le * n3;
  const int64_t e = (int64_t)lblk * epb + le;
  const bool active = le < epb && e < v.E;
  real *const sm = sA[le < epb ? le : 0];
  const int64_t Ev = v.E * n3, Ef = v.E * 6 * n2;
  const uint32_t vi = (uint32_t)(e * n3 + a), fb = (uint32_t)(e * 6 * n2);
  // the element's metrics: scalar loads where a workgroup holds one element
  const int64_t em = epb == 1 ? (int64_t)lblk : (active ? e : 0);
  const real gam = v.gamma, rR = v.rRgas, mu = v.mu, lam = v.lambda;
  const Bg<real> bg{v.bg_p, v.bg_H};
  const real *tr = v.cur ? v.Utr1 : v.Utr0;
  const int i = a % n, j = (a / n) % n, k = a / n2;
  constexpr bool plane_waves = L::plane_waves;
  real dk[n];  // row k of D-hat: wave-uniform when a wave is one k-plane
  if constexpr (plane_waves) {
    const int ku = __builtin_amdgcn_readfirstlane(k);
    const BasisOffsets o(n);
#pragma unroll
    for (int al = 0; al < n; ++al) dk[al] = v.basis[o.Dhat + ku * n + al];
  }
  real U[5], pf[L::upt][L::fpu][4];
  bool prim[L::upt][L::fpu];
  real tUo[L::fpu][5], tUn[L::fpu][5];
  // both sides' traces at the face nodes of work unit t = a + r n3
  auto fetch = [&](int r, int d, int s0, int pq) {
#pragma unroll
    for (int u = 0; u < L::fpu; ++u) {
      const int f = 2 * d + s0 + u;
      const int2 c = v.conn[e * 6 + f];
      prim[r][u] = (c.y >> 3) & 1;
      int pp, qq;
      orient_map(c.y & 7, pq % n, pq / n, N, pp, qq);
      const uint32_t io = fb + f * n2 + pq, in = (uint32_t)c.x * n2 + pp + n * qq;
#pragma unroll
      for (int s = 0; s < 5; ++s) {
        tUo[u][s] = (tr + s * Ef)[io];
        tUn[u][s] = (tr + s * Ef)[in];
      }
    }
  };
  if (active) {
#pragma unroll
    for (int c = 0; c < 5; ++c) U[c] = to_real(ld<NT>(v.U + c * Ev + vi), c, v);
    // the first unit's traces beside the state (a second one's, at N = 1,
    // where it is used: held from here they spilled)
    if (a < L::units) {
      int d, s0, pq;
      face_unit<n, L::fpu, plane_waves>(a, d, s0, pq);
      fetch(0, d, s0, pq);
    }
  }
  real Ja[9];
#pragma unroll
  for (int c = 0; c < 9; ++c) Ja[c] = (v.Ja + c * Ev)[em * n3];
  const real iJ = v.invJ[em * n3];
  real mun = mu;
  if (active) {
    real P[6];
    cons2prim(U, gam, rR, P, bg);
    sm[L::V + a] = P[1];
    sm[L::V + n3 + a] = P[2];
    sm[L::V + 2 * n3 + a] = P[3];
    sm[L::V + 3 * n3 + a] = P[5];
    if (SUTH) mun = sutherland(P[5], mu, v.rTref);
    // Lift_FillFlux: the BR1 average of both sides' traces
#pragma unroll
    for (int r = 0; r < L::upt; ++r) {
      const int t = a + r * n3;
      if (t < L::units) {
        int d, s0, pq;
        face_unit<n, L::fpu, plane_waves>(t, d, s0, pq);
        if (r > 0) fetch(r, d, s0, pq);
#pragma unroll
        for (int u = 0; u < L::fpu; ++u) {
          const int fn = (2 * d + s0 + u) * n2 + pq;
          real Po[6], Pn[6];
          cons2prim(tUo[u], gam, rR, Po, bg);
          cons2prim(tUn[u], gam, rR, Pn, bg);
          const real vo[4] = {Po[1], Po[2], Po[3], Po[5]}, vn[4] = {Pn[1], Pn[2], Pn[3], Pn[5]};
#pragma unroll
          for (int s = 0; s < 4; ++s) sm[L::Avg + s * nf + fn] = real(0.5) * (vo[s] + vn[s]);
#pragma unroll
          for (int dd = 0; dd < 3; ++dd) pf[r][u][dd] = Po[1 + dd];
          pf[r][u][3] = SUTH ? sutherland(Po[5], mu, v.rTref) : mu;
        }
      }
    }
  }
  __syncthreads();
  real g[12];
  if (active) {
    // Lift_VolInt and Lift_SurfInt of u, v, w, T along the three directions
    // (n shat of the faces of direction i is -+ Ja^i), then the metrics
    real w[3][4];
    if constexpr (L::mfma) {
      const PlaneMfma M(sb.Dh);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const real *plane = sm + L::V + s * n3 + n2 * k;
        w[0][s] = M.xi(plane, 0.0);
        w[1][s] = M.eta(plane, 0.0);
      }
    } else {
#pragma unroll
      for (int ci = 0; ci < 2; ++ci) {
#pragma unroll
        for (int s = 0; s < 4; ++s) w[ci][s] = real(0);
#pragma unroll
        for (int al = 0; al < n; ++al) {
          const int src = ci == 0 ? vnode(n, al, j, k) : vnode(n, i, al, k);
          const real dh = sb.Dh[(ci == 0 ? i : j) * (n + 1) + al];
#pragma unroll
          for (int s = 0; s < 4; ++s) w[ci][s] += dh * sm[L::V + s * n3 + src];
        }
      }
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) w[2][s] = real(0);
#pragma unroll
    for (int al = 0; al < n; ++al) {
      const real dh = plane_waves ? dk[al] : sb.Dh[k * (n + 1) + al];
#pragma unroll
      for (int s = 0; s < 4; ++s) w[2][s] += dh * sm[L::V + s * n3 + vnode(n, i, j, al)];
    }
    const int lf[3] = {i, j, k};
    const int pqf[3] = {j + n * k, i + n * k, i + n * j};
#pragma unroll
    for (int f = 0; f < 6; ++f) {
      const int d = f >> 1;
      // (on Gauss-Lobatto nodes l-hat vanishes off the end nodes: skipping
      // those terms put six branches here and 51 spilled registers at N = 5)
      const real lh = (f & 1) ? sb.lhp[lf[d]] : -sb.lhm[lf[d]];
#pragma unroll
      for (int s = 0; s < 4; ++s) w[d][s] += lh * sm[L::Avg + s * nf + f * n2 + pqf[d]];
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
#pragma unroll
      for (int d = 0; d < 3; ++d) g[d * 4 + s] = iJ * (Ja[d] * w[0][s] + Ja[3 + d] * w[1][s] + Ja[6 + d] * w[2][s]);
    }
  }
  real Fc[15];  // contravariant fluxes Ja^i . (F_adv - F_v)
  if (active) {
    real P[6];
    cons2prim(U, gam, rR, P, bg);
    const real lamn = SUTH ? mun * v.kappa : lam;
    real Fx[5], Fy[5], Fz[5], Vx[5], Vy[5], Vz[5];
    flux_adv<0>(U, P, Fx, bg);
    flux_adv<1>(U, P, Fy, bg);
    flux_adv<2>(U, P, Fz, bg);
    flux_visc<0>(P, g, mun, lamn, Vx);
    flux_visc<1>(P, g, mun, lamn, Vy);
    flux_visc<2>(P, g, mun, lamn, Vz);
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      Fx[c] -= Vx[c];
      Fy[c] -= Vy[c];
      Fz[c] -= Vz[c];
    }
#pragma unroll
    for (int ci = 0; ci < 3; ++ci)
#pragma unroll
      for (int c = 0; c < 5; ++c) Fc[5 * ci + c] = Ja[3 * ci] * Fx[c] + Ja[3 * ci + 1] * Fy[c] + Ja[3 * ci + 2] * Fz[c];
  }
  __syncthreads();  // the rows read above are covered by g
  if (active) {
    const int pa = Pad<n>::at(i, j, k);
#pragma unroll
    for (int c = 0; c < 12; ++c) sm[L::G + c * L::gsz + pa] = g[c];
  }
  __syncthreads();
  if (active) {
    // Lift_ProlongToFace of g, then this side's viscous normal flux
#pragma unroll
    for (int r = 0; r < L::upt; ++r) {
      const int t = a + r * n3;
      if (t < L::units) {
        int d, s0, pq;
        face_unit<n, L::fpu, plane_waves>(t, d, s0, pq);
        int base, stride;
        Pad<n>::face_line(2 * d, pq, base, stride);
        const BasisOffsets o(n);
        const real *lw[L::fpu];
#pragma unroll
        for (int u = 0; u < L::fpu; ++u) {
          const bool plus = (s0 + u) != 0;
          lw[u] = plane_waves ? v.basis + (plus ? o.lp : o.lm) : (plus ? sb.lp : sb.lm);
        }
        real gt[L::fpu][12];
        if constexpr (LGL) {
#pragma unroll
          for (int u = 0; u < L::fpu; ++u) {
            const real *row = sm + L::G + base + ((s0 + u) != 0 ? (n - 1) * stride : 0);
#pragma unroll
            for (int s = 0; s < 12; ++s) gt[u][s] = row[s * L::gsz];
          }
        } else {
#pragma unroll
          for (int u = 0; u < L::fpu; ++u)
#pragma unroll
            for (int s = 0; s < 12; ++s) gt[u][s] = real(0);
#pragma unroll
          for (int l = 0; l < n; ++l) {
            const real *row = sm + L::G + base + l * stride;
#pragma unroll
            for (int s = 0; s < 12; ++s) {
              const real gv = row[s * L::gsz];
#pragma unroll
              for (int u = 0; u < L::fpu; ++u) gt[u][s] += lw[u][l] * gv;
            }
          }
        }
        // n shat in the primary side's orientation: -+ Ja^d
        const real m0 = d == 0 ? Ja[0] : (d == 1 ? Ja[3] : Ja[6]);
        const real m1 = d == 0 ? Ja[1] : (d == 1 ? Ja[4] : Ja[7]);
        const real m2 = d == 0 ? Ja[2] : (d == 1 ? Ja[5] : Ja[8]);
#pragma unroll
        for (int u = 0; u < L::fpu; ++u) {
          const int fn = (2 * d + s0 + u) * n2 + pq;
          const real sg = ((s0 + u) != 0) == prim[r][u] ? real(1) : real(-1);
          const real nsv[3] = {m0 * sg, m1 * sg, m2 * sg};
          const real muf = pf[r][u][3];
          const real lamf = SUTH ? muf * v.kappa : lam;
          real H[5];
          flux_visc_face(pf[r][u], gt[u], muf, lamf, nsv, H);
#pragma unroll
          for (int s = 1; s < 5; ++s) st<NT>(H[s], v.Hv + (s - 1) * Ef + fb + fn);
        }
      }
    }
  }
  __syncthreads();  // g is read above; the flux rows cover it
  if (active) {
#pragma unroll
    for (int c = 0; c < 15; ++c) sm[L::F + c * n3 + a] = Fc[c];
  }
  __syncthreads();
  if (active) {
    // VolInt
    real Vi[5] = {0, 0, 0, 0, 0};
    if constexpr (L::mfma) {
      const PlaneMfma M(sb.Dh);
#pragma unroll
      for (int c = 0; c < 5; ++c) {
        Vi[c] = M.xi(sm + L::F + c * n3 + n2 * k, 0.0);
        Vi[c] = M.eta(sm + L::F + (5 + c) * n3 + n2 * k, Vi[c]);
      }
    } else {
#pragma unroll
      for (int ci = 0; ci < 2; ++ci)
#pragma unroll
        for (int al = 0; al < n; ++al) {
          const int src = ci == 0 ? vnode(n, al, j, k) : vnode(n, i, al, k);
          const real dh = sb.Dh[(ci == 0 ? i : j) * (n + 1) + al];
#pragma unroll
          for (int c = 0; c < 5; ++c) Vi[c] += dh * sm[L::F + (5 * ci + c) * n3 + src];
        }
    }
#pragma unroll
    for (int al = 0; al < n; ++al) {
      const real dh = plane_waves ? dk[al] : sb.Dh[k * (n + 1) + al];
#pragma unroll
      for (int c = 0; c < 5; ++c) Vi[c] += dh * sm[L::F + (10 + c) * n3 + vnode(n, i, j, al)];
    }
#pragma unroll
    for (int c = 0; c < 5; ++c) st<NT>(Vi[c], v.Vol + c * Ev + vi);
  }
}

// The surface sweep at N = 6 in FP64 where the working set streams from HBM: one
// face node per thread, its operands (the neighbour's trace, n shat, the sum of
// both sides' viscous fluxes) fetched beside the state and no loop.  That takes 96 VGPRs, so three of the
// six-wave workgroups share a CU instead of two: 20^3 on Gauss nodes 270 -> 209
// us (Roe), on Gauss-Lobatto nodes 184 -> 165 us (LLF); the general loop within
// 96 VGPRs spilled, 344 us.  Roe on Gauss-Lobatto nodes fits two workgroups
// with 108 VGPRs and spilled at 96 (63 -> 80 us on 14^3): it keeps the loop.  At
// the other degrees the bound gains no workgroup and the loop is the faster
// form (by 16% at N = 9).  Meshes that the caches hold fill the workgroups less
// and take the loop too: with Roe's solver on Gauss nodes the fetch cost 8% of a
// step at 6^3 (4 x 4 x 4) and 6% at 9^3.
template <int N, typename real, int SH, bool LGL, int RS, bool NT>
constexpr bool surf_early = NT && N == 6 && sizeof(real) == sizeof(double) && SH != 2 && !(LGL && RS == 1);

// ---------------------------------------------------------------------------
// Surface sweep of one workgroup of elements: FillFlux from this side's
// recomputed U trace, the neighbour's stored one and the mean of both sides'
// H; SurfInt gather, ApplyJac, the stage update (mode 0) or R (mode 1), and
// the next U traces.  SH = 1 (shock capturing, first pass) also forms the
// blending factors and hands a workgroup with a blended element to the blend
// pass; SH = 2 (the blend pass) adds the FV subcell operator, and with SPLIT
// takes the split form's advective volume integral for the blend.  ONE (the
// blend pass after the one-sweep Euler kernel): there is no stored volume
// integral, the advective one formed here is the whole of it.
// ---------------------------------------------------------------------------
template <int N, typename real, int SH, bool LGL, int RS, bool SPLIT = false, bool NT = false, bool ONE = false>
__device__ __forceinline__ void surface_body(const View<real> &v, const int lblk, const int mode, const int tid) {
  using S = Sz<N>;
  constexpr int n = S::n, n2 = S::n2, n3 = S::n3, nf = S::nf, epb = S::epb;
  constexpr bool SHOCK = SH != 0, FV = SH == 2;
  __shared__ Smem<N, real> sb;
  __shared__ real sB[epb][5][Pad<n>::size];
  __shared__ real sS[epb][5][nf];
  // the blend pass: 16 rows per element for the subcell operator and the
  // advective volume integral, the 1-D operators of the subcells
  __shared__ real sX[FV ? epb * 16 * n3 : 1];
  __shared__ real sFV[FV ? SubOps<n>::size : 1];
  __shared__ real sAl[epb];
  load_basis<N, real>(sb, v.basis, tid);
  // the first pass clears the count of the next sweep (which alternates
  // entries, so no pass reads a count that another pass clears)
  if (SH == 1 && lblk == 0 && tid == 0) v.bcnt[1 - v.bpar] = 0;
  if constexpr (FV) {
    using Q = SubOps<n>;
    const BasisOffsets o(n);
    for (int t = tid; t < n * n; t += blockDim.x) sFV[Q::D + t] = v.basis[o.D + t];
    for (int t = tid; t < n; t += blockDim.x) {
      const real w = v.basis[o.w + t], x = v.basis[o.x + t];
      sFV[Q::w + t] = w;
      sFV[Q::rw + t] = real(1) / w;
      // from the node to its two subcell interfaces, and 1/(distance to the next node)
      sFV[Q::lo + t] = x - v.basis[o.xhalf + t];
      sFV[Q::hi + t] = v.basis[o.xhalf + t + 1] - x;
      sFV[Q::rdx + t] = t + 1 < n ? real(1) / (v.basis[o.x + t + 1] - x) : real(0);
    }
  }
  const int le = tid / n3, a = tid - le * n3;
  const int64_t e = (int64_t)lblk * epb + le;
  const bool active = le < epb && e < v.E;
  const int64_t Ev = v.E * n3, Ef = v.E * 6 * n2;
  const uint32_t vi = (uint32_t)(e * n3 + a), fb = (uint32_t)(e * 6 * n2);
  const uint32_t gi = one_node(v) ? (uint32_t)(e * n3) : vi;  // where this node's metrics stand
  const real gam = v.gamma, rR = v.rRgas;
  const Bg<real> bg{v.bg_p, v.bg_H};
  const bool visc = v.viscous != 0;  // the same for the whole grid
  const real *tr = v.cur ? v.Utr1 : v.Utr0;
  const int i = a % n, j = (a / n) % n, k = a / n2;
  constexpr bool plane_waves = n2 == 64 && epb == 1;  // a wave is one face of one element
  real *const su = &sB[le < epb ? le : 0][0][0];
  const int pa = Pad<n>::at(i, j, k);
  // the state, in LDS for this element's own traces and for the update.  The
  // FP64 copy is exact, so it is read back after the face phase instead of
  // being held in registers through it (they would spill); the mixed form
  // keeps the FP64 values, and so does the blend pass, whose occupancy its
  // LDS sets.
  constexpr bool exact_lds = sizeof(real) == sizeof(double) && !FV;
  double Uold[5] = {0, 0, 0, 0, 0};
  constexpr bool early = surf_early<N, real, SH, LGL, RS, NT>;
  static_assert(!early || nf <= n3, "one face node per thread");
  real Ue[5], ne[3], He[4] = {0, 0, 0, 0};
  bool pe = false;
  if (active) {
#pragma unroll
    for (int c = 0; c < 5; ++c) Uold[c] = ld<NT>(v.U + c * Ev + vi);
    if constexpr (early) {
      if (a < nf) {
        const int f = a / n2, pq = a - f * n2;
        const int2 c = v.conn[e * 6 + f];
        pe = (c.y >> 3) & 1;
        int pp, qq;
        orient_map(c.y & 7, pq % n, pq / n, N, pp, qq);
        const uint32_t io = fb + a, in = (uint32_t)c.x * n2 + pp + n * qq;
#pragma unroll
        for (int s = 0; s < 5; ++s) Ue[s] = (tr + s * Ef)[in];
#pragma unroll
        for (int d = 0; d < 3; ++d) ne[d] = (v.NS + d * Ef)[one_node(v) ? fb + f * n2 : io];
        if (visc) {
#pragma unroll
          for (int s = 0; s < 4; ++s) He[s] = (v.Hv + s * Ef)[io] + (v.Hv + s * Ef)[in];
        }
      }
    }
#pragma unroll
    for (int c = 0; c < 5; ++c) su[c * Pad<n>::size + pa] = to_real(Uold[c], c, v);
  }
  if (SHOCK && le < epb && a == 0) {
    // blending factor: frozen, or the element's own indicator value, an
    // operator local to the element (Sec. 2.3); with alpha_smooth raised to
    // half of its face neighbours' values, then clipped again.  Zero past the
    // last element.
    real a0 = real(0);
    if (active) {
      if (v.alpha_in) {
        a0 = v.alpha_in[e];
      } else {
        a0 = v.alpha_raw[e];
        if (v.alpha_smooth) {
#pragma unroll
          for (int f = 0; f < 6; ++f) a0 = fmax(a0, real(0.5) * v.alpha_raw[v.conn[e * 6 + f].x / 6]);
          if (a0 < v.alpha_min) a0 = real(0);
          a0 = fmin(a0, v.alpha_max);
        }
      }
    }
    sAl[le] = a0;
  }
  __syncthreads();
  real al = real(0);
  bool any = false;  // some element of the workgroup is blended
  if constexpr (SHOCK) {
#pragma unroll
    for (int q = 0; q < epb; ++q) any = any || sAl[q] > real(0);
    if (active) {
      al = sAl[le];
      if (a == 0) v.alpha[e] = al;
    }
    if constexpr (SH == 1) {
      // a workgroup with a blended element is left to the blend pass
      if (any) {
        if (tid == 0) v.blist[atomicAdd(v.bcnt + v.bpar, 1)] = lblk;
        return;
      }
    }
  }
  if constexpr (early) {
    if (active && a < nf) {
      const int f = a / n2;
      int base, stride;
      Pad<n>::face_line(f, a - f * n2, base, stride);
      real Uo[5], Um[5], Us[5], Pm[6], Ps[6], nv[3], Fs[5];
      face_state<n, LGL>(su, (f & 1) ? sb.lp : sb.lm, base, stride, f & 1, Uo);
#pragma unroll
      for (int s = 0; s < 5; ++s) {
        Um[s] = pe ? Uo[s] : Ue[s];
        Us[s] = pe ? Ue[s] : Uo[s];
      }
      cons2prim(Um, gam, rR, Pm, bg);
      cons2prim(Us, gam, rR, Ps, bg);
      const real sh = sqrt(ne[0] * ne[0] + ne[1] * ne[1] + ne[2] * ne[2]);
      const real ish = pe ? real(1) / sh : real(-1) / sh;
#pragma unroll
      for (int d = 0; d < 3; ++d) nv[d] = ne[d] * ish;
      riemann<RS>(v.riemann, Um, Pm, Us, Ps, nv, gam, Fs, bg);
#pragma unroll
      for (int s = 0; s < 5; ++s) {
        // rounded twice as in the loop below: a request's bits do not depend on
        // whether its batch streams
#pragma clang fp contract(off)
        const real F = Fs[s] * sh - (s > 0 ? real(0.5) * He[s > 0 ? s - 1 : 0] : real(0));
        sS[le][s][a] = pe ? F : -F;
      }
    }
  } else if (active) {
    // FillFlux: Riemann flux of the U traces minus the mean of both sides' H.
    // This side's trace is recomputed from the state (the same bits as the
    // stored one); the neighbour's is read.
    for (int fn = a; fn < nf; fn += n3) {
      int f = fn / n2;
      if constexpr (plane_waves) f = __builtin_amdgcn_readfirstlane(f);
      const int pq = fn - f * n2, p = pq % n, q = pq / n;
      const int2 c = v.conn[e * 6 + f];
      const bool primary = (c.y >> 3) & 1;
      int pp, qq;
      orient_map(c.y & 7, p, q, N, pp, qq);
      const uint32_t io = fb + fn, in = (uint32_t)c.x * n2 + pp + n * qq;
      const uint32_t im = primary ? io : in, is = primary ? in : io;
      real Uo[5], Un[5];
      {
        int base, stride;
        Pad<n>::face_line(f, pq, base, stride);
        face_state<n, LGL>(su, (f & 1) ? sb.lp : sb.lm, base, stride, f & 1, Uo);
      }
#pragma unroll
      for (int s = 0; s < 5; ++s) Un[s] = (tr + s * Ef)[in];
      real Um[5], Us[5], Pm[6], Ps[6];
#pragma unroll
      for (int s = 0; s < 5; ++s) {
        Um[s] = primary ? Uo[s] : Un[s];
        Us[s] = primary ? Un[s] : Uo[s];
      }
      cons2prim(Um, gam, rR, Pm, bg);
      cons2prim(Us, gam, rR, Ps, bg);
      real nsv[3];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const real ns = (v.NS + d * Ef)[one_node(v) ? fb + f * n2 : io];
        nsv[d] = primary ? ns : -ns;
      }
      const real sh = sqrt(nsv[0] * nsv[0] + nsv[1] * nsv[1] + nsv[2] * nsv[2]);
      const real ish = kScaledVisc<real> ? real(1) / sh : real(0);
      const real nv[3] = {kScaledVisc<real> ? nsv[0] * ish : nsv[0] / sh, kScaledVisc<real> ? nsv[1] * ish : nsv[1] / sh,
                          kScaledVisc<real> ? nsv[2] * ish : nsv[2] / sh};
      real Fs[5];
      if (RS == 2 ? v.riemann == 1 : RS == 1) riemann_roe(Um, Pm, Us, Ps, nv, gam, Fs, bg);
      else riemann_llf(Um, Pm, Us, Ps, nv, gam, Fs, bg);
      if constexpr (kScaledVisc<real>) {
#pragma unroll
        for (int s = 0; s < 5; ++s) Fs[s] *= sh;
      }
      if (visc) {
#pragma unroll
        for (int s = 1; s < 5; ++s) Fs[s] -= real(0.5) * ((v.Hv + (s - 1) * Ef)[im] + (v.Hv + (s - 1) * Ef)[is]);
      }
#pragma unroll
      for (int s = 0; s < 5; ++s) {
        if constexpr (kScaledVisc<real>) sS[le][s][fn] = primary ? Fs[s] : -Fs[s];
        else sS[le][s][fn] = primary ? Fs[s] * sh : -(Fs[s] * sh);
      }
    }
  }
  __syncthreads();
  if constexpr (exact_lds) {
    if (active) {
#pragma unroll
      for (int c = 0; c < 5; ++c) Uold[c] = su[c * Pad<n>::size + pa];
    }
  }
  // blended elements: alpha (V_FV - V_adv) joins the stored volume integral,
  // i.e. (1 - alpha) V_adv + alpha V_FV + V_visc
  real Vb[5] = {0, 0, 0, 0, 0};
  if constexpr (FV) {
    if (any) {  // the same on every thread of the workgroup
      real *rows = sX + (le < epb ? le : 0) * 16 * n3;
      real U[5], P[6], Ja[9];
      if (active) {
#pragma unroll
        for (int c = 0; c < 5; ++c) U[c] = to_real(Uold[c], c, v);
        cons2prim(U, gam, rR, P, bg);
#pragma unroll
        for (int c = 0; c < 9; ++c) Ja[c] = (v.Ja + c * Ev)[gi];
      }
      real Vfv[5] = {0, 0, 0, 0, 0};
      fv_subcells<N, real>(rows, sFV, active, a, i, j, k, P, Ja, gam, rR, bg, Vfv);
      if constexpr (SPLIT) {
        // the split form's advective volume integral: two-point fluxes of
        // the primitives (rows 0-4, still those of the subcell pass), the
        // metric rows (5-13) and the specific total enthalpy (14)
        if (active) {
#pragma unroll
          for (int c = 0; c < 9; ++c) rows[(5 + c) * n3 + a] = Ja[c];
          rows[14 * n3 + a] = (U[4] + P[4]) / P[0];
        }
        __syncthreads();
      } else {
        // the advective DG volume integral, the three directions at once
        if (active) {
          real Fx[5], Fy[5], Fz[5];
          flux_adv<0>(U, P, Fx, bg);
          flux_adv<1>(U, P, Fy, bg);
          flux_adv<2>(U, P, Fz, bg);
#pragma unroll
          for (int ci = 0; ci < 3; ++ci)
#pragma unroll
            for (int c = 0; c < 5; ++c)
              rows[(5 * ci + c) * n3 + a] = Ja[3 * ci + 0] * Fx[c] + Ja[3 * ci + 1] * Fy[c] + Ja[3 * ci + 2] * Fz[c];
        }
        __syncthreads();
      }
      if (active && (ONE || al > real(0))) {
        real Va[5] = {0, 0, 0, 0, 0};
        const real Hn = SPLIT ? rows[14 * n3 + a] : real(0);
#pragma unroll
        for (int ci = 0; ci < 3; ++ci) {
          const int idx = ci == 0 ? i : (ci == 1 ? j : k);
#pragma unroll
          for (int alp = 0; alp < n; ++alp) {
            const int src = ci == 0 ? vnode(n, alp, j, k) : (ci == 1 ? vnode(n, i, alp, k) : vnode(n, i, j, alp));
            const real dh = sb.Dh[idx * (n + 1) + alp];
            if constexpr (SPLIT) {
              const real ds = sFV[SubOps<n>::D + idx * n + alp] + dh;  // D + D-hat
              real F[5];
              two_point_kep(P[0], P[1], P[2], P[3], P[4], Hn, rows[src], rows[n3 + src], rows[2 * n3 + src],
                            rows[3 * n3 + src], rows[4 * n3 + src], rows[14 * n3 + src],
                            real(0.5) * (Ja[3 * ci + 0] + rows[(5 + 3 * ci) * n3 + src]),
                            real(0.5) * (Ja[3 * ci + 1] + rows[(6 + 3 * ci) * n3 + src]),
                            real(0.5) * (Ja[3 * ci + 2] + rows[(7 + 3 * ci) * n3 + src]), F);
#pragma unroll
              for (int c = 0; c < 5; ++c) Va[c] += ds * F[c];
            } else {
#pragma unroll
              for (int c = 0; c < 5; ++c) Va[c] += dh * rows[(5 * ci + c) * n3 + src];
            }
          }
        }
#pragma unroll
        for (int c = 0; c < 5; ++c) Vb[c] = al > real(0) ? al * (Vfv[c] - Va[c]) : real(0);
        if constexpr (ONE) {
#pragma unroll
          for (int c = 0; c < 5; ++c) Vb[c] += Va[c];
        }
      }
    }
  }
  double Unew[5] = {0, 0, 0, 0, 0};
  if (active) {
    real V[5];
#pragma unroll
    for (int c = 0; c < 5; ++c) V[c] = ONE ? Vb[c] : ld<NT>(v.Vol + c * Ev + vi) + Vb[c];
    // 1/J and the RK register, loaded with the volume integral: their latency
    // overlaps the gather, and the register's five loads precede its five
    // stores (which the compiler could not move them across)
    const real iJ = v.invJ[gi];
    double dUo[5];
#pragma unroll
    for (int c = 0; c < 5; ++c) dUo[c] = (mode == 0 && v.rkA != 0.0) ? ld<NT>(v.dU + c * Ev + vi) : 0.0;
    // SurfInt gather (one writer per entry) and ApplyJac
    const int pqf[3] = {j + n * k, i + n * k, i + n * j};
    const int lf[3] = {i, j, k};
#pragma unroll
    for (int f = 0; f < 6; ++f) {
      const int d = f >> 1;
      // at Gauss-Lobatto nodes l-hat vanishes off the end node of the line
      const real lh = (f & 1) ? sb.lhp[lf[d]] : sb.lhm[lf[d]];
#pragma unroll
      for (int c = 0; c < 5; ++c) V[c] += sS[le][c][f * n2 + pqf[d]] * lh;
    }
    double R[5];
#pragma unroll
    for (int c = 0; c < 5; ++c) R[c] = (double)(-(V[c] * iJ));
    if (v.source == 1) {
      const double x = v.Xs[vi], y = (v.Xs + Ev)[vi], z = (v.Xs + 2 * Ev)[vi];
      const double cs = 0.1 * M_PI * cos(M_PI * (x + y + z - v.t));
      const double gg = (double)gam;
      R[0] += 2.0 * cs;
      R[1] += 3.0 * cs;
      R[2] += 3.0 * cs;
      R[3] += 3.0 * cs;
      R[4] += 2.0 * (3.0 * gg - 2.0) / (gg - 1.0) * cs;
    }
    if (mode == 1) {
#pragma unroll
      for (int c = 0; c < 5; ++c) (v.R + c * Ev)[vi] = R[c];
    } else {
#pragma unroll
      for (int c = 0; c < 5; ++c) {
        double *dUc = v.dU + c * Ev;
        // the first stage (A = 0) does not read the register: whatever it
        // holds (a restored state, an aborted step) cannot leak into the step
        const double du = (v.rkA != 0.0 ? v.rkA * dUo[c] : 0.0) + v.dt * R[c];
        st<NT>(du, dUc + vi);
        Unew[c] = Uold[c] + v.rkB * du;
        st<NT>(Unew[c], v.U + c * Ev + vi);
      }
    }
  }
  if (mode == 0) {
    // ProlongToFace of the updated state for the next stage
    // (every face-phase read of the old state is behind the barrier above)
    if (active) {
#pragma unroll
      for (int c = 0; c < 5; ++c) su[c * Pad<n>::size + pa] = to_real(Unew[c], c, v);
    }
    __syncthreads();
    if (active) {
      real *trn = v.cur ? v.Utr0 : v.Utr1;
      for (int fn = a; fn < nf; fn += n3) {
        int f = fn / n2;
        if constexpr (plane_waves) f = __builtin_amdgcn_readfirstlane(f);
        const int pq = fn - f * n2;
        int base, stride;
        Pad<n>::face_line(f, pq, base, stride);
        real t[5];
        face_state<n, LGL>(su, (f & 1) ? sb.lp : sb.lm, base, stride, f & 1, t);
#pragma unroll
        for (int c = 0; c < 5; ++c) st<NT>(t[c], trn + c * Ef + fb + fn);
      }
    }
  }
}


// Surface sweep: SH = 0 without shock capturing; SH = 1 with it, for the
// workgroups without a blended element (the others are listed for k_blend).
template <int N, typename real, int SH, bool LGL, bool NT, int RS>
__global__ void __launch_bounds__(Sz<N>::threads, (surf_early<N, real, SH, LGL, RS, NT> ? 5 : Sz<N>::minw)) k_surface(const View<real> *views, const int *blk_start,
                                                                          int nreq, View<real> single, int mode) {
  int lblk;
  const View<real> v = select_view(views, blk_start, nreq, single, lblk);
  surface_body<N, real, SH, LGL, RS, false, NT>(v, lblk, mode, threadIdx.x);
}

// Blend pass: the surface sweep with the FV subcell blend, for the workgroups
// that the sweep before it listed, request by request; a fixed grid strides
// over each list.  The view's 100 scalar registers live across the loop, so
// the compiler takes about 250 VGPRs: two 256-thread workgroups per CU, one
// of 512.  Its time is the latency of a workgroup (about 19 us at N = 5, 30 us
// at N = 7) times the rounds.  The thread index is opaque to the loop: hoisted
// address arithmetic took another 45 registers and with them the second
// workgroup.  An out-of-line body needs 134 VGPRs, but its call stack made
// every launch, empty ones included, 8 us slower; the view reloaded in each
// round needs 197 and was 10% slower.
template <int N, typename real, bool LGL, bool SPLIT, bool ONE = false>
__global__ void __launch_bounds__(Sz<N>::threads, Sz<N>::minw) k_blend(const View<real> *views, int nreq,
                                                                        View<real> single, int mode) {
  const int nr = nreq == 0 ? 1 : nreq;
  for (int r = 0; r < nr; ++r) {
    const View<real> v = nreq == 0 ? single : rebase(views[r], single.base);
    const int cnt = v.bcnt[v.bpar];
    for (int idx = blockIdx.x; idx < cnt; idx += gridDim.x) {
      int tid = threadIdx.x;
      asm volatile("" : "+v"(tid));
      surface_body<N, real, 2, LGL, 2, SPLIT, false, ONE>(v, v.blist[idx], mode, tid);
      __syncthreads();  // LDS is reused by the next listed workgroup
    }
  }
}

// workgroups of the blend pass: as many as the GPU holds at once
template <int N>
constexpr int kBlendBlocks = Sz<N>::threads <= 256 ? 512 : 256;

// the volume sweep with the viscosity law of the view (a template flag)
template <int N, typename real, bool SHOCK, bool LGL, bool SPLIT>
static void volume_sweep(dim3 grid, const View<real> *views, const int *blk_start, int nreq, const View<real> &v0,
                         hipStream_t st) {
  constexpr int threads = VolLds<N, real, SHOCK, SPLIT>::threads;
  if constexpr (!SHOCK && !SPLIT && sizeof(real) == sizeof(double)) {
    // a mesh of parallelepipeds, in FP64 (the mixed form keeps the order of its
    // roundings, see kScaledVisc; its general sweep reads one node's metrics)
    if (v0.affine && v0.viscous) {
      // streaming hints where the working set streams: 2 to 5% of a pass at N = 3 to
      // 9 (26^3 at N = 5: 4.87 -> 4.71 ms, the surface sweep's share as much as its
      // own); at N <= 2 they made the sweep 15 to 19% slower
      constexpr bool hints = N >= 3;
      const int at = Sz<N>::threads;
      if (hints && v0.nt) {
        if (v0.visc_law) k_volume_affine<N, real, LGL, true, hints><<<grid, at, 0, st>>>(views, blk_start, nreq, v0);
        else k_volume_affine<N, real, LGL, false, hints><<<grid, at, 0, st>>>(views, blk_start, nreq, v0);
      } else {
        if (v0.visc_law) k_volume_affine<N, real, LGL, true, false><<<grid, at, 0, st>>>(views, blk_start, nreq, v0);
        else k_volume_affine<N, real, LGL, false, false><<<grid, at, 0, st>>>(views, blk_start, nreq, v0);
      }
      return;
    }
  }
  if (v0.nt) {
    if (v0.visc_law)
      k_volume<N, real, SHOCK, LGL, SPLIT, true, false, true><<<grid, threads, 0, st>>>(views, blk_start, nreq, v0);
    else
      k_volume<N, real, SHOCK, LGL, SPLIT, false, false, true><<<grid, threads, 0, st>>>(views, blk_start, nreq, v0);
  } else {
    if (v0.visc_law)
      k_volume<N, real, SHOCK, LGL, SPLIT, true><<<grid, threads, 0, st>>>(views, blk_start, nreq, v0);
    else
      k_volume<N, real, SHOCK, LGL, SPLIT, false><<<grid, threads, 0, st>>>(views, blk_start, nreq, v0);
  }
}

// the sweeps that form face fluxes, with the Riemann solver of the view (a
// template flag: together the two took more registers than either, with
// spills, and the code of both; the mixed form fits its registers with both)
template <int N, typename real, int SH, bool LGL>
static void surface_sweep(dim3 grid, dim3 block, const View<real> *views, const int *blk_start, int nreq,
                          const View<real> &v0, int mode, hipStream_t st) {
  if constexpr (sizeof(real) == sizeof(float)) {
    if (v0.nt) k_surface<N, real, SH, LGL, true, 2><<<grid, block, 0, st>>>(views, blk_start, nreq, v0, mode);
    else k_surface<N, real, SH, LGL, false, 2><<<grid, block, 0, st>>>(views, blk_start, nreq, v0, mode);
  } else if (v0.riemann == 1) {
    if (v0.nt) k_surface<N, real, SH, LGL, true, 1><<<grid, block, 0, st>>>(views, blk_start, nreq, v0, mode);
    else k_surface<N, real, SH, LGL, false, 1><<<grid, block, 0, st>>>(views, blk_start, nreq, v0, mode);
  } else {
    if (v0.nt) k_surface<N, real, SH, LGL, true, 0><<<grid, block, 0, st>>>(views, blk_start, nreq, v0, mode);
    else k_surface<N, real, SH, LGL, false, 0><<<grid, block, 0, st>>>(views, blk_start, nreq, v0, mode);
  }
}

template <int N, typename real, bool SHOCK, bool LGL>
static void euler_sweep(dim3 grid, dim3 block, const View<real> *views, const int *blk_start, int nreq,
                        const View<real> &v0, int mode, hipStream_t st) {
  // on Lobatto nodes at N <= 2 the recomputed traces (an end node's state) pay from
  // one workgroup per CU on, small meshes lose by the state's way through LDS
  // (N = 2 mixed: 1.05 times the time at 78 workgroups, 0.96 at a thousand)
  // and at N = 4 both forms of streaming pay up to a few million nodes only (FP64
  // 0.97 of the time at 1.6 million, 1.03 at 8 million; mixed 0.95 at 3.6, 1.02 at 8)
  const bool large4 = !SHOCK && N == 4 && (int64_t)grid.x * Sz<N>::epb * Sz<N>::n3 >= 5000000;
  const bool nt = (v0.nt && !large4) || (!SHOCK && LGL && N <= 2 && grid.x >= 256);
  if constexpr (sizeof(real) == sizeof(float)) {
    if (nt) k_rhs<N, real, SHOCK, LGL, true, 2><<<grid, block, 0, st>>>(views, blk_start, nreq, v0, mode);
    else k_rhs<N, real, SHOCK, LGL, false, 2><<<grid, block, 0, st>>>(views, blk_start, nreq, v0, mode);
  } else if (v0.riemann == 1) {
    if (nt) k_rhs<N, real, SHOCK, LGL, true, 1><<<grid, block, 0, st>>>(views, blk_start, nreq, v0, mode);
    else k_rhs<N, real, SHOCK, LGL, false, 1><<<grid, block, 0, st>>>(views, blk_start, nreq, v0, mode);
  } else {
    if (nt) k_rhs<N, real, SHOCK, LGL, true, 0><<<grid, block, 0, st>>>(views, blk_start, nreq, v0, mode);
    else k_rhs<N, real, SHOCK, LGL, false, 0><<<grid, block, 0, st>>>(views, blk_start, nreq, v0, mode);
  }
}

template <int N, typename real, bool LGL>
static hipError_t launch_nl(Kernel k, int mode, const View<real> *views, const int *blk_start, int nreq, int blocks,
                           const View<real> &v0, hipStream_t st) {
  dim3 grid(blocks), block(Sz<N>::threads);
  switch (k) {
    case K_TRACE:
      k_trace<N, real, LGL><<<grid, block, 0, st>>>(views, blk_start, nreq, v0);
      break;
    case K_LIFT:
      // volume sweep: indicator (shock capturing), lifting (viscous), VolInt
      // (standard or split form)
      if (v0.split) {
        if constexpr (LGL) {  // the split form takes Gauss-Lobatto nodes only
          if (v0.shock) {
            if constexpr (N >= 2 && N <= 7) {  // the degrees shock capturing accepts
              volume_sweep<N, real, true, true, true>(grid, views, blk_start, nreq, v0, st);
            } else {
              return hipErrorInvalidValue;
            }
          } else {
            volume_sweep<N, real, false, true, true>(grid, views, blk_start, nreq, v0, st);
          }
        } else {
          return hipErrorInvalidValue;
        }
      } else if (v0.shock) {
        if constexpr (N >= 2 && N <= 7) {
          volume_sweep<N, real, true, LGL, false>(grid, views, blk_start, nreq, v0, st);
        } else {
          return hipErrorInvalidValue;
        }
      } else {
        volume_sweep<N, real, false, LGL, false>(grid, views, blk_start, nreq, v0, st);
      }
      break;
    case K_DIAG:
      // the lifting of the volume sweep and the dissipation sums
      if (v0.nt)
        k_volume<N, real, false, LGL, false, false, true, true>
            <<<grid, (VolLds<N, real, false, false>::threads), 0, st>>>(views, blk_start, nreq, v0);
      else
        k_volume<N, real, false, LGL, false, false, true, false>
            <<<grid, (VolLds<N, real, false, false>::threads), 0, st>>>(views, blk_start, nreq, v0);
      break;
    case K_RHS:
      // surface sweep (after a volume sweep), or the one-sweep Euler operator
      if (v0.shock) {
        if constexpr (N >= 2 && N <= 7) {  // the degrees shock capturing accepts
          const int bb = std::min(blocks, kBlendBlocks<N>);
          if (v0.one) {
            if constexpr (LGL) {
              euler_sweep<N, real, true, true>(grid, block, views, blk_start, nreq, v0, mode, st);
              k_blend<N, real, true, false, true><<<bb, block, 0, st>>>(views, nreq, v0, mode);
            } else {
              return hipErrorInvalidValue;
            }
          } else {
            surface_sweep<N, real, 1, LGL>(grid, block, views, blk_start, nreq, v0, mode, st);
            if (!v0.split) {
              k_blend<N, real, LGL, false><<<bb, block, 0, st>>>(views, nreq, v0, mode);
            } else if constexpr (LGL) {
              k_blend<N, real, LGL, true><<<bb, block, 0, st>>>(views, nreq, v0, mode);
            } else {
              return hipErrorInvalidValue;
            }
          }
        } else {
          return hipErrorInvalidValue;
        }
      } else if (v0.one) {
        euler_sweep<N, real, false, LGL>(grid, block, views, blk_start, nreq, v0, mode, st);
      } else {
        surface_sweep<N, real, 0, LGL>(grid, block, views, blk_start, nreq, v0, mode, st);
      }
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Gauss-Lobatto nodes take their own instantiations (face values are end nodes)
template <int N, typename real>
hipError_t launch_n(Kernel k, int mode, const View<real> *views, const int *blk_start, int nreq, int blocks,
                           const View<real> &v0, hipStream_t st) {
  return v0.lgl ? launch_nl<N, real, true>(k, mode, views, blk_start, nreq, blocks, v0, st)
                : launch_nl<N, real, false>(k, mode, views, blk_start, nreq, blocks, v0, st);
}

}  // namespace dg
