// One whole Runge-Kutta step of a 1D problem (linear advection, Burgers, Euler)
// per launch, and several steps of a small problem in one launch.
//
// A step of the cache-resident 1D problems is a chain of latencies, not of
// arithmetic: a launch per stage pays the dependent launch, the table and state
// loads and the stores three times over, and the limiter and the CFL maximum
// expand the new state at the random nodes again.  Here a workgroup owns EB
// consecutive elements, stages them with H neighbours on each side (H stages: an
// element's right-hand side reaches one element across each face) in LDS, and
// runs every stage there; each stage's valid window is one element shorter on
// either side, and the neighbours' part of it is computed by both workgroups (the
// same operations, so the same values).  The expansion of a stage's output at the
// nodes serves the limiter test, the next stage's fluxes and the CFL maximum.
//
// Within a stage (st), thread (slot, node):
//   A. expands its element at its node (Sec. 2.1), takes the fluxes and the
//      traces, and publishes the traces;
//   B. forms the interactive fluxes (Sec. 3.3; for a system each face once, by the
//      element on its right; a scalar flux is cheaper than a barrier, so there both
//      faces) and the nodal residual (Sec. 3.4) into LDS;
//   C. wave tasks (block of KB modes, 64 rows (variable, element, point)): Galerkin
//      projection and the stage combination, into the stage state in LDS.  The mode
//      block is uniform over a wave, so the weighted basis comes through scalar loads.
// After the last stage: detector and modal filter, limiter, CFL maximum.
//
// Every sum takes its terms in one fixed order, the order of k_stage1d, which takes
// the same step with one launch per stage: both give the same bits.
//
// Measured (FP64, per step, against one launch per stage): Burgers 1024 elements 24.1 -> 13.7 us,
// Sod 2048 elements 50 -> 33, Sod with HLL and Bogacki-Shampine, 1501 elements, 57 -> 34, one
// RK4 step of the 64-element wave problem 32.8 -> 15.8; 64-element advection, every step in one
// launch, 13.4 -> 6.9.  What is left is latency: a wave alone on its SIMD issues an FP64
// instruction every 8 cycles or so, which is why a thread holds one node (two nodes per thread
// halve the LDS reads but measured 14.5 on Burgers, and spill on Sod), and why a system's
// workgroup takes 512 threads (a fourteenth faster than 384) although its node phases fill fewer.
//
// The step does not run in place (a workgroup reads its neighbours' elements at its
// own time), except where one workgroup holds the whole mesh.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "device_common.hpp"
#include "internal.hpp"

namespace frsg {
namespace step1d {

typedef __attribute__((address_space(4))) double ConstD;  // read through the scalar cache where uniform
// A uniform pointer whose loads the compiler may not move above this point.  The operator
// tables are read again in every phase that uses them (a scalar-cache hit): hoisted out of
// the stage loop they filled every scalar register and spilled.
__device__ __forceinline__ const ConstD* pin(const double* p) {
  const ConstD* c = (const ConstD*)p;
  asm volatile("" : "+s"(c));
  return c;
}
// offsets in the block of point operators (DevTab::op1) of n points
template <int n>
struct Op {
  static constexpr int lL = 0, lR = n, dhL = 2 * n, dhR = 3 * n, mean = 4 * n, D = 5 * n, Vinv = D + n * n,
                       V = Vinv + n * n;
};
// Quotients by one positive number: its reciprocal, and for each numerator the product corrected by
// its remainder, which rounds like the division (three operations beside the shared reciprocal
// instead of a dozen).  So the Euler equations in FP64 round as in the stage kernel: where the
// limiter has set a pressure to its floor, the next stage's test on it is a tie that the last bit
// decides.  (The FP32-mixed loop keeps the divisions of the stage kernel.)  It holds for
// normal numbers.  A divisor of zero, or a numerator or quotient that overflows, gives NaN where
// the division gives an infinity: a density of zero fails the limiter's density test, a mean is refused
// and a wave speed counts as infinite either way; only a nodal momentum whose square overflows
// (above 1e154) passes the pressure test as NaN, which minus infinity would fail.
struct Quotient {
  double r, d;
  __device__ __forceinline__ explicit Quotient(double x) : r(recip(x)), d(x) {}
  __device__ __forceinline__ double operator()(double a) const {
    const double q = a * r;
    return fma(fma(-d, q, a), r, q);
  }
};
__device__ __forceinline__ double euler1_p(const double* U, const Quotient& by_rho, double g) {
  const double kin = by_rho(0.5 * U[1] * U[1]);
  return (g - 1.0) * (U[2] - kin);
}
__device__ __forceinline__ void euler1_f(const double* U, double v, double p, double* F) {
  F[0] = U[1];
  F[1] = U[1] * v + p;
  F[2] = (U[2] + p) * v;
}
template <int EQ, typename R>
__device__ __forceinline__ R pressure_of(const R* U, R g) {
  if constexpr (EQ == kEuler1 && sizeof(R) == sizeof(double)) return euler1_p(U, Quotient(U[0]), g);
  else return pressure<EQ>(U, g);
}
template <int EQ, typename R>
__device__ __forceinline__ void flux_of(const R* U, R* F, R adv, R g) {
  if constexpr (EQ == kEuler1 && sizeof(R) == sizeof(double)) {
    const Quotient by_rho(U[0]);
    euler1_f(U, by_rho(U[1]), euler1_p(U, by_rho, g), F);
  } else {
    flux<EQ, 0>(U, F, adv, g);
  }
}
template <int EQ>
__device__ __forceinline__ double speed_of(const double* U, double adv, double g) {
  if constexpr (EQ == kEuler1) {
    const Quotient by_rho(U[0]);
    const double c = sqrt(by_rho(g * euler1_p(U, by_rho, g)));
    return fabs(by_rho(U[1])) + c;
  } else {
    return speed<EQ, 0>(U, adv, g);
  }
}
template <int EQ, typename R>
__device__ __forceinline__ void interface_of(int kind, const R* L, const R* Rt, R* Fs, R adv, R g) {
  if constexpr (EQ == kEuler1 && sizeof(R) == sizeof(double)) {
    double fL[3], fR[3], vL, vR, cL, cR;
    auto side = [&](const double* U, double* f, double& v, double& c) {
      const Quotient by_rho(U[0]);
      v = by_rho(U[1]);
      const double p = euler1_p(U, by_rho, g);
      euler1_f(U, v, p, f);
      c = sqrt(by_rho(g * p));
    };
    side(L, fL, vL, cL);
    side(Rt, fR, vR, cR);
    if (kind == FRSG_FLUX_HLL) {
      const double SL = fmin(vL - cL, vR - cR), SR = fmax(vL + cL, vR + cR);
      const Quotient by_fan(SR - SL);
#pragma unroll
      for (int s = 0; s < 3; ++s)
        Fs[s] = (SL >= 0.0) ? fL[s]
              : (SR <= 0.0) ? fR[s]
                            : by_fan(SR * fL[s] - SL * fR[s] + (SL * SR) * (Rt[s] - L[s]));
    } else {
      const double lam = fmax(fabs(vL) + cL, fabs(vR) + cR);
#pragma unroll
      for (int s = 0; s < 3; ++s) Fs[s] = 0.5 * (fL[s] + fR[s]) - 0.5 * lam * (Rt[s] - L[s]);
    }
  } else {
    interface_flux<EQ, 0>(kind, L, Rt, Fs, adv, g);
  }
}

constexpr int KB = kProjBlock;  // modes per projection task
constexpr int kMaxStages = 4;

struct Args {
  const double* in;   // state at the start of the step
  double* out;        // state at its end (may equal in where one workgroup covers the mesh)
  double* w1;         // first and second stage state handed out (SSP-RK3), or null
  double* w2;
  const double* PWB;  // weighted basis by blocks of KB modes: [block][node][KB], zeros past the last mode
  int EB, H, W;       // owned elements, neighbours on each side, slots (W = EB + 2 H)
  int NqS;            // row length of the nodal arrays
  int nst;            // stages
  double a[kMaxStages][kMaxStages];  // Butcher form: row i forms the state after right-hand side i
  int limit;          // positivity limiter on every stage output
  unsigned char *f0, *f1, *f2, *f3;  // per element: limiter (stage 1, 2), filter, limiter; null or all set
  int dt_source;      // 1: dt_fixed; 2: from the maximum over lam_in[0 .. nlam)
  double dt_fixed;
  const double* lam_in;
  int nlam;
  double* lam_out;    // per workgroup: CFL maximum of its part of the result (or null)
  double* dt_used;    // or null
  // several steps in one launch
  int nsteps;
  unsigned char* flags;  // [nsteps][4][E] or null
  double* dts;           // [nsteps] or null
};

// sizes in doubles of the LDS regions (each rounded up to an even count, so that pairs of
// nodes stay 16-byte aligned)
struct Lds {
  int u, a, k, tr, r, phi, total;  // offsets
  int nk;                          // stored right-hand sides (tab)
};
__host__ __device__ inline int even(int x) { return (x + 1) & ~1; }
__host__ __device__ inline Lds lds_layout(int S, int M, int n, int W, int NqS, int nk) {
  Lds L;
  const int st = even(W * S * M * n);
  L.nk = nk;
  L.u = 0;
  L.a = st;
  L.k = 2 * st;
  L.tr = L.k + nk * st;
  L.r = L.tr + W * 2 * S * NqS;
  L.phi = L.r + W * S * n * NqS;
  L.total = L.phi + even(M * NqS);
  return L;
}
// rows of nodal values: even (16-byte pairs) and 2 mod 4, so that 16 lanes reading a pair
// each from consecutive rows touch different banks
__host__ __device__ inline int node_row(int Nq) {
  int r = (Nq + 1) & ~1;
  return (r & 3) == 2 ? r : r + 2;
}

// The step loop of one workgroup.  RES: the workgroup holds the whole mesh (slots =
// elements, wrapped on periodic meshes) and takes A.nsteps steps; otherwise one step of
// the window that starts at element e0 - H.
template <int EQ, int N, typename R, bool TAB, bool RES>
__device__ __forceinline__ void run(const KParams& P, const Args& A, double* smem) {
  // products fuse with the sum of the same expression only, as in the stage kernel
#pragma clang fp contract(on)
  constexpr int S = nstate<EQ>();
  constexpr int n = N;
  constexpr bool F64 = std::is_same<R, double>::value;
  using O = Op<n>;
  const int E = P.E, W = A.W, H = A.H;
  int M = P.M, Nq = P.Nq, NqS = A.NqS, ncoef = S * M * n;
  const long EN = (long)E * n;
  const int tid = threadIdx.x, BS = blockDim.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nwaves = BS >> 6;
  const bool periodic = P.bc[0] == FRSG_BC_PERIODIC;
  const int e0 = RES ? 0 : blockIdx.x * A.EB;
  const int base = e0 - H;                                   // element of slot 0 (before wrapping)
  const int nown = RES ? E : min(A.EB, E - e0);
  const Lds L = lds_layout(S, M, n, W, NqS, TAB ? A.nst - 1 : 0);
  double* sU = smem + L.u;      // [W][S][M][n] state at the start of the step
  double* sA = smem + L.a;      // [W][S][M][n] stage state
  double* sK = smem + L.k;      // [nk][W][S][M][n] right-hand sides (tab)
  double* sTr = smem + L.tr;    // [W][2][S][NqS] traces (a system's side 0: the left face's flux)
  double* sR = smem + L.r;      // [W][S][n][NqS] nodal residual; scratch between stages
  double* sPhi = smem + L.phi;  // [M][NqS] chaos basis, the padding repeating the last node
  const int kst = even(W * ncoef);
  __shared__ int sAny, sBad[256];  // limiter: some / this slot's bound failed
  __shared__ double sRed[16];
  constexpr int kRing = 256;
  __shared__ double sdt[RES ? kRing : 1];

  // state window and chaos basis: a thread's loads are all in flight before the first
  // one is waited for (a wave takes rows (variable, mode) of the window)
  double lam = 0.0;
  {
    constexpr int LD = 9;
    const int span = W * n;
    for (int c0 = 0; c0 < span; c0 += 64) {
      const int c = c0 + lane;
      const int sl = c / n, j = c - sl * n;
      int ge = base + sl;
      if (ge < 0 || ge >= E) {
        if (periodic) {
          ge %= E;
          if (ge < 0) ge += E;
        } else {
          ge = min(max(ge, 0), E - 1);  // outside the mesh: never used
        }
      }
      const double* src = A.in + (long)ge * n + j;
      double* dst = sU + sl * ncoef + j;
      for (int r0 = 0; r0 < S * M; r0 += LD * nwaves) {
        double v[LD];
#pragma unroll
        for (int i = 0; i < LD; ++i)
          if (c < span && r0 + wave + i * nwaves < S * M) v[i] = src[(long)(r0 + wave + i * nwaves) * EN];
        if (r0 == 0 && c0 == 0) {
          // the time step: the maximum over the workgroups of the previous launch
          if (RES || A.dt_source == 2)
            for (int i0 = 0; i0 < A.nlam; i0 += 256) {
              double x[4];
#pragma unroll
              for (int i = 0; i < 4; ++i) x[i] = A.lam_in[min(i0 + i * 64 + lane, A.nlam - 1)];
#pragma unroll
              for (int i = 0; i < 4; ++i) lam = fmax(lam, x[i]);
            }
          for (int i = tid; i < M * NqS; i += BS) {
            const int k = i / NqS, q = i - k * NqS;
            sPhi[i] = P.tab.Phi[k * Nq + min(q, Nq - 1)];
          }
        }
#pragma unroll
        for (int i = 0; i < LD; ++i)
          if (c < span && r0 + wave + i * nwaves < S * M) dst[(r0 + wave + i * nwaves) * n] = v[i];
      }
    }
  }
  if (tid == 0) sAny = 0;
  if (tid < 256) sBad[tid] = 0;
  if (RES || A.dt_source == 2)
    for (int o = 32; o > 0; o >>= 1) lam = fmax(lam, __shfl_xor(lam, o));
  __syncthreads();

  const int ls = tid / Nq, q = tid - ls * Nq;
  const bool slot = ls < W;
  const int g = base + ls;                                  // element of this thread's slot
  const bool exists = slot && (RES ? ls < E : (periodic || (g >= 0 && g < E)));
  const bool owned = exists && (RES || (ls >= H && ls < H + nown));
  const int eg = RES ? ls : g;                               // element index where owned
  const int left = (RES && ls == 0) ? E - 1 : ls - 1;
  const int right = (RES && periodic && ls == E - 1) ? 0 : ls + 1;
  const bool at_lo = !periodic && g == 0, at_hi = !periodic && g == E - 1;
  const R adv = (R)P.adv, gam = (R)P.gamma;

  // nodal values of a state at this thread's nodes: mode by mode into independent sums
  auto expand = [&](const double* X, auto& U) {
    using T = typename std::remove_reference<decltype(U[0][0])>::type;
    const double* C = X + ls * ncoef;
    const double* ph = sPhi + q;
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int j = 0; j < n; ++j) U[s][j] = T(0);
    // MC modes at a time, their reads in flight together; past the last mode the factor is 0
    // (x + 0 y is x for every finite y)
    constexpr int MC = S == 1 ? 5 : 1;
#pragma unroll 1
    for (int k = 0; k < M; k += MC) {
      double f[MC], c[MC][S][n];
#pragma unroll
      for (int i = 0; i < MC; ++i) {
        const int ki = min(k + i, M - 1);
        f[i] = ph[ki * NqS];
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
          for (int j = 0; j < n; ++j) c[i][s][j] = C[(s * M + ki) * n + j];
        if (k + i >= M) f[i] = 0.0;
      }
#pragma unroll
      for (int i = 0; i < MC; ++i)
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
          for (int j = 0; j < n; ++j) U[s][j] += (T)c[i][s][j] * (T)f[i];
    }
  };
  auto traces = [&](const auto& U, auto& tm, auto& tp) {
    using T = typename std::remove_reference<decltype(tm[0])>::type;
    const ConstD* op = pin(P.tab.op1);
#pragma unroll
    for (int s = 0; s < S; ++s) {
      T a = T(0), b = T(0);
#pragma unroll
      for (int j = 0; j < n; ++j) {
        a += (T)op[O::lL + j] * U[s][j];
        b += (T)op[O::lR + j] * U[s][j];
      }
      tm[s] = a;
      tp[s] = b;
    }
  };
  auto trow = [&](int sl, int side, int s) { return sTr + ((sl * 2 + side) * S + s) * NqS + q; };

  R U[S][N];            // nodal values of the stage input
  double Ud[S][N];      // FP32-mixed: the FP64 ones, for the limiter and the CFL maximum

  // ---- positivity limiter (Sec. 4.3) on the state in sA, whose nodal values are in V ----
  // test: does density or pressure fall below the threshold at one of this thread's nodes?
  auto mean_state = [&](double* ub, double& eps) {
    const double* C = sA + ls * ncoef;
    const ConstD* op = pin(P.tab.op1);
#pragma unroll
    for (int s = 0; s < S; ++s) {
      double acc = 0.0;
#pragma unroll
      for (int j = 0; j < n; ++j) acc += C[(s * M) * n + j] * op[O::mean + j];
      ub[s] = acc;
    }
    const double pb = pressure_of<EQ>(ub, P.gamma);
    bool finite = true;
#pragma unroll
    for (int s = 0; s < S; ++s) finite = finite && isfinite(ub[s]);
    eps = fmin(1e-8, fmin(ub[0], pb));
    return ub[0] > 0.0 && pb > 0.0 && finite;
  };
  // value pt at a node: the n solution points, then the two faces
  auto point = [&](const double (&V)[S][N], const double (&fm)[S], const double (&fp)[S], int pt, double* X) {
#pragma unroll
    for (int s = 0; s < S; ++s) X[s] = pt < n ? V[s][pt] : (pt == n ? fm[s] : fp[s]);
  };
  auto limit_test = [&](const double (&V)[S][N]) {
    if constexpr (S > 1) {
      double ub[S], eps;
      if (!mean_state(ub, eps)) {
        if (q == 0) atomicOr(P.status, kStatusNotRealizable);
        return;
      }
      double fm[S], fp[S];
      traces(V, fm, fp);
      double rmin = INFINITY, pmin = INFINITY;
#pragma unroll
      for (int pt = 0; pt < n + 2; ++pt) {
        double X[S];
        point(V, fm, fp, pt, X);
        rmin = fmin(rmin, X[0]);
        pmin = fmin(pmin, pressure_of<EQ>(X, P.gamma));
      }
      sR[ls * 2 * NqS + q] = rmin;
      if (fmin(rmin, pmin) < eps) {
        sBad[ls] = 1;
        sAny = 1;
      }
    }
  };
  // the elements that failed the test (every thread calls it, after a barrier): beta1 from the
  // nodes' density minima that the test left, pressure roots, beta2; then the coefficients in
  // sA, from which the pass expands the nodal values anew (taking them along through the affine map
  // saves 1.5 us per step of Sod, but rounds differently).  Near a shock some workgroup comes here
  // in most stages, and
  // the launch lasts as long as that one
  auto limit_fix = [&](double (&V)[S][N]) {
    if constexpr (S > 1) {
      const bool bad = exists && sBad[ls];
      double ub[S], eps = 0.0, beta1 = 1.0;
      double* mine = sR + (slot ? ls : 0) * 2 * NqS;  // [2][NqS] per slot
      auto row_min = [&](const double* r, double x) {  // the smallest of a row's Nq values
        int qq = 0;
#pragma unroll 1
        for (; qq + 8 <= Nq; qq += 8) {
          double2 a[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) a[i] = *reinterpret_cast<const double2*>(r + qq + 2 * i);
#pragma unroll
          for (int i = 0; i < 4; ++i) x = fmin(x, fmin(a[i].x, a[i].y));
        }
        for (; qq < Nq; ++qq) x = fmin(x, r[qq]);
        return x;
      };
      if (bad) {
        mean_state(ub, eps);
        double fm[S], fp[S];
        traces(V, fm, fp);
        const double rmin = row_min(mine, INFINITY);
        beta1 = (rmin >= eps) ? 1.0 : (ub[0] - eps) / (ub[0] - rmin);
        double bmin = 1.0;
#pragma unroll
        for (int pt = 0; pt < n + 2; ++pt) {
          double X[S];
          point(V, fm, fp, pt, X);
          X[0] = beta1 * (X[0] - ub[0]) + ub[0];
          if (pressure_of<EQ>(X, P.gamma) < eps) bmin = fmin(bmin, pressure_root<EQ>(ub, X, eps, P.gamma));
        }
        mine[NqS + q] = bmin;
      }
      __syncthreads();
      if (bad) {
        const double beta2 = row_min(mine + NqS, 1.0);
        double* C = sA + ls * ncoef;
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll 1
          for (int it = q; it < M * n; it += Nq) {
            const double m0 = (it < n) ? 1.0 : 0.0;
            double v = C[s * M * n + it];
            if (s == 0) v = beta1 * (v - ub[0] * m0) + ub[0] * m0;
            C[s * M * n + it] = beta2 * (v - ub[s] * m0) + ub[s] * m0;
          }
      }
    }
  };

  R F[S][N], tm[S], tp[S];
  auto fluxes_and_traces = [&]() {
    traces(U, tm, tp);
#pragma unroll
    for (int j = 0; j < n; ++j) {
      R Uj[S], Fj[S];
#pragma unroll
      for (int s = 0; s < S; ++s) Uj[s] = U[s][j];
      flux_of<EQ>(Uj, Fj, adv, gam);
#pragma unroll
      for (int s = 0; s < S; ++s) F[s][j] = Fj[s];
    }
#pragma unroll
    for (int s = 0; s < S; ++s) {
      if constexpr (S == 1) *trow(ls, 0, s) = (double)tm[s];
      *trow(ls, 1, s) = (double)tp[s];
    }
  };

  for (int step = 0; step < (RES ? A.nsteps : 1); ++step) {
    // dt = CFL dx / ((p+1) lambda_max)
    const double dt = (RES || A.dt_source == 2) ? P.cfl * P.dx / (P.np1 * lam) : A.dt_fixed;
    if (tid == 0 && blockIdx.x == 0) {
      if (!(dt > 0.0) || !isfinite(dt)) atomicOr(P.status, kStatusNonFinite);
      if (RES) {
        sdt[step % kRing] = dt;
      } else {
        *P.dt = dt;
        if (A.dt_used) *A.dt_used = dt;
      }
    }
    unsigned char *f0 = A.f0, *f1 = A.f1, *f2 = A.f2, *f3 = A.f3;
    if (RES && A.flags) {
      f0 = A.flags + step * 4l * E;
      f1 = f0 + E, f2 = f0 + 2l * E, f3 = f0 + 3l * E;
    }
    const double* X = sU;  // the stage input
    int limited = 0;       // Butcher form: the limiter acted on a stage state
    bool lim_last = false, tested = false;
    double rate = 0.0;
    // pass nst only expands the result, for the limiter and the CFL maximum
    const int passes = (A.nst + ((S > 1 && A.limit) || A.lam_out || RES ? 1 : 0));
#pragma unroll 1
    for (int st = 0; st < passes;) {
      // sizes the compiler may not see through: the addresses that follow from them are formed
      // where they are used; hoisted out of this loop they took more registers than there are
      asm volatile("" : "+s"(M), "+s"(Nq), "+s"(NqS), "+s"(ncoef));
      const bool last = st == A.nst - 1, done = st == A.nst;
      const int lo = RES ? 0 : st + 1, hi = RES ? E : W - st - 1;  // slots with a valid output
      const bool in_slot = done ? owned : exists && (RES || (ls >= st && ls < W - st));
      const bool out_slot = exists && ls >= lo && ls < hi;
      const bool test = S > 1 && A.limit && st > 0 && !tested;
      if (in_slot && !(tested && !sBad[ls])) {
        if constexpr (F64) {
          expand(X, U);
          if (test) limit_test(U);
        } else {
          if (test || done) expand(X, Ud);
          if (test) limit_test(Ud);
          if (!done) expand(X, U);
        }
        if (!done) fluxes_and_traces();
      }
      __syncthreads();
      if (S > 1 && !tested && sAny) {
        // the limiter acts on the previous stage's output (uniform over the workgroup); the
        // pass starts over for the elements it changed
        if constexpr (F64) limit_fix(U);
        else limit_fix(Ud);
        if (owned && q == 0 && sBad[ls]) {
          if (done) {
            lim_last = true;
          } else {
            limited = 1;
            if (!TAB && f0) (st == 1 ? f0 : f1)[eg] = 1;
          }
        }
        tested = true;
        __syncthreads();
        continue;
      }
      tested = false;
      if (done) break;

      // B. interactive fluxes and nodal residual
      R FL[S], FR[S];
      if constexpr (S == 1) {
        if (out_slot) {
          R UL[1] = {(R)*trow(left, 1, 0)}, UR[1] = {(R)*trow(right, 0, 0)};
          if (at_lo) ghost<EQ>(P, 0, tm, UL);
          interface_of<EQ>(P.flux, UL, tm, FL, adv, gam);
          if (at_hi) ghost<EQ>(P, 1, tp, UR);
          interface_of<EQ>(P.flux, tp, UR, FR, adv, gam);
        }
      } else {
        // left faces of the output slots and of the slot after them (past the mesh: the
        // boundary face of the last element)
        const bool past = !periodic && g == E;
        const bool face = slot && ls >= lo && ls <= hi && (exists || past);
        if (face) {
          R Lt[S], Rt[S];
          if (!at_lo) {
#pragma unroll
            for (int s = 0; s < S; ++s) Lt[s] = (R)*trow(left, 1, s);
          }
          if (past) {
            ghost<EQ>(P, 1, Lt, Rt);
          } else {
#pragma unroll
            for (int s = 0; s < S; ++s) Rt[s] = tm[s];
            if (at_lo) ghost<EQ>(P, 0, Rt, Lt);
          }
          interface_of<EQ>(P.flux, Lt, Rt, FL, adv, gam);
#pragma unroll
          for (int s = 0; s < S; ++s) *trow(ls, 0, s) = (double)FL[s];
        }
        __syncthreads();
        if (out_slot) {
#pragma unroll
          for (int s = 0; s < S; ++s) FR[s] = (R)*trow(right, 0, s);
        }
      }
      if (out_slot) {
        const R iJ = (R)(1.0 / P.Jx);
        double* Ro = sR + (ls - lo) * S * n * NqS + q;
        const ConstD* op = pin(P.tab.op1);
#pragma unroll
        for (int s = 0; s < S; ++s) {
          R fdl = R(0), fdr = R(0);
#pragma unroll
          for (int l = 0; l < n; ++l) {
            fdl += (R)op[O::lL + l] * F[s][l];
            fdr += (R)op[O::lR + l] * F[s][l];
          }
#pragma unroll
          for (int j = 0; j < n; ++j) {
            R acc = R(0);
#pragma unroll
            for (int l = 0; l < n; ++l) acc += (R)op[O::D + j * n + l] * F[s][l];
            acc = acc + (FL[s] - fdl) * (R)op[O::dhL + j] + (FR[s] - fdr) * (R)op[O::dhR + j];
            Ro[(s * n + j) * NqS] = (double)(-acc * iJ);
          }
        }
      }
      __syncthreads();

      // C. projection and stage combination
      if (tid == 0) sAny = 0;
      if (tid < 256) sBad[tid] = 0;
      {
        const int ospan = (hi - lo) * n, rows = S * ospan;
        const int nkb = (M + KB - 1) / KB, nrb = (rows + 63) >> 6;
        const double cu = st == 0 ? 0.0 : st == 1 ? 0.75 : 1.0 / 3.0;
        const double cw = st == 0 ? 1.0 : st == 1 ? 0.25 : 2.0 / 3.0;
        for (int t = wave; t < nkb * nrb; t += nwaves) {
          const int rb = t / nkb, kb = t - rb * nkb, k0 = kb * KB;
          const int row = min(rb * 64 + lane, rows - 1);  // (the last rows' lanes past the end repeat one)
          const bool mine = rb * 64 + lane < rows;
          const int s = S == 1 ? 0 : (row >= ospan) + (row >= 2 * ospan), rem = row - s * ospan;
          const int eo = rem / n, j = rem - eo * n;
          const double* Rq = sR + ((eo * S + s) * n + j) * NqS;
          const ConstD* pw = (const ConstD*)(A.PWB) + kb * Nq * KB;
          const int idx0 = (lo + eo) * ncoef + (s * M + k0) * n + j;
          int idx[KB];
          double uv[KB], wv[KB];  // the combination's inputs, read before the sums
#pragma unroll
          for (int i = 0; i < KB; ++i) {
            idx[i] = idx0 + min(i, M - 1 - k0) * n;
            uv[i] = sU[idx[i]];
            if constexpr (!TAB) wv[i] = X[idx[i]];
          }
          double ad[KB];
          R ar[KB];
#pragma unroll
          for (int i = 0; i < KB; ++i) {
            ad[i] = 0.0;
            ar[i] = R(0);
          }
          auto add = [&](double r, const ConstD* w) {
#pragma unroll
            for (int i = 0; i < KB; ++i) {
              if constexpr (F64) {
                ad[i] += w[i] * r;
              } else {  // the mean mode in FP64
                if (i == 0) ad[0] += w[0] * r;
                ar[i] += (R)w[i] * (R)r;
              }
            }
          };
          int qq = 0;
#pragma unroll 1
          for (; qq + 8 <= Nq; qq += 8) {
            double2 r[4];
#pragma unroll
            for (int h = 0; h < 4; ++h) r[h] = *reinterpret_cast<const double2*>(Rq + qq + 2 * h);
#pragma unroll
            for (int h = 0; h < 4; ++h) {
              add(r[h].x, pw + (qq + 2 * h) * KB);
              add(r[h].y, pw + (qq + 2 * h + 1) * KB);
            }
          }
#pragma unroll 1
          for (; qq < Nq; ++qq) add(Rq[qq], pw + qq * KB);
#pragma unroll
          for (int i = 0; i < KB; ++i) {
            if (k0 + i >= M) break;
            const double acc = (F64 || (i == 0 && k0 == 0)) ? ad[i] : (double)ar[i];
            double v;
            if constexpr (TAB) {
              double tsum = 0.0;
#pragma unroll
              for (int m = 0; m < kMaxStages - 1; ++m)
                if (m < st && A.a[st][m] != 0.0) tsum = tsum + A.a[st][m] * sK[m * kst + idx[i]];
              if (A.a[st][st] != 0.0) tsum = tsum + A.a[st][st] * acc;
              v = uv[i] + dt * tsum;
              if (mine && !last) sK[st * kst + idx[i]] = acc;
            } else {
              v = cu * uv[i] + cw * (wv[i] + dt * acc);
            }
            if (mine) {
              sA[idx[i]] = v;
              if constexpr (!RES && !TAB && S == 1) {
                const int eo1 = lo + eo - H;
                if (!last && A.w1 && eo1 >= 0 && eo1 < nown)  // stage states handed out
                  (st == 0 ? A.w1 : A.w2)[(long)(k0 + i) * EN + (long)(e0 + eo1) * n + j] = v;
              }
            }
          }
        }
      }
      X = sA;
      if (f0 && owned && q == 0 && !last && !TAB) (st == 0 ? f0 : f1)[eg] = 0;
      __syncthreads();
      if (last) {
        // detector and modal filter (Sec. 4.2, 4.1): thread q owns the chaos mode k = q
        if (P.filter != FRSG_FILTER_NONE) {
          const int k = q;
          const bool has = owned && k < M;
          double ut[S][N];
          double* C = sA + (slot ? ls : 0) * ncoef + k * n;  // + s M n
          double* en = sTr + (slot ? ls : 0) * 2 * S * NqS;  // [M][2] energies of the slot's modes
          double* la = sR + (slot ? ls : 0) * 2 * S;         // Lasso: |u~| of the two highest pure modes
          const ConstD* op = pin(P.tab.op1);
          if (has) {
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
              for (int m = 0; m < n; ++m) {
                double acc = 0.0;
#pragma unroll
                for (int j = 0; j < n; ++j) acc += op[O::Vinv + m * n + j] * C[s * M * n + j];
                ut[s][m] = acc;
              }
            double num = 0.0, den = 0.0;
#pragma unroll
            for (int m = 0; m < n; ++m) {
              const double e2 = ut[0][m] * ut[0][m];
              num += e2 * P.tab.shell[k * n + m];
              den += e2;
            }
            en[2 * k] = num;
            en[2 * k + 1] = den;
            if (P.filter == FRSG_FILTER_LASSO) {
              if (k == 0)
#pragma unroll
                for (int s = 0; s < S; ++s) la[s] = fabs(ut[s][n - 1]);
              if (k == M - 1)
#pragma unroll
                for (int s = 0; s < S; ++s) la[S + s] = fabs(ut[s][0]);
            }
          }
          __syncthreads();
          if (owned) {
            double tn = 0.0, td = 0.0;
#pragma unroll 4
            for (int i = 0; i < M; ++i) {
              tn += en[2 * i];
              td += en[2 * i + 1];
            }
            const bool flag = (P.sensor == FRSG_SENSOR_ALWAYS) || (td > 0.0 && tn / td > P.sensor_thr);
            if (flag && has) {
              if (P.filter == FRSG_FILTER_LASSO) {
                // Eq. LassoFilterFunction: soft threshold of every (spatial, chaos)
                // coefficient; filt holds ||Psi_m Phi_k||_1
#pragma unroll
                for (int s = 0; s < S; ++s) {
                  const double a1 = la[s] / ((double)(n * (n - 1)) * P.tab.filt[n - 1]);
                  const double a2 = (M > 1) ? la[S + s] / ((double)((M - 1) * M) * P.tab.filt[(M - 1) * n]) : 0.0;
#pragma unroll
                  for (int m = 0; m < n; ++m) {
                    const double pen = (a1 * (double)(m * (m + 1)) + a2 * (double)(k * (k + 1))) * P.tab.filt[k * n + m];
                    const double au = fabs(ut[s][m]);
                    const double f = (au > 0.0) ? 1.0 - pen / au : 0.0;
                    ut[s][m] = (f > 0.0 ? f : 0.0) * ut[s][m];
                  }
#pragma unroll
                  for (int j = 0; j < n; ++j) {
                    double acc = 0.0;
#pragma unroll
                    for (int m = 0; m < n; ++m) acc += op[O::V + j * n + m] * ut[s][m];
                    C[s * M * n + j] = acc;
                  }
                }
              } else {
                double lamk[N];
#pragma unroll
                for (int m = 0; m < n; ++m) {
                  const double f = P.tab.filt[k * n + m];
                  lamk[m] = (P.filter == FRSG_FILTER_EXP) ? exp(-P.alpha * dt * f) : f;
                }
#pragma unroll
                for (int s = 0; s < S; ++s)
#pragma unroll
                  for (int j = 0; j < n; ++j) {
                    double acc = 0.0;
#pragma unroll
                    for (int m = 0; m < n; ++m) acc += op[O::V + j * n + m] * (ut[s][m] * lamk[m]);
                    C[s * M * n + j] = acc;
                  }
              }
            }
            if (q == 0 && f2) f2[eg] = flag ? 1 : 0;
          }
          __syncthreads();
        } else if (owned && q == 0 && f2) {
          f2[eg] = 0;
        }
      }
      ++st;
    }

    // CFL maximum of the result
    if ((A.lam_out || RES) && owned) {
      auto wave_speed = [&](const double (&V)[S][N]) {
#pragma unroll
        for (int j = 0; j < n; ++j) {
          double Uj[S];
#pragma unroll
          for (int s = 0; s < S; ++s) Uj[s] = V[s][j];
          double r = speed_of<EQ>(Uj, P.adv, P.gamma);
          if (!(r == r)) r = __longlong_as_double(0x7ff0000000000000ll);  // NaN -> +inf, dt -> 0
          rate = fmax(rate, r);
        }
      };
      if constexpr (F64) wave_speed(U);
      else wave_speed(Ud);
    }
    if (owned && q == 0 && f0) {
      if (TAB) {
        f0[eg] = limited ? 1 : 0;
        f1[eg] = 0;
      }
      f3[eg] = lim_last ? 1 : 0;
    }
    if (A.lam_out || RES) {
      for (int o = 32; o > 0; o >>= 1) rate = fmax(rate, __shfl_xor(rate, o));
      if (lane == 0) sRed[tid >> 6] = rate;
      __syncthreads();
      double r = sRed[0];
      for (int w = 1; w < nwaves; ++w) r = fmax(r, sRed[w]);
      if (RES) lam = r;
      else if (tid == 0) A.lam_out[blockIdx.x] = r;
    }

    if constexpr (RES) {
      // the result is the next step's start: trade the two buffers (U holds its nodal values)
      double* t = sU;
      sU = sA;
      sA = t;
      if (step % kRing == kRing - 1 || step == A.nsteps - 1) {
        __syncthreads();
        const int first = step - step % kRing;
        if (A.dts)
          for (int i = tid; i <= step - first; i += BS) A.dts[first + i] = sdt[i];
        __syncthreads();
        if (step == A.nsteps - 1 && tid == 0) *P.dt = dt;
      }
    }
  }

  // the owned elements of the result
  {
    const double* Z = RES ? sU : sA;
    const int span = nown * n;
    for (int c0 = 0; c0 < span; c0 += 64) {
      const int c = c0 + lane;
      if (c >= span) continue;
      const int l = c / n, j = c - l * n;
      const double* src = Z + (l + H) * ncoef + j;
      double* dst = A.out + (long)(e0 + l) * n + j;
#pragma unroll 4
      for (int sk = wave; sk < S * M; sk += nwaves) dst[(long)sk * EN] = src[sk * n];
    }
  }
  if (RES && tid == 0 && A.lam_out) A.lam_out[0] = lam;
}

}  // namespace step1d
}  // namespace frsg
