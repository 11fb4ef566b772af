// Fused FR-SG stage kernel in FP64 for the 2D Euler equations on quadrilaterals with p = 3 or
// p = 2 (N x N Legendre-Gauss solution points, N = 4 or 3), any gPC size M and random node
// count NQ fixed at compile time, on any mesh: the whole right-hand side of a stage (Sec. 2.1,
// Sec. 3.2-3.5) and its epilogue (stage combination, detector, filter, limiter, CFL maximum,
// Sec. 4), as k_stage2d (kernels_euler2d.hip) does it with two variables per lane.
//
// A wave owns one element, a workgroup a 2 x 2 tile of them.  Lane (h, j): row h of 16 lanes,
// solution point j.  For the chaos expansion and the projection h is the conserved variable, and
// the lane keeps that variable's M coefficients and its residual in registers; random nodes go
// in groups of four, and a 4 x 4 transposition over the rows gives row h all four variables at
// node q0 + h, where fluxes, traces, interface fluxes and the nodal residual are formed once
// per point and node; the residuals are transposed back and projected.
//
// One variable per lane needs half of k_stage2d's registers, so four waves fit a SIMD (128
// registers, 40 KB of LDS per workgroup), in workgroups that are at different places of the
// stage: while one waits for its coefficients or its halo traces, others are in the node loop.
// To stay within 128 registers the lane's point weights are read from LDS in every group, the
// flux divergence is summed before the interface flux, and the weights' and the lane's place are
// computed anew where they are used.
//
// Measured with 15 modes and 25 nodes, p = 3: 90 us per Butcher-row stage at 100 x 50 elements
// (k_stage2d 136), 92 per SSP stage at 112 x 56 (99).  At 192 x 96 the vector units issue two
// thirds of the time, at about 2.1 GHz, and the states pass at 2.3 of the 5.4 TB/s of a large copy;
// the rest is waits at the ends of a workgroup.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device_common.hpp"
#include "internal.hpp"
#include "quad_device.hpp"
#include "stage2d.hpp"

namespace frsg {
namespace {

constexpr int WX = kWaveTile, WY = kWaveTile, WE = WX * WY;  // elements per workgroup
constexpr int WHF = 2 * (WX + WY);           // element faces on the tile boundary
constexpr int WBLK = 64 * WE;                // threads per workgroup
using Table = const __attribute__((address_space(4))) double*;

// value of lane 16 r of the wave in every lane (uniform)
__device__ __forceinline__ double row_value(double v, int r) {
  const long long x = __double_as_longlong(v);
  const unsigned lo = __builtin_amdgcn_readlane((int)x, 16 * r), hi = __builtin_amdgcn_readlane((int)(x >> 32), 16 * r);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// minimum over the wave, in every lane
__device__ __forceinline__ double wave_min(double v) {
  v = ymin4(xmin4(v));
  return fmin(fmin(row_value(v, 0), row_value(v, 1)), fmin(row_value(v, 2), row_value(v, 3)));
}

// Weights of the lanes in LDS (k_stage2w): rows of LS doubles, an odd number of 16-byte units so
// that the 16 rows start in different banks
constexpr int LS = 18;
// rotated l(-1), l(+1) for x (row a) and y (column b)
struct FaceOps {
  double lx[4], rx[4], ly[4], ry[4];
};
__device__ __forceinline__ void make_face_ops(const double* lane, int a, int b, FaceOps& L) {
  const double *lo = lane + 12, *hi = lane + NP * LS + 12;  // the weights of an x-lo and an x-hi flux point
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    L.lx[k] = lo[(a + k) & 3];
    L.rx[k] = hi[(a + k) & 3];
    L.ly[k] = lo[(b - k) & 3];
    L.ry[k] = hi[(b - k) & 3];
  }
}

// variable h of the lane's point at nodes q .. q + 3 (the last node repeated past the end)
template <int M, int NQ>
__device__ __forceinline__ void expand4(const double (&o)[M], Table phi, int q, double (&v)[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const Table row = phi + min(q + i, NQ - 1) * M;
    double t = 0.0;
#pragma unroll
    for (int k = 0; k < M; ++k) t += o[k] * row[k];
    v[i] = t;
  }
}

// Positivity limiter on the wave's element (Sec. 4.3); o: the lane's coefficients.  The decision
// is first taken from rigorous modal bounds at every solution and face point (|Phi_k(z_q)| <=
// cmax_k); only an element whose bound comes within a margin of the threshold is evaluated node
// by node, so both routes give the node-by-node decision.
template <int M, int NQ, int N>
__device__ __forceinline__ int limit_wave(const KParams& P, Table phi, double (&o)[M], int a, int b, Table cmax, const double* lane,
                          bool point) {
  const int h = (threadIdx.x >> 4) & 3;
  const double g = P.gamma;
  // element x random mean: sum_j (w_a/2)(w_b/2) o(j, mode 0)
  double ub[4];
  {
    const double mean = ysum4(xsum4(o[0] * lane[(a + NP * b) * LS + 16]));
#pragma unroll
    for (int s = 0; s < 4; ++s) ub[s] = row_value(mean, s);
  }
  const double pb = euler_p(ub, g);
  const bool realizable = ub[0] > 0.0 && pb > 0.0 && isfinite(ub[0]) && isfinite(ub[1]) && isfinite(ub[2]) &&
                          isfinite(ub[3]);
  if (!realizable) {
    if ((threadIdx.x & 63) == 0) atomicOr(P.status, kStatusNotRealizable);
    return 0;
  }
  const double eps = fmin(1e-8, fmin(ub[0], pb));

  // rigorous bounds: value(z) = mean + sum_{k>=1} c_k Phi_k(z)
  auto safe = [&](const double* mn, const double* vr) {
    const double rlo = mn[0] - vr[0];
    const double elo = mn[3] - vr[3];
    const double mx = fabs(mn[1]) + vr[1];
    const double my = fabs(mn[2]) + vr[2];
    const double tol_r = 1e-10 * (fabs(mn[0]) + vr[0]);
    if (!(rlo > eps + tol_r)) return false;
    const double kin = 0.5 * (mx * mx + my * my) / rlo;
    const double plo = (g - 1.0) * (elo - kin);
    const double tol_p = 1e-10 * (g - 1.0) * (fabs(mn[3]) + vr[3] + kin);
    return plo > eps + tol_p;
  };
  bool ok;
  {
    double var = 0.0;
#pragma unroll
    for (int k = 1; k < M; ++k) var += fabs(o[k]) * cmax[k];
    // the four face points of the lane's line and column: row h tests the h-th
    double fl[4], fv[4], mn[4] = {o[0], o[0], o[0], o[0]}, vr[4] = {var, var, var, var};
    double w[4];
    auto weights = [&](bool x, bool hi) {
#pragma unroll
      for (int k = 0; k < 4; ++k) w[k] = lane[(hi ? NP * LS : 0) + 12 + ((x ? a + k : b - k) & 3)];
    };
    auto absolute = [&]() {
#pragma unroll
      for (int k = 0; k < 4; ++k) w[k] = fabs(w[k]);
      return w;
    };
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      weights(i < 2, i & 1);
      fl[i] = i < 2 ? xdot(w, o[0]) : ydot(w, o[0]);
      fv[i] = i < 2 ? xdot(absolute(), var) : ydot(absolute(), var);
    }
    transpose_rows(mn);
    transpose_rows(vr);
    transpose_rows(fl);
    transpose_rows(fv);
    ok = (safe(mn, vr) && safe(fl, fv)) || !point;
  }
  if (__ballot(!ok) == 0) return 0;

  FaceOps L;
  make_face_ops(lane, a, b, L);
  // node-by-node test: four nodes at a time, row h the h-th at the solution point; per node
  // row h the h-th face point
  double rmin = INFINITY, pmin = INFINITY;
  auto at_nodes = [&](auto&& test) {
#pragma unroll 1
    for (int q = 0; q < NQ; q += 4) {
      double v[4], U[4];
      expand4<M, NQ>(o, phi, q, v);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        U[0] = xdot(L.lx, v[i]);
        U[1] = xdot(L.rx, v[i]);
        U[2] = ydot(L.ly, v[i]);
        U[3] = ydot(L.ry, v[i]);
        transpose_rows(U);
        test(U);
      }
      transpose_rows(v);
      test(v);
    }
  };
  at_nodes([&](double* U) {
    rmin = fmin(rmin, U[0]);
    pmin = fmin(pmin, euler_p(U, g));
  });
  if (!point) rmin = pmin = INFINITY;
  rmin = wave_min(rmin);
  pmin = wave_min(pmin);
  if (!(fmin(rmin, pmin) < eps)) return 0;
  const double beta1 = (rmin >= eps) ? 1.0 : (ub[0] - eps) / (ub[0] - rmin);
  double bmin = 1.0;
  at_nodes([&](double* U) {
    U[0] = beta1 * (U[0] - ub[0]) + ub[0];
    if (euler_p(U, g) < eps) bmin = fmin(bmin, pressure_root<kEuler2>(ub, U, eps, g));
  });
  if (!point) bmin = 1.0;
  const double beta2 = wave_min(bmin);
  const double us = h == 0 ? ub[0] : h == 1 ? ub[1] : h == 2 ? ub[2] : ub[3];
#pragma unroll
  for (int k = 0; k < M; ++k) {
    const double m0 = (k == 0) ? 1.0 : 0.0;
    double v = o[k];
    if (h == 0) v = beta1 * (v - us * m0) + us * m0;
    o[k] = beta2 * (v - us * m0) + us * m0;
  }
  return 1;
}

// what the filter reads per lane and mode, staged by the workgroup
template <int M, int N>
struct FilterLds {
  double lam[M * N * N], shell[M * N * N];  // filter factors, weights of the detector's outer shell
  double V[NP * NP], Vinv[NP * NP];         // padded to 4 x 4
};

// detector and modal filter on the wave's element (Sec. 4.1, 4.2)
template <int M, int N>
__device__ __forceinline__ int filter_wave(const KParams& P, double (&o)[M], int a, int b, int jp,
                                           const FilterLds<M, N>& F) {
  constexpr int NS = N * N;
  double vix[4], viy[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    vix[k] = F.Vinv[a * NP + ((a + k) & 3)];
    viy[k] = F.Vinv[b * NP + ((b - k) & 3)];
  }
  if (P.sensor != FRSG_SENSOR_ALWAYS) {
    // energies of the first variable's spatial-chaos modes (row 0)
    double num = 0.0, den = 0.0;
#pragma unroll
    for (int k = 0; k < M; ++k) {
      const double t = ydot(viy, xdot(vix, o[k]));
      const double e2 = t * t;
      num += e2 * F.shell[k * NS + jp];  // t is 0 on padding lanes
      den += e2;
    }
    num = row_value(ysum4(xsum4(num)), 0);
    den = row_value(ysum4(xsum4(den)), 0);
    if (!(den > 0.0 && num / den > P.sensor_thr)) return 0;
  }
  double vx[4], vy[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    vx[k] = F.V[a * NP + ((a + k) & 3)];
    vy[k] = F.V[b * NP + ((b - k) & 3)];
  }
#pragma unroll
  for (int k = 0; k < M; ++k) {
    const double t = ydot(viy, xdot(vix, o[k])) * F.lam[k * NS + jp];
    o[k] = ydot(vy, xdot(vx, t));
  }
  return 1;
}

// SSP: a stage of SSP-RK3 (out = cu u + cw (in + dt R)); otherwise the right-hand side alone or a
// Butcher row (an instance of its own: with both ends in one kernel the residuals spill)
template <int M, int NQ, int FLUX, int N, bool SSP>
__global__ void __launch_bounds__(WBLK, 4)
k_stage2w(KParams P, StageArgs A, const double* __restrict__ PhiT, const double* __restrict__ PWT,
          const double* __restrict__ in, const double* uin, double* out) {
  constexpr int NS = N * N;
  using H2 = Half2<double>;
  // The loop's LDS.  sU: nodal values of an element at the group's nodes, [row][variable pair]
  // [point]; the interface fluxes take its place (written and read by the element's own wave).
  // sT: traces at the faces inside the tile, for the neighbour, [row][variable
  // pair][direction: the tile's inner x or y face][face point]; one buffer, which the barrier at the
  // end of a group keeps until the neighbour has read it.  sH: traces of the elements around the tile at every node.
  struct LoopLds {
    H2 sU[WE][4][2][NSP];
    H2 sT[WE][4][2][2][NP];
    Quad4<double> sH[NQ][WHF][NP];
  };
  __shared__ union {
    LoopLds loop;
    double sO[WE][4][NSP][M];  // the output, for its face traces
    FilterLds<M, N> filt;
    double red[WE];
  } lds;
  __shared__ __attribute__((aligned(16))) double sLane[NSP][LS];
  auto& sU = lds.loop.sU;
  auto& sT = lds.loop.sT;
  auto& sH = lds.loop.sH;

  const int tid0 = threadIdx.x, tid = tid0;
  const int le = __builtin_amdgcn_readfirstlane(tid >> 6), h = (tid >> 4) & 3, j = tid & 15;
  const int a = j & 3, b = j >> 2;
  const int lx = le % WX, ly = le / WX;
  // XCD-aware order: each XCD gets a contiguous band of tiles (neighbouring halos then share
  // its L2), walked in blocks of 8 x 8 tiles
  const int ntx = (P.nx + WX - 1) / WX, nty = (P.ny + WY - 1) / WY, ntiles = ntx * nty;
  int tile = blockIdx.x;
  if (ntiles % 8 == 0) tile = (tile % 8) * (ntiles / 8) + tile / 8;
  int tx, ty;
  if (ntx % 8 == 0 && nty % 8 == 0) {
    const int blk = tile >> 6, w = tile & 63, nbx = ntx / 8;
    tx = (blk % nbx) * 8 + (w & 7);
    ty = (blk / nbx) * 8 + (w >> 3);
  } else {
    tx = tile % ntx;
    ty = tile / ntx;
  }
  // the last tile of a row or column may be cut short (tnx x tny elements); waves past the mesh
  // and the lanes past the N x N points of an element run along on a neighbouring element's or
  // point's data and take no part in any result
  const int tnx = min(WX, P.nx - WX * tx), tny = min(WY, P.ny - WY * ty);
  const bool inside = lx < tnx && ly < tny;
  const bool point = N == NP || (a < N && b < N);
  const int ix = WX * tx + min(lx, tnx - 1), iy = WY * ty + min(ly, tny - 1);
  const int jp = N == NP ? j : min(a, N - 1) + N * min(b, N - 1);  // point index in the state arrays
  const int e = iy * P.nx + ix;
  const long EN = (long)P.E * NS;
  const Table phi = (Table)PhiT, pwt = (Table)PWT;

  // own coefficients: variable h (the state is below 4 GiB, checked by the host)
  const unsigned sbytes = (unsigned)(4 * M * EN * (long)sizeof(double));
  const unsigned voff = (unsigned)(((long)h * M * EN + (long)e * NS + jp) * (long)sizeof(double));
  auto soff = [&](int k) { return (unsigned)((long)k * EN * (long)sizeof(double)); };
  // point weights of a lane, scaled: -1/Jx Dt and -1/Jy Dt (rotated for xdot, ydot), the
  // correction's derivatives at the point's line and column, the weights of flux point j
  const int fside = j >> 2, fi = j & 3;
  const bool lo_side = (fside & 1) == 0;
  // traces of the elements around the tile at every node: one thread per (face hf, face point
  // hfp, variable hs) and half of the nodes; faces: WY x-lo, WY x-hi, WX y-lo, WX y-hi
  constexpr int TPT = WHF * 4 * N * M;
  constexpr int HALO = WHF * NP * 4, Q1 = (NQ / 2 + 3) & ~3;
  static_assert(HALO % 64 == 0 && 2 * HALO <= WBLK, "halo threads fill whole waves");
  const int hq = 64 * le < HALO ? 0 : 1, ht = tid - hq * HALO;
  const int hf = ht >> 4, hs = tid & 3;
  double th[M];
  if (tid < 2 * HALO) {  // uniform per wave
    const int hfp = N == NP ? (tid >> 2) & 3 : min((tid >> 2) & 3, N - 1);
    int nix, niy;
    bool along_x, from_lo;  // from_lo: the face is the neighbour's lo face (trace at -1)
    if (hf < WY) { nix = WX * tx - 1; niy = WY * ty + hf; along_x = true; from_lo = false; }
    else if (hf < 2 * WY) { nix = WX * tx + tnx; niy = WY * ty + hf - WY; along_x = true; from_lo = true; }
    else if (hf < 2 * WY + WX) { nix = WX * tx + hf - 2 * WY; niy = WY * ty - 1; along_x = false; from_lo = false; }
    else { nix = WX * tx + hf - 2 * WY - WX; niy = WY * ty + tny; along_x = false; from_lo = true; }
    // rows and columns past the mesh have no neighbour
    bool valid = along_x ? (hf < WY ? hf : hf - WY) < tny : (hf < 2 * WY + WX ? hf - 2 * WY : hf - 2 * WY - WX) < tnx;
    if (nix < 0) { if (P.bc[0] == FRSG_BC_PERIODIC) nix += P.nx; else valid = false; }
    if (nix >= P.nx) { if (P.bc[1] == FRSG_BC_PERIODIC) nix -= P.nx; else valid = false; }
    if (niy < 0) { if (P.bc[2] == FRSG_BC_PERIODIC) niy += P.ny; else valid = false; }
    if (niy >= P.ny) { if (P.bc[3] == FRSG_BC_PERIODIC) niy -= P.ny; else valid = false; }
    // a face without a neighbour (domain boundary) reads tile or element 0 instead, and its
    // trace is never used: the lanes on that face take the ghost state
    if (A.tr_in) {  // uniform: the traces were written by the launch that wrote the input
      // the neighbour tile's face slot that faces this one (x-lo halo <- x-hi slot, ...)
      const int slot = hf < WY ? WY + hf
                     : hf < 2 * WY ? hf - WY
                     : hf < 2 * WY + WX ? hf + WX
                     : hf - WX;
      const int nt = valid ? (niy / WY) * ntx + nix / WX : 0;
      const auto rtr = state_rsrc(A.tr_in, (unsigned)((long)ntiles * TPT * (long)sizeof(double)));
      const unsigned to = (unsigned)(((long)nt * TPT + (slot * M * N + hfp) * 4 + hs) * (long)sizeof(double));
#pragma unroll
      for (int k = 0; k < M; ++k) th[k] = bload(rtr, to, (unsigned)(k * N * 4 * sizeof(double)));
    } else {
      const int ne = valid ? niy * P.nx + nix : 0;
      const auto rh = state_rsrc(in, sbytes);
      unsigned ho[N];
#pragma unroll
      for (int c = 0; c < N; ++c)
        ho[c] = (unsigned)((((long)hs * M) * EN + (long)ne * NS + (along_x ? c + N * hfp : hfp + N * c)) *
                           (long)sizeof(double));
#pragma unroll
      for (int k = 0; k < M; ++k) {
        double t = 0.0;
#pragma unroll
        for (int c = 0; c < N; ++c) t += (from_lo ? P.tab.lL[c] : P.tab.lR[c]) * bload(rh, ho[c], soff(k));
        th[k] = t;
        if (k % 5 == 4) __builtin_amdgcn_sched_barrier(0);  // not all 4 M loads in registers at once
      }
    }
  }
  double m[M];
  {
    const auto rin = state_rsrc(in, sbytes);
#pragma unroll
    for (int k = 0; k < M; ++k) m[k] = bload_stream(rin, voff, soff(k));
  }

  if (tid < NSP) {
    const double iJx = -1.0 / P.Jx, iJy = -1.0 / P.Jy;
    double* w = sLane[j];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      w[k] = iJx * mpad<N>(A.Dt, a, (a + k) & 3);
      w[4 + k] = iJy * mpad<N>(A.Dt, b, (b - k) & 3);
      w[12 + k] = wpad<N>(lo_side ? P.tab.lL : P.tab.lR, k);
    }
    w[8] = iJx * wpad<N>(P.tab.dhL, a);
    w[9] = iJx * wpad<N>(P.tab.dhR, a);
    w[10] = iJy * wpad<N>(P.tab.dhL, b);
    w[11] = iJy * wpad<N>(P.tab.dhR, b);
    w[16] = 0.25 * wpad<N>(P.tab.w, a) * wpad<N>(P.tab.w, b);  // share of the point in the element mean
  }

  if (tid < 2 * HALO) {
    const int fp = (tid >> 2) & 3, qe = hq ? NQ : Q1;
#pragma unroll 1
    for (int q = hq * Q1; q < qe; q += 4) {
      double t[4];
      expand4<M, NQ>(th, phi, q, t);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (q + i < qe) sH[q + i][hf][fp].v[hs] = t[i];
    }
  }

  // face-point role: flux point j of this element, side = j >> 2 (x-lo, x-hi, y-lo, y-hi)
  int nbr_le = -1, nbr_halo = 0;
  bool boundary = false;
  if (fside == 0) {
    if (lx > 0) nbr_le = le - 1;
    else if (ix == 0 && P.bc[0] != FRSG_BC_PERIODIC) boundary = true;
    else nbr_halo = ly;
  } else if (fside == 1) {
    if (lx < tnx - 1) nbr_le = le + 1;
    else if (ix == P.nx - 1 && P.bc[1] != FRSG_BC_PERIODIC) boundary = true;
    else nbr_halo = WY + ly;
  } else if (fside == 2) {
    if (ly > 0) nbr_le = le - WX;
    else if (iy == 0 && P.bc[2] != FRSG_BC_PERIODIC) boundary = true;
    else nbr_halo = 2 * WY + lx;
  } else {
    if (ly < tny - 1) nbr_le = le + WX;
    else if (iy == P.ny - 1 && P.bc[3] != FRSG_BC_PERIODIC) boundary = true;
    else nbr_halo = 2 * WY + WX + lx;
  }
  const bool wave_at_boundary = __ballot(boundary) != 0;
  // where the lane reads the neighbour's trace: in sT or in sH
  const bool inner = nbr_le >= 0;
  const H2* const nb_base = inner ? &sT[nbr_le][h][0][fside >> 1][fi]
                                  : reinterpret_cast<const H2*>(&sH[0][nbr_halo][fi]);

  double acc[M];
#pragma unroll
  for (int k = 0; k < M; ++k) acc[k] = 0.0;
  auto wave_sync = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  __syncthreads();

#pragma unroll 1
  for (int q0 = 0; q0 < NQ; q0 += 4) {
    // the lane's place and weights are computed and read anew for each group, to keep the
    // registers free
    int t = tid0;
    asm volatile("" : "+v"(t));
    const int h = (t >> 4) & 3, j = t & 15, a = j & 3, b = j >> 2, fside = b, fi = a;
    const bool lo_side = (fside & 1) == 0;
    const double* W = sLane[j];
    H2(*const X)[NSP] = sU[le][h];
    // (1) all four variables at (j, q0 + h), and the flux divergence there
    double U[4], r[4];
    expand4<M, NQ>(m, phi, q0, U);
    transpose_rows(U);
    X[0][j] = H2{U[0], U[1]};
    X[1][j] = H2{U[2], U[3]};
    {
      const double ir = recip(U[0]);
      const double p = (P.gamma - 1.0) * (U[3] - 0.5 * (U[1] * U[1] + U[2] * U[2]) * ir);
      const double vx = U[1] * ir, vy = U[2] * ir;
      const double Ep = U[3] + p;
      double w[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) w[k] = W[k];
      r[0] = xdot(w, U[1]);
      r[1] = xdot(w, U[1] * vx + p);
      r[2] = xdot(w, U[2] * vx);
      r[3] = xdot(w, Ep * vx);
#pragma unroll
      for (int k = 0; k < 4; ++k) w[k] = W[4 + k];
      r[0] += ydot(w, U[2]);
      r[1] += ydot(w, U[1] * vy);
      r[2] += ydot(w, U[2] * vy + p);
      r[3] += ydot(w, Ep * vy);
      // finished here: the compiler would move the sums behind the interface flux and carry
      // their 24 rotated operands through it
#pragma unroll
      for (int s = 0; s < 4; ++s) asm volatile("" : "+v"(r[s]));
    }
    wave_sync();
    // (2) solution trace at flux point j, along its line of solution points
    double T[4];
    {
      const int l0 = fside < 2 ? NP * fi : fi, ls = fside < 2 ? 1 : NP;
#pragma unroll
      for (int v = 0; v < 2; ++v) {
#pragma unroll
        for (int c = 0; c < N; ++c) {
          const double w = W[12 + c];
          const H2 x = X[v][l0 + ls * c];
          T[2 * v] = c == 0 ? w * x.x : T[2 * v] + w * x.x;
          T[2 * v + 1] = c == 0 ? w * x.y : T[2 * v + 1] + w * x.y;
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (inner) {
      H2* const to = &sT[le][h][0][fside >> 1][fi];
      to[0] = H2{T[0], T[1]};
      to[2 * NP] = H2{T[2], T[3]};
    }
    __syncthreads();
    // (3) interface flux at flux point j
    {
      const int qh = min(q0 + h, NQ - 1);
      const H2* src = nb_base + (inner ? 0 : qh * (int)(sizeof(sH[0]) / sizeof(H2)));
      const H2 n0 = src[0], n1 = src[inner ? 2 * NP : 1];
      double nb[4] = {n0.x, n0.y, n1.x, n1.y};
      if (wave_at_boundary) {  // uniform: only waves with a domain-boundary face pay for the ghosts
        const int gkind = P.bc[fside], gnormal = fside < 2 ? 1 : 2;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          double gh = (gkind == FRSG_BC_DIRICHLET) ? P.bc_state[fside][s] : T[s];
          if (gkind == FRSG_BC_REFLECT && s == gnormal) gh = -gh;
          nb[s] = boundary ? gh : nb[s];
        }
      }
      double Fs[4];
      // as on an x face, the normal momentum first
      auto turn = [&](double* v) {
        const double x = v[1];
        v[1] = fside < 2 ? x : v[2];
        v[2] = fside < 2 ? v[2] : x;
      };
      turn(T);
      turn(nb);
      if constexpr (FLUX == FRSG_FLUX_HLL)
        hll_e2(T, nb, lo_side, Fs, P.gamma, 0);
      else
        rusanov_e2(T, nb, lo_side, Fs, P.gamma, 0);
      turn(Fs);
      X[0][j] = H2{Fs[0], Fs[1]};
      X[1][j] = H2{Fs[2], Fs[3]};
    }
    wave_sync();
    // (4) nodal residual at (j, q0 + h); back to variable h at the four nodes, projected
    {
#pragma unroll
      for (int v = 0; v < 2; ++v) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const double w = W[8 + c];
          const H2 x = X[v][(c < 2 ? b : a) + NP * c];
          r[2 * v] += w * x.x;
          r[2 * v + 1] += w * x.y;
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      transpose_rows(r);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (q0 + i < NQ) {
#pragma unroll
          for (int k = 0; k < M; ++k) acc[k] += pwt[(q0 + i) * M + k] * r[i];
        }
    }
    __syncthreads();  // fluxes and traces are read before the next group's take their place
  }

  {
  // ----------------------------------------------------------------- epilogue
  // the lane's place anew, so that it need not be kept through the loop
  int te = tid0;
  asm volatile("" : "+v"(te));
  const int tid = te, h = (tid >> 4) & 3, j = tid & 15, a = j & 3, b = j >> 2;
  const bool point = N == NP || (a < N && b < N);
  const int jp = N == NP ? j : min(a, N - 1) + N * min(b, N - 1);
  const unsigned voff = (unsigned)(((long)h * M * EN + (long)e * NS + jp) * (long)sizeof(double));
  const auto rout = state_rsrc(out, sbytes);
  const bool own = inside && point;  // the lane's point belongs to the state
  if (!SSP && A.stage == 0) {
    if (own) {
#pragma unroll
      for (int k = 0; k < M; ++k) bstore(acc[k], rout, voff, soff(k));
    }
    return;
  }
  const double dt = stage_dt(P, A.sdt);
  double o[M];
  if constexpr (!SSP) {
    // the earlier stages' terms first, in stage order, then this stage's
#pragma unroll
    for (int k = 0; k < M; ++k) o[k] = 0.0;
    for (int t = 0; t < A.nt; ++t) {
      const auto rk = state_rsrc(A.kk[t], sbytes);
      const double at = A.ka[t];
#pragma unroll
      for (int k = 0; k < M; ++k) o[k] = o[k] + at * bload_stream(rk, voff, soff(k));
    }
    const auto ru = state_rsrc(uin, sbytes);
    const auto rko = state_rsrc(A.k_out, A.k_out ? sbytes : 0u);  // no k_out: an empty range drops the stores
    if (own) {
#pragma unroll
      for (int k = 0; k < M; ++k) bstore(acc[k], rko, voff, soff(k));
    }
    if (A.ka_cur != 0.0) {
#pragma unroll
      for (int k = 0; k < M; ++k) o[k] += A.ka_cur * acc[k];
    }
    __builtin_amdgcn_sched_barrier(0);  // acc is done with before u takes its registers
#pragma unroll
    for (int k = 0; k < M; ++k) o[k] = bload_stream(ru, voff, soff(k)) + dt * o[k];
  } else {
    const auto ru = state_rsrc(uin, A.cu != 0.0 ? sbytes : 0u);
#pragma unroll
    for (int k = 0; k < M; ++k) o[k] = A.cw * (m[k] + dt * acc[k]);
    __builtin_amdgcn_sched_barrier(0);  // m and acc are done with before u takes their registers
#pragma unroll
    for (int k = 0; k < M; ++k) o[k] += A.cu * bload_stream(ru, voff, soff(k));  // 0 from an empty range when cu = 0
  }

  if (A.stage == 3) {
    int ff = 0;
    if (P.filter != FRSG_FILTER_NONE) {
      __syncthreads();  // the node loop's LDS is free
      for (int i = tid; i < M * NS; i += WBLK) {
        const double f = P.tab.filt[i];
        lds.filt.lam[i] = (P.filter == FRSG_FILTER_EXP) ? exp(-P.alpha * dt * f) : f;
        lds.filt.shell[i] = P.tab.shell[i];
      }
      if (tid < NP * NP) {
        lds.filt.V[tid] = mpad<N>(P.tab.V, tid / NP, tid % NP);
        lds.filt.Vinv[tid] = mpad<N>(P.tab.Vinv, tid / NP, tid % NP);
      }
      __syncthreads();
      ff = filter_wave<M, N>(P, o, a, b, jp, lds.filt);
    }
    if (tid % 64 == 0 && inside && A.flag_filt) A.flag_filt[e] = (unsigned char)ff;
  }
  if (P.limiter) {
    const int lf = inside ? limit_wave<M, NQ, N>(P, phi, o, a, b, (Table)A.cmax, &sLane[0][0], point) : 0;
    if (tid % 64 == 0 && inside && A.flag_lim && (lf || !A.flag_or)) A.flag_lim[e] = (unsigned char)lf;
  } else if (tid % 64 == 0 && inside && A.flag_lim && !A.flag_or) {
    A.flag_lim[e] = 0;
  }
  if (!SSP && tid % 64 == 0 && inside && A.flag_zero) A.flag_zero[e] = 0;

  if (own) {
#pragma unroll
    for (int k = 0; k < M; ++k) bstore(o[k], rout, voff, soff(k));
  }

  // modal face traces of the new state on the tile's boundary faces, for the next launch's
  // neighbours: [face slot][mode][face point][variable], the order of the lanes that read them
  if (A.tr_out) {  // uniform
    __syncthreads();
#pragma unroll
    for (int k = 0; k < M; ++k) lds.sO[le][h][j][k] = o[k];
    __syncthreads();
    const int tile_id = ty * ntx + tx;
    const auto rtr = state_rsrc(A.tr_out, (unsigned)((long)ntiles * TPT * (long)sizeof(double)));
    const unsigned tbase = (unsigned)((long)tile_id * TPT * (long)sizeof(double));
    // thread (slot, variable, face point) and every KS-th mode
    constexpr int KS = WBLK / (WHF * 16);
    const int sv = tid & 3, fp = (tid >> 2) & 3, slot = (tid >> 4) % WHF, k0 = (tid >> 4) / WHF;
    int el, at, step;  // the element, the first point of the line through the face point and its stride
    bool lo;
    if (slot < 2 * WY) {
      lo = slot < WY;
      el = (lo ? 0 : tnx - 1) + WX * (lo ? slot : slot - WY);
      at = NP * fp;
      step = 1;
    } else {
      lo = slot < 2 * WY + WX;
      el = (lo ? slot - 2 * WY : slot - 2 * WY - WX) + (lo ? 0 : WX * (tny - 1));
      at = fp;
      step = NP;
    }
    double w[N];
#pragma unroll
    for (int c = 0; c < N; ++c) w[c] = sLane[lo ? 0 : NP][12 + c];
    if (k0 < KS && fp < N) {
      const unsigned to = tbase + (unsigned)(((slot * M * N + fp) * 4 + sv) * (int)sizeof(double));
#pragma unroll
      for (int i = 0; i < (M + KS - 1) / KS; ++i) {
        const int k = k0 + KS * i;
        if (k < M) {
          double t = 0.0;
#pragma unroll
          for (int c = 0; c < N; ++c) t += w[c] * lds.sO[el][sv][at + step * c][k];
          bstore(t, rtr, to + (unsigned)(k * N * 4 * (int)sizeof(double)), 0u);
        }
      }
    }
  }

  // CFL maximum of the new state for the next step
  if (A.stage == 3 && A.lam_next) {
    const double gd = P.gamma, idx = 1.0 / P.dx, idy = 1.0 / P.dy;
    double rate = 0.0;
#pragma unroll 1
    for (int q = 0; q < NQ; q += 4) {
      // (|vx| + c) / dx + (|vy| + c) / dy at node q + h; NaN counts as infinity
      double U[4];
      expand4<M, NQ>(o, phi, q, U);
      transpose_rows(U);
      const double ir = recip(U[0]);
      const double vx = U[1] * ir, vy = U[2] * ir;
      const double p = (gd - 1.0) * (U[3] - 0.5 * (U[1] * vx + U[2] * vy));
      const double c = sqrt(gd * p * ir);
      const double r = (fabs(vx) + c) * idx + (fabs(vy) + c) * idy;
      rate = fmax(rate, (r == r) ? r : __longlong_as_double(0x7ff0000000000000ll));
    }
    if (!own) rate = 0.0;
    for (int w = 32; w > 0; w >>= 1) rate = fmax(rate, __shfl_xor(rate, w));
    __syncthreads();
    if ((tid & 63) == 0) lds.red[le] = rate;
    __syncthreads();
    if (tid == 0) {
      double r = lds.red[0];
      for (int w = 1; w < WE; ++w) r = fmax(r, lds.red[w]);
      atomicMax(A.lam_next, (unsigned long long)__double_as_longlong(r));
    }
  }
  }
}

template <int M, int NQ>
hipError_t launch_t(const KParams& P, const StageArgs& A, const FusedStage& S, hipStream_t s) {
  const int ntiles = wave2d_tiles(P.nx, P.ny);
  const bool ssp = S.stage != 0 && !S.tab;
#define FRSG_WAVE_T(FLUX, NN, SSP)                                                                                 \
  hipLaunchKernelGGL((k_stage2w<M, NQ, FLUX, NN, SSP>), dim3(ntiles), dim3(WBLK), 0, s, P, A, S.PhiT, S.PWT, S.in, S.u, \
                     S.out)
#define FRSG_WAVE(FLUX, NN)                    \
  do {                                         \
    if (ssp) FRSG_WAVE_T(FLUX, NN, true);      \
    else FRSG_WAVE_T(FLUX, NN, false);         \
  } while (0)
  if (P.flux == FRSG_FLUX_HLL) {
    if (P.np1 == 3) FRSG_WAVE(FRSG_FLUX_HLL, 3);
    else FRSG_WAVE(FRSG_FLUX_HLL, NP);
  } else {
    if (P.np1 == 3) FRSG_WAVE(FRSG_FLUX_RUSANOV, 3);
    else FRSG_WAVE(FRSG_FLUX_RUSANOV, NP);
  }
#undef FRSG_WAVE
#undef FRSG_WAVE_T
  return hipGetLastError();
}

}  // namespace

hipError_t launch_wave_stage(const KParams& P, const FusedStage& S, hipStream_t s) {
  if (P.eq != kEuler2 || (P.np1 != 3 && P.np1 != 4) || S.fp32) return hipErrorInvalidValue;
  const StageArgs A = stage_args(S);
#define X(MM, QQ)                                                           \
  if constexpr (wave2d_nodes(QQ))                                           \
    if (P.M == MM && P.Nq == QQ) return launch_t<MM, QQ>(P, A, S, s);
  FRSG_FUSED_SIZES(X)
#undef X
  return hipErrorInvalidValue;
}

}  // namespace frsg
