// Triangle path of the 2D Euler right-hand side (Sec. 3.5 multi-dimensional FR
// on the triangles of Sec. 3.1).  First the multi-pass kernels, for the mode and
// node counts that the fused stage below is not compiled for: as on the generic
// quadrilateral path the nodal values and fluxes at (node, element, solution
// point) come from the shared nodal pass; these add the interactive fluxes at
// the flux points, the nodal residual (flux divergence plus the correction-field
// lifting) and the CFL maximum.  Nodal arrays: [S][Nq][E][N_p]; face jumps:
// [S][Nq][E][3 nfp].  Then the fused stage, one launch per Runge-Kutta stage.
#include "device_common.hpp"

namespace frsg {
namespace {

constexpr int kBlockT = 256;

__device__ __forceinline__ double euler2_p(const double* U, double gamma) {
  return (gamma - 1.0) * (U[3] - 0.5 * (U[1] * U[1] + U[2] * U[2]) / U[0]);
}

// normal flux F . n of the 2D Euler equations, unit normal (nx, ny)
__device__ __forceinline__ void normal_flux(const double* U, double nx, double ny, double gamma, double* F,
                                            double& vn, double& c) {
  const double p = euler2_p(U, gamma);
  vn = (U[1] * nx + U[2] * ny) / U[0];
  c = sqrt(gamma * p / U[0]);
  F[0] = U[0] * vn;
  F[1] = U[1] * vn + p * nx;
  F[2] = U[2] * vn + p * ny;
  F[3] = (U[3] + p) * vn;
}

// interactive flux along the normal, per random node: Lax-Friedrichs with the
// larger of |v.n| + c on the two sides, or HLL with Davis's speeds
__device__ __forceinline__ void flux_n(int kind, const double* L, const double* R, double nx, double ny, double gamma,
                                       double* Fs) {
  double FL[4], FR[4], uL, cL, uR, cR;
  normal_flux(L, nx, ny, gamma, FL, uL, cL);
  normal_flux(R, nx, ny, gamma, FR, uR, cR);
  if (kind == FRSG_FLUX_HLL) {
    const double SL = fmin(uL - cL, uR - cR), SR = fmax(uL + cL, uR + cR);
#pragma unroll
    for (int s = 0; s < 4; ++s)
      Fs[s] = (SL >= 0.0) ? FL[s] : (SR <= 0.0) ? FR[s] : (SR * FL[s] - SL * FR[s] + (SL * SR) * (R[s] - L[s])) / (SR - SL);
  } else {
    const double lam = fmax(fabs(uL) + cL, fabs(uR) + cR);
#pragma unroll
    for (int s = 0; s < 4; ++s) Fs[s] = 0.5 * (FL[s] + FR[s]) - 0.5 * lam * (R[s] - L[s]);
  }
}

// 1/x: hardware estimate and two Newton steps (full double accuracy for the
// positive densities it is applied to)
__device__ __forceinline__ double rcp2(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = fma(-x, r, 1.0);
  r = fma(r, e, r);
  e = fma(-x, r, 1.0);
  return fma(r, e, r);
}

// a[s] for a run-time s without indexing a private array
__device__ __forceinline__ double pick4(const double* a, int s) {
  return s == 0 ? a[0] : (s == 1 ? a[1] : (s == 2 ? a[2] : a[3]));
}

// interactive flux along the unit normal with one reciprocal of the density per side
__device__ __forceinline__ void interactive_n(int kind, const double* L, const double* R, double nx, double ny,
                                              double gamma, double* Fs) {
  const double iL = rcp2(L[0]), iR = rcp2(R[0]);
  const double uL = (L[1] * nx + L[2] * ny) * iL, uR = (R[1] * nx + R[2] * ny) * iR;
  const double pL = (gamma - 1.0) * (L[3] - 0.5 * (L[1] * L[1] + L[2] * L[2]) * iL);
  const double pR = (gamma - 1.0) * (R[3] - 0.5 * (R[1] * R[1] + R[2] * R[2]) * iR);
  const double cL = sqrt(gamma * pL * iL), cR = sqrt(gamma * pR * iR);
  const double FL[4] = {L[0] * uL, L[1] * uL + pL * nx, L[2] * uL + pL * ny, (L[3] + pL) * uL};
  const double FR[4] = {R[0] * uR, R[1] * uR + pR * nx, R[2] * uR + pR * ny, (R[3] + pR) * uR};
  if (kind == FRSG_FLUX_HLL) {
    const double SL = fmin(uL - cL, uR - cR), SR = fmax(uL + cL, uR + cR), iw = rcp2(SR - SL);
#pragma unroll
    for (int s = 0; s < 4; ++s)
      Fs[s] = (SL >= 0.0) ? FL[s] : (SR <= 0.0) ? FR[s] : (SR * FL[s] - SL * FR[s] + (SL * SR) * (R[s] - L[s])) * iw;
  } else {
    const double hl = 0.5 * fmax(fabs(uL) + cL, fabs(uR) + cR);
#pragma unroll
    for (int s = 0; s < 4; ++s) Fs[s] = 0.5 * (FL[s] + FR[s]) - hl * (R[s] - L[s]);
  }
}

// ghost state outside a boundary face of kind bc[side] (reflection about the face)
__device__ __forceinline__ void ghost_n(const KParams& P, int side, const double* in, double nx, double ny,
                                        double* out) {
  const int kind = P.bc[side];
#pragma unroll
  for (int s = 0; s < 4; ++s) out[s] = (kind == FRSG_BC_DIRICHLET) ? P.bc_state[side][s] : in[s];
  if (kind == FRSG_BC_REFLECT) {
    const double mn = in[1] * nx + in[2] * ny;
    out[1] = in[1] - 2.0 * mn * nx;
    out[2] = in[2] - 2.0 * mn * ny;
  }
}

// thread per (node q, element e, face f, flux point k): traces of both sides
// (the neighbour runs the shared face the other way), interactive flux minus the
// interpolated flux along the outward normal, times (face length / reference
// face length / det) for the lifting
__global__ void __launch_bounds__(kBlockT) k_faces_tri(KParams P, const double* __restrict__ Un,
                                                       const double* __restrict__ Fn, const double* __restrict__ Gn,
                                                       double* __restrict__ Jump) {
  const int np = P.nsp, nfp = P.nfp, E = P.E;
  const long NF = (long)P.Nq * E * 3 * nfp;
  const long t = blockIdx.x * (long)kBlockT + threadIdx.x;
  if (t >= NF) return;
  const int k = (int)(t % nfp);
  const int f = (int)((t / nfp) % 3);
  const long qe = t / (3 * nfp);
  const int e = (int)(qe % E);
  const long q = qe / E;
  const long total = (long)P.Nq * E * np;
  const double* geo = P.tri_geo + (long)e * kTriGeo;
  const double nx = geo[kGeoN0 + 2 * f], ny = geo[kGeoN0 + 2 * f + 1];
  const double* Lrow = P.tri_Lf + (f * nfp + k) * np;
  const long base = qe * np;
  double UL[4], FD[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    double u = 0.0, fx = 0.0, fy = 0.0;
    for (int i = 0; i < np; ++i) {
      const double l = Lrow[i];
      u += l * Un[s * total + base + i];
      fx += l * Fn[s * total + base + i];
      fy += l * Gn[s * total + base + i];
    }
    UL[s] = u;
    FD[s] = nx * fx + ny * fy;
  }
  double UR[4];
  const int nb = P.tri_nbr[e * 6 + f];
  if (nb >= 0) {
    const int g = P.tri_nbr[e * 6 + 3 + f];
    const double* Lnb = P.tri_Lf + (g * nfp + (nfp - 1 - k)) * np;
    const long nbase = (q * E + nb) * np;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      double u = 0.0;
      for (int i = 0; i < np; ++i) u += Lnb[i] * Un[s * total + nbase + i];
      UR[s] = u;
    }
  } else {
    ghost_n(P, -1 - nb, UL, nx, ny, UR);
  }
  double Fs[4];
  flux_n(P.flux, UL, UR, nx, ny, P.gamma, Fs);
  const double sc = geo[kGeoSc0 + f];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    Jump[s * NF + t] = (Fs[s] - FD[s]) * sc;
  }
}

// thread per (node q, element e, solution point j): -(div F^D + sum_fk lift_jfk jump_fk)
__global__ void __launch_bounds__(kBlockT) k_resid_tri(KParams P, const double* __restrict__ Fn,
                                                       const double* __restrict__ Gn,
                                                       const double* __restrict__ Jump, double* __restrict__ Rn) {
  const int np = P.nsp, nf = 3 * P.nfp, E = P.E;
  const long total = (long)P.Nq * E * np;
  const long t = blockIdx.x * (long)kBlockT + threadIdx.x;
  if (t >= total) return;
  const int j = (int)(t % np);
  const long qe = t / np;
  const int e = (int)(qe % E);
  const double* geo = P.tri_geo + (long)e * kTriGeo;
  const double rx = geo[kGeoRx], ry = geo[kGeoRy], sx = geo[kGeoSx], sy = geo[kGeoSy];
  const double* Dr = P.tri_Dr + j * np;
  const double* Ds = P.tri_Ds + j * np;
  const double* lift = P.tri_lift + j * nf;
  const long NF = (long)P.Nq * E * nf;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const double* F = Fn + s * total + qe * np;
    const double* G = Gn + s * total + qe * np;
    double dr = 0.0, ds = 0.0;
    for (int i = 0; i < np; ++i) {
      const double fr = rx * F[i] + ry * G[i];
      const double fs = sx * F[i] + sy * G[i];
      dr += Dr[i] * fr;
      ds += Ds[i] * fs;
    }
    const double* J = Jump + s * NF + qe * nf;
    double c = 0.0;
    for (int m = 0; m < nf; ++m) c += lift[m] * J[m];
    Rn[s * total + t] = -(dr + ds + c);
  }
}

// CFL maximum over (node, element, solution point) of (|v| + c) / d_e, from the
// nodal values; exact max, so the reduction order does not matter
__global__ void __launch_bounds__(kBlockT) k_cfl_tri(KParams P, const double* __restrict__ Un) {
  __shared__ double sm[kBlockT];
  const int np = P.nsp, E = P.E;
  const long total = (long)P.Nq * E * np;
  const long t = blockIdx.x * (long)kBlockT + threadIdx.x;
  double rate = 0.0;
  if (t < total) {
    const int e = (int)((t / np) % E);
    double U[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) U[s] = Un[s * total + t];
    const double p = euler2_p(U, P.gamma);
    const double lam = sqrt(U[1] * U[1] + U[2] * U[2]) / U[0] + sqrt(P.gamma * p / U[0]);
    rate = lam / P.tri_geo[(long)e * kTriGeo + kGeoDin];
    if (!(rate == rate)) rate = __longlong_as_double(0x7ff0000000000000ll);  // NaN -> +inf, dt -> 0
  }
  sm[threadIdx.x] = rate;
  __syncthreads();
  for (int o = kBlockT / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) sm[threadIdx.x] = fmax(sm[threadIdx.x], sm[threadIdx.x + o]);
    __syncthreads();
  }
  if (threadIdx.x == 0) atomicMax(P.lam_bits, (unsigned long long)__double_as_longlong(sm[0]));
}

unsigned blocks(long n) { return (unsigned)((n + kBlockT - 1) / kBlockT); }

}  // namespace

hipError_t launch_faces_tri(const KParams& P, const double* Un, const double* Fn, const double* Gn, double* Jump,
                            hipStream_t s) {
  if (P.eq != FRSG_EULER2D || P.nsp > kTriMaxNp || P.nfp < 1) return hipErrorInvalidValue;
  const long NF = (long)P.Nq * P.E * 3 * P.nfp;
  hipLaunchKernelGGL(k_faces_tri, dim3(blocks(NF)), dim3(kBlockT), 0, s, P, Un, Fn, Gn, Jump);
  return hipGetLastError();
}

hipError_t launch_resid_tri(const KParams& P, const double* Fn, const double* Gn, const double* Jump, double* Rn,
                            hipStream_t s) {
  if (P.eq != FRSG_EULER2D || P.nsp > kTriMaxNp) return hipErrorInvalidValue;
  const long total = (long)P.Nq * P.E * P.nsp;
  hipLaunchKernelGGL(k_resid_tri, dim3(blocks(total)), dim3(kBlockT), 0, s, P, Fn, Gn, Jump, Rn);
  return hipGetLastError();
}

hipError_t launch_cfl_tri(const KParams& P, const double* Un, hipStream_t s) {
  if (P.eq != FRSG_EULER2D) return hipErrorInvalidValue;
  const long total = (long)P.Nq * P.E * P.nsp;
  hipLaunchKernelGGL(k_cfl_tri, dim3(blocks(total)), dim3(kBlockT), 0, s, P, Un);
  return hipGetLastError();
}


// ---------------------------------------------------------------------------
// fused stage kernel: one launch per Runge-Kutta stage on triangles
// ---------------------------------------------------------------------------
// Each element gets 4 x SLOTS threads, thread (state s, slot): slot < N_p is
// solution point j, slot < 3 nfp is flux point fk.  A thread keeps its own
// chaos coefficients of state s at point j, the neighbour's modal trace at flux
// point fk and the projection accumulators of (s, j) in registers; per group of
// four random nodes it expands both, and the element's nodal values, fluxes,
// traces and interactive fluxes pass through LDS (k_stage_tri).  The residual is
// projected on the fly and combined with the stage inputs in the epilogue, so a
// stage reads the state once and writes it once; the neighbours' modal traces
// (E x 3 nfp x S x M doubles) were written by the launch that wrote the stage
// input, or by a trace pass (k_limit_tri) before the first.
namespace {

template <int PD>
struct TriShape {
  static constexpr int NPT = (PD + 1) * (PD + 2) / 2;
  static constexpr int NFP = PD + 1;
  static constexpr int NF = 3 * NFP;
  static constexpr int SLOTS = NPT > NF ? NPT : NF;
  static constexpr int TPE = 4 * SLOTS;           // threads per element
  static constexpr int EPB = kTriEPB;             // elements per block
  static constexpr int RG = tri_row_groups(PD);   // row groups of the element operators: waves per block
  static constexpr int RT = tri_trace_rows(PD), RD = tri_point_rows(PD);  // rows per group
  static constexpr int NT = 64 * RG;              // threads per block
};

// Modal traces at the flux points, Tm[e][face][k][s][flux point of the face]: the values of one
// mode at a face are contiguous, in the order of the lanes (flux point, s) that read them, so a
// wave's load of one mode fetches whole cache lines (at p = 3 a 128-byte line per face and mode).
template <int PD, int M>
__device__ __forceinline__ long tri_trace_index(long e, int f, int k, int s, int kk) {
  return (((e * 3 + f) * M + k) * 4 + s) * (PD + 1) + kk;
}

// Place of a lane of the stage and limiter kernels: lane = 4 slot + s within its element's lanes
template <int PD>
struct TriLane {
  using Sh = TriShape<PD>;
  int rem, slot, s, e, le, ec, f, kk;
  bool active, pt, fp;
  __device__ __forceinline__ TriLane(int tid, int e0, int E) {
    const int el = tid / Sh::TPE;
    rem = tid % Sh::TPE;
    slot = rem >> 2;
    s = rem & 3;
    e = e0 + el;
    active = el < Sh::EPB && e < E;
    le = active ? el : 0;   // idle lanes point at the block's first element,
    ec = active ? e : e0;   // which exists, and use nothing of it
    pt = active && slot < Sh::NPT;
    fp = active && slot < Sh::NF;
    f = fp ? slot / Sh::NFP : 0;
    kk = fp ? slot % Sh::NFP : 0;
  }
  // mode 0 of variable s at the lane's point
  __device__ __forceinline__ long state_at(int E, int M) const {
    return ((long)s * M * E + ec) * Sh::NPT + (pt ? slot : 0);
  }
};

// Blocks are dealt to the eight dies in turn: block b works on the (b / 8)-th set of elements of
// the (b % 8)-th eighth, so that the lines shared by neighbouring sets, and most neighbours'
// traces, stay in one die's L2.  (The grid is a multiple of 8; sets past the last are empty.)
constexpr int kDies = 8;
__device__ __forceinline__ int tri_block() {
  return (int)(blockIdx.x % kDies) * (int)(gridDim.x / kDies) + (int)(blockIdx.x / kDies);
}
inline unsigned tri_grid(int E) { return (unsigned)((E + kDies * kTriEPB - 1) / (kDies * kTriEPB)) * kDies; }

// broadcast lane C of each group of four lanes (DPP quad permutation, all lanes active)
template <int C>
__device__ __forceinline__ double quad_bcast(double v) {
  constexpr int ctrl = C * 85;  // quad_perm(C, C, C, C)
  const long long x = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)x, ctrl, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(x >> 32), ctrl, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

__device__ __forceinline__ void quad_gather(double v, double* all) {
  all[0] = quad_bcast<0>(v);
  all[1] = quad_bcast<1>(v);
  all[2] = quad_bcast<2>(v);
  all[3] = quad_bcast<3>(v);
}

// LDS of the end-of-stage work below, per block
template <int PD, int M>
struct TriPostShared {
  using Sh = TriShape<PD>;
  double lam[M * Sh::NPT];  // filter factors of the step (exponential: exp(-alpha dt f))
  double num[Sh::EPB][Sh::NPT], den[Sh::EPB][Sh::NPT];
  double mn[Sh::EPB][2][Sh::TPE];
  int need[Sh::EPB], any;  // elements whose bound fails, and whether there is one
  // by the callers, before a barrier that comes ahead of post_tri: any of its waves sets them
  __device__ __forceinline__ void clear() {
    if ((int)threadIdx.x < Sh::EPB) need[threadIdx.x] = 0;
    if (threadIdx.x == 0) any = 0;
  }
};

// End-of-stage work on triangles with the stage kernel's lane layout: the sensor-gated
// modal filter (Sec. 4.1, 4.2), then the positivity limiter (Sec. 4.3).  Lane (slot, s)
// keeps the coefficients c[] of variable s at solution point `slot`; sC holds those of
// the block's elements.  The limiter decision first uses rigorous bounds per point
// (|Phi_k(z_q)| <= cmax_k, a relative margin of 1e-10 for their rounding) at the
// solution point and, as a flux-point lane, at flux point `slot`; only blocks holding an
// element whose bound fails run the node-by-node minimum and the pressure roots, so the
// decision is the node-by-node one.  The element mean is the constant chaos mode
// averaged with the triangle's quadrature weights.  c[] and sC are updated in place; a[]
// receives the final modal traces at flux point `slot` (flux-point lanes), which the limiter
// needs and the next launch reads.  Returns whether the lane's element changed.  Every thread
// of the block calls it, with sC complete and sh.need, sh.any cleared, both visible.
//
// The sums over an element's points are taken by every lane from LDS (one barrier), and the
// detector's transform of the first variable is shared out over the four lanes of a point:
// serial loops of one lane per element would leave the rest idle through some fifty dependent
// LDS reads.
template <int PD, int M, int NQ>
__device__ __forceinline__ bool post_tri(const KParams& P, double (&c)[M], double (&a)[M],
                                         double (&sC)[TriShape<PD>::EPB][4][M][TriShape<PD>::NPT],
                                         const double* sLf, TriPostShared<PD, M>& sh, const int e, const int le,
                                         const int rem, const bool active, const double dt, const TriPost& post) {
  using Sh = TriShape<PD>;
  constexpr int NPT = Sh::NPT, NF = Sh::NF, TPE = Sh::TPE;
  const int slot = rem >> 2, s = rem & 3;
  const bool pt = active && slot < NPT;
  const bool fp = active && slot < NF;
  bool filtered = false;
  if (post.filter) {
    for (int i = threadIdx.x; i < M * NPT; i += blockDim.x) {
      const double f = P.tab.filt[i];
      sh.lam[i] = P.filter == FRSG_FILTER_EXP ? exp(-P.alpha * dt * f) : f;
    }
    double vi[NPT];  // row `slot` of V^-1
#pragma unroll
    for (int l = 0; l < NPT; ++l) vi[l] = pt ? P.tri_Vinv[slot * NPT + l] : 0.0;
    // detector: energy of the outer shell over the total, first variable; lane s of a point
    // takes the chaos modes s, s + 4, ...
    if (P.sensor == FRSG_SENSOR_DETECTOR) {
      double num = 0.0, den = 0.0;
      if (pt) {
#pragma unroll
        for (int k0 = 0; k0 < M; k0 += 4) {
          const int k = k0 + s;
          if (k < M) {
            double t = 0.0;
#pragma unroll
            for (int l = 0; l < NPT; ++l) t += vi[l] * sC[le][0][k][l];
            const double e2 = t * t;
            num += e2 * P.tab.shell[k * NPT + slot];
            den += e2;
          }
        }
      }
      double N4[4], D4[4];
      quad_gather(num, N4);
      quad_gather(den, D4);
      if (pt && s == 0) {
        sh.num[le][slot] = (N4[0] + N4[1]) + (N4[2] + N4[3]);
        sh.den[le][slot] = (D4[0] + D4[1]) + (D4[2] + D4[3]);
      }
    }
    __syncthreads();
    bool flag = P.sensor != FRSG_SENSOR_DETECTOR;
    if (P.sensor == FRSG_SENSOR_DETECTOR) {
      double n = 0.0, d = 0.0;
#pragma unroll
      for (int i = 0; i < NPT; ++i) {
        n += sh.num[le][i];
        d += sh.den[le][i];
      }
      flag = d > 0.0 && n / d > P.sensor_thr;
    }
    filtered = active && flag;
    if (active && rem == 0 && post.flag_filt) post.flag_filt[e] = filtered ? 1 : 0;
    if (__syncthreads_or(filtered)) {
      // u_j <- sum_m V[j][m] (lambda_km (V^-1 u)_m), the damped modes staged in sC
      double um[M];
#pragma unroll
      for (int k = 0; k < M; ++k) {
        double acc = 0.0;
        if (filtered && pt) {
#pragma unroll
          for (int l = 0; l < NPT; ++l) acc += vi[l] * sC[le][s][k][l];
        }
        um[k] = acc;
      }
      __syncthreads();
      if (filtered && pt) {
#pragma unroll
        for (int k = 0; k < M; ++k) sC[le][s][k][slot] = um[k] * sh.lam[k * NPT + slot];
      }
      __syncthreads();
      if (filtered && pt) {
#pragma unroll
        for (int l = 0; l < NPT; ++l) vi[l] = P.tri_V[slot * NPT + l];
#pragma unroll
        for (int k = 0; k < M; ++k) {
          double acc = 0.0;
#pragma unroll
          for (int m = 0; m < NPT; ++m) acc += vi[m] * sC[le][s][k][m];
          c[k] = acc;
        }
      }
      __syncthreads();
      if (filtered && pt) {
#pragma unroll
        for (int k = 0; k < M; ++k) sC[le][s][k][slot] = c[k];
      }
      __syncthreads();
    }
  }
  // flux-point lanes: all modes interpolated to their flux point
  auto flux_traces = [&]() {
    double l[NPT];
#pragma unroll
    for (int j = 0; j < NPT; ++j) l[j] = sLf[(fp ? slot : 0) * NPT + j];
#pragma unroll
    for (int k = 0; k < M; ++k) {
      double acc = 0.0;
#pragma unroll
      for (int j = 0; j < NPT; ++j) acc += l[j] * sC[le][s][k][j];
      a[k] = acc;
    }
  };
  if (fp) flux_traces();
  if (!post.limit) return filtered;
  // element means of the four variables: lane s takes its own
  double ub[4];
  {
    double acc = 0.0;
#pragma unroll
    for (int j = 0; j < NPT; ++j) acc += sC[le][s][0][j] * P.tab.swts[j];
    quad_gather(acc, ub);
  }
  const double pb = (P.gamma - 1.0) * (ub[3] - 0.5 * (ub[1] * ub[1] + ub[2] * ub[2]) / ub[0]);
  const bool real = ub[0] > 0.0 && pb > 0.0 && isfinite(ub[0]) && isfinite(ub[1]) && isfinite(ub[2]) &&
                    isfinite(ub[3]);
  const double eps = fmin(1e-8, fmin(ub[0], pb));
  // rigorous bounds at the solution point and the flux point of this lane
  auto bound_ok = [&](const double* coef, bool on) {
    double mn = coef[0], vr = 0.0;
#pragma unroll
    for (int k = 1; k < M; ++k) vr += fabs(coef[k]) * P.tab.cmax[k];
    double MN[4], VR[4];
    quad_gather(mn, MN);
    quad_gather(vr, VR);
    if (!on) return true;
    const double rlo = MN[0] - VR[0];
    const double tol_r = 1e-10 * (fabs(MN[0]) + VR[0]);
    if (!(rlo > eps + tol_r)) return false;
    double m2 = 0.0;
#pragma unroll
    for (int v = 1; v < 3; ++v) {
      const double mx = fabs(MN[v]) + VR[v];
      m2 += mx * mx;
    }
    const double ke = 0.5 * m2 / rlo;
    const double elo = MN[3] - VR[3];
    const double plo = (P.gamma - 1.0) * (elo - ke);
    const double tol_p = 1e-10 * (P.gamma - 1.0) * (fabs(MN[3]) + VR[3] + ke);
    return plo > eps + tol_p;
  };
  const bool ok_sp = bound_ok(c, pt && real);
  const bool ok_fp = bound_ok(a, fp && real);
  if (active && real && !(ok_sp && ok_fp)) {
    sh.need[le] = 1;
    sh.any = 1;
  }
  if (active && !real && slot == 0 && s == 0) atomicOr(P.status, kStatusNotRealizable);
  __syncthreads();
  bool act = false;
  if (sh.any) {
    const bool need = active && real && sh.need[le];
    // node-by-node minima of density and pressure over solution and flux points
    double rmin = INFINITY, pmin = INFINITY;
#pragma unroll 1
    for (int q = 0; q < NQ; ++q) {
      double vs = 0.0, vf = 0.0;
#pragma unroll
      for (int k = 0; k < M; ++k) {
        const double ph = P.tab.PhiT[q * M + k];
        vs += ph * c[k];
        vf += ph * a[k];
      }
      double Us[4], Uf[4];
      quad_gather(vs, Us);
      quad_gather(vf, Uf);
      if (need && pt) {
        rmin = fmin(rmin, Us[0]);
        pmin = fmin(pmin, (P.gamma - 1.0) * (Us[3] - 0.5 * (Us[1] * Us[1] + Us[2] * Us[2]) / Us[0]));
      }
      if (need && fp) {
        rmin = fmin(rmin, Uf[0]);
        pmin = fmin(pmin, (P.gamma - 1.0) * (Uf[3] - 0.5 * (Uf[1] * Uf[1] + Uf[2] * Uf[2]) / Uf[0]));
      }
    }
    // minimum over an element's points, by every lane (the four lanes of a point hold the same)
    auto elem_min = [&](int row, double x) {
      for (int i = 0; i < TPE; i += 4) x = fmin(x, sh.mn[le][row][i]);
      return x;
    };
    if (active) {
      sh.mn[le][0][rem] = rmin;
      sh.mn[le][1][rem] = pmin;
    }
    __syncthreads();
    const double Rmin = elem_min(0, INFINITY), Pmin = elem_min(1, INFINITY);
    act = need && fmin(Rmin, Pmin) < eps;
    const double beta1 = (Rmin >= eps) ? 1.0 : (ub[0] - eps) / (ub[0] - Rmin);
    // beta2: smallest root over the points whose pressure stays below eps after beta1
    double bmin = 1.0;
#pragma unroll 1
    for (int q = 0; q < NQ; ++q) {
      double vs = 0.0, vf = 0.0;
#pragma unroll
      for (int k = 0; k < M; ++k) {
        const double ph = P.tab.PhiT[q * M + k];
        vs += ph * c[k];
        vf += ph * a[k];
      }
      double Us[4], Uf[4];
      quad_gather(vs, Us);
      quad_gather(vf, Uf);
      if (act && pt) {
        Us[0] = beta1 * (Us[0] - ub[0]) + ub[0];
        if ((P.gamma - 1.0) * (Us[3] - 0.5 * (Us[1] * Us[1] + Us[2] * Us[2]) / Us[0]) < eps)
          bmin = fmin(bmin, pressure_root<kEuler2>(ub, Us, eps, P.gamma));
      }
      if (act && fp) {
        Uf[0] = beta1 * (Uf[0] - ub[0]) + ub[0];
        if ((P.gamma - 1.0) * (Uf[3] - 0.5 * (Uf[1] * Uf[1] + Uf[2] * Uf[2]) / Uf[0]) < eps)
          bmin = fmin(bmin, pressure_root<kEuler2>(ub, Uf, eps, P.gamma));
      }
    }
    __syncthreads();
    if (active) sh.mn[le][0][rem] = bmin;
    __syncthreads();
    const double beta2 = elem_min(0, 1.0);
    // no lane reads sC past the last barrier: rewrite it in place
    if (act && pt) {
#pragma unroll
      for (int k = 0; k < M; ++k) {
        const double m0 = (k == 0) ? 1.0 : 0.0;
        double v = c[k];
        if (s == 0) v = beta1 * (v - ub[0] * m0) + ub[0] * m0;
        v = beta2 * (v - pick4(ub, s) * m0) + pick4(ub, s) * m0;
        c[k] = v;
        sC[le][s][k][slot] = v;
      }
    }
    __syncthreads();
    if (act && fp) flux_traces();
  }
  if (active && rem == 0 && post.flag_lim) post.flag_lim[e] = act ? 1 : 0;
  return filtered || act;
}

// A block holds four elements, and a group of four random nodes passes through four layouts:
//   A  lane (point, variable s): the chaos expansion of variable s at the point (its
//      coefficients stay in registers) for the four nodes; then, as lane (point, node), the
//      contravariant flux of all four variables;
//   B  lane (element, node, variable), each wave one group of rows: own traces and flux
//      divergence.  A row's coefficients are the same for the whole wave, so they are scalar
//      operands and a lane reads each nodal value of its column once;
//   I  lane (flux point, node): the interactive flux of all four variables, once per point;
//   C  as B: the correction's lifting, added to the divergence kept in registers;
//   D  as A: projection of the residual of variable s onto the chaos.
// The element operators take 42 x 10 products per node and variable at p = 3; with lanes on
// points (the layout of A throughout) every product needs its own table and nodal value from
// LDS, and the LDS rate, not the arithmetic, bounds the stage.  The last group repeats the last
// node, unprojected.
//
// The flux divergence uses Dr~ = Dr - lift (nr L), Ds~ likewise (nr, ns the reference normals):
// the interpolated flux at the faces, which the correction subtracts, folded into the
// derivative, so that the correction lifts the interactive flux alone.
//
// Three blocks' worth of waves per SIMD need at most 168 registers, for which the lane's place,
// the geometry and the tables are read or computed anew where they are used, the divergence is
// parked in LDS over I, and u of the combination arrives in the registers of the neighbour's
// traces once the last group has expanded them.
//
// Measured at 16,384 triangles, p = 3, 15 modes, 25 nodes: 227 us per stage (423 us with lanes
// on points throughout and one node at a time).  It moves 0.43 GB, 79 us at the rate of a large
// copy, and issues 82 us of vector instructions; the rest is LDS and waits at the block's
// start and end.  Four blocks fit a compute unit by LDS (40 KB).
template <int PD, int M, int NQ>
__global__ void __launch_bounds__(TriShape<PD>::NT, 3)
    k_stage_tri(KParams P, const double* __restrict__ in, const double* u, double* out, double cu, double cw, int rhs_only,
                const double* __restrict__ Tm, double* __restrict__ Tm_out, TriPost post, TriDt tdt) {
  using Sh = TriShape<PD>;
  constexpr int NPT = Sh::NPT, NFP = Sh::NFP, NF = Sh::NF, EPB = Sh::EPB, NT = Sh::NT;
  constexpr int RG = Sh::RG, RT = Sh::RT, RD = Sh::RD;
  static_assert(NPT <= NF && EPB * 16 == 64, "layouts of the kernel");
  struct Quad {
    double v[4];
  };
  struct alignas(16) Pair {
    double v[2];
  };
  // The nodal arrays of the loop, [element][point][node] quads of the four variables.  A point's
  // row is half of the 64 banks: the number of rows is odd so that two elements' rows for the
  // same point fall into different halves, the node's place in a row is rotated by point / 2 so
  // that eight neighbouring points cover all banks, and the quad's halves are swapped for every
  // other pair of points so that 16-byte accesses do too.  kT holds the own traces, then the
  // interactive fluxes, kU the nodal values, then the flux divergence and the residual.
  constexpr int ROWS = (RG * RT > RG * RD ? RG * RT : RG * RD) | 1, AR = EPB * ROWS * 16;
  constexpr int kU = 0, kFr = AR, kGs = 2 * AR, kT = 3 * AR, kX = 4 * AR;
  // place of (node i, variable v) in the row of point j
  auto place = [](int j, int i, int v) { return 4 * ((i + (j >> 1)) & 3) + (v ^ (j & 2)); };
  __shared__ union {
    alignas(16) double loop[5 * AR];
    double O[EPB][4][M][NPT];  // the output, for the filter, the limiter and its traces
  } lds;
  __shared__ double sLf[NF * NPT], sGeo[EPB * kTriGeo];
  __shared__ TriPostShared<PD, M> sh;
  const int E = P.E, e0 = tri_block() * EPB;
  if (e0 >= E) return;
  sh.clear();
  for (int i = threadIdx.x; i < NF * NPT; i += NT) sLf[i] = P.tri_Lf[i];
  {
    const int n = min(EPB, E - e0) * kTriGeo;
    for (int i = threadIdx.x; i < EPB * kTriGeo; i += NT) sGeo[i] = i < n ? P.tri_geo[(long)e0 * kTriGeo + i] : 0.0;
  }
  const TriLane<PD> at_start((int)threadIdx.x, e0, E);
  const int slot = at_start.slot, s = at_start.s, le = at_start.le, ec = at_start.ec, f = at_start.f, kk = at_start.kk;
  const bool pt = at_start.pt, fp = at_start.fp;
  const long EN = (long)E * NPT;

  const int nb = P.tri_nbr[(long)ec * 6 + f], g = nb < 0 ? 0 : P.tri_nbr[(long)ec * 6 + 3 + f];

  double uc[M], tn[M], acc[M];
  {
    const double* pu = in + at_start.state_at(E, M);
    const double* pn = Tm + tri_trace_index<PD, M>(nb < 0 ? ec : nb, g, 0, s, NFP - 1 - kk);
#pragma unroll
    for (int k = 0; k < M; ++k) {
      uc[k] = pu[k * EN];
      tn[k] = pn[k * 4 * NFP];
      acc[k] = 0.0;
    }
  }
  __syncthreads();
  double* const L = lds.loop;
  // row of the lane's point: its quad of node q0 + s, variable s at node q0 + i
  const int qb = (le * ROWS + slot) * 16, mine = qb + place(slot, s, 0) - (slot & 2), half = slot & 2;
  int w[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) w[i] = qb + place(slot, i, s);
  auto load_quad = [&](int array) {
    const Pair a = *(const Pair*)(L + array + mine + half), b = *(const Pair*)(L + array + mine + (half ^ 2));
    return Quad{{a.v[0], a.v[1], b.v[0], b.v[1]}};
  };
  auto store_quad = [&](int array, const Quad& x) {
    *(Pair*)(L + array + mine + half) = Pair{{x.v[0], x.v[1]}};
    *(Pair*)(L + array + mine + (half ^ 2)) = Pair{{x.v[2], x.v[3]}};
  };
  // the row group of this wave and the lane's column in it
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int cb = ((threadIdx.x & 63) >> 4) * ROWS * 16, cn = (threadIdx.x >> 2) & 3;
  int at[4];  // the column's double in the row of point j: 16 j + at[(j >> 1) & 3]
#pragma unroll
  for (int j = 0; j < 4; ++j) at[j] = cb + place(2 * j, cn, s);
  auto row_at = [&](int row) { return cb + 16 * row + place(row, cn, s); };
  using Rows = const __attribute__((address_space(4))) double*;
  Rows phi = (Rows)P.tab.PhiT, pwt = (Rows)P.tab.PWT;  // node-major
  const Rows rows = (Rows)(P.tri_rows + wave * (NPT * (RT + 2 * RD) + NF * RD));
  // the four lanes of a point write and read its row within one wave
  auto wave_sync = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };

  // the stages combine with the input itself (uc holds it) and read u only where cu != 0
  const bool need_u = (cu != 0.0);
#pragma unroll 1
  for (int q0 = 0; q0 < NQ; q0 += 4) {
    // read and computed anew for each group, to keep the registers free
    int gi = le * kTriGeo, tid = threadIdx.x;
    asm volatile("" : "+v"(gi), "+v"(tid));
    const double* geo = sGeo + gi;
    // A
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int q = min(q0 + i, NQ - 1);
      double v = 0.0, vr = 0.0;
#pragma unroll
      for (int k = 0; k < M; ++k) {
        const double ph = phi[q * M + k];
        v += ph * uc[k];
        vr += ph * tn[k];
      }
      if (pt) L[kU + w[i]] = v;
      if (fp) L[kX + w[i]] = vr;
    }
    if (q0 + 4 >= NQ && need_u) {  // the neighbour's traces are done with: u arrives meanwhile
      const TriLane<PD> me(tid, e0, E);
      const double* pu = u + me.state_at(E, M);
#pragma unroll
      for (int k = 0; k < M; ++k) tn[k] = pu[k * EN];
    }
    wave_sync();
    if (pt) {
      const Quad U = load_quad(kU);
      const double rx = geo[kGeoRx], ry = geo[kGeoRy], sx = geo[kGeoSx], sy = geo[kGeoSy];
      const double ir = rcp2(U.v[0]);
      const double vx = U.v[1] * ir, vy = U.v[2] * ir;
      const double p = (P.gamma - 1.0) * (U.v[3] - 0.5 * (U.v[1] * vx + U.v[2] * vy));
      const double vr = rx * vx + ry * vy, vs = sx * vx + sy * vy, H = U.v[3] + p;
      store_quad(kFr, Quad{{U.v[0] * vr, U.v[1] * vr + rx * p, U.v[2] * vr + ry * p, H * vr}});
      store_quad(kGs, Quad{{U.v[0] * vs, U.v[1] * vs + sx * p, U.v[2] * vs + sy * p, H * vs}});
    }
    __syncthreads();
    // B
    double d[RD];
    // The tables are streamed: the part of step j is loaded when the products of step j - 2 are
    // done (without the order the compiler loads all of it first, and spills).
    Rows ro[2] = {rows, rows};
    auto in_order = [&](int j, auto& x) {
      Rows& part = ro[j & 1];
#pragma unroll
      for (auto& v : x) asm volatile("" : "+s"(part), "+v"(v));
    };
    {
      double T[RT];
#pragma unroll
      for (int r = 0; r < RT; ++r) T[r] = 0.0;
#pragma unroll
      for (int r = 0; r < RD; ++r) d[r] = 0.0;
#pragma unroll
      for (int j = 0; j < NPT; ++j) {
        const Rows c = ro[j & 1] + j * (RT + 2 * RD);
        const int x = 16 * j + at[(j >> 1) & 3];
        const double U = L[kU + x], Fr = L[kFr + x], Gs = L[kGs + x];
#pragma unroll
        for (int r = 0; r < RT; ++r) T[r] += c[r] * U;
#pragma unroll
        for (int r = 0; r < RD; ++r) {
          d[r] += c[RT + r] * Fr;
          d[r] += c[RT + RD + r] * Gs;
        }
        in_order(j, T);
        in_order(j, d);
      }
#pragma unroll
      for (int r = 0; r < RT; ++r) L[kT + row_at(wave * RT + r)] = T[r];
    }
    __syncthreads();
    // I
#pragma unroll
    for (int r = 0; r < RD; ++r) L[kU + row_at(wave * RD + r)] = d[r];  // parked, to free registers
    if (fp) {
      const double fnx = geo[kGeoN0 + 2 * f], fny = geo[kGeoN0 + 2 * f + 1], fsc = geo[kGeoSc0 + f];
      const Quad Lt = load_quad(kT);
      Quad Rt = load_quad(kX);
      if (nb < 0) ghost_n(P, -1 - nb, Lt.v, fnx, fny, Rt.v);  // domain boundary: the ghost state
      Quad Fs;
      interactive_n(P.flux, Lt.v, Rt.v, fnx, fny, P.gamma, Fs.v);
#pragma unroll
      for (int t = 0; t < 4; ++t) Fs.v[t] *= fsc;
      store_quad(kT, Fs);
    }
    __syncthreads();
    // C
#pragma unroll
    for (int r = 0; r < RD; ++r) d[r] = L[kU + row_at(wave * RD + r)];
#pragma unroll
    for (int m = 0; m < NF; ++m) {
      const Rows c = ro[(m >> 1) & 1] + NPT * (RT + 2 * RD) + m * RD;
      const double J = L[kT + 16 * m + at[(m >> 1) & 3]];
#pragma unroll
      for (int r = 0; r < RD; ++r) d[r] += c[r] * J;
      if (m & 1) in_order(m >> 1, d);
    }
#pragma unroll
    for (int r = 0; r < RD; ++r) L[kU + row_at(wave * RD + r)] = d[r];
    __syncthreads();
    // D
    if (pt) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (q0 + i < NQ) {
          const double Rq = -L[kU + w[i]];
#pragma unroll
          for (int k = 0; k < M; ++k) acc[k] += pwt[(q0 + i) * M + k] * Rq;
        }
      }
    }
    wave_sync();  // the rows are read before the next group's writes
  }
  const bool do_post = post.filter || post.limit;
  // the lane's place anew, so that it need not be kept through the loop
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const TriLane<PD> me(tid, e0, E);
  // the time step: from the CFL maximum (first stage of a CFL step; the first block publishes
  // it), or as an earlier launch left it
  double dt = 0.0;
  if (!rhs_only) {
    if (tdt.from_lam) {
      dt = P.cfl / (P.np1 * __longlong_as_double((long long)*P.lam_bits));
      if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (!(dt > 0.0) || !isfinite(dt)) atomicOr(P.status, kStatusNonFinite);
        *P.dt = dt;
        if (tdt.dt_used) *tdt.dt_used = dt;
      }
    } else {
      dt = *P.dt;
      if (blockIdx.x == 0 && threadIdx.x == 0 && tdt.dt_used) *tdt.dt_used = dt;
    }
  }

  __syncthreads();  // the loop's LDS is free
  const long mine_at = me.state_at(E, M);
  if (me.pt) {
    double* po = out + mine_at;
#pragma unroll
    for (int k = 0; k < M; ++k) {
      const double uv = need_u ? tn[k] : 0.0;
      const double o = rhs_only ? acc[k] : cu * uv + cw * (uc[k] + dt * acc[k]);
      acc[k] = o;
      if (!rhs_only) lds.O[me.le][me.s][k][me.slot] = o;
      if (!do_post) po[k * EN] = o;
    }
  }
  if (!do_post && !Tm_out) return;
  __syncthreads();
  // the limiter after the stage, or the end-of-step filter and limiter, on the output, and the
  // modal traces of the final output at the flux points
  double tr[M];
  post_tri<PD, M, NQ>(P, acc, tr, lds.O, sLf, sh, me.e, me.le, me.rem, me.active, dt, post);
  if (do_post && me.pt) {
    double* po = out + mine_at;
#pragma unroll
    for (int k = 0; k < M; ++k) po[k * EN] = acc[k];
  }
  if (Tm_out && me.fp) {
    double* pm = Tm_out + tri_trace_index<PD, M>(me.e, me.f, 0, me.s, me.kk);
#pragma unroll
    for (int k = 0; k < M; ++k) pm[k * 4 * NFP] = tr[k];
  }
}

// CFL maximum of a modal state: (|v| + c) / d_e over solution points and nodes
__global__ void __launch_bounds__(256) k_cfl_tri_modal(KParams P, const double* __restrict__ u) {
  __shared__ double sm[256];
  const int np = P.nsp, E = P.E, M = P.M, Nq = P.Nq;
  const long EN = (long)E * np;
  const long t = blockIdx.x * 256l + threadIdx.x;
  double rate = 0.0;
  if (t < EN) {
    const int e = (int)(t / np);
    const double din = P.tri_geo[(long)e * kTriGeo + kGeoDin];
    for (int q = 0; q < Nq; ++q) {
      double U[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        double v = 0.0;
        for (int k = 0; k < M; ++k) v += P.tab.Phi[k * Nq + q] * u[((long)s * M + k) * EN + t];
        U[s] = v;
      }
      const double p = euler2_p(U, P.gamma);
      double r = (sqrt(U[1] * U[1] + U[2] * U[2]) / U[0] + sqrt(P.gamma * p / U[0])) / din;
      if (!(r == r)) r = __longlong_as_double(0x7ff0000000000000ll);
      rate = fmax(rate, r);
    }
  }
  sm[threadIdx.x] = rate;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) sm[threadIdx.x] = fmax(sm[threadIdx.x], sm[threadIdx.x + o]);
    __syncthreads();
  }
  if (threadIdx.x == 0) atomicMax(P.lam_bits, (unsigned long long)__double_as_longlong(sm[0]));
}

// the same for the (M, N_q) pairs of the fused stage: the thread's coefficients stay in registers
template <int M, int NQ>
__global__ void __launch_bounds__(256) k_cfl_tri_mq(KParams P, const double* __restrict__ u) {
  __shared__ double sm[256];
  const int np = P.nsp;
  const long EN = (long)P.E * np;
  const long t = blockIdx.x * 256l + threadIdx.x;
  double rate = 0.0;
  if (t < EN) {
    const double din = P.tri_geo[(t / np) * kTriGeo + kGeoDin];
    double c[4][M];
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int k = 0; k < M; ++k) c[s][k] = u[((long)s * M + k) * EN + t];
    for (int q = 0; q < NQ; ++q) {
      double U[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        double v = 0.0;
#pragma unroll
        for (int k = 0; k < M; ++k) v += P.tab.PhiT[q * M + k] * c[s][k];
        U[s] = v;
      }
      const double ir = rcp2(U[0]);
      const double m2 = U[1] * U[1] + U[2] * U[2];
      const double p = (P.gamma - 1.0) * (U[3] - 0.5 * m2 * ir);
      double r = sqrt(m2) * ir + sqrt(P.gamma * p * ir);
      if (!(r == r)) r = __longlong_as_double(0x7ff0000000000000ll);
      rate = fmax(rate, r);
    }
    rate = rate / din;
  }
  sm[threadIdx.x] = rate;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) sm[threadIdx.x] = fmax(sm[threadIdx.x], sm[threadIdx.x + o]);
    __syncthreads();
  }
  if (threadIdx.x == 0) atomicMax(P.lam_bits, (unsigned long long)__double_as_longlong(sm[0]));
}

// the filter and/or limiter in place on a state, as a pass of its own, and/or its modal traces
template <int PD, int M, int NQ>
__global__ void __launch_bounds__(TriShape<PD>::NT) k_limit_tri(KParams P, const double* in, double* out,
                                                                double* __restrict__ Tm_out, TriPost post) {
  using Sh = TriShape<PD>;
  constexpr int NPT = Sh::NPT, EPB = Sh::EPB;
  __shared__ double sC[EPB][4][M][NPT];
  __shared__ double sLf[Sh::NF * NPT];
  __shared__ TriPostShared<PD, M> sh;
  const int E = P.E, e0 = tri_block() * EPB;
  if (e0 >= E) return;
  sh.clear();
  for (int i = threadIdx.x; i < Sh::NF * NPT; i += Sh::NT) sLf[i] = P.tri_Lf[i];
  const TriLane<PD> me((int)threadIdx.x, e0, E);
  const long EN = (long)E * NPT, mine_at = me.state_at(E, M);
  double c[M];
#pragma unroll
  for (int k = 0; k < M; ++k) {
    c[k] = in[mine_at + k * EN];
    if (me.pt) sC[me.le][me.s][k][me.slot] = c[k];
  }
  __syncthreads();
  double tr[M];
  const bool changed = post_tri<PD, M, NQ>(P, c, tr, sC, sLf, sh, me.e, me.le, me.rem, me.active,
                                           post.filter ? *P.dt : 0.0, post);
  if (changed && me.pt) {
#pragma unroll
    for (int k = 0; k < M; ++k) out[mine_at + k * EN] = c[k];
  }
  if (Tm_out && me.fp) {
    double* pm = Tm_out + tri_trace_index<PD, M>(me.e, me.f, 0, me.s, me.kk);
#pragma unroll
    for (int k = 0; k < M; ++k) pm[k * 4 * Sh::NFP] = tr[k];
  }
}

template <int PD, int M, int NQ>
hipError_t go_stage_tri(const KParams& P, const double* in, const double* u, double* out, double cu, double cw,
                        int rhs_only, double* Tm, int traces_ready, double* Tm_out, const TriPost& post,
                        const TriDt& tdt, hipStream_t s) {
  using Sh = TriShape<PD>;
  if (!traces_ready) {
    hipLaunchKernelGGL((k_limit_tri<PD, M, NQ>), dim3(tri_grid(P.E)), dim3(Sh::NT), 0, s, P, in, (double*)nullptr, Tm,
                       TriPost());
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k_stage_tri<PD, M, NQ>), dim3(tri_grid(P.E)), dim3(Sh::NT), 0, s, P, in, u, out, cu, cw, rhs_only,
                     (const double*)Tm, Tm_out, post, tdt);
  return hipGetLastError();
}

template <int PD>
hipError_t dispatch_mq(const KParams& P, const double* in, const double* u, double* out, double cu, double cw,
                       int rhs_only, double* Tm, int traces_ready, double* Tm_out, const TriPost& post,
                       const TriDt& tdt, hipStream_t s) {
#define FRSG_TRI_MQ(MM, QQ)                                                                                 \
  if (P.M == MM && P.Nq == QQ)                                                                               \
    return go_stage_tri<PD, MM, QQ>(P, in, u, out, cu, cw, rhs_only, Tm, traces_ready, Tm_out, post, tdt, s);
  FRSG_TRI_MQ(15, 25) FRSG_TRI_MQ(10, 16) FRSG_TRI_MQ(6, 9) FRSG_TRI_MQ(5, 5) FRSG_TRI_MQ(3, 4)
#undef FRSG_TRI_MQ
  return hipErrorInvalidValue;
}

}  // namespace

template <int PD>
hipError_t dispatch_limit(const KParams& P, double* u, const TriPost& post, hipStream_t s) {
  using Sh = TriShape<PD>;
#define FRSG_TRI_LIM(MM, QQ)                                                                        \
  if (P.M == MM && P.Nq == QQ) {                                                                     \
    hipLaunchKernelGGL((k_limit_tri<PD, MM, QQ>), dim3(tri_grid(P.E)), dim3(Sh::NT), 0, s, P, u, u,      \
                       (double*)nullptr, post);                                                        \
    return hipGetLastError();                                                                        \
  }
  FRSG_TRI_LIM(15, 25) FRSG_TRI_LIM(10, 16) FRSG_TRI_LIM(6, 9) FRSG_TRI_LIM(5, 5) FRSG_TRI_LIM(3, 4)
#undef FRSG_TRI_LIM
  return hipErrorInvalidValue;
}

bool tri_fused_supported(const KParams& P) {
  if (P.eq != FRSG_EULER2D || P.nfp < 2 || P.nfp > 5) return false;
  const int mq[5][2] = {{15, 25}, {10, 16}, {6, 9}, {5, 5}, {3, 4}};
  for (auto& x : mq)
    if (P.M == x[0] && P.Nq == x[1]) return true;
  return false;
}

// one stage: out = cu u + cw (in + dt R(in)), or R(in) with rhs_only, the neighbours' traces
// of `in` from Tm (filled by a trace pass first unless traces_ready); with Tm_out the
// traces of `out` are written there for the next stage
hipError_t launch_stage_tri(const KParams& P, const double* in, const double* u, double* out, double cu, double cw,
                            int rhs_only, double* Tm, int traces_ready, double* Tm_out, hipStream_t s,
                            const TriPost& post, const TriDt& tdt) {
  if (!tri_fused_supported(P) || (post.filter && P.filter == FRSG_FILTER_LASSO) || (rhs_only && (post.filter || post.limit)))
    return hipErrorInvalidValue;
  switch (P.nfp - 1) {
    case 1: return dispatch_mq<1>(P, in, u, out, cu, cw, rhs_only, Tm, traces_ready, Tm_out, post, tdt, s);
    case 2: return dispatch_mq<2>(P, in, u, out, cu, cw, rhs_only, Tm, traces_ready, Tm_out, post, tdt, s);
    case 3: return dispatch_mq<3>(P, in, u, out, cu, cw, rhs_only, Tm, traces_ready, Tm_out, post, tdt, s);
    case 4: return dispatch_mq<4>(P, in, u, out, cu, cw, rhs_only, Tm, traces_ready, Tm_out, post, tdt, s);
    default: return hipErrorInvalidValue;
  }
}

// the sensor-gated filter and/or the limiter in place with the fused lane layout (the
// fused (p, M, N_q) set)
hipError_t launch_post_tri(const KParams& P, double* u, const TriPost& post, hipStream_t s) {
  if (!tri_fused_supported(P) || (post.filter && P.filter == FRSG_FILTER_LASSO)) return hipErrorInvalidValue;
  switch (P.nfp - 1) {
    case 1: return dispatch_limit<1>(P, u, post, s);
    case 2: return dispatch_limit<2>(P, u, post, s);
    case 3: return dispatch_limit<3>(P, u, post, s);
    case 4: return dispatch_limit<4>(P, u, post, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_limit_tri(const KParams& P, double* u, unsigned char* flags, hipStream_t s) {
  TriPost post;
  post.limit = 1;
  post.flag_lim = flags;
  return launch_post_tri(P, u, post, s);
}

hipError_t launch_cfl_tri_modal(const KParams& P, const double* u, hipStream_t s) {
  if (P.eq != FRSG_EULER2D) return hipErrorInvalidValue;
  const long n = (long)P.E * P.nsp;
#define FRSG_TRI_CFL(MM, QQ)                                                                    \
  if (P.M == MM && P.Nq == QQ) {                                                                 \
    hipLaunchKernelGGL((k_cfl_tri_mq<MM, QQ>), dim3(blocks(n)), dim3(256), 0, s, P, u);          \
    return hipGetLastError();                                                                    \
  }
  FRSG_TRI_CFL(15, 25) FRSG_TRI_CFL(10, 16) FRSG_TRI_CFL(6, 9) FRSG_TRI_CFL(5, 5) FRSG_TRI_CFL(3, 4)
#undef FRSG_TRI_CFL
  hipLaunchKernelGGL(k_cfl_tri_modal, dim3(blocks(n)), dim3(256), 0, s, P, u);
  return hipGetLastError();
}

}  // namespace frsg
