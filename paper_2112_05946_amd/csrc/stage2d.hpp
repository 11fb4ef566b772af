// What the 2D Euler stage kernels share: arguments of a stage, the tile of elements a
// workgroup owns, exchange between the 16-lane rows of a wave, padded point weights.
#pragma once

#include <hip/hip_runtime.h>

#include "internal.hpp"
#include "quad_device.hpp"

namespace frsg {
namespace {

using namespace quad;

// ---------------------------------------------------------------------------
// arguments
// ---------------------------------------------------------------------------
struct StageArgs {
  double cu, cw;             // out = cu u + cw (in + dt R)
  int stage;                 // 0: right-hand side only; 1, 2: limited stage output; 3: end of step
  unsigned char* flag_lim;   // per element: limiter acted on the output (stages 1-3)
  unsigned char* flag_filt;  // per element: filter acted (stage 3)
  unsigned long long* lam_next;  // stage 3: CFL accumulator of the new state (may be null)
  const double* Dt;          // 4 x 4 modified derivative matrix
  const double* cmax;        // [M] max_q |Phi_k(z_q)|
  const double* tr_in;       // modal face traces of the input, or null: interpolate from the neighbours
  double* tr_out;            // modal face traces of the output (may be null)
  // Butcher-row form (tab) instead of cu u + cw (in + dt R): out = u + dt (sum_m ka[m] kk[m]
  // + ka_cur R) over the earlier stage right-hand sides with nonzero coefficients, in stage
  // order, R last (skipped when ka_cur is 0); R is also stored in k_out (may be null)
  int tab, nt;
  const double* kk[kRkMaxTerms];
  double ka[kRkMaxTerms];
  double ka_cur;
  double* k_out;
  int flag_or;               // limiter flags OR-ed into flag_lim (set only where it acts)
  unsigned char* flag_zero;  // flags cleared by this stage (may be null)
  StageDt sdt;
};

inline StageArgs stage_args(const FusedStage& S) {
  StageArgs A;
  A.cu = S.cu;
  A.cw = S.cw;
  A.stage = S.stage;
  A.flag_lim = S.flag_lim;
  A.flag_filt = S.flag_filt;
  A.lam_next = S.lam_next;
  A.Dt = S.Dt;
  A.cmax = S.cmax;
  A.tr_in = S.tr_in;
  A.tr_out = S.tr_out;
  A.tab = S.tab;
  A.nt = S.tab ? S.terms.n : 0;
  for (int t = 0; t < kRkMaxTerms; ++t) {
    A.kk[t] = t < A.nt ? S.terms.K[t] : nullptr;
    A.ka[t] = t < A.nt ? S.terms.a[t] : 0.0;
  }
  A.ka_cur = S.ka_cur;
  A.k_out = S.k_out;
  A.flag_or = S.flag_or;
  A.flag_zero = S.flag_zero;
  A.sdt = S.sdt;
  return A;
}

// (M, N_q) of the fused kernels
#define FRSG_FUSED_SIZES(X) X(15, 25) X(10, 16) X(6, 9) X(3, 4) X(5, 5)

constexpr int TX = 4, TY = 2;
constexpr int TE = TX * TY;          // elements per tile
constexpr int NHF = 2 * (TX + TY);   // element faces on the tile boundary
// modal face traces of one tile: per boundary face slot (x-lo rows, x-hi rows,
// y-lo columns, y-hi columns), variable, face point and mode
template <int M, int N>
constexpr int TRACE_PER_TILE = NHF * 4 * N * M;

// Exchange between the two 16-lane rows of each 32-lane half (v_permlane16_swap
// of a and b): afterwards b in row 0 holds row 1's a and a in row 1 holds row
// 0's b, while a in row 0 and b in row 1 keep their values.  Every lane of the
// wave must be active.
__device__ __forceinline__ void swap_rows_u32(unsigned& a, unsigned& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}
__device__ __forceinline__ void swap_rows(float& a, float& b) {
  unsigned x = __float_as_uint(a), y = __float_as_uint(b);
  swap_rows_u32(x, y);
  a = __uint_as_float(x);
  b = __uint_as_float(y);
}
__device__ __forceinline__ void swap_rows(double& a, double& b) {
  const unsigned long long x = (unsigned long long)__double_as_longlong(a);
  const unsigned long long y = (unsigned long long)__double_as_longlong(b);
  unsigned xl = (unsigned)x, xh = (unsigned)(x >> 32), yl = (unsigned)y, yh = (unsigned)(y >> 32);
  swap_rows_u32(xl, yl);
  swap_rows_u32(xh, yh);
  a = __longlong_as_double((long long)(((unsigned long long)xh << 32) | xl));
  b = __longlong_as_double((long long)(((unsigned long long)yh << 32) | yl));
}

// 4 x 4 transposition over the four 16-lane rows of a wave: afterwards v[s] in row i holds what
// v[i] held in row s.  Every lane of the wave must be active.
__device__ __forceinline__ void swap_halves(double& a, double& b) {
  const unsigned long long x = (unsigned long long)__double_as_longlong(a);
  const unsigned long long y = (unsigned long long)__double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  a = __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0]));
  b = __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1]));
}
__device__ __forceinline__ void transpose_rows(double (&v)[4]) {
  swap_rows(v[0], v[1]);
  swap_rows(v[2], v[3]);
  swap_halves(v[0], v[2]);
  swap_halves(v[1], v[3]);
}

// entry c of an N-vector of point weights, 0 on the padding of a 16-lane row (c >= N)
template <int N>
__device__ __forceinline__ double wpad(const double* w, int c) {
  return (N == NP || c < N) ? w[N == NP ? c : min(c, N - 1)] : 0.0;
}
// entry (r, c) of an N x N point matrix, 0 on the padding
template <int N>
__device__ __forceinline__ double mpad(const double* m, int r, int c) {
  if constexpr (N == NP) return m[r * NP + c];
  else return (r < N && c < N) ? m[min(r, N - 1) * N + min(c, N - 1)] : 0.0;
}
}  // namespace
}  // namespace frsg
