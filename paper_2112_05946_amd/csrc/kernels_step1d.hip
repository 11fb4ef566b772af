// Kernels and launchers of the one-launch 1D step (step1d.hpp): the windowed step, the
// steps of a small problem in one workgroup, and the CFL maximum of a state.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "step1d.hpp"

namespace frsg {
namespace {

using step1d::Args;

constexpr int kMaxThreads = 512;
constexpr int kMaxThreadsRes = 1024;
constexpr int kBlockCfl = 256;
constexpr int kMaxLam = 1024;           // per-workgroup maxima that a step reads by itself
constexpr size_t kMaxLds = 150 * 1024;  // of the compute unit's 160 KB

template <int EQ, int N, typename R, bool TAB>
__global__ void __launch_bounds__(kMaxThreads) k_step1d(KParams P, Args A) {
  extern __shared__ __attribute__((aligned(16))) double smem[];
  step1d::run<EQ, N, R, TAB, false>(P, A, smem);
}

// THREADS: 512 (up to 256 registers per lane) or 1024 (128)
template <int EQ, int N, int THREADS>
__global__ void __launch_bounds__(THREADS) k_steps1d_resident(KParams P, Args A) {
  extern __shared__ __attribute__((aligned(16))) double smem[];
  step1d::run<EQ, N, double, false, true>(P, A, smem);
}

// CFL maximum of a state, per workgroup into part[blockIdx.x]; with copy, the state also
// goes there (the step after it then reads the copy and writes the state).  A workgroup
// stages the coefficients of EB elements in LDS; thread (element, node)
template <int EQ, int N>
__global__ void __launch_bounds__(kBlockCfl) k_cfl1d_part(KParams P, const double* __restrict__ u, int EB, double* part,
                                                          double* copy) {
  constexpr int S = nstate<EQ>(), n = N;
  extern __shared__ __attribute__((aligned(16))) double sC[];  // [EB][S][M][n]
  __shared__ double sm[kBlockCfl / 64];
  const int E = P.E, M = P.M, Nq = P.Nq, tid = threadIdx.x, lane = tid & 63;
  const long EN = (long)E * n;
  const int e0 = blockIdx.x * EB, nloc = min(EB, E - e0);
  const int ncoef = S * M * n, span = nloc * n;
  for (int c = lane; c < span; c += 64) {
    const int le = c / n, j = c - le * n;
    const long at = (long)(e0 + le) * n + j;
#pragma unroll 4
    for (int sk = tid >> 6; sk < S * M; sk += kBlockCfl / 64) {
      const double v = u[(long)sk * EN + at];
      sC[le * ncoef + sk * n + j] = v;
      if (copy) copy[(long)sk * EN + at] = v;
    }
  }
  __syncthreads();
  const int le = tid / Nq, q = tid - le * Nq;
  double rate = 0.0;
  if (le < nloc) {
    const double* C = sC + le * ncoef;
    double V[S][N];
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int j = 0; j < n; ++j) V[s][j] = 0.0;
#pragma unroll 3
    for (int k = 0; k < M; ++k) {
      const double phi = P.tab.Phi[k * Nq + q];
#pragma unroll
      for (int s = 0; s < S; ++s)
#pragma unroll
        for (int j = 0; j < n; ++j) V[s][j] += C[(s * M + k) * n + j] * phi;
    }
#pragma unroll
    for (int j = 0; j < n; ++j) {
      double U[S];
#pragma unroll
      for (int s = 0; s < S; ++s) U[s] = V[s][j];
      double r = speed<EQ, 0>(U, P.adv, P.gamma);
      if (!(r == r)) r = __longlong_as_double(0x7ff0000000000000ll);  // NaN -> +inf, dt -> 0
      rate = fmax(rate, r);
    }
  }
  for (int o = 32; o > 0; o >>= 1) rate = fmax(rate, __shfl_xor(rate, o));
  if (lane == 0) sm[tid >> 6] = rate;
  __syncthreads();
  if (tid == 0) {
    double r = sm[0];
    for (int w = 1; w < kBlockCfl / 64; ++w) r = fmax(r, sm[w]);
    part[blockIdx.x] = r;
  }
}

// the maximum of many per-workgroup maxima
__global__ void __launch_bounds__(256) k_fold_max(const double* __restrict__ part, int n, double* out) {
  __shared__ double sm[4];
  double r = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) r = fmax(r, part[i]);
  for (int o = 32; o > 0; o >>= 1) r = fmax(r, __shfl_xor(r, o));
  if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = r;
  __syncthreads();
  if (threadIdx.x == 0) *out = fmax(fmax(sm[0], sm[1]), fmax(sm[2], sm[3]));
}

__global__ void __launch_bounds__(256) k_copy_state(const double* __restrict__ a, double* __restrict__ b, long n) {
  for (long i = blockIdx.x * 256l + threadIdx.x; i < n; i += gridDim.x * 256l) b[i] = a[i];
}

struct Plan {
  int EB = 0, W = 0, NqS = 0, threads = 0, grid = 0;
  size_t lds = 0;
};

// a system's projection and staging have use for every wave; a scalar problem's for four
int least_threads(const KParams& P) { return P.S > 1 ? kMaxThreads : 256; }

// stages kept: right-hand sides a tableau step holds beside the two states
Plan plan_of(const KParams& P, int nst, int nk) {
  Plan L;
  L.NqS = step1d::node_row(P.Nq);
  const int H = nst;
  // about one workgroup per compute unit: fewer elements only repeat more of the
  // neighbours' work, more leave compute units idle.  Beyond 16 elements only where a large
  // mesh has so few nodes that 16 would leave the workgroup's threads idle, and with two
  // workgroups per compute unit left, scalar four (Sod, 3 nodes, 49,152 elements, four steps:
  // 470 us with a launch per stage, 814 with 16 elements, 262 with 79).  12 to 14 nodes fill a
  // scalar problem's four waves with a few elements less (Burgers, 12 nodes, 16,384 elements:
  // 199 us with a launch per stage, 203 with 16 elements, 151 with 15)
  int EB = std::min(16, std::max(4, (P.E + 255) / 256));
  const int least = least_threads(P), wide = least / P.Nq - 2 * H;
  if (wide > 16) EB = std::max(EB, std::min(wide, P.E / (P.S > 1 ? 512 : 1024)));
  else if (P.S == 1 && wide >= 12 && P.E > 8192) EB = wide;
  for (; EB >= 4; --EB) {
    L.W = EB + 2 * H;
    const int need = (L.W * P.Nq + 63) / 64 * 64;
    L.lds = sizeof(double) * (size_t)step1d::lds_layout(P.S, P.M, P.np1, L.W, L.NqS, nk).total;
    if (need > kMaxThreads || L.lds > kMaxLds || L.W > 256) continue;
    L.threads = std::max(least, need);
    L.EB = EB;
    L.grid = (P.E + EB - 1) / EB;
    return L;
  }
  return Plan();
}

int cfl_eb(const KParams& P) {
  const int by_lds = (int)(60 * 1024 / (sizeof(double) * (size_t)P.S * P.M * P.np1));
  return std::min(kBlockCfl / P.Nq, by_lds);
}

template <typename K>
hipError_t allow_lds(K kernel, size_t bytes) {
  if (bytes <= 64 * 1024) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)bytes);
}

template <int EQ, int N, typename R, bool TAB>
hipError_t go_step(const KParams& P, const Args& A, const Plan& L, hipStream_t s) {
  const hipError_t e = allow_lds(&k_step1d<EQ, N, R, TAB>, L.lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_step1d<EQ, N, R, TAB>), dim3(L.grid), dim3(L.threads), L.lds, s, P, A);
  return hipGetLastError();
}

template <typename F>
hipError_t with_eq_n(const KParams& P, F&& f) {
  auto with_n = [&](auto eq) -> hipError_t {
    switch (P.np1) {
#define FRSG_N(NN) case NN: return f(eq, std::integral_constant<int, NN>{});
      FRSG_N(2) FRSG_N(3) FRSG_N(4) FRSG_N(5)
#undef FRSG_N
      default: return hipErrorInvalidValue;
    }
  };
  switch (P.eq) {
    case kAdvection: return with_n(std::integral_constant<int, kAdvection>{});
    case kBurgers: return with_n(std::integral_constant<int, kBurgers>{});
    case kEuler1: return with_n(std::integral_constant<int, kEuler1>{});
    default: return hipErrorInvalidValue;
  }
}

// Whether the step in one launch is the faster one.  With at most one workgroup per compute unit a
// step is a chain of latencies, and it always is (on each of 676 problems of 2048 elements or more).
// Beyond that the work counts: a workgroup computes EB + 2 (stages - 1), .. EB elements for EB, the stage
// kernel EB' + 2 per launch for EB' = 256 / N_q - 2.  Over 3 to 64 nodes and up to 49,152
// elements (figures: four steps, against a launch per stage) one launch loses
//  - on p = 4 scalar problems of more than 256 threads, whose registers leave one workgroup per
//    compute unit (Burgers, 40 nodes, RK4, 16,384 elements: 1379 us against 902); not with 16 or 32
//    and more nodes and 8 elements, where the stage kernel's own rows collide in LDS or hold few
//    elements (0.7 to 0.95 of its time), and not where its three passes over the state miss
//    the L2 caches (24 nodes, 49,152 elements: 979 against 1233);
//  - on FP32-mixed systems, which expand the state in both types, with few elements per workgroup
//    or an almost empty second round (Sod, 24 nodes, 4096 elements: 317 against 292);
//  - on four-stage steps of systems, whose stored right-hand sides leave room for few elements
//    (p = 4 Sod, RK4, 16,384 elements, five per workgroup: 1988 against 1277).
bool pays(const KParams& P, const Plan& L, int stages, bool tab) {
  if (L.grid <= 256) return true;
  const bool p4 = P.np1 == 5, few = L.EB >= 8 && (P.Nq % 16 == 0 || (p4 && P.Nq >= 32));
  if (P.S == 1)
    return !p4 || L.threads <= 256 || few || (P.eq == kAdvection && P.fp32) ||
           (!tab && L.EB >= 6 && sizeof(double) * (double)P.M * P.E * P.np1 >= 16e6);
  if (P.fp32) return few || (L.grid >= 512 && L.EB >= (P.np1 <= 3 ? 8 : 10));
  if (stages < 4) return few || !p4 || L.grid >= 512;
  return L.EB >= 10 || (L.EB >= 6 && P.Nq >= 32);
}

}  // namespace

// Steps of up to four stages of FR degree 1..4 (FP32-mixed: SSP-RK3 only) whose window of at
// least four elements fits a workgroup's threads and LDS; higher degrees (whose nodal values
// would spill) and larger node counts take one launch per stage
bool step1d_supported(const KParams& P, int stages, bool tab) {
  if (P.dim != 1 || P.bf16 || (P.fp32 && tab) || P.np1 < 2 || P.np1 > 5) return false;
  if (stages < 1 || stages > step1d::kMaxStages) return false;
  const Plan L = plan_of(P, stages, tab ? stages - 1 : 0);
  return L.EB > 0 && cfl_eb(P) >= 1 && pays(P, L, stages, tab);
}
// per-workgroup maxima of a step or of a CFL pass, at most
long step1d_partials(const KParams& P) { return std::max<long>((P.E + 3) / 4, cfl_eb(P) > 0 ? (P.E + cfl_eb(P) - 1) / cfl_eb(P) : 0) + 1; }
bool step1d_one_workgroup(const KParams& P, int stages, bool tab) {
  return plan_of(P, stages, tab ? stages - 1 : 0).grid == 1;
}

// the per-workgroup maxima part[0 .. n) as a step reads them: few as they are, many folded
// into part[n]
static hipError_t fold(double* part, int& n, const double*& at, hipStream_t s) {
  at = part;
  if (n <= kMaxLam) return hipSuccess;
  hipLaunchKernelGGL(k_fold_max, dim3(1), dim3(256), 0, s, part, n, part + n);
  at = part + n;
  n = 1;
  return hipGetLastError();
}

hipError_t launch_cfl1d_part(const KParams& P, const double* u, double* part, double* copy, Lam1d* lam, hipStream_t s) {
  const int EB = cfl_eb(P);
  if (EB < 1) return hipErrorInvalidValue;
  const size_t shmem = sizeof(double) * (size_t)EB * P.S * P.M * P.np1;
  const int grid = (P.E + EB - 1) / EB;
  const hipError_t e = with_eq_n(P, [&](auto eq, auto nn) -> hipError_t {
    hipLaunchKernelGGL((k_cfl1d_part<decltype(eq)::value, decltype(nn)::value>), dim3(grid), dim3(kBlockCfl), shmem, s, P,
                       u, EB, part, copy);
    return hipGetLastError();
  });
  if (e != hipSuccess) return e;
  lam->n = grid;
  return fold(part, lam->n, lam->at, s);
}

hipError_t launch_copy_state(const double* a, double* b, long n, hipStream_t s) {
  const unsigned grid = (unsigned)std::min<long>(2048, (n + 255) / 256);
  hipLaunchKernelGGL(k_copy_state, dim3(grid), dim3(256), 0, s, a, b, n);
  return hipGetLastError();
}

hipError_t launch_step1d(const KParams& P, const Step1D& T, Lam1d* lam_out, hipStream_t s) {
  const Plan L = plan_of(P, T.stages, T.tab ? T.stages - 1 : 0);
  if (L.EB == 0 || (T.in == T.out && L.grid > 1) || T.stages > step1d::kMaxStages) return hipErrorInvalidValue;
  Args A{};
  A.in = T.in, A.out = T.out, A.w1 = T.w1, A.w2 = T.w2, A.PWB = P.tab.PWB;
  A.EB = L.EB, A.H = T.stages, A.W = L.W, A.NqS = L.NqS, A.nst = T.stages;
  if (T.tab)
    for (int i = 0; i < T.stages; ++i)
      for (int j = 0; j <= i; ++j) A.a[i][j] = T.rows[i][j];
  A.limit = T.limit;
  if (T.flags) A.f0 = T.flags, A.f1 = T.flags + P.E, A.f2 = T.flags + 2l * P.E, A.f3 = T.flags + 3l * P.E;
  A.dt_source = T.dt > 0.0 ? 1 : 2;
  A.dt_fixed = T.dt > 0.0 ? T.dt : 0.0;
  A.lam_in = T.lam.at, A.nlam = T.lam.n, A.lam_out = T.lam_part, A.dt_used = T.dt_used;
  const hipError_t e = with_eq_n(P, [&](auto eq, auto nn) -> hipError_t {
    constexpr int EQ = decltype(eq)::value, N = decltype(nn)::value;
    if (P.fp32) return T.tab ? hipErrorInvalidValue : go_step<EQ, N, float, false>(P, A, L, s);
    return T.tab ? go_step<EQ, N, double, true>(P, A, L, s) : go_step<EQ, N, double, false>(P, A, L, s);
  });
  if (e != hipSuccess || !T.lam_part || !lam_out) return e;
  lam_out->n = L.grid;
  return fold(T.lam_part, lam_out->n, lam_out->at, s);
}

// the one-workgroup multi-step kernel: FP64 scalar equations of FR degree <= 3, every element
// and two more in 1024 (element, node) pairs (at 1024 threads a lane has 128 registers: the Euler
// and higher-degree instances would spill), and a stage's coefficients, traces and residuals (once
// each, unpadded) and the chaos tables within 64 KB.  That is a cap on the work of one compute
// unit, not on its LDS: the launch lays out at most 127 KB under it.  It lies about where a step of
// one workgroup takes as long as a window step (Burgers, 9 modes, 16 nodes: 12.1 us at 40
// elements, 14.4 at 56, against 13.8 at 57; p = 1, 3 nodes: 9.8 at 339, against 10.9 at 340).
constexpr int kMaxNRes = 4;
constexpr size_t kWorkRes = 64 * 1024;
static size_t resident_state_bytes(const KParams& P) { return sizeof(double) * (size_t)P.S * P.M * P.np1 * P.E; }
static size_t resident_work(const KParams& P) {
  const size_t nc = (size_t)P.S * P.M * P.np1, E = (size_t)P.E;
  return sizeof(double) * ((E + 2) * nc + (E + 2) * P.Nq * 2 * P.S + E * P.S * P.np1 * P.Nq + 2 * (size_t)P.M * P.Nq +
                           16 + 256);
}
bool fr1d_resident_fits(const KParams& P) {
  if (P.dim != 1 || P.fp32 || P.bf16 || P.eq == kEuler1 || P.np1 < 2 || P.np1 > kMaxNRes) return false;
  if ((long)(P.E + 2) * P.Nq > kMaxThreadsRes) return false;
  return resident_work(P) <= kWorkRes;
}
bool fr1d_resident_small(const KParams& P) {
  return fr1d_resident_fits(P) && resident_work(P) + 3 * resident_state_bytes(P) <= kWorkRes;
}

template <int EQ, int N, int THREADS>
static hipError_t go_resident(const KParams& P, const Args& A, int threads, size_t lds, hipStream_t s) {
  const hipError_t e = allow_lds(&k_steps1d_resident<EQ, N, THREADS>, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_steps1d_resident<EQ, N, THREADS>), dim3(1), dim3(threads), lds, s, P, A);
  return hipGetLastError();
}

hipError_t launch_steps1d_resident(const KParams& P, double* u, int nsteps, int limit, unsigned char* flags,
                                   double* dt_used, const Lam1d& lam_in, double* lam_out, hipStream_t s) {
  if (!fr1d_resident_fits(P)) return hipErrorInvalidValue;
  Args A{};
  A.in = u, A.out = u, A.PWB = P.tab.PWB;
  A.EB = P.E, A.H = 0, A.W = P.E;
  A.NqS = step1d::node_row(P.Nq);
  A.nst = 3, A.limit = limit, A.dt_source = 2;
  A.lam_in = lam_in.at, A.nlam = lam_in.n, A.lam_out = lam_out;
  A.nsteps = nsteps, A.flags = flags, A.dts = dt_used;
  const int threads = std::max(256, (A.W * P.Nq + 63) / 64 * 64);
  const bool small = threads <= kMaxThreads;
  const size_t lds = sizeof(double) * (size_t)step1d::lds_layout(P.S, P.M, P.np1, A.W, A.NqS, 0).total;
  if (threads > kMaxThreadsRes || lds > kMaxLds) return hipErrorInvalidValue;
  auto go = [&](auto eq) -> hipError_t {
    constexpr int EQ = decltype(eq)::value;
    switch (P.np1) {
#define FRSG_N(NN)                                                                        \
  case NN:                                                                                \
    return small ? go_resident<EQ, NN, kMaxThreads>(P, A, threads, lds, s)  \
                 : go_resident<EQ, NN, kMaxThreadsRes>(P, A, threads, lds, s);
      FRSG_N(2) FRSG_N(3) FRSG_N(4)
#undef FRSG_N
      default: return hipErrorInvalidValue;
    }
  };
  switch (P.eq) {
    case kAdvection: return go(std::integral_constant<int, kAdvection>{});
    case kBurgers: return go(std::integral_constant<int, kBurgers>{});
    default: return hipErrorInvalidValue;
  }
}

}  // namespace frsg
