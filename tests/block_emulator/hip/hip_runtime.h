// Stand-in for the HIP runtime header under which a kernel source compiles as host code, for the
// block emulator (emulator.hpp): the language keywords, the types that the declarations name, and
// the intrinsics of the kernels that it runs.  A kernel is called as an ordinary function by the
// emulator; a launch is not (the launchers compile and launch nothing).
#pragma once

#include <cmath>
#include <cstdint>
#include <cstring>
#include <functional>
#include <string>
#include <type_traits>
#include <vector>

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ static
// register pins (asm volatile("" : ...)) have no effect on values
#define asm
#define volatile(...)

using hipStream_t = void*;
using hipEvent_t = void*;
using hipError_t = int;
constexpr hipError_t hipSuccess = 0, hipErrorInvalidValue = 1;
inline hipError_t hipGetLastError() { return hipSuccess; }
struct dim3 {
  unsigned x, y, z;
  dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
#define hipLaunchKernelGGL(...) ((void)0)

namespace emu {
void block_barrier();            // every thread of the block
int block_or(int v);             // ... and the OR over them
int wave_read(int v, int lane);  // the value of a lane of the wave; every lane of the wave calls it
int lane();
}  // namespace emu
extern thread_local dim3 threadIdx, blockIdx, blockDim, gridDim;

inline void __syncthreads() { emu::block_barrier(); }
inline int __syncthreads_or(int v) { return emu::block_or(v); }
inline int mov_quad_perm(int v, int ctrl) {  // the quad permutations of a DPP move
  const int l = emu::lane();
  return emu::wave_read(v, (l & ~3) | ((ctrl >> (2 * (l & 3))) & 3));
}
#define __builtin_amdgcn_mov_dpp(v, ctrl, rows, banks, bound) mov_quad_perm(v, ctrl)
#define __builtin_amdgcn_rcp(x) (1.0 / (x))
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_fence(order, scope) ((void)0)
// lanes exchange through LDS between two of these without a block barrier
#define __builtin_amdgcn_wave_barrier() ((void)emu::wave_read(0, 0))

template <typename A, typename B>
B as_bits(A a) {
  static_assert(sizeof(A) == sizeof(B), "");
  B b;
  std::memcpy(&b, &a, sizeof b);
  return b;
}
inline long long __double_as_longlong(double x) { return as_bits<double, long long>(x); }
inline double __longlong_as_double(long long x) { return as_bits<long long, double>(x); }
inline unsigned atomicOr(unsigned* p, unsigned v) { const unsigned o = *p; *p |= v; return o; }
inline unsigned long long atomicMax(unsigned long long* p, unsigned long long v) {
  const unsigned long long o = *p;
  if (v > o) *p = v;
  return o;
}
inline int min(int a, int b) { return a < b ? a : b; }
using std::fabs;
using std::fma;
using std::fmax;
using std::fmin;
using std::isfinite;
using std::sqrt;
