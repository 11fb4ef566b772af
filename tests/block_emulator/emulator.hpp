// Runs one workgroup of a kernel on the CPU, its threads as fibers, the waves in a chosen order: a
// wave runs up to the next block barrier before the next one in the order starts.  The hardware
// may take any order, so a kernel whose results depend on it lacks a barrier.
#pragma once

#include <ucontext.h>

#include <cstdio>
#include <cstdlib>
#include <functional>
#include <vector>

#include <hip/hip_runtime.h>

thread_local dim3 threadIdx, blockIdx, blockDim, gridDim;

namespace emu {

struct Fiber {
  ucontext_t ctx;
  std::vector<char> stack;
  enum { kRun, kWave, kBlock, kDone } at = kRun;
  int value = 0;   // handed in at a wave operation or a block OR
};
inline std::vector<Fiber> g_fibers;
inline ucontext_t g_sched;
inline int g_cur = 0, g_or = 0;
inline std::function<void()> g_body;
inline std::vector<int> g_wave;  // values of the wave operation in hand, by thread

inline int lane() { return g_cur & 63; }
inline void yield(int at, int v) {
  Fiber& f = g_fibers[g_cur];
  f.at = static_cast<decltype(f.at)>(at);
  f.value = v;
  swapcontext(&f.ctx, &g_sched);
}
inline void block_barrier() { yield(Fiber::kBlock, 0); }
inline int block_or(int v) {
  yield(Fiber::kBlock, v);
  return g_or;
}
inline int wave_read(int v, int from) {
  yield(Fiber::kWave, v);
  return g_wave[(g_cur & ~63) + from];
}
inline void enter() {
  g_body();
  g_fibers[g_cur].at = Fiber::kDone;
  swapcontext(&g_fibers[g_cur].ctx, &g_sched);
}

// one block of `threads` threads; order: the waves, first to last
inline void run_block(int threads, const std::vector<int>& order, std::function<void()> body) {
  g_body = std::move(body);
  g_fibers = std::vector<Fiber>(threads);
  g_wave.assign(threads, 0);
  blockDim = dim3(threads);
  for (int t = 0; t < threads; ++t) {
    Fiber& f = g_fibers[t];
    f.stack.resize(256 * 1024);
    getcontext(&f.ctx);
    f.ctx.uc_stack.ss_sp = f.stack.data();
    f.ctx.uc_stack.ss_size = f.stack.size();
    f.ctx.uc_link = nullptr;
    makecontext(&f.ctx, enter, 0);
  }
  for (bool live = true; live;) {
    for (int w : order) {
      for (;;) {  // the wave up to the block barrier: all lanes to the next meeting point, again and again
        int at[4] = {0, 0, 0, 0};
        for (int t = 64 * w; t < 64 * w + 64; ++t) {
          g_cur = t;
          threadIdx = dim3(t);
          if (g_fibers[t].at == Fiber::kRun) swapcontext(&g_sched, &g_fibers[t].ctx);
          ++at[g_fibers[t].at];
        }
        if (at[Fiber::kWave] == 0) break;
        if (at[Fiber::kWave] != 64) {
          std::fprintf(stderr, "wave %d: %d lanes at a wave operation\n", w, at[Fiber::kWave]);
          std::exit(2);
        }
        for (int t = 64 * w; t < 64 * w + 64; ++t) {
          g_wave[t] = g_fibers[t].value;
          g_fibers[t].at = Fiber::kRun;
        }
      }
    }
    int barrier = 0, done = 0;
    g_or = 0;
    for (Fiber& f : g_fibers) {
      barrier += f.at == Fiber::kBlock;
      done += f.at == Fiber::kDone;
      if (f.at == Fiber::kBlock) g_or |= f.value;
    }
    if (barrier + done != threads || (barrier && done)) {
      std::fprintf(stderr, "%d threads at a block barrier, %d done, of %d\n", barrier, done, threads);
      std::exit(2);
    }
    for (Fiber& f : g_fibers)
      if (f.at == Fiber::kBlock) f.at = Fiber::kRun;
    live = barrier != 0;
  }
}

}  // namespace emu
