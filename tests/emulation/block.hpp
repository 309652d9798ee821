// One block of a kernel on the CPU: every lane is a fiber, and the caller says
// which wave runs next, so that single waves can be let far ahead of the others
// between two barriers. Device text included after this header sees the block's
// names (threadIdx, __syncthreads, __ballot, ...) and ordinary memory.
#pragma once
#include <ucontext.h>

#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <vector>

constexpr int kWave = 64;
struct Dim { unsigned x; };
static Dim threadIdx, blockDim;

struct Lane {
  ucontext_t ctx;
  std::vector<char> stack;
  int wait = 0;       // 0 runs, 1 at a wave exchange, 2 at a block barrier, 3 ended
  long long value = 0;
};
static std::vector<Lane> lanes;
static ucontext_t driver;
static int current;
static std::vector<long long> exchanged;  // per lane: the values of its wave's last exchange
static std::vector<long> barriers;         // per wave

static void pause_lane(int why) {
  const int me = current;
  lanes[me].wait = why;
  swapcontext(&lanes[me].ctx, &driver);
}
static int lane_id() { return current % kWave; }
static const long long *exchange(long long v) {
  lanes[current].value = v;
  pause_lane(1);
  return &exchanged[current / kWave * kWave];
}
[[maybe_unused]] static uint64_t __ballot(bool b) {
  const long long *v = exchange(b);
  uint64_t m = 0;
  for (int i = 0; i < kWave; ++i) m |= uint64_t(v[i] != 0) << i;
  return m;
}
template <class T> static T lane_read(T v, int src) { return T(exchange((long long)v)[src]); }
[[maybe_unused]] static unsigned lanes_below(uint64_t m) {
  return unsigned(__builtin_popcountll(m & ((1ull << lane_id()) - 1)));
}
[[maybe_unused]] static int __popcll(uint64_t m) { return __builtin_popcountll(m); }
[[maybe_unused]] static int __ffsll(long long m) { return __builtin_ffsll(m); }
template <class T, class U> static T atomicAdd(T *p, U v) {
  const T old = *p;
  *p += T(v);
  return old;
}
[[maybe_unused]] static double __shfl_xor(double v, int o, int) {
  long long x;
  std::memcpy(&x, &v, 8);
  x = exchange(x)[lane_id() ^ o];
  std::memcpy(&v, &x, 8);
  return v;
}
static void __syncthreads() { pause_lane(2); }
using std::min;
#define __device__
#define __forceinline__ inline

static std::function<void()> block_body;
static void entry() {
  block_body();
  pause_lane(3);
}

// Runs the block to its end; pick(waves that can run) names the next wave. A
// wave runs until all its lanes stand at a barrier or have ended. False if
// waves are left waiting for a barrier that the others never reach.
static bool run(int nw, const std::function<int(const std::vector<int> &)> &pick) {
  lanes = std::vector<Lane>(size_t(nw) * kWave);
  exchanged.assign(lanes.size(), 0);
  barriers.assign(nw, 0);
  blockDim.x = unsigned(lanes.size());
  for (Lane &l : lanes) {
    l.stack.resize(32 << 10);
    getcontext(&l.ctx);
    l.ctx.uc_stack.ss_sp = l.stack.data();
    l.ctx.uc_stack.ss_size = l.stack.size();
    l.ctx.uc_link = nullptr;
    makecontext(&l.ctx, entry, 0);
  }
  std::vector<int> at(nw, 0);
  for (;;) {
    std::vector<int> ready;
    for (int w = 0; w < nw; ++w)
      if (at[w] == 0) ready.push_back(w);
    if (ready.empty()) {
      // a barrier opens once every wave that has not ended stands at one
      bool some = false;
      for (int w = 0; w < nw; ++w)
        if (at[w] == 2) {
          at[w] = 0;
          ++barriers[w];
          some = true;
        }
      if (!some) return std::all_of(barriers.begin(), barriers.end(),
                                    [&](long b) { return b == barriers[0]; });
      for (Lane &l : lanes)
        if (l.wait == 2) l.wait = 0;
      continue;
    }
    const int w = pick(ready);
    while (at[w] == 0) {
      for (int i = 0; i < kWave; ++i) {
        current = w * kWave + i;
        threadIdx.x = unsigned(current);
        if (lanes[current].wait == 0) swapcontext(&driver, &lanes[current].ctx);
      }
      const int why = lanes[w * kWave].wait;
      for (int i = 0; i < kWave; ++i)
        if (lanes[w * kWave + i].wait != why) {
          std::printf("wave %d diverged at an exchange\n", w);
          std::exit(2);
        }
      if (why == 1)
        for (int i = 0; i < kWave; ++i) {
          exchanged[w * kWave + i] = lanes[w * kWave + i].value;
          lanes[w * kWave + i].wait = 0;
        }
      else
        at[w] = why;
    }
  }
}

// Schedules: waves in order, backwards, each wave first in turn, then random ones.
static int schedules(int nw) { return 2 + nw + 8; }
static std::function<int(const std::vector<int> &)> schedule(int s, int nw) {
  return [s, nw, seed = unsigned(s)](const std::vector<int> &ready) mutable {
    if (s == 0) return ready.front();
    if (s == 1) return ready.back();
    if (s < 2 + nw) {
      for (int w : ready)
        if (w == s - 2) return w;
      return ready.front();
    }
    seed = seed * 1664525u + 1013904223u;
    return ready[(seed >> 8) % ready.size()];
  };
}
