// One block of a kernel on the CPU: every lane is a fiber, and the driver says
// which wave runs next. Runs the append step of the bottom-up normal visit (its
// text comes from the sources: append.inc and step.inc) under schedules in
// which one wave is let far ahead of the others between two barriers.
//   append_step WAVES CAP STEPS DENSITY
#include <ucontext.h>

#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
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
static uint64_t __ballot(bool b) {
  const long long *v = exchange(b);
  uint64_t m = 0;
  for (int i = 0; i < kWave; ++i) m |= uint64_t(v[i] != 0) << i;
  return m;
}
template <class T> static T lane_read(T v, int src) { return T(exchange((long long)v)[src]); }
static unsigned lanes_below(uint64_t m) {
  return unsigned(__builtin_popcountll(m & ((1ull << lane_id()) - 1)));
}
static int __popcll(uint64_t m) { return __builtin_popcountll(m); }
static int __ffsll(long long m) { return __builtin_ffsll(m); }
template <class T, class U> static T atomicAdd(T *p, U v) {
  const T old = *p;
  *p += T(v);
  return old;
}
static void __syncthreads() { pause_lane(2); }
using std::min;
#define __device__
#define __forceinline__ inline
#include "append.inc"

static int g_cap, g_steps;
static double g_density;
static std::vector<int32_t> lds, out_q, out_c;
static unsigned long long tails;
static struct { int qcount, ccount; unsigned long long qbase, cbase; } S;

static bool draw(int step, int tid, int which) {
  uint64_t z = (uint64_t(step) * 1024 + tid) * 2 + which + 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return double((z ^ (z >> 31)) >> 11) / double(1ull << 53) < g_density;
}

static void body() {
  const int cap = g_cap;
  BlockAppend qa{lds.data(), &S.qcount, &S.qbase, cap, &tails, out_q.data()};
  BlockAppend ca{lds.data() + cap, &S.ccount, &S.cbase, cap, &tails, out_c.data(), 32};
  qa.init();
  ca.init();
  __syncthreads();
  for (int step = 0; step < g_steps; ++step) {
    const int tid = int(threadIdx.x), v = step * int(blockDim.x) + tid, pos = v;
    const bool won = draw(step, tid, 0), ok = true, visited = false;
    const bool found = !draw(step, tid, 1);
#include "step.inc"
  }
  flush_pair(qa, ca);
}

static void entry() {
  body();
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

int main(int argc, char **argv) {
  if (argc != 5) return 64;
  const int nw = std::atoi(argv[1]);
  g_cap = std::atoi(argv[2]);
  g_steps = std::atoi(argv[3]);
  g_density = std::atof(argv[4]);
  const int total = g_steps * nw * kWave;
  std::vector<int32_t> want_q, want_c;
  for (int step = 0; step < g_steps; ++step)
    for (int t = 0; t < nw * kWave; ++t) {
      if (draw(step, t, 0)) want_q.push_back(step * nw * kWave + t);
      if (draw(step, t, 1)) want_c.push_back(step * nw * kWave + t);
    }
  unsigned seed = 1;
  for (int s = 0; s < 2 + nw + 8; ++s) {
    auto pick = [&](const std::vector<int> &ready) {
      if (s == 0) return ready.front();
      if (s == 1) return ready.back();
      if (s < 2 + nw) {  // one wave first, the others in order
        for (int w : ready)
          if (w == s - 2) return w;
        return ready.front();
      }
      seed = seed * 1664525u + 1013904223u;
      return ready[(seed >> 8) % ready.size()];
    };
    lds.assign(2 * size_t(g_cap), -1);
    out_q.assign(size_t(total) + 64, -1);
    out_c.assign(size_t(total) + 64, -1);
    tails = 0;
    S = {};
    const bool matched = run(nw, pick);
    const size_t nq = size_t(tails & 0xffffffffull), nc = size_t(tails >> 32);
    std::vector<int32_t> q(out_q.begin(), out_q.begin() + std::min(nq, out_q.size()));
    std::vector<int32_t> c(out_c.begin(), out_c.begin() + std::min(nc, out_c.size()));
    std::sort(q.begin(), q.end());
    std::sort(c.begin(), c.end());
    if (!matched || q != want_q || c != want_c) {
      std::printf("schedule %d: barriers %s, queue %zu of %zu%s, candidates %zu of %zu%s\n", s,
                  matched ? "match" : "do not match", nq, want_q.size(),
                  q == want_q ? "" : " (wrong entries)", nc, want_c.size(),
                  c == want_c ? "" : " (wrong entries)");
      return 1;
    }
  }
  std::printf("append step ok\n");
  return 0;
}
