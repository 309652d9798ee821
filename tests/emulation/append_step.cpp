// The append step of the bottom-up normal visit (its text comes from the
// sources: append.inc and step.inc) as one block under many wave schedules.
//   append_step WAVES CAP STEPS DENSITY
#include "block.hpp"
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
  block_body = body;
  for (int s = 0; s < schedules(nw); ++s) {
    lds.assign(2 * size_t(g_cap), -1);
    out_q.assign(size_t(total) + 64, -1);
    out_c.assign(size_t(total) + 64, -1);
    tails = 0;
    S = {};
    const bool matched = run(nw, schedule(s, nw));
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
