// The shape rule of one-launch searches (its text comes from the sources:
// shape.inc) on the host: reads "mode forced factor0 n m max_degree" lines, writes
// blocks and threads.
#include <algorithm>
#include <cstdint>
#include <cstdio>

#include "dsbfs.h"
#include "shape.inc"

int main() {
  dsbfs_run_opts o{};
  long long n, m, x;
  while (std::scanf("%d %d %lf %lld %lld %lld", &o.mode, &o.forced, &o.factor0[0], &n, &m, &x) == 6) {
    const OneLaunch r = one_launch_shape(n, m, x, o);
    std::printf("%d %d\n", r.blocks, r.threads);
  }
  return 0;
}
