// The block sums of PageRank's delegate pull (their text comes from the
// sources: sum.inc and rows.inc) as one block under many wave schedules.
//   pr_lead_rows ROWS
#include "block.hpp"

#include <cmath>
using std::fabs;
#include "sum.inc"

constexpr int kDW = 8;
struct Step { double alpha; };
static int g_rows;
static double sh[kDW], total;
static std::vector<double> got;
static const int32_t *vid_of;

static double part(int r, int w) { return 1.0 + r * 16 + w; }
static void pr_deleg_done(const Step &, int32_t, int64_t r, int32_t, int64_t, double x,
                          double &delta) {
  got[r] = x;
  delta += x;
}

static void body() {
  const Step a{1.0};
  const double base = 0.0;
  const int l = lane_id(), w = int(threadIdx.x) / kWave;
  double delta = 0.0;
  for (int64_t r = 0; r < g_rows; ++r) {
    const int32_t k = 0;
    const int64_t b = 0, e = 1;
    const double s = part(int(r), w);
#include "rows.inc"
  block_add_f64(&total, delta, sh);
}

int main(int argc, char **argv) {
  if (argc != 2) return 64;
  g_rows = std::atoi(argv[1]);
  const int32_t none[1] = {0};
  vid_of = none;
  block_body = body;
  for (int s = 0; s < schedules(kDW); ++s) {
    got.assign(g_rows, -1.0);
    total = 0.0;
    const bool matched = run(kDW, schedule(s, kDW));
    double want = 0.0;
    for (int r = 0; r < g_rows; ++r) {
      double x = 0.0;
      for (int w = 0; w < kDW; ++w) x += part(r, w);
      want += x;
      if (!matched || got[r] != x) {
        std::printf("schedule %d: row %d is %g, not %g\n", s, r, got[r], x);
        return 1;
      }
    }
    if (total != want) {
      std::printf("schedule %d: total %g, not %g\n", s, total, want);
      return 1;
    }
  }
  std::printf("rows ok\n");
  return 0;
}
