// The compute-unit gate (its text comes from the sources: gate.inc) on the host,
// with devices of different sizes.
#include <algorithm>
#include <atomic>
#include <chrono>
#include <condition_variable>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <memory>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

static int device = 0, units_of[3] = {256, 32, 80};
enum { hipDeviceAttributeMultiprocessorCount };
static int hipGetDevice(int *d) { *d = device; return 0; }
static int hipDeviceGetAttribute(int *v, int, int d) { *v = units_of[d]; return 0; }
#define HIPCHK(x) (void)(x)
enum { DSBFS_ERR_INVALID_ARG };
[[noreturn]] static void fail(int, const std::string &) { std::abort(); }
struct ResidentLease {
  int units = 0;
  void *gate = nullptr;
  ResidentLease(int blocks, bool wait);
  ~ResidentLease();
  bool wanted() const;
};
#include "gate.inc"

#define CHECK(x) \
  if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); std::exit(1); }

int main() {
  using L = std::unique_ptr<ResidentLease>;
  auto take = [](int b, bool w) { return L(new ResidentLease(b, w)); };
  for (device = 0; device < 3; ++device) {
    const int u = units_of[device];
    // a grid that may not run: more blocks than units
    CHECK(take(u + 1, false)->units == 0);
    L a = take(u, false);
    CHECK(a->units == u);
    CHECK(take(1, false)->units == 0);
    a.reset();
    L b = take(u / 2, false), c = take(u - u / 2, false);
    CHECK(b->units && c->units && take(1, false)->units == 0);
    CHECK(!b->wanted() && !c->wanted());
    // two that wait (several blocks a unit): served in order, and none that does
    // not wait goes before them, though units are free meanwhile
    std::vector<int> order;
    std::mutex mu;
    std::atomic<int> waiting{0};
    std::vector<std::thread> t;
    for (int i = 0; i < 2; ++i) {
      t.emplace_back([&, i] {
        ++waiting;
        L w = take(4 * u, true);
        std::lock_guard<std::mutex> lk(mu);
        if (w->units == u) order.push_back(i);
      });
      while (waiting <= i) std::this_thread::yield();
      std::this_thread::sleep_for(std::chrono::milliseconds(50));
    }
    CHECK(b->wanted() && c->wanted());
    c.reset();
    CHECK(take(1, false)->units == 0);
    b.reset();
    for (std::thread &x : t) x.join();
    CHECK(order == (std::vector<int>{0, 1}));
    CHECK(take(u, false)->units == u);
  }
  std::printf("gate ok\n");
  return 0;
}
