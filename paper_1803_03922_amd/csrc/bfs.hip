// Single-source BFS on one GPU.
//
// Mode 1 is the paper's degree-separated direction-optimized BFS at p = 1
// (Section IV): the normal frontier is a compacted queue, the delegate
// frontier a bitmask (Section IV-A). A level is up to four phases:
//   previsit  - delegate mask: Fd = Cd & ~Vd, Vd = Cd, dd/dn workloads of the
//               frontier; normal queue: nn/nd workloads, normal frontier
//               bitmap, and the nn top-down visit (nn is always forward and
//               its claims change none of the decision's inputs);
//   list      - (levels with a forward dd or dn visit) the frontier delegates
//               with the prefix sum of their forward row lengths;
//   forward   - top-down nd from the normal queue, dd and dn from that list,
//               balanced over edges;
//   backward  - bottom-up dn over the nd source list, dd and nd over the
//               unvisited delegates, each stopping at the first frontier parent.
// The direction decision (Section IV-B: FV vs BV = |U|(q+s)/q with factor0 /
// factor1, per kernel dd, dn, nd) falls between previsit and the rest. Every
// block makes it for itself from the level's counters, so it costs neither a
// launch nor a barrier.
// Exactly-once discovery comes from atomic test-and-set on the claimed
// bitmaps (normals: Vn; delegates: Cd = visited or found this level), so
// queues hold no duplicates and depth/parent are written once per vertex. (The
// heavy nn visits of long normal rows store first and claim afterwards, one
// thread a vertex: scatter_step, settle.)
//
// Mode 0 is plain top-down BFS over the plain CSR (the paper's "BFS" beside
// "DOBFS", Section VI-C): a list phase (degrees of the queue's rows) and an
// expansion balanced over edges.
//
// Two drivers run the same phases:
//   one launch   - a grid small enough to be resident at once runs all levels,
//                  its phases separated by a grid barrier (small graphs, where
//                  dispatch would cost more than the work);
//   level by level - a kernel per phase, the host one level ahead.
#include <algorithm>
#include <cmath>
#include <condition_variable>
#include <cstring>
#include <memory>
#include <mutex>
#include <string>

#include "internal.hpp"

namespace dsbfs {

void msbfs_release(Workspace *ws);

Workspace::~Workspace() {
  msbfs_release(this);
  if (hstat && !borrowed) (void)hipHostFree(hstat);
  for (hipEvent_t e : events) (void)hipEventDestroy(e);
}

namespace {

constexpr int kSegs = 256;  // segments of a forward list (one block each)

// Per-level counters of a search (device). Three copies rotate: level L adds
// into ctr[L % 3], reads the queue lengths the previous level left in
// ctr[(L + 2) % 3] and clears ctr[(L + 1) % 3].
//
// Sums are kept in kCtrCopies parts, each word on a 128-byte line of its own:
// 2048 blocks adding four counts to one line at the end of a large level cost
// it about 100 us. A block adds to part blockIdx % kCtrCopies.
constexpr int kCtrCopies = 8;
enum { kFvNn, kQNn, kFvNd, kQNd, kFdn, kFvDd, kQDd, kFvDn, kQDn, kPrevSums,
       kClDn = kPrevSums,  // delegates with a dn edge claimed by this level
       kNumSums };
struct LevelCtr {
  // Tails of the next normal queue (bits 0..31: the queue length of the next
  // level) and of the next bottom-up normal candidate list (bits 32..63), in
  // one word: the bottom-up normal pass appends to both and reserves both
  // with one atomic. Neither count reaches 2^31, so no carry crosses.
  CtrLine qn_nc;
  CtrLine sum[kNumSums][kCtrCopies];
};

// A level's counts, summed over the parts.
struct LevelCounts {
  unsigned long long v[kNumSums];
};

// State of a search between levels.
struct LevelState {
  int32_t level;
  int32_t done;        // the frontier is empty: every later kernel returns
  int32_t dir[4];      // current direction per kernel dd, dn, nd, nn (0 forward, 1 backward)
  int32_t cand_state;  // -1: the next bottom-up normal pass scans the whole nd source list
  int32_t nc_pending;  // the previous pass compacted a candidate list of unknown length
  int32_t marked;      // the previous level marked its normal frontier bitmap
  int32_t pad;
  int64_t rem[4];      // unvisited: delegates with a dd edge, with a dn edge, nd-list
                       // normals, normals with an nn edge
  int64_t nc;          // candidates of the next bottom-up normal pass
};

// Totals over the levels so far that the decision keeps (statistics only).
struct LevelTotals {
  unsigned long long deg_sum;                    // sum of frontier degrees
  unsigned long long kept;                       // bottom-up candidates kept
  unsigned long long units0[DSBFS_NUM_KERNELS];  // queue / list entries per kernel
  int64_t launches[DSBFS_NUM_KERNELS];           // visits that had work
};

// What a level does after its previsit.
struct Plan {
  int32_t nd_td, dd_td, dn_td, dn_bu, dd_bu, nd_bu, nn_td, nn_bu;
  int32_t cin_sel, cout_sel;  // bottom-up candidate list read (-1: all) and written
  int64_t nc, qn;
};

// What the host learns of each level (a ring of 4 slots, slot = level & 3):
// written by the level's last kernel into pinned host memory, seq last.
struct LevelStatus {
  int32_t done, level;
  dsbfs_level_stats rec;
  int32_t pad;
  int32_t seq;       // level + 1 once the rest is written
};
constexpr int kStatusSlots = 4;

// Grid barrier: arrivals per group of blocks, groups complete, and one release
// word per group, each on its own 128-byte line.
constexpr int kBarGroups = 8;
constexpr int kMaxOneLaunch = 256;  // blocks of a one-launch search at most
struct GridBar {
  CtrLine arrive[kBarGroups], top, release[kBarGroups];
  CtrLine err;  // 1: a wait exceeded its bound; every block leaves
  uint32_t started[kMaxOneLaunch];  // 1: the block runs
};

// Control block of a search (device memory).
struct SearchCtl {
  GridBar bar;
  LevelState st[2];  // level L reads st[L & 1], its last kernel writes the other
  LevelCtr ctr[3];
  LevelTotals tot;
  unsigned long long units[DSBFS_NUM_KERNELS][4];  // work units per kernel so far
  int64_t seg_len[kSegs];   // edges of each segment of the forward list
  int32_t seg_cnt[kSegs];   // its entries
  int32_t levels;           // one launch: levels with a non-empty frontier
  int32_t pad;
  int64_t left;             // where a further launch goes on from (with st[0]):
                            // normals in no frontier so far
};

// Arguments of every kernel of a search.
struct Search {
  // graph (see Graph)
  const uint64_t *noff, *doff;
  const uint16_t *nlen;
  const int32_t *ncol;
  const uint32_t *nnoff;
  const int32_t *nncol, *dcol, *vid_of, *ndsrc, *nds_col, *nnsrc;
  const int64_t *nds_off;
  const int2 *nds_first, *dd_first;
  const uint32_t *ddm, *dnm;
  const int64_t *poff;
  const int32_t *pcol, *did;
  int32_t n, d, nwords, dwords;
  int64_t n_ndsrc, n_nnsrc;
  // results
  int32_t *depth, *parent;
  // scratch (see Workspace)
  uint32_t *Vn, *Fn0, *Fn1, *Vd, *Fd, *Cd;
  int32_t *Q0, *Q1, *C0, *C1, *dlist;
  int64_t *dscan;
  SearchCtl *ctl;
  LevelStatus *hs;
  double nn_mean;  // nn edges per normal vertex
  int32_t nn_rows;  // rows of about 256 nn edges together, a power of two up to 64
  // options
  double f0[4], f1[4];
  uint64_t forced_seed;
  int32_t forced, nn_do;
  // Output of delegates and of bottom-up claims by a dense pass at the end
  // (k_output), from arrays by delegate and by position of the nd source list.
  int32_t compact;
  int2 *dout;
  int32_t *ppar;
  uint8_t *plev;
  const RankDir *drank, *nrank;
  int32_t count;  // statistics are wanted: keep work units and every workload sum
  int32_t source, mode;
  long long bar_ticks;  // bound of a wait of the grid barrier
  // one launch: its first level (a multiple of 6: levels are counted from 0 in each
  // launch, and buffers alternate by level parity and level % 3)
  int32_t level0;

  __device__ __forceinline__ uint32_t *fn(int p) const { return p ? Fn1 : Fn0; }
  __device__ __forceinline__ int32_t *q(int p) const { return p ? Q1 : Q0; }
  __device__ __forceinline__ int32_t *cand(int p) const { return p ? C1 : C0; }
  __device__ __forceinline__ void put(int32_t v, int32_t p, int32_t dep) const {
    depth[v] = dep + level0;
    if (parent) parent[v] = p;
  }
  // a delegate claimed
  __device__ __forceinline__ void put_deleg(int32_t k, int32_t p, int32_t dep) const {
    if (compact) dout[k] = int2{p, dep + 1};
    else put(vid_of[k], p, dep);
  }
  // position pos of the nd source list (vertex v) claimed bottom-up
  __device__ __forceinline__ void put_pos(int32_t pos, int32_t v, int32_t p, int32_t dep) const {
    if (compact && dep < 256) {
      plev[pos] = uint8_t(dep);
      if (parent) ppar[pos] = p;
    } else {
      put(v, p, dep);
    }
  }
};

__host__ __device__ inline uint64_t mix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
  return z ^ (z >> 31);
}

// Backward workload estimate |U|(q+s)/q (Section IV-B), 0 when q or |U| is 0.
__host__ __device__ inline double bv_estimate(int64_t U, int64_t q, int64_t s) {
  if (q <= 0 || U <= 0) return 0.0;
  return double(U) * (double(q) + double(s)) / double(q);
}

// ---------------------------------------------------------------------------
// block scratch and small helpers
// ---------------------------------------------------------------------------
// LDS of one wave: the 64 rows it walks together.
struct WaveRows {
  int32_t excl[kWave];  // exclusive prefix of the row lengths
  int32_t aux[kWave];   // parent vertex (forward), first hit (backward), mask word
  int64_t beg[kWave];   // row starts
  int64_t mid[kWave];   // where the row's second part starts
};

template <int NW> struct Scratch {
  // entries of each append buffer (four waves: eight blocks fit a compute unit's 160 KB)
  static constexpr int kCap = NW <= 4 ? 1408 : 3072;
  WaveRows w[NW];
  int32_t buf[2 * kCap];  // queue and candidate buffers, or one buffer per wave
  int qcount, ccount;
  unsigned long long qbase, cbase;
  unsigned long long red[16];
  int64_t sh[NW];
  int64_t seg[kSegs + 1];  // prefix of the forward list's segments
  unsigned long long units[DSBFS_NUM_KERNELS * 4];
  LevelCounts now;
  LevelState st, ns;
  Plan plan;
  int64_t qn, nc_prev, q_dn;
  int mark, ok;
};

// Wave totals through DPP scans; the value is the same in every lane.
__device__ __forceinline__ uint32_t wave_total(uint32_t x) {
  return uint32_t(lane_read(wave_incl_scan(int32_t(x)), kWave - 1));
}
__device__ __forceinline__ unsigned long long wave_total(unsigned long long x) {
  // low and high parts separately: 64 values below 2^24 sum below 2^30
  const uint32_t lo = wave_total(uint32_t(x & 0xffffffull));
  const uint32_t hi = wave_total(uint32_t(x >> 24));
  return (static_cast<unsigned long long>(hi) << 24) + lo;
}

__device__ __forceinline__ unsigned long long ctr_load(const unsigned long long *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Adds a thread's counts to word j.. of the block's sums (LDS), one LDS atomic a wave.
template <class T> __device__ __forceinline__ void block_acc(unsigned long long *dst, T x) {
  const T t = wave_total(x);
  if (lane_id() == 0 && t) atomicAdd(dst, static_cast<unsigned long long>(t));
}

// Work units of a kernel (only kept when statistics are wanted): into the
// block's sums, which go to memory once per launch.
template <int NW>
__device__ __forceinline__ void count_units(const Search &a, Scratch<NW> &S, int k, uint32_t x0,
                                            uint32_t x1, uint32_t x2, uint32_t x3) {
  if (!a.count) return;
  block_acc(&S.units[k * 4 + 0], x0);
  block_acc(&S.units[k * 4 + 1], x1);
  block_acc(&S.units[k * 4 + 2], x2);
  block_acc(&S.units[k * 4 + 3], x3);
}

template <int NW> __device__ __forceinline__ void units_open(const Search &a, Scratch<NW> &S) {
  for (int i = threadIdx.x; i < DSBFS_NUM_KERNELS * 4; i += blockDim.x) S.units[i] = 0;
  for (int i = threadIdx.x; i < 16; i += blockDim.x) S.red[i] = 0;
  __syncthreads();
}
template <int NW> __device__ __forceinline__ void units_close(const Search &a, Scratch<NW> &S) {
  __syncthreads();
  if (!a.count) return;
  for (int i = threadIdx.x; i < DSBFS_NUM_KERNELS * 4; i += blockDim.x)
    if (S.units[i]) atomicAdd(&a.ctl->units[i / 4][i % 4], S.units[i]);
}

// Adds the block's sums red[k0 .. k1) to the level's counters and clears them
// (block-uniform).
template <int NW>
__device__ __forceinline__ void red_flush(Scratch<NW> &S, LevelCtr &c, int k0, int k1) {
  __syncthreads();
  const int k = k0 + int(threadIdx.x);
  if (k < k1) {
    const unsigned long long t = S.red[k];
    if (t) atomicAdd(&c.sum[k][blockIdx.x % kCtrCopies].v, t);
    S.red[k] = 0;
  }
  __syncthreads();
}

// Clears a level's counters (by block 0).
__device__ __forceinline__ void ctr_clear(LevelCtr &c) {
  if (blockIdx.x != 0) return;
  for (int i = threadIdx.x; i < kNumSums * kCtrCopies; i += blockDim.x)
    c.sum[i / kCtrCopies][i % kCtrCopies].v = 0;
  if (threadIdx.x == 0) c.qn_nc.v = 0;
}

// Largest index lo in [0, 64) with ex[lo] <= e (ex non-decreasing, ex[0] <= e).
__device__ __forceinline__ int owner64(const int32_t *ex, int32_t e) {
  int lo = 0;
#pragma unroll
  for (int step = 32; step > 0; step >>= 1) {
    const int c = lo + step;
    if (ex[c] <= e) lo = c;
  }
  return lo;
}

// Position of the r-th (from 0) set bit of x, r < popcount(x).
__device__ __forceinline__ int nth_bit(uint32_t x, int r) {
  int pos = 0;
#pragma unroll
  for (int s = 16; s > 0; s >>= 1) {
    const int c = __popc(x & ((1u << s) - 1u));
    if (r >= c) {
      r -= c;
      x >>= s;
      pos += s;
    }
  }
  return pos;
}

// Append buffer of one wave in LDS: a full buffer goes out with one atomic on
// the list's counter (device-scope atomics on one address serialize across
// the chip, 12.6 ns each, so waves never do one per step).
struct WaveAppend {
  int32_t *buf;
  int cap;  // at least 2 * kWave
  unsigned long long *gcount;  // bits 0..31 count this list
  int32_t *gout;
  int cnt;

  __device__ __forceinline__ void push(bool want, int32_t v) {
    const uint64_t m = __ballot(want);
    if (m == 0) return;
    if (want) buf[cnt + int(lanes_below(m))] = v;
    cnt += __popcll(m);
    if (cnt > cap - kWave) flush();
  }
  __device__ void flush() {
    if (cnt == 0) return;
    wave_sync();
    unsigned long long b = 0;
    if (lane_id() == 0) b = atomicAdd(gcount, (unsigned long long)cnt) & 0xffffffffull;
    b = lane_read(b, 0);
    for (int i = lane_id(); i < cnt; i += kWave) gout[b + i] = buf[i];
    wave_sync();
    cnt = 0;
  }
};

// What the block's waves have left in their buffers, with one atomic (a flush
// per wave had up to 8192 of them wait on the tail at a level's end: RMAT 22
// 402 -> 381 us, RMAT 26 2340 -> 2230).
template <int NW> __device__ __forceinline__ void flush_block(Scratch<NW> &S, WaveAppend &qa) {
  const int nw = blockDim.x / kWave, w = threadIdx.x / kWave;
  if (lane_id() == 0) S.sh[w] = qa.cnt;
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t all = 0;
    for (int i = 0; i < nw; ++i) {
      const int64_t c = S.sh[i];
      S.sh[i] = all;
      all += c;
    }
    S.qbase = all ? atomicAdd(qa.gcount, (unsigned long long)all) & 0xffffffffull : 0ull;
  }
  __syncthreads();
  const int64_t to = int64_t(S.qbase) + S.sh[w];
  for (int i = lane_id(); i < qa.cnt; i += kWave) qa.gout[to + i] = qa.buf[i];
  qa.cnt = 0;
  __syncthreads();
}

// The block's two append buffers as one buffer per wave.
template <int NW>
__device__ __forceinline__ WaveAppend wave_append_buf(Scratch<NW> &S, unsigned long long *gcount,
                                                      int32_t *gout) {
  constexpr int per = 2 * Scratch<NW>::kCap / NW;
  return WaveAppend{S.buf + (threadIdx.x / kWave) * per, per, gcount, gout, 0};
}

// ---------------------------------------------------------------------------
// grid barrier (one-launch searches)
// ---------------------------------------------------------------------------
// Two levels: a block counts its arrival on its group's line, the group's last
// arrival counts on `top`, the last of those releases every group. Blocks poll
// their own group's line with relaxed loads; every block fences on both sides
// (agent scope), so plain stores before the barrier are visible after it.
// Counters only grow (k_init zeroes them), so nothing is reset between
// barriers. Measured, empty: 1.9 us for 16 blocks, 2.5 for 64, 3.4 for 128,
// 5.2 for 256, 9 for 512: the fences of each block are served one after the
// other, which is why a one-launch search runs few, wide blocks.
// A wait is bounded: past the bound every block leaves (returns false) and the
// host runs the search level by level instead. Blocks that do not run yet (other
// kernels hold their compute units, and may for long) are not waited for as blocks
// at work are: the widest shape's blocks of 1024 threads with 128 registers need
// every compute unit to themselves, and beside a long one-wave kernel such a
// search lost the whole bound, then 0.2 s. (Held at 112 registers they would fit
// beside it, at 2 to 5% of every search.)
constexpr long long kStartTicks = 200000;     // 2 ms of the 100 MHz wall clock
constexpr long long kBarTicks = 2000000000;   // 20 s

// Tells the others that this block runs (a store: a count on one line is 2 us).
__device__ __forceinline__ void grid_start(GridBar &b) {
  if (threadIdx.x == 0)
    __hip_atomic_store(&b.started[blockIdx.x], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ bool grid_started(const GridBar &b) {
  for (unsigned i = 0; i < gridDim.x; ++i)
    if (!__hip_atomic_load(&b.started[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return false;
  return true;
}

__device__ bool grid_sync(GridBar &b, unsigned long long epoch, int *ok, long long bound) {
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned G = gridDim.x, grp = blockIdx.x % kBarGroups;
    const unsigned gsize = G / kBarGroups + (grp < G % kBarGroups ? 1u : 0u);
    const unsigned ngrp = G < kBarGroups ? G : kBarGroups;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    const unsigned long long t = __hip_atomic_fetch_add(
        &b.arrive[grp].v, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (t + 1 == epoch * gsize) {
      // the group's arrivals happen before this one's count on top
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "agent");
      const unsigned long long u = __hip_atomic_fetch_add(
          &b.top.v, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (u + 1 == epoch * ngrp) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "agent");
        for (unsigned i = 0; i < ngrp; ++i)
          __hip_atomic_store(&b.release[i].v, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    const long long t0 = wall_clock64();
    long long limit = min(bound, kStartTicks);
    int good = 1;
    while (ctr_load(&b.release[grp].v) < epoch) {
      if (ctr_load(&b.err.v)) {
        good = 0;
        break;
      }
      if (wall_clock64() - t0 > limit) {
        if (limit < bound && grid_started(b)) {
          limit = bound;
          continue;
        }
        __hip_atomic_store(&b.err.v, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        good = 0;
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    *ok = good;
  }
  __syncthreads();
  return *ok != 0;
}

// ---------------------------------------------------------------------------
// init
// ---------------------------------------------------------------------------
// Clears bitmaps and the control block, fills the outputs (or, in compact
// mode, clears what the output pass reads) and seeds the source: a delegate is
// claimed (the first previsit moves it to the frontier mask), a normal vertex
// enters the queue. The counters of "level -1" hold the level-0 queue length.
// Bound by the output fill: 6.5 TB/s at 67M vertices.
__global__ void k_init(Search a, LevelState init) {
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  const int64_t t0 = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const int32_t s = a.source;
  const int32_t k = a.mode == 1 ? a.did[s] : -1;
  if (a.compact) {
    for (int64_t i = t0; i < a.d; i += stride) a.dout[i] = i == k ? int2{s, 1} : int2{-1, 0};
    for (int64_t i = t0; i < (a.n_ndsrc + 3) / 4; i += stride)
      reinterpret_cast<uint32_t *>(a.plev)[i] = 0;
    if (k < 0 && t0 == 0) a.put(s, s, 0);
  } else {
    for (int64_t v = t0; v < a.n; v += stride) {
      a.depth[v] = v == s ? 0 : -1;
      if (a.parent) a.parent[v] = v == s ? s : -1;
    }
  }
  for (int64_t w = t0; w < a.nwords; w += stride) {
    a.Vn[w] = k < 0 && w == (s >> 5) ? 1u << (s & 31) : 0u;
    a.Fn0[w] = 0;
    a.Fn1[w] = 0;
  }
  for (int64_t w = t0; w < a.dwords; w += stride) {
    a.Vd[w] = 0;
    a.Fd[w] = 0;
    a.Cd[w] = k >= 0 && w == (k >> 5) ? 1u << (k & 31) : 0u;
  }
  if (blockIdx.x == 0) {
    unsigned long long *c = reinterpret_cast<unsigned long long *>(a.ctl);
    for (int i = threadIdx.x; i < int(sizeof(SearchCtl) / 8); i += blockDim.x) c[i] = 0;
    __syncthreads();
    if (threadIdx.x == 0) {
      a.ctl->st[0] = init;
      LevelCtr &before = a.ctl->ctr[2];
      before.qn_nc.v = k < 0 ? 1u : 0u;
      before.sum[kClDn][0].v = k >= 0 && bit_test(a.dnm, uint32_t(k)) ? 1u : 0u;
      if (k < 0) a.Q0[0] = s;
    }
  }
}

// Compact mode's output: every vertex once, in order, so that depth and parent
// leave as whole lines. A delegate's come from dout, a normal vertex claimed
// bottom-up has its depth at its position of the nd source list, an unvisited
// one gets -1, and a normal vertex claimed top-down was written by its claim.
// Storing each claim where it belongs had the heavy level of RMAT 26 make 16.5M
// write requests of a few bytes, 26 G/s (its delegates alone 7.8M), which
// bound it; the arrays here take 3M, and this pass writes 8 bytes a vertex in
// place of the fill before the search.
//
// A thread has kOutRow vertices in a row: one directory entry of each kind
// and one word of visited bits for all of them, entries of the arrays that
// follow each other, and one 16-byte store where all are put (the caller's
// arrays may begin at any int32: then, and beside vertices that a claim wrote,
// one store each). Loads have no branches (a lane with nothing to read takes
// entry 0), so that all are in flight at once. RMAT 26, 537 MB out: 244 us; with
// a vertex a thread, four apart, 292 us, and with the loads behind branches, a
// chain of round trips, 310 us. The stores alone take 100 us; each of the three
// gathers adds 35 to 48 us.
constexpr int kOutRow = 4;
template <bool VEC> __global__ void __launch_bounds__(256) k_output(Search a) {
  const int64_t stride = int64_t(gridDim.x) * blockDim.x * kOutRow;
  for (int64_t v0 = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) * kOutRow; v0 < a.n;
       v0 += stride) {
    const RankDir dr = a.drank[v0 >> 5], nr = a.nrank[v0 >> 5];
    const uint32_t vis = a.Vn[v0 >> 5];
    int32_t k[kOutRow], pos[kOutRow];
    bool is_d[kOutRow], is_n[kOutRow], seen[kOutRow];
#pragma unroll
    for (int u = 0; u < kOutRow; ++u) {
      const int32_t v = int32_t(v0) + u;
      is_d[u] = dr.has(v);
      seen[u] = (vis >> (v & 31)) & 1u;
      is_n[u] = !is_d[u] && seen[u] && nr.has(v);
      k[u] = is_d[u] ? dr.rank(v) : 0;
      pos[u] = is_n[u] ? nr.rank(v) : 0;
    }
    int2 o[kOutRow];
    int32_t lev[kOutRow], pp[kOutRow];
#pragma unroll
    for (int u = 0; u < kOutRow; ++u) {
      o[u] = a.dout[k[u]];
      lev[u] = a.plev[pos[u]];
      pp[u] = a.parent ? a.ppar[pos[u]] : 0;
    }
    int32_t dep[kOutRow], par[kOutRow];
    bool put[kOutRow], all = VEC;
#pragma unroll
    for (int u = 0; u < kOutRow; ++u) {
      dep[u] = is_d[u] ? o[u].y - 1 : (is_n[u] ? lev[u] : -1);
      par[u] = is_d[u] ? (o[u].y ? o[u].x : -1) : (is_n[u] ? pp[u] : -1);
      // a visited normal vertex without a depth here was written by its claim
      put[u] = v0 + u < a.n && (is_d[u] || !seen[u] || (is_n[u] && lev[u] != 0));
      all = all && put[u];
    }
    if (all) {
      *reinterpret_cast<int4 *>(a.depth + v0) = int4{dep[0], dep[1], dep[2], dep[3]};
      if (a.parent)
        *reinterpret_cast<int4 *>(a.parent + v0) = int4{par[0], par[1], par[2], par[3]};
      continue;
    }
#pragma unroll
    for (int u = 0; u < kOutRow; ++u) {
      if (!put[u]) continue;
      a.depth[v0 + u] = dep[u];
      if (a.parent) a.parent[v0 + u] = par[u];
    }
  }
}

// ---------------------------------------------------------------------------
// decision
// ---------------------------------------------------------------------------
// Opens level L in the block: the queue length and candidate count the
// previous level left, and whether this level marks the normal frontier
// bitmap Fn. Fn is read only by a bottom-up nd visit (which needs an unvisited
// delegate with a dn edge left after this level's frontier) and, with nn_do,
// by a bottom-up nn visit.
template <int NW>
__device__ __forceinline__ void level_open(const Search &a, Scratch<NW> &S, int L) {
  const LevelCtr &prev = a.ctl->ctr[(L + 2) % 3];
  // the first wave: lanes 0..7 the parts of the claim count, lane 8 the tails
  if (threadIdx.x < kWave) {
    const int l = lane_id();
    unsigned long long x = 0;
    if (l < kCtrCopies) x = ctr_load(&prev.sum[kClDn][l].v);
    else if (l == kCtrCopies) x = ctr_load(&prev.qn_nc.v);
    const uint32_t claimed = wave_total(l < kCtrCopies ? uint32_t(x) : 0u);
    const unsigned long long t = lane_read(x, kCtrCopies);
    if (l == 0) {
      S.q_dn = int64_t(claimed);
      S.qn = int64_t(t & 0xffffffffull);
      S.nc_prev = int64_t(t >> 32);
      S.mark = S.st.rem[1] - S.q_dn > 0 || (a.nn_do && S.st.rem[3] > 0);
    }
  }
  __syncthreads();
}

// Direction decision of Section IV-B for dd, dn, nd (indices 0, 1, 2) from
// the level's previsit counts c, in FP64 with the same expression as the
// oracle's replay, the bookkeeping of the remaining counts, and the plan of
// the rest of the level. One thread, on its own copies; rec (may be NULL) gets
// the level's record.
__device__ __forceinline__ void decide_level(const Search &a, LevelState &t, const LevelCounts &c,
                                             int64_t qn, int64_t nc_prev, int mark, Plan &p,
                                             LevelStatus *rec) {
  const int32_t L = t.level;
  const int64_t fdn = int64_t(c.v[kFdn]);
  if (t.nc_pending) {
    // length of the candidate list the previous bottom-up normal pass compacted
    t.nc = nc_prev;
    t.nc_pending = 0;
  }
  t.level = L + 1;
  t.marked = 0;
  if (rec) {
    rec->level = L;
    rec->done = 0;
  }
  if (qn == 0 && fdn == 0) {
    t.done = 1;
    if (rec) rec->done = 1;
    return;
  }
  t.marked = mark;
  const int64_t q[3] = {int64_t(c.v[kQDd]), int64_t(c.v[kQDn]), int64_t(c.v[kQNd])};
  const int64_t FV[3] = {int64_t(c.v[kFvDd]), int64_t(c.v[kFvDn]), int64_t(c.v[kFvNd])};
  const int64_t q_nn = int64_t(c.v[kQNn]), fv_nn = int64_t(c.v[kFvNn]);
  t.rem[0] -= q[0];
  t.rem[1] -= q[1];
  t.rem[2] -= q[2];
  t.rem[3] -= q_nn;
  const int64_t U[3] = {t.rem[0], t.rem[2], t.rem[1]};
  const int64_t R[3] = {t.rem[0], t.rem[1], t.rem[2]};
  auto choose = [&](int k, int64_t qk, int64_t fvk, double bvk) {
    int d = t.dir[k];
    if (a.forced == 1) d = 0;
    else if (a.forced == 2) d = L >= 1 ? 1 : 0;
    else if (a.forced == 3)
      d = int(mix64(a.forced_seed + uint64_t(L) * 3 + k + (k == 3 ? 0x5bd1e995ull : 0)) & 1);
    else if (qk > 0) {
      if (d == 0 && double(fvk) > a.f0[k] * bvk) d = 1;
      else if (d == 1 && double(fvk) < a.f1[k] * bvk) d = 0;
    }
    t.dir[k] = d;
  };
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double bv = bv_estimate(U[k], q[k], R[k]);
    choose(k, q[k], FV[k], bv);
    if (rec) {
      rec->rec.q[k] = q[k];
      rec->rec.s[k] = R[k];
      rec->rec.U[k] = U[k];
      rec->rec.FV[k] = FV[k];
      rec->rec.BV[k] = bv;
      rec->rec.dir[k] = t.dir[k];
    }
  }
  // nn (nn_do only): U = s = unvisited normals with an nn edge (symmetric)
  const double bv_nn = a.nn_do ? bv_estimate(t.rem[3], q_nn, t.rem[3]) : 0.0;
  if (a.nn_do) choose(3, q_nn, fv_nn, bv_nn);
  p.qn = qn;
  p.nn_td = a.nn_do && t.dir[3] == 0 && q_nn > 0;
  p.nn_bu = a.nn_do && t.dir[3] == 1 && q_nn > 0 && t.rem[3] > 0;
  // without nn_do, nn went top-down inside the previsit already
  p.dd_td = t.dir[0] == 0 && q[0] > 0;
  p.dn_td = t.dir[1] == 0 && q[1] > 0;
  p.nd_td = t.dir[2] == 0 && q[2] > 0;
  p.dd_bu = t.dir[0] == 1 && q[0] > 0 && U[0] > 0;
  p.dn_bu = t.dir[1] == 1 && q[1] > 0 && U[1] > 0 && t.nc > 0;
  p.nd_bu = t.dir[2] == 1 && q[2] > 0 && U[2] > 0;
  p.nc = t.nc;
  if (p.dn_bu) {
    p.cin_sel = t.cand_state;
    p.cout_sel = t.cand_state < 0 ? 0 : (t.cand_state ^ 1);
    t.cand_state = p.cout_sel;
    t.nc_pending = 1;
  }
  if (rec) {
    rec->rec.U_nn = a.nn_do ? t.rem[3] : 0;
    rec->rec.s_nn = rec->rec.U_nn;
    rec->rec.BV_nn = bv_nn;
    rec->rec.dir_nn = a.nn_do ? t.dir[3] : 0;
    rec->rec.FV_nn = fv_nn;
    rec->rec.q_nn = q_nn;
    rec->rec.frontier_normal = qn;
    rec->rec.frontier_delegate = fdn;
  }
}

// Adds level st's contribution to the totals (one thread of one block, after
// the decision; only when statistics are wanted).
__device__ inline void account_level(const Search &a, const LevelState &st, const LevelState &ns,
                                     const LevelCounts &c, int64_t qn, int64_t nc_prev,
                                     const Plan &p, LevelTotals &t) {
  const int64_t fdn = int64_t(c.v[kFdn]);
  t.units0[DSBFS_K_PREV_NORMAL] += qn;
  t.units0[DSBFS_K_PREV_DELEG] += fdn;
  ++t.launches[DSBFS_K_PREV_NORMAL];
  if (a.d > 0) ++t.launches[DSBFS_K_PREV_DELEG];
  t.deg_sum += c.v[kFvNn] + c.v[kFvNd] + c.v[kFvDd] + c.v[kFvDn];
  if (st.nc_pending) t.kept += nc_prev;
  if (ns.done) return;
  ++t.launches[DSBFS_K_CLOSE];
  if (ns.marked) t.units0[DSBFS_K_CLOSE] += a.nwords;
  if (p.nd_td) t.units0[DSBFS_K_TD_NORMAL] += qn;
  if (p.nn_td) t.units0[DSBFS_K_TD_NN] += qn;
  if (p.dd_td || p.dn_td) t.units0[DSBFS_K_TD_DELEG] += fdn;
  t.launches[DSBFS_K_TD_NORMAL] += p.nd_td;
  t.launches[DSBFS_K_TD_DELEG] += p.dd_td || p.dn_td;
  t.launches[DSBFS_K_BU_NORMAL] += p.dn_bu;
  t.launches[DSBFS_K_BU_DELEG] += p.dd_bu || p.nd_bu;
  t.launches[DSBFS_K_TD_NN] += p.nn_td;
  t.launches[DSBFS_K_BU_NN] += p.nn_bu;
}

// The decision of level L, made by every block for itself (S.ns, S.plan).
// level_open has run for L.
template <int NW>
__device__ __forceinline__ void level_plan(const Search &a, Scratch<NW> &S, int L,
                                           LevelStatus *rec = nullptr) {
  const LevelCtr &c = a.ctl->ctr[L % 3];
  // the first wave, eight lanes a sum: nine sums in two rounds of loads
  static_assert(kPrevSums <= 2 * kWave / kCtrCopies, "two rounds");
  if (threadIdx.x < kWave) {
    const int l = lane_id(), part = l % kCtrCopies;
    unsigned long long x[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int k = r * (kWave / kCtrCopies) + l / kCtrCopies;
      x[r] = k < kPrevSums ? ctr_load(&c.sum[k][part].v) : 0ull;
    }
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int k = r * (kWave / kCtrCopies) + l / kCtrCopies;
      unsigned long long t = x[r];
      for (int o = 1; o < kCtrCopies; o <<= 1) t += __shfl_xor(t, o, kWave);
      if (part == 0 && k < kPrevSums) S.now.v[k] = t;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const LevelCounts now = S.now;
    LevelState t = S.st;
    Plan p{};
    decide_level(a, t, now, S.qn, S.nc_prev, S.mark, p, rec);
    S.ns = t;
    S.plan = p;
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------
// previsit
// ---------------------------------------------------------------------------
// Mask words of one wave step of the delegate passes: a power of two, small
// enough that every wave of the grid has a step when there are that many words.
__device__ __forceinline__ int mask_step(int32_t words, int64_t nwaves, int least) {
  int c = kWave;
  while (c > least && int64_t(words) < c * nwaves) c >>= 1;
  return c;
}

// Delegates claimed by the previous level become the frontier mask, with their
// dd/dn counts. Workloads (degree sums) need the row offsets of every frontier
// delegate; they are read only while a decision can still depend on them or
// statistics want them: under the heuristic schedule with factor1 = 0 a kernel
// that went backward never switches back. A wave enumerates the set bits of
// its words 64 at a time, one delegate per lane, so the offset reads are
// coalesced and dense whatever the density of the mask (one thread per word,
// walking its bits alone, took 54 us at 1.7M frontier delegates of RMAT 26).
template <int NW> __device__ void prev_deleg(const Search &a, Scratch<NW> &S) {
  const bool need_fv = a.count || a.forced != 0 || S.st.dir[0] == 0 || S.st.dir[1] == 0 ||
                       a.f1[0] != 0.0 || a.f1[1] != 0.0;
  const int l = lane_id();
  const int64_t nwaves = int64_t(gridDim.x) * (blockDim.x / kWave);
  const int64_t wid = int64_t(blockIdx.x) * (blockDim.x / kWave) + threadIdx.x / kWave;
  const int cw = mask_step(a.dwords, nwaves, 2);
  WaveRows &R = S.w[threadIdx.x / kWave];
  uint32_t cnt = 0, q_dd = 0, q_dn = 0;
  unsigned long long fv_dd = 0, fv_dn = 0;
  for (int64_t w0 = wid * cw; w0 < a.dwords; w0 += nwaves * cw) {
    const int64_t w = w0 + l;
    uint32_t f = 0;
    if (l < cw && w < a.dwords) {
      const uint32_t cd = a.Cd[w];
      f = cd & ~a.Vd[w];
      a.Fd[w] = f;
      if (f) {
        a.Vd[w] = cd;
        cnt += __popc(f);
        q_dd += __popc(f & a.ddm[w]);
        q_dn += __popc(f & a.dnm[w]);
      }
    }
    if (!need_fv) continue;
    const int32_t c = __popc(f);
    const int32_t incl = wave_incl_scan(c);
    const int32_t T = lane_read(incl, kWave - 1);
    if (T == 0) continue;
    wave_sync();
    R.excl[l] = incl - c;
    R.aux[l] = int32_t(f);
    wave_sync();
    for (int32_t i = l; i < T; i += kWave) {
      const int o = owner64(R.excl, i);
      const int64_t k = (w0 + o) * 32 + nth_bit(uint32_t(R.aux[o]), i - R.excl[o]);
      const uint64_t x0 = a.doff[k], x1 = a.doff[k + 1];
      const int64_t dd = row_first(x0);
      fv_dd += dd;
      fv_dn += row_start(x1) - row_start(x0) - dd;
    }
  }
  block_acc(&S.red[kFdn], cnt);
  block_acc(&S.red[kQDd], q_dd);
  block_acc(&S.red[kQDn], q_dn);
  if (need_fv) {
    block_acc(&S.red[kFvDd], fv_dd);
    block_acc(&S.red[kFvDn], fv_dn);
  }
}

// Forward expansion of one part of the rows of up to 64 normal vertices, one
// per lane (u: vertex, len: part length, beg: its start): the lengths are
// prefix-summed across the wave, which walks the concatenated entries 64 at a
// time, so lanes stay busy whatever the mix of degrees (all are <= TH). Four
// steps of a long walk go together: their column loads, then their tests,
// then their atomics are in flight at once, since a step alone waits for
// three dependent round trips. to_normal: nn (claims normals, enqueues them),
// else nd (claims delegates in Cd).
template <bool to_normal, int U>
__device__ __forceinline__ void expand_step(const Search &a, const WaveRows &R,
                                            const int32_t *col, int32_t e0, int32_t T,
                                            int32_t dep, WaveAppend &qa, uint32_t &claimed,
                                            uint32_t &with_dn) {
  const int l = lane_id();
  int32_t v[U];
  int o[U];
  uint32_t wd[U], old[U];
  uint32_t *const bm = to_normal ? a.Vn : a.Cd;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int32_t e = min(e0 + u * kWave + l, T - 1);
    o[u] = owner64(R.excl, e);
    v[u] = col[R.beg[o[u]] + (e - R.excl[o[u]])];
  }
#pragma unroll
  for (int u = 0; u < U; ++u) wd[u] = bm[uint32_t(v[u]) >> 5];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t b = 1u << (v[u] & 31);
    old[u] = b;
    // a stale word can only lack a bit: the atomic decides
    if (e0 + u * kWave + l < T && !(wd[u] & b)) old[u] = atomicOr(&bm[uint32_t(v[u]) >> 5], b);
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const bool won = !(old[u] & (1u << (v[u] & 31)));
    if (won) {
      ++claimed;
      if (to_normal) {
        a.put(v[u], R.aux[o[u]], dep);
      } else {
        a.put_deleg(v[u], R.aux[o[u]], dep);
        with_dn += bit_test(a.dnm, uint32_t(v[u]));
      }
    }
    if (to_normal) qa.push(won, v[u]);
  }
}

template <bool to_normal>
__device__ __forceinline__ void expand_rows(const Search &a, WaveRows &R, const int32_t *col,
                                            int32_t u, int32_t len, int64_t beg, int32_t dep,
                                            WaveAppend &qa, uint32_t &edges, uint32_t &claimed,
                                            uint32_t &with_dn) {
  const int l = lane_id();
  const int32_t incl = wave_incl_scan(len);
  const int32_t T = lane_read(incl, kWave - 1);
  if (T == 0) return;
  wave_sync();
  R.excl[l] = incl - len;
  R.aux[l] = u;
  R.beg[l] = beg;
  wave_sync();
  if (l == 0) edges += uint32_t(T);
  int32_t e0 = 0;
  for (; T - e0 > 2 * kWave; e0 += 4 * kWave)
    expand_step<to_normal, 4>(a, R, col, e0, T, dep, qa, claimed, with_dn);
  for (; e0 < T; e0 += kWave)
    expand_step<to_normal, 1>(a, R, col, e0, T, dep, qa, claimed, with_dn);
}

// A heavy level's nn visit: every edge to a vertex that no earlier level
// claimed stores its row's vertex there, and settle() collects what was
// stored. Atomics bound such a level otherwise: 26 G/s on this card whatever
// they touch (random 4-byte stores 80 G/s), and as a wave's cached bitmap words
// do not show the other chiplets' claims, nearly every edge to a vertex
// unvisited at the level's start needs one.
// ER 2^22 of mean degree 16: its two heavy levels 685 and 501 us before, 270 and
// 370 with 20 each for settle(); the second is bound by 51M bit tests (200 G/s)
// and gains from rows read in order.
template <int U>
__device__ __forceinline__ void scatter_step(const Search &a, const WaveRows &R,
                                             const int32_t *col, int32_t e0, int32_t T,
                                             int32_t dep) {
  const int l = lane_id();
  int32_t v[U];
  int o[U];
  uint32_t wd[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int32_t e = min(e0 + u * kWave + l, T - 1);
    o[u] = owner64(R.excl, e);
    v[u] = col[R.beg[o[u]] + (e - R.excl[o[u]])];
  }
#pragma unroll
  for (int u = 0; u < U; ++u) wd[u] = a.Vn[uint32_t(v[u]) >> 5];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    // (the lanes past the end repeat the last edge)
    if ((wd[u] >> (v[u] & 31)) & 1u) continue;
    if (a.parent) a.parent[v[u]] = R.aux[o[u]];
    else a.depth[v[u]] = dep + a.level0;
  }
}

__device__ __forceinline__ void scatter_rows(const Search &a, WaveRows &R, const int32_t *col,
                                             int32_t u, int32_t len, int64_t beg, int32_t dep,
                                             uint32_t &edges) {
  const int l = lane_id();
  const int32_t incl = wave_incl_scan(len);
  const int32_t T = lane_read(incl, kWave - 1);
  if (T == 0) return;
  wave_sync();
  R.excl[l] = incl - len;
  R.aux[l] = u;
  R.beg[l] = beg;
  wave_sync();
  if (l == 0) edges += uint32_t(T);
  int32_t e0 = 0;
  for (; T - e0 > 2 * kWave; e0 += 4 * kWave) scatter_step<4>(a, R, col, e0, T, dep);
  for (; e0 < T; e0 += kWave) scatter_step<1>(a, R, col, e0, T, dep);
}

// Claims what the scatter of level L stored: the normal vertices whose parent
// (or depth, where the caller wants no parents) is set and that no level has
// claimed yet. A wave has a contiguous share of the vertices, 64 groups of 64
// at a time, and the block reserves room for all its claims of a round with one
// atomic (a buffer per wave had 10K atomics on the tail, 115 us at 3.2M claims;
// now 20). The next level reads the rows in near-ascending order, too. Runs
// beside the delegate list, which reads nothing of it.
template <int NW> __device__ void settle(const Search &a, Scratch<NW> &S, int L) {
  constexpr int U = 4;
  const int l = lane_id(), nw = blockDim.x / kWave;
  const int64_t nwaves = int64_t(gridDim.x) * nw;
  const int64_t wid = int64_t(blockIdx.x) * nw + threadIdx.x / kWave;
  const int64_t groups = (int64_t(a.n) + kWave - 1) / kWave;
  const int64_t per = (groups + nwaves - 1) / nwaves;
  const int64_t gb = min(wid * per, groups), ge = min(gb + per, groups);
  const int32_t *const set = a.parent ? a.parent : a.depth;
  int32_t *const out = a.q((L + 1) & 1);
  uint32_t claimed = 0;
  for (int64_t r0 = 0; r0 < per; r0 += kWave) {
    unsigned long long mine = 0;  // lane i: the claims of group gb + r0 + i
    const int64_t re = min(ge, gb + r0 + kWave);
    for (int64_t g0 = gb + r0; g0 < re; g0 += U) {
      int32_t x[U];
      uint32_t vis[U], dl[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t v = min((g0 + u) * kWave + l, int64_t(a.n) - 1);
        x[u] = set[v];
        vis[u] = a.Vn[v >> 5];
        dl[u] = a.drank[v >> 5].bits;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t v = (g0 + u) * kWave + l;
        const bool won =
            g0 + u < re && v < a.n && x[u] != -1 && !(((vis[u] | dl[u]) >> (v & 31)) & 1u);
        const unsigned long long m = __ballot(won);
        const uint32_t half = uint32_t(l < 32 ? m : m >> 32);
        if ((l & 31) == 0 && half) a.Vn[v >> 5] = vis[u] | half;
        if (won && a.parent) a.depth[v] = L + 1 + a.level0;
        if (l == int(g0 + u - gb - r0)) mine = m;
      }
    }
    const int32_t c = __popcll(mine);
    claimed += c;
    const int32_t incl = wave_incl_scan(c);
    if (l == kWave - 1) S.sh[threadIdx.x / kWave] = incl;
    __syncthreads();
    if (threadIdx.x == 0) {
      int64_t all = 0;
      for (int w = 0; w < nw; ++w) {
        const int64_t k = S.sh[w];
        S.sh[w] = all;
        all += k;
      }
      S.qbase = all ? atomicAdd(&a.ctl->ctr[L % 3].qn_nc.v, (unsigned long long)all) & 0xffffffffull
                    : 0ull;
    }
    __syncthreads();
    const int64_t to = int64_t(S.qbase) + S.sh[threadIdx.x / kWave];
    for (int g = 0; gb + r0 + g < re; ++g) {
      const unsigned long long m = lane_read(mine, g);
      const int32_t at = lane_read(incl - c, g);
      if ((m >> l) & 1ull)
        out[to + at + int(lanes_below(m))] = int32_t((gb + r0 + g) * kWave + l);
    }
    __syncthreads();
  }
  count_units(a, S, DSBFS_K_PREV_NORMAL, 0, 0, claimed, 0);
}

// A wave's rows of a queue of q entries: as few a step as give every wave of the
// grid one, but no fewer than nn_rows and no more than 64, dealt out over the
// blocks. A wave expands its rows in a chain of steps: with 64 rows of 16 edges
// a wave, the waves in blocks in a row, a level of 3170 rows took 67 us, now 20
// (ER 2^22, 1199 -> 1100 us; RMAT 22, nearly all rows in full steps, gains 3%
// from the dealing alone). Rows of one edge or two are not spread: it would
// only add atomics to Fn. A queue short enough for 256 blocks is left to those:
// a block that claims costs an atomic on the queue's tail.
struct QueueShare {
  int64_t first, stride;
  int rows;
  // the whole block has none
  __device__ __forceinline__ bool none(int64_t q) const {
    return rows == 0 || int64_t(blockIdx.x) * rows >= q;
  }
};
__device__ __forceinline__ QueueShare queue_share(const Search &a, int64_t q) {
  const int nw = blockDim.x / kWave;
  const int64_t grid =
      q <= 256 * int64_t(blockDim.x) ? min(int64_t(gridDim.x), int64_t(256)) : int64_t(gridDim.x);
  const int rows = mask_step(int32_t(q), grid * nw, a.nn_rows);
  if (blockIdx.x >= grid) return {q, 0, 0};
  return {(int64_t(threadIdx.x / kWave) * grid + blockIdx.x) * rows, grid * nw * rows, rows};
}

// The nn part of row u: its length and, when `start` is set, where it begins
// (in the compact nn copy if there is one, else in the full rows).
__device__ __forceinline__ void nn_part(const Search &a, int32_t u, bool start, int32_t &nn,
                                        int64_t &nd, int64_t &beg) {
  // part lengths from 2 bytes per vertex; the start only for rows with nn
  // edges (most normal rows of a scale-free graph have none)
  const uint32_t lw = a.nlen[u];
  if (lw == kLenWide) {
    const uint64_t w0 = a.noff[u], w1 = a.noff[u + 1];
    nn = int32_t(row_first(w0));
    nd = row_start(w1) - row_start(w0) - nn;
    beg = a.nnoff ? int64_t(a.nnoff[u]) : row_start(w0);
  } else {
    nn = int32_t(lw & 0xFFu);
    nd = int64_t(lw >> 8);
    if (nn > 0 && start) beg = a.nnoff ? int64_t(a.nnoff[u]) : row_start(a.noff[u]);
  }
}

// One pass over the normal queue: previsit (nn/nd workloads and counts of the
// frontier, normal frontier bitmap Fn) fused with the nn top-down visit. With
// nn under the direction decision (nn_do) it only counts and marks.
// scatter: the visit of a heavy level (settle() follows).
template <int NW>
__device__ void prev_normal(const Search &a, Scratch<NW> &S, int L, bool scatter) {
  const int64_t qn = S.qn;
  const QueueShare sh = queue_share(a, qn);
  if (sh.none(qn)) return;
  const int mark = S.mark, expand = !a.nn_do;
  const int32_t *const Q = a.q(L & 1);
  uint32_t *const Fn = a.fn(L & 1);
  WaveRows &R = S.w[threadIdx.x / kWave];
  WaveAppend qa = wave_append_buf(S, &a.ctl->ctr[L % 3].qn_nc.v, a.q((L + 1) & 1));
  uint32_t q_nn = 0, q_nd = 0, edges = 0, claimed = 0, none = 0;
  unsigned long long fv_nn = 0, fv_nd = 0;
  for (int64_t i0 = sh.first; i0 < qn; i0 += sh.stride) {
    const int64_t i = i0 + lane_id();
    const bool ok = lane_id() < sh.rows && i < qn;
    int32_t u = 0, nn = 0;
    int64_t beg = 0;
    if (ok) {
      int64_t nd = 0;
      u = Q[i];
      nn_part(a, u, expand, nn, nd, beg);
      fv_nn += nn;
      q_nn += nn > 0;
      fv_nd += nd;
      q_nd += nd > 0;
    }
    // queues filled by the bottom-up pass are in ascending order: mark word by word
    if (mark) wave_bit_set(Fn, uint32_t(u), ok, true);
    if (scatter)
      scatter_rows(a, R, a.nnoff ? a.nncol : a.ncol, u, nn, beg, L + 1, edges);
    else if (expand)
      expand_rows<true>(a, R, a.nnoff ? a.nncol : a.ncol, u, nn, beg, L + 1, qa, edges, claimed,
                        none);
  }
  // (few waves: their atomics are done before the block's waves have met)
  if (qn > 256 * sh.rows) flush_block(S, qa);
  else qa.flush();
  block_acc(&S.red[kQNd], q_nd);
  // the other sums only where a decision or the statistics read them
  if (a.count || a.forced != 0 || S.st.dir[2] == 0 || a.f1[2] != 0.0)
    block_acc(&S.red[kFvNd], fv_nd);
  if (a.count || a.nn_do) {
    block_acc(&S.red[kFvNn], fv_nn);
    block_acc(&S.red[kQNn], q_nn);
  }
  // units: queue entries (counted by the decision), nn edges, normals claimed
  count_units(a, S, DSBFS_K_PREV_NORMAL, 0, edges, claimed, 0);
}

// Previsit of level L: kDeleg and kNormal parts, and kClear: the frontier
// bitmap that the previous level marked (two alternate by level, so clearing
// one does not wait for the marking of the other) and the counters of level
// L + 1.
enum { kDeleg = 1, kNormal = 2, kClear = 4, kNn = 8, kCommit = 16 };
template <int NW, int parts>
__device__ __forceinline__ void previsit(const Search &a, Scratch<NW> &S, int L,
                                         bool scatter = false) {
  if (parts & kClear) {
    if (S.st.marked) {
      uint32_t *const F = a.fn((L + 1) & 1);
      for (int64_t w = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; w < a.nwords;
           w += int64_t(gridDim.x) * blockDim.x)
        F[w] = 0;
    }
    ctr_clear(a.ctl->ctr[(L + 1) % 3]);
  }
  if (parts & kDeleg) prev_deleg(a, S);
  if (parts & kNormal) prev_normal(a, S, L, scatter);
  if (parts & (kDeleg | kNormal)) red_flush(S, a.ctl->ctr[L % 3], 0, kPrevSums);
}

// ---------------------------------------------------------------------------
// edge-balanced expansion of a list of rows
// ---------------------------------------------------------------------------
// The list is cut into segments, one per listing block: segment b's entries
// start at b * stride of the list, dscan holds each entry's exclusive prefix
// within its segment, seg_len its total. Totals meet in the expansion, where
// every block scans the (at most kSegs) segment lengths in LDS: the list needs
// no device-wide scan (three kernels before).

// Exclusive scan of x over the block; *total = sum.
template <int NW>
__device__ __forceinline__ int64_t block_scan(Scratch<NW> &S, int64_t x, int64_t *total) {
  const int w = threadIdx.x / kWave, nw = blockDim.x / kWave;
  const int64_t incl = wave_incl_scan(x);
  if (lane_id() == kWave - 1) S.sh[w] = incl;
  __syncthreads();
  int64_t before = 0, all = 0;
  for (int i = 0; i < nw; ++i) {
    const int64_t t = S.sh[i];
    before += i < w ? t : 0;
    all += t;
  }
  *total = all;
  __syncthreads();
  return before + incl - x;
}

__device__ __forceinline__ int list_segs() { return min(int(gridDim.x), kSegs); }

// Entries of a segment of mode 0's list: an even share of the queue, but no
// less than kMinSeg, so that a wave's share of a short queue lies in one
// segment (a wave takes the segments of its share one after the other).
constexpr int64_t kMinSeg = 1024;
__device__ __forceinline__ int64_t plain_seg(int64_t qn, int ns) {
  return max((qn + ns - 1) / ns, kMinSeg);
}

// Frontier delegates with the lengths of their forward parts (dd if dd_td, dn
// if dn_td). Segment b lists the delegates of its share of the mask words.
template <int NW> __device__ void list_deleg(const Search &a, Scratch<NW> &S) {
  const int ns = list_segs();
  if (int(blockIdx.x) >= ns) return;
  const int dd_td = S.plan.dd_td, dn_td = S.plan.dn_td;
  const int64_t per = (int64_t(a.dwords) + ns - 1) / ns;
  const int64_t wb = blockIdx.x * per, we = min(wb + per, int64_t(a.dwords));
  const int64_t out0 = wb * 32;
  int64_t done = 0, sum = 0;
  for (int64_t w0 = wb; w0 < we; w0 += blockDim.x) {
    const int64_t w = w0 + threadIdx.x;
    const uint32_t f = w < we ? a.Fd[w] : 0u;
    int64_t len = 0;
    for (uint32_t g = f; g; g &= g - 1) {
      const int64_t k = w * 32 + __ffs(g) - 1;
      const uint64_t x0 = a.doff[k], x1 = a.doff[k + 1];
      const int64_t dd = row_first(x0), dn = row_start(x1) - row_start(x0) - dd;
      len += (dd_td ? dd : 0) + (dn_td ? dn : 0);
    }
    int64_t all, alln;
    int64_t at = sum + block_scan(S, len, &all);
    int64_t pos = out0 + done + block_scan(S, int64_t(__popc(f)), &alln);
    for (uint32_t g = f; g; g &= g - 1) {
      const int64_t k = w * 32 + __ffs(g) - 1;
      const uint64_t x0 = a.doff[k], x1 = a.doff[k + 1];
      const int64_t dd = row_first(x0), dn = row_start(x1) - row_start(x0) - dd;
      a.dlist[pos] = int32_t(k);
      a.dscan[pos] = at;
      ++pos;
      at += (dd_td ? dd : 0) + (dn_td ? dn : 0);
    }
    sum += all;
    done += alln;
  }
  if (threadIdx.x == 0) {
    a.ctl->seg_len[blockIdx.x] = sum;
    a.ctl->seg_cnt[blockIdx.x] = int32_t(done);
  }
}

// Mode 0: the whole queue, with the degrees of its rows.
template <int NW> __device__ void list_plain(const Search &a, Scratch<NW> &S, int L) {
  const int ns = list_segs();
  if (int(blockIdx.x) >= ns) return;
  const int32_t *const Q = a.q(L & 1);
  const int64_t per = plain_seg(S.qn, ns);
  const int64_t b = min(blockIdx.x * per, S.qn), e = min(b + per, S.qn);
  int64_t sum = 0;
  for (int64_t i0 = b; i0 < e; i0 += blockDim.x) {
    const int64_t i = i0 + threadIdx.x;
    int64_t len = 0;
    if (i < e) {
      const int32_t u = Q[i];
      len = a.poff[u + 1] - a.poff[u];
    }
    int64_t all;
    const int64_t at = sum + block_scan(S, len, &all);
    if (i < e) a.dscan[i] = at;
    sum += all;
  }
  if (threadIdx.x == 0) {
    a.ctl->seg_len[blockIdx.x] = sum;
    a.ctl->seg_cnt[blockIdx.x] = int32_t(e - b);
  }
}

// Largest i in [0, cnt) with p[i] <= x (p non-decreasing, p[0] <= x), for a
// whole wave: 64 probes a round.
__device__ __forceinline__ int64_t wave_search(const int64_t *p, int64_t cnt, int64_t x) {
  int64_t lo = 0, len = cnt;
  while (len > 1) {
    const int64_t step = (len + kWave - 1) / kWave;
    const int64_t at = int64_t(lane_id()) * step;
    const uint64_t m = __ballot(at < len && p[lo + min(at, len - 1)] <= x);
    const int64_t j = (63 - __builtin_clzll(m)) * step;  // lane 0 always holds
    lo += j;
    len = min(step, len - j);
  }
  return lo;
}

// One step of the expansion: the entries [e0, lim) of the window in R, U * 64
// of them at most (plain: claims normals; else dd entries claim delegates, dn
// entries normals). R.beg[o] + e is entry e's column, R.mid[o] where row o's
// dn part begins.
template <bool plain, int U>
__device__ __forceinline__ void list_step(const Search &a, const WaveRows &R, int64_t ew,
                                          int64_t e0, int64_t lim, int32_t dep, WaveAppend &qa,
                                          uint32_t &cl_n, uint32_t &cl_d, uint32_t &with_dn) {
  const int l = lane_id();
  int32_t x[U];
  int o[U];
  bool ok[U], dd[U];
  uint32_t wd[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int64_t e = e0 + u * kWave + l;
    ok[u] = e < lim;
    const int64_t ec = ok[u] ? e : lim - 1;
    o[u] = owner64(R.excl, int32_t(ec - ew));
    dd[u] = !plain && ec < R.mid[o[u]];
    x[u] = (plain ? a.pcol : a.dcol)[R.beg[o[u]] + ec];
  }
#pragma unroll
  for (int u = 0; u < U; ++u) wd[u] = (dd[u] ? a.Cd : a.Vn)[uint32_t(x[u]) >> 5];
  if (plain) {
    // columns by neighbour degree: no two lanes share a word by design
    uint32_t old[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t b = 1u << (x[u] & 31);
      old[u] = b;
      if (ok[u] && !(wd[u] & b)) old[u] = atomicOr(&a.Vn[uint32_t(x[u]) >> 5], b);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool won = !(old[u] & (1u << (x[u] & 31)));
      if (won) {
        a.put(x[u], R.aux[o[u]], dep);
        ++cl_n;
      }
      qa.push(won, x[u]);
    }
    return;
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    // claims: the word read above first (most edges lead to vertices already
    // claimed), then one atomic per run of lanes sharing a bitmap word (dn
    // parts are ascending)
    const bool want = ok[u] && !((wd[u] >> (x[u] & 31)) & 1u);
    if (__ballot(want && dd[u])) {
      if (wave_bit_claim(a.Cd, uint32_t(x[u]), ok[u] && dd[u], want && dd[u])) {
        a.put_deleg(x[u], R.aux[o[u]], dep);
        with_dn += bit_test(a.dnm, uint32_t(x[u]));
        ++cl_d;
      }
    }
    if (__ballot(want && !dd[u])) {
      const bool won = wave_bit_claim(a.Vn, uint32_t(x[u]), ok[u] && !dd[u], want && !dd[u]);
      if (won) {
        a.put(x[u], R.aux[o[u]], dep);
        ++cl_n;
      }
      qa.push(won, x[u]);
    }
  }
}

// Top-down over the listed rows, balanced over edges: every wave takes one
// contiguous share of the concatenated rows. It finds the first row by search
// and then stages 64 rows at a time in LDS (prefix, first column, parent); a
// step finds its entries' rows there. Steps of four column loads, tests and
// atomics in flight, as in the normal expansion: a step alone is a chain of
// round trips.
template <bool plain, int NW>
__device__ void expand_list(const Search &a, Scratch<NW> &S, int L, uint32_t &with_dn) {
  const int ns = list_segs();
  const int l = lane_id(), w = threadIdx.x / kWave, nw = blockDim.x / kWave;
  // exclusive prefix of the segment lengths
  {
    int64_t run = 0;
    for (int i0 = 0; i0 < ns; i0 += blockDim.x) {
      const int i = i0 + threadIdx.x;
      int64_t all;
      const int64_t at = run + block_scan(S, i < ns ? a.ctl->seg_len[i] : 0, &all);
      if (i < ns) S.seg[i] = at;
      run += all;
    }
    if (threadIdx.x == 0) S.seg[ns] = run;
    __syncthreads();
  }
  const int64_t E = S.seg[ns];
  const int64_t nwaves = int64_t(gridDim.x) * nw;
  const int64_t share = ((E + nwaves - 1) / nwaves + kWave - 1) / kWave * kWave;
  const int64_t eb = (int64_t(blockIdx.x) * nw + w) * share, ee = min(E, eb + share);
  const int32_t *const list = plain ? a.q(L & 1) : a.dlist;
  const int64_t stride = plain ? plain_seg(S.qn, ns) : (int64_t(a.dwords) + ns - 1) / ns * 32;
  WaveRows &R = S.w[w];
  WaveAppend qa = wave_append_buf(S, &a.ctl->ctr[L % 3].qn_nc.v, a.q((L + 1) & 1));
  const int dd_td = !plain && S.plan.dd_td;
  uint32_t cl_n = 0, cl_d = 0;
  for (int64_t e = eb; e < ee;) {
    // segment of e (the last one starting at or before it; empty ones share
    // their start with the next)
    int sg = 0;
    for (int step = kSegs / 2; step > 0; step >>= 1)
      if (sg + step < ns && S.seg[sg + step] <= e) sg += step;
    const int64_t s0 = S.seg[sg], s1 = S.seg[sg + 1];
    const int64_t lim = min(ee, s1) - s0;
    const int64_t base = sg * stride, cnt = a.ctl->seg_cnt[sg];
    int64_t own = wave_search(a.dscan + base, cnt, e - s0);
    for (int64_t ew = e - s0; ew < lim;) {
      const int64_t i = own + l;
      const bool in = i < cnt;
      int32_t u = 0;
      int64_t pre = 0, beg = 0, mid = 0;
      if (in) {
        u = list[base + i];
        pre = a.dscan[base + i];
        if (plain) {
          beg = a.poff[u] - pre;
        } else {
          const uint64_t x0 = a.doff[u];
          const int64_t dd = row_first(x0);
          beg = row_start(x0) + (dd_td ? 0 : dd) - pre;
          mid = dd_td ? pre + dd : 0;
          u = a.vid_of[u];
        }
      }
      const int64_t wend = own + kWave < cnt ? a.dscan[base + own + kWave] : s1 - s0;
      const int64_t stop = min(lim, wend);
      wave_sync();
      // a row that began before ew has a negative prefix (rows are shorter
      // than 2^24 entries, 64 of them sum below 2^31)
      R.excl[l] = in ? int32_t(pre - ew) : INT32_MAX;
      R.aux[l] = u;
      R.beg[l] = beg;
      R.mid[l] = mid;
      wave_sync();
      int64_t p = ew;
      for (; stop - p > 2 * kWave; p += 4 * kWave)
        list_step<plain, 4>(a, R, ew, p, stop, L + 1, qa, cl_n, cl_d, with_dn);
      for (; p < stop; p += kWave)
        list_step<plain, 1>(a, R, ew, p, stop, L + 1, qa, cl_n, cl_d, with_dn);
      ew = stop;
      own += kWave;
    }
    e = s0 + lim;
  }
  qa.flush();
  const uint32_t edges = l == 0 && eb < ee ? uint32_t(ee - eb) : 0u;
  if (plain) {
    // units: queue entries (counted by the caller), edges, claimed
    count_units(a, S, DSBFS_K_PLAIN, 0, edges, cl_n, 0);
  } else {
    // units: -, edges, normals claimed, delegates claimed
    count_units(a, S, DSBFS_K_TD_DELEG, 0, edges, cl_n, cl_d);
  }
}

// ---------------------------------------------------------------------------
// forward visits of the normal queue
// ---------------------------------------------------------------------------
// Top-down nd (levels where nd goes forward), and nn when it is under the
// direction decision and goes forward.
template <int NW, int parts>
__device__ void td_normal(const Search &a, Scratch<NW> &S, int L, uint32_t &with_dn) {
  const int64_t qn = S.plan.qn;
  const int nd_td = (parts & kNormal) && S.plan.nd_td, nn_td = (parts & kNn) && S.plan.nn_td;
  if (!nd_td && !nn_td) return;
  const QueueShare sh = queue_share(a, qn);
  if (sh.none(qn)) return;
  const int l = lane_id();
  const int32_t *const Q = a.q(L & 1);
  WaveRows &R = S.w[threadIdx.x / kWave];
  WaveAppend qa = wave_append_buf(S, &a.ctl->ctr[L % 3].qn_nc.v, a.q((L + 1) & 1));
  uint32_t nd_e = 0, nd_c = 0, nn_e = 0, nn_c = 0, none = 0;
  for (int64_t i0 = sh.first; i0 < qn; i0 += sh.stride) {
    const int64_t i = i0 + l;
    const bool ok = l < sh.rows && i < qn;
    const int32_t u = ok ? Q[i] : 0;
    if (nd_td) {
      int32_t len = 0;
      int64_t beg = 0;
      if (ok) {
        const uint64_t w0 = a.noff[u], w1 = a.noff[u + 1];
        beg = row_start(w0) + row_first(w0);
        len = int32_t(row_start(w1) - beg);
      }
      expand_rows<false>(a, R, a.ncol, u, len, beg, L + 1, qa, nd_e, nd_c, with_dn);
    }
    if (nn_td) {
      int32_t nn = 0;
      int64_t nd = 0, beg = 0;
      if (ok) nn_part(a, u, true, nn, nd, beg);
      expand_rows<true>(a, R, a.nnoff ? a.nncol : a.ncol, u, nn, beg, L + 1, qa, nn_e, nn_c,
                        none);
    }
  }
  qa.flush();
  // units: -, edges, -, delegates claimed / -, edges, normals claimed, -
  if (nd_td) count_units(a, S, DSBFS_K_TD_NORMAL, 0, nd_e, 0, nd_c);
  if (nn_td) count_units(a, S, DSBFS_K_TD_NN, 0, nn_e, nn_c, 0);
}

// Forward visits of level L, of the parts asked for.
template <int NW, int parts>
__device__ __forceinline__ void forward(const Search &a, Scratch<NW> &S, int L) {
  uint32_t with_dn = 0;
  if (parts & (kNormal | kNn)) td_normal<NW, parts>(a, S, L, with_dn);
  __syncthreads();
  if ((parts & kDeleg) && (S.plan.dd_td || S.plan.dn_td)) expand_list<false>(a, S, L, with_dn);
  block_acc(&S.red[kClDn], with_dn);
  red_flush(S, a.ctl->ctr[L % 3], kClDn, kClDn + 1);
}

// ---------------------------------------------------------------------------
// bottom-up visits
// ---------------------------------------------------------------------------
// Walks the concatenated rows of a wave's 64 candidates (R.excl, R.beg set,
// lane l's row has len entries), 64 entries per step, until every row has a
// hit or ends: R.aux[l] gets the first hit of row l (an index into the
// concatenation), kNone if there is none. hit(o, q) tests entry q of row o.
constexpr int32_t kNone = 0x7fffffff;
template <class F>
__device__ __forceinline__ void walk_rows(WaveRows &R, int32_t T, int32_t len, uint32_t &edges,
                                          F &&hit) {
  const int l = lane_id();
  uint64_t remaining = __ballot(len > 0);
  for (int32_t e0 = 0; e0 < T && remaining; e0 += kWave) {
    const int32_t e = e0 + l;
    if (e < T) {
      const int o = owner64(R.excl, e);
      // a row whose parent an earlier step found is not read further: a scan
      // stops at its first frontier neighbour (Section IV-B)
      if (R.aux[o] == kNone) {
        ++edges;
        if (hit(o, R.beg[o] + (e - R.excl[o]))) atomicMin(&R.aux[o], e);
      }
    }
    wave_sync();
    remaining = __ballot(len > 0 && R.aux[l] == kNone);
  }
}

// Bottom-up nn (nn_do, levels where nn goes backward): every normal vertex
// with an nn edge that is still unvisited scans its nn part (ascending IDs)
// for a vertex of the level's normal frontier Fn, stopping at the first. A
// candidate is one lane's and no other visit claims normals meanwhile, so
// claims set bits without reading them back.
template <int NW> __device__ void bu_nn(const Search &a, Scratch<NW> &S, int L) {
  const uint32_t *const Fn = a.fn(L & 1);
  WaveRows &R = S.w[threadIdx.x / kWave];
  WaveAppend qa = wave_append_buf(S, &a.ctl->ctr[L % 3].qn_nc.v, a.q((L + 1) & 1));
  const int l = lane_id();
  uint32_t reads = 0, scanned = 0, edges = 0, claimed = 0;
  for (int64_t b0 = int64_t(blockIdx.x) * blockDim.x; b0 < a.n_nnsrc;
       b0 += int64_t(gridDim.x) * blockDim.x) {
    const int64_t i = b0 + threadIdx.x;
    const bool ok = i < a.n_nnsrc;
    int32_t v = 0, len = 0;
    int64_t beg = 0;
    if (ok) {
      v = a.nnsrc[i];
      ++reads;
      if (!bit_test(a.Vn, uint32_t(v))) {
        ++scanned;
        const uint32_t lw = a.nlen[v];
        const uint64_t w0 = a.noff[v];
        beg = row_start(w0);
        len = lw == kLenWide ? int32_t(row_first(w0)) : int32_t(lw & 0xFFu);
      }
    }
    const int32_t incl = wave_incl_scan(len);
    const int32_t T = lane_read(incl, kWave - 1);
    wave_sync();
    R.excl[l] = incl - len;
    R.beg[l] = beg;
    R.aux[l] = kNone;
    wave_sync();
    walk_rows(R, T, len, edges,
              [&](int, int64_t q) { return bit_test(Fn, uint32_t(a.ncol[q])); });
    const int32_t fe = R.aux[l];
    const bool won = ok && len > 0 && fe != kNone;
    wave_bit_set(a.Vn, uint32_t(v), ok, won);
    if (won) {
      a.put(v, a.ncol[beg + (fe - (incl - len))], L + 1);
      ++claimed;
    }
    qa.push(won, v);
  }
  qa.flush();
  // units: list entries read, unvisited scanned, edges inspected, claimed
  count_units(a, S, DSBFS_K_BU_NN, reads, scanned, edges, claimed);
}

// Bottom-up dn (destination: normal vertices). Candidates are positions in
// the nd source list; row p of the source-list-ordered nd copy holds the
// delegate neighbours of ndsrc[p]. Each wave takes 64 candidates, drops the
// visited ones, and walks the concatenation of the remaining rows
// (consecutive candidates have consecutive rows, so the first pass over the
// whole list streams them). Candidates still unvisited are compacted (as
// positions) for the next bottom-up level.
template <int NW> __device__ void bu_normal(const Search &a, Scratch<NW> &S, int L) {
  // first pass: every position of the nd source list (dense); later passes:
  // the positions the previous pass left unvisited
  const int dense = S.plan.cin_sel < 0;
  const int32_t *const cin = a.cand(S.plan.cin_sel);
  const int64_t nc = S.plan.nc;
  constexpr int cap = Scratch<NW>::kCap;
  unsigned long long *const tails = &a.ctl->ctr[L % 3].qn_nc.v;
  BlockAppend qa{S.buf, &S.qcount, &S.qbase, cap, tails, a.q((L + 1) & 1)};
  BlockAppend ca{S.buf + cap, &S.ccount, &S.cbase, cap, tails, a.cand(S.plan.cout_sel), 32};
  qa.init();
  ca.init();
  __syncthreads();
  WaveRows &R = S.w[threadIdx.x / kWave];
  const int l = lane_id();
  uint32_t reads = 0, scanned = 0, edges = 0, claimed = 0;
  for (int64_t b0 = int64_t(blockIdx.x) * blockDim.x; b0 < nc;
       b0 += int64_t(gridDim.x) * blockDim.x) {
    const int64_t i = b0 + threadIdx.x;
    const bool ok = i < nc;
    int32_t pos = 0, v = 0, len = 0;
    int64_t beg = 0;
    bool visited = true;
    int32_t hit0 = -1;  // delegate found at the first entry of the row
    int32_t pk0 = 0;    // vertex of the row's first delegate (its parent if it is a hit)
    if (ok) {
      pos = dense ? int32_t(i) : cin[i];
      // The loads are ordered to keep the chain of dependent accesses short:
      // the vertex and its row bounds both depend on pos only; the row's
      // first entry (rows in the list are never empty) does not wait for the
      // visited test, and the parent candidate is fetched beside the
      // frontier test.
      v = a.ndsrc[pos];
      // Rows start with their highest-degree delegate, the likeliest to be in
      // the frontier: a hit there skips the wave's walk for this row. The
      // first entry and its vertex come from a dense array (8 bytes per
      // candidate, read in list order); its frontier bit is tested whether
      // or not the candidate turns out to be visited, so that the loads
      // overlap the visited test instead of following it.
      const int2 f = a.nds_first[pos];
      const int32_t k0 = f.x;
      pk0 = f.y;
      const bool f0 = bit_test(a.Fd, uint32_t(k0));
      ++reads;
      visited = bit_test(a.Vn, uint32_t(v));
      hit0 = (!visited && f0) ? k0 : -1;
      scanned += !visited;
      edges += !visited;
      if (!visited && !f0) {
        // a miss: the rest of the row is walked below
        beg = a.nds_off[pos] + 1;
        len = int32_t(a.nds_off[pos + 1] - beg);
      }
    }
    const int32_t incl = wave_incl_scan(len);
    const int32_t T = lane_read(incl, kWave - 1);
    wave_sync();
    R.excl[l] = incl - len;
    R.beg[l] = beg;
    R.aux[l] = kNone;
    wave_sync();
    walk_rows(R, T, len, edges,
              [&](int, int64_t q) { return bit_test(a.Fd, uint32_t(a.nds_col[q])); });
    const int32_t fe = R.aux[l];
    const bool found = hit0 >= 0 || (len > 0 && fe != kNone);
    // A vertex is the candidate of one lane only, and no other visit claims
    // normal vertices meanwhile (the level's forward visits are complete), so
    // a found candidate is this lane's: its bit is set without waiting for
    // the atomic's old value. Candidates are ascending: set word by word.
    const bool won = ok && found;
    wave_bit_set(a.Vn, uint32_t(v), ok, won);
    if (won) {
      a.put_pos(pos, v, hit0 >= 0 ? pk0 : a.vid_of[a.nds_col[beg + (fe - (incl - len))]], L + 1);
      ++claimed;
    }
    qa.push(won, v);
    ca.push(ok && !visited && !found, pos);
    flush_pair_if_full(qa, ca, int(blockDim.x));
  }
  flush_pair(qa, ca);
  // units: list entries read, unvisited scanned, edges inspected, claimed
  count_units(a, S, DSBFS_K_BU_NORMAL, reads, scanned, edges, claimed);
}

// Bottom-up dd and/or nd (destination: delegates): unclaimed delegates with
// an edge in a subgraph scanned bottom-up this level. A wave takes a few bytes
// of the masks and enumerates their candidates 64 at a time, one per lane, so no
// candidate list is written. Each lane first tests the first entry of its
// scanned range (dd parts start with their highest-degree neighbour, the
// likeliest to be in the frontier); the rows that miss are then walked
// together. dd entries are tested against Fd, dn entries against the normal
// frontier bitmap Fn. The bytes are this wave's alone: claims are collected in
// LDS and the byte stored once. Bytes, not words, so that few delegates still
// spread over the waves: a wave walks its candidates' rows in a chain of steps
// (a search of 2^12 vertices: 43 of its 127 us with 64 delegates a wave,
// 14 of 95 with eight).
template <int NW> __device__ void bu_deleg(const Search &a, Scratch<NW> &S, int L,
                                           uint32_t &with_dn) {
  const int dd_bu = S.plan.dd_bu, nd_bu = S.plan.nd_bu;
  const uint32_t *const Fn = a.fn(L & 1);
  const int l = lane_id();
  const int64_t nwaves = int64_t(gridDim.x) * (blockDim.x / kWave);
  const int64_t wid = int64_t(blockIdx.x) * (blockDim.x / kWave) + threadIdx.x / kWave;
  const int32_t dbytes = a.dwords * 4;
  const int cw = mask_step(dbytes, nwaves, 1);
  uint8_t *const Cd = reinterpret_cast<uint8_t *>(a.Cd);
  const uint8_t *const ddm = reinterpret_cast<const uint8_t *>(a.ddm);
  const uint8_t *const dnms = reinterpret_cast<const uint8_t *>(a.dnm);
  WaveRows &R = S.w[threadIdx.x / kWave];
  // this wave's part of the append buffers: mask words and their prefix, and
  // the bits claimed
  int32_t *const wpre = S.buf + (threadIdx.x / kWave) * (3 * kWave);
  int32_t *const wbits = wpre + kWave;
  unsigned int *const wgot = reinterpret_cast<unsigned int *>(wpre + 2 * kWave);
  uint32_t cands = 0, edges = 0, claimed = 0;
  for (int64_t w0 = wid * cw; w0 < dbytes; w0 += nwaves * cw) {
    const int64_t w = w0 + l;
    uint32_t c = 0, cd = 0, dnm = 0;
    if (l < cw && w < dbytes) {
      cd = Cd[w];
      dnm = dnms[w];
      c = ~cd & ((dd_bu ? ddm[w] : 0u) | (nd_bu ? dnm : 0u));
    }
    const int32_t pc = __popc(c);
    const int32_t pincl = wave_incl_scan(pc);
    const int32_t total = lane_read(pincl, kWave - 1);
    if (total == 0) continue;
    wave_sync();
    wpre[l] = pincl - pc;
    wbits[l] = int32_t(c);
    wgot[l] = 0;
    wave_sync();
    for (int32_t i0 = 0; i0 < total; i0 += kWave) {
      const int32_t i = i0 + l;
      const bool ok = i < total;
      int32_t k = 0, len = 0, px = 0;
      int64_t p = 0, mid = 0, hit = -1;
      int wo = 0, bit = 0;
      if (ok) {
        wo = owner64(wpre, i);
        bit = nth_bit(uint32_t(wbits[wo]), i - wpre[wo]);
        k = int32_t((w0 + wo) * 8 + bit);
        const uint64_t x0 = a.doff[k], x1 = a.doff[k + 1];
        const int2 f = a.dd_first[k];  // fetched beside the row bounds
        const int64_t beg = row_start(x0);
        mid = beg + row_first(x0);
        p = dd_bu ? beg : mid;
        const int64_t hi = nd_bu ? row_start(x1) : mid;
        if (p < hi) {
          ++cands;
          const bool in_dd = p < mid;
          const int32_t x = in_dd ? f.x : a.dcol[p];
          ++edges;
          px = in_dd ? f.y : x;  // the parent if this entry is a hit
          if (in_dd ? bit_test(a.Fd, uint32_t(x)) : bit_test(Fn, uint32_t(x))) hit = p;
          else ++p;
          // delegate degrees are below 2^24, so 64 rows sum below 2^31
          if (hit < 0) len = int32_t(hi - p);
        }
      }
      const bool probe_hit = hit >= 0;
      const int32_t incl = wave_incl_scan(len);
      const int32_t T = lane_read(incl, kWave - 1);
      if (T > 0) {
        wave_sync();
        R.excl[l] = incl - len;
        R.beg[l] = p;
        R.mid[l] = mid;
        R.aux[l] = kNone;
        wave_sync();
        walk_rows(R, T, len, edges, [&](int o, int64_t q) {
          const uint32_t x = uint32_t(a.dcol[q]);
          return q < R.mid[o] ? bit_test(a.Fd, x) : bit_test(Fn, x);
        });
        const int32_t fe = R.aux[l];
        if (len > 0 && fe != kNone) hit = p + (fe - (incl - len));
      }
      if (ok && hit >= 0) {
        atomicOr(&wgot[wo], 1u << bit);
        int32_t par = px;
        if (!probe_hit) {
          const int32_t x = a.dcol[hit];
          par = hit < mid ? a.vid_of[x] : x;
        }
        a.put_deleg(k, par, L + 1);
        ++claimed;
      }
    }
    wave_sync();
    const uint32_t got = wgot[l];
    if (got) {
      Cd[w] = uint8_t(cd | got);
      with_dn += __popc(got & dnm);
    }
  }
  // units: candidates scanned, edges inspected, claimed
  count_units(a, S, DSBFS_K_BU_DELEG, cands, edges, claimed, 0);
}

// Bottom-up dn and dd/nd of level L, of the parts asked for. They touch
// different bitmaps (Vn and the queues; Cd), so one phase runs both.
template <int NW, int parts>
__device__ __forceinline__ void backward(const Search &a, Scratch<NW> &S, int L) {
  uint32_t with_dn = 0;
  if ((parts & kNormal) && S.plan.dn_bu) bu_normal(a, S, L);
  __syncthreads();
  if ((parts & kDeleg) && (S.plan.dd_bu || S.plan.nd_bu)) {
    bu_deleg(a, S, L, with_dn);
    block_acc(&S.red[kClDn], with_dn);
    red_flush(S, a.ctl->ctr[L % 3], kClDn, kClDn + 1);
  }
}
// ---------------------------------------------------------------------------
// level by level: one kernel per phase
// ---------------------------------------------------------------------------
// Every per-level kernel is a grid-stride loop over a bounded grid (8
// workgroups per CU), reads the level's state and returns at once when its
// plan has no work. Host launches run one level ahead of the device.
constexpr int kBS = 256;
constexpr int kNW = kBS / kWave;

// Loads the state of level L into the block; false if the search has ended.
template <int NW>
__device__ __forceinline__ bool level_enter(const Search &a, Scratch<NW> &S, int L) {
  const uint32_t *from = reinterpret_cast<const uint32_t *>(&a.ctl->st[L & 1]);
  uint32_t *to = reinterpret_cast<uint32_t *>(&S.st);
  for (int i = threadIdx.x; i < int(sizeof(LevelState) / 4); i += blockDim.x) to[i] = from[i];
  units_open(a, S);
  if (S.st.done) return false;
  level_open(a, S, L);
  return true;
}

template <int parts>
__global__ void __launch_bounds__(kBS, 8) k_previsit(Search a, int L) {
  __shared__ Scratch<kNW> S;
  if (!level_enter(a, S, L)) return;
  previsit<kNW, parts>(a, S, L);
  units_close(a, S);
}

__global__ void __launch_bounds__(kBS, 8) k_list(Search a, int L) {
  __shared__ Scratch<kNW> S;
  if (!level_enter(a, S, L)) return;
  level_plan(a, S, L);
  if (S.plan.dd_td || S.plan.dn_td) list_deleg(a, S);
}

template <int parts>
__global__ void __launch_bounds__(kBS, 8) k_forward(Search a, int L) {
  __shared__ Scratch<kNW> S;
  if (!level_enter(a, S, L)) return;
  level_plan(a, S, L);
  if (S.ns.done) return;
  forward<kNW, parts>(a, S, L);
  units_close(a, S);
}

__global__ void __launch_bounds__(kBS, 8) k_bu_nn(Search a, int L) {
  __shared__ Scratch<kNW> S;
  if (!level_enter(a, S, L)) return;
  level_plan(a, S, L);
  if (!S.plan.nn_bu) return;
  bu_nn(a, S, L);
  units_close(a, S);
}

// Publishes a level's record to the host: the record, then its sequence number.
template <int NW>
__device__ void publish(const Search &a, const LevelStatus &rec, int L) {
  __syncthreads();
  LevelStatus *const to = a.hs + (L & (kStatusSlots - 1));
  const uint32_t *f = reinterpret_cast<const uint32_t *>(&rec);
  uint32_t *t = reinterpret_cast<uint32_t *>(to);
  for (int i = threadIdx.x; i < int(offsetof(LevelStatus, seq) / 4); i += blockDim.x) t[i] = f[i];
  __threadfence_system();
  __syncthreads();
  if (threadIdx.x == 0)
    __hip_atomic_store(&to->seq, L + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The level's last kernel: bottom-up visits; with kCommit, block 0 also
// commits the state of the next level and publishes this level's record.
template <int parts>
__global__ void __launch_bounds__(kBS, 8) k_backward(Search a, int L) {
  __shared__ Scratch<kNW> S;
  LevelStatus &rec = *reinterpret_cast<LevelStatus *>(S.seg);  // segments are not used here
  const bool commit = (parts & kCommit) && blockIdx.x == 0;
  if (!level_enter(a, S, L)) {
    // levels launched behind the last one: the end stays visible to both slots
    if (commit && threadIdx.x == 0) a.ctl->st[(L + 1) & 1].done = 1;
    return;
  }
  level_plan(a, S, L, commit ? &rec : nullptr);
  if (commit) {
    if (threadIdx.x == 0) {
      a.ctl->st[(L + 1) & 1] = S.ns;
      if (a.count) account_level(a, S.st, S.ns, S.now, S.qn, S.nc_prev, S.plan, a.ctl->tot);
    }
    publish<kNW>(a, rec, L);
  }
  if (S.ns.done) return;
  backward<kNW, parts>(a, S, L);
  units_close(a, S);
}

// Mode 0, one level: the queue's degrees, then the expansion.
template <int NW> __device__ __forceinline__ bool plain_open(const Search &a, Scratch<NW> &S, int L) {
  if (threadIdx.x == 0) {
    S.qn = int64_t(ctr_load(&a.ctl->ctr[(L + 2) % 3].qn_nc.v) & 0xffffffffull);
    S.plan = Plan{};
  }
  __syncthreads();
  return S.qn > 0;
}
__global__ void __launch_bounds__(kBS, 8) k_plain_list(Search a, int L) {
  __shared__ Scratch<kNW> S;
  ctr_clear(a.ctl->ctr[(L + 1) % 3]);
  if (plain_open(a, S, L)) list_plain(a, S, L);
}

__global__ void __launch_bounds__(kBS, 8) k_plain_expand(Search a, int L) {
  __shared__ Scratch<kNW> S;
  LevelStatus &rec = *reinterpret_cast<LevelStatus *>(S.seg);  // before the segments
  units_open(a, S);
  const bool work = plain_open(a, S, L);
  if (blockIdx.x == 0) {
    for (int i = threadIdx.x; i < int(sizeof(LevelStatus) / 4); i += blockDim.x)
      reinterpret_cast<uint32_t *>(&rec)[i] = 0;
    __syncthreads();
    if (threadIdx.x == 0) {
      rec.done = !work;
      rec.level = L;
      rec.rec.frontier_normal = S.qn;
      if (a.count && work) {
        a.ctl->tot.units0[DSBFS_K_PLAIN] += S.qn;
        ++a.ctl->tot.launches[DSBFS_K_PLAIN];
      }
    }
    publish<kNW>(a, rec, L);
    __syncthreads();
  }
  if (!work) return;
  uint32_t none = 0;
  expand_list<true>(a, S, L, none);
  units_close(a, S);
}

// ---------------------------------------------------------------------------
// one launch: all levels of a search in one resident grid
// ---------------------------------------------------------------------------
// For graphs whose levels are a few microseconds of work: a kernel boundary
// costs 4.5 us (12 kernels and a 13 us graph hand-over per level before:
// of the 642 us of an RMAT 22 search 380 were dispatch), a grid barrier of 64 wide
// blocks 2.5 us and there are two or three per level. Every block follows the
// search's state by itself, so a level needs no other exchange than its
// counters.
constexpr int kWideNW = 16;
constexpr double kHeavyEdges = 1 << 18;

// A launch ends after this many levels, and the host launches the next: between
// them a batch that waits for compute units gets them. A path of 30000 vertices
// kept one waiting for a quarter of a second. Most graphs have fewer levels; a
// launch more is some 15 us after 2 ms.
constexpr int kLaunchLevels = 252;
static_assert(kLaunchLevels % 6 == 0, "see Search::level0");

// How block 0 left: kDone, kGaveUp where a barrier wait exceeded its bound, kGoOn
// with levels left.
enum { kDone = 1, kGoOn = 2, kGaveUp = -1 };
__device__ __forceinline__ void one_launch_end(const Search &a, int how, int levels) {
  if (blockIdx.x != 0) return;
  __syncthreads();
  if (threadIdx.x == 0) {
    a.ctl->levels = levels;
    a.hs->level = levels;
    __threadfence_system();
    __hip_atomic_store(&a.hs->seq, how, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// Whether a level's nn visit scatters (scatter_step): its edges to unvisited
// vertices, as the mean nn row and the share of normals left predict them, are
// at least n / 16 + 2^18. settle() reads and writes about 12 bytes a vertex and
// costs a barrier, 8 us and 7 per million vertices; an edge saves an atomic for
// a store, 26 us per million. ER 2^22 with n / 4, n / 16, n / 16 + 2^18, n / 16 +
// 2^20: 1448, 1409, 1412, 1485 us (1812 without); the smaller lines without the
// constant cost searches of 2^17 vertices 3%.
__device__ __forceinline__ bool heavy_level(const Search &a, int64_t qn, int64_t left) {
  const double n = a.n;
  return double(qn) * a.nn_mean * double(left) >= n * (n / 16 + kHeavyEdges);
}

// HEAVY: levels may scatter (heavy_graph()).
template <bool HEAVY> __global__ void __launch_bounds__(1024) k_search(Search a) {
  __shared__ Scratch<kWideNW> S;
  GridBar &bar = a.ctl->bar;
  grid_start(bar);
  if (threadIdx.x == 0) S.st = a.ctl->st[0];
  units_open(a, S);
  unsigned long long ep = 0;
  int L = 0;
  bool ok = true;
  // normals in no frontier so far
  int64_t left = HEAVY && a.level0 > 0 ? a.ctl->left : int64_t(a.n) - a.d;
  for (; L < kLaunchLevels; ++L) {
    level_open(a, S, L);
    left -= S.qn;
    const bool heavy = HEAVY && heavy_level(a, S.qn, left);
    previsit<kWideNW, kDeleg | kNormal | kClear>(a, S, L, heavy);
    if (!(ok = grid_sync(bar, ++ep, &S.ok, a.bar_ticks))) break;
    level_plan(a, S, L);
    if (a.count && blockIdx.x == 0 && threadIdx.x == 0)
      account_level(a, S.st, S.ns, S.now, S.qn, S.nc_prev, S.plan, a.ctl->tot);
    if (S.ns.done) break;
    const Plan &p = S.plan;
    if (heavy) settle(a, S, L);
    if (p.dd_td || p.dn_td) list_deleg(a, S);
    if (heavy || p.dd_td || p.dn_td) {
      if (!(ok = grid_sync(bar, ++ep, &S.ok, a.bar_ticks))) break;
    }
    if (p.dd_td || p.dn_td || p.nd_td || p.nn_td) {
      forward<kWideNW, kDeleg | kNormal | kNn>(a, S, L);
      if (!(ok = grid_sync(bar, ++ep, &S.ok, a.bar_ticks))) break;
    }
    if (p.nn_bu) {
      bu_nn(a, S, L);
      if (!(ok = grid_sync(bar, ++ep, &S.ok, a.bar_ticks))) break;
    }
    if (p.dn_bu || p.dd_bu || p.nd_bu) {
      backward<kWideNW, kDeleg | kNormal>(a, S, L);
      if (!(ok = grid_sync(bar, ++ep, &S.ok, a.bar_ticks))) break;
    }
    __syncthreads();
    if (threadIdx.x == 0) S.st = S.ns;
    __syncthreads();
  }
  units_close(a, S);
  const bool more = ok && L == kLaunchLevels;
  if (more && blockIdx.x == 0 && threadIdx.x == 0) {
    a.ctl->st[0] = S.st;
    a.ctl->left = left;
  }
  one_launch_end(a, more ? kGoOn : ok ? kDone : kGaveUp, a.level0 + L);
}

__global__ void __launch_bounds__(1024) k_plain_search(Search a) {
  __shared__ Scratch<kWideNW> S;
  GridBar &bar = a.ctl->bar;
  grid_start(bar);
  unsigned long long ep = 0;
  units_open(a, S);
  int L = 0;
  bool ok = true;
  for (; L < kLaunchLevels; ++L) {
    if (!plain_open(a, S, L)) break;
    ctr_clear(a.ctl->ctr[(L + 1) % 3]);
    if (a.count && blockIdx.x == 0 && threadIdx.x == 0) {
      a.ctl->tot.units0[DSBFS_K_PLAIN] += S.qn;
      ++a.ctl->tot.launches[DSBFS_K_PLAIN];
    }
    list_plain(a, S, L);
    if (!(ok = grid_sync(bar, ++ep, &S.ok, a.bar_ticks))) break;
    uint32_t none = 0;
    expand_list<true>(a, S, L, none);
    if (!(ok = grid_sync(bar, ++ep, &S.ok, a.bar_ticks))) break;
  }
  units_close(a, S);
  one_launch_end(a, !ok ? kGaveUp : L == kLaunchLevels ? kGoOn : kDone, a.level0 + L);
}

// Before a launch that goes on: the barrier as at the first one's start.
__global__ void k_clear_bar(GridBar *bar) {
  uint32_t *const w = reinterpret_cast<uint32_t *>(bar);
  for (int i = threadIdx.x; i < int(sizeof(GridBar) / 4); i += blockDim.x) w[i] = 0;
}

// Number of resident waves worth of blocks for grid-stride kernels.
int stride_grid() { return 256 * 8; }

// Shape of a one-launch search (blocks = 0: level by level instead). A barrier
// costs more the more blocks there are, a level's work less the more waves, so
// the grid grows with the graph. Measured (us a search, RMAT edge factor 16,
// parents; 32x256 / 64x256 / 64x512 / 128x512 / 128x1024 / 256x512 / 256x1024 /
// level by level):
//   n = 2^12   125 /  127 /  128 / 136 / 143 / 154 / 162 / 188
//   n = 2^14   118 /  117 /  118 / 128 / 135 / 148 / 155 / 187
//   n = 2^15   141 /  133 /  130 / 136 / 144 / 158 / 167 / 192
//   n = 2^17   170 /  151 /  143 / 148 / 155 / 169 / 179 / 212
//   n = 2^18   491 /  349 /  279 / 250 / 231 / 246 / 246 / 297
//   n = 2^20   594 /  389 /  301 / 260 / 261 / 271 / 282 / 357
//   n = 2^21  1023 /  605 /  425 / 328 / 294 / 304 / 300 / 379
//   n = 2^22  1857 / 1020 /  643 / 429 / 354 / 353 / 329 / 398
//   n = 2^23  4431 / 2310 / 1386 / 831 / 613 / 583 / 488 / 527
//   n = 2^24  9663 / 4999 / 2909 / 1695 / 1252 / 1144 / 908 / 854
// ER, mean degree 16, n = 2^20  1453 / 843 / 618 / 444 / 424 / 393 / 396 / 748
// Plain top-down searches read every edge, about four times the work a vertex:
//   n = 2^16  264 / 206 / 181 / 186 / - / 224 / 292 / 284
//   n = 2^20 3728 / 2058 / 1457 / 1030 / - / 903 / 943 / 957
// Denser graphs take the shape of a larger one (m directed edges; the same columns):
//   plain, n = 2^14, m = 23M   949 /  534 /  359 /  289 / 289 / 330 / 371 / 316
//   plain, ER 2^14, m = 106M  4423 / 2257 / 1248 /  711 / 506 / 481 / 404 / 346
//   plain, ER 2^18, m = 134M  6126 / 3133 / 1875 / 1025 / 979 / 650 / 684 / 750
// where all of them are read, that is in plain searches and in those that stay
// top-down; a direction-optimized search of a graph with hubs reads few of them,
// however many there are, but one of a uniform graph scans long rows before it
// meets its frontier:
//   RMAT 2^14, m = 23M          93 /   91 /   93 /  102 / 108 / 118 / 126 / 161
//   ER 2^14, m = 32M          1208 /  673 /  387 /  240 / 165 / 169 / 179 / 205
//   ER 2^16, m = 132M         5525 / 2837 / 1504 /  807 / 473 / 456 / 290 / 243
//   ER 2^20, m = 134M        14180 / 7145 / 3972 / 2081 / 1270 / 1138 / 746 / 671
struct OneLaunch {
  int blocks, threads;
};

// Whether the search's levels may scatter: nn rows long enough for it to pay,
// a graph in which some level can pass heavy_level (qn * left is at most
// n^2 / 4), and nn outside the direction decision. The other searches run the
// kernel without that code, which costs them 1.5 to 3% (more registers and
// instructions at every level).
bool heavy_graph(const Search &a) {
  return !a.nn_do && a.nn_mean >= 4 && a.nn_mean * a.n / 4 >= a.n / 16.0 + kHeavyEdges;
}

// w: vertices of a graph of edge factor 16 with about as much work.
OneLaunch plain_shape(int64_t n, int64_t w) {
  if (w <= 1 << 13) return {32, 256};
  if (w <= 1 << 15) return {64, 256};
  if (w <= 3 << 15) return {64, 512};
  if (w <= 3 << 17) return {128, 512};
  // (many edges of many vertices: 650 and 684 us at 2^18 and 134M, 1101 and 1170 at 2^20)
  if (w <= 3 << 19 || (n >= 1 << 17 && n <= 3 << 19)) return {256, 512};
  if (n <= 3 << 20) return {256, 1024};
  return {0, 0};
}

OneLaunch one_launch_shape(int64_t n, int64_t m, int64_t max_degree, const dsbfs_run_opts &o) {
  // (below 2^20 edges the columns differ by less than runs do)
  const bool dense = m > 1 << 20;
  const OneLaunch plain = plain_shape(n, dense ? std::max(n, m / 64) : n);
  if (o.mode == 0) return plain;
  // uniform: the largest degree is 1.1 to 1.3 times the mean in ER graphs, 2.9 times
  // and more in the densest RMAT ones (where a source sees most of the graph at once
  // there is nothing to scan: ER 2^12 with 15M edges 67 us in 32 blocks, 84 in 128)
  const bool uniform = dense && max_degree * n <= 2 * m && 2 * max_degree <= n;
  const int64_t w = uniform ? std::max(n, m / 32) : n;
  OneLaunch r{256, 1024};
  if (n > 3 << 22) return {0, 0};
  if (w <= 1 << 14) r = {32, 256};
  else if (w <= 3 << 16) r = {64, 512};
  else if (w <= 3 << 20) r = {128, 1024};
  // a search that stays top-down, by its schedule or its factor
  const bool forward = o.forced == 1 || (o.forced == 0 && o.factor0[0] >= 1.0);
  if (forward && dense && plain.blocks * plain.threads > r.blocks * r.threads) r = plain;
  return r;
}

}  // namespace

// Where the dense output's arrays lie: in the part of dscan that a degree-separated
// search leaves unused, then behind the bitmap in dlen, which may grow to 4 n
// bytes for it (and 4 KB, for the smallest graphs' lines). Every graph with
// d <= n / 2 has room: 16 d bytes of dscan's 8 n, then 5 bytes a position (at most
// n - d) in the 8 (n - 2 d) left there and dlen's 3.9 n. Arrays of their own took 5
// bytes a position and 8 a delegate of every workspace. Graphs with more delegates
// than normals write depths and parents where they belong as they go: consecutive
// delegates are near-consecutive vertices there, which is what the arrays are for
// (16M vertices, 73 and 100% delegates: 4602 and 3265 us, with arrays 4619 and 3303).
static void place_output(Workspace *ws, const Alloc *al, hipStream_t s) {
  const Graph *g = ws->g;
  const size_t n = size_t(g->n), d = size_t(g->d), nds = size_t(g->st.n_ndsrc);
  struct Room {
    size_t at, end;
    bool take(size_t bytes, size_t &where) {
      const size_t b = (at + 255) / 256 * 256;
      if (b + bytes > end) return false;
      where = b;
      at = b + bytes;
      return true;
    }
  };
  const size_t fn = size_t(g->nwords()) * 4;
  Room scan{d * 8, (n + 1) * 8}, len{fn, n * 4 + 4096};
  const size_t size[3] = {std::max<size_t>(d, 1) * 8, std::max<size_t>(nds, 1) * 4,
                          (std::max<size_t>(nds, 1) + 3) / 4 * 4};
  size_t at[3];
  bool in_scan[3], fits = true;
  for (int i = 0; i < 3 && fits; ++i) {
    in_scan[i] = scan.take(size[i], at[i]);
    fits = in_scan[i] || len.take(size[i], at[i]);
  }
  ws->dlen.alloc(al, fits ? len.at : fn, s);
  if (!fits) return;
  void **const to[3] = {&ws->dout, &ws->ppar, &ws->plev};
  for (int i = 0; i < 3; ++i) *to[i] = (in_scan[i] ? ws->dscan : ws->dlen).as<char>() + at[i];
}

Workspace *workspace_create(const Graph *g, int32_t max_lanes) {
  if (max_lanes != 0 && max_lanes != 64)
    fail(DSBFS_ERR_INVALID_ARG, "max_lanes must be 0 or 64");
  Workspace *ws = new Workspace();
  try {
    ws->g = g;
    ws->max_lanes = max_lanes;
    const Alloc *al = &g->al;
    hipStream_t s = g->stream;
    const int64_t n = g->n, d = g->d;
    ws->Vn.alloc(al, size_t(g->nwords()) * 4, s);
    ws->Fn.alloc(al, size_t(g->nwords()) * 4, s);
    ws->Vd.alloc(al, size_t(g->dwords()) * 4, s);
    ws->Fd.alloc(al, size_t(g->dwords()) * 4, s);
    ws->Cd.alloc(al, size_t(g->dwords()) * 4, s);
    ws->q0.alloc(al, size_t(n) * 4, s);
    ws->q1.alloc(al, size_t(n) * 4, s);
    ws->dlist.alloc(al, size_t(d) * 4, s);
    ws->dscan.alloc(al, size_t(std::max(n, d) + 1) * 8, s);
    ws->c0.alloc(al, size_t(g->st.n_ndsrc) * 4, s);
    ws->c1.alloc(al, size_t(g->st.n_ndsrc) * 4, s);
    ws->ctl.alloc(al, sizeof(SearchCtl), s);
    place_output(ws, al, s);
    HIPCHK(hipHostMalloc(&ws->hstat, kStatusSlots * sizeof(LevelStatus), hipHostMallocDefault));
    std::memset(ws->hstat, 0, kStatusSlots * sizeof(LevelStatus));
    return ws;
  } catch (...) {
    delete ws;
    throw;
  }
}

void workspace_destroy(Workspace *ws) { delete ws; }

static dsbfs_run_opts default_opts() {
  dsbfs_run_opts o{};
  o.mode = 1;
  o.want_parent = 1;
  // tuned for this layout (see the header); the paper's are DSBFS_PAPER_FACTOR0_*
  o.factor0[0] = 0.02;
  o.factor0[1] = 0.001;
  o.factor0[2] = 1e-6;
  o.factor1[0] = o.factor1[1] = o.factor1[2] = 0.0;
  o.forced = 0;
  o.forced_seed = 0;
  o.nn_do = 0;
  o.factor0_nn = 1e-3;
  o.factor1_nn = 0.0;
  return o;
}

void run_opts_default(dsbfs_run_opts *o) { *o = default_opts(); }

// Blocks of grids that wait for their own blocks (one-launch searches, the
// persistent multi-source kernel) may not be resident in part beside each
// other: two such grids could hold the compute units each needs to complete.
// Each takes its blocks' worth of compute units from its device's gate before
// the launch and returns them once the launch has completed. Callers that wait
// (batches) are served in order of arrival, and while one does, a caller that
// can do without (a search, which then goes level by level) takes no units:
// searches that overlap each other would keep a batch from the whole chip for
// as long as they go on.
namespace {
struct ResidentGate {
  std::mutex mu;
  std::condition_variable cv;
  int units = 0, used = 0;         // compute units of the device, and those taken
  uint64_t next = 0, serving = 0;  // tickets of the callers that wait
};
ResidentGate &resident_gate() {
  static ResidentGate gates[64];
  int dev = 0;
  HIPCHK(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64) fail(DSBFS_ERR_INVALID_ARG, "device index out of range");
  ResidentGate &g = gates[dev];
  std::lock_guard<std::mutex> lk(g.mu);
  if (!g.units)
    HIPCHK(hipDeviceGetAttribute(&g.units, hipDeviceAttributeMultiprocessorCount, dev));
  return g;
}
}  // namespace

// More blocks than compute units are either several to a unit by the launch's own
// occupancy check (the batches' kernel, wait = true) or too many.
ResidentLease::ResidentLease(int blocks, bool wait) {
  ResidentGate &g = resident_gate();
  std::unique_lock<std::mutex> lk(g.mu);
  const int want = wait ? std::min(blocks, g.units) : blocks;
  if (wait) {
    const uint64_t ticket = g.next++;
    g.cv.wait(lk, [&] { return g.serving == ticket && g.used + want <= g.units; });
    ++g.serving;
    g.cv.notify_all();  // the next in line may fit beside this one
  } else if (g.serving != g.next || g.used + want > g.units) {
    return;
  }
  g.used += want;
  units = want;
  gate = &g;
}

bool ResidentLease::wanted() const {
  ResidentGate &g = *static_cast<ResidentGate *>(gate);
  std::lock_guard<std::mutex> lk(g.mu);
  return g.serving != g.next;
}

ResidentLease::~ResidentLease() {
  if (!gate) return;
  ResidentGate &g = *static_cast<ResidentGate *>(gate);
  {
    std::lock_guard<std::mutex> lk(g.mu);
    g.used -= units;
  }
  g.cv.notify_all();
}

namespace {

// Per-kernel HIP-event timing of a profiled search.
struct Prof {
  bool on = false;
  hipStream_t s = nullptr;
  Workspace *ws = nullptr;
  size_t next = 0;
  struct Span { int k, b, e, level; };
  std::vector<Span> spans;
  int64_t launches_seen[DSBFS_NUM_KERNELS] = {};

  hipEvent_t ev() {
    if (next == ws->events.size()) {
      hipEvent_t e;
      HIPCHK(hipEventCreate(&e));
      ws->events.push_back(e);
    }
    return ws->events[next++];
  }
  template <class F> void timed(int k, int level, F &&f) {
    if (!on) {
      f();
      return;
    }
    const int b = int(next);
    HIPCHK(hipEventRecord(ev(), s));
    f();
    const int e = int(next);
    HIPCHK(hipEventRecord(ev(), s));
    spans.push_back({k, b, e, level});
  }
};

Search search_args(const Graph *g, Workspace *ws, const dsbfs_run_opts &o, int32_t source,
                   int32_t *depth, int32_t *parent, bool count) {
  Search a{};
  a.noff = g->noff.as<uint64_t>();
  a.doff = g->doff.as<uint64_t>();
  a.nlen = g->nlen.as<uint16_t>();
  a.ncol = g->ncol.as<int32_t>();
  a.nnoff = g->nnoff.as<uint32_t>();
  a.nncol = g->nncol.as<int32_t>();
  a.dcol = g->dcol.as<int32_t>();
  a.vid_of = g->vid_of.as<int32_t>();
  a.ndsrc = g->ndsrc.as<int32_t>();
  a.nds_col = g->nds_col.as<int32_t>();
  a.nnsrc = g->nnsrc.as<int32_t>();
  a.nds_off = g->nds_off.as<int64_t>();
  a.nds_first = g->nds_first.as<int2>();
  a.dd_first = g->dd_first.as<int2>();
  a.ddm = g->ddsrc_mask.as<uint32_t>();
  a.dnm = g->dnsrc_mask.as<uint32_t>();
  a.poff = g->poff.as<int64_t>();
  a.pcol = g->pcol.as<int32_t>();
  a.did = g->did.as<int32_t>();
  a.n = g->n;
  a.d = g->d;
  a.nwords = g->nwords();
  a.dwords = g->dwords();
  a.n_ndsrc = g->st.n_ndsrc;
  a.n_nnsrc = g->st.n_nnsrc;
  a.depth = depth;
  a.parent = parent;
  a.Vn = ws->Vn.as<uint32_t>();
  // two normal frontier bitmaps alternate by level
  a.Fn0 = ws->Fn.as<uint32_t>();
  a.Fn1 = ws->dlen.as<uint32_t>();
  a.Vd = ws->Vd.as<uint32_t>();
  a.Fd = ws->Fd.as<uint32_t>();
  a.Cd = ws->Cd.as<uint32_t>();
  a.Q0 = ws->q0.as<int32_t>();
  a.Q1 = ws->q1.as<int32_t>();
  a.C0 = ws->c0.as<int32_t>();
  a.C1 = ws->c1.as<int32_t>();
  a.dlist = ws->dlist.as<int32_t>();
  a.dscan = ws->dscan.as<int64_t>();
  a.dout = static_cast<int2 *>(ws->dout);
  a.ppar = static_cast<int32_t *>(ws->ppar);
  a.plev = static_cast<uint8_t *>(ws->plev);
  a.drank = g->drank.as<RankDir>();
  a.nrank = g->nrank.as<RankDir>();
  a.ctl = ws->ctl.as<SearchCtl>();
  a.hs = static_cast<LevelStatus *>(ws->hstat);
  a.nn_mean = double(g->st.e_nn) / double(std::max(g->n - g->d, 1));
  a.nn_rows = kWave;
  while (a.nn_rows > 1 && a.nn_mean * (a.nn_rows / 2) >= 4 * kWave) a.nn_rows >>= 1;
  for (int k = 0; k < 3; ++k) {
    a.f0[k] = o.factor0[k];
    a.f1[k] = o.factor1[k];
  }
  a.f0[3] = o.factor0_nn;
  a.f1[3] = o.factor1_nn;
  a.forced_seed = o.forced_seed;
  a.forced = o.forced;
  a.nn_do = o.nn_do;
  a.count = count;
  a.source = source;
  a.mode = o.mode;
  a.bar_ticks = ws->bar_ticks ? ws->bar_ticks : kBarTicks;
  return a;
}

LevelState first_state(const Graph *g) {
  LevelState t{};
  t.cand_state = -1;
  t.rem[0] = g->st.n_ddsrc;
  t.rem[1] = g->st.n_dnsrc;
  t.rem[2] = g->st.n_ndsrc;
  t.rem[3] = g->st.n_nnsrc;
  t.nc = g->st.n_ndsrc;
  return t;
}

// The kernels of level L, level by level. skip: forward kernels that cannot
// have work (bit 0 all of them, bit 1 the delegate list).
void launch_level(const Search &a, int L, int skip, hipStream_t s) {
  const dim3 G(stride_grid()), B(kBS);
  if (a.mode == 0) {
    hipLaunchKernelGGL(k_plain_list, dim3(kSegs), B, 0, s, a, L);
    hipLaunchKernelGGL(k_plain_expand, G, B, 0, s, a, L);
    HIPCHK(hipGetLastError());
    return;
  }
  hipLaunchKernelGGL((k_previsit<kDeleg | kNormal | kClear>), G, B, 0, s, a, L);
  if (!(skip & 3) && a.d > 0) hipLaunchKernelGGL(k_list, dim3(kSegs), B, 0, s, a, L);
  if (!(skip & 1) && (a.d > 0 || a.nn_do))
    hipLaunchKernelGGL((k_forward<kDeleg | kNormal | kNn>), G, B, 0, s, a, L);
  if (a.nn_do && a.n_nnsrc > 0) hipLaunchKernelGGL(k_bu_nn, G, B, 0, s, a, L);
  hipLaunchKernelGGL((k_backward<kDeleg | kNormal | kCommit>), G, B, 0, s, a, L);
  HIPCHK(hipGetLastError());
}

// The same level with a kernel per visit, each timed (profile = 1).
void launch_level_profiled(const Search &a, int L, Prof &P) {
  const dim3 G(stride_grid()), B(kBS);
  hipStream_t s = P.s;
  if (a.mode == 0) {
    P.timed(DSBFS_K_PLAIN, L, [&] { launch_level(a, L, 0, s); });
    return;
  }
  if (a.d > 0)
    P.timed(DSBFS_K_PREV_DELEG, L,
            [&] { hipLaunchKernelGGL((k_previsit<kDeleg>), G, B, 0, s, a, L); });
  P.timed(DSBFS_K_CLOSE, L, [&] { hipLaunchKernelGGL((k_previsit<kClear>), G, B, 0, s, a, L); });
  P.timed(DSBFS_K_PREV_NORMAL, L,
          [&] { hipLaunchKernelGGL((k_previsit<kNormal>), G, B, 0, s, a, L); });
  if (a.nn_do)
    P.timed(DSBFS_K_TD_NN, L, [&] { hipLaunchKernelGGL((k_forward<kNn>), G, B, 0, s, a, L); });
  if (a.d > 0) {
    P.timed(DSBFS_K_TD_NORMAL, L,
            [&] { hipLaunchKernelGGL((k_forward<kNormal>), G, B, 0, s, a, L); });
    P.timed(DSBFS_K_TD_DELEG, L, [&] {
      hipLaunchKernelGGL(k_list, dim3(kSegs), B, 0, s, a, L);
      hipLaunchKernelGGL((k_forward<kDeleg>), G, B, 0, s, a, L);
    });
  }
  if (a.nn_do && a.n_nnsrc > 0)
    P.timed(DSBFS_K_BU_NN, L, [&] { hipLaunchKernelGGL(k_bu_nn, G, B, 0, s, a, L); });
  P.timed(DSBFS_K_BU_NORMAL, L,
          [&] { hipLaunchKernelGGL((k_backward<kNormal>), G, B, 0, s, a, L); });
  P.timed(DSBFS_K_BU_DELEG, L,
          [&] { hipLaunchKernelGGL((k_backward<kDeleg | kCommit>), G, B, 0, s, a, L); });
  HIPCHK(hipGetLastError());
}

// Waits until the device has published level L's record (pinned memory).
const LevelStatus &await_status(Workspace *ws, int L, hipStream_t s) {
  LevelStatus *st = static_cast<LevelStatus *>(ws->hstat) + (L & (kStatusSlots - 1));
  for (int64_t spin = 1;; ++spin) {
    if (__atomic_load_n(&st->seq, __ATOMIC_ACQUIRE) == L + 1) return *st;
    if (spin % 4096 == 0) {
      // the stream running dry (or failing) without the record is an error
      const hipError_t e = hipStreamQuery(s);
      if (e == hipErrorNotReady) continue;
      HIPCHK(e);
      if (__atomic_load_n(&st->seq, __ATOMIC_ACQUIRE) == L + 1) return *st;
      fail(DSBFS_ERR_DEVICE, "search ended without a level record");
    }
  }
}

void launch_init(const Search &a, const LevelState &st, hipStream_t s) {
  hipLaunchKernelGGL(k_init, dim3(grid_for(std::max(a.n, 1), kBS, 4096)), dim3(kBS), 0, s, a, st);
  HIPCHK(hipGetLastError());
}

void launch_output(const Search &a, hipStream_t s) {
  if (!a.compact) return;
  const dim3 grid(grid_for(a.n, 256 * kOutRow, 65536)), block(256);
  const bool vec = (uintptr_t(a.depth) | uintptr_t(a.parent)) % 16 == 0;
  if (vec)
    hipLaunchKernelGGL(k_output<true>, grid, block, 0, s, a);
  else
    hipLaunchKernelGGL(k_output<false>, grid, block, 0, s, a);
  HIPCHK(hipGetLastError());
}

// Level by level; seen gets the records of the levels with a frontier.
void run_levels(const Graph *g, Workspace *ws, Search a, const dsbfs_run_opts &o, Prof &P,
                std::vector<LevelStatus> &seen, hipStream_t s) {
  // (no arrays: the allocation-free search, graphs with many delegates)
  a.compact = o.mode == 1 && ws->dout;
  LevelStatus *hs = static_cast<LevelStatus *>(ws->hstat);
  if (!ws->borrowed)
    for (int i = 0; i < kStatusSlots; ++i) hs[i].seq = 0;
  P.timed(DSBFS_K_INIT, -1, [&] { launch_init(a, first_state(g), s); });
  if (P.on || ws->borrowed) {
    // a synchronization per level, so that only visits with work keep their
    // spans; the allocation-free search copies the record from device memory
    for (int32_t L = 0;; ++L) {
      const size_t sp0 = P.spans.size();
      if (P.on) launch_level_profiled(a, L, P);
      else launch_level(a, L, 0, s);
      LevelStatus st;
      if (ws->borrowed)
        HIPCHK(hipMemcpyAsync(&st, hs + (L & (kStatusSlots - 1)), sizeof(LevelStatus),
                              hipMemcpyDeviceToHost, s));
      HIPCHK(hipStreamSynchronize(s));
      if (!ws->borrowed) st = hs[L & (kStatusSlots - 1)];
      if (st.seq != L + 1) fail(DSBFS_ERR_DEVICE, "search ended without a level record");
      if (P.on) {
        LevelTotals tot;
        HIPCHK(hipMemcpy(&tot, &a.ctl->tot, sizeof(tot), hipMemcpyDeviceToHost));
        std::vector<Prof::Span> keep;
        for (size_t i = sp0; i < P.spans.size(); ++i)
          if (tot.launches[P.spans[i].k] > P.launches_seen[P.spans[i].k]) keep.push_back(P.spans[i]);
        for (int k = 0; k < DSBFS_NUM_KERNELS; ++k) P.launches_seen[k] = tot.launches[k];
        P.spans.resize(sp0);
        P.spans.insert(P.spans.end(), keep.begin(), keep.end());
      }
      if (st.done) break;
      seen.push_back(st);
    }
    P.timed(DSBFS_K_INIT, -1, [&] { launch_output(a, s); });
    HIPCHK(hipStreamSynchronize(s));
    return;
  }
  // The host stays one level ahead and stops once a level reports an empty
  // frontier (the level queued behind it returns at once). The level it
  // launches next leaves out forward kernels that cannot have work, from the
  // latest record it has seen: under the heuristic schedule with factor1 = 0 a
  // subgraph that went backward never switches back (FV < 0 * BV never holds).
  const bool monotone = o.forced == 0 && !o.nn_do && o.factor1[0] == 0.0 &&
                        o.factor1[1] == 0.0 && o.factor1[2] == 0.0;
  int skip = 0;
  for (int32_t L = 0;; ++L) {
    launch_level(a, L, skip, s);
    if (L < 1) continue;
    const LevelStatus &st = await_status(ws, L - 1, s);
    if (st.done) break;
    seen.push_back(st);
    if (monotone && o.mode == 1 && st.rec.dir[0] == 1 && st.rec.dir[1] == 1)
      skip = st.rec.dir[2] == 1 ? 1 : 2;
  }
  launch_output(a, s);
  // the level behind the last one is still queued: the workspace is free for
  // a search on another stream only after it
  HIPCHK(hipStreamSynchronize(s));
}

// The whole search in one launch (deep ones in several, see kLaunchLevels); false
// if a grid could not run (its workspace is then to be initialized again). After a launch that gave up on a
// wait, the workspace's next searches go level by level without trying, 16 at
// first and four times as many after every further one in a row: what the wait
// cost is spread over them while whatever holds the compute units stays.
bool run_one_launch(const Graph *g, Workspace *ws, Search a, const OneLaunch &shape,
                    hipStream_t s, int32_t *levels) {
  Backoff &back = ws->back;
  if (back.skip > 0) {
    --back.skip;
    return false;
  }
  stream_drain(s);
  auto lease = std::make_unique<ResidentLease>(shape.blocks, false);
  if (!lease->units) return false;
  LevelStatus *hs = static_cast<LevelStatus *>(ws->hstat);
  launch_init(a, first_state(g), s);
  LevelStatus st;
  for (;;) {
    if (!ws->borrowed) hs->seq = 0;
    if (a.mode == 1 && heavy_graph(a))
      hipLaunchKernelGGL(k_search<true>, dim3(shape.blocks), dim3(shape.threads), 0, s, a);
    else if (a.mode == 1)
      hipLaunchKernelGGL(k_search<false>, dim3(shape.blocks), dim3(shape.threads), 0, s, a);
    else
      hipLaunchKernelGGL(k_plain_search, dim3(shape.blocks), dim3(shape.threads), 0, s, a);
    HIPCHK(hipGetLastError());
    if (ws->borrowed)
      HIPCHK(hipMemcpyAsync(&st, hs, sizeof(LevelStatus), hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    if (!ws->borrowed) st = *hs;
    if (st.seq != kGoOn) break;
    a.level0 = st.level;
    hipLaunchKernelGGL(k_clear_bar, dim3(1), dim3(kBS), 0, s, &a.ctl->bar);
    if (lease->wanted()) {
      // behind those that wait now
      lease.reset();
      lease = std::make_unique<ResidentLease>(shape.blocks, true);
    }
  }
  *levels = st.level;
  if (st.seq == kDone) {
    back = Backoff{};
    return true;
  }
  back.len = back.len ? std::min(4 * back.len, 4096) : 16;
  back.skip = back.len;
  return false;
}

}  // namespace

void bfs_run(const Graph *g, Workspace *ws, int32_t source, const dsbfs_run_opts *opts_in,
             int32_t *depth, int32_t *parent, dsbfs_run_stats *stats, hipStream_t s) {
  if (!ws || ws->g != g) fail(DSBFS_ERR_INVALID_ARG, "workspace does not belong to this graph");
  if (source < 0 || source >= g->n) fail(DSBFS_ERR_INVALID_ARG, "source outside [0, n)");
  if (!depth) fail(DSBFS_ERR_INVALID_ARG, "depth must not be NULL");
  const dsbfs_run_opts o = opts_in ? *opts_in : default_opts();
  if (o.mode != 0 && o.mode != 1) fail(DSBFS_ERR_INVALID_ARG, "mode must be 0 or 1");
  if (o.want_parent && !parent) fail(DSBFS_ERR_INVALID_ARG, "parent is NULL but want_parent");
  if (o.mode == 0 && !g->pcol.p && g->m > 0)
    fail(DSBFS_ERR_INVALID_ARG, "mode 0 needs the plain CSR (keep_plain_csr)");
  if (o.forced < 0 || o.forced > 3) fail(DSBFS_ERR_INVALID_ARG, "forced must be 0..3");
  if (o.nn_do != 0 && o.nn_do != 1) fail(DSBFS_ERR_INVALID_ARG, "nn_do must be 0 or 1");

  const Search a = search_args(g, ws, o, source, depth, o.want_parent ? parent : nullptr,
                               stats != nullptr);
  Prof P;
  P.on = o.profile != 0 && stats != nullptr;
  P.s = s;
  P.ws = ws;
  std::vector<LevelStatus> seen;
  int32_t num_levels = 0;
  // One launch unless the caller wants a record per level.
  const bool records = stats && stats->levels && stats->capacity > 0;
  const OneLaunch shape = one_launch_shape(g->n, g->m, g->st.max_degree, o);
  if (!(shape.blocks && !P.on && !records &&
        run_one_launch(g, ws, a, shape, s, &num_levels))) {
    run_levels(g, ws, a, o, P, seen, s);
    num_levels = int32_t(seen.size());
  }
  if (!stats) return;

  LevelTotals tot;
  unsigned long long U[DSBFS_NUM_KERNELS][4];
  HIPCHK(hipMemcpyAsync(&tot, &a.ctl->tot, sizeof(tot), hipMemcpyDeviceToHost, s));
  HIPCHK(hipMemcpyAsync(U, a.ctl->units, sizeof(U), hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  // queue and list entries are counted by the decision
  for (int k = 0; k < DSBFS_NUM_KERNELS; ++k)
    if (k != DSBFS_K_BU_NORMAL && k != DSBFS_K_BU_DELEG && k != DSBFS_K_BU_NN)
      U[k][0] = tot.units0[k];
  U[DSBFS_K_INIT][0] = (unsigned long long)g->n;
  stats->num_levels = num_levels;
  for (int32_t i = 0; i < int32_t(seen.size()) && i < stats->capacity && stats->levels; ++i) {
    stats->levels[i] = seen[i].rec;
    for (double &t : stats->levels[i].kernel_ms) t = 0.0;  // filled from the spans below
  }
  // Every reached vertex sits in exactly one level's frontier, whose previsit
  // (or plain expansion) summed its full degree; each vertex but the source
  // was claimed exactly once. So the component's size and edge count come
  // from the level counters without another pass over depth[].
  stats->reached = 1 + int64_t(U[DSBFS_K_PREV_NORMAL][2] + U[DSBFS_K_TD_NORMAL][3] +
                               U[DSBFS_K_TD_DELEG][2] + U[DSBFS_K_TD_DELEG][3] +
                               U[DSBFS_K_BU_NORMAL][3] + U[DSBFS_K_BU_DELEG][2] +
                               U[DSBFS_K_PLAIN][2] + U[DSBFS_K_TD_NN][2] + U[DSBFS_K_BU_NN][3]);
  stats->edges_cc = int64_t((o.mode == 0 ? U[DSBFS_K_PLAIN][1] : tot.deg_sum) / 2);

  // Algorithmic bytes per kernel from its unit counts (see dsbfs.h).
  const int64_t out_b = o.want_parent ? 8 : 4;  // depth (+ parent) per vertex
  auto u = [&](int k, int j) { return int64_t(U[k][j]); };
  int64_t bytes[DSBFS_NUM_KERNELS] = {};
  int64_t edges[DSBFS_NUM_KERNELS] = {};
  bytes[DSBFS_K_INIT] = u(DSBFS_K_INIT, 0) * out_b;
  bytes[DSBFS_K_PREV_DELEG] = u(DSBFS_K_PREV_DELEG, 0) * (4 + 16);
  for (int k : {DSBFS_K_PREV_NORMAL, DSBFS_K_PLAIN, DSBFS_K_TD_NN}) {
    bytes[k] = u(k, 0) * (4 + 16) + u(k, 1) * 4 + u(k, 2) * (out_b + 4);
    edges[k] = u(k, 1);
  }
  bytes[DSBFS_K_TD_NORMAL] = u(DSBFS_K_TD_NORMAL, 0) * (4 + 16) + u(DSBFS_K_TD_NORMAL, 1) * 4 +
                             u(DSBFS_K_TD_NORMAL, 3) * (out_b + 4);
  edges[DSBFS_K_TD_NORMAL] = u(DSBFS_K_TD_NORMAL, 1);
  bytes[DSBFS_K_TD_DELEG] = u(DSBFS_K_TD_DELEG, 0) * (4 + 16) + u(DSBFS_K_TD_DELEG, 1) * 4 +
                            (u(DSBFS_K_TD_DELEG, 2) + u(DSBFS_K_TD_DELEG, 3)) * (out_b + 4 + 4);
  edges[DSBFS_K_TD_DELEG] = u(DSBFS_K_TD_DELEG, 1);
  for (int k : {DSBFS_K_BU_NORMAL, DSBFS_K_BU_NN}) {
    bytes[k] = u(k, 0) * 4 + u(k, 1) * 16 + u(k, 2) * 4 + u(k, 3) * (out_b + 4 + 4);
    edges[k] = u(k, 2);
  }
  bytes[DSBFS_K_BU_NORMAL] += int64_t(tot.kept) * 4;
  bytes[DSBFS_K_BU_DELEG] = u(DSBFS_K_BU_DELEG, 0) * (4 + 4 + 16) + u(DSBFS_K_BU_DELEG, 1) * 4 +
                            u(DSBFS_K_BU_DELEG, 2) * (out_b + 4 + 4);
  edges[DSBFS_K_BU_DELEG] = u(DSBFS_K_BU_DELEG, 1);
  bytes[DSBFS_K_CLOSE] = u(DSBFS_K_CLOSE, 0) * 4;
  double ms[DSBFS_NUM_KERNELS] = {};
  for (const Prof::Span &sp : P.spans) {
    float t = 0.f;
    HIPCHK(hipEventElapsedTime(&t, ws->events[sp.b], ws->events[sp.e]));
    ms[sp.k] += double(t);
    if (sp.level >= 0 && sp.level < stats->num_levels && sp.level < stats->capacity &&
        stats->levels)
      stats->levels[sp.level].kernel_ms[sp.k] += double(t);
  }
  for (int k = 0; k < DSBFS_NUM_KERNELS; ++k) {
    stats->kernels[k].ms = ms[k];
    stats->kernels[k].launches = k == DSBFS_K_INIT ? 1 : tot.launches[k];
    stats->kernels[k].bytes = bytes[k];
    stats->kernels[k].edges = edges[k];
  }
}

// ---------------------------------------------------------------------------
// Allocation-free single-source search
// ---------------------------------------------------------------------------
// For callers that cannot allocate device memory: the search's scratch (the
// workspace's bitmaps, queues, candidate lists, counters, control block and
// level status ring) is carved out of one file-scope device array. Each GPU
// holds its own copy of the array, at its own address, from the library's
// load until the process ends; host code never uses the array's name as an
// address, only the device address hipGetSymbolAddress returns for the
// current device.
// What grows with the graph has kScratchBytes; the control block and the status
// ring, of fixed size, lie before it (behind it, 64 MB from all else that a search
// reads, they cost it 2 us).
constexpr size_t kScratchBytes = size_t(64) << 20;
constexpr size_t round256(size_t b) { return ((b < 256 ? 256 : b) + 255) / 256 * 256; }
constexpr size_t kFixedBytes =
    round256(sizeof(SearchCtl)) + round256(kStatusSlots * sizeof(LevelStatus));
static __device__ __align__(256) unsigned char scratch[kFixedBytes + kScratchBytes];

namespace {

constexpr int kMaxDevices = 64;

struct ScratchSlot {
  std::mutex mu;         // one search at a time per device
  void *ptr = nullptr;   // device address of `scratch` on this device
  Backoff back;          // of the searches in it, as a workspace's
};

ScratchSlot &scratch_slot(int dev) {
  static ScratchSlot slots[kMaxDevices];
  return slots[dev];
}

}  // namespace

// What decides whether a graph is taken (about 25 bytes per vertex). It is
// more than the search carves out of kScratchBytes now (every part carved below
// is a term here; those marked "room" have no part): the limit on graphs stays
// where callers know it.
size_t noalloc_scratch_bytes(const Graph *g) {
  const int64_t n = g->n, d = g->d, nm = std::max(n, d);
  const size_t tiles = (size_t((d + 2047) / 2048 + 1) * 8 + 255) / 256 * 256;
  size_t t = 0;
  t += 2 * round256(size_t(g->nwords()) * 4);          // Vn, Fn
  t += 3 * round256(size_t(g->dwords()) * 4);          // Vd, Fd, Cd
  t += 2 * round256(size_t(n) * 4);                    // q0, q1
  t += 2 * round256(size_t(d) * 4);                    // dlist; room
  t += round256(size_t(nm) * 4);                       // dlen, and room
  t += round256(size_t(nm + 1) * 8);                   // dscan
  t += 2 * round256(size_t(g->st.n_ndsrc) * 4);        // c0, c1
  t += round256(scan_tmp_bytes(nm));                   // room
  t += round256(2 * tiles);                            // room
  t += 3328;                                           // room
  return t;
}

void bfs_run_noalloc(const Graph *g, int32_t source, const dsbfs_run_opts *opts, int32_t *depth,
                     int32_t *parent, dsbfs_run_stats *stats, hipStream_t s) {
  if (!g) fail(DSBFS_ERR_INVALID_ARG, "graph must not be NULL");
  if (opts && opts->profile)
    fail(DSBFS_ERR_INVALID_ARG, "profile = 1 needs timing events; the allocation-free search "
                                "does not create them");
  const size_t need = noalloc_scratch_bytes(g);
  if (need > kScratchBytes)
    fail(DSBFS_ERR_RANGE, "graph needs " + std::to_string(need) +
                              " bytes of search scratch; the allocation-free search holds " +
                              std::to_string(kScratchBytes) + " (use a workspace)");
  int dev = 0;
  HIPCHK(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) fail(DSBFS_ERR_INVALID_ARG, "device index out of range");
  ScratchSlot &sl = scratch_slot(dev);
  std::lock_guard<std::mutex> lock(sl.mu);
  if (!sl.ptr) {
    void *ptr = nullptr;
    HIPCHK(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) fail(DSBFS_ERR_HIP, "hipGetSymbolAddress returned NULL for the search scratch");
    sl.ptr = ptr;
  }
  char *base = static_cast<char *>(sl.ptr);
  size_t off = 0;
  auto carve = [&](DevBuf &b, size_t bytes) {
    b.p = base + off;
    b.bytes = round256(bytes);
    b.al = nullptr;   // not owned: nothing is freed
    b.s = s;
    off += b.bytes;
  };
  const int64_t n = g->n, d = g->d, nm = std::max(n, d);
  Workspace ws;
  ws.g = g;
  ws.borrowed = true;
  carve(ws.ctl, sizeof(SearchCtl));
  DevBuf ring;
  carve(ring, kStatusSlots * sizeof(LevelStatus));
  carve(ws.Vn, size_t(g->nwords()) * 4);
  carve(ws.Fn, size_t(g->nwords()) * 4);
  carve(ws.Vd, size_t(g->dwords()) * 4);
  carve(ws.Fd, size_t(g->dwords()) * 4);
  carve(ws.Cd, size_t(g->dwords()) * 4);
  carve(ws.q0, size_t(n) * 4);
  carve(ws.q1, size_t(n) * 4);
  carve(ws.dlist, size_t(d) * 4);
  carve(ws.dlen, size_t(g->nwords()) * 4);
  carve(ws.dscan, size_t(nm + 1) * 8);
  carve(ws.c0, size_t(g->st.n_ndsrc) * 4);
  carve(ws.c1, size_t(g->st.n_ndsrc) * 4);
  if (off > kFixedBytes + kScratchBytes)
    fail(DSBFS_ERR_RANGE, "allocation-free search scratch exceeded");
  ws.hstat = ring.p;
  ws.back = sl.back;
  bfs_run(g, &ws, source, opts, depth, parent, stats, s);
  sl.back = ws.back;
  // the next call reuses the array: this one's work must be complete
  HIPCHK(hipStreamSynchronize(s));
}

}  // namespace dsbfs
