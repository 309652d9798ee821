// Internal declarations of the dsbfs HIP library (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "dsbfs.h"

namespace dsbfs {

constexpr int kWave = 64;
constexpr uint64_t kOffMask = (1ull << 40) - 1;  // packed row offset: start in bits 0..39
constexpr int kOffShift = 40;                    // length of the first part in bits 40..63
constexpr int64_t kMaxFirstPart = (1ll << 24) - 1;

// ---------------------------------------------------------------------------
// Errors: internal code throws dsbfs::Error; the C-ABI layer catches it.
// ---------------------------------------------------------------------------
struct Error {
  dsbfs_status status;
  std::string msg;
};

[[noreturn]] void fail(dsbfs_status st, const std::string &msg);
void hip_check(hipError_t e, const char *what, const char *file, int line);
#define HIPCHK(x) ::dsbfs::hip_check((x), #x, __FILE__, __LINE__)

// ---------------------------------------------------------------------------
// Device memory through the caller's allocator (or hipMalloc).
// ---------------------------------------------------------------------------
struct Alloc {
  dsbfs_allocator a{};
  bool custom = false;
  void *get(size_t bytes, hipStream_t s) const;
  void put(void *p, hipStream_t s) const;
};

// Owning device buffer bound to an allocator.
struct DevBuf {
  void *p = nullptr;
  size_t bytes = 0;
  const Alloc *al = nullptr;
  hipStream_t s = nullptr;
  DevBuf() = default;
  DevBuf(const DevBuf &) = delete;
  DevBuf &operator=(const DevBuf &) = delete;
  DevBuf(DevBuf &&o) noexcept { *this = std::move(o); }
  DevBuf &operator=(DevBuf &&o) noexcept {
    if (this != &o) {
      reset();
      p = o.p; bytes = o.bytes; al = o.al; s = o.s;
      o.p = nullptr; o.bytes = 0;
    }
    return *this;
  }
  ~DevBuf() { reset(); }
  void alloc(const Alloc *a, size_t nbytes, hipStream_t st) {
    reset();
    al = a; s = st; bytes = nbytes;
    p = a->get(nbytes < 256 ? 256 : nbytes, st);
  }
  void reset() {
    if (p && al) al->put(p, s);
    p = nullptr; bytes = 0;
  }
  template <class T> T *as() const { return static_cast<T *>(p); }
};

// ---------------------------------------------------------------------------
// Graph: the degree-separated layout (Section III-C) plus the plain CSR.
//   Normal rows  (n rows, indexed by vertex ID; empty for delegates):
//     [ nn neighbours (vertex IDs) | nd neighbours (delegate IDs) ]
//   Delegate rows (d rows, indexed by delegate ID):
//     [ dd neighbours (delegate IDs) | dn neighbours (vertex IDs) ]
//   noff/doff are packed: start (bits 0..39) | first-part length << 40.
// ---------------------------------------------------------------------------
constexpr uint16_t kLenWide = 0xFFFF;

// Directory of a set of vertices, one entry per 32: their bits, and the rank
// (position among all of the set, ascending) of the first of them.
struct RankDir {
  uint32_t bits;
  int32_t base;
  __host__ __device__ bool has(int32_t v) const { return (bits >> (v & 31)) & 1u; }
  __device__ int32_t rank(int32_t v) const {
    return base + __popc(bits & ((1u << (v & 31)) - 1u));
  }
};

struct Graph {
  Alloc al;
  hipStream_t stream = nullptr;
  int device = 0;
  int32_t n = 0, d = 0, TH = 0;
  int64_t m = 0;
  dsbfs_graph_stats st{};
  DevBuf deg, did, vid_of, noff, ncol, doff, dcol, ndsrc, ddsrc_mask, dnsrc_mask;
  // nd rows again, in nd-source-list order (row i = nd part of ndsrc[i]), so
  // bottom-up passes over the source list stream them: int64 [n_ndsrc+1],
  // int32 [e_nd] delegate IDs.
  DevBuf nds_off, nds_col, nds_first;
  DevBuf dd_first;  // per delegate: (first dd neighbour, its vertex), or (-1, -1)
  // per vertex, uint16: nn length | nd length << 8 of a normal row (0 for a
  // delegate), kLenWide when either is 255 or more (read noff instead); the
  // normal previsit reads these 2 bytes instead of two 8-byte row offsets
  DevBuf nlen;
  // ranks of the delegates (their IDs) and of the nd source list (positions),
  // RankDir [ceil(n / 32)]
  DevBuf drank, nrank;
  DevBuf nnsrc;     // normal vertices with a normal neighbour, ascending (nn_do bottom-up)
  // nn parts again, concatenated in vertex order (int32 [e_nn] vertex IDs),
  // and the start of each vertex's part (uint32 [n]): a forward nn visit
  // reads 4 bytes per frontier vertex and a column array of 4 bytes per nn
  // edge, where most parts are one or two entries, instead of the 8-byte
  // packed offset and a line of the full row. Not built (null) when
  // e_nn >= 2^32; the kernels then read noff and ncol.
  DevBuf nnoff, nncol;
  DevBuf poff, pcol;  // plain CSR: int64 offsets [n+1], int32 columns [m]
  // PageRank's gather-friendly copy, built by its first call and kept with
  // the graph: pr_order = the delegates by descending degree bucket (ties by
  // ID), pr_lead the leading ones whose rows a block pulls, and pr_col = dcol
  // with every dd entry replaced by its rank in that order, so the
  // contributions of the most-gathered delegates sit together (int32 [d],
  // [e_dd + e_dn]).
  mutable DevBuf pr_order, pr_col;
  mutable int32_t pr_lead = 0;
  mutable std::mutex pr_mu;
  int32_t dwords() const { return (d + 31) / 32; }
  int32_t nwords() const { return (n + 31) / 32; }
};

// Searches that do not try a single launch after one that had to give up.
struct Backoff {
  int skip = 0;  // of them left
  int len = 0;   // how many the last one set
};

// Scratch of one search at a time (single-source and multi-source).
struct Workspace {
  const Graph *g = nullptr;
  int32_t max_lanes = 0;
  // uint32 bitmaps: visited / frontier normals; visited at level start,
  // frontier, and claimed (visited or found this level) delegates
  DevBuf Vn, Fn, Vd, Fd, Cd;
  DevBuf q0, q1;               // normal queues, int32[n]
  DevBuf dlist;                // frontier delegates of a forward visit, int32[d]
  DevBuf dlen;                 // second Fn bitmap
  DevBuf dscan;                // int64[max(n, d) + 1]: prefix of top-down lengths
  DevBuf c0, c1;               // bottom-up normal candidates, int32[n_ndsrc]
  // what bottom-up visits and delegate claims find, until a dense pass at the
  // end of the search writes it out (bfs.hip): per position of the nd source
  // list parent (int32) and depth (uint8, 0: none), per delegate (parent,
  // depth + 1). They lie in dscan, of which a degree-separated search uses d
  // entries, and behind dlen's bitmap; NULL where they do not fit there
  // (place_output).
  void *ppar = nullptr, *plev = nullptr, *dout = nullptr;
  DevBuf ctl;                  // control block of the search in progress (bfs.hip)
  std::vector<hipEvent_t> events;  // profiling event pool
  void *hstat = nullptr;       // pinned ring of per-level status records
  Backoff back;
  int64_t bar_ticks = 0;       // bound of a one-launch search's waits; 0: the usual one
  // multi-source lane state
  void *ms_state = nullptr;           // launch state of multi-source BFS (msbfs.hip)
  // borrowed: every buffer points into memory the workspace does not own (the
  // allocation-free search's static scratch); hstat is then device memory,
  // read by copies
  bool borrowed = false;
  ~Workspace();
};

// Compute units held for a launch whose blocks wait for each other (bfs.hip):
// taken before the launch, returned once it has completed. wait = false: units
// is 0 when there are not enough now. The launch's stream has nothing else to do
// first (stream_drain): units held behind a long kernel of the caller's would
// keep every batch of the device waiting for it.
struct ResidentLease {
  int units = 0;
  void *gate = nullptr;
  ResidentLease(int blocks, bool wait);
  ~ResidentLease();
  bool wanted() const;  // others wait for units
  ResidentLease(const ResidentLease &) = delete;
  ResidentLease &operator=(const ResidentLease &) = delete;
};

// A counter on a 128-byte line of its own: device-scope atomics on one line are
// served one after the other, 12.6 ns each.
struct alignas(128) CtrLine {
  unsigned long long v;
  unsigned long long pad[15];
};

// Sources of the lanes admitted at one level (by value: no copy per level).
struct SeedList {
  int32_t src[64];
};

// Control block of one level of the server's batches (device; two alternate):
// the next frontier's size and lanes, in parts that the reader sums, and the
// length of a top-down level's list.
constexpr int kLvParts = 16;
struct LvCtl {
  CtrLine active[kLvParts], alive[kLvParts], td_count;
};

// Rows written by one flush of the server's level ring (see k_lv_flush).
struct LaneFlush {
  int32_t *res[64];    // result row of each lane (int32[n]) or NULL if the lane is idle
  int32_t start[64];   // level at which each lane's source had depth 0
  uint64_t valid[16];  // per level jlo + o: the lanes whose unwritten levels include it
  uint64_t lanes;      // lanes considered
  int32_t jlo, jhi;    // levels [jlo, jhi], jhi - jlo < 16
  int32_t final;       // 1: only lanes whose frontier ran empty; write -1 where unreached
};

// ---------------------------------------------------------------------------
// Device helpers.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int lane_id() { return __lane_id(); }

// Number of set bits of mask in lanes below the calling lane.
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u));
}

template <class T> __device__ __forceinline__ T wave_sum(T v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

// Cross-lane moves through DPP (data-parallel primitives: a VALU operand
// modifier, no LDS round trip, unlike ds_bpermute behind __shfl). Lanes whose
// source is outside the row / wave, or whose row is masked off, read `old`.
constexpr int kDppRowShr = 0x110;   // + n (1..15): lane l reads l - n within its 16-lane row
constexpr int kDppWaveShl1 = 0x130; // lane l reads l + 1
constexpr int kDppWaveShr1 = 0x138; // lane l reads l - 1
constexpr int kDppBcast15 = 0x142;  // rows 1..3 read lane 15 of the previous row
constexpr int kDppBcast31 = 0x143;  // rows 2..3 read lane 31
template <int Ctrl, int RowMask = 0xf>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t old, uint32_t v) {
  return uint32_t(__builtin_amdgcn_update_dpp(int(old), int(v), Ctrl, RowMask, 0xf, false));
}

// Lane `src` (wave-uniform) of v, through a scalar register.
__device__ __forceinline__ int32_t lane_read(int32_t v, int src) {
  return __builtin_amdgcn_readlane(v, src);
}
__device__ __forceinline__ int64_t lane_read(int64_t v, int src) {
  const uint32_t lo = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(uint64_t(v))), src));
  const uint32_t hi = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(uint64_t(v) >> 32)), src));
  return int64_t((static_cast<uint64_t>(hi) << 32) | lo);
}
__device__ __forceinline__ unsigned long long lane_read(unsigned long long v, int src) {
  const uint32_t lo = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(v)), src));
  const uint32_t hi = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(v >> 32)), src));
  return (static_cast<unsigned long long>(hi) << 32) | lo;
}

// OR of a 64-bit value over the wave, returned to every lane (DPP inclusive
// OR-scan of each half, then lane 63 through a scalar register). The whole
// wave must be active.
__device__ __forceinline__ uint32_t wave_or_dpp_u32(uint32_t x) {
  x |= dpp_u32<kDppRowShr + 1>(0u, x);
  x |= dpp_u32<kDppRowShr + 2>(0u, x);
  x |= dpp_u32<kDppRowShr + 4>(0u, x);
  x |= dpp_u32<kDppRowShr + 8>(0u, x);
  x |= dpp_u32<kDppBcast15, 0xa>(0u, x);
  x |= dpp_u32<kDppBcast31, 0xc>(0u, x);
  return uint32_t(__builtin_amdgcn_readlane(int(x), kWave - 1));
}
__device__ __forceinline__ uint64_t wave_or_all(uint64_t x) {
  const uint32_t lo = wave_or_dpp_u32(uint32_t(x));
  const uint32_t hi = wave_or_dpp_u32(uint32_t(x >> 32));
  return (uint64_t(hi) << 32) | lo;
}

// Inclusive prefix sum across the 64 lanes of a wave.
template <class T> __device__ __forceinline__ T wave_incl_scan(T v) {
  const int l = lane_id();
  for (int o = 1; o < kWave; o <<= 1) {
    T t = __shfl_up(v, o, kWave);
    if (l >= o) v += t;
  }
  return v;
}
// 32-bit version with DPP: Hillis-Steele inside each 16-lane row, then the
// row totals carried across rows by two broadcasts.
template <> __device__ __forceinline__ int32_t wave_incl_scan<int32_t>(int32_t v) {
  uint32_t x = uint32_t(v);
  x += dpp_u32<kDppRowShr + 1>(0u, x);
  x += dpp_u32<kDppRowShr + 2>(0u, x);
  x += dpp_u32<kDppRowShr + 4>(0u, x);
  x += dpp_u32<kDppRowShr + 8>(0u, x);
  x += dpp_u32<kDppBcast15, 0xa>(0u, x);
  x += dpp_u32<kDppBcast31, 0xc>(0u, x);
  return int32_t(x);
}

// Wave-aggregated append: every lane with `want` gets a distinct slot of
// *counter (returned), one atomic per wave. Lanes without `want` get -1.
__device__ __forceinline__ int64_t wave_append(bool want, unsigned long long *counter) {
  uint64_t m = __ballot(want);
  if (m == 0) return -1;
  int leader = __ffsll(static_cast<long long>(m)) - 1;
  unsigned long long base = 0;
  if (lane_id() == leader) base = atomicAdd(counter, static_cast<unsigned long long>(__popcll(m)));
  base = lane_read(base, leader);
  return want ? static_cast<int64_t>(base + lanes_below(m)) : -1;
}

__device__ __forceinline__ bool bit_test(const uint32_t *bm, uint32_t v) {
  return (bm[v >> 5] >> (v & 31)) & 1u;
}

// Wave-cooperative bitmap update for lanes whose bits tend to share words
// (vertices visited in ascending order). Adjacent lanes with the same word
// form a run; a segmented OR-scan combines the run's bits and the run's last
// lane issues the one atomicOr. Atomics on one word from many lanes of one
// instruction serialize in the cache, so this is several times faster than a
// per-lane atomicOr on ascending patterns. Must be called by the whole wave.
//   claim: returns true for exactly one lane per bit that was 0 before the
//   call (a bit wanted by several lanes of one run goes to the lowest lane).
struct WaveBits {
  uint32_t word, bit, incl, old;
  bool want, head;
  // valid: v is a vertex (its word joins a run even without a bit, so the
  // runs of an ascending list are not cut by lanes that want nothing)
  __device__ __forceinline__ void run(uint32_t *bm, uint32_t v, bool valid, bool w,
                                      bool need_old) {
    const int l = lane_id();
    want = valid && w;
    word = valid ? (v >> 5) : 0xffffffffu;
    bit = want ? (1u << (v & 31)) : 0u;
    // neighbours' words (lane 0 / lane 63 read a value no word can take)
    const uint32_t prev_word = dpp_u32<kDppWaveShr1>(0xfffffffeu, word);
    const uint32_t next_word = dpp_u32<kDppWaveShl1>(0xfffffffeu, word);
    head = l == 0 || prev_word != word;
    const bool tail = l == kWave - 1 || next_word != word;
    // segmented inclusive OR-scan (incl = OR of the bits from the run's head
    // to this lane) with DPP; f marks that a head lies within the span so far
    incl = bit;
    uint32_t f = head ? 1u : 0u, t, tf;
#define DSBFS_SEG_STEP(CTRL, MASK)              \
    t = dpp_u32<CTRL, MASK>(0u, incl);           \
    tf = dpp_u32<CTRL, MASK>(0u, f);             \
    if (!f) incl |= t;                           \
    f |= tf;
    DSBFS_SEG_STEP(kDppRowShr + 1, 0xf)
    DSBFS_SEG_STEP(kDppRowShr + 2, 0xf)
    DSBFS_SEG_STEP(kDppRowShr + 4, 0xf)
    DSBFS_SEG_STEP(kDppRowShr + 8, 0xf)
    DSBFS_SEG_STEP(kDppBcast15, 0xa)
    DSBFS_SEG_STEP(kDppBcast31, 0xc)
#undef DSBFS_SEG_STEP
    old = 0;
    if (tail && word != 0xffffffffu && incl) old = atomicOr(&bm[word], incl);
    if (need_old) {
      // the run's tail is the first tail lane at or after this lane
      const uint64_t tails = __ballot(tail);
      const int tp = l + __builtin_ctzll(tails >> l);
      old = uint32_t(__shfl(int(old), tp, kWave));
    }
  }
  // true iff this lane set its bit first (bit was 0 and no lower lane of the run wanted it)
  __device__ __forceinline__ bool won() const {
    const uint32_t before = dpp_u32<kDppWaveShr1>(0u, incl);
    const uint32_t excl = head ? 0u : before;
    return want && !(old & bit) && !(excl & bit);
  }
};

__device__ __forceinline__ bool wave_bit_claim(uint32_t *bm, uint32_t v, bool valid, bool want) {
  WaveBits wb;
  wb.run(bm, v, valid, want, true);
  return wb.won();
}

__device__ __forceinline__ void wave_bit_set(uint32_t *bm, uint32_t v, bool valid, bool want) {
  WaveBits wb;
  wb.run(bm, v, valid, want, false);
}

// Orders LDS traffic of one wave around a point where lanes read what other
// lanes of the same wave wrote.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Block-level append buffer in LDS for grid-stride kernels: lanes reserve
// slots with one LDS atomic per wave; the block writes the buffer out with a
// single global atomic per flush, coalesced. Device-scope atomics on one
// global counter serialize across the chip, so kernels never do one per wave.
// Appends beyond the buffer (only possible if one iteration produces more
// than `cap - margin` entries) fall back to a wave-aggregated global append.
struct BlockAppend {
  int32_t *buf;              // LDS, cap entries
  int *count;                // LDS
  unsigned long long *base;  // LDS
  int cap;
  unsigned long long *gcount;
  int32_t *gout;
  int shift = 0;  // the 32-bit half of *gcount that counts this list (0 or 32)

  // Reserves n entries of the list: the old count of its half of *gcount.
  __device__ unsigned long long reserve(unsigned long long n) const {
    return (atomicAdd(gcount, n << shift) >> shift) & 0xffffffffull;
  }

  __device__ void init() {
    if (threadIdx.x == 0) *count = 0;
  }
  // Called by every lane of a wave (wave-uniform).
  __device__ void push(bool want, int32_t v) {
    const uint64_t m = __ballot(want);
    if (m == 0) return;
    const int leader = __ffsll(static_cast<long long>(m)) - 1;
    int p = 0;
    if (lane_id() == leader) p = atomicAdd(count, __popcll(m));
    p = lane_read(p, leader);
    const int pos = p + int(lanes_below(m));
    const bool over = want && pos >= cap;
    if (want && !over) buf[pos] = v;
    const uint64_t mo = __ballot(over);
    if (mo) {
      const int lo = __ffsll(static_cast<long long>(mo)) - 1;
      unsigned long long b = 0;
      if (lane_id() == lo) b = reserve(__popcll(mo));
      b = lane_read(b, lo);
      if (over) gout[b + lanes_below(mo)] = v;
    }
  }
};

// Writes out two append buffers that count in the two halves of one word
// (q: bits 0..31, c: bits 32..63) with a single atomic (block-uniform).
__device__ inline void flush_pair(BlockAppend &q, BlockAppend &c) {
  __syncthreads();
  const int nq = min(*q.count, q.cap), nc = min(*c.count, c.cap);
  if (threadIdx.x == 0) {
    unsigned long long b = 0;
    if (nq || nc)
      b = atomicAdd(q.gcount, (static_cast<unsigned long long>(nc) << 32) |
                                  static_cast<unsigned long long>(nq));
    *q.base = b & 0xffffffffull;
    *c.base = b >> 32;
  }
  __syncthreads();
  const unsigned long long bq = *q.base, bc = *c.base;
  for (int i = threadIdx.x; i < nq; i += blockDim.x) q.gout[bq + i] = q.buf[i];
  for (int i = threadIdx.x; i < nc; i += blockDim.x) c.gout[bc + i] = c.buf[i];
  __syncthreads();
  if (threadIdx.x == 0) {
    *q.count = 0;
    *c.count = 0;
  }
  __syncthreads();
}

// Writes both buffers out once one may not hold another step's entries (at
// most `margin`). Block-uniform: the decision is read between two barriers,
// where no push can change the counts. With the first alone, a wave could push
// its next step's entries before another had read the counts of this one: the
// two then parted at the barriers of flush_pair, and entries were lost.
__device__ inline void flush_pair_if_full(BlockAppend &q, BlockAppend &c, int margin) {
  __syncthreads();
  const bool full = *q.count > q.cap - margin || *c.count > c.cap - margin;
  __syncthreads();
  if (full) flush_pair(q, c);
}

__device__ __forceinline__ int64_t row_start(uint64_t w) { return static_cast<int64_t>(w & kOffMask); }
__device__ __forceinline__ int64_t row_first(uint64_t w) { return static_cast<int64_t>(w >> kOffShift); }

// Appends both directions of up to N pairs per thread that are not loops as
// keys (u << B) | v, with one atomic per block (block-uniform call). A pair
// that is not there is given as a loop.
template <int N>
__device__ __forceinline__ void pack_pairs(const int32_t (&u)[N], const int32_t (&v)[N], int B,
                                           uint64_t *keys, unsigned long long *cursor) {
  __shared__ unsigned long long wbase[16];
  const int w = threadIdx.x / kWave, nw = blockDim.x / kWave;
  int total = 0;
#pragma unroll
  for (int i = 0; i < N; ++i) total += __popcll(__ballot(u[i] != v[i]));
  __syncthreads();
  if (lane_id() == 0) wbase[w] = (unsigned long long)total;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long sum = 0;
    for (int i = 0; i < nw; ++i) sum += wbase[i];
    unsigned long long run = atomicAdd(cursor, sum);
    for (int i = 0; i < nw; ++i) {
      const unsigned long long t = wbase[i];
      wbase[i] = run;
      run += t;
    }
  }
  __syncthreads();
  unsigned long long pos = wbase[w];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const bool keep = u[i] != v[i];
    const uint64_t m = __ballot(keep);
    if (keep) {
      const uint64_t a = uint64_t(uint32_t(u[i])), b = uint64_t(uint32_t(v[i]));
      uint64_t *const to = keys + 2 * (pos + lanes_below(m));
      to[0] = (a << B) | b;
      to[1] = (b << B) | a;
    }
    pos += __popcll(m);
  }
}

// Degree bucket of a vertex on a log scale (8 buckets per power of two), so
// that ordering by bucket orders neighbours by degree with a one-byte key.
__host__ __device__ __forceinline__ uint32_t deg_bucket(int32_t deg) {
  if (deg <= 1) return 0;
#ifdef __HIP_DEVICE_COMPILE__
  const uint32_t lg = 31u - __clz(uint32_t(deg));          // floor(log2)
#else
  const uint32_t lg = 31u - uint32_t(__builtin_clz(uint32_t(deg)));
#endif
  const uint32_t frac = lg >= 3 ? (uint32_t(deg) >> (lg - 3)) & 7u : (uint32_t(deg) << (3 - lg)) & 7u;
  const uint32_t b = lg * 8u + frac;
  return b > 254u ? 254u : b;
}

inline int grid_for(int64_t items, int per_block, int cap = 65536) {
  int64_t g = (items + per_block - 1) / per_block;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return static_cast<int>(g);
}

// ---------------------------------------------------------------------------
// Device-wide primitives (prims.hip).
// ---------------------------------------------------------------------------
// out[i] = sum of in[0..i), i in [0, N]; out has N+1 entries. tmp is scratch
// of scan_tmp_bytes(N) bytes.
size_t scan_tmp_bytes(int64_t N);
void scan_excl_i32_to_i64(const int32_t *in, int64_t *out, int64_t N, void *tmp, hipStream_t s);

// Stable LSD radix sort of N uint64 keys on bits [lo_bit, hi_bit) (bits above
// hi_bit are equal in all keys; keys already ordered below lo_bit keep that
// order among equal sort fields). Returns the array that holds the result, keys
// or alt (both of N keys). tmp: radix_tmp_bytes(N).
size_t radix_tmp_bytes(int64_t N);
uint64_t *radix_sort_u64_bits(uint64_t *keys, uint64_t *alt, int64_t N, int lo_bit, int hi_bit,
                              void *tmp, hipStream_t s);

// Order-preserving compaction of indices i in [0, N) with flag[i] != 0 into
// out; *count (device) gets the number kept. tmp: compact_tmp_bytes(N).
size_t compact_tmp_bytes(int64_t N);
void compact_flags_u8(const uint8_t *flag, int64_t N, int32_t *out, int64_t *count, void *tmp,
                      hipStream_t s);
// The distinct keys of a sorted array as CSR rows: key = (row << B) | column.
// unique_count_u64 counts them (and leaves the tiles' prefix in tmp),
// unique_to_csr, called next with the same tmp, writes their columns (col, m of
// them) and the row offsets off[n + 1]. tmp: unique_tmp_bytes(N).
size_t unique_tmp_bytes(int64_t N);
void unique_count_u64(const uint64_t *keys, int64_t N, int64_t *count, void *tmp, hipStream_t s);
void unique_to_csr(const uint64_t *keys, int64_t N, int64_t m, int B, int32_t n, int64_t *off,
                   int32_t *col, void *tmp, hipStream_t s);

// Host helpers.
// Waits for the work queued on s, if any (an idle stream costs the query, 0.1 us
// to 0.5 us).
inline void stream_drain(hipStream_t s) {
  const hipError_t e = hipStreamQuery(s);
  if (e == hipErrorNotReady) {
    (void)hipGetLastError();
    HIPCHK(hipStreamSynchronize(s));
  } else {
    HIPCHK(e);
  }
}
template <class T> T d2h_scalar(const T *dptr, hipStream_t s) {
  T v{};
  HIPCHK(hipMemcpyAsync(&v, dptr, sizeof(T), hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  return v;
}

}  // namespace dsbfs
