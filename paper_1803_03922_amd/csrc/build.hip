// Graph construction on the device.
//
// Edge list -> simple symmetric graph (edge doubling, Section VI-A; symmetric
// graph assumption, Section II-A; self-loops and duplicates dropped) ->
// plain CSR -> degree separation at TH (Section III-A: delegate iff degree >
// TH; delegates renumbered in ascending vertex ID, Fig. 2 caption) -> the
// four subgraphs (Section III-C) stored as two row sets with packed offsets:
//   normal row v   = [nn neighbours (vertex IDs) | nd neighbours (delegate IDs)]
//   delegate row k = [dd neighbours (delegate IDs) | dn neighbours (vertex IDs)]
// and the source list of nd plus the source masks of dd and dn (Section IV-B).
//
// At one GPU every vertex is local, so nn columns are 32-bit vertex IDs too
// (the paper keeps them 64-bit only because they may be remote), and the
// offsets are 64-bit because one GPU holds more than 2^32 edges at scale 26.
#include <algorithm>

#include "internal.hpp"

namespace dsbfs {

namespace {

constexpr int kBS = 256;

// Pairs with an endpoint outside [0, n) (ctr[0]) and, of the others, those that
// are not loops (ctr[1]), which is what the keys need room for: room for every
// pair would be four times a list's own size too much where most are loops. One
// pass over the list, both counts with one atomic a block.
constexpr int kPackItems = 16;
__global__ void __launch_bounds__(kBS) k_count_pairs(const int32_t *src, const int32_t *dst,
                                                     int64_t g, int32_t n,
                                                     unsigned long long *ctr) {
  constexpr int64_t tile = int64_t(kBS) * kPackItems;
  __shared__ unsigned long long sh[2];
  if (threadIdx.x < 2) sh[threadIdx.x] = 0;
  __syncthreads();
  unsigned long long bad = 0, keep = 0;
  for (int64_t t0 = int64_t(blockIdx.x) * tile; t0 < g; t0 += int64_t(gridDim.x) * tile) {
    int32_t u[kPackItems], v[kPackItems];
#pragma unroll
    for (int i = 0; i < kPackItems; ++i) {
      const int64_t e = t0 + i * kBS + threadIdx.x;
      u[i] = e < g ? src[e] : 0;
      v[i] = e < g ? dst[e] : 0;
    }
#pragma unroll
    for (int i = 0; i < kPackItems; ++i) {
      const bool out = uint32_t(u[i]) >= uint32_t(n) || uint32_t(v[i]) >= uint32_t(n);
      bad += out;
      keep += !out && u[i] != v[i];
    }
  }
  bad = wave_sum(bad);
  keep = wave_sum(keep);
  if (lane_id() == 0) {
    if (bad) atomicAdd(&sh[0], bad);
    if (keep) atomicAdd(&sh[1], keep);
  }
  __syncthreads();
  if (threadIdx.x < 2 && sh[threadIdx.x]) atomicAdd(&ctr[threadIdx.x], sh[threadIdx.x]);
}

// Both directions of every non-loop pair as 64-bit keys (u << B) | v, in any
// order (they are sorted next). A block packs kPackItems pairs per thread and
// reserves their places with one atomic: one per wave step, on one address,
// took 12.6 ms for 67M pairs (12.6 ns each, one after the other). Bound by the
// 24 bytes a pair moves: 0.28 ms.
__global__ void __launch_bounds__(kBS) k_pack(const int32_t *src, const int32_t *dst, int64_t g,
                                              int B, uint64_t *keys, unsigned long long *cursor) {
  constexpr int64_t tile = int64_t(kBS) * kPackItems;
  for (int64_t t0 = int64_t(blockIdx.x) * tile; t0 < g; t0 += int64_t(gridDim.x) * tile) {
    const int64_t w0 = t0 + int64_t(threadIdx.x / kWave) * (kWave * kPackItems) + lane_id();
    int32_t u[kPackItems], v[kPackItems];
#pragma unroll
    for (int i = 0; i < kPackItems; ++i) {
      const int64_t e = w0 + i * kWave;
      u[i] = e < g ? src[e] : 0;
      v[i] = e < g ? dst[e] : 0;
    }
    pack_pairs<kPackItems>(u, v, B, keys, cursor);
  }
}

__global__ void k_degrees(const int64_t *poff, int32_t n, int32_t *deg) {
  for (int64_t v = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; v < n;
       v += int64_t(gridDim.x) * blockDim.x)
    deg[v] = int32_t(poff[v + 1] - poff[v]);
}

__global__ void k_flag_gt(const int32_t *deg, int32_t n, int32_t th, uint8_t *flag) {
  for (int64_t v = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; v < n;
       v += int64_t(gridDim.x) * blockDim.x)
    flag[v] = deg[v] > th;
}

__global__ void k_fill_i32(int32_t *p, int64_t N, int32_t val) {
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < N;
       i += int64_t(gridDim.x) * blockDim.x)
    p[i] = val;
}

__global__ void k_did_scatter(const int32_t *vid_of, int32_t d, int32_t *did) {
  for (int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; k < d;
       k += int64_t(gridDim.x) * blockDim.x)
    did[vid_of[k]] = int32_t(k);
}

__global__ void k_row_lengths(const int32_t *deg, const int32_t *did, const int32_t *vid_of,
                              int32_t n, int32_t d, int32_t *nlen, int32_t *dlen) {
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t v = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; v < n; v += stride)
    nlen[v] = did[v] < 0 ? deg[v] : 0;
  for (int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; k < d; k += stride)
    dlen[k] = deg[vid_of[k]];
}

__global__ void k_pack_offsets(const int64_t *nstart, const int64_t *dstart, const int32_t *deg,
                               const int32_t *did, const int32_t *vid_of, const int32_t *cnt_del,
                               int32_t n, int32_t d, uint64_t *noff, uint64_t *doff) {
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t v = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; v <= n; v += stride) {
    uint64_t first = 0;
    if (v < n && did[v] < 0) first = uint64_t(deg[v] - cnt_del[v]);  // nn part
    noff[v] = uint64_t(nstart[v]) | (first << kOffShift);
  }
  for (int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; k <= d; k += stride) {
    uint64_t first = k < d ? uint64_t(cnt_del[vid_of[k]]) : 0;      // dd part
    doff[k] = uint64_t(dstart[k]) | (first << kOffShift);
  }
}

// Compact part lengths of the normal rows (see Graph::nlen).
__global__ void k_pack_lens(const int32_t *deg, const int32_t *did, const int32_t *cnt_del,
                            int32_t n, uint16_t *nlen) {
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t v = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; v < n; v += stride) {
    uint16_t x = 0;
    if (did[v] < 0) {
      const int32_t nd = cnt_del[v], nn = deg[v] - nd;
      x = (nn < 255 && nd < 255) ? uint16_t(nn | (nd << 8)) : kLenWide;
    }
    nlen[v] = x;
  }
}

// nn length of every vertex (0 for a delegate): the part sizes of the
// compact nn copy.
__global__ void k_nn_counts(const int32_t *deg, const int32_t *did, const int32_t *cnt_del,
                            int32_t n, int32_t *cnt) {
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t v = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; v < n; v += stride)
    cnt[v] = did[v] < 0 ? deg[v] - cnt_del[v] : 0;
}

// Copies the nn part of every normal row (its first part) to its place in
// the compact nn copy and records where it starts.
__global__ void k_nn_fill(const int64_t *start, const int32_t *cnt, const uint64_t *noff,
                          const int32_t *ncol, int32_t n, uint32_t *nnoff, int32_t *nncol) {
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t v = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; v < n; v += stride) {
    const int64_t o = start[v];
    nnoff[v] = uint32_t(o);
    const int32_t c = cnt[v];
    if (c > 0) {
      const int64_t b = row_start(noff[v]);
      for (int32_t j = 0; j < c; ++j) nncol[o + j] = ncol[b + j];
    }
  }
}

// ---------------------------------------------------------------------------
// arranging the rows
// ---------------------------------------------------------------------------
// What the arrangement needs of a neighbour, in arrays that stay in the L2: a
// byte per vertex with its degree bucket, plus one for delegates (degrees
// above TH: delegate iff code > bucket(TH), bucket = code minus that one), and
// the delegates' rank directory for their IDs. The degree and delegate ID
// arrays would be a line from beyond the L2 per entry (16 MB each at 4M
// vertices): 3.3 ms for the dd keys of RMAT 22 alone.
__global__ void k_codes(const int32_t *deg, const int32_t *did, int32_t n, int32_t th,
                        uint8_t *code, RankDir *rank) {
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t v0 = int64_t(blockIdx.x) * blockDim.x; v0 < n; v0 += stride) {
    const int64_t v = v0 + threadIdx.x;
    int32_t k = -1;
    if (v < n) {
      k = did[v];
      code[v] = uint8_t(deg_bucket(deg[v]) + (deg[v] > th));
    }
    const uint64_t m = __ballot(k >= 0);
    const int l = lane_id();
    const uint32_t bits = uint32_t(l < 32 ? m : m >> 32);
    const int first = (l < 32 ? 0 : 32) + (bits ? __ffs(bits) - 1 : 0);
    const int32_t base = __shfl(k, first, kWave);
    if ((l & 31) == 0 && v < n) rank[v >> 5] = RankDir{bits, base};
  }
}

struct Arrange {
  const int64_t *poff;
  const int32_t *pcol;     // rows of the plain CSR, ascending
  const uint8_t *code;
  const RankDir *rank;
  const int32_t *deg, *did;
  const int64_t *nstart, *dstart;
  int32_t n;
  int32_t bth;             // bucket of TH
  int32_t *plain;          // plain rows by bucket, highest first (NULL: not wanted)
  int32_t *ncol, *dcol;    // split rows
  int32_t *cnt_del;        // delegate neighbours of each row

  __device__ __forceinline__ bool is_del(uint32_t c) const { return int32_t(c) > bth; }
  __device__ __forceinline__ int32_t del_id(int32_t v) const {
    return rank[v >> 5].rank(v);
  }
  // where row u's split entries go
  __device__ __forceinline__ int32_t *split_row(int32_t u, bool &del) const {
    const int32_t k = did[u];
    del = k >= 0;
    return del ? dcol + dstart[k] : ncol + nstart[u];
  }
  // order of an entry in the plain row: bucket, highest first
  __device__ __forceinline__ uint32_t plain_key(uint32_t c) const {
    return 255u - (c - (is_del(c) ? 1u : 0u));
  }
  // and in the split row: a delegate's row has its dd entries by bucket,
  // highest first, then the dn entries; a normal row nn, then nd
  __device__ __forceinline__ uint32_t split_key(uint32_t c, bool del) const {
    return del ? (is_del(c) ? 255u - c : 255u) : (is_del(c) ? 1u : 0u);
  }
};

// Rows with at most kShortRow entries. A wave takes 16 rows (or 8 at a time
// when they are long), stages their entries in LDS and places each entry by
// counting the entries of its row that go before it: plain by (bucket
// descending, ID), dd by the same, dn and nn by ID, nd by (degree descending,
// ID). Bound by the gathers of the code bytes; the walk over the row costs
// len LDS reads per entry.
constexpr int kShortRow = 64;
constexpr int kShortCap = 512;  // entries a wave holds

struct ShortWave {
  int32_t col[kShortCap];
  int32_t deg[kShortCap];
  uint8_t code[kShortCap];
  int32_t ex[kWave];    // exclusive prefix of the row lengths
  int64_t beg[16];
};

__device__ __forceinline__ int owner_of(const int32_t *ex, int32_t e) {
  int lo = 0;
#pragma unroll
  for (int step = 32; step > 0; step >>= 1)
    if (ex[lo + step] <= e) lo += step;
  return lo;
}

__global__ void __launch_bounds__(kBS) k_rows_short(Arrange a) {
  __shared__ ShortWave s_w[kBS / kWave];
  ShortWave &S = s_w[threadIdx.x / kWave];
  const int l = lane_id();
  const int64_t wid = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) / kWave;
  const int64_t nw = int64_t(gridDim.x) * blockDim.x / kWave;
  for (int64_t v0 = wid * 16; v0 < a.n; v0 += nw * 16) {
    int64_t b = 0;
    int32_t all = 0;
    bool mine = false;
    if (l < 16 && v0 + l < a.n) {
      b = a.poff[v0 + l];
      all = int32_t(a.poff[v0 + l + 1] - b);
      mine = all <= kShortRow;
      if (!mine) all = 0;
      if (mine && all == 0) a.cnt_del[v0 + l] = 0;
    }
    // 16 rows at once, or 8 and 8
    const int32_t sum = lane_read(wave_incl_scan(all), kWave - 1);
    if (sum == 0) continue;
    for (int half = 0; half < (sum <= kShortCap ? 1 : 2); ++half) {
      const bool take = sum <= kShortCap || l / 8 == half;
      const int32_t len = take ? all : 0;
      const int32_t incl = wave_incl_scan(len);
      const int32_t T = lane_read(incl, kWave - 1);
      wave_sync();
      S.ex[l] = incl - len;
      if (l < 16) S.beg[l] = b;
      wave_sync();
      for (int32_t e = l; e < T; e += kWave) {
        const int o = owner_of(S.ex, e);
        const int32_t v = a.pcol[S.beg[o] + (e - S.ex[o])];
        const uint8_t c = a.code[v];
        S.col[e] = v;
        S.code[e] = c;
        // exact degrees order the nd entries of normal rows
        S.deg[e] = a.is_del(c) ? a.deg[v] : 0;
      }
      wave_sync();
      for (int32_t e = l; e < T; e += kWave) {
        const int o = owner_of(S.ex, e);
        const int32_t r0 = S.ex[o], r1 = o < kWave - 1 ? S.ex[o + 1] : T;
        const uint32_t c = S.code[e];
        const uint32_t pk = a.plain_key(c);
        const int32_t dg = S.deg[e];
        int32_t before = 0;   // entries of the plain row before this one
        int32_t del = 0;      // delegate entries of the row
        int32_t del_b = 0, del_d = 0;  // delegates before, by bucket / by degree
        int32_t nor_b = 0;    // normals before, by ID
        for (int32_t j = r0; j < r1; ++j) {
          const uint32_t cj = S.code[j];
          const uint32_t kj = a.plain_key(cj);
          const bool dj = a.is_del(cj), ahead = j < e;
          const int32_t gj = S.deg[j];
          before += kj < pk || (kj == pk && ahead);
          del += dj;
          del_b += dj && (cj > c || (cj == c && ahead));
          del_d += dj && (gj > dg || (gj == dg && ahead));
          nor_b += !dj && ahead;
        }
        const int32_t v = S.col[e];
        const int64_t u = v0 + o;
        if (a.plain) a.plain[S.beg[o] + before] = v;
        bool row_del;
        int32_t *out = a.split_row(int32_t(u), row_del);
        const bool is_del = a.is_del(c);
        const int32_t len_o = r1 - r0;
        int32_t pos;
        if (row_del) pos = is_del ? del_b : del + nor_b;
        else pos = is_del ? (len_o - del) + del_d : nor_b;
        out[pos] = is_del ? a.del_id(v) : v;
        if (e == r0) a.cnt_del[u] = del;
      }
      wave_sync();
    }
  }
}

// Longer rows: a stable counting sort by one-byte keys, for the plain row and
// the split row together: counts, their prefix, then the entries 64 per wave
// step, ranked inside the step by matching keys with ballots (their order, so
// ascending IDs, is kept among equal keys). A wave per row up to kHugeRow
// entries; past that a block of 16 waves per row. (Before: keys of 8 bytes
// and four or five radix passes over all rows for each of the two orders.)
constexpr int kHugeRow = 8192;

// Lanes with the same key as this one, among `active`.
__device__ __forceinline__ uint64_t match_key(uint32_t key, uint64_t active) {
  uint64_t m = active;
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    const bool bit = (key >> b) & 1u;
    const uint64_t bal = __ballot(bit);
    m &= bit ? bal : ~bal;
  }
  return m;
}

// Exclusive prefix of 256 counts by one wave, in place (4 counts a lane).
__device__ __forceinline__ void prefix256(int32_t *cnt) {
  const int l = lane_id();
  int32_t c[4], t = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    c[i] = cnt[4 * l + i];
    t += c[i];
  }
  int32_t run = wave_incl_scan(t) - t;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    cnt[4 * l + i] = run;
    run += c[i];
  }
}

__global__ void __launch_bounds__(kBS) k_rows_long(Arrange a, const int32_t *rows,
                                                   const int64_t *nrows) {
  __shared__ int32_t s_p[kBS / kWave][256], s_s[kBS / kWave][256];
  int32_t *const cp = s_p[threadIdx.x / kWave], *const cs = s_s[threadIdx.x / kWave];
  const int l = lane_id();
  const int64_t wid = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) / kWave;
  const int64_t nw = int64_t(gridDim.x) * blockDim.x / kWave;
  const int64_t R = *nrows;
  for (int64_t i = wid; i < R; i += nw) {
    const int32_t u = rows[i];
    const int64_t b = a.poff[u];
    const int32_t len = int32_t(a.poff[u + 1] - b);
    if (len > kHugeRow) continue;
    bool del;
    int32_t *const out = a.split_row(u, del);
    wave_sync();
    for (int k = l; k < 256; k += kWave) cp[k] = cs[k] = 0;
    wave_sync();
    int32_t ndel = 0;
    // four steps' loads together (a step alone is a chain of two gathers);
    // slots past the row end load its last entry again
    for (int32_t j0 = 0; j0 < len; j0 += 4 * kWave) {
      int32_t v[4];
      uint32_t c[4];
#pragma unroll
      for (int x = 0; x < 4; ++x) v[x] = a.pcol[b + min(j0 + x * kWave + l, len - 1)];
#pragma unroll
      for (int x = 0; x < 4; ++x) c[x] = a.code[v[x]];
#pragma unroll
      for (int x = 0; x < 4; ++x)
        if (j0 + x * kWave + l < len) {
          ndel += a.is_del(c[x]);
          if (a.plain) atomicAdd(&cp[a.plain_key(c[x])], 1);
          atomicAdd(&cs[a.split_key(c[x], del)], 1);
        }
    }
    ndel = wave_sum(ndel);
    if (l == 0) a.cnt_del[u] = ndel;
    wave_sync();
    prefix256(cp);
    prefix256(cs);
    wave_sync();
    for (int32_t j0 = 0; j0 < len; j0 += 4 * kWave) {
      int32_t v4[4], id4[4];
      uint32_t c4[4];
#pragma unroll
      for (int x = 0; x < 4; ++x) v4[x] = a.pcol[b + min(j0 + x * kWave + l, len - 1)];
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        c4[x] = a.code[v4[x]];
        const int32_t id = a.del_id(v4[x]);
        id4[x] = a.is_del(c4[x]) ? id : v4[x];
      }
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const bool ok = j0 + x * kWave + l < len;
        const uint64_t act = __ballot(ok);
        if (act == 0) break;
        const uint32_t ks = a.split_key(c4[x], del);
        const uint64_t ms = match_key(ks, act);
        if (ok) out[cs[ks] + int32_t(lanes_below(ms))] = id4[x];
        uint32_t kp = 0;
        uint64_t mp = 0;
        if (a.plain) {
          kp = a.plain_key(c4[x]);
          mp = match_key(kp, act);
          if (ok) a.plain[b + cp[kp] + int32_t(lanes_below(mp))] = v4[x];
        }
        wave_sync();
        if (ok && lanes_below(ms) == 0) cs[ks] += __popcll(ms);
        if (a.plain && ok && lanes_below(mp) == 0) cp[kp] += __popcll(mp);
        wave_sync();
      }
    }
  }
}

constexpr int kHugeBS = 1024, kHugeNW = kHugeBS / kWave;

// One ordering of a huge row: counts per wave of each 1024-entry round, so that
// entries of equal keys keep their order across the block's waves.
template <class Key, class Put>
__device__ void huge_order(int32_t len, int32_t (*wcnt)[256], int32_t *base, Key &&key,
                           Put &&put) {
  const int w = threadIdx.x / kWave, l = lane_id();
  __syncthreads();
  if (threadIdx.x < 256) base[threadIdx.x] = 0;
  __syncthreads();
  for (int32_t j = threadIdx.x; j < len; j += kHugeBS) atomicAdd(&base[key(j)], 1);
  __syncthreads();
  if (w == 0) prefix256(base);
  __syncthreads();
  for (int32_t j0 = 0; j0 < len; j0 += kHugeBS) {
    const int32_t j = j0 + threadIdx.x;
    const bool ok = j < len;
    const uint32_t k = ok ? key(j) : 0u;
    const uint64_t m = match_key(k, __ballot(ok));
    for (int i = l; i < 256; i += kWave) wcnt[w][i] = 0;
    wave_sync();
    if (ok && lanes_below(m) == 0) wcnt[w][k] = __popcll(m);
    __syncthreads();
    if (threadIdx.x < 256) {
      int32_t run = base[threadIdx.x];
#pragma unroll
      for (int i = 0; i < kHugeNW; ++i) {
        const int32_t c = wcnt[i][threadIdx.x];
        wcnt[i][threadIdx.x] = run;
        run += c;
      }
      base[threadIdx.x] = run;
    }
    __syncthreads();
    if (ok) put(j, wcnt[w][k] + int32_t(lanes_below(m)));
    __syncthreads();
  }
}

__global__ void __launch_bounds__(kHugeBS) k_rows_huge(Arrange a, const int32_t *rows,
                                                       const int64_t *nrows) {
  __shared__ int32_t wcnt[kHugeNW][256];
  __shared__ int32_t base[256];
  __shared__ int32_t ndel;
  const int64_t R = *nrows;
  for (int64_t i = blockIdx.x; i < R; i += gridDim.x) {
    const int32_t u = rows[i];
    const int64_t b = a.poff[u];
    const int32_t len = int32_t(a.poff[u + 1] - b);
    bool del;
    int32_t *const out = a.split_row(u, del);
    if (threadIdx.x == 0) ndel = 0;
    __syncthreads();
    int32_t nd = 0;
    for (int32_t j = threadIdx.x; j < len; j += kHugeBS) nd += a.is_del(a.code[a.pcol[b + j]]);
    nd = wave_sum(nd);
    if (lane_id() == 0) atomicAdd(&ndel, nd);
    __syncthreads();
    if (threadIdx.x == 0) a.cnt_del[u] = ndel;
    auto code = [&](int32_t j) { return uint32_t(a.code[a.pcol[b + j]]); };
    huge_order(len, wcnt, base, [&](int32_t j) { return a.split_key(code(j), del); },
               [&](int32_t j, int32_t pos) {
                 const int32_t v = a.pcol[b + j];
                 out[pos] = a.is_del(a.code[v]) ? a.del_id(v) : v;
               });
    if (a.plain)
      huge_order(len, wcnt, base, [&](int32_t j) { return a.plain_key(code(j)); },
                 [&](int32_t j, int32_t pos) { a.plain[b + pos] = a.pcol[b + j]; });
    __syncthreads();
  }
}

__global__ void k_flag_ndsrc(const int32_t *did, const int32_t *cnt_del, int32_t n, uint8_t *flag) {
  for (int64_t u = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; u < n;
       u += int64_t(gridDim.x) * blockDim.x)
    flag[u] = did[u] < 0 && cnt_del[u] > 0;
}

// Normal vertices with a normal neighbour (bottom-up nn candidates).
__global__ void k_flag_nnsrc(const int32_t *deg, const int32_t *did, const int32_t *cnt_del,
                             int32_t n, uint8_t *flag) {
  for (int64_t u = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; u < n;
       u += int64_t(gridDim.x) * blockDim.x)
    flag[u] = did[u] < 0 && deg[u] > cnt_del[u];
}

__global__ void k_source_masks(const int32_t *vid_of, const int32_t *deg, const int32_t *cnt_del,
                               int32_t d, uint32_t *ddm, uint32_t *dnm) {
  const int32_t W = (d + 31) / 32;
  for (int64_t w = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; w < W;
       w += int64_t(gridDim.x) * blockDim.x) {
    uint32_t a = 0, b = 0;
    for (int i = 0; i < 32; ++i) {
      const int64_t k = w * 32 + i;
      if (k >= d) break;
      const int32_t u = vid_of[k];
      if (cnt_del[u] > 0) a |= 1u << i;
      if (deg[u] - cnt_del[u] > 0) b |= 1u << i;
    }
    ddm[w] = a;
    dnm[w] = b;
  }
}

// Rank directory of the nd source list (cleared before).
__global__ void k_nd_rank(const int32_t *ndsrc, int64_t cnt, RankDir *rank) {
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < cnt;
       i += int64_t(gridDim.x) * blockDim.x) {
    const int32_t v = ndsrc[i];
    if (i == 0 || (ndsrc[i - 1] >> 5) != (v >> 5)) rank[v >> 5].base = int32_t(i);
    atomicOr(&rank[v >> 5].bits, 1u << (v & 31));
  }
}

__global__ void k_nds_len(const int32_t *ndsrc, int64_t cnt, const int32_t *cnt_del,
                          int32_t *len) {
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < cnt;
       i += int64_t(gridDim.x) * blockDim.x)
    len[i] = cnt_del[ndsrc[i]];
}

// Copies the nd part of row ndsrc[i] to row i of the source-list-ordered copy,
// and its first entry (delegate ID, then that delegate's vertex) to pair i of
// nds_first, the dense array a bottom-up pass probes first.
__global__ void k_nds_fill(const int32_t *ndsrc, int64_t cnt, const uint64_t *noff,
                           const int32_t *ncol, const int32_t *vid_of, const int64_t *nds_off,
                           int32_t *nds_col, int32_t *nds_first) {
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < cnt;
       i += int64_t(gridDim.x) * blockDim.x) {
    const int32_t v = ndsrc[i];
    const uint64_t w0 = noff[v];
    const int64_t from = row_start(w0) + row_first(w0);
    const int64_t to = nds_off[i], len = nds_off[i + 1] - to;
    for (int64_t j = 0; j < len; ++j) nds_col[to + j] = ncol[from + j];
    // rows of the list are never empty
    nds_first[2 * i] = ncol[from];
    nds_first[2 * i + 1] = vid_of[ncol[from]];
  }
}

// [0] e_nn [1] e_nd [2] e_dn [3] e_dd [4] n_ndsrc [5] n_ddsrc [6] n_dnsrc [7] max degree
__global__ void k_stats(const int32_t *deg, const int32_t *did, const int32_t *cnt_del, int32_t n,
                        unsigned long long *out) {
  unsigned long long a[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  unsigned long long mx = 0;
  for (int64_t u = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; u < n;
       u += int64_t(gridDim.x) * blockDim.x) {
    const unsigned long long dg = deg[u], cd = cnt_del[u], cn = dg - cd;
    if (did[u] < 0) {
      a[0] += cn; a[1] += cd; a[4] += cd > 0; a[7] += cn > 0;
    } else {
      a[2] += cn; a[3] += cd; a[5] += cd > 0; a[6] += cn > 0;
    }
    mx = dg > mx ? dg : mx;
  }
  // one atomic a block and count (one a wave, on one line, took 1.6 ms at 4M vertices)
  __shared__ unsigned long long sh[9];
  if (threadIdx.x < 9) sh[threadIdx.x] = 0;
  __syncthreads();
  for (int i = 0; i < 8; ++i) {
    const unsigned long long s = wave_sum(a[i]);
    // out[7] is the maximum degree; the count of normals with an nn edge is out[8]
    if (lane_id() == 0 && s) atomicAdd(&sh[i < 7 ? i : 8], s);
  }
  for (int o = 32; o > 0; o >>= 1) {
    unsigned long long t = __shfl_xor(mx, o, kWave);
    mx = t > mx ? t : mx;
  }
  if (lane_id() == 0) atomicMax(&sh[7], mx);
  __syncthreads();
  if (threadIdx.x < 9 && sh[threadIdx.x]) {
    if (threadIdx.x == 7) atomicMax(&out[7], sh[7]);
    else atomicAdd(&out[threadIdx.x], sh[threadIdx.x]);
  }
}

int bits_for(int64_t n) {
  int B = 1;
  while ((int64_t(1) << B) < n) ++B;
  return B;
}

// First entry of every dd part (its highest-degree neighbour) and that
// neighbour's vertex, as a dense pair per delegate; (-1, -1) if the part is
// empty. The bottom-up dd visit probes it before walking the row.
__global__ void k_dd_first(const uint64_t *doff, const int32_t *dcol, const int32_t *vid_of,
                           int32_t d, int32_t *out) {
  for (int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; k < d;
       k += int64_t(gridDim.x) * blockDim.x) {
    const uint64_t w = doff[k];
    const int32_t x = row_first(w) > 0 ? dcol[row_start(w)] : -1;
    out[2 * k] = x;
    out[2 * k + 1] = x >= 0 ? vid_of[x] : -1;
  }
}

// nd parts of normal rows longer than kShortRow (TH above it; shorter rows are
// ordered where they are arranged): insertion sort by neighbour degree,
// highest first, ties by delegate ID. Parts longer than 64 entries keep
// ascending ID order.
__global__ void k_nd_sort(const uint64_t *noff, int32_t n, const int32_t *did, int32_t *ncol,
                          const int32_t *vid_of, const int32_t *deg) {
  for (int64_t v = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; v < n;
       v += int64_t(gridDim.x) * blockDim.x) {
    if (did[v] >= 0) continue;
    const uint64_t w0 = noff[v], w1 = noff[v + 1];
    const int64_t b = row_start(w0) + row_first(w0), e = row_start(w1);
    if (e - row_start(w0) <= kShortRow || e - b < 2 || e - b > 64) continue;
    for (int64_t i = b + 1; i < e; ++i) {
      const int32_t x = ncol[i];
      const int32_t dx = deg[vid_of[x]];
      int64_t j = i - 1;
      while (j >= b) {
        const int32_t y = ncol[j];
        const int32_t dy = deg[vid_of[y]];
        if (dy > dx || (dy == dx && y < x)) break;
        ncol[j + 1] = y;
        --j;
      }
      ncol[j + 1] = x;
    }
  }
}

}  // namespace

int64_t rmat_pack_keys(const dsbfs_rmat_spec *sp, int B, uint64_t *keys, unsigned long long *cursor,
                       hipStream_t s);

// Builds the layout from an edge list (src, dst: g pairs), or, with rmat
// set, from the RMAT generator writing the symmetrized keys directly.
Graph *graph_create(const int32_t *src, const int32_t *dst, int64_t g, int32_t n,
                    const dsbfs_build_opts *opts, const dsbfs_allocator *alloc, hipStream_t s,
                    const dsbfs_rmat_spec *rmat) {
  if (rmat) {
    if (rmat->scale < 1 || rmat->scale > 31)
      fail(DSBFS_ERR_INVALID_ARG, "scale must be in [1, 31]");
    if (rmat->scale == 31) fail(DSBFS_ERR_RANGE, "2^31 vertices do not fit int32 IDs");
    n = int32_t(int64_t(1) << rmat->scale);
    g = rmat->num_edges;
    src = dst = nullptr;
  }
  if (n < 1) fail(DSBFS_ERR_INVALID_ARG, "num_vertices must be >= 1");
  if (g < 0) fail(DSBFS_ERR_INVALID_ARG, "num_edges must be >= 0");
  if (g > 0 && !rmat && (!src || !dst)) fail(DSBFS_ERR_INVALID_ARG, "src/dst must not be NULL");
  dsbfs_build_opts o{};
  o.threshold = 32;
  o.keep_plain_csr = 1;
  if (opts) o = *opts;
  if (o.threshold < 0) fail(DSBFS_ERR_INVALID_ARG, "threshold must be >= 0");
  if (o.skip_nn_copy != 0 && o.skip_nn_copy != 1)
    fail(DSBFS_ERR_INVALID_ARG, "skip_nn_copy must be 0 or 1");
  if (g > (int64_t(1) << 38)) fail(DSBFS_ERR_RANGE, "too many edges for the packed offsets");

  Graph *G = new Graph();
  try {
    if (alloc && alloc->alloc && alloc->free) {
      G->al.a = *alloc;
      G->al.custom = true;
    }
    HIPCHK(hipGetDevice(&G->device));
    G->stream = s;
    G->n = n;
    G->TH = o.threshold;
    const Alloc *al = &G->al;
    const int B = bits_for(n);

    // 1. edges on the device, checked and counted (or generated: step 2)
    DevBuf esrc, edst;
    const int32_t *ds = src, *dd = dst;
    if (!rmat && !o.edges_on_device && g > 0) {
      esrc.alloc(al, size_t(g) * 4, s);
      edst.alloc(al, size_t(g) * 4, s);
      HIPCHK(hipMemcpyAsync(esrc.p, src, size_t(g) * 4, hipMemcpyHostToDevice, s));
      HIPCHK(hipMemcpyAsync(edst.p, dst, size_t(g) * 4, hipMemcpyHostToDevice, s));
      ds = esrc.as<int32_t>();
      dd = edst.as<int32_t>();
    }
    DevBuf ctr;
    ctr.alloc(al, 16 * sizeof(unsigned long long), s);
    HIPCHK(hipMemsetAsync(ctr.p, 0, 16 * sizeof(unsigned long long), s));
    unsigned long long *c = ctr.as<unsigned long long>();
    int64_t M2 = 2 * g;   // upper bound for the generator (self-loops are dropped)
    if (!rmat && g > 0) {
      hipLaunchKernelGGL(k_count_pairs, dim3(grid_for(g, kBS * kPackItems, 2048)), dim3(kBS), 0, s,
                         ds, dd, g, n, c);
      HIPCHK(hipGetLastError());
      unsigned long long hc[2];
      HIPCHK(hipMemcpyAsync(hc, c, sizeof(hc), hipMemcpyDeviceToHost, s));
      HIPCHK(hipStreamSynchronize(s));
      if (hc[0]) fail(DSBFS_ERR_INVALID_ARG, "edge endpoint outside [0, num_vertices)");
      M2 = 2 * int64_t(hc[1]);
    }

    // 2. symmetrize into keys, sort, de-duplicate
    DevBuf keys, alt;
    keys.alloc(al, size_t(M2) * 8, s);
    alt.alloc(al, size_t(M2) * 8, s);
    if (rmat) {
      M2 = rmat_pack_keys(rmat, B, keys.as<uint64_t>(), c, s);
    } else if (M2 > 0) {
      hipLaunchKernelGGL(k_pack, dim3(grid_for(g, kBS * kPackItems, 8192)), dim3(kBS), 0, s, ds,
                         dd, g, B, keys.as<uint64_t>(), c);
      HIPCHK(hipGetLastError());
    }
    esrc.reset();
    edst.reset();
    // 3. plain CSR and degrees: the sorted keys' distinct ones
    int64_t m = 0;
    {
      DevBuf tmp;
      tmp.alloc(al, std::max(radix_tmp_bytes(M2), unique_tmp_bytes(M2)), s);
      if (radix_sort_u64_bits(keys.as<uint64_t>(), alt.as<uint64_t>(), M2, 0, 2 * B, tmp.p, s) !=
          keys.as<uint64_t>())
        std::swap(keys, alt);
      alt.reset();
      int64_t *cnt = reinterpret_cast<int64_t *>(c + 2);
      unique_count_u64(keys.as<uint64_t>(), M2, cnt, tmp.p, s);
      m = d2h_scalar(cnt, s);
      G->m = m;
      G->poff.alloc(al, size_t(n + 1) * 8, s);
      G->pcol.alloc(al, size_t(m) * 4, s);
      G->deg.alloc(al, size_t(n) * 4, s);
      unique_to_csr(keys.as<uint64_t>(), M2, m, B, n, G->poff.as<int64_t>(),
                    G->pcol.as<int32_t>(), tmp.p, s);
    }
    keys.reset();
    hipLaunchKernelGGL(k_degrees, dim3(grid_for(n, kBS, 16384)), dim3(kBS), 0, s,
                       G->poff.as<int64_t>(), n, G->deg.as<int32_t>());
    HIPCHK(hipGetLastError());

    // 4. degree separation: delegate iff degree > TH, IDs in ascending vertex ID
    DevBuf flag, tmp;
    flag.alloc(al, size_t(n), s);
    tmp.alloc(al, compact_tmp_bytes(n), s);
    G->vid_of.alloc(al, size_t(n) * 4, s);  // shrunk below once d is known
    G->did.alloc(al, size_t(n) * 4, s);
    hipLaunchKernelGGL(k_flag_gt, dim3(grid_for(n, kBS, 8192)), dim3(kBS), 0, s,
                       G->deg.as<int32_t>(), n, o.threshold, flag.as<uint8_t>());
    HIPCHK(hipGetLastError());
    int64_t *cnt = reinterpret_cast<int64_t *>(c + 2);
    compact_flags_u8(flag.as<uint8_t>(), n, G->vid_of.as<int32_t>(), cnt, tmp.p, s);
    const int64_t d = d2h_scalar(cnt, s);
    G->d = int32_t(d);
    {
      DevBuf v2;
      v2.alloc(al, size_t(d) * 4, s);
      if (d > 0)
        HIPCHK(hipMemcpyAsync(v2.p, G->vid_of.p, size_t(d) * 4, hipMemcpyDeviceToDevice, s));
      G->vid_of = std::move(v2);
    }
    hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(n, kBS, 8192)), dim3(kBS), 0, s,
                       G->did.as<int32_t>(), int64_t(n), -1);
    HIPCHK(hipGetLastError());
    if (d > 0) {
      hipLaunchKernelGGL(k_did_scatter, dim3(grid_for(d, kBS, 8192)), dim3(kBS), 0, s,
                         G->vid_of.as<int32_t>(), int32_t(d), G->did.as<int32_t>());
      HIPCHK(hipGetLastError());
    }

    // 5. columns into the split rows (and the plain rows by neighbour degree,
    //    highest first: a bottom-up pass over them meets hubs first). dd parts
    //    come by degree bucket, nd parts by degree; the four subgraphs do not
    //    depend on the order.
    DevBuf cnt_del, nstart, dstart;
    cnt_del.alloc(al, size_t(n) * 4, s);
    nstart.alloc(al, size_t(n + 1) * 8, s);
    dstart.alloc(al, size_t(d + 1) * 8, s);
    {
      DevBuf nlen, dlen, stmp;
      nlen.alloc(al, size_t(n) * 4, s);
      dlen.alloc(al, size_t(d) * 4, s);
      stmp.alloc(al, scan_tmp_bytes(std::max<int64_t>(n, d)), s);
      hipLaunchKernelGGL(k_row_lengths, dim3(grid_for(n, kBS, 8192)), dim3(kBS), 0, s,
                         G->deg.as<int32_t>(), G->did.as<int32_t>(), G->vid_of.as<int32_t>(), n,
                         int32_t(d), nlen.as<int32_t>(), dlen.as<int32_t>());
      HIPCHK(hipGetLastError());
      scan_excl_i32_to_i64(nlen.as<int32_t>(), nstart.as<int64_t>(), n, stmp.p, s);
      scan_excl_i32_to_i64(dlen.as<int32_t>(), dstart.as<int64_t>(), d, stmp.p, s);
    }
    const int64_t ncols = d2h_scalar(nstart.as<int64_t>() + n, s);
    G->ncol.alloc(al, size_t(ncols) * 4, s);
    G->dcol.alloc(al, size_t(m - ncols) * 4, s);
    {
      DevBuf code, rows, sorted;
      code.alloc(al, size_t(n), s);
      G->drank.alloc(al, size_t(G->nwords()) * sizeof(RankDir), s);
      if (o.keep_plain_csr) sorted.alloc(al, size_t(m) * 4, s);
      hipLaunchKernelGGL(k_codes, dim3(grid_for(n, kBS, 8192)), dim3(kBS), 0, s,
                         G->deg.as<int32_t>(), G->did.as<int32_t>(), n, o.threshold,
                         code.as<uint8_t>(), G->drank.as<RankDir>());
      HIPCHK(hipGetLastError());
      Arrange a{};
      a.poff = G->poff.as<int64_t>();
      a.pcol = G->pcol.as<int32_t>();
      a.code = code.as<uint8_t>();
      a.rank = G->drank.as<RankDir>();
      a.deg = G->deg.as<int32_t>();
      a.did = G->did.as<int32_t>();
      a.nstart = nstart.as<int64_t>();
      a.dstart = dstart.as<int64_t>();
      a.n = n;
      a.bth = int32_t(deg_bucket(o.threshold));
      a.plain = sorted.as<int32_t>();
      a.ncol = G->ncol.as<int32_t>();
      a.dcol = G->dcol.as<int32_t>();
      a.cnt_del = cnt_del.as<int32_t>();
      hipLaunchKernelGGL(k_rows_short, dim3(grid_for(n, 16 * kBS / kWave, 4096)), dim3(kBS), 0, s,
                         a);
      HIPCHK(hipGetLastError());
      rows.alloc(al, size_t(n) * 4, s);
      hipLaunchKernelGGL(k_flag_gt, dim3(grid_for(n, kBS, 8192)), dim3(kBS), 0, s,
                         G->deg.as<int32_t>(), n, kShortRow, flag.as<uint8_t>());
      HIPCHK(hipGetLastError());
      compact_flags_u8(flag.as<uint8_t>(), n, rows.as<int32_t>(), cnt, tmp.p, s);
      hipLaunchKernelGGL(k_rows_long, dim3(4096), dim3(kBS), 0, s, a, rows.as<int32_t>(), cnt);
      HIPCHK(hipGetLastError());
      hipLaunchKernelGGL(k_flag_gt, dim3(grid_for(n, kBS, 8192)), dim3(kBS), 0, s,
                         G->deg.as<int32_t>(), n, kHugeRow, flag.as<uint8_t>());
      HIPCHK(hipGetLastError());
      compact_flags_u8(flag.as<uint8_t>(), n, rows.as<int32_t>(), cnt, tmp.p, s);
      hipLaunchKernelGGL(k_rows_huge, dim3(512), dim3(kHugeBS), 0, s, a, rows.as<int32_t>(), cnt);
      HIPCHK(hipGetLastError());
      HIPCHK(hipStreamSynchronize(s));
      if (o.keep_plain_csr) std::swap(G->pcol, sorted);
    }
    if (!o.keep_plain_csr) {
      G->poff.reset();
      G->pcol.reset();
    }

    // 6. statistics and the packed-offset range check
    HIPCHK(hipMemsetAsync(c, 0, 9 * sizeof(unsigned long long), s));
    hipLaunchKernelGGL(k_stats, dim3(grid_for(n, kBS, 1024)), dim3(kBS), 0, s,
                       G->deg.as<int32_t>(), G->did.as<int32_t>(), cnt_del.as<int32_t>(), n, c);
    HIPCHK(hipGetLastError());
    unsigned long long hs[9];
    HIPCHK(hipMemcpyAsync(hs, c, sizeof(hs), hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    if (int64_t(hs[7]) > kMaxFirstPart)
      fail(DSBFS_ERR_RANGE, "a vertex degree exceeds the packed row-offset limit (2^24-1)");

    // 7. row offsets of the two row sets
    {
      G->noff.alloc(al, size_t(n + 1) * 8, s);
      G->doff.alloc(al, size_t(d + 1) * 8, s);
      hipLaunchKernelGGL(k_pack_offsets, dim3(grid_for(n + 1, kBS, 8192)), dim3(kBS), 0, s,
                         nstart.as<int64_t>(), dstart.as<int64_t>(), G->deg.as<int32_t>(),
                         G->did.as<int32_t>(), G->vid_of.as<int32_t>(), cnt_del.as<int32_t>(), n,
                         int32_t(d), G->noff.as<uint64_t>(), G->doff.as<uint64_t>());
      HIPCHK(hipGetLastError());
      G->nlen.alloc(al, size_t(n) * 2, s);
      hipLaunchKernelGGL(k_pack_lens, dim3(grid_for(n, kBS, 8192)), dim3(kBS), 0, s,
                         G->deg.as<int32_t>(), G->did.as<int32_t>(), cnt_del.as<int32_t>(), n,
                         G->nlen.as<uint16_t>());
      HIPCHK(hipGetLastError());
      // (the copy below is the largest a build of few edges ever is)
      nstart.reset();
      dstart.reset();
      flag.reset();
    }
    const int64_t e_nn = hs[0], e_nd = hs[1], e_dn = hs[2], e_dd = hs[3];
    // 8. compact copy of the nn parts (the forward nn visit's rows), while
    //     its 32-bit starts can address it
    if (e_nn < (int64_t(1) << 32) && !o.skip_nn_copy) {
      DevBuf cnt_nn, start, stmp;
      cnt_nn.alloc(al, size_t(n) * 4, s);
      start.alloc(al, size_t(n + 1) * 8, s);
      stmp.alloc(al, scan_tmp_bytes(n), s);
      hipLaunchKernelGGL(k_nn_counts, dim3(grid_for(n, kBS, 8192)), dim3(kBS), 0, s,
                         G->deg.as<int32_t>(), G->did.as<int32_t>(), cnt_del.as<int32_t>(), n,
                         cnt_nn.as<int32_t>());
      HIPCHK(hipGetLastError());
      scan_excl_i32_to_i64(cnt_nn.as<int32_t>(), start.as<int64_t>(), n, stmp.p, s);
      G->nnoff.alloc(al, size_t(n) * 4, s);
      G->nncol.alloc(al, size_t(std::max<int64_t>(e_nn, 1)) * 4, s);
      hipLaunchKernelGGL(k_nn_fill, dim3(grid_for(n, kBS, 8192)), dim3(kBS), 0, s,
                         start.as<int64_t>(), cnt_nn.as<int32_t>(), G->noff.as<uint64_t>(),
                         G->ncol.as<int32_t>(), n, G->nnoff.as<uint32_t>(),
                         G->nncol.as<int32_t>());
      HIPCHK(hipGetLastError());
      HIPCHK(hipStreamSynchronize(s));
    }

    G->dd_first.alloc(al, size_t(d) * 8, s);
    if (d > 0) {
      hipLaunchKernelGGL(k_dd_first, dim3(grid_for(d, kBS, 4096)), dim3(kBS), 0, s,
                         G->doff.as<uint64_t>(), G->dcol.as<int32_t>(), G->vid_of.as<int32_t>(),
                         int32_t(d), G->dd_first.as<int32_t>());
      HIPCHK(hipGetLastError());
    }
    if (d > 0 && e_nd > 1 && o.threshold > kShortRow) {
      hipLaunchKernelGGL(k_nd_sort, dim3(grid_for(n, kBS, 16384)), dim3(kBS), 0, s,
                         G->noff.as<uint64_t>(), n, G->did.as<int32_t>(), G->ncol.as<int32_t>(),
                         G->vid_of.as<int32_t>(), G->deg.as<int32_t>());
      HIPCHK(hipGetLastError());
    }

    // 9. source list of nd, source masks of dd and dn
    flag.alloc(al, size_t(n), s);
    hipLaunchKernelGGL(k_flag_ndsrc, dim3(grid_for(n, kBS, 8192)), dim3(kBS), 0, s,
                       G->did.as<int32_t>(), cnt_del.as<int32_t>(), n, flag.as<uint8_t>());
    HIPCHK(hipGetLastError());
    G->ndsrc.alloc(al, size_t(hs[4]) * 4, s);
    compact_flags_u8(flag.as<uint8_t>(), n, G->ndsrc.as<int32_t>(), cnt, tmp.p, s);
    hipLaunchKernelGGL(k_flag_nnsrc, dim3(grid_for(n, kBS, 8192)), dim3(kBS), 0, s,
                       G->deg.as<int32_t>(), G->did.as<int32_t>(), cnt_del.as<int32_t>(), n,
                       flag.as<uint8_t>());
    HIPCHK(hipGetLastError());
    G->nnsrc.alloc(al, size_t(hs[8]) * 4, s);
    compact_flags_u8(flag.as<uint8_t>(), n, G->nnsrc.as<int32_t>(), cnt, tmp.p, s);
    {
      const int64_t nsrc = int64_t(hs[4]);
      DevBuf len, stmp;
      len.alloc(al, size_t(nsrc) * 4, s);
      stmp.alloc(al, scan_tmp_bytes(nsrc), s);
      G->nds_off.alloc(al, size_t(nsrc + 1) * 8, s);
      G->nds_col.alloc(al, size_t(e_nd) * 4, s);
      G->nds_first.alloc(al, size_t(nsrc) * 8, s);
      G->nrank.alloc(al, size_t(G->nwords()) * sizeof(RankDir), s);
      HIPCHK(hipMemsetAsync(G->nrank.p, 0, size_t(G->nwords()) * sizeof(RankDir), s));
      if (nsrc > 0) {
        hipLaunchKernelGGL(k_nd_rank, dim3(grid_for(nsrc, kBS, 8192)), dim3(kBS), 0, s,
                           G->ndsrc.as<int32_t>(), nsrc, G->nrank.as<RankDir>());
        hipLaunchKernelGGL(k_nds_len, dim3(grid_for(nsrc, kBS, 8192)), dim3(kBS), 0, s,
                           G->ndsrc.as<int32_t>(), nsrc, cnt_del.as<int32_t>(),
                           len.as<int32_t>());
        HIPCHK(hipGetLastError());
      }
      scan_excl_i32_to_i64(len.as<int32_t>(), G->nds_off.as<int64_t>(), nsrc, stmp.p, s);
      if (nsrc > 0) {
        hipLaunchKernelGGL(k_nds_fill, dim3(grid_for(nsrc, kBS, 16384)), dim3(kBS), 0, s,
                           G->ndsrc.as<int32_t>(), nsrc, G->noff.as<uint64_t>(),
                           G->ncol.as<int32_t>(), G->vid_of.as<int32_t>(),
                           G->nds_off.as<int64_t>(), G->nds_col.as<int32_t>(),
                           G->nds_first.as<int32_t>());
        HIPCHK(hipGetLastError());
      }
      HIPCHK(hipStreamSynchronize(s));
    }
    G->ddsrc_mask.alloc(al, size_t(G->dwords()) * 4, s);
    G->dnsrc_mask.alloc(al, size_t(G->dwords()) * 4, s);
    if (d > 0) {
      hipLaunchKernelGGL(k_source_masks, dim3(grid_for(G->dwords(), kBS, 4096)), dim3(kBS), 0, s,
                         G->vid_of.as<int32_t>(), G->deg.as<int32_t>(), cnt_del.as<int32_t>(),
                         int32_t(d), G->ddsrc_mask.as<uint32_t>(), G->dnsrc_mask.as<uint32_t>());
      HIPCHK(hipGetLastError());
    }
    HIPCHK(hipStreamSynchronize(s));

    dsbfs_graph_stats &st = G->st;
    std::memset(&st, 0, sizeof(st));
    st.n = n;
    st.m_dir = m;
    st.d = d;
    st.e_nn = e_nn; st.e_nd = e_nd; st.e_dn = e_dn; st.e_dd = e_dd;
    st.n_ndsrc = hs[4]; st.n_ddsrc = hs[5]; st.n_dnsrc = hs[6];
    st.max_degree = hs[7];
    st.n_nnsrc = int64_t(hs[8]);
    st.threshold = o.threshold;
    // the four subgraphs; the source-list-ordered nd copy is reported apart
    st.bytes_layout = int64_t(n + 1) * 8 + int64_t(d + 1) * 8 + 4 * m;
    st.bytes_plain = o.keep_plain_csr ? int64_t(n + 1) * 8 + 4 * m : 0;
    return G;
  } catch (...) {
    delete G;
    throw;
  }
}

void graph_destroy(Graph *G) { delete G; }

void graph_export(const Graph *G, int32_t which, void *host_out, int64_t cap, int64_t *bytes) {
  const DevBuf *b = nullptr;
  int64_t nb = 0;
  const int64_t n = G->n, d = G->d;
  switch (which) {
    case 0: b = &G->deg; nb = n * 4; break;
    case 1: b = &G->did; nb = n * 4; break;
    case 2: b = &G->vid_of; nb = d * 4; break;
    case 3: b = &G->noff; nb = (n + 1) * 8; break;
    case 4: b = &G->ncol; nb = (G->st.e_nn + G->st.e_nd) * 4; break;
    case 5: b = &G->doff; nb = (d + 1) * 8; break;
    case 6: b = &G->dcol; nb = (G->st.e_dn + G->st.e_dd) * 4; break;
    case 7: b = &G->ndsrc; nb = G->st.n_ndsrc * 4; break;
    case 8: b = &G->ddsrc_mask; nb = int64_t(G->dwords()) * 4; break;
    case 9: b = &G->dnsrc_mask; nb = int64_t(G->dwords()) * 4; break;
    case 10: b = &G->poff; nb = G->poff.p ? (n + 1) * 8 : 0; break;
    case 11: b = &G->pcol; nb = G->pcol.p ? G->m * 4 : 0; break;
    case 12: b = &G->nds_off; nb = (G->st.n_ndsrc + 1) * 8; break;
    case 13: b = &G->nds_col; nb = G->st.e_nd * 4; break;
    case 14: b = &G->nds_first; nb = G->st.n_ndsrc * 8; break;
    case 15: b = &G->dd_first; nb = d * 8; break;
    case 16: b = &G->nlen; nb = n * 2; break;
    case 17: b = &G->nnsrc; nb = G->st.n_nnsrc * 4; break;
    case 18: b = &G->nnoff; nb = G->nnoff.p ? n * 4 : 0; break;
    case 19: b = &G->nncol; nb = G->nncol.p ? G->st.e_nn * 4 : 0; break;
    default: fail(DSBFS_ERR_INVALID_ARG, "unknown array index");
  }
  *bytes = nb;
  if (!host_out || cap < nb || nb == 0) return;
  HIPCHK(hipMemcpyAsync(host_out, b->p, size_t(nb), hipMemcpyDeviceToHost, G->stream));
  HIPCHK(hipStreamSynchronize(G->stream));
}

}  // namespace dsbfs
