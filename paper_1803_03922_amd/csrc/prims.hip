// Device-wide primitives for the graph builder and the search drivers:
// exclusive scan, order-preserving compaction and LSD radix sort of 64-bit
// keys. Tiles are wave64-native: block-level scans are built from wave
// shuffles plus one LDS slot per wave, and the radix scatter ranks keys inside
// a wave by digit matching with a ballot a bit (stable) and stages the keys in
// LDS.
#include "internal.hpp"

namespace dsbfs {

namespace {

constexpr int kBS = 256;             // threads per block of scans/compactions
constexpr int kItems = 8;            // consecutive items per thread
constexpr int64_t kTile = kBS * kItems;
constexpr int kNW = kBS / kWave;

constexpr int kRadixBS = 512;
constexpr int kRadixNW = kRadixBS / kWave;
constexpr int kRadixItems = 16;      // keys per thread
constexpr int64_t kRadixTile = int64_t(kRadixBS) * kRadixItems;
constexpr int kRadixBits = 9;        // digits of at most 9 bits
constexpr int kRadixBins = 1 << kRadixBits;

inline size_t align256(size_t b) { return (b + 255) & ~size_t(255); }
inline int64_t ntiles(int64_t N, int64_t tile) { return (N + tile - 1) / tile; }

// Exclusive scan of one value per thread over the block; *total = block sum.
__device__ int64_t block_excl_scan(int64_t v, int64_t *sh, int64_t *total) {
  const int tid = threadIdx.x, w = tid / kWave, l = tid % kWave;
  int64_t incl = wave_incl_scan(v);
  if (l == kWave - 1) sh[w] = incl;
  __syncthreads();
  if (tid == 0) {
    int64_t run = 0;
    for (int i = 0; i < kNW; ++i) {
      int64_t t = sh[i];
      sh[i] = run;
      run += t;
    }
    sh[kNW] = run;
  }
  __syncthreads();
  int64_t r = sh[w] + incl - v;
  *total = sh[kNW];
  __syncthreads();
  return r;
}

__device__ int64_t block_sum(int64_t v, int64_t *sh) {
  int64_t t;
  block_excl_scan(v, sh, &t);
  return t;
}

template <class T>
__global__ void __launch_bounds__(kBS) k_scan_reduce(const T *in, int64_t N, int64_t *bsum) {
  __shared__ int64_t sh[kNW + 1];
  const int64_t base = int64_t(blockIdx.x) * kTile + int64_t(threadIdx.x) * kItems;
  int64_t s = 0;
#pragma unroll
  for (int k = 0; k < kItems; ++k)
    if (base + k < N) s += static_cast<int64_t>(in[base + k]);
  s = block_sum(s, sh);
  if (threadIdx.x == 0) bsum[blockIdx.x] = s;
}

// (in and out may be one array: a block reads its tile before it writes it)
template <class T, class O>
__global__ void __launch_bounds__(kBS) k_scan_down(const T *in, O *out, int64_t N,
                                                    const int64_t *bscan) {
  __shared__ int64_t sh[kNW + 1];
  const int64_t base = int64_t(blockIdx.x) * kTile + int64_t(threadIdx.x) * kItems;
  T v[kItems];
  int64_t s = 0;
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    v[k] = base + k < N ? in[base + k] : T(0);
    s += static_cast<int64_t>(v[k]);
  }
  int64_t total;
  int64_t pre = block_excl_scan(s, sh, &total);
  const int64_t boff = bscan ? bscan[blockIdx.x] : 0;
  pre += boff;
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    if (base + k < N) out[base + k] = O(pre);
    pre += static_cast<int64_t>(v[k]);
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) out[N] = O(boff + total);
}

template <class T, class O = int64_t>
void scan_impl(const T *in, O *out, int64_t N, void *tmp, hipStream_t s) {
  const int64_t nb = ntiles(N, kTile);
  if (N == 0) {
    HIPCHK(hipMemsetAsync(out, 0, sizeof(O), s));
    return;
  }
  if (nb == 1) {
    hipLaunchKernelGGL((k_scan_down<T, O>), dim3(1), dim3(kBS), 0, s, in, out, N,
                       static_cast<const int64_t *>(nullptr));
    HIPCHK(hipGetLastError());
    return;
  }
  char *t = static_cast<char *>(tmp);
  int64_t *bsum = reinterpret_cast<int64_t *>(t);
  t += align256(size_t(nb) * 8);
  int64_t *bscan = reinterpret_cast<int64_t *>(t);
  t += align256(size_t(nb + 1) * 8);
  hipLaunchKernelGGL(k_scan_reduce<T>, dim3(unsigned(nb)), dim3(kBS), 0, s, in, N, bsum);
  HIPCHK(hipGetLastError());
  scan_impl<int64_t>(bsum, bscan, nb, t, s);
  hipLaunchKernelGGL((k_scan_down<T, O>), dim3(unsigned(nb)), dim3(kBS), 0, s, in, out, N,
                     static_cast<const int64_t *>(bscan));
  HIPCHK(hipGetLastError());
}

// ---- compaction -----------------------------------------------------------

struct FlagPred {
  const uint8_t *f;
  __device__ bool operator()(int64_t i) const { return f[i] != 0; }
};
struct FlagOut {
  int32_t *out;
  __device__ void operator()(int64_t pos, int64_t i) const { out[pos] = static_cast<int32_t>(i); }
};
template <class P>
__global__ void __launch_bounds__(kBS) k_compact_count(P pred, int64_t N, int64_t *bsum) {
  __shared__ int64_t sh[kNW + 1];
  const int64_t base = int64_t(blockIdx.x) * kTile + int64_t(threadIdx.x) * kItems;
  int64_t c = 0;
#pragma unroll
  for (int k = 0; k < kItems; ++k)
    if (base + k < N && pred(base + k)) ++c;
  c = block_sum(c, sh);
  if (threadIdx.x == 0) bsum[blockIdx.x] = c;
}

template <class P, class O>
__global__ void __launch_bounds__(kBS) k_compact_write(P pred, O out, int64_t N,
                                                        const int64_t *bscan, int64_t *count) {
  __shared__ int64_t sh[kNW + 1];
  const int64_t base = int64_t(blockIdx.x) * kTile + int64_t(threadIdx.x) * kItems;
  bool keep[kItems];
  int64_t c = 0;
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    keep[k] = base + k < N && pred(base + k);
    c += keep[k];
  }
  int64_t total;
  int64_t pos = block_excl_scan(c, sh, &total);
  const int64_t boff = bscan ? bscan[blockIdx.x] : 0;
  pos += boff;
#pragma unroll
  for (int k = 0; k < kItems; ++k)
    if (keep[k]) out(pos++, base + k);
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *count = boff + total;
}

template <class P, class O>
void compact_impl(P pred, O out, int64_t N, int64_t *count, void *tmp, hipStream_t s) {
  if (N == 0) {
    HIPCHK(hipMemsetAsync(count, 0, sizeof(int64_t), s));
    return;
  }
  const int64_t nb = ntiles(N, kTile);
  if (nb == 1) {
    hipLaunchKernelGGL((k_compact_write<P, O>), dim3(1), dim3(kBS), 0, s, pred, out, N,
                       static_cast<const int64_t *>(nullptr), count);
    HIPCHK(hipGetLastError());
    return;
  }
  char *t = static_cast<char *>(tmp);
  int64_t *bsum = reinterpret_cast<int64_t *>(t);
  t += align256(size_t(nb) * 8);
  int64_t *bscan = reinterpret_cast<int64_t *>(t);
  t += align256(size_t(nb + 1) * 8);
  hipLaunchKernelGGL((k_compact_count<P>), dim3(unsigned(nb)), dim3(kBS), 0, s, pred, N, bsum);
  HIPCHK(hipGetLastError());
  scan_impl<int64_t>(bsum, bscan, nb, t, s);
  hipLaunchKernelGGL((k_compact_write<P, O>), dim3(unsigned(nb)), dim3(kBS), 0, s, pred, out, N,
                     static_cast<const int64_t *>(bscan), count);
  HIPCHK(hipGetLastError());
}

// ---- distinct keys of a sorted array -> CSR ---------------------------------
// Tiles of kUniqTile keys; a wave takes its keys 64 at a time, so that reads
// and writes are coalesced and positions come from ballots.
constexpr int kUniqItems = 16;
constexpr int64_t kUniqTile = int64_t(kBS) * kUniqItems;

__device__ __forceinline__ bool uniq_at(const uint64_t *keys, int64_t i, int64_t N, uint64_t &key,
                                        uint64_t &prev) {
  key = prev = 0;
  if (i >= N) return false;
  key = keys[i];
  prev = i > 0 ? keys[i - 1] : ~key;
  return key != prev;
}

__global__ void __launch_bounds__(kBS) k_uniq_count(const uint64_t *keys, int64_t N,
                                                    int64_t *bsum) {
  __shared__ int64_t sh[kNW + 1];
  const int64_t w0 = int64_t(blockIdx.x) * kUniqTile +
                     int64_t(threadIdx.x / kWave) * (kWave * kUniqItems) + lane_id();
  int64_t c = 0;
#pragma unroll
  for (int k = 0; k < kUniqItems; ++k) {
    uint64_t key, prev;
    c += uniq_at(keys, w0 + int64_t(k) * kWave, N, key, prev);
  }
  c = block_sum(c, sh);
  if (threadIdx.x == 0) bsum[blockIdx.x] = c;
}

// Columns of the distinct keys at their positions, and the offset of every row
// that begins between a distinct key and the one before it (rows without a
// key begin where the next one does).
__global__ void __launch_bounds__(kBS) k_uniq_csr(const uint64_t *keys, int64_t N, int64_t m,
                                                  int B, int32_t n, const int64_t *bscan,
                                                  int64_t *off, int32_t *col) {
  __shared__ int wtot[kNW];
  const int w = threadIdx.x / kWave;
  const uint64_t mask = (uint64_t(1) << B) - 1;
  const int64_t w0 = int64_t(blockIdx.x) * kUniqTile + int64_t(w) * (kWave * kUniqItems) +
                     lane_id();
  uint64_t key[kUniqItems], prev[kUniqItems];
  uint64_t bal[kUniqItems];
  int tot = 0;
#pragma unroll
  for (int k = 0; k < kUniqItems; ++k) {
    bal[k] = __ballot(uniq_at(keys, w0 + int64_t(k) * kWave, N, key[k], prev[k]));
    tot += __popcll(bal[k]);
  }
  if (lane_id() == 0) wtot[w] = tot;
  __syncthreads();
  int64_t pos = bscan[blockIdx.x];
  for (int i = 0; i < w; ++i) pos += wtot[i];
#pragma unroll
  for (int k = 0; k < kUniqItems; ++k) {
    const int64_t i = w0 + int64_t(k) * kWave;
    if ((bal[k] >> lane_id()) & 1ull) {
      const int64_t p = pos + lanes_below(bal[k]);
      col[p] = int32_t(key[k] & mask);
      const int64_t row = int64_t(key[k] >> B), before = i > 0 ? int64_t(prev[k] >> B) : -1;
      for (int64_t x = before + 1; x <= row; ++x) off[x] = p;
    }
    // rows after the last key
    if (i == N - 1)
      for (int64_t x = int64_t(key[k] >> B) + 1; x <= n; ++x) off[x] = m;
    pos += __popcll(bal[k]);
  }
}

__global__ void k_fill_i64(int64_t *p, int64_t N, int64_t v) {
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < N;
       i += int64_t(gridDim.x) * blockDim.x)
    p[i] = v;
}

// ---- radix sort -----------------------------------------------------------

__global__ void __launch_bounds__(kRadixBS) k_radix_hist(const uint64_t *keys, int64_t N,
                                                          int shift, int bits, int64_t nb,
                                                          uint32_t *ghist) {
  __shared__ uint32_t hist[kRadixBins];
  const uint32_t dmask = (1u << bits) - 1u;
  hist[threadIdx.x] = 0;
  __syncthreads();
  const int64_t tile = int64_t(blockIdx.x) * kRadixTile;
#pragma unroll
  for (int r = 0; r < kRadixItems; ++r) {
    const int64_t i = tile + int64_t(r) * kRadixBS + threadIdx.x;
    if (i < N) atomicAdd(&hist[uint32_t(keys[i] >> shift) & dmask], 1u);
  }
  __syncthreads();
  if (threadIdx.x <= dmask) ghist[int64_t(threadIdx.x) * nb + blockIdx.x] = hist[threadIdx.x];
}

// Stable scatter of one tile of 8192 keys. Wave w holds the tile's keys
// [1024 w, 1024 w + 1024), 64 at a time; lanes with equal digits are matched
// with ballots, so a key's rank among the equal digits of its wave is a count
// the wave keeps in LDS plus a popcount, with no block barrier between steps.
// The keys then go to LDS in digit order and out from there: runs of the same
// digit leave as whole lines (about 16 keys, 128 bytes, of random data), where
// writing them one by one from registers kept 256 partly filled lines per
// block open in the L2. 128M keys: 1.4 ms a pass of 8 bits before, 0.8 ms a
// pass of 9 bits now (44 bits: five passes instead of six).
template <class O>
__global__ void __launch_bounds__(kRadixBS) k_radix_scatter(const uint64_t *keys, uint64_t *out,
                                                             int64_t N, int shift, int bits,
                                                             int64_t nb, const O *gscan) {
  __shared__ uint64_t stage[kRadixTile];
  __shared__ uint16_t wcnt[kRadixNW][kRadixBins];  // below 8192: two blocks fit a compute unit
  __shared__ int64_t base[kRadixBins];  // where the tile's keys of a digit go, less their
                                        // position in the tile's order
  __shared__ int wsum[kRadixNW];
  const int tid = threadIdx.x, w = tid / kWave, l = lane_id();
  const uint32_t dmask = (1u << bits) - 1u;
  const int64_t tile = int64_t(blockIdx.x) * kRadixTile;
  const int64_t w0 = tile + int64_t(w) * (kWave * kRadixItems) + l;
  uint64_t key[kRadixItems];
  int rank[kRadixItems];
#pragma unroll
  for (int r = 0; r < kRadixItems; ++r) {
    const int64_t i = w0 + int64_t(r) * kWave;
    key[r] = i < N ? keys[i] : 0;
  }
  for (int i = l; i < kRadixBins; i += kWave) wcnt[w][i] = 0;
  wave_sync();
#pragma unroll
  for (int r = 0; r < kRadixItems; ++r) {
    const bool ok = w0 + int64_t(r) * kWave < N;
    const uint32_t dig = uint32_t(key[r] >> shift) & dmask;
    uint64_t m = __ballot(ok);
    for (int b = 0; b < bits; ++b) {
      const bool bit = (dig >> b) & 1u;
      const uint64_t bal = __ballot(bit);
      m &= bit ? bal : ~bal;
    }
    const int below = int(lanes_below(m));
    if (ok) rank[r] = wcnt[w][dig] + below;
    wave_sync();
    if (ok && below == 0) wcnt[w][dig] = uint16_t(wcnt[w][dig] + __popcll(m));
    wave_sync();
  }
  __syncthreads();
  // thread = digit: prefix over the waves, then over the digits
  int total = 0;
#pragma unroll
  for (int k = 0; k < kRadixNW; ++k) {
    const int c = wcnt[k][tid];
    wcnt[k][tid] = uint16_t(total);
    total += c;
  }
  const int incl = wave_incl_scan(total);
  if (l == kWave - 1) wsum[w] = incl;
  __syncthreads();
  int first = incl - total;
  for (int k = 0; k < w; ++k) first += wsum[k];
#pragma unroll
  for (int k = 0; k < kRadixNW; ++k) wcnt[k][tid] = uint16_t(wcnt[k][tid] + first);
  if (uint32_t(tid) <= dmask) base[tid] = int64_t(gscan[int64_t(tid) * nb + blockIdx.x]) - first;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kRadixItems; ++r)
    if (w0 + int64_t(r) * kWave < N)
      stage[wcnt[w][uint32_t(key[r] >> shift) & dmask] + rank[r]] = key[r];
  __syncthreads();
  const int cnt = int(min(kRadixTile, N - tile));
  for (int i = tid; i < cnt; i += kRadixBS) {
    const uint64_t k = stage[i];
    out[base[uint32_t(k >> shift) & dmask] + i] = k;
  }
}

}  // namespace

size_t scan_tmp_bytes(int64_t N) {
  const int64_t nb = ntiles(N, kTile);
  if (nb <= 1) return 256;
  return align256(size_t(nb) * 8) + align256(size_t(nb + 1) * 8) + scan_tmp_bytes(nb);
}

void scan_excl_i32_to_i64(const int32_t *in, int64_t *out, int64_t N, void *tmp, hipStream_t s) {
  scan_impl<int32_t>(in, out, N, tmp, s);
}

size_t compact_tmp_bytes(int64_t N) { return scan_tmp_bytes(N); }

void compact_flags_u8(const uint8_t *flag, int64_t N, int32_t *out, int64_t *count, void *tmp,
                      hipStream_t s) {
  compact_impl(FlagPred{flag}, FlagOut{out}, N, count, tmp, s);
}

size_t unique_tmp_bytes(int64_t N) {
  const int64_t nb = ntiles(N, kUniqTile);
  return align256(size_t(nb) * 8) + align256(size_t(nb + 1) * 8) + scan_tmp_bytes(nb);
}

void unique_count_u64(const uint64_t *keys, int64_t N, int64_t *count, void *tmp, hipStream_t s) {
  if (N == 0) {
    HIPCHK(hipMemsetAsync(count, 0, sizeof(int64_t), s));
    return;
  }
  const int64_t nb = ntiles(N, kUniqTile);
  char *t = static_cast<char *>(tmp);
  int64_t *bsum = reinterpret_cast<int64_t *>(t);
  t += align256(size_t(nb) * 8);
  int64_t *bscan = reinterpret_cast<int64_t *>(t);
  t += align256(size_t(nb + 1) * 8);
  hipLaunchKernelGGL(k_uniq_count, dim3(unsigned(nb)), dim3(kBS), 0, s, keys, N, bsum);
  HIPCHK(hipGetLastError());
  scan_impl<int64_t>(bsum, bscan, nb, t, s);
  HIPCHK(hipMemcpyAsync(count, bscan + nb, sizeof(int64_t), hipMemcpyDeviceToDevice, s));
}

void unique_to_csr(const uint64_t *keys, int64_t N, int64_t m, int B, int32_t n, int64_t *off,
                   int32_t *col, void *tmp, hipStream_t s) {
  if (N == 0) {
    hipLaunchKernelGGL(k_fill_i64, dim3(grid_for(int64_t(n) + 1, 256, 4096)), dim3(256), 0, s, off,
                       int64_t(n) + 1, int64_t(0));
    HIPCHK(hipGetLastError());
    return;
  }
  const int64_t nb = ntiles(N, kUniqTile);
  const int64_t *bscan = reinterpret_cast<const int64_t *>(static_cast<char *>(tmp) +
                                                           align256(size_t(nb) * 8));
  hipLaunchKernelGGL(k_uniq_csr, dim3(unsigned(nb)), dim3(kBS), 0, s, keys, N, m, B, n, bscan, off,
                     col);
  HIPCHK(hipGetLastError());
}

// Up to this many keys their places fit 32 bits, and the counts are scanned where
// they are: 0.25 bytes of scratch a key instead of 0.75 (the 512 digits of a pass
// took a build that just fitted 1.5% over its limit).
constexpr int64_t kRadix32 = UINT32_MAX;

size_t radix_tmp_bytes(int64_t N) {
  const int64_t nb = ntiles(N, kRadixTile);
  const int64_t H = kRadixBins * (nb > 0 ? nb : 1);
  return (N <= kRadix32 ? align256(size_t(H + 1) * 4)
                        : align256(size_t(H) * 4) + align256(size_t(H + 1) * 8)) +
         scan_tmp_bytes(H);
}

uint64_t *radix_sort_u64_bits(uint64_t *keys, uint64_t *alt, int64_t N, int lo_bit, int hi_bit,
                              void *tmp, hipStream_t s) {
  if (N <= 1 || hi_bit <= lo_bit) return keys;
  const int64_t nb = ntiles(N, kRadixTile);
  // the fewest passes of at most kRadixBits bits, of even widths
  const int passes = (hi_bit - lo_bit + kRadixBits - 1) / kRadixBits;
  const int width = (hi_bit - lo_bit + passes - 1) / passes;
  const int64_t H = (int64_t(1) << width) * nb;
  char *t = static_cast<char *>(tmp);
  uint32_t *ghist = reinterpret_cast<uint32_t *>(t);
  t += align256(size_t(N <= kRadix32 ? H + 1 : H) * 4);
  int64_t *gscan = reinterpret_cast<int64_t *>(t);
  if (N > kRadix32) t += align256(size_t(H + 1) * 8);
  uint64_t *src = keys, *dst = alt;
  for (int shift = lo_bit; shift < hi_bit; shift += width) {
    hipLaunchKernelGGL(k_radix_hist, dim3(unsigned(nb)), dim3(kRadixBS), 0, s, src, N, shift,
                       width, nb, ghist);
    HIPCHK(hipGetLastError());
    if (N <= kRadix32) {
      scan_impl(ghist, ghist, H, t, s);
      hipLaunchKernelGGL(k_radix_scatter<uint32_t>, dim3(unsigned(nb)), dim3(kRadixBS), 0, s, src,
                         dst, N, shift, width, nb, ghist);
    } else {
      scan_impl(ghist, gscan, H, t, s);
      hipLaunchKernelGGL(k_radix_scatter<int64_t>, dim3(unsigned(nb)), dim3(kRadixBS), 0, s, src,
                         dst, N, shift, width, nb, gscan);
    }
    HIPCHK(hipGetLastError());
    uint64_t *x = src;
    src = dst;
    dst = x;
  }
  return src;
}

}  // namespace dsbfs
