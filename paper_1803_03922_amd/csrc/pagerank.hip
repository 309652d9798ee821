// PageRank on the degree-separated layout.
//
// The paper names other graph primitives on degree-separated graphs as future
// work, where delegates carry multi-bit state instead of the one-bit masks of
// BFS (Sections VI-D, VII). Here the delegate state is each delegate's rank
// contribution r/deg, kept in a compact array indexed by delegate ID (the
// array that would be replicated across GPUs, as the BFS masks are); normal
// vertices keep theirs in an array indexed by vertex ID. One FP64 power
// iteration step from r to r':
//   D = rank of the degree-0 vertices (spread uniformly),
//   r'[v] = (1 - alpha) / n + alpha * (D / n + sum over neighbours u of
//           r[u] / deg(u)),
// as two kernels: the pull over normal rows (nn part from the normal array, nd
// part from the delegate array; rows have at most TH entries: one thread per
// row), and the pull over delegate rows (dd part from the delegate array, dn
// part from the normal array; a wave per row, a block per long row). Each pull
// also writes its vertex's contribution to the next step (a row's length is
// its degree), into the other of two arrays, so no kernel reads the ranks back;
// the ranks themselves are written by the last two steps only (the last one's
// L1 change needs the one before), or by every step when a tolerance asks for
// the change of each. Row sums run in a fixed order; the dangling mass and the
// L1 change are summed with atomics, whose order can move the last bits between
// runs.
//
// The dd part is 90% of the edges at RMAT 26, and on scale-free graphs most
// of its gathers land on the few highest-degree delegates, which delegate IDs
// (ascending vertex IDs) scatter over the whole contribution array. The
// delegate pull therefore reads its dd entries from a copy of the delegate
// columns in which each dd entry is the neighbour's rank by descending degree
// bucket, and gathers from the contributions stored by that rank: the hot ones
// share lines and stay in the L2, neighbouring entries of a row (ordered by
// the same buckets) share lines too, and the columns stream past (nontemporal
// loads). Rows are also taken in that order, longest first.
#include "internal.hpp"

namespace dsbfs {

namespace {

constexpr int kPB = 256;

// Sums over all vertices, in kAccParts parts on lines of their own: one atomic
// a block on a single address was served every 12.6 ns, 0.1 ms for 8192 blocks
// in each of the three kernels of a step.
constexpr int kAccParts = 64;
struct alignas(128) PrPart {
  double dangling;  // rank of degree-0 vertices after the step (spread by the next)
  double delta;     // L1 change of the step
  double pad[14];
};
struct PrAcc {
  PrPart part[kAccParts];
};

__device__ __forceinline__ double wave_sum_f64(double x) {
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, kWave);
  return x;
}

// Block sum of one double per thread, added to *dst with one atomic.
__device__ __forceinline__ void block_add_f64(double *dst, double x, double *sh) {
  x = wave_sum_f64(x);
  const int w = threadIdx.x / kWave;
  if (lane_id() == 0) sh[w] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int i = 0; i < int(blockDim.x) / kWave; ++i) t += sh[i];
    if (t != 0.0) atomicAdd(dst, t);
  }
  __syncthreads();
}

__device__ __forceinline__ void pr_clear(PrAcc *acc) {
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i < kAccParts; i += blockDim.x)
      acc->part[i].dangling = acc->part[i].delta = 0.0;
}

// Clears an accumulator and, when r is given, fills the ranks with v.
__global__ void k_pr_fill(double *r, int32_t n, double v, PrAcc *acc) {
  if (r)
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += int64_t(gridDim.x) * blockDim.x)
      r[i] = v;
  pr_clear(acc);
}

// Sort keys of the delegates: (255 - degree bucket) above the delegate ID, so
// ascending keys are descending buckets, ties by ID: the order of the entries
// of every dd part, whose columns as ranks are therefore ascending.
__global__ void k_pr_keys(const int32_t *vid_of, const int32_t *deg, int32_t d, uint64_t *keys) {
  for (int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; k < d;
       k += int64_t(gridDim.x) * blockDim.x)
    keys[k] = (uint64_t(255u - deg_bucket(deg[vid_of[k]])) << 32) | uint64_t(uint32_t(k));
}

// Rank of each delegate, the delegates in rank order, and the number of leading
// ones whose bucket is at least `bucket`.
__global__ void k_pr_ranks(const uint64_t *keys, int32_t d, uint32_t bucket, int32_t *rank,
                           int32_t *order, int32_t *lead) {
  for (int64_t r = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; r < d;
       r += int64_t(gridDim.x) * blockDim.x) {
    const int32_t k = int32_t(uint32_t(keys[r]));
    rank[k] = int32_t(r);
    order[r] = k;
    const bool in = uint32_t(keys[r] >> 32) <= 255u - bucket;
    const bool next = r + 1 < d && uint32_t(keys[r + 1] >> 32) <= 255u - bucket;
    if (in && !next) *lead = int32_t(r + 1);
    if (r == 0 && !in) *lead = 0;
  }
}

// pr_col: the delegate rows with dd entries as ranks, dn entries as they are.
__global__ void __launch_bounds__(kPB) k_pr_cols(const uint64_t *doff, const int32_t *dcol,
                                                 const int32_t *rank, int32_t d, int32_t *pcol) {
  const int l = lane_id();
  const int64_t wid = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) / kWave;
  const int64_t nw = int64_t(gridDim.x) * blockDim.x / kWave;
  for (int64_t k = wid; k < d; k += nw) {
    const uint64_t w0 = doff[k], w1 = doff[k + 1];
    const int64_t b = row_start(w0), mid = b + row_first(w0), e = row_start(w1);
    for (int64_t i = b + l; i < e; i += kWave) {
      const int32_t c = dcol[i];
      pcol[i] = i < mid ? rank[c] : c;
    }
  }
}

// Contributions of every vertex at rank x0, and the dangling mass.
__global__ void __launch_bounds__(kPB) k_pr_first(double x0, const int32_t *deg,
                                                  const int32_t *did, const int32_t *vid_of,
                                                  const int32_t *order, int32_t n, int32_t d,
                                                  double *cn, double *cd, double *cdr,
                                                  PrAcc *acc) {
  __shared__ double sh[kPB / kWave];
  double dang = 0.0;
  for (int64_t v0 = int64_t(blockIdx.x) * blockDim.x; v0 < n;
       v0 += int64_t(gridDim.x) * blockDim.x) {
    const int64_t v = v0 + threadIdx.x;
    if (v < n) {
      const int32_t dg = deg[v];
      if (dg == 0) dang += x0;
      if (did[v] < 0) cn[v] = dg > 0 ? x0 / double(dg) : 0.0;
    }
  }
  for (int64_t r = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; r < d;
       r += int64_t(gridDim.x) * blockDim.x) {
    const int32_t k = order[r];
    cd[k] = cdr[r] = x0 / double(deg[vid_of[k]]);  // a delegate has neighbours
  }
  block_add_f64(&acc->part[blockIdx.x % kAccParts].dangling, dang, sh);
}

// What one step reads and writes.
struct PrStep {
  int32_t n, d;
  double alpha;
  // contributions: normals, delegates by ID and by rank; and those of the next
  // step (cd is written by the delegate pull, which does not read it, after the
  // normal pull has)
  const double *cn, *cdr;
  double *cd, *cn1, *cdr1;
  const PrAcc *in;              // dangling mass of r
  PrAcc *out;                   // L1 change, dangling mass of r'
  PrAcc *clear;                 // the next step's `out`
  double *rank;                 // r -> r' in place, or NULL
  int delta;                    // sum |r' - r| (rank holds r)
};

// (1 - alpha) / n + alpha D / n, by every wave for itself (whole wave).
__device__ __forceinline__ double pr_base(const PrStep &a) {
  const double dang = wave_sum_f64(a.in->part[lane_id()].dangling);
  return (1.0 - a.alpha) / double(a.n) + a.alpha * dang / double(a.n);
}

__device__ __forceinline__ void pr_rank(const PrStep &a, int32_t v, double x, double &delta) {
  if (!a.rank) return;
  if (a.delta) delta += fabs(x - a.rank[v]);
  a.rank[v] = x;
}

// Normal rows: nn part (vertex IDs, normal contributions), then nd part
// (delegate IDs, delegate contributions). A thread sums its row in stored
// order, four entries at a time: four column loads, then four gathers, then
// the four additions. Slots past the row end re-load its last entry and add
// +0.0 (the partial sum is non-negative), as in the delegate pull.
constexpr int kPrRowUnroll = 4;

__global__ void __launch_bounds__(kPB) k_pr_normal(PrStep a, const uint64_t *noff,
                                                   const int32_t *ncol, const int32_t *did) {
  __shared__ double sh[kPB / kWave];
  const double *const cd = a.cd;
  const double base = pr_base(a);
  double delta = 0.0, dang = 0.0;
  pr_clear(a.clear);
  for (int64_t v0 = int64_t(blockIdx.x) * blockDim.x; v0 < a.n;
       v0 += int64_t(gridDim.x) * blockDim.x) {
    const int64_t v = v0 + threadIdx.x;
    if (v < a.n && did[v] < 0) {
      const uint64_t w0 = noff[v], w1 = noff[v + 1];
      const int64_t b = row_start(w0), mid = b + row_first(w0), e = row_start(w1);
      double s = 0.0;
      for (int64_t i0 = b; i0 < e; i0 += kPrRowUnroll) {
        int32_t c[kPrRowUnroll];
        double y[kPrRowUnroll];
#pragma unroll
        for (int u = 0; u < kPrRowUnroll; ++u) c[u] = ncol[i0 + u < e ? i0 + u : e - 1];
#pragma unroll
        for (int u = 0; u < kPrRowUnroll; ++u) {
          const int64_t j = i0 + u;
          const double g = ((j < e ? j : e - 1) < mid ? a.cn : cd)[c[u]];
          y[u] = j < e ? g : 0.0;
        }
#pragma unroll
        for (int u = 0; u < kPrRowUnroll; ++u) s += y[u];
      }
      const double x = base + a.alpha * s;
      pr_rank(a, int32_t(v), x, delta);
      a.cn1[v] = e > b ? x / double(e - b) : 0.0;
      if (e == b) dang += x;
    }
  }
  PrPart &p = a.out->part[blockIdx.x % kAccParts];
  block_add_f64(&p.delta, delta, sh);
  block_add_f64(&p.dangling, dang, sh);
}

// Delegate rows: dd part (delegate ranks, contributions by rank), then dn part
// (vertex IDs, normal contributions), U entries per lane at a time: U column
// loads, then U gathers, then the U additions, so U gathers are in flight per
// lane. A slot past the end loads the row's last entry again (no branch, so no
// wait between the loads) and adds +0.0, which leaves the non-negative partial
// sum unchanged. The lane's entries start at i0 and step by U * 64 * waves.
template <int U>
__device__ __forceinline__ double pr_pull(const PrStep &a, const int32_t *pcol, int64_t i0,
                                          int64_t mid, int64_t e, int64_t step) {
  double s = 0.0;
  for (; i0 < e; i0 += step) {
    int32_t c[U];
    double x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t j = i0 + int64_t(u) * kWave;
      c[u] = __builtin_nontemporal_load(pcol + (j < e ? j : e - 1));
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t j = i0 + int64_t(u) * kWave;
      const double v = ((j < e ? j : e - 1) < mid ? a.cdr : a.cn)[c[u]];
      x[u] = j < e ? v : 0.0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) s += x[u];
  }
  return s;
}

__device__ __forceinline__ void pr_deleg_done(const PrStep &a, int32_t k, int64_t r, int32_t v,
                                              int64_t deg, double x, double &delta) {
  pr_rank(a, v, x, delta);
  const double c = x / double(deg);  // a delegate has more than TH >= 0 neighbours
  a.cd[k] = c;
  a.cdr1[r] = c;
}

// Rows in rank order: the `lead` first (over kLeadRow entries) a block each,
// the others a wave each. One wave per row whatever its length left the pull
// waiting for the longest: RMAT 22's row of 170K entries took one wave 0.8 of
// the kernel's 0.87 ms. Eight gathers in flight cost 80 VGPRs (6 waves per
// SIMD) and beat four at 64.
constexpr int kPrUnroll = 8;
constexpr int kLeadRow = 4096;
constexpr int kDB = 512, kDW = kDB / kWave;

__global__ void __launch_bounds__(kDB) k_pr_deleg(PrStep a, const uint64_t *doff,
                                                  const int32_t *pcol, const int32_t *vid_of,
                                                  const int32_t *order, int32_t lead) {
  __shared__ double sh[kDW];
  const double base = pr_base(a);
  const int l = lane_id(), w = threadIdx.x / kWave;
  double delta = 0.0;
  for (int64_t r = blockIdx.x; r < lead; r += gridDim.x) {
    const int32_t k = order[r];
    const uint64_t w0 = doff[k], w1 = doff[k + 1];
    const int64_t b = row_start(w0), mid = b + row_first(w0), e = row_start(w1);
    const double s = wave_sum_f64(pr_pull<kPrUnroll>(
        a, pcol, b + int64_t(w) * (kPrUnroll * kWave) + l, mid, e, kDW * kPrUnroll * kWave));
    if (l == 0) sh[w] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
      double t = 0.0;
      for (int i = 0; i < kDW; ++i) t += sh[i];
      pr_deleg_done(a, k, r, vid_of[k], e - b, base + a.alpha * t, delta);
    }
    // before anything else is written to sh: the next row's sums, or, where no
    // row is left for this block, those of block_add_f64
    __syncthreads();
  }
  const int64_t nw = int64_t(gridDim.x) * kDW;
  for (int64_t r = lead + int64_t(blockIdx.x) * kDW + w; r < a.d; r += nw) {
    const int32_t k = order[r];
    const uint64_t w0 = doff[k], w1 = doff[k + 1];
    const int64_t b = row_start(w0), mid = b + row_first(w0), e = row_start(w1);
    double s;
    if (e - b <= kWave) s = pr_pull<1>(a, pcol, b + l, mid, e, kWave);
    else if (e - b <= 2 * kWave) s = pr_pull<2>(a, pcol, b + l, mid, e, 2 * kWave);
    else if (e - b <= 4 * kWave) s = pr_pull<4>(a, pcol, b + l, mid, e, 4 * kWave);
    else s = pr_pull<kPrUnroll>(a, pcol, b + l, mid, e, kPrUnroll * kWave);
    s = wave_sum_f64(s);
    if (l == 0) pr_deleg_done(a, k, r, vid_of[k], e - b, base + a.alpha * s, delta);
  }
  block_add_f64(&a.out->part[blockIdx.x % kAccParts].delta, delta, sh);
}

}  // namespace

void pagerank_run(const Graph *g, double alpha, int32_t max_iter, double tol, double *rank,
                  int32_t *iters_done, double *last_delta, hipStream_t s) {
  if (!rank) fail(DSBFS_ERR_INVALID_ARG, "rank must not be NULL");
  if (!(alpha >= 0.0 && alpha <= 1.0)) fail(DSBFS_ERR_INVALID_ARG, "alpha must be in [0, 1]");
  if (max_iter < 0) fail(DSBFS_ERR_INVALID_ARG, "max_iterations must be >= 0");
  const int32_t n = g->n, d = g->d;
  const Alloc *al = &g->al;
  if (d > 0) {
    std::lock_guard<std::mutex> lk(g->pr_mu);
    if (!g->pr_col.p) {
      DevBuf keys, alt, tmp, rank, order, lead, pcol;
      keys.alloc(al, size_t(d) * 8, s);
      alt.alloc(al, size_t(d) * 8, s);
      tmp.alloc(al, radix_tmp_bytes(d), s);
      rank.alloc(al, size_t(d) * 4, s);
      order.alloc(al, size_t(d) * 4, s);
      lead.alloc(al, 4, s);
      const int64_t ecols = g->st.e_dd + g->st.e_dn;
      pcol.alloc(al, size_t(std::max<int64_t>(ecols, 1)) * 4, s);
      const int G0 = grid_for(d, kPB, 8192);
      hipLaunchKernelGGL(k_pr_keys, dim3(G0), dim3(kPB), 0, s, g->vid_of.as<int32_t>(),
                         g->deg.as<int32_t>(), d, keys.as<uint64_t>());
      HIPCHK(hipGetLastError());
      // keys start in ascending ID order: a stable sort on the bucket field
      // alone leaves ties in ID order
      const uint64_t *sorted = radix_sort_u64_bits(keys.as<uint64_t>(), alt.as<uint64_t>(), d, 32,
                                                   40, tmp.p, s);
      hipLaunchKernelGGL(k_pr_ranks, dim3(G0), dim3(kPB), 0, s, sorted, d,
                         deg_bucket(kLeadRow), rank.as<int32_t>(), order.as<int32_t>(),
                         lead.as<int32_t>());
      HIPCHK(hipGetLastError());
      hipLaunchKernelGGL(k_pr_cols, dim3(grid_for(int64_t(d) * kWave, kPB, 8192)), dim3(kPB), 0,
                         s, g->doff.as<uint64_t>(), g->dcol.as<int32_t>(), rank.as<int32_t>(), d,
                         pcol.as<int32_t>());
      HIPCHK(hipGetLastError());
      g->pr_lead = d2h_scalar(lead.as<int32_t>(), s);
      g->pr_order = std::move(order);
      g->pr_col = std::move(pcol);
    }
  }
  // contributions; those that a pull reads while it writes the next step's are
  // kept twice, alternating by step
  DevBuf cn[2], cd, cdr[2], acc;
  for (int i = 0; i < 2; ++i) {
    cn[i].alloc(al, size_t(n) * 8, s);
    cdr[i].alloc(al, size_t(std::max(d, 1)) * 8, s);
  }
  cd.alloc(al, size_t(std::max(d, 1)) * 8, s);
  // accumulators: step i reads the dangling mass of A[i % 3] and adds into
  // A[(i + 1) % 3]; the third is cleared meanwhile
  acc.alloc(al, 3 * sizeof(PrAcc), s);
  PrAcc *A = acc.as<PrAcc>();
  const int G1 = grid_for(n, kPB, 8192);
  for (int i = 0; i < 3; ++i)
    hipLaunchKernelGGL(k_pr_fill, dim3(i == 0 ? G1 : 1), dim3(kPB), 0, s,
                       i == 0 ? rank : nullptr, n, 1.0 / double(n), A + i);
  HIPCHK(hipGetLastError());
  int32_t it = 0;
  double dl = 0.0;
  if (max_iter > 0) {
    hipLaunchKernelGGL(k_pr_first, dim3(G1), dim3(kPB), 0, s, 1.0 / double(n),
                       g->deg.as<int32_t>(), g->did.as<int32_t>(), g->vid_of.as<int32_t>(),
                       g->pr_order.as<int32_t>(), n, d, cn[0].as<double>(), cd.as<double>(),
                       cdr[0].as<double>(), A);
    HIPCHK(hipGetLastError());
  }
  for (; it < max_iter; ++it) {
    const int p = it & 1, q = p ^ 1;
    const bool last = it + 1 == max_iter;
    PrStep a{};
    a.n = n;
    a.d = d;
    a.alpha = alpha;
    a.cn = cn[p].as<double>();
    a.cd = cd.as<double>();
    a.cdr = cdr[p].as<double>();
    a.cn1 = cn[q].as<double>();
    a.cdr1 = cdr[q].as<double>();
    a.in = A + it % 3;
    a.out = A + (it + 1) % 3;
    a.rank = tol > 0.0 || it + 2 >= max_iter ? rank : nullptr;
    a.delta = tol > 0.0 || last;
    a.clear = A + (it + 2) % 3;
    hipLaunchKernelGGL(k_pr_normal, dim3(G1), dim3(kPB), 0, s, a, g->noff.as<uint64_t>(),
                       g->ncol.as<int32_t>(), g->did.as<int32_t>());
    if (d > 0)
      hipLaunchKernelGGL(k_pr_deleg, dim3(grid_for(int64_t(d) * kWave, kDB, 4096)), dim3(kDB), 0,
                         s, a, g->doff.as<uint64_t>(), g->pr_col.as<int32_t>(),
                         g->vid_of.as<int32_t>(), g->pr_order.as<int32_t>(), g->pr_lead);
    HIPCHK(hipGetLastError());
    if (tol > 0.0 || last) {
      std::vector<PrAcc> h(1);
      HIPCHK(hipMemcpyAsync(h.data(), a.out, sizeof(PrAcc), hipMemcpyDeviceToHost, s));
      HIPCHK(hipStreamSynchronize(s));
      dl = 0.0;
      for (const PrPart &x : h[0].part) dl += x.delta;
      if (tol > 0.0 && dl < tol) {
        ++it;
        break;
      }
    }
  }
  HIPCHK(hipStreamSynchronize(s));
  if (iters_done) *iters_done = it;
  if (last_delta) *last_delta = dl;
}

}  // namespace dsbfs
