// Graph ingest: CSR validation and packing of weight-sorted arcs.
//
// The graph model of Section 2 is an undirected graph with positive integer
// weights.  A symmetric CSR is validated (columns in range, rows strictly
// increasing, no self loops, weights >= 1, every arc matched by its reverse
// with the same weight) and each arc is packed as (w << 32) | col.  Rows are
// then re-sorted by (w, col) so that the light arcs of a node (w <= Delta,
// Section 3) are a prefix of its row, and the heavy ones a suffix.
#include <string.h>

#include <utility>
#include <vector>

#include "common.h"

namespace cld {
size_t scan_ws_bytes(int64_t n);
size_t radix_ws_bytes(int64_t n);
int radix_sort_u64(uint64_t *keys, uint64_t *vals, int64_t n, int begin_bit, int end_bit, uint64_t *ktmp,
                   uint64_t *vtmp, bool *in_tmp, void *ws, size_t ws_bytes, hipStream_t stream);
}  // namespace cld

namespace {

constexpr int kT = 256;
constexpr int kTile = 2048;       // arcs of one validation tile
// A tile that spans more rows searches for those of its arcs: some 100 dependent
// reads a thread, where visiting 16 rows per arc of the tile is 128 that overlap
// (324 and 328 us for a 512 x 512 mesh with 63 nodes without arcs after each).
constexpr int kWalkRows = 8 * kTile;
constexpr int kThreadRow = 16;    // rows of up to 8 or 16 arcs: sorting network of one thread
constexpr int kWaveRow = 64;      // ... one arc per lane of a wave
constexpr int kWaveRow4 = 256;    // ... four
constexpr int kBlockRow = 2048;   // ... bitonic sort in 16 KB of LDS, 256 threads
constexpr int kLdsRow = 8192;     // ... in 64 KB, 1024 threads
constexpr int64_t kBatchArcs = (int64_t)1 << 26;   // hub-row arcs sorted together (at least n)

enum : uint32_t {
  BAD_ROWPTR = 1, BAD_COL = 2, BAD_SELF = 4, BAD_ORDER = 8, BAD_WEIGHT = 16, BAD_ASYM = 32,
};

// Row size classes that are sorted from lists.
enum : int { ROWS_WAVE = 0, ROWS_WAVE4 = 1, ROWS_BLOCK = 2, ROWS_LDS = 3, ROWS_BIG = 4, ROW_CLASSES = 5 };

struct IngestCtl {
  uint32_t bad;
  uint32_t count[ROW_CLASSES];
  uint32_t wbits;   // all weights, or'ed
  uint32_t pad;
  unsigned long long wsum;
  unsigned long long diff;   // arcs that look their reverse up minus arcs that are looked up (mod 2^64)
};

// Checks the row offsets: two reads a row, whatever they hold.
__global__ void __launch_bounds__(kT) k_check_rows(const int64_t *rp, int32_t n, int64_t m, IngestCtl *ctl) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t a0 = rp[i], a1 = rp[i + 1];
    bool ok = a0 <= a1 && a0 >= 0 && a1 <= m;
    if (i == 0) ok = ok && a0 == 0;
    if (i == n - 1) ok = ok && a1 == m;
    if (!ok) atomicOr(&ctl->bad, BAD_ROWPTR);
  }
}

// The row that arc a lies in: the last of the n rows to start at or before a
// (rows without arcs that start there come before it).  The offsets have been
// checked.  Every lane of the wave calls it with the same arguments; each step
// samples 64 offsets, three to five dependent reads in all.
__device__ __forceinline__ int32_t row_of_arc(const int64_t *rp, int32_t n, int64_t a) {
  const int64_t lane = threadIdx.x & 63;
  int64_t lo = 0, hi = n;   // rp[lo] <= a < rp[hi]
  while (hi - lo > 1) {
    const int64_t step = (hi - lo + 63) >> 6, p = lo + lane * step;
    lo += (__popcll(__ballot(p < hi && rp[p < hi ? p : lo] <= a)) - 1) * step;
    hi = lo + step < hi ? lo + step : hi;
  }
  return (int32_t)lo;
}

// The same by one thread, among the rows lo .. hi, which hold a.
__device__ __forceinline__ int32_t row_between(const int64_t *rp, int32_t lo, int32_t hi, int64_t a) {
  while (lo < hi) {
    const int32_t mid = lo + ((hi - lo + 1) >> 1);
    if (rp[mid] <= a) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Validates and packs tiles of kTile consecutive arcs, one arc per thread and
// step, so that a hub's row is spread over many workgroups (one wave per row
// left the longest row alone with 20 ms of R-MAT scale 21's ingest).  An arc's
// row comes from a maximum scan over the row starts inside the tile; the rows of
// the tile's first and last arc are searched for (noted by the row check they took
// work in the product of rows and arcs when the offsets were malformed).  A tile
// whose arcs lie more than kWalkRows rows apart, with a long run of rows without
// arcs between them, searches for each thread's rows instead of visiting them all
// (16 million such rows, at the end of a 1000 x 1000 mesh or amid it: 0.35 ms,
// 18.5 when one workgroup visited them).
//
// Bound by scattered reads: 3.5 ms for the 62M arcs of R-MAT scale 21 (far row
// offsets of every arc, a search per edge), 1.0 ms for the road-like 4096 x
// 4096 mesh, whose short rows left most lanes of a wave per row idle (8.3 ms).
//
// Symmetry: of the two arcs of an edge the one whose far row is shorter (ties:
// the smaller id) looks its reverse up there, by binary search.  When every
// look-up succeeds, the arcs looked up are as many as the look-ups (rows hold
// a column once), and all arcs are matched if no others are left: the two
// kinds of arcs must be equally many.
__global__ void __launch_bounds__(kT) k_validate_pack(const int64_t *rp, const int32_t *col, const uint32_t *w,
                                                      int32_t n, int64_t m, uint64_t *arcs, IngestCtl *ctl) {
  __shared__ int32_t row[kTile];
  __shared__ int32_t wmax[kT / 64];
  __shared__ int32_t ends[2];   // rows of the tile's first and last arc
  if (ctl->bad & BAD_ROWPTR) return;   // nothing is indexed with malformed offsets
  constexpr int kPer = kTile / kT;
  const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t tiles = (m + kTile - 1) / kTile;
  uint32_t bad = 0, wbits = 0;
  unsigned long long wsum = 0, diff = 0;
  for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
    const int64_t a0 = t * kTile;
    const int len = (int)(m - a0 < kTile ? m - a0 : kTile);
    if (wave < 2) {
      const int32_t r = row_of_arc(rp, n, wave == 0 ? a0 : a0 + len - 1);
      if (lane == 0) ends[wave] = r;
    }
    for (int i = tid; i < kTile; i += kT) row[i] = 0;
    __syncthreads();
    const int32_t row0 = ends[0], row1 = ends[1];
    if (row1 - row0 > kWalkRows) {
      int32_t r = row0;
      for (int i = tid * kPer; i < (tid + 1) * kPer && i < len; ++i) {
        if (i == tid * kPer || rp[r + 1] <= a0 + i) r = row_between(rp, r, row1, a0 + i);
        row[i] = r - row0;
      }
    } else {
      for (int64_t r = (int64_t)row0 + 1 + tid; r <= row1; r += kT) atomicMax(&row[rp[r] - a0], (int32_t)(r - row0));
      __syncthreads();
      // inclusive maximum scan, kPer consecutive entries per thread
      int32_t mx[kPer], run = 0;
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        const int32_t x = row[tid * kPer + j];
        run = x > run ? x : run;
        mx[j] = run;
      }
      int32_t incl = run;
      for (int o = 1; o < 64; o <<= 1) {
        const int32_t y = __shfl_up(incl, o);
        if (lane >= o && y > incl) incl = y;
      }
      if (lane == 63) wmax[wave] = incl;
      int32_t before = __shfl_up(incl, 1);
      if (lane == 0) before = 0;
      __syncthreads();
      for (int k = 0; k < wave; ++k) before = wmax[k] > before ? wmax[k] : before;
#pragma unroll
      for (int j = 0; j < kPer; ++j) row[tid * kPer + j] = mx[j] > before ? mx[j] : before;
    }
    __syncthreads();
#pragma unroll 2
    for (int j = 0; j < kPer; ++j) {
      const int i = j * kT + tid;
      if (i >= len) break;
      const int64_t a = a0 + i;
      const int32_t u = row0 + row[i], v = col[a];
      const uint32_t wt = w[a];
      const int64_t ua = rp[u], ub = rp[u + 1];
      wsum += wt;
      wbits |= wt;
      if (v < 0 || v >= n) { bad |= BAD_COL; continue; }
      if (a > ua && col[a - 1] >= v) bad |= BAD_ORDER;
      if (wt == 0) bad |= BAD_WEIGHT;
      arcs[a] = ((uint64_t)wt << 32) | (uint32_t)v;
      if (v == u) { bad |= BAD_SELF; continue; }
      int64_t lo = rp[v], hi = rp[v + 1];
      const int64_t du = ub - ua, dv = hi - lo;
      if (dv > du || (dv == du && v > u)) { --diff; continue; }
      ++diff;
      bool found = false;
      while (lo < hi) {
        const int64_t mid = lo + ((hi - lo) >> 1);
        const int32_t c = col[mid];
        if (c == u) { found = w[mid] == wt; break; }
        if (c < u) lo = mid + 1; else hi = mid;
      }
      if (!found) bad |= BAD_ASYM;
    }
    __syncthreads();
  }
  for (int o = 32; o >= 1; o >>= 1) {
    bad |= __shfl_xor(bad, o);
    wbits |= __shfl_xor(wbits, o);
    wsum += __shfl_xor(wsum, o);
    diff += __shfl_xor(diff, o);
  }
  if (lane == 0) {
    if (bad) atomicOr(&ctl->bad, bad);
    if (wbits) atomicOr(&ctl->wbits, wbits);
    if (wsum) atomicAdd(&ctl->wsum, wsum);
    if (diff) atomicAdd(&ctl->diff, diff);
  }
}

__device__ __forceinline__ void order(uint64_t &x, uint64_t &y) {
  const uint64_t a = x < y ? x : y, b = x < y ? y : x;
  x = a;
  y = b;
}

// Batcher's odd-even merge sort of N registers.
template <int N>
__device__ __forceinline__ void network(uint64_t (&x)[N]) {
#pragma unroll
  for (int p = 1; p < N; p <<= 1)
#pragma unroll
    for (int k = p; k >= 1; k >>= 1)
#pragma unroll
      for (int j = k % p; j + k < N; j += 2 * k)
#pragma unroll
        for (int i = 0; i < k; ++i)
          if (i + j + k < N && (i + j) / (2 * p) == (i + j + k) / (2 * p)) order(x[i + j], x[i + j + k]);
}

template <int N>
__device__ __forceinline__ void sort_row(uint64_t *row, int deg) {
  uint64_t x[N];
#pragma unroll
  for (int i = 0; i < N; ++i) x[i] = i < deg ? row[i] : ~0ull;
  network<N>(x);
#pragma unroll
  for (int i = 0; i < N; ++i)
    if (i < deg) row[i] = x[i];
}

// Rows of up to kThreadRow arcs are sorted by one thread each; longer rows are
// queued by size class, with one reservation per class for 1024 rows (one per
// wave made the counters' line the bottleneck: 0.47 instead of 0.05 ms on
// R-MAT scale 21).
constexpr int kSmallThreads = 1024;

__global__ void __launch_bounds__(kSmallThreads) k_small_sort(const int64_t *rp, int32_t n, uint64_t *arcs,
                                                              int32_t *rows, IngestCtl *ctl) {
  __shared__ uint32_t cnt[ROW_CLASSES], at0[ROW_CLASSES];
  if (ctl->bad & BAD_ROWPTR) return;
  const int64_t stride = (int64_t)gridDim.x * kSmallThreads;
  for (int64_t base = (int64_t)blockIdx.x * kSmallThreads; base < n; base += stride) {
    const int64_t u = base + threadIdx.x;
    if (threadIdx.x < ROW_CLASSES) cnt[threadIdx.x] = 0;
    int64_t a0 = 0, deg = 0;
    if (u < n) {
      a0 = rp[u];
      deg = rp[u + 1] - a0;
    }
    __syncthreads();
    int cls = -1;
    uint32_t at = 0;
    if (deg > kThreadRow) {
      cls = deg <= kWaveRow ? ROWS_WAVE
                            : (deg <= kWaveRow4 ? ROWS_WAVE4
                                                : (deg <= kBlockRow ? ROWS_BLOCK : (deg <= kLdsRow ? ROWS_LDS : ROWS_BIG)));
      at = atomicAdd(&cnt[cls], 1u);
    }
    __syncthreads();
    if (threadIdx.x < ROW_CLASSES && cnt[threadIdx.x])
      at0[threadIdx.x] = atomicAdd(&ctl->count[threadIdx.x], cnt[threadIdx.x]);
    __syncthreads();
    if (cls >= 0) rows[(int64_t)cls * n + at0[cls] + at] = (int32_t)u;
    else if (deg > 8) sort_row<16>(arcs + a0, (int)deg);
    else if (deg > 1) sort_row<8>(arcs + a0, (int)deg);
    __syncthreads();
  }
}

// One wave per row of up to 64 * E arcs: bitonic sort of E arcs per lane (arc
// e * 64 + lane), across the lanes and, from distance 64 on, within each lane.
template <int E>   // 1, 2 or 4
__global__ void __launch_bounds__(kT) k_wave_sort(const int64_t *rp, const int32_t *rows, const uint32_t *count,
                                                  uint64_t *arcs) {
  const int lane = threadIdx.x & 63;
  const uint32_t waves = gridDim.x * (kT / 64);
  for (uint32_t r = blockIdx.x * (kT / 64) + (threadIdx.x >> 6); r < *count; r += waves) {
    const int32_t u = rows[r];
    const int64_t a0 = rp[u];
    const int deg = (int)(rp[u + 1] - a0);
    uint64_t x[E];
#pragma unroll
    for (int e = 0; e < E; ++e) x[e] = e * 64 + lane < deg ? arcs[a0 + e * 64 + lane] : ~0ull;
#pragma unroll
    for (int lk = 1; lk <= 6 + (E > 1) + (E > 2); ++lk) {
      const int k = 1 << lk;
      if (k < 2 * deg) {   // else the first k / 2 arcs are all, and in order
#pragma unroll
        for (int lj = lk - 1; lj >= 0; --lj) {
          const int j = 1 << lj;
#pragma unroll
          for (int e = 0; e < E; ++e) {
            if (j >= 64) {
              const int f = e ^ (j >> 6);
              if (f > e) {
                const bool up = ((e * 64) & k) == 0, swap = (x[e] > x[f]) == up;
                const uint64_t lo = swap ? x[f] : x[e], hi = swap ? x[e] : x[f];
                x[e] = lo;
                x[f] = hi;
              }
            } else {
              const uint64_t y = __shfl_xor(x[e], j);
              const bool up = ((e * 64 + lane) & k) == 0, low = (lane & j) == 0;
              x[e] = (low == up) == (x[e] < y) ? x[e] : y;
            }
          }
        }
      }
    }
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (e * 64 + lane < deg) arcs[a0 + e * 64 + lane] = x[e];
  }
}

// One workgroup per longer row: bitonic sort in LDS.  (Every row of 33 to 8192
// arcs in the 64 KB form, two workgroups per CU, took 4.4 ms on R-MAT scale
// 21; the four classes of today take 1.4 ms.)
template <int kThreads, int kCap>
__global__ void __launch_bounds__(kThreads) k_lds_sort(const int64_t *rp, const int32_t *rows, const uint32_t *count,
                                                       uint64_t *arcs) {
  __shared__ uint64_t s[kCap];
  for (uint32_t r = blockIdx.x; r < *count; r += gridDim.x) {
    const int32_t u = rows[r];
    const int64_t a0 = rp[u];
    const int32_t deg = (int32_t)(rp[u + 1] - a0);
    int size = 1;
    while (size < deg) size <<= 1;
    for (int i = threadIdx.x; i < size; i += kThreads) s[i] = i < deg ? arcs[a0 + i] : ~(uint64_t)0;
    __syncthreads();
    for (int k = 2; k <= size; k <<= 1) {
      for (int j = k >> 1; j > 0; j >>= 1) {
        // thread i takes the i-th pair (x, x + j)
        for (int i = threadIdx.x; i < size / 2; i += kThreads) {
          const int x = ((i & ~(j - 1)) << 1) | (i & (j - 1)), y = x | j;
          const bool up = (x & k) == 0;
          const uint64_t sx = s[x], sy = s[y];
          if ((sx > sy) == up) { s[x] = sy; s[y] = sx; }
        }
        __syncthreads();
      }
    }
    for (int i = threadIdx.x; i < deg; i += kThreads) arcs[a0 + i] = s[i];
    __syncthreads();
  }
}

// Rows longer than kLdsRow arcs are sorted in batches: their arcs are copied
// side by side (with the row's ordinal in the batch as value), radix-sorted by
// arc, then stably by ordinal, which regroups every row in place with its
// arcs in order; a batch holds up to the batch capacity of arcs.
struct BigRow {
  int64_t a0;      // first arc of the row
  uint32_t start;  // its first slot in the batch
  uint32_t deg;
};

__global__ void k_big_rows(const int64_t *rp, const int32_t *big, uint32_t nbig, int64_t *out) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nbig; i += (int64_t)gridDim.x * blockDim.x) {
    const int32_t u = big[i];
    out[2 * i] = rp[u];
    out[2 * i + 1] = rp[u + 1] - rp[u];
  }
}

__global__ void k_batch_gather(const uint64_t *arcs, const BigRow *rows, uint32_t nrows, uint64_t *key,
                               uint64_t *ord) {
  for (uint32_t r = blockIdx.x; r < nrows; r += gridDim.x) {
    const BigRow b = rows[r];
    for (uint32_t j = threadIdx.x; j < b.deg; j += blockDim.x) {
      key[b.start + j] = arcs[b.a0 + j];
      ord[b.start + j] = r;
    }
  }
}

__global__ void k_batch_scatter(uint64_t *arcs, const BigRow *rows, uint32_t nrows, const uint64_t *key) {
  for (uint32_t r = blockIdx.x; r < nrows; r += gridDim.x) {
    const BigRow b = rows[r];
    for (uint32_t j = threadIdx.x; j < b.deg; j += blockDim.x) arcs[b.a0 + j] = key[b.start + j];
  }
}

int64_t batch_cap(int32_t n, int64_t m) {
  const int64_t want = kBatchArcs > (int64_t)n ? kBatchArcs : (int64_t)n;   // every row fits one batch
  return m + 1 < want ? m + 1 : want;
}

int significant(uint32_t x) {   // bits of the values 0 .. x, at least 1
  int b = 1;
  while (b < 32 && x >> b) ++b;
  return b;
}

int64_t big_rows_cap(int64_t m) { return m / (kLdsRow + 1) + 1; }

}  // namespace

extern "C" size_t cldiam_load_csr_workspace_size(int32_t n, int64_t m) {
  if (n < 1 || m < 0) return 0;
  cld::Sizer s;
  s.take<IngestCtl>(1);
  s.take<int32_t>((size_t)ROW_CLASSES * n);        // rows by size class
  const int64_t nb = big_rows_cap(m), B = batch_cap(n, m);
  s.take<int64_t>(2 * (size_t)nb);   // (offset, degree) of every big row
  s.take<BigRow>((size_t)nb);
  for (int i = 0; i < 4; ++i) s.take<uint64_t>((size_t)B);   // batch keys, ordinals and their radix buffers
  s.used += cld::radix_ws_bytes(B);
  return s.used;
}

extern "C" int cldiam_load_csr(const cldiam_csr *g, uint64_t *d_arcs, uint64_t *h_weight_sum, void *ws,
                               size_t ws_bytes, void *stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  if (!g || g->n < 1 || g->m < 0 || g->m >= ((int64_t)1 << 40) || !g->d_row_ptr || (g->m && (!g->d_col || !g->d_w || !d_arcs))) {
    cld::set_error("load_csr: invalid arguments");
    return CLDIAM_EINVAL;
  }
  const int32_t n = g->n;
  const int64_t m = g->m;
  cld::Arena a(ws, ws_bytes);
  IngestCtl *ctl = a.take<IngestCtl>(1);
  int32_t *rows = a.take<int32_t>((size_t)ROW_CLASSES * n);
  const int64_t nbcap = big_rows_cap(m), B = batch_cap(n, m);
  int64_t *binfo = a.take<int64_t>(2 * (size_t)nbcap);
  BigRow *brows = a.take<BigRow>((size_t)nbcap);
  uint64_t *bk = a.take<uint64_t>((size_t)B), *bo = a.take<uint64_t>((size_t)B);
  uint64_t *bkt = a.take<uint64_t>((size_t)B), *bot = a.take<uint64_t>((size_t)B);
  if (!ctl || !rows || !binfo || !brows || !bk || !bo || !bkt || !bot) {
    cld::set_error("load_csr: workspace of %zu bytes, %zu needed", ws_bytes, cldiam_load_csr_workspace_size(n, m));
    return CLDIAM_ENOMEM;
  }
  CLD_HIP(hipMemsetAsync(ctl, 0, sizeof(IngestCtl), stream));
  const int32_t *list[ROW_CLASSES];
  for (int c = 0; c < ROW_CLASSES; ++c) list[c] = rows + (int64_t)c * n;
  k_check_rows<<<cld::blocks_for(n, kT, 4096), kT, 0, stream>>>(g->d_row_ptr, n, m, ctl);
  CLD_LAUNCH_CHECK("k_check_rows");
  if (m > 0) {
    // malformed row offsets end the next two kernels at once
    k_validate_pack<<<cld::blocks_for(m, kTile, 4096), kT, 0, stream>>>(g->d_row_ptr, g->d_col, g->d_w, n, m, d_arcs,
                                                                       ctl);
    CLD_LAUNCH_CHECK("k_validate_pack");
    k_small_sort<<<cld::blocks_for(n, kSmallThreads, 4096), kSmallThreads, 0, stream>>>(g->d_row_ptr, n, d_arcs, rows, ctl);
    CLD_LAUNCH_CHECK("k_small_sort");
  }
  IngestCtl h;
  CLD_HIP(hipMemcpyAsync(&h, ctl, sizeof h, hipMemcpyDeviceToHost, stream));
  CLD_HIP(hipStreamSynchronize(stream));
  if (h.bad & BAD_ROWPTR) { cld::set_error("load_csr: malformed row offsets"); return CLDIAM_EINVAL; }
  if (h.diff) h.bad |= BAD_ASYM;
  if (m > 0) {
    if (h.bad) {
      cld::set_error("load_csr: malformed CSR (flags 0x%x: 1 row offsets, 2 column range, 4 self loop, "
                     "8 row order, 16 zero weight, 32 not symmetric)", h.bad);
      return CLDIAM_EINVAL;
    }
    if (h.count[ROWS_WAVE]) {
      k_wave_sort<1><<<cld::blocks_for(h.count[ROWS_WAVE], kT / 64, 8192), kT, 0, stream>>>(
          g->d_row_ptr, list[ROWS_WAVE], &ctl->count[ROWS_WAVE], d_arcs);
      CLD_LAUNCH_CHECK("k_wave_sort");
    }
    if (h.count[ROWS_WAVE4]) {
      k_wave_sort<4><<<cld::blocks_for(h.count[ROWS_WAVE4], kT / 64, 8192), kT, 0, stream>>>(
          g->d_row_ptr, list[ROWS_WAVE4], &ctl->count[ROWS_WAVE4], d_arcs);
      CLD_LAUNCH_CHECK("k_wave_sort");
    }
    if (h.count[ROWS_BLOCK]) {
      k_lds_sort<256, kBlockRow><<<cld::blocks_for(h.count[ROWS_BLOCK], 1, 8192), 256, 0, stream>>>(
          g->d_row_ptr, list[ROWS_BLOCK], &ctl->count[ROWS_BLOCK], d_arcs);
      CLD_LAUNCH_CHECK("k_lds_sort");
    }
    if (h.count[ROWS_LDS]) {
      k_lds_sort<1024, kLdsRow><<<cld::blocks_for(h.count[ROWS_LDS], 1, 4096), 1024, 0, stream>>>(
          g->d_row_ptr, list[ROWS_LDS], &ctl->count[ROWS_LDS], d_arcs);
      CLD_LAUNCH_CHECK("k_lds_sort");
    }
    const uint32_t nbig = h.count[ROWS_BIG];
    const int32_t *big = list[ROWS_BIG];
    if (nbig) {
      if ((int64_t)nbig > nbcap) { cld::set_error("load_csr: hub row count out of range"); return CLDIAM_EHIP; }
      k_big_rows<<<cld::blocks_for(nbig, kT, 1024), kT, 0, stream>>>(g->d_row_ptr, big, nbig, binfo);
      CLD_LAUNCH_CHECK("k_big_rows");
      std::vector<int64_t> info(2 * (size_t)nbig);
      CLD_HIP(hipMemcpyAsync(info.data(), binfo, 16 * (size_t)nbig, hipMemcpyDeviceToHost, stream));
      CLD_HIP(hipStreamSynchronize(stream));
      // batches of whole rows, at most B arcs each (every row has at most n - 1 < B arcs)
      std::vector<BigRow> desc(nbig);
      std::vector<std::pair<uint32_t, uint32_t>> batches;   // (first row, row count)
      int64_t fill = 0;
      uint32_t first = 0;
      for (uint32_t i = 0; i < nbig; ++i) {
        const int64_t deg = info[2 * i + 1];
        if (fill + deg > B) {
          batches.push_back({first, i - first});
          first = i;
          fill = 0;
        }
        desc[i] = {info[2 * i], (uint32_t)fill, (uint32_t)deg};
        fill += deg;
      }
      batches.push_back({first, nbig - first});
      CLD_HIP(hipMemcpyAsync(brows, desc.data(), sizeof(BigRow) * desc.size(), hipMemcpyHostToDevice, stream));
      for (const auto &bt : batches) {
        const BigRow &last = desc[bt.first + bt.second - 1];
        const int64_t total = (int64_t)last.start + last.deg;
        int ob = 1;
        while (ob < 64 && (bt.second - 1) >> ob) ++ob;
        k_batch_gather<<<bt.second < 4096 ? bt.second : 4096, 1024, 0, stream>>>(d_arcs, brows + bt.first,
                                                                                bt.second, bk, bo);
        CLD_LAUNCH_CHECK("k_batch_gather");
        // by column, weight and the row's ordinal in turn, each on its
        // significant bits (stable, so the last key counts most); the arcs are
        // the keys of the first two, the ordinals of the last
        uint64_t *k1 = bk, *o1 = bo, *k2 = bkt, *o2 = bot;
        const auto by = [&](uint64_t *&k, uint64_t *&v, uint64_t *&kt, uint64_t *&vt, int lo, int bits) {
          bool moved = false;
          const int rc = cld::radix_sort_u64(k, v, total, lo, lo + bits, kt, vt, &moved, a.base + a.used,
                                             a.cap - a.used, stream);
          if (moved) { std::swap(k, kt); std::swap(v, vt); }
          return rc;
        };
        int rc = by(k1, o1, k2, o2, 0, significant(n - 1));
        if (!rc) rc = by(k1, o1, k2, o2, 32, significant(h.wbits));
        if (!rc) rc = by(o1, k1, o2, k2, 0, ob);
        if (rc) return rc;
        k_batch_scatter<<<bt.second < 4096 ? bt.second : 4096, 1024, 0, stream>>>(d_arcs, brows + bt.first,
                                                                                 bt.second, k1);
        CLD_LAUNCH_CHECK("k_batch_scatter");
      }
      CLD_HIP(hipStreamSynchronize(stream));   // desc is read by the copies above
    }
  }
  CLD_HIP(hipStreamSynchronize(stream));
  if (h_weight_sum) *h_weight_sum = h.wsum;
  return CLDIAM_OK;
}
