// Diameter estimate (Section 4 of arXiv:1506.03265):
//   Phi_approx = Phi(G_C) + 2 * radius,
// where Phi(G_C) is the largest finite shortest-path distance between two
// nodes of the quotient graph.  G_C is small (the number of clusters), so it
// is solved exactly: every workgroup runs single-source shortest paths from
// one quotient node at a time (label-correcting relaxation with a
// deduplicated queue; all distances exact at the fixpoint), keeping distances
// and queues in LDS when they fit, in a per-workgroup workspace slice
// otherwise.
//
// A search's time is its rounds (about the hops of its longest shortest path)
// times a round's chain of reads (queue, row offsets, arcs, distance).  So a
// row is read by a group of lanes at once (one thread per row took a read's
// latency per arc, 700 in a row on R-MAT's star-like quotients), a row longer
// than kWideRow by the whole workgroup, and the quotient graph itself is copied
// to LDS where it fits beside the search's arrays.
//
// Few searches are needed: once node v's eccentricity ecc(v) is known, no node
// u of its component has a larger one than ecc(v) + d(u, v), so a node whose
// bound is not above the largest eccentricity found so far is skipped (on a
// symmetric quotient: see k_check_symmetry).  The order spreads the first sources
// over the ids.  How the searches are launched:
//   - kPilots first, one workgroup of 1024 threads per CU.  Their bounds exclude
//     nearly all others on quotients of meshes and social graphs, and on a ring or
//     a torus, whose eccentricities are all alike, none;
//   - then wide searches again if at most kFewLeft sources are left, else as many
//     of 256 threads as the card holds, which a few nodes' frontier leaves free;
//   - a quotient of short rows (fewer than kThinRow arcs a node) that the card holds
//     a search for every node of has them all at once, of 128 threads: bounds would
//     come no sooner than the results;
//   - in global memory, with longer rows, wide searches alone take sources from a
//     counter (waiting for the pilots cost 40% on 32,000 nodes of 25 arcs).
//
// A quotient of 2228 nodes and 12028 arcs takes some 320 us (1771 us with a search
// from every node, 256 threads each, one thread per row), the star-like one of R-MAT
// scale 24 60 us (356).  A ring of 1000 nodes takes 0.47 ms (1.68 with one search per
// CU throughout), of 3000 5.8 (14.4), of 13,000 192 (592), a torus of 50 x 60 0.48
// (0.93), a mesh of 55 x 55 0.39 (0.45).
#include <algorithm>
#include <mutex>
#include <numeric>
#include <vector>

#include "common.h"

namespace {

constexpr int kT = 256;
constexpr int kWideT = 1024;   // threads of a search ...
constexpr int kThinT = 256;    // ... where many are left
constexpr int kSmallT = 128;   // ... in a quotient of short rows that the card holds a search for every node of
constexpr int64_t kThinRow = 3;
constexpr int kCus = 256;
constexpr int kCuThreads = 2048;
constexpr int kPilots = kCus;        // searches that run first, for their bounds
constexpr uint32_t kFewLeft = 4 * kCus;   // wide searches follow for no more than these
constexpr int kMaxSlices = 1024;     // searches in global memory at most
constexpr size_t kLdsTotal = 160 * 1024, kLdsOwn = 2048;   // a CU's, and of a search for its own small variables
constexpr size_t kLdsBytes = kLdsTotal - kLdsOwn;          // for a search's arrays
constexpr int kLdsMaxK = 12800;  // 12.1 bytes per node -> 155 KB

// Bytes of one workgroup's distances, queues and queued set in global memory: a
// multiple of 8, so that every workgroup's 64-bit distances are aligned (a
// 64-bit atomic on an address that is not faults).
__host__ __device__ constexpr size_t slice_bytes(int32_t k) { return ((size_t)k * 20 + 7) & ~(size_t)7; }

struct ECtl {
  unsigned long long phi;   // largest eccentricity found
  uint32_t next;            // sources that the shared counter has handed out
  uint32_t bad;        // the quotient CSR is malformed: nothing is indexed with it
  uint32_t directed;   // some arc has no reverse of its weight where its row's order has it: no bounds
};

// The quotient graph in global memory.
struct Csr {
  const int64_t *rp;
  const int32_t *col;
  const uint64_t *w;
};

// The quotient CSR must have row offsets from 0 to qm, non-decreasing, and
// columns in [0, k); anything else fails the call before the APSP reads it.
__global__ void k_check_quotient(int32_t k, int64_t qm, const int64_t *rp, const int32_t *col, uint32_t *bad) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < k; i += stride) {
    bool ok = rp[i] <= rp[i + 1];
    if (i == 0) ok = ok && rp[0] == 0;
    if (i == k - 1) ok = ok && rp[k] == qm;
    if (!ok) *bad = 1u;
  }
  for (int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; a < qm; a += stride)
    if ((uint32_t)col[a] >= (uint32_t)k) *bad = 1u;
}

// The bounds on eccentricities hold where distances are the same both ways, so
// every arc's reverse is looked up, a wave per row and an arc per lane, by binary
// search in the far row.  An arc whose reverse is not where a row in ascending order
// has it makes the estimate search from every node.
__global__ void __launch_bounds__(kT) k_check_symmetry(int32_t k, Csr g, ECtl *ctl) {
  if (ctl->bad) return;   // nothing is indexed with malformed offsets
  const int64_t at = (int64_t)blockIdx.x * kT + threadIdx.x;
  bool directed = false;
  for (int64_t u = at >> 6; u < k; u += (int64_t)gridDim.x * (kT / 64)) {
    const int64_t a1 = g.rp[u + 1];
    for (int64_t a = g.rp[u] + (at & 63); a < a1; a += 64) {
      const int32_t v = g.col[a];
      int64_t lo = g.rp[v], hi = g.rp[v + 1];
      bool found = false;
      while (lo < hi) {
        const int64_t mid = lo + ((hi - lo) >> 1);
        const int32_t c = g.col[mid];
        if (c == u) { found = g.w[mid] == g.w[a]; break; }
        if (c < u) lo = mid + 1; else hi = mid;
      }
      if (!found) directed = true;
    }
  }
  if (directed) ctl->directed = 1u;
}

constexpr int kGroup = 8;      // lanes per row
constexpr int kWideRow = 128;  // longer rows are read by the whole workgroup
constexpr int kWideCap = 128;  // such rows per pass (others are read by their group)

// Distances, queues and the set of queued nodes of one workgroup's search.
template <class Id>
struct Search {
  uint64_t *dist;
  Id *queue[2];
  uint32_t *queued;   // bitmap
};

// The quotient graph copied to LDS.
struct LdsCsr {
  const uint32_t *rp;
  const uint16_t *col;
  const uint64_t *w;
};

template <class Id>
__device__ __forceinline__ void relax_arc(const Search<Id> &x, int32_t v, uint64_t nd, uint32_t *qn, Id *next) {
  if (nd >= x.dist[v]) return;
  if (nd >= atomicMin((unsigned long long *)&x.dist[v], (unsigned long long)nd)) return;
  const uint32_t bit = 1u << (v & 31);
  if (!(atomicOr(&x.queued[v >> 5], bit) & bit)) next[atomicAdd(qn, 1u)] = (Id)v;
}

template <class Id>
__device__ __forceinline__ uint64_t distance(const Search<Id> &x, int32_t u) {
  return __hip_atomic_load(&x.dist[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Exact distances from s; returns the largest finite one.
template <int T, class Graph, class Id>
__device__ __forceinline__ unsigned long long sssp_block(int32_t k, const Graph &g, int32_t s, const Search<Id> &x) {
  __shared__ uint32_t qn[2], nwide;
  __shared__ Id wide[kWideCap];
  __shared__ unsigned long long bmax;
  const int32_t tid = (int32_t)threadIdx.x, lane = tid % kGroup;
  for (int32_t v = tid; v < k; v += T) x.dist[v] = CLD_INF64;
  for (int32_t i = tid; i < (k + 31) / 32; i += T) x.queued[i] = 0;
  if (tid == 0) { qn[0] = 1; qn[1] = 0; nwide = 0; bmax = 0; }
  __syncthreads();
  if (tid == 0) { x.dist[s] = 0; x.queue[0][0] = (Id)s; x.queued[s >> 5] = 1u << (s & 31); }
  __syncthreads();
  for (int q = 0;; q ^= 1) {
    const uint32_t n = qn[q];
    if (n == 0) break;
    const Id *cur = x.queue[q];
    Id *next = x.queue[q ^ 1];
    for (uint32_t i0 = 0; i0 < n; i0 += T / kGroup) {
      const uint32_t i = i0 + (uint32_t)(tid / kGroup);
      if (i < n) {
        const int32_t u = (int32_t)cur[i];
        const auto a0 = g.rp[u], a1 = g.rp[u + 1];
        // off the set before its distance is read (the value returned is
        // waited for): an improvement after this queues u again, one before it
        // is seen by the read, which does not go through the L1
        const uint32_t bit = 1u << (u & 31);
        uint32_t was = 0;
        if (lane == 0) was = atomicAnd(&x.queued[u >> 5], ~bit);
        bool mine = (__shfl(was, 0, kGroup) & bit) != 0;
        if (a1 - a0 > kWideRow) {
          uint32_t slot = 0;
          if (lane == 0) slot = atomicAdd(&nwide, 1u);
          slot = __shfl(slot, 0, kGroup);
          mine = slot >= kWideCap;
          if (!mine && lane == 0) wide[slot] = (Id)u;
        }
        if (mine) {
          const uint64_t du = distance(x, u);
          for (auto a = a0 + lane; a < a1; a += kGroup) relax_arc(x, (int32_t)g.col[a], du + g.w[a], &qn[q ^ 1], next);
        }
      }
    }
    __syncthreads();
    const uint32_t nw = nwide < kWideCap ? nwide : kWideCap;
    for (uint32_t i = 0; i < nw; ++i) {
      const int32_t u = (int32_t)wide[i];
      const uint64_t du = distance(x, u);
      const auto a1 = g.rp[u + 1];
      for (auto a = g.rp[u] + tid; a < a1; a += T) relax_arc(x, (int32_t)g.col[a], du + g.w[a], &qn[q ^ 1], next);
    }
    __syncthreads();
    if (tid == 0) { qn[q] = 0; nwide = 0; }
    __syncthreads();
  }
  unsigned long long m = 0;
  for (int32_t v = tid; v < k; v += T)
    if (x.dist[v] != CLD_INF64 && x.dist[v] > m) m = x.dist[v];
  for (int o = 32; o >= 1; o >>= 1) {
    const unsigned long long y = __shfl_xor(m, o);
    m = y > m ? y : m;
  }
  if ((tid & 63) == 0 && m) atomicMax(&bmax, m);
  __syncthreads();
  return bmax;
}

// Bytes of a search's arrays for ids of `id` bytes, the distances first.
__host__ __device__ inline size_t search_bytes(int32_t k, size_t id) {
  return (size_t)k * 8 + (((size_t)k + 31) / 32) * 4 + 2 * (size_t)k * id;
}

template <class Id>
__device__ __forceinline__ Search<Id> place(char *base, int32_t k) {
  uint64_t *dist = (uint64_t *)base;
  uint32_t *queued = (uint32_t *)(dist + k);
  Id *q = (Id *)(queued + (k + 31) / 32);
  return Search<Id>{dist, {q, q + k}, queued};
}

// Sources of a launch: those at places first .. end - 1 in the order
// i * step mod k; workgroup b's at first + b, first + b + blocks, ..., or whichever
// is next (`shared`: a counter, 25 ns a source).  ub[v] bounds v's eccentricity from
// above.
struct Sources {
  uint32_t k, step, first, end;
  bool shared;
  uint32_t most;   // the launch makes no search where more are left
  uint64_t *ub;
  ECtl *ctl;
  __device__ __forceinline__ int32_t at(uint32_t i) const { return (int32_t)((uint64_t)i * step % k); }
  // whether no node beats the largest eccentricity found when its own is that of source i
  __device__ __forceinline__ bool excluded(uint32_t i) const {
    return !ctl->directed && __hip_atomic_load(&ub[at(i)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <=
                                 __hip_atomic_load(&ctl->phi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
};

// Whether the workgroup has any search to make: some source of its own is not
// excluded, and no more than q.most of all are.
__device__ __forceinline__ bool some_left(const Sources &q) {
  if (q.ctl->bad) return false;
  const uint32_t tid = threadIdx.x, threads = blockDim.x;
  bool some = false;
  for (uint64_t i = q.first + blockIdx.x + (uint64_t)tid * gridDim.x; i < q.end; i += (uint64_t)threads * gridDim.x)
    some = some || !q.excluded((uint32_t)i);
  if (!__syncthreads_or(some)) return false;
  if (q.most >= q.k) return true;
  if (q.ctl->directed) return false;   // nothing is ever excluded
  uint32_t left = 0;
  for (uint32_t i = q.first; i < q.end && left <= q.most; i += threads)
    left += (uint32_t)__syncthreads_count(i + tid < q.end && !q.excluded(i + tid));
  return left <= q.most;
}

template <int T, class Graph, class Id>
__device__ __forceinline__ void search_all(const Graph &g, const Search<Id> &x, const Sources &q) {
  __shared__ int32_t src;
  const int32_t k = (int32_t)q.k;
  uint64_t i = q.first + blockIdx.x;   // thread 0's place
  for (;;) {
    if (threadIdx.x == 0) {
      for (;;) {
        if (q.shared) i = q.first + (uint64_t)atomicAdd(&q.ctl->next, 1u);
        src = i < q.end ? q.at((uint32_t)i) : -1;
        if (src < 0 || !q.excluded((uint32_t)i)) break;
        i += gridDim.x;
      }
      i += gridDim.x;
    }
    __syncthreads();
    const int32_t s = src;
    if (s < 0) return;
    const unsigned long long ecc = sssp_block<T>(k, g, s, x);
    if (threadIdx.x == 0 && ecc > __hip_atomic_load(&q.ctl->phi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      atomicMax(&q.ctl->phi, ecc);
    for (int32_t v = threadIdx.x; v < k; v += T) {
      const uint64_t d = x.dist[v];
      if (d != CLD_INF64 && d + ecc >= ecc) atomicMin((unsigned long long *)&q.ub[v], (unsigned long long)(d + ecc));
    }
    __syncthreads();
  }
}

// The graph's copy follows the search's arrays (from an 8-byte boundary).
__host__ __device__ inline size_t copy_at(int32_t k) { return (search_bytes(k, 2) + 7) & ~(size_t)7; }
__host__ __device__ inline size_t resident_bytes(int32_t k, int64_t qm) {
  return copy_at(k) + (size_t)qm * 10 + ((size_t)k + 1) * 4;
}

template <int T, bool kResident>
__global__ void __launch_bounds__(T) k_apsp_lds(int64_t qm, Csr g, Sources q) {
  if (!some_left(q)) return;
  extern __shared__ uint64_t lds[];
  const int32_t k = (int32_t)q.k;
  const Search<uint16_t> x = place<uint16_t>((char *)lds, k);
  if (kResident) {
    uint64_t *w = (uint64_t *)((char *)lds + copy_at(k));
    uint32_t *rp = (uint32_t *)(w + qm);
    uint16_t *col = (uint16_t *)(rp + k + 1);
    for (int32_t a = threadIdx.x; a < (int32_t)qm; a += T) {
      w[a] = g.w[a];
      col[a] = (uint16_t)g.col[a];
    }
    for (int32_t v = threadIdx.x; v <= k; v += T) rp[v] = (uint32_t)g.rp[v];
    __syncthreads();
    search_all<T>(LdsCsr{rp, col, w}, x, q);
  } else {
    search_all<T>(g, x, q);
  }
}

template <int T>
__global__ void __launch_bounds__(T) k_apsp_global(Csr g, Sources q, char *slices) {
  if (!some_left(q)) return;
  search_all<T>(g, place<int32_t>(slices + slice_bytes((int32_t)q.k) * blockIdx.x, (int32_t)q.k), q);
}

// A step near k / golden ratio without a common divisor with k: multiples of
// it visit every node, far apart.
uint32_t spread_step(int32_t k) {
  uint32_t step = (uint32_t)((uint64_t)k * 618033989u / 1000000000u);
  if (step < 1) step = 1;
  while (std::gcd(step, (uint32_t)k) != 1) ++step;
  return step;
}

// Slices of global memory for quotients above kLdsMaxK nodes, one per workgroup.
int slices_for(int32_t k) { return k < kMaxSlices ? k : kMaxSlices; }

// Searches of T threads that the card holds with `bytes` of LDS each for arrays.
template <int T>
int resident_searches(size_t bytes) {
  const int by_lds = (int)(kLdsTotal / (bytes + kLdsOwn)), by_threads = kCuThreads / T;
  return kCus * (by_lds < by_threads ? by_lds : by_threads);
}

// The searches of q by at most `most` workgroups of T threads.  nslices: slices of
// global memory that there are for quotients above kLdsMaxK nodes.
template <int T>
int search(int64_t qm, const Csr &g, const Sources &q, char *slices, int nslices, int most, hipStream_t stream) {
  if (q.first >= q.end) return CLDIAM_OK;
  const int32_t k = (int32_t)q.k;
  int grid = (int)(q.end - q.first);
  if (grid > most) grid = most;
  if (k > kLdsMaxK) {
    if (grid > nslices) grid = nslices;   // workgroup b works in slice b
    k_apsp_global<T><<<grid, T, 0, stream>>>(g, q, slices);
    CLD_LAUNCH_CHECK("k_apsp_global");
    return CLDIAM_OK;
  }
  // wide searches take the copy of the graph where it fits at all, the others where
  // it does not cost them places
  const size_t bare = search_bytes(k, 2), with = qm <= (int64_t)kLdsBytes ? resident_bytes(k, qm) : kLdsTotal;
  const bool copy = with <= kLdsBytes && (T == kWideT || resident_searches<T>(with) == resident_searches<T>(bare));
  const int fit = resident_searches<T>(copy ? with : bare);
  if (grid > fit) grid = fit;
  if (copy) k_apsp_lds<T, true><<<grid, T, with, stream>>>(qm, g, q);
  else k_apsp_lds<T, false><<<grid, T, bare, stream>>>(qm, g, q);
  CLD_LAUNCH_CHECK("k_apsp_lds");
  return CLDIAM_OK;
}

// Fresh control block and bounds (a kernel rather than a memset node, so that a
// caller may capture the call in a graph).
__global__ void __launch_bounds__(kT) k_zero_ctl(ECtl *ctl, uint64_t *ub, int32_t k) {
  const int64_t at = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (int64_t v = at; v < k; v += (int64_t)gridDim.x * blockDim.x) ub[v] = CLD_INF64;
  if (at == 0) { ctl->phi = 0; ctl->next = 0; ctl->bad = 0; ctl->directed = 0; }
}

// Checks, APSP and readback, with the control block, the bounds and the
// `nslices` per-workgroup slices already placed.
int estimate_run(int32_t k, int64_t qm, const int64_t *rp, const int32_t *col, const uint64_t *w, uint64_t radius,
                 uint64_t *h_phi_gc, uint64_t *h_phi_approx, ECtl *ctl, uint64_t *ub, char *slices, int nslices,
                 hipStream_t stream) {
  k_zero_ctl<<<cld::blocks_for(k, kT, 256), kT, 0, stream>>>(ctl, ub, k);
  CLD_LAUNCH_CHECK("k_zero_ctl");
  k_check_quotient<<<cld::blocks_for(k > qm ? (int64_t)k : qm, kT, 1024), kT, 0, stream>>>(k, qm, rp, col,
                                                                                           &ctl->bad);
  CLD_LAUNCH_CHECK("k_check_quotient");
  const Csr g{rp, col, w};
  k_check_symmetry<<<cld::blocks_for((int64_t)k * 64, kT, 1024), kT, 0, stream>>>(k, g, ctl);
  CLD_LAUNCH_CHECK("k_check_symmetry");
  Sources q{(uint32_t)k, spread_step(k), 0, (uint32_t)k, false, (uint32_t)k, ub, ctl};
  const bool thin = qm < kThinRow * (int64_t)k, in_lds = k <= kLdsMaxK;
  int rc = CLDIAM_OK;
  if (thin && in_lds && k <= resident_searches<kSmallT>(search_bytes(k, 2))) {
    rc = search<kSmallT>(qm, g, q, slices, nslices, k, stream);
  } else if (!thin && !in_lds) {
    q.shared = true;
    rc = search<kWideT>(qm, g, q, slices, nslices, kPilots, stream);
  } else {
    q.end = (uint32_t)(k < kPilots ? k : kPilots);
    rc = search<kWideT>(qm, g, q, slices, nslices, kPilots, stream);
    q.first = q.end;
    q.end = (uint32_t)k;
    if (!rc && !thin) {
      q.most = kFewLeft;
      rc = search<kWideT>(qm, g, q, slices, nslices, kCus, stream);
      q.most = (uint32_t)k;
    }
    if (!rc) rc = search<kThinT>(qm, g, q, slices, nslices, k, stream);
  }
  if (rc) return rc;
  ECtl h;
  CLD_HIP(hipMemcpyAsync(&h, ctl, sizeof h, hipMemcpyDeviceToHost, stream));
  CLD_HIP(hipStreamSynchronize(stream));
  if (h.bad) {
    cld::set_error("estimate_diameter: malformed quotient CSR (row offsets or a column out of range)");
    return CLDIAM_EINVAL;
  }
  *h_phi_gc = h.phi;
  *h_phi_approx = h.phi + 2 * radius;
  return CLDIAM_OK;
}

// ----------------------------------------------- no-allocation variant --
// Scratch of cldiam_estimate_diameter_noalloc: the control block at offset 0,
// the bounds, then the per-workgroup APSP slices of quotients above kLdsMaxK nodes.  Each
// device holds its own copy from the library's load until the process ends.
constexpr size_t kStaticBytes = (size_t)32 << 20;
constexpr size_t kStaticCtl = 256;
constexpr size_t kStaticUb = (size_t)CLDIAM_NOALLOC_MAX_K * 8;   // the bounds, after the control block
static_assert(sizeof(ECtl) <= kStaticCtl, "control block fits its slot");
static_assert(kStaticCtl + kStaticUb + slice_bytes(CLDIAM_NOALLOC_MAX_K) <= kStaticBytes, "a slice for every k");
static __device__ __align__(256) char scratch[kStaticBytes];

// Device address of `scratch` on each device, resolved once per device with
// that device current (the host-side name is not a device address).
std::mutex g_scratch_mu;
std::vector<char *> g_scratch_ptr;

int scratch_on_current_device(char **out) {
  int dev = 0, count = 0;
  CLD_HIP(hipGetDevice(&dev));
  CLD_HIP(hipGetDeviceCount(&count));
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if ((int)g_scratch_ptr.size() < count) g_scratch_ptr.resize(count, nullptr);
  if (dev < 0 || dev >= count) { cld::set_error("estimate_diameter_noalloc: no current device"); return CLDIAM_EHIP; }
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    CLD_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    g_scratch_ptr[dev] = (char *)p;
  }
  *out = g_scratch_ptr[dev];
  return CLDIAM_OK;
}

}  // namespace

extern "C" size_t cldiam_estimate_workspace_size(int32_t k, int64_t qm) {
  (void)qm;
  if (k < 1) return 0;
  cld::Sizer s;
  s.take<ECtl>(1);
  s.take<uint64_t>((size_t)k);
  if (k > kLdsMaxK) s.take<char>(slice_bytes(k) * slices_for(k));
  return s.used;
}

extern "C" int cldiam_estimate_diameter(int32_t k, int64_t qm, const int64_t *d_qrow_ptr, const int32_t *d_qcol,
                                        const uint64_t *d_qw, uint64_t radius, uint64_t *h_phi_gc,
                                        uint64_t *h_phi_approx, void *ws, size_t ws_bytes, void *stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  if (k < 1 || qm < 0 || !d_qrow_ptr || (qm && (!d_qcol || !d_qw)) || !h_phi_gc || !h_phi_approx) {
    cld::set_error("estimate_diameter: invalid arguments");
    return CLDIAM_EINVAL;
  }
  cld::Arena a(ws, ws_bytes);
  ECtl *ctl = a.take<ECtl>(1);
  uint64_t *ub = a.take<uint64_t>((size_t)k);
  char *slices = nullptr;
  if (k > kLdsMaxK) slices = a.take<char>(slice_bytes(k) * slices_for(k));
  if (!ctl || !ub || (k > kLdsMaxK && !slices)) {
    cld::set_error("estimate_diameter: workspace of %zu bytes, %zu needed", ws_bytes,
                   cldiam_estimate_workspace_size(k, qm));
    return CLDIAM_ENOMEM;
  }
  return estimate_run(k, qm, d_qrow_ptr, d_qcol, d_qw, radius, h_phi_gc, h_phi_approx, ctl, ub, slices,
                      slices_for(k), stream);
}

extern "C" int cldiam_estimate_diameter_noalloc(int32_t k, int64_t qm, const int64_t *d_qrow_ptr,
                                                const int32_t *d_qcol, const uint64_t *d_qw, uint64_t radius,
                                                uint64_t *h_phi_gc, uint64_t *h_phi_approx, void *stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  if (k < 1 || qm < 0 || !d_qrow_ptr || (qm && (!d_qcol || !d_qw)) || !h_phi_gc || !h_phi_approx) {
    cld::set_error("estimate_diameter_noalloc: invalid arguments");
    return CLDIAM_EINVAL;
  }
  if (k > CLDIAM_NOALLOC_MAX_K) {
    cld::set_error("estimate_diameter_noalloc: k = %d above the maximum %d of the static scratch", k,
                   CLDIAM_NOALLOC_MAX_K);
    return CLDIAM_EINVAL;
  }
  char *base = nullptr;
  int rc = scratch_on_current_device(&base);
  if (rc) return rc;
  // the slices that fit (at least 1 for every k up to the maximum)
  int nslices = slices_for(k);
  if (k > kLdsMaxK) {
    const size_t fit = (kStaticBytes - kStaticCtl - kStaticUb) / slice_bytes(k);
    if ((size_t)nslices > fit) nslices = (int)fit;
  }
  return estimate_run(k, qm, d_qrow_ptr, d_qcol, d_qw, radius, h_phi_gc, h_phi_approx, (ECtl *)base,
                      (uint64_t *)(base + kStaticCtl), base + kStaticCtl + kStaticUb, nslices, stream);
}
