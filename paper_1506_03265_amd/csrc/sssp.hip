// Delta-stepping single-source shortest paths (Meyer and Sanders), the
// competitor of Section 5 of arXiv:1506.03265: twice the largest finite
// distance from one source is a 2-approximation of the diameter.
//
// The nodes still to be relaxed are a bitmap.  One launch (a step) relaxes
// those below theta = (smallest distance in the bitmap) + delta and leaves the
// others for later steps, which orders the search by buckets of width delta.
// A workgroup owns a range of bitmap words, so it meets its nodes in ascending
// order (neighbouring nodes share cache lines), and carries the search on from
// the nodes that it improves in local rounds over an LDS queue.
//
// Every improvement of a distance is the responsibility of the thread that
// made it: it goes into the workgroup's queue, or, when it lies beyond theta,
// finds the queue full or is left over when the rounds end, into the next
// step's bitmap.  A queued improvement is dropped only when a smaller distance
// has been written since, which is some other thread's responsibility.  So at
// the end of a step every node whose distance has not been relaxed is in the
// bitmap, nodes relaxed in local rounds are not visited again, and none of the
// atomics (minimum on the distance, or on the bitmap) has to return a value.
// Distances are exact (u32, overflow checked); the schedule only changes the
// work.
//
// A row is relaxed by four lanes together, one arc each at a time: a local
// round of a few dozen nodes, the usual case, costs latency and a wave's
// instructions, which this quarters (one lane per row with four arcs in flight:
// 5.2 instead of 3.6 ms on a 700 x 900 grid, 3.0 instead of 2.0 on an R-GG of
// 100,000 nodes).  No load is under a branch of its own, so they overlap.
//
// What bounds it: the number of hops (8,600 on the road-like 4096 x 4096 mesh)
// times the chain of dependent accesses of one (queue, row offsets and
// distance, arcs, far distances: 3.5 us where they miss the L2).  That mesh
// takes 28 to 33 ms at the default width, depending on the GPU; with node lists,
// returning atomics and one hop per launch it took 190 to 205.  Looking up an
// improved node's row together with its distance, which makes the chain one
// access shorter, gained nothing (four times the offset loads).
#include <chrono>
#include <thread>

#include "common.h"

namespace {

constexpr int kT = 256;
// Eight workgroups per CU, whose chains of accesses interleave: the road-like
// 4096 x 4096 mesh takes 34.7 ms, on one GPU, with 8 of 256 threads, 43 with 4, 36.7 with 16
// (more than are resident), 43 with 4 of 512, 47 with 2 of 1024.  The list and
// the queue are no longer than lets eight share a CU's LDS.
constexpr int kStepThreads = 256;
constexpr int kBlocksPerCu = 2048 / kStepThreads;
constexpr int kList = 4 * kStepThreads;    // nodes of one expansion of a bitmap window
constexpr int kQueue = 2 * kStepThreads;   // improved nodes of one local round
constexpr int kRowLanes = 4;      // lanes that relax a row together
constexpr int kMidRow = 32;       // longer rows are relaxed by one wave ...
constexpr int kBigRow = 4096;     // ... and these by the whole workgroup
constexpr int kMidCap = kStepThreads;
constexpr int kBigCap = 64;
// Fewest bitmap words of a workgroup: as many as hold kMinArcs arcs on average, but
// no more than kMinWords (a launch of more workgroups costs more: R-MAT scale 18 at
// width 5000 takes 5.9 ms with 16 words, 6.5 with 9, 8.7 with 4).  A frontier of
// neighbouring nodes with long rows otherwise falls to one or two workgroups: a
// band of 200,000 nodes joined to the 80 nearest takes 742 ms with 6 words, 1110
// with 16, the complete graph of 3000 nodes 1.7 with one word, 14.1 with 16.
constexpr int kMinWords = 16;
constexpr int64_t kMinArcs = 16384;
// Local rounds: on sparse graphs a round carries the search a hop further for
// a quarter of a step's cost (road-like 4096 x 4096 mesh: 145 ms without, 37 with
// 16 or 32, 39 with 64 and a longer queue).  On graphs of more than kDenseDegree arcs per
// node a few hops reach everything and distances taken early are mostly
// improved again (R-MAT scale 20: 4.0 ms without, 5.3 with one round, 20 with 32).
constexpr uint32_t kRounds = 32;
constexpr int64_t kDenseDegree = 16;
constexpr uint32_t kLead = 16;    // steps that the host queues ahead of the device

// Results of one step, in a ring: step t reads slot t - 1, writes slot t and
// clears slot t + 1.
struct alignas(128) SSlot {
  uint32_t fmin;   // smallest distance in the next bitmap (CLD_INF32: none)
  uint32_t pad[31];
};

struct SCtl {
  SSlot slot[4];
  uint32_t maybe;      // some offer did not fit in 32 bits
  uint32_t overflow;   // some node's final distance plus one of its arcs does not
  unsigned long long mx;
};

struct SJob {
  const int64_t *rp;
  const uint64_t *arcs;
  int32_t n;
  uint32_t words;    // bitmap words
  uint32_t chunk;    // bitmap words of one workgroup
  uint32_t delta;
  uint32_t rounds;   // most local rounds of a step
  uint32_t *dist;
  uint32_t *front[2];
  SCtl *ctl;
  uint32_t *mirror;  // mapped host words {last step begun, done}
};

struct SStep {
  int32_t list[kList];
  uint2 queue[2][kQueue];   // (node, distance to relax it with)
  uint2 mid[kMidCap];       // rows for one wave each
  uint2 big[kBigCap];       // rows for the whole workgroup
  uint32_t qn[3];           // queued nodes, by round modulo 3
  uint32_t nmid[2], nbig[2];   // rows set aside by the even and the odd passes (see relax_long)
  uint32_t wsum[kStepThreads / 64];
  uint32_t fmin;
};

// What a thread carries through a step.
struct Walk {
  const SJob &j;
  SStep &S;
  uint32_t *next;
  uint32_t theta;
  uint32_t q = 0, qslot = 0;   // queue and counter that improvements go to
  uint32_t pass = 0;
  uint32_t fmin = CLD_INF32;   // smallest distance that this thread has left for the next step
};

__device__ __forceinline__ void leave(Walk &k, uint32_t v, uint32_t d) {
  atomicOr(&k.next[v >> 5], 1u << (v & 31));
  if (d < k.fmin) k.fmin = d;
}

// Offers u's distance du over one arc per lane (in: the lane has one).  An
// improvement is queued, one reservation per wave.  The load of the
// neighbour's distance is not under a branch (a lane without an arc reads
// node 0's): loads under branches do not overlap.
__device__ __forceinline__ void offer(Walk &k, uint32_t du, bool in, uint64_t arc) {
  const uint64_t x = (uint64_t)du + (arc >> 32);
  const bool fits = x < CLD_INF32;
  const uint32_t v = in && fits ? (uint32_t)arc : 0u, nd = (uint32_t)x, old = k.j.dist[v];
  if (in && !fits) k.j.ctl->maybe = 1u;
  const bool better = in && fits && nd < old, near = better && nd < k.theta;
  if (better) atomicMin(&k.j.dist[v], nd);
  const uint64_t m = __ballot(near);
  if (m) {
    const int first = __ffsll((long long)m) - 1;
    uint32_t base = 0;
    if ((int)(threadIdx.x & 63) == first) base = atomicAdd(&k.S.qn[k.qslot], (uint32_t)__popcll(m));
    base = (uint32_t)__builtin_amdgcn_readlane((int)base, first);
    const uint32_t slot = base + (uint32_t)__popcll(m & ((1ull << (threadIdx.x & 63)) - 1ull));
    if (near && slot < kQueue) k.S.queue[k.q][slot] = make_uint2(v, nd);
    else if (near) leave(k, v, nd);
  }
  if (better && !near) leave(k, v, nd);
}

__device__ __forceinline__ uint32_t row_lane() { return threadIdx.x & (kRowLanes - 1); }

// Relaxes u's row (degree deg, first arc a0) with distance du by the kRowLanes
// lanes of a group together, one arc each at a time.  Long rows are set aside
// for the relax_long that ends the pass.
__device__ __forceinline__ void relax_row(Walk &k, uint32_t u, uint32_t du, int64_t a0, int32_t deg) {
  if (deg > kMidRow) {
    uint32_t aside = 0;
    if (row_lane() == 0) {
      const uint32_t p = k.pass & 1;
      const uint32_t slot = atomicAdd(deg > kBigRow ? &k.S.nbig[p] : &k.S.nmid[p], 1u);
      aside = slot < (uint32_t)(deg > kBigRow ? kBigCap : kMidCap);
      if (aside) (deg > kBigRow ? k.S.big : k.S.mid)[slot] = make_uint2(u, du);
    }
    if (__shfl((int)aside, (int)(threadIdx.x & 63 & ~(kRowLanes - 1)))) return;
  }
  const uint64_t *row = k.j.arcs + a0;
  for (int32_t base = 0; base < deg; base += kRowLanes) {
    const int32_t a = base + (int32_t)row_lane();
    offer(k, du, a < deg, row[a < deg ? a : base]);
  }
}

// Ends a pass: relaxes the long rows that it set aside.  The counters alternate
// between passes: a wave that is late to read this pass's sees none of the next
// pass's rows, so every wave takes the same branch after the one barrier.
__device__ __forceinline__ void relax_long(Walk &k) {
  SStep &S = k.S;
  __syncthreads();
  const uint32_t p = k.pass++ & 1;
  const uint32_t nm = S.nmid[p] < kMidCap ? S.nmid[p] : kMidCap, nb = S.nbig[p] < kBigCap ? S.nbig[p] : kBigCap;
  if (nm == 0 && nb == 0) return;
  for (uint32_t r = threadIdx.x >> 6; r < nm; r += kStepThreads / 64) {
    const uint2 x = S.mid[r];
    const int64_t a0 = k.j.rp[x.x];
    const int32_t deg = (int32_t)(k.j.rp[x.x + 1] - a0);
    for (int32_t a = (int32_t)(threadIdx.x & 63); a < deg; a += 64) offer(k, x.y, true, k.j.arcs[a0 + a]);
  }
  for (uint32_t r = 0; r < nb; ++r) {
    const uint2 x = S.big[r];
    const int64_t a0 = k.j.rp[x.x];
    const int32_t deg = (int32_t)(k.j.rp[x.x + 1] - a0);
    for (int32_t a = (int32_t)threadIdx.x; a < deg; a += kStepThreads) offer(k, x.y, true, k.j.arcs[a0 + a]);
  }
  __syncthreads();
  if (threadIdx.x == 0) { S.nmid[p] = 0; S.nbig[p] = 0; }
  __syncthreads();
}

__global__ void __launch_bounds__(kStepThreads) k_sssp_step(SJob j, uint32_t t) {
  __shared__ SStep S;
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t low = j.ctl->slot[(t + 3) & 3].fmin;
  if (blockIdx.x == 0 && tid == 0) {
    j.ctl->slot[(t + 1) & 3].fmin = CLD_INF32;
    __hip_atomic_store(&j.mirror[0], t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (low == CLD_INF32) __hip_atomic_store(&j.mirror[1], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
  if (low == CLD_INF32) return;
  const uint32_t theta = low < CLD_INF32 - j.delta ? low + j.delta : CLD_INF32;
  uint32_t *cur = j.front[t & 1], *next = j.front[(t + 1) & 1];
  if (tid == 0) { S.qn[0] = S.qn[1] = S.qn[2] = S.nmid[0] = S.nmid[1] = S.nbig[0] = S.nbig[1] = 0; S.fmin = CLD_INF32; }
  // Workgroups go to the XCDs in turn; each XCD takes one eighth of the words,
  // so that neighbouring ranges share an L2 (2 to 6% faster than in turn).
  const uint32_t range = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  const uint32_t lo = range * j.chunk < j.words ? range * j.chunk : j.words;
  const uint32_t hi = lo + j.chunk < j.words ? lo + j.chunk : j.words;
  Walk k{j, S, next, theta};
  uint32_t ahead = lo + tid < hi ? cur[lo + tid] : 0u;
  for (uint32_t w0 = lo; w0 < hi; w0 += kStepThreads) {
    const uint32_t word = ahead, w = w0 + tid;
    ahead = w + kStepThreads < hi ? cur[w + kStepThreads] : 0u;
    if (word) cur[w] = 0;
    // position of this word's first node among the window's nodes
    uint32_t incl = __popc(word);
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(incl, o);
      if (lane >= (uint32_t)o) incl += y;
    }
    __syncthreads();
    if (lane == 63) S.wsum[wave] = incl;
    __syncthreads();
    uint32_t at = incl - __popc(word), total = 0;
    for (uint32_t i = 0; i < kStepThreads / 64; ++i) {
      if (i < wave) at += S.wsum[i];
      total += S.wsum[i];
    }
    for (uint32_t r0 = 0; r0 < total; r0 += kList) {
      uint32_t p = at;
      for (uint32_t x = word; x; x &= x - 1, ++p)
        if (p - r0 < kList) S.list[p - r0] = (int32_t)((w << 5) + (uint32_t)__ffs((int)x) - 1);
      __syncthreads();
      const uint32_t n = total - r0 < kList ? total - r0 : kList;
      for (uint32_t i0 = 0; i0 < n; i0 += kStepThreads) {
        for (uint32_t i = i0 + tid / kRowLanes; i < n && i < i0 + kStepThreads; i += kStepThreads / kRowLanes) {
          const uint32_t u = (uint32_t)S.list[i], du = j.dist[u];
          const int64_t a0 = j.rp[u], a1 = j.rp[u + 1];
          if (du < theta) relax_row(k, u, du, a0, (int32_t)(a1 - a0));
          else if (row_lane() == 0) leave(k, u, du);
        }
        relax_long(k);
      }
      __syncthreads();
    }
  }
  // Round i reads queue i & 1 and counter i % 3 and fills the other queue and
  // the next counter; the third counter is cleared meanwhile, so the barrier
  // that ends a round's last pass is the only one.
  uint32_t n = 0, q = 0, slot = 0;
  __syncthreads();
  for (uint32_t round = 0;; ++round) {
    n = S.qn[slot] < kQueue ? S.qn[slot] : kQueue;
    if (n == 0 || round >= j.rounds) break;
    k.q = q ^ 1;
    k.qslot = slot == 2 ? 0 : slot + 1;
    if (tid == 0) S.qn[slot == 0 ? 2 : slot - 1] = 0;
    for (uint32_t i0 = 0; i0 < n; i0 += kStepThreads) {
      for (uint32_t i = i0 + tid / kRowLanes; i < n && i < i0 + kStepThreads; i += kStepThreads / kRowLanes) {
        const uint2 x = S.queue[q][i];
        const uint32_t d = j.dist[x.x];
        const int64_t a0 = j.rp[x.x], a1 = j.rp[x.x + 1];
        if (d >= x.y) relax_row(k, x.x, x.y, a0, (int32_t)(a1 - a0));
      }
      relax_long(k);
    }
    q = k.q;
    slot = k.qslot;
  }
  for (uint32_t i = tid; i < n; i += kStepThreads) {
    const uint2 x = S.queue[q][i];
    leave(k, x.x, x.y);
  }
  if (__any(k.fmin != CLD_INF32)) {
    for (int o = 32; o >= 1; o >>= 1) {
      const uint32_t y = __shfl_xor(k.fmin, o);
      k.fmin = y < k.fmin ? y : k.fmin;
    }
    if (lane == 0) atomicMin(&S.fmin, k.fmin);
  }
  __syncthreads();
  if (tid == 0 && S.fmin != CLD_INF32) atomicMin(&j.ctl->slot[t & 3].fmin, S.fmin);
}

__global__ void __launch_bounds__(kT) k_sssp_init(SJob j, int32_t src) {
  const int64_t at = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t v = at; v < j.n; v += stride) j.dist[v] = v == src ? 0u : CLD_INF32;
  for (int64_t w = at; w < j.words; w += stride) {
    j.front[1][w] = w == (src >> 5) ? 1u << (src & 31) : 0u;   // step 1 reads front[1]
    j.front[0][w] = 0;
  }
  if (at == 0) {
    for (int i = 0; i < 4; ++i) j.ctl->slot[i].fmin = i == 0 ? 0u : CLD_INF32;
    j.ctl->maybe = 0;
    j.ctl->overflow = 0;
    j.ctl->mx = 0;
  }
}

__global__ void __launch_bounds__(kT) k_sssp_max(SJob j) {
  unsigned long long m = 0;
  for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < j.n; v += (int64_t)gridDim.x * blockDim.x)
    if (j.dist[v] != CLD_INF32 && j.dist[v] > m) m = j.dist[v];
  for (int o = 32; o >= 1; o >>= 1) {
    unsigned long long x = __shfl_xor(m, o);
    m = x > m ? x : m;
  }
  if ((threadIdx.x & 63) == 0 && m) atomicMax(&j.ctl->mx, m);
}

// Whether some reached node's distance plus its longest arc (the last one of
// its row) does not fit in 32 bits.  Offers made from tentative distances may
// not fit although the final ones do, so this looks at the final ones.
__global__ void __launch_bounds__(kT) k_sssp_overflow(SJob j) {
  for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < j.n; v += (int64_t)gridDim.x * blockDim.x) {
    const uint32_t d = j.dist[v];
    if (d == CLD_INF32 || j.rp[v + 1] == j.rp[v]) continue;
    if ((uint64_t)d + (j.arcs[j.rp[v + 1] - 1] >> 32) >= CLD_INF32) j.ctl->overflow = 1u;
  }
}

// Sum of all arc weights (the high words of the packed arcs), for the default
// bucket width.
__global__ void __launch_bounds__(kT) k_sssp_weight_sum(const uint64_t *arcs, int64_t m, unsigned long long *sum) {
  unsigned long long s = 0;
  for (int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; a < m; a += (int64_t)gridDim.x * blockDim.x)
    s += arcs[a] >> 32;
  for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o);
  if ((threadIdx.x & 63) == 0 && s) atomicAdd(sum, s);
}

// Default bucket width: kDefaultWidth mean arc weights (at least 1, at most
// 2^31); 1 on a graph without arcs.
constexpr uint64_t kDefaultWidth = 16;
constexpr int kLimitSeconds = 60;

uint32_t bitmap_words(int32_t n) { return (uint32_t)(((int64_t)n + 31) >> 5); }

}  // namespace

extern "C" size_t cldiam_sssp_workspace_size(int32_t n, int64_t m) {
  (void)m;
  if (n < 1) return 0;
  cld::Sizer s;
  s.take<SCtl>(1);
  for (int i = 0; i < 2; ++i) s.take<uint32_t>(bitmap_words(n));
  return s.used;
}

extern "C" int cldiam_sssp_delta_stepping(int32_t n, int64_t m, const int64_t *d_row_ptr, const uint64_t *d_arcs,
                                          int32_t source, uint32_t bucket_delta, uint32_t *d_dist,
                                          uint64_t *h_max_dist, void *ws, size_t ws_bytes, void *stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  if (n < 1 || m < 0 || source < 0 || source >= n || !d_row_ptr || (m && !d_arcs) || !d_dist || !h_max_dist) {
    cld::set_error("sssp: invalid arguments");
    return CLDIAM_EINVAL;
  }
  cld::Arena a(ws, ws_bytes);
  SJob j;
  j.ctl = a.take<SCtl>(1);
  j.front[0] = a.take<uint32_t>(bitmap_words(n));
  j.front[1] = a.take<uint32_t>(bitmap_words(n));
  if (!j.front[1]) {
    cld::set_error("sssp: workspace of %zu bytes, %zu needed", ws_bytes, cldiam_sssp_workspace_size(n, m));
    return CLDIAM_ENOMEM;
  }
  if (bucket_delta == 0) {
    // default width from the mean arc weight (ctl->mx serves as the sum's slot)
    uint64_t wsum = 0;
    if (m > 0) {
      CLD_HIP(hipMemsetAsync(&j.ctl->mx, 0, 8, stream));
      k_sssp_weight_sum<<<cld::blocks_for(m, kT, 4096), kT, 0, stream>>>(d_arcs, m, &j.ctl->mx);
      CLD_LAUNCH_CHECK("k_sssp_weight_sum");
      unsigned long long hs = 0;
      CLD_HIP(hipMemcpyAsync(&hs, &j.ctl->mx, 8, hipMemcpyDeviceToHost, stream));
      CLD_HIP(hipStreamSynchronize(stream));
      wsum = hs;
    }
    uint64_t b = m > 0 ? kDefaultWidth * (wsum / (uint64_t)m) : 1;
    if (b < 1) b = 1;
    if (b > CLD_DELTA_MAX) b = CLD_DELTA_MAX;
    bucket_delta = (uint32_t)b;
  }
  int dev = 0, cus = 0;
  CLD_HIP(hipGetDevice(&dev));
  CLD_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  j.rp = d_row_ptr;
  j.arcs = d_arcs;
  j.n = n;
  j.delta = bucket_delta;
  j.dist = d_dist;
  j.words = bitmap_words(n);
  const uint32_t most = (uint32_t)(cus * kBlocksPerCu);
  j.chunk = (j.words + most - 1) / most;
  const int64_t fit = m > 0 ? kMinArcs * n / (32 * m) : kMinWords;
  const uint32_t least = fit < 1 ? 1u : (fit < kMinWords ? (uint32_t)fit : (uint32_t)kMinWords);
  if (j.chunk < least) j.chunk = least;
  const int blocks = (int)(((j.words + j.chunk - 1) / j.chunk + 7) / 8 * 8);   // a multiple of the XCDs
  j.rounds = m > kDenseDegree * n ? 0 : kRounds;
  cld::Pinned<SCtl> pinned;   // readback buffer; its first line mirrors the device's progress during the search
  if (!pinned.p) { cld::set_error("sssp: pinned host buffer allocation failed"); return CLDIAM_EHIP; }
  volatile uint32_t *hm = (volatile uint32_t *)pinned.p;
  cld::Drain drain{stream, true};   // queued steps write the mirror
  hm[0] = 0;
  hm[1] = 0;
  CLD_HIP(hipHostGetDevicePointer((void **)&j.mirror, (void *)pinned.p, 0));
  k_sssp_init<<<cld::blocks_for(n, kT, 8192), kT, 0, stream>>>(j, source);
  CLD_LAUNCH_CHECK("k_sssp_init");
  // The host queues steps at most kLead ahead of the device and stops once a
  // step reports that the step before it left nothing to relax.  The time limit
  // counts from the first step: the stream may have other work before it.
  std::chrono::steady_clock::time_point t0;
  bool begun = false;
  uint32_t queued = 0;
  while (!hm[1]) {
    if (queued < hm[0] + kLead) {
      ++queued;
      k_sssp_step<<<blocks, kStepThreads, 0, stream>>>(j, queued);
      CLD_LAUNCH_CHECK("k_sssp_step");
      continue;
    }
    const auto now = std::chrono::steady_clock::now();
    if (!begun && hm[0]) {
      begun = true;
      t0 = now;
    }
    if (begun && now - t0 > std::chrono::seconds(kLimitSeconds)) {
      cld::set_error("sssp: search exceeded its time limit");
      return CLDIAM_ETIMEOUT;
    }
    std::this_thread::yield();
  }
  k_sssp_max<<<cld::blocks_for(n, kT, 2048), kT, 0, stream>>>(j);
  CLD_LAUNCH_CHECK("k_sssp_max");
  CLD_HIP(hipMemcpyAsync(pinned.p, j.ctl, sizeof(SCtl), hipMemcpyDeviceToHost, stream));
  CLD_HIP(hipStreamSynchronize(stream));
  drain.armed = false;
  if (pinned.p->maybe) {
    k_sssp_overflow<<<cld::blocks_for(n, kT, 4096), kT, 0, stream>>>(j);
    CLD_LAUNCH_CHECK("k_sssp_overflow");
    CLD_HIP(hipMemcpyAsync(pinned.p, j.ctl, sizeof(SCtl), hipMemcpyDeviceToHost, stream));
    CLD_HIP(hipStreamSynchronize(stream));
    if (pinned.p->overflow) { cld::set_error("sssp: a distance does not fit in 32 bits"); return CLDIAM_EOVERFLOW; }
  }
  *h_max_dist = pinned.p->mx;
  return CLDIAM_OK;
}
