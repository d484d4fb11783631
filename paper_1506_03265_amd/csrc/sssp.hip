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
// What bounds it: the number of hops (8,600 on the road-like 4096 x 4096 mesh)
// times the chain of dependent accesses of one (queue, row offsets and
// distance, arcs, far distances: 4.6 us where they miss the L2).  That mesh
// takes 44 ms at the default width, R-MAT scale 20 4 ms; with node lists,
// returning atomics and one hop per launch they took 255 and 237 ms.  Looking
// up an improved node's row together with its distance, which makes the chain
// one access shorter, gained nothing (47 ms: four times the offset loads).
#include <chrono>
#include <thread>

#include "common.h"

namespace {

constexpr int kT = 256;
// Four workgroups per CU, whose chains of accesses interleave: the road-like
// 4096 x 4096 mesh takes 43 ms with 256 threads, 45 with 512, 50 with 1024.
constexpr int kStepThreads = 256;
constexpr int kBlocksPerCu = 1024 / kStepThreads;
constexpr int kList = 8 * kStepThreads;    // nodes of one expansion of a bitmap window
constexpr int kQueue = 4 * kStepThreads;   // improved nodes of one local round
constexpr int kMidRow = 32;       // longer rows are relaxed by one wave ...
constexpr int kBigRow = 4096;     // ... and these by the whole workgroup
constexpr int kMidCap = 2 * kStepThreads;
constexpr int kBigCap = 64;
constexpr int kMinWords = 16;     // fewest bitmap words of a workgroup
// Local rounds: on sparse graphs a round carries the search a hop further for
// a third of a step's cost (road-like 4096 x 4096 mesh: 145 ms without, 45 with
// 16, 44 with 32, 46 with 64).  On graphs of more than kDenseDegree arcs per
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
  uint32_t qn[2];
  uint32_t nmid[2], nbig[2];   // rows set aside by the even and the odd passes (see relax_long)
  uint32_t wsum[kStepThreads / 64];
  uint32_t fmin;
};

__device__ __forceinline__ void leave(const SJob &j, SStep &S, uint32_t *next, uint32_t v, uint32_t d) {
  atomicOr(&next[v >> 5], 1u << (v & 31));
  if (d < S.fmin) atomicMin(&S.fmin, d);
}

// Applies a thread's K offers nd[i] to v[i] that beat the distances read
// (better[i]), and queues them: one reservation per wave.
template <int K>
__device__ __forceinline__ void improve(const SJob &j, SStep &S, uint32_t *next, int q, uint32_t theta,
                                        const bool (&better)[K], const uint32_t (&v)[K], const uint32_t (&nd)[K]) {
  const uint64_t below = (1ull << (threadIdx.x & 63)) - 1ull;
  uint32_t at[K], total = 0;
  bool near[K];
#pragma unroll
  for (int i = 0; i < K; ++i) {
    if (better[i]) atomicMin(&j.dist[v[i]], nd[i]);
    near[i] = better[i] && nd[i] < theta;
    const uint64_t m = __ballot(near[i]);
    at[i] = total + (uint32_t)__popcll(m & below);
    total += (uint32_t)__popcll(m);
  }
  if (total) {
    uint32_t base = 0;
    const int first = __ffsll((long long)__ballot(true)) - 1;
    if ((int)(threadIdx.x & 63) == first) base = atomicAdd(&S.qn[q], total);
    base = __shfl(base, first);
#pragma unroll
    for (int i = 0; i < K; ++i) {
      if (!near[i]) continue;
      if (base + at[i] < kQueue) S.queue[q][base + at[i]] = make_uint2(v[i], nd[i]);
      else leave(j, S, next, v[i], nd[i]);
    }
  }
#pragma unroll
  for (int i = 0; i < K; ++i)
    if (better[i] && !near[i]) leave(j, S, next, v[i], nd[i]);
}

__device__ __forceinline__ void offer(const SJob &j, SStep &S, uint32_t *next, int q, uint32_t theta, uint32_t du,
                                      uint64_t arc) {
  const uint64_t x = (uint64_t)du + (arc >> 32);
  const uint32_t v[1] = {(uint32_t)arc}, nd[1] = {(uint32_t)x};
  if (x >= CLD_INF32) j.ctl->maybe = 1u;
  const bool better[1] = {x < CLD_INF32 && nd[0] < j.dist[v[0]]};
  improve<1>(j, S, next, q, theta, better, v, nd);
}

// Relaxes u's row (degree deg, first arc a0) with distance du; improvements
// go to queue q.  Arcs are taken four at a time so that their loads overlap.
// Long rows are set aside for the relax_long that ends the pass.
__device__ __forceinline__ void relax_row(const SJob &j, SStep &S, uint32_t *next, int q, uint32_t theta,
                                          uint32_t pass, uint32_t u, uint32_t du, int64_t a0, int32_t deg) {
  if (deg > kMidRow) {
    if (deg > kBigRow) {
      const uint32_t slot = atomicAdd(&S.nbig[pass & 1], 1u);
      if (slot < kBigCap) { S.big[slot] = make_uint2(u, du); return; }
    } else {
      const uint32_t slot = atomicAdd(&S.nmid[pass & 1], 1u);
      if (slot < kMidCap) { S.mid[slot] = make_uint2(u, du); return; }
    }
  }
  const uint64_t *row = j.arcs + a0;
  for (int32_t base = 0; base < deg; base += 4) {
    uint64_t arc[4];
    uint32_t v[4], nd[4];
    bool ok[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) arc[i] = base + i < deg ? row[base + i] : ~0ull;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint64_t x = (uint64_t)du + (arc[i] >> 32);
      ok[i] = base + i < deg && x < CLD_INF32;
      if (base + i < deg && !ok[i]) j.ctl->maybe = 1u;
      nd[i] = (uint32_t)x;
      v[i] = (uint32_t)arc[i];
      ok[i] = ok[i] && nd[i] < j.dist[v[i]];
    }
    improve<4>(j, S, next, q, theta, ok, v, nd);
  }
}

// Ends a pass: relaxes the long rows that it set aside.  The counters alternate
// between passes: a wave that is late to read this pass's sees none of the next
// pass's rows, so every wave takes the same branch after the one barrier.
__device__ void relax_long(const SJob &j, SStep &S, uint32_t *next, int q, uint32_t theta, uint32_t &pass) {
  __syncthreads();
  const uint32_t p = pass++ & 1;
  const uint32_t nm = S.nmid[p] < kMidCap ? S.nmid[p] : kMidCap, nb = S.nbig[p] < kBigCap ? S.nbig[p] : kBigCap;
  if (nm == 0 && nb == 0) return;
  for (uint32_t r = threadIdx.x >> 6; r < nm; r += kStepThreads / 64) {
    const uint2 x = S.mid[r];
    const int64_t a0 = j.rp[x.x];
    const int32_t deg = (int32_t)(j.rp[x.x + 1] - a0);
    for (int32_t a = (int32_t)(threadIdx.x & 63); a < deg; a += 64) offer(j, S, next, q, theta, x.y, j.arcs[a0 + a]);
  }
  for (uint32_t r = 0; r < nb; ++r) {
    const uint2 x = S.big[r];
    const int64_t a0 = j.rp[x.x];
    const int32_t deg = (int32_t)(j.rp[x.x + 1] - a0);
    for (int32_t a = (int32_t)threadIdx.x; a < deg; a += kStepThreads) offer(j, S, next, q, theta, x.y, j.arcs[a0 + a]);
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
  if (tid == 0) { S.qn[0] = S.qn[1] = S.nmid[0] = S.nmid[1] = S.nbig[0] = S.nbig[1] = 0; S.fmin = CLD_INF32; }
  // Workgroups go to the XCDs in turn; each XCD takes one eighth of the words,
  // so that neighbouring ranges share an L2 (2 to 6% faster than in turn).
  const uint32_t range = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  const uint32_t lo = range * j.chunk < j.words ? range * j.chunk : j.words;
  const uint32_t hi = lo + j.chunk < j.words ? lo + j.chunk : j.words;
  uint32_t pass = 0;
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
    for (uint32_t k = 0; k < kStepThreads / 64; ++k) {
      if (k < wave) at += S.wsum[k];
      total += S.wsum[k];
    }
    for (uint32_t r0 = 0; r0 < total; r0 += kList) {
      uint32_t p = at;
      for (uint32_t x = word; x; x &= x - 1, ++p)
        if (p - r0 < kList) S.list[p - r0] = (int32_t)((w << 5) + (uint32_t)__ffs((int)x) - 1);
      __syncthreads();
      const uint32_t n = total - r0 < kList ? total - r0 : kList;
      for (uint32_t i0 = 0; i0 < n; i0 += kStepThreads) {
        const uint32_t i = i0 + tid;
        if (i < n) {
          const uint32_t u = (uint32_t)S.list[i], du = j.dist[u];
          const int64_t a0 = j.rp[u], a1 = j.rp[u + 1];
          if (du >= theta) leave(j, S, next, u, du);
          else relax_row(j, S, next, 0, theta, pass, u, du, a0, (int32_t)(a1 - a0));
        }
        relax_long(j, S, next, 0, theta, pass);
      }
      __syncthreads();
    }
  }
  int q = 0;
  uint32_t n = 0;
  for (uint32_t round = 0;; ++round) {
    __syncthreads();
    n = S.qn[q] < kQueue ? S.qn[q] : kQueue;
    if (n == 0 || round >= j.rounds) break;
    if (tid == 0) S.qn[q ^ 1] = 0;
    __syncthreads();
    for (uint32_t i0 = 0; i0 < n; i0 += kStepThreads) {
      const uint32_t i = i0 + tid;
      if (i < n) {
        const uint2 x = S.queue[q][i];
        const uint32_t d = j.dist[x.x];
        const int64_t a0 = j.rp[x.x], a1 = j.rp[x.x + 1];
        if (d >= x.y) relax_row(j, S, next, q ^ 1, theta, pass, x.x, x.y, a0, (int32_t)(a1 - a0));
      }
      relax_long(j, S, next, q ^ 1, theta, pass);
    }
    q ^= 1;
  }
  for (uint32_t i = tid; i < n; i += kStepThreads) {
    const uint2 x = S.queue[q][i];
    leave(j, S, next, x.x, x.y);
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
  if (j.chunk < kMinWords) j.chunk = kMinWords;
  const int blocks = (int)(((j.words + j.chunk - 1) / j.chunk + 7) / 8 * 8);   // a multiple of the XCDs
  j.rounds = m > kDenseDegree * n ? 0 : kRounds;
  cld::Pinned<SCtl> pinned;   // readback buffer; its first line mirrors the device's progress during the search
  if (!pinned.p) { cld::set_error("sssp: pinned host buffer allocation failed"); return CLDIAM_EHIP; }
  volatile uint32_t *hm = (volatile uint32_t *)pinned.p;
  hm[0] = 0;
  hm[1] = 0;
  CLD_HIP(hipHostGetDevicePointer((void **)&j.mirror, (void *)pinned.p, 0));
  k_sssp_init<<<cld::blocks_for(n, kT, 8192), kT, 0, stream>>>(j, source);
  CLD_LAUNCH_CHECK("k_sssp_init");
  // The host queues steps at most kLead ahead of the device and stops once a
  // step reports that the step before it left nothing to relax.
  const auto t0 = std::chrono::steady_clock::now();
  uint32_t queued = 0;
  while (!hm[1]) {
    if (queued < hm[0] + kLead) {
      ++queued;
      k_sssp_step<<<blocks, kStepThreads, 0, stream>>>(j, queued);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) {
        (void)hipStreamSynchronize(stream);   // queued steps still write the mirror
        return cld::hip_fail(e, "k_sssp_step");
      }
      continue;
    }
    if (std::chrono::steady_clock::now() - t0 > std::chrono::seconds(kLimitSeconds)) {
      CLD_HIP(hipStreamSynchronize(stream));
      cld::set_error("sssp: search exceeded its time limit");
      return CLDIAM_ETIMEOUT;
    }
    std::this_thread::yield();
  }
  k_sssp_max<<<cld::blocks_for(n, kT, 2048), kT, 0, stream>>>(j);
  CLD_LAUNCH_CHECK("k_sssp_max");
  CLD_HIP(hipMemcpyAsync(pinned.p, j.ctl, sizeof(SCtl), hipMemcpyDeviceToHost, stream));
  CLD_HIP(hipStreamSynchronize(stream));
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
