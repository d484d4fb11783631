// Weighted quotient graph G_C (Section 4 of arXiv:1506.03265).
//
// Clusters are numbered densely by ascending center id (ranks in a bitmap of
// the centers).  Every edge {u, v} of G whose endpoints lie in different
// clusters a < b gives the pair key a << kb | b (kb = bits of k-1) and the
// value w(u,v) + D_u + D_v.  Pairs are folded to their minimum in an LDS table
// of each workgroup and then in one table in global memory.  When that table
// holds them all (up to kTableMost pairs, a clustering of thousands of
// clusters), one kernel ranks the keys of both directions and writes the CSR.
// Pairs that find the table full go to a list instead; then the list and the
// table's pairs are radix sorted, the first element of each run marks a
// quotient arc and an atomic minimum over the run keeps the lightest.
#include <vector>

#include "common.h"

namespace cld {
size_t scan_ws_bytes(int64_t n);
size_t radix_ws_bytes(int64_t n);
int scan_exclusive_u32(const uint32_t *in, uint32_t *out, int64_t n, uint32_t *d_total, void *ws, size_t ws_bytes,
                       hipStream_t stream);
int radix_sort_u64(uint64_t *keys, uint64_t *vals, int64_t n, int begin_bit, int end_bit, uint64_t *ktmp,
                   uint64_t *vtmp, bool *in_tmp, void *ws, size_t ws_bytes, hipStream_t stream);
}  // namespace cld

namespace {

constexpr int kT = 256;

struct QCtl {
  unsigned long long pairs;   // directed pairs on the list
  uint32_t k;
  uint32_t uniq;    // pairs in the table (each stands for both directions); later: quotient arcs
  uint32_t bad;     // some label is out of range or not a center
  uint32_t chunk;   // chunks of rows taken beyond each workgroup's first
};

// ------------------------------------------------------------ numbering --

constexpr int kNumThreads = 1024;
constexpr int kNumWaves = kNumThreads / 64;
constexpr int kNumBlocks = 4096;    // wanted workgroups at most; a wave takes 4 to 64 bitmap words
constexpr int kPackBlocks = 512;

// Bitmap of the centers and ranks in it: words[w] holds nodes 64 w .. 64 w + 63,
// before[w] counts the centers of the workgroup's earlier words, total[] those
// of each workgroup.
struct Ranks {
  uint64_t *words;
  uint32_t *before;
  uint32_t *total;
  uint32_t per;      // words per workgroup
  uint32_t blocks;
};

// Center bits; a label that is out of range or names a node that is not its
// own center is reported (the caller then gets CLDIAM_EINVAL, no kernel
// indexes with it).
__global__ void __launch_bounds__(kNumThreads) k_centers(const int32_t *cluster, int32_t n, Ranks r, QCtl *ctl) {
  __shared__ uint32_t wsum[kNumWaves];
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t nwords = (uint32_t)(((int64_t)n + 63) >> 6), wpw = r.per / kNumWaves;
  const uint32_t w0 = blockIdx.x * r.per + wave * wpw;
  uint64_t mine = 0;   // lane l keeps word w0 + l
  bool bad = false;
  for (uint32_t j = 0; j < wpw; j += 4) {
    int32_t c[4];
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) {
      const int64_t v = ((int64_t)(w0 + j + i) << 6) + lane;
      c[i] = v < n ? cluster[v] : -1;
    }
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) {
      const int64_t v = ((int64_t)(w0 + j + i) << 6) + lane;
      const bool center = v < n && c[i] == (int32_t)v;
      if (v < n && !center) {
        if ((uint32_t)c[i] >= (uint32_t)n) bad = true;
        else if (cluster[c[i]] != c[i]) bad = true;
      }
      const uint64_t x = __ballot(center);
      if (lane == j + i) mine = x;
    }
  }
  if (bad) ctl->bad = 1u;
  const uint32_t count = (uint32_t)__popcll(mine), incl = cld_wave_scan_u32(count);
  if (lane == 63) wsum[wave] = incl;
  __syncthreads();
  uint32_t at = incl - count, all = 0;
  for (uint32_t i = 0; i < (uint32_t)kNumWaves; ++i) {
    if (i < wave) at += wsum[i];
    all += wsum[i];
  }
  if (lane < wpw && w0 + lane < nwords) {
    r.words[w0 + lane] = mine;
    r.before[w0 + lane] = at;
  }
  if (threadIdx.x == 0) r.total[blockIdx.x] = all;
}

__device__ __forceinline__ int bits_for_dev(uint32_t x) {  // bits needed for values 0..x, at least 1
  return x ? 32 - __clz(x) : 1;
}

// Dense cluster index of every node, 16 bits each while they suffice (an arc's
// far end then costs a 2-byte gather), and the list of centers.
__global__ void __launch_bounds__(kNumThreads) k_number(const int32_t *cluster, int32_t n, Ranks r, QCtl *ctl,
                                                        void *cid, int32_t *qcenter) {
  extern __shared__ uint32_t base[];   // centers before each workgroup of k_centers
  __shared__ uint32_t wsum[kNumWaves];
  if (ctl->bad) return;
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t each = (r.blocks + kNumThreads - 1) / kNumThreads;
  uint32_t sum = 0;
  for (uint32_t i = 0; i < each; ++i)
    if (tid * each + i < r.blocks) sum += r.total[tid * each + i];
  const uint32_t incl = cld_wave_scan_u32(sum);
  if (lane == 63) wsum[wave] = incl;
  __syncthreads();
  uint32_t at = incl - sum, k = 0;
  for (uint32_t i = 0; i < (uint32_t)kNumWaves; ++i) {
    if (i < wave) at += wsum[i];
    k += wsum[i];
  }
  for (uint32_t i = 0; i < each; ++i)
    if (tid * each + i < r.blocks) {
      base[tid * each + i] = at;
      at += r.total[tid * each + i];
    }
  __syncthreads();
  if (blockIdx.x == 0 && tid == 0) ctl->k = k;
  const bool narrow = k <= 65536;
  for (int64_t v = (int64_t)blockIdx.x * kNumThreads + tid; v < n; v += (int64_t)gridDim.x * kNumThreads) {
    const uint32_t c = (uint32_t)cluster[v], w = c >> 6;
    const uint32_t id = base[w / r.per] + r.before[w] + (uint32_t)__popcll(r.words[w] & ((1ull << (c & 63)) - 1ull));
    if (narrow) ((uint16_t *)cid)[v] = (uint16_t)id;
    else ((uint32_t *)cid)[v] = id;
    if (c == (uint32_t)v) qcenter[id] = (int32_t)v;
  }
}

// ------------------------------------------------------------- emission --

// The table of all pairs in global memory.
constexpr uint32_t kTableSlots = 32768;
constexpr uint32_t kTableMost = 8192;   // pairs the table is meant for (a few more may slip in)
constexpr int kTableProbes = 32;

struct Table {
  unsigned long long *key, *val;
  uint32_t *slot;              // slots in the order they were taken
  uint64_t *keys, *vals;       // the list: directed pairs
  QCtl *ctl;
  int kb;
};

__global__ void __launch_bounds__(kT) k_clear(Table t) {
  const uint32_t at = blockIdx.x * blockDim.x + threadIdx.x;
  for (uint32_t i = at; i < kTableSlots; i += gridDim.x * blockDim.x) {
    t.key[i] = ~0ull;
    t.val[i] = ~0ull;
  }
  if (at == 0) *t.ctl = QCtl{};
}

__device__ __forceinline__ uint64_t reversed(uint64_t key, int kb) {
  return (key & ((1ull << kb) - 1ull)) << kb | key >> kb;
}

// Room for `each` entries of every active lane of a wave, one addition in all:
// the first entry of this lane's.  Out of line: inlined wherever a pair is
// emitted it cost the arc pass 4% (R-MAT scale 20, 2 clusters: 2.16, now 2.06 ms).
template <class T>
__device__ __attribute__((noinline)) T reserve(T *counter, uint32_t each) {
  const uint64_t m = __ballot(true);
  const int lane = (int)(threadIdx.x & 63), first = __ffsll((long long)m) - 1;
  T base = 0;
  if (lane == first) base = atomicAdd(counter, (T)(each * (uint32_t)__popcll(m)));
  return __shfl(base, first) + (T)(each * (uint32_t)__popcll(m & ((1ull << lane) - 1ull)));
}

// Lowers key's value in the table; a new key's slot is noted in claims[] (up to
// claim_cap, counted in *claimed) for one reservation later, or at once.  False:
// the table has no room for the key.  *full: the table takes no new keys.
__device__ __forceinline__ bool put_pair(const Table &t, uint32_t *full, uint64_t key, uint64_t val, int32_t *claims,
                                         uint32_t claim_cap, uint32_t *claimed) {
  uint32_t h = (uint32_t)((key * 0xD6E8FEB86659FD93ull) >> 44) & (kTableSlots - 1);
  for (int p = 0; p < kTableProbes; ++p) {
    unsigned long long at = __hip_atomic_load(&t.key[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (at == ~0ull) {
      if (*full) return false;
      at = atomicCAS(&t.key[h], ~0ull, (unsigned long long)key);
      if (at == ~0ull) {
        const uint32_t i = claim_cap ? atomicAdd(claimed, 1u) : 0u;
        if (i < claim_cap) {
          claims[i] = (int32_t)h;
        } else {
          const uint32_t c = reserve(&t.ctl->uniq, 1u);
          t.slot[c] = h;
          if (c >= kTableMost) *full = 1;
        }
        at = key;
      }
    }
    if (at == key) {
      if (val < __hip_atomic_load(&t.val[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMin(&t.val[h], (unsigned long long)val);
      return true;
    }
    h = (h + 1) & (kTableSlots - 1);
  }
  *full = 1;
  return false;
}

// Both directions of a pair at `at` on the list.
__device__ __forceinline__ void list_pair(const Table &t, uint64_t at, uint64_t key, uint64_t val) {
  t.keys[at] = key;
  t.vals[at] = val;
  t.keys[at + 1] = reversed(key, t.kb);
  t.vals[at + 1] = val;
}

// The rows are cut into up to kEmitChunks chunks, the first of each workgroup
// fixed, the others for whichever is free (hubs make them unequal); rows of up to
// kEmitThreadDeg arcs are walked by one thread, longer rows are deferred to LDS
// and walked by one wave (64 lanes) or, above kEmitBlockDeg, by the whole
// workgroup.  Every pair first goes into an LDS hash table of the workgroup
// that keeps the minimum per key, and from there, whenever it is half full
// after a round and at the end, to the table of all pairs.  A pair that finds
// no slot after a few probes goes straight there.
//
// Bound by the gathers of the arcs' far ends (260 million on R-MAT scale 24).
// So a far end's 2-byte cluster index is read first; most arcs end there: both
// ends in one cluster, or the arc's weight plus the near end's D already no
// better than the pair's value in the LDS table (R-MAT's few large clusters:
// 61% of the arcs join two, and their values fall early), and D is read for
// the rest only.  R-MAT scale 24: 3.55 ms (6.65 with an 8-byte word of index and
// D gathered for every arc, both directions folded apart), scale 18: 0.11
// (0.24), the road-like 4096 x 4096 mesh: 0.30 (0.32).
constexpr int kEmitThreads = 1024;
constexpr int kEmitThreadDeg = 16;
constexpr int kEmitBlockDeg = 4096;
constexpr int kEmitDefer = 512;     // deferred rows per round
constexpr int kHashCap = 4096;      // LDS hash slots (power of two)
constexpr int kHashProbes = 16;
constexpr int kEmitBatch = 4;       // arcs of a row in flight per thread

struct EmitState {
  unsigned long long hkey[kHashCap];
  unsigned long long hval[kHashCap];
  int32_t mid[kEmitDefer];
  int32_t big[kEmitDefer];
  uint32_t nmid, nbig, used;
  uint32_t chunk, base;
  uint32_t listed;            // of a flush: pairs for the list ...
  unsigned long long list;    // ... and their place
  uint32_t full;   // the table of all pairs takes no new keys (from the last flush on, or met since)
  uint32_t blind;  // ... and holds so few of this workgroup's that they go to the list unseen
  Table table;
};

__device__ __forceinline__ uint32_t hash_slot(uint64_t key) {
  uint64_t x = key * 0x9E3779B97F4A7C15ull;
  return (uint32_t)(x >> 40) & (kHashCap - 1);
}

// Whether the LDS table holds a value for key that is no larger than x.
__device__ __forceinline__ bool no_better(const EmitState &E, uint64_t key, uint64_t x) {
  uint32_t h = hash_slot(key);
  for (int p = 0; p < kHashProbes; ++p) {
    const unsigned long long at = E.hkey[h];
    if (at == key) return E.hval[h] <= x;
    if (at == ~0ull) return false;
    h = (h + 1) & (kHashCap - 1);
  }
  return false;
}

__device__ __forceinline__ void emit_pair(EmitState &E, uint64_t key, uint64_t val) {
  uint32_t h = hash_slot(key);
  for (int p = 0; p < kHashProbes; ++p) {
    unsigned long long at = E.hkey[h];
    if (at == ~0ull) {
      at = atomicCAS(&E.hkey[h], ~0ull, (unsigned long long)key);
      if (at == ~0ull) {
        atomicAdd(&E.used, 1u);
        at = key;
      }
    }
    if (at == key) {
      atomicMin(&E.hval[h], (unsigned long long)val);
      return;
    }
    h = (h + 1) & (kHashCap - 1);
  }
  if (E.blind || !put_pair(E.table, &E.full, key, val, nullptr, 0, nullptr))
    list_pair(E.table, reserve(&E.table.ctl->pairs, 2u), key, val);
}

__device__ void hash_flush(EmitState &E) {
  // One look at the count and one reservation per flush, of new keys as of pairs
  // for the list: with one of each per new key, the count's line took 200 of the
  // arc pass's 300 us on a road-like 2048 x 2048 mesh of 2228 clusters, and with
  // one per listed pair a 2048 x 2048 mesh of 5000 scattered clusters, 4 million
  // such pairs, took 104 ms (4.3 now).  A workgroup whose pairs are hardly ever in
  // the full table stops looking there (blind).
  if (threadIdx.x == 0) {
    E.nmid = 0;   // E.mid holds the slots of new keys meanwhile: their count is reserved once
    E.listed = 0;
    E.full = __hip_atomic_load(&E.table.ctl->uniq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= kTableMost;
  }
  __syncthreads();
  uint32_t mine = 0;
  for (uint32_t i = threadIdx.x; i < kHashCap; i += kEmitThreads) {
    const uint64_t key = E.hkey[i];
    if (key == ~0ull) continue;
    if (!E.blind && put_pair(E.table, &E.full, key, E.hval[i], E.mid, kEmitDefer, &E.nmid)) {
      E.hkey[i] = ~0ull;
      E.hval[i] = ~0ull;
    } else {
      ++mine;
    }
  }
  const uint32_t incl = cld_wave_scan_u32(mine), all = cld_last_lane(incl);
  uint32_t at = 0;
  if (all) {
    if ((threadIdx.x & 63) == 0) at = atomicAdd(&E.listed, all);
    at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + incl - mine;
  }
  __syncthreads();
  const uint32_t n = E.nmid < kEmitDefer ? E.nmid : kEmitDefer;
  if (threadIdx.x == 0) {
    E.blind = E.listed > E.used / 8 * 7;
    E.used = 0;
    E.base = n ? atomicAdd(&E.table.ctl->uniq, n) : 0u;
    E.list = E.listed ? atomicAdd(&E.table.ctl->pairs, 2ull * E.listed) : 0ull;
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < n; i += kEmitThreads) E.table.slot[E.base + i] = (uint32_t)E.mid[i];
  if (mine) {
    for (uint32_t i = threadIdx.x; i < kHashCap; i += kEmitThreads) {
      const uint64_t key = E.hkey[i];
      if (key == ~0ull) continue;
      list_pair(E.table, E.list + 2ull * at++, key, E.hval[i]);
      E.hkey[i] = ~0ull;
      E.hval[i] = ~0ull;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) E.nmid = 0;
  __syncthreads();
}

// One pending pair per thread, in registers.  A stage has few clusters, so
// consecutive arcs of a row mostly lead to the same cluster: their pairs fold
// here and only a change of key touches the LDS table (whose random slots
// cost bank conflicts).  Flushed at the end of each row part.
struct PairCache {
  uint64_t key = ~0ull, val = ~0ull;
};

__device__ __forceinline__ void cache_flush(PairCache &pc, EmitState &E) {
  if (pc.key != ~0ull) emit_pair(E, pc.key, pc.val);
  pc.key = ~0ull;
}

// Arcs first, first + stride, ... of u's row.  The graph is symmetric with
// equal weights both ways and w + D_u + D_v is symmetric, so each edge is taken
// once, from its smaller end (u < v).
template <class Id>
__device__ __forceinline__ void emit_row(int32_t u, const uint64_t *row, int32_t deg, int32_t first, int32_t stride,
                                         const Id *cid, const uint64_t *D, EmitState &E, int kb) {
  const uint32_t cu = cid[u];
  const uint64_t du = D[u];
  PairCache pc;
  for (int32_t a = first; a < deg; a += stride * kEmitBatch) {
    uint64_t arc[kEmitBatch];
    uint32_t cv[kEmitBatch];
#pragma unroll
    for (int i = 0; i < kEmitBatch; ++i) arc[i] = a + i * stride < deg ? row[a + i * stride] : 0ull;
#pragma unroll
    for (int i = 0; i < kEmitBatch; ++i) cv[i] = (int32_t)(uint32_t)arc[i] > u ? cid[(uint32_t)arc[i]] : cu;
#pragma unroll
    for (int i = 0; i < kEmitBatch; ++i) {
      if (cv[i] == cu) continue;
      const uint64_t key = cu < cv[i] ? (uint64_t)cu << kb | cv[i] : (uint64_t)cv[i] << kb | cu;
      const uint64_t least = (arc[i] >> 32) + du;
      if (key == pc.key) {
        if (least >= pc.val) continue;
      } else if (no_better(E, key, least)) {
        continue;
      }
      const uint64_t val = least + D[(uint32_t)arc[i]];
      if (key != pc.key) {
        cache_flush(pc, E);
        pc.key = key;
        pc.val = val;
      } else if (val < pc.val) {
        pc.val = val;
      }
    }
  }
  cache_flush(pc, E);
}

template <class Id>
__device__ __forceinline__ void emit_rows(const int64_t *rp, const uint64_t *arcs, int32_t n, const Id *cid,
                                          const uint64_t *D, EmitState &E, int kb, uint32_t chunk, int64_t per) {
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6;
  const int64_t lo = (int64_t)chunk * per;
  const int64_t hi = lo + per < n ? lo + per : n;
  for (int64_t r = lo; r < hi; r += blockDim.x) {
    const int64_t u = r + threadIdx.x;
    if (u < hi) {
      const int64_t a0 = rp[u];
      const int32_t deg = (int32_t)(rp[u + 1] - a0);
      bool done = false;
      if (deg > kEmitThreadDeg) {
        uint32_t *cnt = deg > kEmitBlockDeg ? &E.nbig : &E.nmid;
        int32_t *lst = deg > kEmitBlockDeg ? E.big : E.mid;
        const uint32_t slot = atomicAdd(cnt, 1u);
        if (slot < kEmitDefer) { lst[slot] = (int32_t)u; done = true; }
      }
      if (!done) emit_row((int32_t)u, arcs + a0, deg, 0, 1, cid, D, E, kb);
    }
    __syncthreads();
    const uint32_t nm = E.nmid < kEmitDefer ? E.nmid : kEmitDefer;
    for (uint32_t i = wave; i < nm; i += nwaves) {
      const int32_t x = E.mid[i];
      const int64_t a0 = rp[x];
      emit_row(x, arcs + a0, (int32_t)(rp[x + 1] - a0), (int32_t)lane, 64, cid, D, E, kb);
    }
    const uint32_t nbg = E.nbig < kEmitDefer ? E.nbig : kEmitDefer;
    for (uint32_t i = 0; i < nbg; ++i) {
      const int32_t x = E.big[i];
      const int64_t a0 = rp[x];
      emit_row(x, arcs + a0, (int32_t)(rp[x + 1] - a0), (int32_t)threadIdx.x, kEmitThreads, cid, D, E, kb);
      __syncthreads();
      const bool full = E.used > kHashCap / 2;
      __syncthreads();
      if (full) hash_flush(E);
    }
    __syncthreads();
    const bool full = E.used > kHashCap / 2;
    if (threadIdx.x == 0) { E.nmid = 0; E.nbig = 0; }
    __syncthreads();
    if (full) hash_flush(E);
  }
}

__global__ void __launch_bounds__(kEmitThreads, 8) k_emit(const int64_t *rp, const uint64_t *arcs, int32_t n,
                                                       const void *cid, const uint64_t *D, int64_t per, Table t) {
  __shared__ EmitState E;
  if (t.ctl->bad) return;
  const uint32_t k = t.ctl->k;
  const int kb = bits_for_dev(k > 0 ? k - 1 : 0u);
  for (uint32_t i = threadIdx.x; i < kHashCap; i += blockDim.x) { E.hkey[i] = ~0ull; E.hval[i] = ~0ull; }
  if (threadIdx.x == 0) {
    E.nmid = 0; E.nbig = 0; E.used = 0; E.full = 0; E.blind = 0;
    E.table = t;
    E.table.kb = kb;
  }
  __syncthreads();
  const uint32_t chunks = (uint32_t)(((int64_t)n + per - 1) / per);
  for (uint32_t chunk = blockIdx.x; chunk < chunks;) {
    if (k <= 65536) emit_rows(rp, arcs, n, (const uint16_t *)cid, D, E, kb, chunk, per);
    else emit_rows(rp, arcs, n, (const uint32_t *)cid, D, E, kb, chunk, per);
    if (threadIdx.x == 0) E.chunk = gridDim.x + atomicAdd(&t.ctl->chunk, 1u);
    __syncthreads();
    chunk = E.chunk;
    __syncthreads();
  }
  hash_flush(E);
}

// -------------------------------------------------------------- ranking --

// With all pairs in the table: every workgroup holds the keys of both
// directions in LDS, and each wave counts, for its keys and row starts, the
// keys below: a key's rank is its place in the CSR, a row's its offset.
// 8 to 35 us for 300 to 12,000 arcs, where sorting, marking and reducing runs of
// the unfolded pairs took 15 launches, two host synchronisations and 150 to 250.
constexpr int kRankThreads = 1024;
constexpr int kRankBlocks = 256;
constexpr int kRankBatch = 8;             // keys ranked by a wave in one walk
constexpr uint32_t kRankMostK = 16384;    // 14-bit indices: keys of 28 bits

__device__ __host__ inline bool table_holds_all(const QCtl &c) {
  return !c.bad && c.pairs == 0 && c.uniq <= kTableMost && c.k <= kRankMostK;
}

__global__ void __launch_bounds__(kRankThreads) k_rank(Table t, int32_t *qcol, uint64_t *qw, int64_t *qrp) {
  extern __shared__ uint4 keys4[];   // both directions' keys, filled up with ~0 to whole steps of a wave
  uint32_t *keys = (uint32_t *)keys4;
  const QCtl c = *t.ctl;
  if (!table_holds_all(c)) return;
  const int kb = bits_for_dev(c.k > 0 ? c.k - 1 : 0u);
  const uint32_t lane = threadIdx.x & 63, n = 2 * c.uniq, steps = (n + 255) / 256, all = n + c.k + 1;
  for (uint32_t i = threadIdx.x; i < 128 * steps; i += kRankThreads) {
    const uint64_t key = i < c.uniq ? t.key[t.slot[i]] : 0ull;
    keys[2 * i] = i < c.uniq ? (uint32_t)key : ~0u;
    keys[2 * i + 1] = i < c.uniq ? (uint32_t)reversed(key, kb) : ~0u;
  }
  __syncthreads();
  const uint32_t wave = blockIdx.x * (kRankThreads / 64) + (threadIdx.x >> 6);
  const uint32_t waves = gridDim.x * (kRankThreads / 64);
  for (uint32_t e0 = wave * kRankBatch; e0 < all; e0 += waves * kRankBatch) {
    uint32_t x[kRankBatch], below[kRankBatch] = {};
#pragma unroll
    for (int j = 0; j < kRankBatch; ++j) x[j] = e0 + j < n ? keys[e0 + j] : (e0 + j - n) << kb;
    for (uint32_t i = 0; i < steps; ++i) {
      const uint4 y = keys4[i * 64 + lane];
#pragma unroll
      for (int j = 0; j < kRankBatch; ++j)
        below[j] += (uint32_t)(y.x < x[j]) + (uint32_t)(y.y < x[j]) + (uint32_t)(y.z < x[j]) + (uint32_t)(y.w < x[j]);
    }
#pragma unroll
    for (int j = 0; j < kRankBatch; ++j) {
      const uint32_t rank = cld_last_lane(cld_wave_scan_u32(below[j])), e = e0 + j;
      if (lane != 0 || e >= all) continue;
      if (e < n) {
        qcol[rank] = (int32_t)(x[j] & ((1u << kb) - 1u));
        qw[rank] = t.val[t.slot[e >> 1]];
      } else {
        qrp[e - n] = rank;
      }
    }
  }
}

// The table's pairs join the list.
__global__ void __launch_bounds__(kT) k_table_to_list(Table t, uint32_t uniq, uint64_t pairs) {
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < uniq; i += gridDim.x * blockDim.x) {
    const uint64_t key = t.key[t.slot[i]], val = t.val[t.slot[i]];
    t.keys[pairs + 2 * i] = key;
    t.vals[pairs + 2 * i] = val;
    t.keys[pairs + 2 * i + 1] = reversed(key, t.kb);
    t.vals[pairs + 2 * i + 1] = val;
  }
}

__global__ void k_heads(const uint64_t *keys, int64_t P, uint32_t *head) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < P; i += (int64_t)gridDim.x * blockDim.x)
    head[i] = (i == 0 || keys[i] != keys[i - 1]) ? 1u : 0u;
}

__global__ void k_fill_inf(uint64_t *x, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    x[i] = CLD_INF64;
}

// Run minimum into the unique slot, one chunk of kRunChunk consecutive
// elements per thread: one atomic per (run, chunk) piece.  Heads also write the
// column and fill the row offsets of every row in (previous row, this row].
constexpr int kRunChunk = 64;

__global__ void k_reduce_runs(const uint64_t *keys, const uint64_t *vals, int64_t P, const uint32_t *head,
                              const uint32_t *idx, int kb, int32_t *qcol, uint64_t *qw, int64_t *qrp) {
  const uint64_t bmask = (kb >= 64) ? ~0ull : ((1ull << kb) - 1ull);
  const int64_t chunks = (P + kRunChunk - 1) / kRunChunk;
  for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < chunks; c += (int64_t)gridDim.x * blockDim.x) {
    const int64_t b = c * kRunChunk, e = b + kRunChunk < P ? b + kRunChunk : P;
    uint32_t slot = idx[b] + head[b] - 1;
    uint64_t best = vals[b];
    for (int64_t i = b; i < e; ++i) {
      if (head[i]) {
        if (i > b) atomicMin((unsigned long long *)&qw[slot], (unsigned long long)best);
        slot = idx[i];
        best = vals[i];
        qcol[slot] = (int32_t)(keys[i] & bmask);
        const int64_t row = (int64_t)(keys[i] >> kb);
        const int64_t prev = (i == 0) ? -1 : (int64_t)(keys[i - 1] >> kb);
        for (int64_t r = prev + 1; r <= row; ++r) qrp[r] = slot;
      } else if (vals[i] < best) {
        best = vals[i];
      }
    }
    atomicMin((unsigned long long *)&qw[slot], (unsigned long long)best);
  }
}

__global__ void k_tail_rows(const uint64_t *keys, int64_t P, int kb, int32_t k, uint32_t uniq, int64_t *qrp) {
  const int64_t last = P > 0 ? (int64_t)(keys[P - 1] >> kb) : -1;
  for (int64_t r = last + 1 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r <= k;
       r += (int64_t)gridDim.x * blockDim.x)
    qrp[r] = uniq;
}

int bits_for(uint32_t x) {  // bits needed for values 0..x
  int b = 1;
  while (b < 32 && (x >> b) != 0) ++b;
  return b;
}

// Two workgroups per CU, each with one table to fold its chunks in (2048
// workgroups of one chunk brought several times the pairs to the table of all
// pairs: 198 instead of 162 us on a road-like 2048 x 2048 mesh of 2228 clusters).
constexpr int kEmitBlocks = 512;
constexpr int kEmitChunks = 2048;

struct Buffers {
  Ranks ranks;
  Table table;
  void *cid;
  uint64_t *ktmp, *vtmp;
  uint32_t *head, *idx;
  bool fits;
};

// Words per workgroup of k_centers: 4 to 64 per wave.
uint32_t words_per_block(int32_t n) {
  const int64_t words = ((int64_t)n + 63) >> 6;
  int64_t wpw = (words + (int64_t)kNumBlocks * kNumWaves - 1) / ((int64_t)kNumBlocks * kNumWaves);
  wpw = wpw < 4 ? 4 : (wpw > 64 ? 64 : (wpw + 3) / 4 * 4);
  return (uint32_t)(wpw * kNumWaves);
}

template <class A>
Buffers carve(A &a, int32_t n, int64_t m) {
  Buffers b{};
  const size_t words = ((size_t)n + 63) / 64;
  b.ranks.per = words_per_block(n);
  b.ranks.blocks = (uint32_t)((words + b.ranks.per - 1) / b.ranks.per);
  b.table.ctl = a.template take<QCtl>(1);
  b.ranks.words = a.template take<uint64_t>(words);
  b.ranks.before = a.template take<uint32_t>(words);
  b.ranks.total = a.template take<uint32_t>(b.ranks.blocks);
  b.cid = a.template take<uint32_t>((size_t)n);
  b.table.key = a.template take<unsigned long long>(kTableSlots);
  b.table.val = a.template take<unsigned long long>(kTableSlots);
  b.table.slot = a.template take<uint32_t>(kTableSlots);
  b.table.keys = a.template take<uint64_t>((size_t)m + 1);
  b.table.vals = a.template take<uint64_t>((size_t)m + 1);
  b.ktmp = a.template take<uint64_t>((size_t)m + 1);
  b.vtmp = a.template take<uint64_t>((size_t)m + 1);
  b.head = a.template take<uint32_t>((size_t)m + 1);
  b.idx = a.template take<uint32_t>((size_t)m + 1);
  b.fits = b.idx != nullptr;
  return b;
}

struct SizeA {
  cld::Sizer s;
  template <class T>
  T *take(size_t n) { s.take<T>(n); return nullptr; }
};

}  // namespace

extern "C" size_t cldiam_quotient_workspace_size(int32_t n, int64_t m) {
  if (n < 1 || m < 0) return 0;
  SizeA s;
  carve(s, n, m);
  size_t extra = cld::radix_ws_bytes(m + 1);
  size_t sc = cld::scan_ws_bytes(m + 1);
  return s.s.used + (extra > sc ? extra : sc);
}

extern "C" int cldiam_build_quotient(int32_t n, int64_t m, const int64_t *d_row_ptr, const uint64_t *d_arcs,
                                     const int32_t *d_cluster, const uint64_t *d_D, int32_t *d_qcenter,
                                     int64_t *d_qrow_ptr, int32_t *d_qcol, uint64_t *d_qw, int32_t *h_k,
                                     int64_t *h_qm, void *ws, size_t ws_bytes, void *stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  if (n < 1 || m < 0 || m >= ((int64_t)1 << 40) || !d_row_ptr || (m && !d_arcs) || !d_cluster || !d_D ||
      !d_qcenter || !d_qrow_ptr || !h_k || !h_qm) {
    cld::set_error("build_quotient: invalid arguments");
    return CLDIAM_EINVAL;
  }
  cld::Arena a(ws, ws_bytes);
  Buffers b = carve(a, n, m);
  if (!b.fits || a.used > ws_bytes) {
    cld::set_error("build_quotient: workspace of %zu bytes, %zu needed", ws_bytes, cldiam_quotient_workspace_size(n, m));
    return CLDIAM_ENOMEM;
  }
  void *rest = a.base + a.used;
  const size_t rest_bytes = a.cap - a.used;
  QCtl *ctl = b.table.ctl;
  k_clear<<<32, kT, 0, stream>>>(b.table);
  CLD_LAUNCH_CHECK("k_clear");
  k_centers<<<b.ranks.blocks, kNumThreads, 0, stream>>>(d_cluster, n, b.ranks, ctl);
  CLD_LAUNCH_CHECK("k_centers");
  k_number<<<cld::blocks_for(n, kNumThreads, kPackBlocks), kNumThreads, (size_t)b.ranks.blocks * 4, stream>>>(
      d_cluster, n, b.ranks, ctl, b.cid, d_qcenter);
  CLD_LAUNCH_CHECK("k_number");
  if (m > 0) {
    const int64_t chunks = n < kEmitChunks * 64 ? ((int64_t)n + 63) / 64 : kEmitChunks, per = (n + chunks - 1) / chunks;
    k_emit<<<(unsigned)(chunks < kEmitBlocks ? chunks : kEmitBlocks), kEmitThreads, 0, stream>>>(
        d_row_ptr, d_arcs, n, b.cid, d_D, per, b.table);
    CLD_LAUNCH_CHECK("k_emit");
  }
  k_rank<<<kRankBlocks, kRankThreads, (size_t)2 * kTableMost * 4, stream>>>(b.table, d_qcol, d_qw, d_qrow_ptr);
  CLD_LAUNCH_CHECK("k_rank");
  cld::Pinned<QCtl> pinned;
  if (!pinned.p) { cld::set_error("build_quotient: pinned host buffer allocation failed"); return CLDIAM_EHIP; }
  CLD_HIP(hipMemcpyAsync(pinned.p, ctl, sizeof(QCtl), hipMemcpyDeviceToHost, stream));
  CLD_HIP(hipStreamSynchronize(stream));
  const QCtl h = *pinned.p;
  if (h.bad) {
    cld::set_error("build_quotient: a cluster label is out of range or not a center (cluster[c] != c)");
    return CLDIAM_EINVAL;
  }
  const int32_t k = (int32_t)h.k;
  if (table_holds_all(h)) {
    *h_k = k;
    *h_qm = 2 * (int64_t)h.uniq;
    return CLDIAM_OK;
  }
  const int kb = bits_for(k > 0 ? (uint32_t)(k - 1) : 0u);
  b.table.kb = kb;
  if (h.uniq) {
    k_table_to_list<<<cld::blocks_for(h.uniq, kT, 256), kT, 0, stream>>>(b.table, h.uniq, h.pairs);
    CLD_LAUNCH_CHECK("k_table_to_list");
  }
  const int64_t P = (int64_t)h.pairs + 2 * (int64_t)h.uniq;
  if (P >= (int64_t)0xffffffff) {
    cld::set_error("build_quotient: %lld distinct cluster pairs exceed the 2^32 - 1 the run numbering holds",
                   (long long)P);
    return CLDIAM_EOVERFLOW;
  }
  uint64_t *keys = b.table.keys, *vals = b.table.vals, *ktmp = b.ktmp, *vtmp = b.vtmp;
  uint32_t *head = b.head, *idx = b.idx;
  bool in_tmp = false;
  int rc = cld::radix_sort_u64(keys, vals, P, 0, 2 * kb, ktmp, vtmp, &in_tmp, rest, rest_bytes, stream);
  if (rc) return rc;
  const uint64_t *sk = in_tmp ? ktmp : keys;
  const uint64_t *sv = in_tmp ? vtmp : vals;
  uint32_t uniq = 0;
  if (P > 0) {
    k_heads<<<cld::blocks_for(P, kT, 8192), kT, 0, stream>>>(sk, P, head);
    CLD_LAUNCH_CHECK("k_heads");
    rc = cld::scan_exclusive_u32(head, idx, P, &ctl->uniq, rest, rest_bytes, stream);
    if (rc) return rc;
    CLD_HIP(hipMemcpyAsync(pinned.p, ctl, sizeof(QCtl), hipMemcpyDeviceToHost, stream));
    CLD_HIP(hipStreamSynchronize(stream));
    uniq = pinned.p->uniq;
    k_fill_inf<<<cld::blocks_for(uniq, kT, 8192), kT, 0, stream>>>(d_qw, uniq);
    CLD_LAUNCH_CHECK("k_fill_inf");
    k_reduce_runs<<<cld::blocks_for((P + kRunChunk - 1) / kRunChunk, kT, 8192), kT, 0, stream>>>(sk, sv, P, head, idx, kb, d_qcol, d_qw,
                                                                    d_qrow_ptr);
    CLD_LAUNCH_CHECK("k_reduce_runs");
  }
  k_tail_rows<<<cld::blocks_for((int64_t)k + 1, kT, 4096), kT, 0, stream>>>(sk, P, kb, k, uniq, d_qrow_ptr);
  CLD_LAUNCH_CHECK("k_tail_rows");
  CLD_HIP(hipStreamSynchronize(stream));
  *h_k = k;
  *h_qm = uniq;
  return CLDIAM_OK;
}
