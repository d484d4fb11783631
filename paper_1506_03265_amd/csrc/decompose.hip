// CLUSTER(G, tau) of Algorithm 1 (Section 3 of arXiv:1506.03265) on gfx950.
//
// Design
// ------
// One device job decomposes a batch of graphs (a single graph is a batch of
// one).  Every graph runs its own state machine
//
//   SELECT -> RELAX* -> NEXT -> [RELAX* -> NEXT]* -> ASSIGN [-> RMAX] -> SELECT ...
//                                                              -> SINGLE -> DONE
//
// and all graphs advance in lock step through "sweeps", one kernel launch
// each.  Between sweeps every graph's control step applies Algorithm 1's
// decisions: coverage test, Delta doubling, stage end, termination.
//
// Node sets are bitmaps: the uncovered nodes, the frontier (current and next)
// and the blocked nodes, one 64-bit word per 64 nodes.  Each graph's words are
// cut into chunks (one per workgroup, or a few per workgroup on large dense
// graphs); workgroup b takes chunk b and further chunks go to whichever
// workgroup asks next.  (Growth chunks of a graph whose arcs lie in a small part of
// the id range are cut at nodes of equal arcs, see kSkew.)  A workgroup owns
// the words of its chunk, so it walks its nodes in ascending order (neighbouring
// nodes share cache lines: frontiers kept as unordered lists moved several times the
// lines) and changes the sets that it walks without atomics.
//
// Node state is one u64 key per node: (growth distance << 32) | center id,
// ~0 when unset.  An offer (d_u + w, c_u) is applied with a 64-bit atomicMin,
// so concurrent offers resolve to the lexicographic minimum and the fixpoint
// of a growth level is unique whatever the order of relaxations; no step
// synchronisation is needed inside a level.  Nodes assigned in earlier
// stages keep key (0, cluster) and are sources of later stages (the effect of
// Procedure Contract); no contracted graph is built.
//
// A relaxation sweep takes only frontier nodes whose tentative distance lies
// in the current distance bucket (a narrower one for nodes with long rows)
// and keeps the others on the frontier, which orders the label-correcting
// growth like Delta-stepping without changing its fixpoint.  It goes on from
// the nodes that it improves in local rounds over a queue in LDS.  Every
// improvement of a key is the responsibility of the thread that made it: it
// goes into the workgroup's queue, or, when it lies beyond the bucket, finds
// the queue full or is left over when the rounds end, on the next frontier.  A
// queued improvement is dropped only when the key has become smaller since,
// which is another thread's responsibility.  So after a sweep every node whose
// key has not been relaxed is on the next frontier, nothing is relaxed twice
// with the same key, and neither the atomicMin on the key nor the atomicOr on
// a bitmap has to return a value (a wave goes on without waiting for them).
//
// A node is blocked when its scan stopped at an arc heavier than Delta - d_u.
// At a level's fixpoint every arc from a reached node into an unreached node
// is such a blocked arc, so NEXT, which looks at the blocked nodes' heavy arcs,
//   - finds the smallest distance at which a new node becomes reachable (Delta
//     doublings below it cannot change anything and are applied without growth);
//   - keeps exactly the blocked nodes with an unreached neighbour as the
//     frontier of the next level, or, when the stage ends, as the sources of
//     the next stage: the other nodes' offers cannot be accepted any more.
// The same sweep counts the covered nodes, so that growth itself keeps no count.
//
// Drivers: host-driven launches of one kernel per sweep (the host polls a done
// flag), or a persistent cooperative kernel with grid barriers.  In a job of
// one graph every workgroup runs the control step by itself at the start of a
// sweep, from the state and the counters that the sweep before left (state in
// a ring of two, counters in a ring of three: last, current, being cleared); it
// costs 1 to 2 us, where a launch of its own cost 6.  Jobs of several graphs
// take a control launch (one thread per graph) before every sweep.

#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <chrono>
#include <thread>
#include <vector>

#include "common.h"

namespace {

enum Phase : uint32_t {
  PH_START = 0,
  PH_SELECT = 1,
  PH_RELAX = 2,
  PH_COUNT = 3,    // covered nodes only (pull mode, or before a switch to it)
  PH_NEXT = 4,
  PH_ASSIGN = 5,
  PH_RMAX = 6,
  PH_SINGLE = 7,
  PH_DONE = 8,
  PH_IDLE = 9,     // slot of a server job that no graph has used yet (a used one stays DONE)
  PH_COMMIT = 10,  // synchronous steps: the last step's updates go into the keys
  PH_C2_INIT = 11,      // CLUSTER2: fresh state for every node
  PH_C2_SELECT = 12,    // CLUSTER2: centers of iteration i with probability 2^i / n, and Contract2's
                        // rescaled edges out of last iteration's clusters
  PH_C2_ASSIGN = 13,    // CLUSTER2: assignment, D = d + Delta2 (i - birth iteration)
  PH_PULL = 14,         // pull mode: unreached nodes take their best offer from reached neighbours
  PH_NEXT_PULL = 15,    // pull mode: NEXT computed from the unreached nodes' side
};

struct GDesc {
  const int64_t *row_ptr;   // n+1 arc offsets
  const uint64_t *arcs;
  int32_t *cluster;
  uint64_t *D;
  int64_t off;       // offset of this graph in node-indexed workspace arrays (a multiple of 64)
  double K;          // (gamma * tau) * log2(n)
  uint64_t seed;
  int32_t n;
  uint32_t words;    // bitmap words: ceil(n / 64)
  uint32_t stop;     // ceil(8 tau log2 n)
  uint32_t delta0;
  uint32_t bucket;   // distance bucket width of RELAX sweeps; 0 = unbounded
  uint32_t variant;  // CLDIAM_VARIANT_*
  uint32_t step_cap; // synchronous steps: most steps per PartialGrowth call (0 = none)
  uint32_t c2_iters; // CLUSTER2: ceil(log2 n) iterations
  int32_t local_rounds;  // workgroup-local relaxation rounds per RELAX run
  int32_t row_shift;     // long rows use a bucket of width Delta >> row_shift; < 0 = none
  int32_t chunk_factor;  // growth chunks per workgroup and sweep
  uint32_t grow_words;   // fewest bitmap words of a growth chunk
  int32_t mid_deg;       // rows of more arcs are relaxed by one wave ("long rows")
  int32_t big_deg;       // rows of more arcs are relaxed by the whole workgroup
  uint32_t lq_cap;       // slots of the local relaxation queue used (at most kLocalCap)
  uint32_t pull_mode;    // CLDIAM_PULL_*: when new levels and stages pull from the unreached side
  uint32_t hub_deg;      // rows of more arcs are hub rows (kHubDegree x the average degree)
  uint64_t hub_min;      // more arcs than this in hub rows: a skewed, low-diameter graph
};

// Control-owned state of one graph.
struct GState {
  uint64_t T;
  uint64_t rounds, updates, msgs;   // synchronous steps
  uint64_t radius;      // max D
  uint64_t radius1;     // CLUSTER2: R_CL of the preliminary CLUSTER run
  uint64_t blk_arcs;    // heavy arcs left on the rows marked blocked in this level (what a push rescan reads)
  uint64_t arcs;        // arcs read by relaxation (diagnostic)
  uint32_t phase, stage, delta;
  uint32_t nU;          // uncovered nodes at the start of the stage
  uint32_t cov;         // covered in this stage, at the last count
  uint32_t centers;     // centers drawn in this stage
  uint32_t cur, nxt, blk, alt;   // roles of the four bitmaps: frontier, next frontier, blocked, spare (empty)
  int32_t status;
  uint32_t levels, sweeps, centers_total, singletons;
  uint32_t theta;       // RELAX sweeps relax frontier nodes with tentative distance below theta
  uint32_t row_base;    // ... and nodes of long rows only below row_limit(row_base)
  uint32_t steps_call;  // synchronous steps of the current PartialGrowth call
  uint32_t merge;       // synchronous steps: the blocked nodes join the frontier of the next RELAX
  uint32_t c2;          // 1 while in CLUSTER2's iterations
  uint32_t pull;        // 1 once the graph grows new levels and stages by pulling (see PH_PULL)
  uint32_t pull_base;   // distance at which the current pulled level starts (its first bucket)
  uint32_t again;       // PULL passes of this level so far
  uint32_t src_blk;     // the next stage's sources are the blocked set (no NEXT has filtered it)
  uint32_t records;     // some long row has a scan record
  uint32_t cuts;        // growth chunks cut at nodes of equal arcs (0: chunks of equal ids)
  uint32_t closed;      // one graph: done, and the books are closed (later sweeps return at once)
};
static_assert(sizeof(GState) % 4 == 0, "copied word by word");

// What a sweep of one graph reports to its next control step.
struct alignas(128) GCount {
  uint32_t fmin;        // RELAX: smallest tentative distance on the next frontier (~0: it is empty)
  uint32_t cov;         // covered nodes (COUNT, NEXT, C2_ASSIGN; synchronous steps: newly covered)
  uint32_t centers;     // centers drawn
  uint32_t upd;         // synchronous steps: nodes updated
  uint32_t records;
  uint32_t pad;
  unsigned long long next;      // NEXT: smallest reach distance
  unsigned long long radius;    // max D of the nodes assigned
  unsigned long long msgs;      // synchronous steps: offers sent
  unsigned long long blk_arcs;
  unsigned long long hub_arcs;  // first SELECT (auto pull mode): arcs in hub rows
  unsigned long long arcs;
};

// Job-wide counters of one sweep.
struct alignas(128) SweepCount {
  uint32_t cursor;   // chunks taken beyond the first nblocks
  uint32_t pad0[31];
  uint32_t idle;     // workgroups that have finished the sweep
  uint32_t pad1[31];
};

struct Ctl {
  uint32_t done;      // 1 when every graph is DONE
  uint32_t total;     // chunks of the current sweep (several graphs)
  uint32_t error;     // first error status (as positive code) or 0
  uint32_t iterations;
  uint32_t timeout;   // barrier wait gave up
  uint32_t pad;
  unsigned long long t_start;   // wall clock at the first control step
  unsigned long long t_limit;   // ticks after which the job stops with a timeout
  SweepCount sc[3];
  CldBarrier bar;
};

struct Job {
  const GDesc *desc;
  GState *st;        // one per graph (one graph: its final state)
  GState *ring;      // one graph: the state after the last sweep and the current one
  GCount *cn;        // one per graph (one graph: a ring of three)
  Ctl *ctl;
  uint32_t *seg;     // [0, G]: exclusive prefix of per-graph chunks; [G+1, 2G]: words per chunk (0: cut)
  int32_t *log;      // G x CLDIAM_STAGE_LOG x 4
  uint64_t *key;
  uint64_t *keyn;    // synchronous steps: updates of the odd steps (see step_state); CLUSTER2's iterations:
                     // growth distance of the assigned nodes; otherwise, for long rows, the key of the
                     // row's last scan
  uint32_t *slim;    // with keyn: the light limit (Delta - d) of that scan; arcs up to it have been offered
  uint64_t *R;       // by center: largest D of its cluster after the last stage; CLUSTER2: birth iteration;
                     // synchronous steps: for nodes with a distance, updates of the even steps as well
  uint64_t *U;       // bitmap: uncovered nodes
  uint64_t *F;       // four bitmaps, one after the other, in the roles of GState
  int32_t *cut;      // graph at node slot off: first node of each of its cuts, from 2 (off / 64) on, and the end
  int64_t fwords;    // words of one
  int32_t G;
  int32_t nblocks;        // workgroups of a sweep launch
  uint32_t *hmirror = nullptr;   // host-driven job: mapped pinned words {control steps done, done flag} that
                                 // the host polls while it queues steps (nullptr: not mirrored)
  uint32_t cutoff;        // a workgroup ends its local rounds once this many workgroups have finished the
                          // sweep (what it leaves is on the next frontier)
};

constexpr int kThreads = 1024;        // control workgroup of many graphs
constexpr int kSweepThreads = 1024;   // sweep workgroup
constexpr int kCuThreads = 1024;      // sweep threads resident per CU
constexpr int kWaves = kSweepThreads / 64;
constexpr int kList = 8 * kSweepThreads;       // nodes of one expansion of a bitmap window
constexpr int kLocalCap = 4 * kSweepThreads;   // LDS local-round queue slots
constexpr int kMidDeg = 32;       // default: rows above this degree are relaxed by one wave
constexpr int kBigDeg = 8192;     // default: rows above this degree are relaxed by the whole workgroup
constexpr int kMidCap = 2 * kSweepThreads;   // deferred wave rows per pass
constexpr int kBigCap = kSweepThreads / 8;   // deferred workgroup rows per pass
constexpr int kLocalRounds = 16;  // default local relaxation rounds per RELAX run
// Default: local rounds do not wait for the other workgroups.  Ended once 75%
// of the workgroups have finished the sweep, the rest of the growth waits for
// the next launch (64 x 64 mesh 0.69 instead of 0.43 ms, 1153 x 1021 mesh 3.05
// instead of 2.36, road-like 4096 x 4096 mesh 9.5 instead of 8.7; 600 meshes of some
// 150 nodes in one job 1.83 instead of 1.66, but 64 geometric graphs of up to a
// million nodes 7.5 instead of 8.7).
constexpr int kLocalCutoffPct = 100;
constexpr int kDenseWaveRow = 128;     // default wave_row_min on graphs of more than kDenseDegree arcs per node
constexpr int kLocalRoundsDense = 2;   // ... on graphs with more than kDenseDegree arcs per node and
constexpr int kDenseDegree = 16;       // more than kDenseLarge nodes (none on smaller dense graphs)
constexpr int32_t kDenseLarge = 1 << 21;
constexpr int32_t kDenseChunks = 3;     // growth chunks per workgroup on dense graphs
constexpr int32_t kRowShiftMin = 5;     // default long-row bucket: Delta >> shift, shift from the arc count
constexpr int32_t kRowShiftMax = 8;
constexpr int kJobSeconds = 60;   // device-side limit of one decomposition job
// Fewest bitmap words of a growth chunk: as many as hold kGrowArcs arcs on average,
// but no more than kGrowWords; and of a node pass's.  (8 words, 512 nodes, whatever
// their rows, left the complete graph of 3000 nodes to six workgroups: 1.45 ms, now
// 0.54.)
constexpr uint32_t kGrowWords = 8;
constexpr int64_t kGrowArcs = 16384;
constexpr uint32_t kPassWords = 16;
// Chunks of equal ids leave most of the card idle where the arcs lie in few of
// them, as in graphs numbered by degree.  So when the fullest of kRanges equal id
// ranges holds more than kSkew times the average, growth chunks are cut at nodes
// where arcs, and kNodeCost for every node, are equal (at least kCutArcs of them):
// R-MAT scale 21 numbered by degree takes 5.1 ms in steps, 10.7 in CLUSTER2 and 5.2
// pushed; in chunks of equal ids 240, 240 and 100.  A relaxation takes kCutChunks per
// workgroup, since a frontier of neighbouring nodes lies in few of them, and passes
// over those without one (a band of 60 arcs a node beside a mesh of a million nodes
// in CLUSTER2: 44 ms with one chunk, 27 with 4, 26 with 8).  Graphs of many nearly
// empty sweeps lose by it (R-MAT scale 17 with its isolated nodes 54 to 74 ms).
// Meshes and R-MAT graphs of random numbers stay below a skew of 2.
constexpr int kRanges = 64;
constexpr uint64_t kSkew = 4;
constexpr uint64_t kNodeCost = 4;
constexpr uint64_t kCutArcs = 4096;
constexpr uint64_t kCutChunks = 4;
constexpr uint32_t kRmaxSlots = 1024;   // RMAX: LDS table of cluster maxima (direct-mapped by center id)
constexpr uint32_t kRmaxFree = 0xffffffffu;
static_assert(kRmaxSlots == 1024, "RMAX slots are the top 10 bits of a 32-bit hash");
constexpr uint32_t kPullArcs = 8;   // pull-mode switch: heavy blocked arcs per unreached node
// PULL is repeated, by then over all uncovered nodes, while a pass changes more
// than one in 2^kPullAgainShift of them.  A repeated pass reads a row only up to
// its node's distance (0.4 to 1 ms on R-MAT scale 24, where pushing from the nodes
// of the first pass took 13 ms and some 380 million arcs), and each hop of the
// last few nodes costs less pushed.  With a wave for every long row (see kPullRow)
// R-MAT scale 24 and 18 (graphs of perf/cases.py, decomposition alone) and two dozen
// mixed requests took 15.4, 1.15 and 11.6 ms with
// one pass, 10.9, 1.16 and 9.8 with a quarter, 10.4, 1.17 and 9.4 with 1/16, 10.6,
// 0.76 and 9.4 with 1/32, 11.2, 0.74 and 9.6 with 1/256.  kPullMost bounds the
// passes where distances take many hops.
constexpr uint32_t kPullAgainShift = 5;
constexpr uint32_t kPullMost = 16;
// A reached node's row is read up to its distance only, a few arcs even of a long
// one, so in pull passes rows of up to kPullRow arcs stay with one thread, 64 rows
// in flight per wave: the same take 8.7, 0.71 and 8.6 ms (10.1 on the benchmark's
// R-MAT scale 24); 10.5, 0.75 and 9.1 with a wave for every row above 128 arcs;
// 9.7, 1.06 and 9.4 with a thread for every row.
constexpr int32_t kPullRow = 1024;
constexpr int64_t kHubDegree = 8;   // hub rows: more than kHubDegree x the average degree ...
constexpr int64_t kHubShare = 8;    // ... holding more than 1/kHubShare of the arcs: pull from the first stage

// ------------------------------------------------------------- control --

// A failing graph stops alone; the other graphs of the job go on.
__device__ __forceinline__ void fail(GState &s, int status) {
  s.status = status;
  s.phase = PH_DONE;
}

__device__ __forceinline__ void finish(const GDesc &d, GState &s);

__device__ __forceinline__ void begin_stage(const GDesc &d, GState &s) {
  s.centers = 0;
  s.cov = 0;
  if (s.nU == 0 || s.nU < d.stop || d.n < 2) {
    s.phase = PH_SINGLE;
    if (s.nU == 0) finish(d, s);   // nobody is left to be a singleton
    return;
  }
  if (s.stage >= CLDIAM_MAX_STAGES) {
    fail(s, CLDIAM_ESTAGES);
    return;
  }
  double p = d.K / (double)s.nU;
  s.T = p >= 1.0 ? ((uint64_t)1 << 32) : (uint64_t)floor(p * 4294967296.0);
  s.phase = PH_SELECT;
}

// Upper end (exclusive) of the distance bucket that starts at lo.
__device__ __forceinline__ uint32_t bucket_limit(const GDesc &d, uint32_t lo) {
  if (d.bucket == 0) return 0xffffffffu;
  const uint64_t t = (uint64_t)lo + d.bucket;
  return t < 0xffffffffull ? (uint32_t)t : 0xffffffffu;
}

// Upper end (exclusive) of the narrower bucket of rows of more than mid_deg
// arcs.  Relaxing such a row before its node's distance is nearly final
// costs a full rescan when the distance drops again, so these rows wait
// until the frontier minimum comes within Delta / 2^row_shift of them.
__device__ __forceinline__ uint32_t row_limit(const GDesc &d, uint32_t delta, uint32_t lo) {
  if (d.row_shift < 0 || lo == 0xffffffffu) return 0xffffffffu;
  const uint32_t w = delta >> d.row_shift;
  const uint64_t t = (uint64_t)lo + (w ? w : 1u);
  return t < 0xffffffffull ? (uint32_t)t : 0xffffffffu;
}

__device__ __forceinline__ void swap_roles(uint32_t &a, uint32_t &b) {
  const uint32_t t = a;
  a = b;
  b = t;
}

// A growth starts at distance lo on the frontier.
__device__ __forceinline__ void begin_growth(const GDesc &d, GState &s, uint32_t lo) {
  s.theta = bucket_limit(d, lo);
  s.row_base = lo;
  s.phase = PH_RELAX;
}

// CLUSTER2: iteration s.stage + 1 draws centers with probability 2^i / n.
__device__ __forceinline__ void c2_begin_iteration(const GDesc &d, GState &s) {
  const int i = (int)s.stage + 1;
  const double p = ldexp(1.0, i) / (double)d.n;
  s.T = p >= 1.0 ? ((uint64_t)1 << 32) : (uint64_t)floor(p * 4294967296.0);
  s.centers = 0;
  s.cov = 0;
  s.phase = PH_C2_SELECT;
}

// Synchronous steps: a new PartialGrowth call at the current Delta.
__device__ __forceinline__ void begin_call(GState &s) {
  s.levels++;
  s.steps_call = 0;
  s.theta = 0xffffffffu;
  s.row_base = 0xffffffffu;
  s.phase = PH_RELAX;
}

// Pull mode pays once the heavy arcs of the blocked rows, which a push rescan
// and a push NEXT read, outweigh kPullArcs arcs per unreached node (about
// what pulling reads per node: its rows are sorted by weight and it stops at
// its first reached neighbour).
__device__ __forceinline__ bool pull_pays(const GState &s, uint32_t unreached) {
  return s.blk_arcs > (uint64_t)kPullArcs * unreached;
}

__device__ __forceinline__ bool double_delta(GState &s) {
  if (2ull * s.delta > CLD_DELTA_MAX) {
    fail(s, CLDIAM_EOVERFLOW);
    return false;
  }
  s.delta *= 2;
  return true;
}

// Doubles Delta to the first value at which a node at distance `reach` is
// reached, one level per doubling.
__device__ __forceinline__ bool raise_delta(GState &s, uint64_t reach) {
  uint64_t dl = s.delta;
  do {
    if (2 * dl > CLD_DELTA_MAX) {
      fail(s, CLDIAM_EOVERFLOW);
      return false;
    }
    dl *= 2;
    s.levels++;
  } while (dl < reach);
  s.delta = (uint32_t)dl;
  s.blk_arcs = 0;
  return true;
}

__device__ __forceinline__ void log_stage(const GState &s, int32_t *log) {
  if (!log || s.stage >= CLDIAM_STAGE_LOG) return;
  int32_t *lg = log + (size_t)s.stage * 4;
  lg[0] = (int32_t)s.nU; lg[1] = (int32_t)s.centers; lg[2] = (int32_t)s.cov; lg[3] = (int32_t)s.delta;
}

// CLUSTER is complete (singletons included): the end, or CLUSTER2's start.
__device__ __forceinline__ void finish(const GDesc &d, GState &s) {
  s.singletons = s.nU;
  s.phase = PH_DONE;
  if (d.variant != CLDIAM_VARIANT_CLUSTER2) return;
  const uint64_t r1 = s.radius;
  if (2 * r1 > CLD_DELTA_MAX) { fail(s, CLDIAM_EOVERFLOW); return; }
  s.radius1 = r1;
  s.delta = (uint32_t)(2 * r1);
  if (d.c2_iters == 0) return;   // one node: its own cluster
  s.c2 = 1;
  s.pull = 0;
  s.stage = 0;
  s.levels = 0;
  s.centers_total = 0;
  s.singletons = 0;
  s.radius = 0;
  s.phase = PH_C2_INIT;
}

// The stage's covered nodes are assigned and off the uncovered set.
__device__ __forceinline__ void end_stage(const GDesc &d, GState &s, int32_t *log) {
  log_stage(s, log);
  s.nU -= s.cov;
  s.stage++;
  if (s.c2) {
    // the blocked set stays: next iteration's Contract2 boundary
    if (s.nU == 0) {
      // iterations without an uncovered node change nothing
      s.centers = 0;
      s.cov = 0;
      for (; s.stage < d.c2_iters; s.stage++) {
        s.levels++;
        log_stage(s, log);
      }
    }
    if (s.stage >= d.c2_iters) s.phase = PH_DONE;
    else c2_begin_iteration(d, s);
    return;
  }
  if (d.variant != CLDIAM_VARIANT_STEPS) {
    // sources of the next stage: the nodes that NEXT kept (already the
    // frontier), or the blocked set; in pull mode none (SELECT and PULL
    // empty both): the uncovered nodes pull from their assigned neighbours
    if (!s.pull && d.pull_mode == CLDIAM_PULL_AUTO && pull_pays(s, s.nU)) s.pull = 1;
    if (s.src_blk) swap_roles(s.cur, s.blk);
    s.src_blk = 0;
    s.blk_arcs = 0;
  }
  // (synchronous steps: the active set and, with s.merge, the blocked set)
  begin_stage(d, s);
}

// Transition of one graph after a sweep of its current phase, whose counters
// are c.  log: its stage log (nullptr: another workgroup writes it).
__device__ __forceinline__ void control_graph(const GDesc &d, GState &s, const GCount &c, int32_t *log) {
  s.arcs += c.arcs;
  s.records |= c.records;
  switch (s.phase) {
    case PH_START:
      s.delta = d.delta0;
      s.stage = 0;
      s.nU = (uint32_t)d.n;
      s.cur = 0; s.nxt = 1; s.blk = 2; s.alt = 3;
      if ((uint64_t)s.delta > CLD_DELTA_MAX) { fail(s, CLDIAM_EOVERFLOW); break; }
      s.pull = d.pull_mode == CLDIAM_PULL_ALWAYS ? 1u : 0u;
      begin_stage(d, s);
      break;
    case PH_SELECT:
      // frontier = sources from the previous stage + the new centers, all at
      // distance 0
      s.centers = c.centers;
      s.cov = c.centers;
      s.centers_total += c.centers;
      if (d.variant == CLDIAM_VARIANT_STEPS) {
        // the outer loop's test comes first: enough new centers end the stage
        if (2ull * s.cov >= (uint64_t)s.nU) { s.phase = PH_ASSIGN; break; }
        begin_call(s);
        break;
      }
      s.levels++;
      // a skewed degree distribution (hub rows holding a large share of the
      // arcs) goes with a low diameter: the growth then reaches most nodes
      // within a few hops, which a pull pass does for less than pushing
      if (!s.pull && s.stage == 0 && d.pull_mode == CLDIAM_PULL_AUTO && c.hub_arcs > d.hub_min) s.pull = 1;
      if (s.pull) {
        // the uncovered nodes pull from the assigned nodes and the new centers
        s.pull_base = 0;
        s.again = 0;
        s.phase = PH_PULL;
        break;
      }
      begin_growth(d, s, 0);
      break;
    case PH_PULL:
      // while a pass changes many nodes another costs less than pushing from
      // them (see kPullAgainShift); then those that it changed are the frontier
      s.again++;
      if (c.upd > s.nU >> kPullAgainShift && s.again < kPullMost) break;
      begin_growth(d, s, c.fmin != 0xffffffffu && c.fmin > s.pull_base ? c.fmin : s.pull_base);
      break;
    case PH_RELAX:
      s.sweeps++;
      if (d.variant == CLDIAM_VARIANT_STEPS) {
        s.rounds++;
        s.steps_call++;
        s.msgs += c.msgs;
        if (s.merge) { swap_roles(s.blk, s.alt); s.merge = 0; }   // the old blocked set is used up
        s.updates += c.upd;
        s.cov += c.cov;
        swap_roles(s.cur, s.nxt);   // the updated nodes are the next active set
        if (c.upd == 0) {
          s.phase = PH_NEXT;      // fixpoint: is any uncovered node reachable?
        } else if (2ull * s.cov >= (uint64_t)s.nU) {
          s.merge = 1;
          s.phase = PH_COMMIT;
        } else if (d.step_cap && s.steps_call >= d.step_cap) {
          if (!double_delta(s)) break;
          s.merge = 1;
          begin_call(s);
        }
        break;
      }
      s.blk_arcs += c.blk_arcs;
      if (c.fmin != 0xffffffffu) {
        swap_roles(s.cur, s.nxt);
        // the next bucket starts at the smallest distance on the frontier
        const uint32_t th = bucket_limit(d, c.fmin);
        if (th > s.theta) s.theta = th;
        if (c.fmin > s.row_base) s.row_base = c.fmin;
      } else if (s.c2) {
        s.phase = PH_C2_ASSIGN;
      } else {
        // fixpoint.  In pull mode, and when a switch to it may pay (blocked
        // heavy arcs for more than 1/16 of the nodes), count before choosing
        // the side that NEXT looks from.
        s.phase = s.pull || (d.pull_mode == CLDIAM_PULL_AUTO && pull_pays(s, s.nU >> 4)) ? PH_COUNT : PH_NEXT;
      }
      break;
    case PH_COUNT:
      s.cov = c.cov;
      if (2ull * s.cov >= (uint64_t)s.nU) {
        s.src_blk = s.pull ? 0u : 1u;
        s.phase = PH_ASSIGN;
        break;
      }
      if (!s.pull && pull_pays(s, s.nU - s.cov)) s.pull = 1;
      s.phase = s.pull ? PH_NEXT_PULL : PH_NEXT;
      break;
    case PH_COMMIT:
      s.phase = PH_ASSIGN;
      break;
    case PH_NEXT:
      if (d.variant == CLDIAM_VARIANT_STEPS) {
        s.merge = 1;
        if (c.next == CLD_INF64) s.phase = PH_ASSIGN;
        else if (double_delta(s)) begin_call(s);
        break;
      }
      s.cov = c.cov;
      if (2ull * s.cov >= (uint64_t)s.nU || c.next == CLD_INF64) s.phase = PH_ASSIGN;
      else if (raise_delta(s, c.next)) begin_growth(d, s, (uint32_t)c.next);
      break;
    case PH_NEXT_PULL:
      if (c.next == CLD_INF64) {
        s.phase = PH_ASSIGN;
      } else if (raise_delta(s, c.next)) {
        s.pull_base = (uint32_t)c.next;
        s.again = 0;
        s.phase = PH_PULL;
      }
      break;
    case PH_ASSIGN:
      if (c.radius > s.radius) s.radius = c.radius;
      if (s.stage > 0) s.phase = PH_RMAX;
      else end_stage(d, s, log);
      break;
    case PH_RMAX:
      end_stage(d, s, log);
      break;
    case PH_SINGLE:
      finish(d, s);
      break;
    case PH_C2_INIT:
      s.nU = (uint32_t)d.n;
      s.cur = 0; s.nxt = 1; s.blk = 2; s.alt = 3;
      c2_begin_iteration(d, s);
      break;
    case PH_C2_SELECT:
      s.centers = c.centers;
      s.centers_total += c.centers;
      s.levels++;
      begin_growth(d, s, 0);
      break;
    case PH_C2_ASSIGN:
      if (c.radius > s.radius) s.radius = c.radius;
      s.cov = c.cov;
      end_stage(d, s, log);
      break;
    default:
      break;
  }
}

__device__ __forceinline__ void clear_count(GCount &c) {
  c.fmin = 0xffffffffu;
  c.cov = c.centers = c.upd = c.records = 0;
  c.next = CLD_INF64;
  c.radius = c.msgs = c.blk_arcs = c.hub_arcs = c.arcs = 0;
}

__device__ __forceinline__ bool is_growth(uint32_t phase) {
  return phase == PH_RELAX || phase == PH_NEXT || phase == PH_PULL || phase == PH_NEXT_PULL;
}

// Bitmap words per chunk of a graph's sweep: chunk_factor chunks per workgroup
// in growth, one in node passes, none smaller than a wave or two of nodes.
__device__ __forceinline__ uint32_t chunk_words(const GDesc &d, uint32_t phase, int32_t nblocks) {
  const bool grow = is_growth(phase);
  const uint32_t nch = (uint32_t)nblocks * (grow ? (uint32_t)d.chunk_factor : 1u);
  const uint32_t per = (d.words + nch - 1) / nch, least = grow ? d.grow_words : kPassWords;
  return per > least ? per : least;
}

// Where the i-th of kRanges equal id ranges begins in the arcs.
__device__ __forceinline__ uint64_t range_start(const GDesc &d, int i) {
  const int64_t at = i * (((int64_t)d.n + kRanges - 1) / kRanges);
  return (uint64_t)d.row_ptr[at < d.n ? at : d.n];
}

// Whether a graph is too small to be cut by arcs.
__device__ __forceinline__ bool below_cuts(const GDesc &d) {
  return (uint64_t)d.row_ptr[d.n] + kNodeCost * (uint64_t)d.n < 2 * kCutArcs;
}

// Growth chunks cut by arcs for a graph whose fullest id range holds `fullest`
// (0: chunks of equal ids will do).
__device__ __forceinline__ uint32_t cuts_for(const GDesc &d, uint64_t fullest, int32_t nblocks) {
  const uint64_t m = (uint64_t)d.row_ptr[d.n];
  if (fullest * kRanges <= kSkew * m) return 0;
  const uint64_t most = kCutChunks * (uint64_t)nblocks * (uint32_t)d.chunk_factor, fit = (m + kNodeCost * (uint64_t)d.n) / kCutArcs;
  uint64_t k = fit < most ? fit : most;
  if (k > d.words) k = d.words;
  return k > 1 ? (uint32_t)k : 0u;
}

// The phases whose chunks are cut so.
__device__ __forceinline__ bool by_arcs(const GState &s) {
  return s.cuts != 0 && (is_growth(s.phase) || s.phase == PH_C2_SELECT);
}

// Chunks of such a phase.  Only a relaxation, whose frontier may lie in a few
// neighbouring ones, takes kCutChunks per workgroup.
__device__ __forceinline__ uint32_t cuts_per_chunk(const GState &s) { return s.phase == PH_RELAX ? 1u : (uint32_t)kCutChunks; }
__device__ __forceinline__ uint32_t cut_chunks(const GState &s) {
  return (s.cuts + cuts_per_chunk(s) - 1) / cuts_per_chunk(s);
}

// The first node of cut i of k: where arcs and nodes before it cost i / k.
__device__ __forceinline__ int32_t cut_at(const GDesc &d, uint32_t i, uint32_t k) {
  const uint64_t m = (uint64_t)d.row_ptr[d.n], want = (m + kNodeCost * (uint64_t)d.n) * i / k;
  int32_t lo = 0, hi = d.n;
  while (lo < hi) {
    const int32_t mid = lo + ((hi - lo) >> 1);
    if ((uint64_t)d.row_ptr[mid] + kNodeCost * (uint64_t)mid < want) lo = mid + 1; else hi = mid;
  }
  return lo;
}

// Device time limit of a job, checked once per control step.
__device__ __forceinline__ void check_time(Ctl *ctl) {
  const unsigned long long now = wall_clock64();
  if (ctl->iterations == 0) ctl->t_start = now;
  else if (now - ctl->t_start > ctl->t_limit && ctl->error == 0) atomicCAS(&ctl->error, 0u, (uint32_t)(-CLDIAM_ETIMEOUT));
}

__device__ __forceinline__ void report(const Job &job, uint32_t iterations, uint32_t done) {
  if (!job.hmirror) return;
  __hip_atomic_store(&job.hmirror[0], iterations, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __hip_atomic_store(&job.hmirror[1], done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// One workgroup of T threads: control of every graph of a job of several,
// then the next sweep's chunks.
// restart: the job's time limit counts from here.
template <int T>
__device__ void control_block(const Job &job, bool restart = false) {
  __shared__ uint32_t scan[T];
  __shared__ uint32_t carry, alldone;
  __shared__ unsigned long long work;
  Ctl *ctl = job.ctl;
  if (threadIdx.x == 0) {
    carry = 0;
    alldone = 1;
    work = 0;
    if (restart) ctl->iterations = 0;
    check_time(ctl);
  }
  __syncthreads();
  for (int base = 0; base < job.G; base += T) {
    const int g = base + (int)threadIdx.x;
    if (g < job.G) {
      GState &s = job.st[g];
      if (s.phase != PH_DONE && s.phase != PH_IDLE) {
        if (s.phase == PH_START && !below_cuts(job.desc[g])) {
          uint64_t fullest = 0, last = 0;
#pragma unroll 16
          for (int i = 1; i <= kRanges; ++i) {
            const uint64_t x = range_start(job.desc[g], i);
            fullest = x - last > fullest ? x - last : fullest;
            last = x;
          }
          s.cuts = cuts_for(job.desc[g], fullest, job.nblocks);
        }
        if (ctl->error == 0) control_graph(job.desc[g], s, job.cn[g], job.log + (size_t)g * CLDIAM_STAGE_LOG * 4);
        else s.phase = PH_DONE;
        clear_count(job.cn[g]);
        if (s.phase != PH_DONE) {
          atomicAdd(&work, (unsigned long long)job.desc[g].words);
          atomicAnd(&alldone, 0u);
        }
      }
    }
  }
  __syncthreads();
  // A chunk is no smaller than half the sweep's average words per workgroup:
  // many small graphs then take a few chunks each, instead of one per
  // workgroup that would pay a chunk's fixed cost for a handful of nodes.
  const unsigned long long avg = work / (2ull * (unsigned long long)job.nblocks);
  for (int base = 0; base < job.G; base += T) {
    const int g = base + (int)threadIdx.x;
    uint32_t chunks = 0;
    if (g < job.G) {
      const uint32_t phase = job.st[g].phase;
      uint32_t per = 0;
      if (by_arcs(job.st[g])) {
        chunks = cut_chunks(job.st[g]);
      } else if (phase != PH_DONE && phase != PH_IDLE) {
        per = chunk_words(job.desc[g], phase, job.nblocks);
        if (per < avg) per = (uint32_t)avg;
        chunks = (job.desc[g].words + per - 1) / per;
      }
      job.seg[job.G + 1 + g] = per;
    }
    scan[threadIdx.x] = chunks;
    __syncthreads();
    for (int o = 1; o < T; o <<= 1) {
      uint32_t x = threadIdx.x >= (unsigned)o ? scan[threadIdx.x - o] : 0;
      __syncthreads();
      scan[threadIdx.x] += x;
      __syncthreads();
    }
    if (g < job.G) job.seg[g] = carry + scan[threadIdx.x] - chunks;
    __syncthreads();
    if (threadIdx.x == T - 1) carry += scan[T - 1];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    job.seg[job.G] = carry;
    ctl->total = carry;
    ctl->sc[0].cursor = 0;
    ctl->sc[0].idle = 0;
    ctl->iterations++;
    ctl->done = alldone;
    report(job, ctl->iterations, alldone);
  }
  __syncthreads();
}

// --------------------------------------------------------------- sweeps --

// LDS of a sweep workgroup.
struct Stage {
  union {
    struct {                     // growth
      int32_t list[kList];       // nodes of the window being walked
      uint64_t qk[2][kLocalCap]; // local relaxation queues: key to relax with ...
      int32_t qv[2][kLocalCap];  // ... and node
      int32_t mid[kMidCap];      // rows deferred to one wave each
      int32_t big[kBigCap];      // rows deferred to the whole workgroup
    };
    struct {                     // RMAX: per-cluster maxima of this workgroup's nodes
      uint32_t tag[kRmaxSlots];
      unsigned long long mx[kRmaxSlots];
    } rmax;
  };
  uint32_t qn[3];              // queued nodes, by round modulo 3
  uint32_t mid_cnt[2], big_cnt[2];   // of the even and the odd passes (see coop_rows)
  unsigned long long blk_min;  // workgroup minimum over a big row (NEXT, PULL)
  unsigned long long row_key;  // key of the big row being scanned
  int32_t row_lo;              // end of its light prefix (index within the row)
  int32_t row_start;           // first arc of its scan (index within the row)
  uint32_t wsum[2][kWaves];
  uint32_t chunk;              // next chunk of this workgroup
  uint32_t stop;               // local rounds end early: most of the grid has finished the sweep
  GCount sum;                  // this workgroup's part of the sweep's counters
  GCount last;                 // one graph: the counters of the sweep before ...
  GState st;                   // ... and the state that the control step made of it
};

// One graph's sweep as a workgroup sees it.
struct Run {
  const Job &job;
  const GDesc &d;
  const GState &s;
  Stage &S;
  uint64_t *key;         // this graph's part of the node arrays and bitmaps
  uint64_t *keyn;
  uint32_t *slim;
  uint64_t *pend, *pnew;   // synchronous steps: updates of the last step and of this one
  uint64_t *cur, *nxt;
  uint64_t *mark;        // where blocked nodes are marked (nullptr: nowhere)
  uint32_t delta, theta, theta_row;
  bool resume;           // long rows resume their last scan
  uint32_t na, nb;       // nodes of a chunk cut by arcs, which may share its first and last word (nb = 0: whole words)
  uint32_t pass = 0;     // list passes so far
  uint32_t q = 0, qslot = 0;   // queue and counter that improvements go to
  // per-thread sums
  uint32_t updated = 0, covered = 0;   // synchronous steps
  uint32_t scanned = 0, heavy = 0, fmin = 0xffffffffu;
  unsigned long long acc = 0;   // NEXT: min; ASSIGN: max; SELECT: hub arcs
};

__device__ __forceinline__ void set_bit(uint64_t *bits, int32_t v) {
  atomicOr((unsigned long long *)&bits[v >> 6], 1ull << (v & 63));
}

// The workgroup's nodes of word w.
__device__ __forceinline__ uint64_t own_bits(const Run &r, uint32_t w) {
  if (r.nb == 0) return ~0ull;
  uint64_t x = ~0ull;
  if (w == r.na >> 6) x <<= r.na & 63;
  if (w == (r.nb - 1) >> 6) x &= ~0ull >> (63 - ((r.nb - 1) & 63));
  return x;
}

// Takes them out of word w of a set that no other workgroup adds to.
__device__ __forceinline__ void drop_bits(const Run &r, uint64_t *bits, uint32_t w) {
  const uint64_t own = own_bits(r, w);
  if (own == ~0ull) bits[w] = 0;
  else atomicAnd((unsigned long long *)&bits[w], (unsigned long long)~own);
}

__device__ __forceinline__ uint64_t take_bits(const Run &r, uint64_t *bits, uint32_t w) {
  const uint64_t x = bits[w] & own_bits(r, w);
  if (x) drop_bits(r, bits, w);
  return x;
}

// v stays for the next sweep, at tentative distance dist.
__device__ __forceinline__ void leave(Run &r, int32_t v, uint32_t dist) {
  set_bit(r.nxt, v);
  if (dist < r.fmin) r.fmin = dist;
}

// u's scan stopped at a heavy arc; `heavy` arcs are left on its row.  word is
// u's word of the blocked set as read before.
__device__ __forceinline__ void mark_blocked(Run &r, int32_t u, uint64_t word, int32_t heavy) {
  if (word >> (u & 63) & 1) return;
  set_bit(r.mark, u);
  r.heavy += (uint32_t)heavy;
}

__device__ __forceinline__ uint64_t marks_of(const Run &r, int32_t u) { return r.mark ? r.mark[u >> 6] : ~0ull; }

// Applies a thread's K offers cand[i] to v[i] that beat the keys read
// (better[i]) and queues them: one reservation per wave.
template <int K>
__device__ __forceinline__ void improve(Run &r, const bool (&better)[K], const int32_t (&v)[K],
                                        const uint64_t (&cand)[K]) {
  const uint64_t below = (1ull << (threadIdx.x & 63)) - 1ull;
  uint32_t at[K], total = 0;
  bool near[K];
#pragma unroll
  for (int i = 0; i < K; ++i) {
    if (better[i]) atomicMin((unsigned long long *)&r.key[v[i]], (unsigned long long)cand[i]);
    near[i] = better[i] && (uint32_t)(cand[i] >> 32) < r.theta;
    const uint64_t m = __ballot(near[i]);
    at[i] = total + (uint32_t)__popcll(m & below);
    total += (uint32_t)__popcll(m);
  }
  if (total) {
    uint32_t base = 0;
    const int first = __ffsll((long long)__ballot(true)) - 1;
    if ((int)(threadIdx.x & 63) == first) base = atomicAdd(&r.S.qn[r.qslot], total);
    base = (uint32_t)__builtin_amdgcn_readlane((int)base, first);
#pragma unroll
    for (int i = 0; i < K; ++i) {
      if (!near[i]) continue;
      const uint32_t slot = base + at[i];
      if (slot < r.d.lq_cap) {
        r.S.qv[r.q][slot] = v[i];
        r.S.qk[r.q][slot] = cand[i];
      } else {
        leave(r, v[i], (uint32_t)(cand[i] >> 32));
      }
    }
  }
#pragma unroll
  for (int i = 0; i < K; ++i)
    if (better[i] && !near[i]) leave(r, v[i], (uint32_t)(cand[i] >> 32));
}

constexpr int kArcBatch = 2;    // arcs of a long row in flight per thread (4 spill registers)
constexpr int kScanBatch = 4;   // ... and of a row that one thread scans (NEXT, PULL)

// Synchronous steps.  A step's offers are judged against the state before it,
// and the lexicographic minimum over a node's offers is its state after it.  A
// step's updates go to one of two arrays in turn (pnew; atomicMin over what an
// earlier step left there, which is never below the node's state) and the nodes
// that have one to the next frontier.  The next step's state of a node is the
// smaller of its key and its entry in that array (then pend): nothing writes
// either in that step but the owner of an updated node, who copies the update
// into the key.  So a step is one sweep, bound by its launch and the chain of
// dependent accesses of one hop (20 us): the road-like 2048 x 2048 mesh takes 8.6
// ms for 371 steps, and took 11.8 with a second sweep that published the updates.
// A node at distance 0 (a center, or assigned) takes no offer: its key alone
// counts, and the arrays hold nothing for it (one is R, by center).
__device__ __forceinline__ uint64_t step_state(uint64_t key, uint64_t pend) {
  return key >> 32 && pend < key ? pend : key;
}

// Applies the offers of a step (state[i]: of v[i] before the step) and counts
// the nodes that it updates and covers: the thread that puts a node on the
// frontier counts it.
template <int K>
__device__ __forceinline__ void improve_sync(Run &r, const bool (&better)[K], const int32_t (&v)[K],
                                             const uint64_t (&cand)[K], const uint64_t (&state)[K]) {
  uint64_t old[K];
#pragma unroll
  for (int i = 0; i < K; ++i) {
    old[i] = ~0ull;
    if (better[i]) {
      atomicMin((unsigned long long *)&r.pnew[v[i]], (unsigned long long)cand[i]);
      old[i] = atomicOr((unsigned long long *)&r.nxt[v[i] >> 6], 1ull << (v[i] & 63));
    }
  }
#pragma unroll
  for (int i = 0; i < K; ++i) {
    const bool first = !(old[i] >> (v[i] & 63) & 1);
    r.updated += first;
    r.covered += first && state[i] == CLD_INF64;
  }
}

// K arcs of u's row (key ku; in[i]: part of the row): the light ones
// (w <= lim) are offered, the first heavy one ends the scan.  Returns the
// number of light arcs; *blocked is set if a heavy one is among them.
template <bool kSync, int K>
__device__ __forceinline__ uint32_t offer(Run &r, uint64_t ku, uint32_t lim, const bool (&in)[K],
                                          const uint64_t (&arc)[K], bool *blocked) {
  bool better[K];
  int32_t v[K];
  uint64_t cand[K];
  uint32_t light = 0;
#pragma unroll
  for (int i = 0; i < K; ++i) {
    const bool ok = in[i] && (uint32_t)(arc[i] >> 32) <= lim;
    if (in[i] && !ok) *blocked = true;
    light += ok;
    v[i] = ok ? (int32_t)(uint32_t)arc[i] : 0;
    cand[i] = ku + (arc[i] & 0xffffffff00000000ull);
    better[i] = ok;
  }
  uint64_t k[K];
#pragma unroll
  for (int i = 0; i < K; ++i) k[i] = r.key[v[i]];
  if (kSync) {
    uint64_t p[K];
#pragma unroll
    for (int i = 0; i < K; ++i) p[i] = r.pend[v[i]];
#pragma unroll
    for (int i = 0; i < K; ++i) k[i] = step_state(k[i], p[i]);
  }
#pragma unroll
  for (int i = 0; i < K; ++i) better[i] = better[i] && (kSync ? (cand[i] >> 32) < (k[i] >> 32) : cand[i] < k[i]);
  if (kSync) improve_sync<K>(r, better, v, cand, k);
  else improve<K>(r, better, v, cand);
  return light;
}

// Queues a long row for the cooperative passes that end this pass; false when
// the queue is full (the caller then handles the row itself).
__device__ __forceinline__ bool defer_row(Run &r, int32_t u, int32_t deg) {
  if (deg > r.d.big_deg) {
    const uint32_t slot = atomicAdd(&r.S.big_cnt[r.pass & 1], 1u);
    if (slot < kBigCap) { r.S.big[slot] = u; return true; }
  } else {
    const uint32_t slot = atomicAdd(&r.S.mid_cnt[r.pass & 1], 1u);
    if (slot < kMidCap) { r.S.mid[slot] = u; return true; }
  }
  return false;
}

// Rows are relaxed by kRowLanes lanes together, one arc each at a time.  A
// local round of a few dozen nodes, the usual case on meshes, takes 2 to 3 us
// of latency and of one wave's instructions, which this cuts to a quarter of
// those of one lane per row with four arcs in flight (CLUSTER2 on the road-like
// 2048 x 2048 mesh 9.4 instead of 13.0 ms, 1153 x 1021 mesh 1.40 instead of
// 1.87, R-MAT scale 18 1.11 instead of 1.27).  Eight lanes leave half of them
// idle on meshes (10.9 and 1.68 ms) and gain 5% on R-MAT scale 24.  All lanes of
// a group have the same arguments.
//
// Loads in flight together are not under branches of their own (lanes without
// an arc or a node read some other): the compiler waits for a load before it
// leaves the branch, which had four far keys follow one another.
constexpr int kRowLanes = 4;
__device__ __forceinline__ uint32_t row_lane() { return threadIdx.x & (kRowLanes - 1); }
__device__ __forceinline__ uint32_t group_sum(uint32_t x) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xb1, 0xf, 0xf, true);   // lanes [1, 0, 3, 2]
  return x + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4e, 0xf, 0xf, true);   // [2, 3, 0, 1]
}

// Relaxes u with key ku; long rows are deferred.
template <bool kSync>
__device__ __forceinline__ void relax_row(Run &r, int32_t u, uint64_t ku, int64_t a0, int32_t deg) {
  if (deg > r.d.mid_deg) {
    uint32_t deferred = 0;
    if (row_lane() == 0) deferred = defer_row(r, u, deg);
    if (group_sum(deferred)) return;
  }
  const uint64_t word = marks_of(r, u);
  const uint64_t *row = r.d.arcs + a0;
  const uint32_t lim = r.delta - (uint32_t)(ku >> 32);
  uint32_t light = 0, heavy = 0;
  for (int32_t base = 0; base < deg && !heavy; base += kRowLanes) {
    const int32_t a = base + (int32_t)row_lane();
    const bool in[1] = {a < deg};
    const uint64_t arc[1] = {row[in[0] ? a : base]};
    bool blocked = false;
    light += offer<kSync, 1>(r, ku, lim, in, arc, &blocked);
    heavy = group_sum(blocked);
  }
  r.scanned += light;
  if (heavy) {
    light = group_sum(light);
    if (row_lane() == 0) mark_blocked(r, u, word, deg - (int32_t)light);
  }
}

// A frontier node.
template <bool kSync>
__device__ __forceinline__ void relax_item(Run &r, int32_t u) {
  uint64_t ku = r.key[u];
  const int64_t a0 = r.d.row_ptr[u];
  const int32_t deg = (int32_t)(r.d.row_ptr[u + 1] - a0);   // indices within a row are 32-bit
  if (kSync) {
    const uint64_t now = step_state(ku, r.pend[u]);
    if (now != ku && row_lane() == 0) r.key[u] = now;
    ku = now;
  }
  const uint32_t dist = (uint32_t)(ku >> 32);
  // beyond the current distance bucket: stays for a later sweep
  if (!kSync && (dist >= r.theta || (deg > r.d.mid_deg && dist >= r.theta_row))) {
    if (row_lane() == 0) leave(r, u, dist);
  } else {
    relax_row<kSync>(r, u, ku, a0, deg);
  }
}

// A queued improvement.
__device__ __forceinline__ void relax_queued(Run &r, int32_t u, uint64_t ku) {
  const uint64_t now = r.key[u];
  const int64_t a0 = r.d.row_ptr[u];
  const int32_t deg = (int32_t)(r.d.row_ptr[u + 1] - a0);
  if (now < ku) return;   // improved again since: another entry's business
  const uint32_t dist = (uint32_t)(ku >> 32);
  if (deg > r.d.mid_deg && dist >= r.theta_row) {
    if (row_lane() == 0) leave(r, u, dist);
  } else {
    relax_row<false>(r, u, ku, a0, deg);
  }
}

// NEXT for a short row: smallest d_u + w over its heavy arcs (w > Delta - d_u)
// into unreached nodes.  Rows are sorted by weight, so the first such arc in
// ascending order gives the minimum.
__device__ __forceinline__ uint64_t next_small(const Run &r, uint64_t ku, int64_t a0, int32_t deg) {
  const uint32_t du = (uint32_t)(ku >> 32), lim = r.delta - du;
  const uint64_t *row = r.d.arcs + a0;
  for (int32_t base = 0; base < deg; base += kScanBatch) {
    uint64_t arc[kScanBatch];
    bool hit[kScanBatch];
#pragma unroll
    for (int i = 0; i < kScanBatch; ++i) arc[i] = row[base + i < deg ? base + i : base];
    uint64_t k[kScanBatch];
#pragma unroll
    for (int i = 0; i < kScanBatch; ++i) hit[i] = (uint32_t)(arc[i] >> 32) > lim;
#pragma unroll
    for (int i = 0; i < kScanBatch; ++i) k[i] = r.key[hit[i] ? (int32_t)(uint32_t)arc[i] : 0];
#pragma unroll
    for (int i = 0; i < kScanBatch; ++i) hit[i] = hit[i] && k[i] == CLD_INF64;
#pragma unroll
    for (int i = 0; i < kScanBatch; ++i)
      if (hit[i]) return (uint64_t)du + (arc[i] >> 32);
  }
  return CLD_INF64;
}

// Long rows remember their last scan (key and light limit).  Within a Delta
// level a node's key only decreases and Delta is fixed, so a record with the
// node's current key means that every arc up to the recorded limit has
// already been offered with this key; once a level is at its fixpoint the
// reached nodes' keys are final, so a larger Delta only has to look past the
// recorded limit; and after a stage the arcs up to it lead to assigned nodes.
// A record read in a race is never larger than what some scan with an equal
// or better key has covered, so skipping up to it drops no useful offer.
// First arc in [lo, hi) of a weight-sorted row with w > x, found by the 64
// lanes of a wave together: each round samples 64 evenly spaced arcs and
// keeps the bracket of the first one above x (two or three dependent loads
// for rows up to 8192 arcs instead of a dozen for a binary search).  Every
// lane of the wave calls it with the same arguments and gets the result.
__device__ __forceinline__ int32_t wave_first_above(const uint64_t *arcs, int32_t lo, int32_t hi, uint32_t x) {
  const int32_t lane = (int32_t)(threadIdx.x & 63);
  while (hi - lo > 64) {
    const int32_t step = (hi - lo + 63) >> 6;
    const int32_t p = lo + lane * step;
    const bool above = p < hi && (uint32_t)(arcs[p] >> 32) > x;
    const unsigned long long m = __ballot(above);
    if (m == 0) {
      // every valid sample is <= x: the answer lies after the last one
      const int32_t last = lo + ((hi - 1 - lo) / step) * step;
      lo = last + 1;
    } else {
      const int32_t f = __ffsll((long long)m) - 1;
      const int32_t nlo = f == 0 ? lo : lo + (f - 1) * step + 1;
      hi = lo + f * step;   // the sample at f is above x
      lo = nlo;
      if (f == 0) return hi;
    }
  }
  const int32_t p = lo + lane;
  const unsigned long long m = __ballot(p < hi && (uint32_t)(arcs[p] >> 32) > x);
  return m ? lo + (__ffsll((long long)m) - 1) : hi;
}

// Resume index within the row [0, end) of u (arcs at row).
__device__ __forceinline__ int32_t resume_at_wave(const Run &r, int32_t u, uint64_t ku, const uint64_t *row,
                                                  int32_t end) {
  if (r.keyn[u] != ku) return 0;
  return wave_first_above(row, 0, end, r.slim[u]);
}

__device__ __forceinline__ void note_scan(Run &r, int32_t u, uint64_t ku, uint32_t lim) {
  r.slim[u] = lim;
  r.keyn[u] = ku;
  r.S.sum.records = 1;
}

// Ends a pass: the rows that it deferred, each wave taking whole mid-size
// rows (64 lanes x kArcBatch arcs per step), then the whole workgroup each big
// row.  The deferral counters alternate between passes, so a wave that is late
// to read this pass's sees none of the next pass's rows and every wave takes
// the same branch after the one barrier.  `mid` handles a row in a wave, `big`
// one in the workgroup (called by every thread, with a barrier behind it).
template <class Mid, class Big>
__device__ __forceinline__ void coop_rows(Run &r, Mid mid, Big big) {
  __syncthreads();
  Stage &S = r.S;
  const uint32_t p = r.pass++ & 1;
  const uint32_t nm = S.mid_cnt[p] < kMidCap ? S.mid_cnt[p] : kMidCap;
  const uint32_t nb = S.big_cnt[p] < kBigCap ? S.big_cnt[p] : kBigCap;
  if (nm == 0 && nb == 0) return;
  for (uint32_t i = threadIdx.x >> 6; i < nm; i += kWaves) {
    const int32_t u = S.mid[i];
    const int64_t a0 = r.d.row_ptr[u];
    mid(u, r.d.arcs + a0, (int32_t)(r.d.row_ptr[u + 1] - a0));
  }
  for (uint32_t h = 0; h < nb; ++h) {
    const int32_t u = S.big[h];
    const int64_t a0 = r.d.row_ptr[u];
    big(u, r.d.arcs + a0, (int32_t)(r.d.row_ptr[u + 1] - a0));
    __syncthreads();
  }
  __syncthreads();
  if (threadIdx.x == 0) { S.mid_cnt[p] = 0; S.big_cnt[p] = 0; }
  __syncthreads();
}

template <bool kSync>
__device__ __forceinline__ void relax_long(Run &r) {
  const int32_t lane = (int32_t)(threadIdx.x & 63), tid = (int32_t)threadIdx.x;
  auto mid = [&](int32_t u, const uint64_t *row, int32_t deg) {
    const uint64_t word = marks_of(r, u), ku = kSync ? step_state(r.key[u], r.pend[u]) : r.key[u];
    const uint32_t lim = r.delta - (uint32_t)(ku >> 32);
    const int32_t start = r.resume ? resume_at_wave(r, u, ku, row, deg) : 0;
    int32_t end = start;   // of the light prefix
    bool any = false;
    for (int32_t base = start; base < deg && !any; base += 64 * kArcBatch) {
      uint64_t arc[kArcBatch];
      bool in[kArcBatch], blocked = false;
#pragma unroll
      for (int i = 0; i < kArcBatch; ++i) {
        const int32_t a = base + 64 * i + lane;
        in[i] = a < deg;
        arc[i] = row[in[i] ? a : deg - 1];
      }
      uint32_t light = offer<kSync, kArcBatch>(r, ku, lim, in, arc, &blocked);
      r.scanned += light;
      any = __any(blocked);
      for (int o = 32; o >= 1; o >>= 1) light += __shfl_xor(light, o);
      end += (int32_t)light;
    }
    if (lane == 0) {
      if (any) mark_blocked(r, u, word, deg - end);
      if (r.resume) note_scan(r, u, ku, lim);
    }
  };
  auto big = [&](int32_t u, const uint64_t *row, int32_t deg) {
    // wave 0 reads u's key once for the whole workgroup (so every thread scans
    // with the same key and the scan record describes all of them) and finds
    // the end of the light prefix and the resume point
    if (threadIdx.x < 64) {
      const uint64_t k = kSync ? step_state(r.key[u], r.pend[u]) : r.key[u];
      const int32_t light_end = wave_first_above(row, 0, deg, r.delta - (uint32_t)(k >> 32));
      const int32_t from = r.resume ? resume_at_wave(r, u, k, row, light_end) : 0;
      if (threadIdx.x == 0) {
        r.S.row_key = k;
        r.S.row_lo = light_end;
        r.S.row_start = from;
      }
    }
    __syncthreads();
    const uint64_t ku = r.S.row_key;
    const uint32_t lim = r.delta - (uint32_t)(ku >> 32);
    const int32_t lo = r.S.row_lo;
    for (int32_t base = r.S.row_start; base < lo; base += kSweepThreads * kArcBatch) {
      uint64_t arc[kArcBatch];
      bool in[kArcBatch], blocked = false;
#pragma unroll
      for (int i = 0; i < kArcBatch; ++i) {
        const int32_t a = base + kSweepThreads * i + tid;
        in[i] = a < lo;
        arc[i] = row[in[i] ? a : lo - 1];
      }
      r.scanned += offer<kSync, kArcBatch>(r, ku, lim, in, arc, &blocked);
    }
    if (threadIdx.x == 0 && lo < deg) mark_blocked(r, u, marks_of(r, u), deg - lo);
    __syncthreads();
    // every thread's part of the row is done: record the scan
    if (r.resume && threadIdx.x == 0) note_scan(r, u, ku, lim);
  };
  coop_rows(r, mid, big);
}

// NEXT: u keeps its place on the frontier (unless the steps are synchronous,
// whose blocked set stays whole) and its reach counts.
__device__ __forceinline__ void next_hit(Run &r, int32_t u, uint64_t reach) {
  if (reach < r.acc) r.acc = reach;
  if (r.d.variant != CLDIAM_VARIANT_STEPS) set_bit(r.cur, u);
}

__device__ __forceinline__ void next_long(Run &r) {
  const int32_t lane = (int32_t)(threadIdx.x & 63);
  auto mid = [&](int32_t u, const uint64_t *row, int32_t deg) {
    const uint32_t du = (uint32_t)(r.key[u] >> 32), lim = r.delta - du;
    // the heavy arcs start after the light prefix
    for (int32_t base = wave_first_above(row, 0, deg, lim); base < deg; base += 64) {
      const int32_t a = base + lane;
      const uint64_t arc = a < deg ? row[a] : 0ull;
      const bool hit = a < deg && (uint32_t)(arc >> 32) > lim && r.key[(int32_t)(uint32_t)arc] == CLD_INF64;
      const unsigned long long m = __ballot(hit);
      if (m) {
        // first hit in ascending order has the smallest weight
        if (lane == __ffsll((long long)m) - 1) next_hit(r, u, (uint64_t)du + (arc >> 32));
        break;
      }
    }
  };
  auto big = [&](int32_t u, const uint64_t *row, int32_t deg) {
    Stage &S = r.S;
    const uint32_t du = (uint32_t)(r.key[u] >> 32);
    if (threadIdx.x < 64) {
      const int32_t lo = wave_first_above(row, 0, deg, r.delta - du);
      if (threadIdx.x == 0) { S.row_lo = lo; S.blk_min = CLD_INF64; }
    }
    __syncthreads();
    for (int32_t base = S.row_lo; base < deg; base += kSweepThreads) {
      const int32_t a = base + (int32_t)threadIdx.x;
      if (a < deg) {
        const uint64_t arc = row[a];
        if (r.key[(int32_t)(uint32_t)arc] == CLD_INF64)
          atomicMin(&S.blk_min, (unsigned long long)((uint64_t)du + (arc >> 32)));
      }
      __syncthreads();
      const bool found = S.blk_min != CLD_INF64;
      __syncthreads();
      if (found) break;
    }
    if (threadIdx.x == 0 && S.blk_min != CLD_INF64) next_hit(r, u, S.blk_min);
  };
  coop_rows(r, mid, big);
}

// Pull mode.  Offers over arcs that were heavy at the previous Delta, or
// from the sources of a new stage, can only reach unreached nodes: they are
// at least the previous Delta, above every reached key.  When the unreached
// nodes are fewer than the blocked ones, they look at their neighbours
// instead: PULL gives an unreached node v the lexicographic minimum over its
// neighbours u with a key of (d_u + w, c_u), d_u + w <= Delta (only v's own
// thread writes v's key, so no atomic is needed); NEXT_PULL folds the smallest
// d_u + w over the same arcs.  Rows are sorted by weight, so both stop early
// (pull_more).  A pass that changed many nodes is followed by another, in which
// the reached nodes look for smaller offers as well.  Every node then has the
// minimum over what its neighbours had after the pass before, so only the nodes
// changed by the last pass have offers left to make and are the frontier.
// One thread per row: four lanes, as in relaxation, took 5% longer.
// A key read while its node is being pulled in the same pass is a real path
// too, so taking it only moves the fixpoint closer.

// Whether an arc of weight w, in a row sorted by weight, can still beat the
// best offer: every offer over it is at least w (d_u >= 0), so PULL stops
// past min(Delta, best distance) (an equal distance may still win on the
// center id) and NEXT_PULL once w reaches the best distance.
__device__ __forceinline__ bool pull_more(uint64_t w, uint64_t best, uint32_t delta, bool next) {
  return next ? w < best : (w <= delta && w <= (best >> 32));
}

// Value (pull) or distance (next) that a neighbour with key k offers to an
// unreached node over an arc of weight w.
__device__ __forceinline__ uint64_t pull_offer(const Run &r, uint64_t w, uint64_t k, bool next) {
  if (k == CLD_INF64) return CLD_INF64;
  const uint64_t du = k >> 32;
  if (next) return du + w;
  return du + w <= r.delta ? k + (w << 32) : CLD_INF64;
}

// now: v's key before.
__device__ __forceinline__ void pull_apply(Run &r, int32_t v, uint64_t now, uint64_t best, bool next) {
  if (next) {
    if (best < r.acc) r.acc = best;
  } else if (best < now) {
    r.key[v] = best;
    set_bit(r.cur, v);
    ++r.updated;
    if ((uint32_t)(best >> 32) < r.fmin) r.fmin = (uint32_t)(best >> 32);
  }
}

// One uncovered node (in a level's first pass an unreached one), its row scanned by this thread (long rows are deferred).
__device__ __forceinline__ void pull_item(Run &r, int32_t v, bool next) {
  const uint64_t now = r.key[v];
  const int64_t a0 = r.d.row_ptr[v];
  const int32_t deg = (int32_t)(r.d.row_ptr[v + 1] - a0);
  if (now != CLD_INF64 && (next || r.s.again == 0)) return;
  if (deg > (now != CLD_INF64 ? kPullRow : r.d.mid_deg) && defer_row(r, v, deg)) return;
  const uint64_t *row = r.d.arcs + a0;
  uint64_t best = now;
  for (int32_t base = 0; base < deg; base += kScanBatch) {
    uint64_t arc[kScanBatch];
    bool ok[kScanBatch];
    bool stop = false;
#pragma unroll
    for (int j = 0; j < kScanBatch; ++j) arc[j] = row[base + j < deg ? base + j : base];
#pragma unroll
    for (int j = 0; j < kScanBatch; ++j) {
      const uint64_t w = arc[j] >> 32;
      ok[j] = base + j < deg && pull_more(w, best, r.delta, next);
      if (base + j < deg && !ok[j]) stop = true;
    }
    uint64_t k[kScanBatch];
#pragma unroll
    for (int j = 0; j < kScanBatch; ++j) k[j] = r.key[ok[j] ? (int32_t)(uint32_t)arc[j] : v];
#pragma unroll
    for (int j = 0; j < kScanBatch; ++j) {
      const uint64_t c = ok[j] ? pull_offer(r, arc[j] >> 32, k[j], next) : CLD_INF64;
      best = c < best ? c : best;
    }
    if (stop) break;
  }
  pull_apply(r, v, now, best, next);
}

__device__ __forceinline__ uint64_t wave_min_all(uint64_t x) {
  for (int o = 32; o >= 1; o >>= 1) {
    const uint64_t y = __shfl_xor(x, o);
    x = y < x ? y : x;
  }
  return x;
}

// The long rows deferred by pull_item: a wave per row, then the whole
// workgroup per hub row.
__device__ __forceinline__ void pull_long(Run &r, bool next) {
  const int32_t lane = (int32_t)(threadIdx.x & 63);
  auto mid = [&](int32_t v, const uint64_t *row, int32_t deg) {
    const uint64_t now = r.key[v];
    uint64_t best = now;
    for (int32_t base = 0; base < deg; base += 64) {
      const int32_t a = base + lane;
      const uint64_t arc = a < deg ? row[a] : ~0ull;
      const bool in = a < deg && pull_more(arc >> 32, best, r.delta, next);
      if (!__any(in)) break;
      const uint64_t c = in ? pull_offer(r, arc >> 32, r.key[(int32_t)(uint32_t)arc], next) : CLD_INF64;
      if (__any(c < best)) best = wave_min_all(c < best ? c : best);
    }
    if (lane == 0) pull_apply(r, v, now, best, next);
  };
  auto big = [&](int32_t v, const uint64_t *row, int32_t deg) {
    Stage &S = r.S;
    const uint64_t now = r.key[v];   // read before thread 0 writes it: every thread passes the barriers below first
    if (threadIdx.x == 0) S.blk_min = now;
    __syncthreads();
    for (int32_t base = 0; base < deg; base += kSweepThreads) {
      const uint64_t cur = S.blk_min;   // the same for every thread: nothing changes it between the barriers
      const int32_t a = base + (int32_t)threadIdx.x;
      __syncthreads();
      if (a < deg) {
        const uint64_t arc = row[a];
        if (pull_more(arc >> 32, cur, r.delta, next)) {
          const uint64_t c = pull_offer(r, arc >> 32, r.key[(int32_t)(uint32_t)arc], next);
          if (c < cur) atomicMin(&S.blk_min, (unsigned long long)c);
        }
      }
      __syncthreads();
      const int32_t nxt = base + kSweepThreads;
      const bool stop = nxt >= deg || !pull_more(row[nxt] >> 32, S.blk_min, r.delta, next);
      if (stop) break;
    }
    if (threadIdx.x == 0) pull_apply(r, v, now, S.blk_min, next);
  };
  coop_rows(r, mid, big);
}

// CLUSTER2, Contract2: u was assigned last iteration at growth distance dl
// (kept in keyn) with label c; every edge with Delta2 - dl < w <= Delta2 is
// the rescaled edge (c, v) of weight dl + w - Delta2.  Rows are sorted by
// weight, so those arcs are one contiguous range.
__device__ __forceinline__ void c2_boundary(Run &r, int32_t u) {
  const uint32_t delta2 = r.delta;
  const uint32_t dl = (uint32_t)r.keyn[u];
  const uint64_t label = r.key[u] & 0xffffffffull;
  const int64_t a0 = r.d.row_ptr[u];
  const int32_t a1 = (int32_t)(r.d.row_ptr[u + 1] - a0);
  const uint64_t *row = r.d.arcs + a0;
  int32_t lo = 0, hi = a1;
  while (lo < hi) {   // first arc with w > delta2 - dl
    const int32_t mid = lo + ((hi - lo) >> 1);
    if ((uint32_t)(row[mid] >> 32) <= delta2 - dl) lo = mid + 1; else hi = mid;
  }
  for (int32_t a = lo; a < a1; ++a) {
    const uint64_t arc = row[a];
    const uint32_t w = (uint32_t)(arc >> 32);
    if (w > delta2) break;
    ++r.scanned;
    const int32_t v = (int32_t)(uint32_t)arc;
    const uint64_t cand = ((uint64_t)(dl + w - delta2) << 32) | label;
    if (cand < r.key[v]) {
      atomicMin((unsigned long long *)&r.key[v], (unsigned long long)cand);
      set_bit(r.cur, v);
    }
  }
}

// Walks the nodes of a set in words [lo, hi), kSweepThreads nodes per pass in
// ascending order.  word(w) gives word w (and may clear it: it is called once
// per word, by the workgroup that owns it); item(v) handles a node and end()
// the pass's end (every thread, with a barrier inside).  Dense words are
// spread by their wave together, sparse ones each by its own thread.
template <int kLanes = 1, class Word, class Item, class End>
__device__ __forceinline__ void list_pass(Run &r, uint32_t lo, uint32_t hi, Word word, Item item, End end) {
  Stage &S = r.S;
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint64_t ahead = lo + tid < hi ? word(lo + tid) : 0ull;
  uint32_t window = 0;
  for (uint32_t w0 = lo; w0 < hi; w0 += kSweepThreads) {
    const uint64_t mine = ahead;
    const uint32_t w = w0 + tid;
    ahead = w + kSweepThreads < hi ? word(w + kSweepThreads) : 0ull;
    const uint32_t count = (uint32_t)__popcll(mine);
    const uint32_t incl = cld_wave_scan_u32(count);
    uint32_t *wsum = S.wsum[window++ & 1];   // the window before may still be read
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    const uint32_t ws = lane < (uint32_t)kWaves ? wsum[lane] : 0u, wincl = cld_wave_scan_u32(ws);
    const uint32_t total = cld_last_lane(wincl);
    const uint32_t at = incl - count + (uint32_t)__shfl(wincl - ws, (int)wave);
    const bool dense = __any(count > 8);
    for (uint32_t r0 = 0; r0 < total; r0 += kList) {
      if (dense) {
        for (uint64_t left = __ballot(count != 0 && at + count > r0 && at < r0 + kList); left; left &= left - 1) {
          const int k = __ffsll((long long)left) - 1;
          const uint64_t x = __shfl(mine, k);
          const uint32_t p = __shfl(at, k) + (uint32_t)__popcll(x & ((1ull << lane) - 1ull)) - r0;
          if ((x >> lane & 1) && p < kList) S.list[p] = (int32_t)(((w0 + wave * 64 + k) << 6) + lane);
        }
      } else {
        uint32_t p = at - r0;
        for (uint64_t x = mine; x; x &= x - 1, ++p)
          if (p < kList) S.list[p] = (int32_t)((w << 6) + (uint32_t)__ffsll((long long)x) - 1);
      }
      __syncthreads();
      const uint32_t n = total - r0 < kList ? total - r0 : kList;
      for (uint32_t i0 = 0; i0 < n; i0 += kSweepThreads) {
        for (uint32_t i = i0 + tid / kLanes; i < n && i < i0 + kSweepThreads; i += kSweepThreads / kLanes) item(S.list[i]);
        end();
      }
      __syncthreads();
    }
  }
}

// Walks the nodes of a set in words [lo, hi) wave by wave, kNodeWords words of
// 64 nodes at a time: load(v) for every node (their loads overlap), then, word
// by word, use(w, v, in, x) by the whole wave (in: v is in the set, x: its
// load).  The wave owns the words.
constexpr int kNodeWords = 8;

template <class Load, class Use>
__device__ __forceinline__ void node_pass(const Run &r, const uint64_t *bits, uint32_t lo, uint32_t hi, Load load, Use use) {
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (uint32_t base = lo + wave * kNodeWords; base < hi; base += kWaves * kNodeWords) {
    const uint64_t mine = lane < (uint32_t)kNodeWords && base + lane < hi ? bits[base + lane] & own_bits(r, base + lane) : 0ull;
    const uint64_t filled = __ballot(mine != 0);
    if (filled == 0) continue;
    const int at = __ffsll((long long)filled) - 1;   // a word with members, and its first
    const int32_t some = (int32_t)(((base + at) << 6) + (uint32_t)__ffsll((long long)__shfl(mine, at)) - 1u);
    uint64_t word[kNodeWords], x[kNodeWords];
    int32_t any[kNodeWords];
#pragma unroll
    for (int j = 0; j < kNodeWords; ++j) {
      word[j] = __shfl(mine, j);
      const bool in = word[j] >> lane & 1;
      // one load whether in or not (a branch around it would wait for the
      // load before): lanes outside the set read a member's
      const uint32_t other = word[j] ? (uint32_t)__ffsll((long long)word[j]) - 1u : lane;
      any[j] = (int32_t)(((base + j) << 6) + (in ? lane : other));
      if (!word[j]) any[j] = some;
    }
#pragma unroll
    for (int j = 0; j < kNodeWords; ++j) x[j] = load(any[j]);
#pragma unroll
    for (int j = 0; j < kNodeWords; ++j)
      if (word[j]) use(base + j, (int32_t)(((base + j) << 6) + lane), (bool)(word[j] >> lane & 1), x[j]);
  }
}

// A covered node's D, for the workgroup's table of cluster maxima: a stage has
// few clusters, so fold in LDS first (the slot of c, once claimed by c), in
// global memory when another center holds the slot.
__device__ __forceinline__ void fold_rmax(Run &r, uint64_t *R, uint32_t c, uint64_t Dv) {
  Stage &S = r.S;
  const uint32_t slot = (c * 2654435761u) >> 22;   // 10 bits: kRmaxSlots
  uint32_t t = S.rmax.tag[slot];
  if (t == kRmaxFree) {
    t = atomicCAS(&S.rmax.tag[slot], kRmaxFree, c);
    if (t == kRmaxFree) t = c;
  }
  if (t == c) {
    if (Dv > S.rmax.mx[slot]) atomicMax(&S.rmax.mx[slot], (unsigned long long)Dv);
  } else if (Dv > R[c]) {
    atomicMax((unsigned long long *)&R[c], (unsigned long long)Dv);
  }
}

// Bitmap words [lo, hi) of graph g, or its nodes [na, nb) there.
__device__ __forceinline__ void process_run(const Job &job, const GDesc &d, const GState &s, GCount &cn, uint32_t *idle, uint32_t lo,
                            uint32_t hi, uint32_t na, uint32_t nb, Stage &S) {
  const uint32_t phase = s.phase, stage = s.stage, lane = threadIdx.x & 63;
  const uint32_t woff = (uint32_t)(d.off >> 6);
  const bool steps = d.variant == CLDIAM_VARIANT_STEPS;
  uint64_t *U = job.U + woff, *R = job.R + d.off;
  uint64_t *F = job.F + woff, *blk = F + s.blk * job.fwords, *alt = F + s.alt * job.fwords;
  const uint32_t row_lim = row_limit(d, s.delta, s.row_base);
  const bool odd = s.rounds & 1;
  Run r{job, d, s, S, job.key + d.off, job.keyn + d.off, job.slim + d.off,
        odd ? R : job.keyn + d.off, odd ? job.keyn + d.off : R, F + s.cur * job.fwords,
        F + s.nxt * job.fwords, s.pull ? nullptr : (s.merge ? alt : blk), s.delta, s.theta, row_lim < s.theta ? row_lim : s.theta,
        !steps && !s.c2, na, nb};
  if (threadIdx.x == 0) {
    clear_count(S.sum);
    S.qn[0] = S.qn[1] = S.qn[2] = 0;
    S.mid_cnt[0] = S.mid_cnt[1] = S.big_cnt[0] = S.big_cnt[1] = 0;
    S.stop = 0;
  }
  const bool table = phase == PH_RMAX || (phase == PH_ASSIGN && stage == 0);
  if (table) {
    for (uint32_t t = threadIdx.x; t < kRmaxSlots; t += kSweepThreads) {
      S.rmax.tag[t] = kRmaxFree;
      S.rmax.mx[t] = 0;
    }
  }
  __syncthreads();
  uint32_t cov = 0;   // per wave: nodes counted
  const auto no_load = [](int32_t) { return 0ull; };
  const auto key_of = [&](int32_t v) { return r.key[v]; };
  const auto no_end = [] {};
  switch (phase) {
    case PH_SELECT:
    case PH_C2_SELECT: {
      const bool c2 = phase == PH_C2_SELECT;
      if (s.pull && stage > 0) {   // pull mode has no pushing sources
        for (uint32_t w = lo + threadIdx.x; w < hi; w += kSweepThreads)
          if (r.cur[w]) r.cur[w] = 0;
        __syncthreads();
      }
      if (!c2 && stage == 0 && lo == 0 && s.cuts != 0)
        for (uint32_t i = threadIdx.x; i <= s.cuts; i += kSweepThreads) job.cut[2 * (d.off >> 6) + i] = cut_at(d, i, s.cuts);
      const bool hubs = !c2 && stage == 0 && d.pull_mode == CLDIAM_PULL_AUTO;
      node_pass(r, U, lo, hi,
                [&](int32_t v) { return hubs ? (uint64_t)(d.row_ptr[v + 1] - d.row_ptr[v]) : 0ull; },
                [&](uint32_t w, int32_t v, bool in, uint64_t deg) {
        if (in && deg > d.hub_deg) r.acc += deg;
        const uint32_t x0 = cld_philox_word0((uint32_t)v, c2 ? stage + 1 : stage, 0u, c2 ? 1u : 0u, (uint32_t)d.seed,
                                             (uint32_t)(d.seed >> 32));
        const bool sel = in && (uint64_t)x0 < s.T;
        if (sel) {
          r.key[v] = (uint64_t)(uint32_t)v;
          R[v] = c2 ? stage + 1 : 0;
        }
        const uint64_t m = __ballot(sel);
        if (m && lane == 0) atomicOr((unsigned long long *)&r.cur[w], (unsigned long long)m);
        cov += (uint32_t)__popcll(m);
      });
      if (c2)
        list_pass(r, lo, hi,
                  [&](uint32_t w) { return take_bits(r, blk, w); },
                  [&](int32_t u) { c2_boundary(r, u); }, no_end);
      break;
    }
    case PH_RELAX:
      if (steps) {
        const bool merge = s.merge != 0;
        list_pass<kRowLanes>(r, lo, hi,
                  [&](uint32_t w) {
                    uint64_t x = take_bits(r, r.cur, w);
                    if (merge) x |= take_bits(r, blk, w);
                    return x;
                  },
                  [&](int32_t u) { relax_item<true>(r, u); }, [&] { relax_long<true>(r); });
      } else {
        list_pass<kRowLanes>(r, lo, hi, [&](uint32_t w) { return take_bits(r, r.cur, w); },
                  [&](int32_t u) { relax_item<false>(r, u); }, [&] { relax_long<false>(r); });
      }
      break;
    case PH_COMMIT:
      node_pass(r, r.cur, lo, hi, key_of, [&](uint32_t, int32_t v, bool in, uint64_t k) {
        if (in) r.key[v] = step_state(k, r.pend[v]);
      });
      break;
    case PH_COUNT:
      node_pass(r, U, lo, hi, key_of, [&](uint32_t, int32_t, bool in, uint64_t k) {
        cov += (uint32_t)__popcll(__ballot(in && k != CLD_INF64));
      });
      break;
    case PH_NEXT:
      r.acc = CLD_INF64;
      if (!steps)
        node_pass(r, U, lo, hi, key_of, [&](uint32_t, int32_t, bool in, uint64_t k) {
          cov += (uint32_t)__popcll(__ballot(in && k != CLD_INF64));
        });
      list_pass(r, lo, hi,
                [&](uint32_t w) { return steps ? blk[w] & own_bits(r, w) : take_bits(r, blk, w); },
                [&](int32_t u) {
                  const uint64_t ku = r.key[u];
                  const int64_t a0 = d.row_ptr[u];
                  const int32_t deg = (int32_t)(d.row_ptr[u + 1] - a0);
                  if (deg > d.mid_deg && defer_row(r, u, deg)) return;
                  const uint64_t reach = next_small(r, ku, a0, deg);
                  if (reach != CLD_INF64) next_hit(r, u, reach);
                },
                [&] { next_long(r); });
      break;
    case PH_PULL:
    case PH_NEXT_PULL: {
      const bool next = phase == PH_NEXT_PULL;
      if (next) r.acc = CLD_INF64;
      for (uint32_t w = lo + threadIdx.x; w < hi; w += kSweepThreads) {
        if (blk[w]) drop_bits(r, blk, w);   // left from before the switch to pull mode
        if (s.again && !next && r.cur[w]) drop_bits(r, r.cur, w);   // every node looks at the changes of the pass before
      }
      __syncthreads();
      list_pass(r, lo, hi, [&](uint32_t w) { return U[w] & own_bits(r, w); }, [&](int32_t v) { pull_item(r, v, next); },
                [&] { pull_long(r, next); });
      break;
    }
    case PH_ASSIGN:
      // D = growth distance + the cluster's radius before this stage (0 in the
      // first, whose pass therefore folds the new radii and takes the covered
      // nodes off the uncovered set as well)
      node_pass(r, U, lo, hi, key_of, [&](uint32_t w, int32_t v, bool in, uint64_t k) {
        const bool got = in && k != CLD_INF64;
        if (got) {
          const uint32_t c = (uint32_t)k;
          const uint64_t Dv = (k >> 32) + (stage > 0 ? R[c] : 0ull);
          d.cluster[v] = (int32_t)c;
          d.D[v] = Dv;
          if (Dv > r.acc) r.acc = Dv;
          if (stage == 0) {
            fold_rmax(r, R, c, Dv);
            r.key[v] = (uint64_t)c;
            if (s.records) r.keyn[v] = (uint64_t)c;
          }
        }
        if (stage == 0) {
          const uint64_t m = __ballot(got);
          if (m && lane == 0) U[w] &= ~m;
        }
      });
      break;
    case PH_RMAX:
      node_pass(r, U, lo, hi, key_of, [&](uint32_t w, int32_t v, bool in, uint64_t k) {
        const bool got = in && k != CLD_INF64;
        if (got) {
          const uint32_t c = (uint32_t)k;
          fold_rmax(r, R, c, d.D[v]);
          r.key[v] = (uint64_t)c;
          if (s.records) r.keyn[v] = (uint64_t)c;
        }
        const uint64_t m = __ballot(got);
        if (m && lane == 0) U[w] &= ~m;
      });
      break;
    case PH_SINGLE:
      node_pass(r, U, lo, hi, no_load, [&](uint32_t, int32_t v, bool in, uint64_t) {
        if (!in) return;
        d.cluster[v] = v;
        d.D[v] = 0;
      });
      break;
    case PH_C2_INIT:
      for (uint32_t w = lo + threadIdx.x; w < hi; w += kSweepThreads) {
        const int64_t left = (int64_t)d.n - ((int64_t)w << 6);
        U[w] = left >= 64 ? ~0ull : (1ull << left) - 1ull;
        for (int i = 0; i < 4; ++i) F[i * job.fwords + w] = 0;
      }
      for (int64_t v = ((int64_t)lo << 6) + threadIdx.x; v < ((int64_t)hi << 6) && v < d.n; v += kSweepThreads)
        r.key[v] = CLD_INF64;
      break;
    case PH_C2_ASSIGN:
      node_pass(r, U, lo, hi, key_of, [&](uint32_t w, int32_t v, bool in, uint64_t k) {
        const bool got = in && k != CLD_INF64;
        if (got) {
          const uint32_t c = (uint32_t)k;
          const uint64_t local = k >> 32;
          const uint64_t Dv = local + (uint64_t)r.delta * (uint64_t)(stage + 1 - R[c]);
          d.cluster[v] = (int32_t)c;
          d.D[v] = Dv;
          r.keyn[v] = local;   // kept for next iteration's rescaled edges
          r.key[v] = (uint64_t)c;
          if (Dv > r.acc) r.acc = Dv;
        }
        const uint64_t m = __ballot(got);
        if (m && lane == 0) U[w] &= ~m;
        cov += (uint32_t)__popcll(m);
      });
      break;
    default:
      break;
  }
  if (phase == PH_RELAX && !steps) {
    // Local rounds: relax the nodes that this workgroup improved.  What is
    // left when they end stays for the next sweep.  Round i reads queue i & 1
    // and counter i % 3 and fills the other queue and the next counter; the
    // third counter is cleared meanwhile, so the barrier that ends a round's
    // last pass is the only one.
    uint32_t n = 0, slot = 0;
    int q = 0;
    __syncthreads();
    for (int round = 0;; ++round) {
      n = S.qn[slot] < d.lq_cap ? S.qn[slot] : d.lq_cap;
      if (n == 0 || round >= d.local_rounds) break;
      if (job.cutoff < (uint32_t)job.nblocks) {
        if (threadIdx.x == 0)
          S.stop = __hip_atomic_load(idle, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= job.cutoff;
        __syncthreads();
        const uint32_t stop = S.stop;
        __syncthreads();
        if (stop) break;
      }
      r.q = q ^ 1;
      r.qslot = slot == 2 ? 0 : slot + 1;
      if (threadIdx.x == 0) S.qn[slot == 0 ? 2 : slot - 1] = 0;
      for (uint32_t i0 = 0; i0 < n; i0 += kSweepThreads) {
        for (uint32_t i = i0 + threadIdx.x / kRowLanes; i < n && i < i0 + kSweepThreads; i += kSweepThreads / kRowLanes)
          relax_queued(r, S.qv[q][i], S.qk[q][i]);
        relax_long<false>(r);
      }
      q ^= 1;
      slot = r.qslot;
    }
    for (uint32_t i = threadIdx.x; i < n; i += kSweepThreads) leave(r, S.qv[q][i], (uint32_t)(S.qk[q][i] >> 32));
  }
  // fold the threads' and waves' sums
  const bool is_min = phase == PH_NEXT || phase == PH_NEXT_PULL;
  if (is_growth(phase) || phase == PH_C2_SELECT) {
    r.scanned = cld_last_lane(cld_wave_scan_u32(r.scanned));
    r.heavy = cld_last_lane(cld_wave_scan_u32(r.heavy));
  }
  if (phase == PH_PULL || (steps && phase == PH_RELAX)) {
    if (steps) cov = cld_last_lane(cld_wave_scan_u32(r.covered));
    const uint32_t upd = cld_last_lane(cld_wave_scan_u32(r.updated));
    if (lane == 0 && upd) atomicAdd(&S.sum.upd, upd);
  }
  if (phase != PH_RELAX && __any(r.acc != (is_min ? CLD_INF64 : 0ull)))
    for (int o = 32; o >= 1; o >>= 1) {
      const unsigned long long y = __shfl_xor(r.acc, o);
      r.acc = is_min ? (y < r.acc ? y : r.acc) : (phase == PH_SELECT ? r.acc + y : (y > r.acc ? y : r.acc));
    }
  if ((phase == PH_RELAX || phase == PH_PULL) && __any(r.fmin != 0xffffffffu)) {
    for (int o = 32; o >= 1; o >>= 1) {
      const uint32_t y = __shfl_xor(r.fmin, o);
      r.fmin = y < r.fmin ? y : r.fmin;
    }
    if (lane == 0) atomicMin(&S.sum.fmin, r.fmin);
  }
  if (lane == 0) {
    if (r.scanned) atomicAdd(&S.sum.arcs, (unsigned long long)r.scanned);
    if (r.heavy) atomicAdd(&S.sum.blk_arcs, (unsigned long long)r.heavy);
    if (cov) atomicAdd(&S.sum.cov, cov);
    if (is_min) {
      if (r.acc != CLD_INF64) atomicMin(&S.sum.next, r.acc);
    } else if (r.acc) {
      if (phase == PH_SELECT) atomicAdd(&S.sum.hub_arcs, r.acc);
      else atomicMax(&S.sum.radius, r.acc);
    }
  }
  __syncthreads();
  if (table) {
    for (uint32_t t = threadIdx.x; t < kRmaxSlots; t += kSweepThreads) {
      const uint32_t c = S.rmax.tag[t];
      if (c == kRmaxFree) continue;
      const unsigned long long m = S.rmax.mx[t];
      if (m > R[c]) atomicMax((unsigned long long *)&R[c], m);
    }
  }
  if (threadIdx.x == 0) {
    const GCount &x = S.sum;
    if (x.fmin != 0xffffffffu) atomicMin(&cn.fmin, x.fmin);
    if (x.cov) atomicAdd(phase == PH_SELECT || phase == PH_C2_SELECT ? &cn.centers : &cn.cov, x.cov);
    if (x.upd) atomicAdd(&cn.upd, x.upd);
    if (x.records) cn.records = 1;
    if (x.next != CLD_INF64) atomicMin(&cn.next, x.next);
    if (x.radius) atomicMax(&cn.radius, x.radius);
    if (steps && phase == PH_RELAX && x.arcs) atomicAdd(&cn.msgs, x.arcs);
    if (x.blk_arcs) atomicAdd(&cn.blk_arcs, x.blk_arcs);
    if (x.hub_arcs) atomicAdd(&cn.hub_arcs, x.hub_arcs);
    if (x.arcs) atomicAdd(&cn.arcs, x.arcs);
  }
  __syncthreads();
}

// Chunk index -> graph (largest g with seg[g] <= i).
__device__ __forceinline__ int graph_of(const Job &job, uint32_t i) {
  int lo = 0, hi = job.G - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (job.seg[mid] <= i) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// First chunk of a workgroup: workgroups go to the XCDs in turn, so each XCD
// takes one eighth of the first chunks and neighbouring ranges share an L2.
__device__ __forceinline__ uint32_t first_chunk(uint32_t block, uint32_t nblocks, uint32_t total) {
  if (nblocks & 7) return block;
  const uint32_t all = total < nblocks ? total : nblocks, per = (all + 7) >> 3;
  const uint32_t i = block >> 3, c = (block & 7) * per + i;
  return i < per && c < all ? c : 0xffffffffu;
}

// Chunks of a sweep; the first of each workgroup, then whichever is next, so
// that costly chunks (hub rows) do not hold up a sweep.
template <class Chunk>
__device__ __forceinline__ void take_chunks(const Job &job, SweepCount &sc, uint32_t total, uint32_t block,
                                            uint32_t nblocks, Stage &S, Chunk chunk) {
  for (uint32_t v = first_chunk(block, nblocks, total); v < total;) {
    chunk(v);
    if (total <= nblocks) break;
    if (threadIdx.x == 0) S.chunk = nblocks + atomicAdd(&sc.cursor, 1u);
    __syncthreads();
    v = S.chunk;
    __syncthreads();
  }
  if (threadIdx.x == 0 && job.cutoff < (uint32_t)job.nblocks) atomicAdd(&sc.idle, 1u);
}

// Chunk c of a graph's sweep: `per` words, or cut by arcs (per = 0).
__device__ __forceinline__ void run_chunk(const Job &job, const GDesc &d, const GState &s, GCount &cn, uint32_t *idle, uint32_t per,
                          uint32_t c, Stage &S) {
  uint32_t lo = c * per, hi = lo + per < d.words ? lo + per : d.words, na = 0, nb = 0;
  if (per == 0) {
    const int32_t *cut = job.cut + 2 * (d.off >> 6);
    const uint32_t f = cuts_per_chunk(s), first = c * f, end = first + f < s.cuts ? first + f : s.cuts;
    na = (uint32_t)__builtin_amdgcn_readfirstlane(cut[first]);
    nb = (uint32_t)__builtin_amdgcn_readfirstlane(cut[end]);
    if (na >= nb) return;   // a row that costs more than a chunk
    lo = na >> 6;
    hi = (nb + 63) >> 6;
    if (s.phase == PH_RELAX) {
      // several chunks per workgroup, most of them without a frontier: not worth
      // a pass's fixed part
      const uint64_t *F = job.F + (d.off >> 6);
      bool any = false;
      for (uint32_t w = lo + threadIdx.x; w < hi; w += kSweepThreads)
        any = any || F[s.cur * job.fwords + w] != 0 || (s.merge && F[s.blk * job.fwords + w] != 0);
      if (!__syncthreads_or(any)) return;
    }
  }
  process_run(job, d, s, cn, idle, lo, hi, na, nb, S);
}

// A sweep of a job of several graphs, after its control launch.
__device__ __forceinline__ void sweep_many(const Job &job, uint32_t block, uint32_t nblocks, Stage &S) {
  const uint32_t total = job.ctl->total;
  SweepCount &sc = job.ctl->sc[0];
  take_chunks(job, sc, total, block, nblocks, S, [&](uint32_t v) {
    const int g = graph_of(job, v);
    const GDesc &d = job.desc[g];
    run_chunk(job, d, job.st[g], job.cn[g], &sc.idle, job.seg[job.G + 1 + g], v - job.seg[g], S);
  });
}

// Sweep t (from 1) of a job of one graph, its control step included; false
// when the graph is done.
__device__ __forceinline__ bool sweep_one(const Job &job, const GDesc &d, uint32_t t, uint32_t block,
                                          uint32_t nblocks, Stage &S) {
  Ctl *ctl = job.ctl;
  const uint32_t tid = threadIdx.x;
  const uint32_t *st = (const uint32_t *)&job.ring[(t - 1) & 1], *cn = (const uint32_t *)&job.cn[(t + 2) % 3];
  for (uint32_t i = tid; i < sizeof(GState) / 4; i += kSweepThreads) ((uint32_t *)&S.st)[i] = st[i];
  for (uint32_t i = tid; i < sizeof(GCount) / 4; i += kSweepThreads) ((uint32_t *)&S.last)[i] = cn[i];
  __syncthreads();
  if (S.st.closed) return false;
  // the last workgroup, which has no chunk in a small graph, keeps the books
  const bool books = block == nblocks - 1;
  if (t == 1 && tid < kRanges) {
    uint64_t x = range_start(d, (int)tid + 1) - range_start(d, (int)tid);
    for (int o = 32; o >= 1; o >>= 1) {
      const uint64_t y = __shfl_xor(x, o);
      x = y > x ? y : x;
    }
    if (tid == 0) S.st.cuts = cuts_for(d, x, (int32_t)nblocks);
  }
  if (tid == 0) control_graph(d, S.st, S.last, books ? job.log : nullptr);
  __syncthreads();
  const bool done = S.st.phase == PH_DONE;
  if (books) {
    uint32_t *to = (uint32_t *)&job.ring[t & 1], *fin = (uint32_t *)&job.st[0];
    for (uint32_t i = tid; i < sizeof(GState) / 4; i += kSweepThreads) {
      const uint32_t x = ((const uint32_t *)&S.st)[i];
      to[i] = x;
      if (done) fin[i] = x;
    }
    __syncthreads();
    if (tid == 0) {
      // past the time limit the next sweep finds the graph done (this one goes
      // on, so that every workgroup ends at the same sweep)
      check_time(ctl);
      if (ctl->error) job.ring[t & 1].phase = PH_DONE;
      clear_count(job.cn[(t + 1) % 3]);
      ctl->sc[(t + 1) % 3].cursor = 0;
      ctl->sc[(t + 1) % 3].idle = 0;
      ctl->iterations = t;
      if (done) {
        ctl->done = 1;
        job.ring[0].closed = job.ring[1].closed = 1;   // whichever the next sweep reads
      }
      report(job, t, done ? 1u : 0u);
    }
  }
  if (done) return false;
  SweepCount &sc = ctl->sc[t % 3];
  uint32_t per = chunk_words(d, S.st.phase, (int32_t)nblocks), total = (d.words + per - 1) / per;
  if (by_arcs(S.st)) {
    per = 0;
    total = cut_chunks(S.st);
  }
  take_chunks(job, sc, total, block, nblocks, S,
              [&](uint32_t v) { run_chunk(job, d, S.st, job.cn[t % 3], &sc.idle, per, v, S); });
  return true;
}

// ---------------------------------------------------------------- kernels --

// The descriptor of a job of one graph, and the job's time limit.
__global__ void k_describe(Job job, GDesc d, unsigned long long t_limit) {
  *const_cast<GDesc *>(job.desc) = d;
  job.ctl->t_limit = t_limit;
}

// Fresh state of the nodes, sets and counters of graph g (a job of one graph
// has three sets of counters).
__device__ __forceinline__ void fresh_nodes(const Job &job, int32_t g, const GDesc &d) {
  if (blockIdx.x == 0 && threadIdx.x < (job.G == 1 ? 3u : 1u)) clear_count(job.cn[g + threadIdx.x]);
  const int64_t at = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = at; i < d.n; i += stride) {
    job.key[d.off + i] = CLD_INF64;
    job.keyn[d.off + i] = CLD_INF64;
    job.slim[d.off + i] = 0;
    if (d.variant == CLDIAM_VARIANT_STEPS) job.R[d.off + i] = CLD_INF64;   // see step_state
  }
  const int64_t woff = d.off >> 6;
  for (int64_t w = at; w < d.words; w += stride) {
    const int64_t left = (int64_t)d.n - (w << 6);
    job.U[woff + w] = left >= 64 ? ~0ull : (1ull << left) - 1ull;
    for (int i = 0; i < 4; ++i) job.F[i * job.fwords + woff + w] = 0;
  }
}

// Every graph of a job: graph first + blockIdx.y.
__global__ void __launch_bounds__(256) k_init(Job job, int32_t first) {
  const int32_t g = first + (int32_t)blockIdx.y;
  fresh_nodes(job, g, job.desc[g]);
}

// A server's graph enters slot g: descriptor, state, stage log and nodes.  One
// launch, with the descriptor as an argument (two copies, a fill and a wait
// for them took 80 us a graph).
__global__ void __launch_bounds__(256) k_admit(Job job, int32_t g, GDesc d) {
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) {
      const_cast<GDesc *>(job.desc)[g] = d;
      job.st[g] = GState{};   // PH_START
    }
    int32_t *log = job.log + (size_t)g * CLDIAM_STAGE_LOG * 4;
    for (int i = threadIdx.x; i < CLDIAM_STAGE_LOG * 4; i += 256) log[i] = 0;
  }
  fresh_nodes(job, g, d);
}

// A job of up to kSmallControl graphs takes a one-wave control step: no
// cross-wave barriers, a 64-entry scan.
template <int T>
__global__ void __launch_bounds__(T) k_control(Job job, bool restart) { control_block<T>(job, restart); }

constexpr int kSmallControl = 64;

// One step: for several graphs the control launch, then the sweep.
__global__ void __launch_bounds__(kSweepThreads, kCuThreads / kSweepThreads) k_sweep_many(Job job) {
  __shared__ Stage S;
  if (job.ctl->done) return;
  sweep_many(job, blockIdx.x, gridDim.x, S);
}

// The descriptor comes as an argument: reading it from memory field by field
// delayed every sweep by 1 to 2 us.
__global__ void __launch_bounds__(kSweepThreads, kCuThreads / kSweepThreads) k_sweep(Job job, GDesc d, uint32_t t) {
  __shared__ Stage S;
  sweep_one(job, d, t, blockIdx.x, gridDim.x, S);
}

void launch_step(const Job &job, const GDesc *one, uint32_t t, hipStream_t stream, bool restart = false) {
  if (one) {
    k_sweep<<<job.nblocks, kSweepThreads, 0, stream>>>(job, *one, t);
    return;
  }
  if (job.G <= kSmallControl) k_control<kSmallControl><<<1, kSmallControl, 0, stream>>>(job, restart);
  else k_control<kThreads><<<1, kThreads, 0, stream>>>(job, restart);
  k_sweep_many<<<job.nblocks, kSweepThreads, 0, stream>>>(job);
}

__global__ void __launch_bounds__(kSweepThreads, kCuThreads / kSweepThreads) k_persistent(Job job) {
  __shared__ Stage S;
  const uint32_t nb = gridDim.x;
  if (job.G == 1) {
    for (uint32_t t = 1; sweep_one(job, job.desc[0], t, blockIdx.x, nb, S); ++t)
      if (!cld_grid_barrier(&job.ctl->bar, &job.ctl->timeout, nb)) return;
    return;
  }
  for (;;) {
    if (blockIdx.x == 0) control_block<kSweepThreads>(job);
    if (!cld_grid_barrier(&job.ctl->bar, &job.ctl->timeout, nb)) return;
    if (job.ctl->done || job.ctl->timeout) return;
    sweep_many(job, blockIdx.x, nb, S);
    if (!cld_grid_barrier(&job.ctl->bar, &job.ctl->timeout, nb)) return;
  }
}

// ------------------------------------------------------------------- host --

struct Layout {
  GDesc *desc;
  char *zero;         // st, ring, ctl and log lie together: cleared at the start, read back at the end
  size_t zero_bytes;
  GState *st, *ring;
  GCount *cn;
  Ctl *ctl;
  uint32_t *seg;
  int32_t *log;
  uint64_t *key, *keyn, *R;
  uint32_t *slim;
  uint64_t *U, *F;
  int32_t *cut;
  int64_t fwords;
};

// Every graph's nodes start at a multiple of 64, so that its bitmap words are
// its own.
constexpr int64_t kNodeAlign = 64;
int64_t aligned_nodes(int64_t n) { return (n + kNodeAlign - 1) / kNodeAlign * kNodeAlign; }

// N: node slots, a multiple of kNodeAlign.
template <class A>
bool carve(A &a, int64_t N, int32_t G, Layout *L) {
  auto p_desc = a.template take<GDesc>(G);
  auto p_st = a.template take<GState>(G);
  auto p_ring = a.template take<GState>(2);
  auto p_ctl = a.template take<Ctl>(1);
  auto p_log = a.template take<int32_t>((size_t)G * CLDIAM_STAGE_LOG * 4);
  auto p_cn = a.template take<GCount>(G < 3 ? 3 : G);
  auto p_seg = a.template take<uint32_t>(2 * (size_t)G + 1);
  auto p_key = a.template take<uint64_t>(N);
  auto p_keyn = a.template take<uint64_t>(N);
  auto p_R = a.template take<uint64_t>(N);
  auto p_slim = a.template take<uint32_t>(N);
  auto p_U = a.template take<uint64_t>(N / 64);
  auto p_F = a.template take<uint64_t>(4 * (N / 64));
  auto p_cut = a.template take<int32_t>(2 * (N / 64));   // at most a chunk for every word, and the end
  if (L) {
    *L = Layout{(GDesc *)p_desc, (char *)p_st, (size_t)((char *)p_cn - (char *)p_st), (GState *)p_st,
                (GState *)p_ring, (GCount *)p_cn, (Ctl *)p_ctl, (uint32_t *)p_seg, (int32_t *)p_log,
                (uint64_t *)p_key, (uint64_t *)p_keyn, (uint64_t *)p_R, (uint32_t *)p_slim, (uint64_t *)p_U,
                (uint64_t *)p_F, (int32_t *)p_cut, N / 64};
    return p_desc && p_cut;
  }
  return true;
}

Job make_job(const Layout &L, int32_t G) {
  Job job{};
  job.desc = L.desc; job.st = L.st; job.ring = L.ring; job.cn = L.cn; job.ctl = L.ctl; job.seg = L.seg;
  job.log = L.log; job.key = L.key; job.keyn = L.keyn; job.R = L.R; job.slim = L.slim; job.U = L.U;
  job.F = L.F; job.cut = L.cut; job.fwords = L.fwords;
  job.G = G;
  return job;
}

// Blocks of k_init for the graphs of a job of N node slots.
dim3 init_grid(int64_t N, int32_t G) { return dim3((unsigned)cld::blocks_for(N / G, 256, G > 1 ? 1024 : 8192), (unsigned)G); }

struct SizeArena {
  cld::Sizer s;
  template <class T>
  void *take(size_t n) { s.take<T>(n); return (void *)1; }
};

struct PtrArena {
  cld::Arena a;
  PtrArena(void *p, size_t c) : a(p, c) {}
  template <class T>
  void *take(size_t n) { return (void *)a.take<T>(n); }
};

constexpr size_t kMirrorOffset = cld::kPinnedBytes - 128;   // host-loop mirror words in the readback buffer
constexpr uint32_t kLeadSteps = 16;   // steps the host queues ahead of the device
constexpr size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }
constexpr size_t kReadback = up256(sizeof(GState)) + up256(2 * sizeof(GState)) + up256(sizeof(Ctl)) +
                             up256(CLDIAM_STAGE_LOG * 16);   // Layout's zero region of one graph
static_assert(kReadback <= kMirrorOffset, "readback and mirror words must fit a pooled pinned buffer");
static_assert(sizeof(Stage) <= 160 * 1024, "a workgroup's LDS");

// Workgroups of the sweep grid: one per CU unless requested (bounded by the
// co-resident maximum for the persistent kernel).
int grid_blocks(int driver, int requested, int *blocks) {
  int coop_blocks = 0;
  int rc = cld::cooperative_blocks((const void *)k_persistent, kSweepThreads, kCuThreads / kSweepThreads,
                                   &coop_blocks);
  if (rc) return rc;
  int dev = 0, cus = 0;
  CLD_HIP(hipGetDevice(&dev));
  CLD_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  int want = requested > 0 ? requested : cus * (kCuThreads / kSweepThreads);
  if (driver == CLDIAM_DRIVER_HOST) {
    *blocks = want;
    return CLDIAM_OK;
  }
  if (coop_blocks == 0) {
    *blocks = 0;
    return CLDIAM_OK;
  }
  *blocks = want < coop_blocks ? want : coop_blocks;
  return CLDIAM_OK;
}

// Finished workgroups after which the others end their local rounds.
uint32_t local_cutoff(const cldiam_tuning *tuning, int blocks) {
  int pct = tuning && tuning->local_cutoff > 0 ? tuning->local_cutoff : kLocalCutoffPct;
  if (pct > 100) pct = 100;
  return (uint32_t)(((int64_t)pct * blocks + 99) / 100);
}

// Descriptor of one graph (node offset set by the caller); returns a status.
int make_desc(const cldiam_graph &x, int g, const cldiam_tuning *tuning, GDesc *out) {
  float bucket_width = tuning ? tuning->bucket_width : 0.f;
  if (x.n < 1 || x.m < 0 || x.m >= ((int64_t)1 << 40) || !x.d_row_ptr || (x.m && !x.d_arcs) || !x.d_cluster ||
      !x.d_D || x.params.tau < 1) {
    cld::set_error("decompose: invalid graph %d (n=%d m=%lld tau=%u)", g, x.n, (long long)x.m, x.params.tau);
    return CLDIAM_EINVAL;
  }
  GDesc &d = *out;
  memset(&d, 0, sizeof d);
  d.row_ptr = x.d_row_ptr;
  d.arcs = x.d_arcs;
  d.cluster = x.d_cluster;
  d.D = x.d_D;
  d.n = x.n;
  d.words = (uint32_t)(((int64_t)x.n + 63) >> 6);
  const double gamma = 4.0 * M_LN2;
  const double L = log2((double)x.n);
  d.K = gamma * x.params.tau * L;
  d.stop = (uint32_t)ceil(8.0 * x.params.tau * L);
  d.seed = x.params.seed;
  if (x.params.variant > CLDIAM_VARIANT_CLUSTER2) {
    cld::set_error("decompose: unknown variant %u (graph %d)", x.params.variant, g);
    return CLDIAM_EINVAL;
  }
  d.variant = x.params.variant;
  d.step_cap = x.params.step_cap;
  // local rounds: the caller's, else many on sparse graphs (long growth
  // paths: each round carries the frontier one more hop without a sweep)
  // and few on dense ones (their rows are long and their growth shallow)
  // long-row bucket: the caller's shift, else the default; none for
  // synchronous steps (their sweeps take every active node)
  // The default narrows with the graph: a narrower bucket saves rescans of
  // long rows but costs sweeps, whose fixed cost weighs more on small graphs.
  const int32_t rs = tuning ? tuning->row_bucket_shift : 0;
  int32_t auto_shift = 0;
  while (auto_shift < 62 && (x.m >> (auto_shift + 1)) > 0) ++auto_shift;   // floor(log2 m)
  auto_shift = auto_shift / 2 - 6;
  auto_shift = auto_shift < kRowShiftMin ? kRowShiftMin : (auto_shift > kRowShiftMax ? kRowShiftMax : auto_shift);
  d.row_shift = (rs < 0 || d.variant == CLDIAM_VARIANT_STEPS) ? -1 : (rs == 0 ? auto_shift : (rs > 31 ? 31 : rs));
  // large dense graphs: the cost of a chunk varies with the hub rows it
  // holds, so cut their frontiers finer and hand the chunks out on demand
  const int32_t cf = tuning ? tuning->chunk_factor : 0;
  d.chunk_factor = cf > 0 ? (cf > 64 ? 64 : cf)
                          : ((x.m > (int64_t)kDenseDegree * x.n && x.n > kDenseLarge) ? kDenseChunks : 1);
  const int64_t fit = x.m > 0 ? kGrowArcs * x.n / (64 * x.m) : kGrowWords;
  d.grow_words = fit < 1 ? 1u : (fit < (int64_t)kGrowWords ? (uint32_t)fit : kGrowWords);
  // row tiers (threads per row) and the local queue's size
  const int32_t wr = tuning ? tuning->wave_row_min : 0, gr = tuning ? tuning->group_row_min : 0;
  const int32_t lqc = tuning ? tuning->local_queue : 0;
  const bool dense = x.m > (int64_t)kDenseDegree * x.n;
  d.mid_deg = wr > 0 ? (wr > (1 << 20) ? (1 << 20) : wr) : (dense ? kDenseWaveRow : kMidDeg);
  d.big_deg = gr > 0 ? (gr > (1 << 30) ? (1 << 30) : gr) : kBigDeg;
  if (d.big_deg < d.mid_deg) d.big_deg = d.mid_deg;
  d.lq_cap = lqc > 0 ? (uint32_t)(lqc < 64 ? 64 : (lqc > kLocalCap ? kLocalCap : lqc)) : (uint32_t)kLocalCap;
  const int32_t pm = tuning ? tuning->pull_mode : 0;
  if (pm < 0 || pm > CLDIAM_PULL_ALWAYS) {
    cld::set_error("decompose: unknown pull mode %d (graph %d)", pm, g);
    return CLDIAM_EINVAL;
  }
  // CLUSTER2 (its preliminary CLUSTER run included) and the literal steps never pull
  d.pull_mode = d.variant == CLDIAM_VARIANT_FIXPOINT ? (uint32_t)pm : (uint32_t)CLDIAM_PULL_NEVER;
  {
    const int64_t hd = x.m / x.n * kHubDegree;
    d.hub_deg = (uint32_t)(hd < 0xffffffffll ? hd : 0xffffffffll);
    d.hub_min = (uint64_t)(x.m / kHubShare);
  }
  if (tuning && tuning->local_rounds >= 0) d.local_rounds = tuning->local_rounds > 64 ? 64 : tuning->local_rounds;
  else if (x.m <= (int64_t)kDenseDegree * x.n) d.local_rounds = kLocalRounds;
  else d.local_rounds = x.n > kDenseLarge ? kLocalRoundsDense : 0;
  d.c2_iters = 0;
  while (((int64_t)1 << d.c2_iters) < (int64_t)x.n) d.c2_iters++;   // ceil(log2 n)
  uint64_t d0 = x.params.delta0;
  if (d0 == 0) d0 = x.m > 0 ? x.weight_sum / (uint64_t)x.m : 1;
  if (d0 < 1) d0 = 1;
  if (d0 > CLD_DELTA_MAX) {
    cld::set_error("decompose: initial Delta %llu above 2^31 (graph %d)", (unsigned long long)d0, g);
    return CLDIAM_EOVERFLOW;
  }
  d.delta0 = (uint32_t)d0;
  // bucket width in mean arc weights -> distance units (0 = unbounded)
  if (bucket_width == 0.f) bucket_width = CLDIAM_BUCKET_DEFAULT;
  d.bucket = 0;
  if (bucket_width > 0.f && x.m > 0 && d.variant != CLDIAM_VARIANT_STEPS) {
    const double b = ceil((double)bucket_width * ((double)x.weight_sum / (double)x.m));
    d.bucket = b >= 4294967295.0 ? 0u : (b < 1.0 ? 1u : (uint32_t)b);
  }
  return CLDIAM_OK;
}

void fill_stats(const GDesc &d, const GState &st, const int32_t *log, cldiam_stats *o) {
  memset(o, 0, sizeof *o);
  o->stages = (int32_t)st.stage;
  o->levels = (int32_t)st.levels;
  o->delta0 = d.delta0;
  o->delta_end = st.delta;
  o->stop = (int32_t)d.stop;
  o->num_clusters = (int32_t)(st.centers_total + st.singletons);
  o->singletons = (int32_t)st.singletons;
  o->sweeps = (int32_t)st.sweeps;
  o->radius = st.radius;
  o->status = st.status;
  o->rounds = st.rounds;
  o->radius1 = st.radius1;
  o->updates = st.updates;
  o->messages = st.msgs;
  for (int s = 0; s < CLDIAM_STAGE_LOG && s < o->stages; ++s) {
    const int32_t *l = log + (size_t)s * 4;
    o->stage_uncovered[s] = l[0];
    o->stage_centers[s] = l[1];
    o->stage_covered[s] = l[2];
    o->stage_delta[s] = (uint32_t)l[3];
  }
}

int read_wall_limit(unsigned long long *limit) {
  int dev = 0, khz = 0;
  CLD_HIP(hipGetDevice(&dev));
  CLD_HIP(hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev));
  if (khz <= 0) khz = 100000;
  *limit = (unsigned long long)khz * 1000ull * kJobSeconds;
  return CLDIAM_OK;
}

}  // namespace

extern "C" size_t cldiam_decompose_workspace_size(int64_t total_n, int32_t num_graphs) {
  if (total_n < 1 || num_graphs < 1) return 0;
  SizeArena s;
  carve(s, aligned_nodes(total_n + (int64_t)(num_graphs - 1) * (kNodeAlign - 1)), num_graphs, nullptr);
  return s.s.used;
}

extern "C" int cldiam_decompose_batch(int32_t G, const cldiam_graph *gs, cldiam_stats *stats, int driver,
                                      const cldiam_tuning *tuning, void *ws, size_t ws_bytes, void *stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  if (G < 1 || !gs) { cld::set_error("decompose: num_graphs < 1 or no graphs"); return CLDIAM_EINVAL; }
  int64_t total = 0, N = 0;   // nodes, node slots
  std::vector<GDesc> desc(G);
  for (int g = 0; g < G; ++g) {
    int rc = make_desc(gs[g], g, tuning, &desc[g]);
    if (rc) return rc;
    desc[g].off = N;
    total += gs[g].n;
    N += aligned_nodes(gs[g].n);
  }
  if (total >= ((int64_t)1 << 31)) { cld::set_error("decompose: more than 2^31 nodes in one job"); return CLDIAM_EINVAL; }
  Layout L;
  PtrArena pa(ws, ws_bytes);
  if (!carve(pa, N, G, &L) || pa.a.used > ws_bytes) {
    cld::set_error("decompose: workspace of %zu bytes, %zu needed", ws_bytes,
                   cldiam_decompose_workspace_size(total, G));
    return CLDIAM_ENOMEM;
  }
  Job job = make_job(L, G);
  const bool one = G == 1;
  unsigned long long limit = 0;
  int rc = read_wall_limit(&limit);
  if (rc) return rc;
  CLD_HIP(hipMemsetAsync(L.zero, 0, L.zero_bytes, stream));
  if (one) {
    k_describe<<<1, 1, 0, stream>>>(job, desc[0], limit);
  } else {
    CLD_HIP(hipMemcpyAsync(L.desc, desc.data(), sizeof(GDesc) * G, hipMemcpyHostToDevice, stream));
    CLD_HIP(hipMemcpyAsync(&L.ctl->t_limit, &limit, sizeof limit, hipMemcpyHostToDevice, stream));
  }
  for (int32_t g = 0; g < G; g += 65535) {
    const int32_t part = G - g < 65535 ? G - g : 65535;
    k_init<<<init_grid(N, part), 256, 0, stream>>>(job, g);
  }
  CLD_LAUNCH_CHECK("k_init");

  int blocks = 0;
  rc = grid_blocks(driver == CLDIAM_DRIVER_PERSISTENT ? driver : CLDIAM_DRIVER_HOST, tuning ? tuning->grid_blocks : 0,
                   &blocks);
  if (rc) return rc;
  if (blocks == 0 && driver == CLDIAM_DRIVER_PERSISTENT) {
    cld::set_error("decompose: device has no cooperative launch");
    return CLDIAM_EINVAL;
  }
  const bool persistent = driver == CLDIAM_DRIVER_PERSISTENT && blocks > 0;
  if (!persistent && blocks <= 0) blocks = 256;
  if (blocks > 65535) blocks = 65535;
  job.nblocks = blocks;
  job.cutoff = local_cutoff(tuning, blocks);
  struct Readback {
    char zero[kReadback];
  };
  cld::Pinned<Readback> pinned;   // back to the pool when the call returns
  if (!pinned.p) { cld::set_error("decompose: pinned host buffer allocation failed"); return CLDIAM_EHIP; }
  cld::Drain drain{stream, true};   // queued steps write the mirror
  const Ctl *hc = (const Ctl *)(pinned.p->zero + ((char *)L.ctl - L.zero));   // one graph: where ctl is read back
  // the last line of the same buffer: the control step's mirror for the host loop
  volatile uint32_t *hm = (volatile uint32_t *)((char *)pinned.p + kMirrorOffset);
  hipEvent_t ev0 = nullptr, ev1 = nullptr;
  CLD_HIP(hipEventCreate(&ev0));
  CLD_HIP(hipEventCreate(&ev1));
  struct EvGuard {
    hipEvent_t a, b;
    ~EvGuard() { if (a) (void)hipEventDestroy(a); if (b) (void)hipEventDestroy(b); }
  } evg{ev0, ev1};
  CLD_HIP(hipEventRecord(ev0, stream));
  if (persistent) {
    void *args[] = {&job};
    CLD_HIP(hipLaunchCooperativeKernel((const void *)k_persistent, dim3(blocks), dim3(kSweepThreads), args, 0,
                                       stream));
  } else {
    // The host queues steps at most kLeadSteps ahead of the control steps the
    // device has finished (read from the mapped mirror, no stream
    // synchronisation), and stops queueing once the device reports the job
    // done: only the steps already queued then run, and they return at once.
    hm[0] = 0;
    hm[1] = 0;
    uint32_t *dm = nullptr;
    CLD_HIP(hipHostGetDevicePointer((void **)&dm, (void *)hm, 0));
    job.hmirror = dm;
    const auto t0 = std::chrono::steady_clock::now();
    uint32_t queued = 0;
    for (;;) {
      if (hm[1]) break;
      if (queued < hm[0] + kLeadSteps) {
        launch_step(job, one ? &desc[0] : nullptr, ++queued, stream);
        if ((queued & 15u) == 0) CLD_LAUNCH_CHECK("k_sweep");
        continue;
      }
      if (std::chrono::steady_clock::now() - t0 > std::chrono::seconds(kJobSeconds + 30)) {
        cld::set_error("decompose: host-driven job exceeded its time limit");
        return CLDIAM_ETIMEOUT;
      }
      std::this_thread::yield();
    }
    CLD_LAUNCH_CHECK("k_sweep");
  }
  CLD_HIP(hipEventRecord(ev1, stream));
  std::vector<char> many(one ? 0 : L.zero_bytes);
  char *back = one ? pinned.p->zero : many.data();
  CLD_HIP(hipMemcpyAsync(back, L.zero, L.zero_bytes, hipMemcpyDeviceToHost, stream));
  CLD_HIP(hipStreamSynchronize(stream));
  drain.armed = false;
  if (!one) hc = (const Ctl *)(back + ((char *)L.ctl - L.zero));
  if (persistent && hc->timeout) { cld::set_error("decompose: grid barrier timed out"); return CLDIAM_ETIMEOUT; }
  if (!hc->done && !(persistent && hc->error)) {
    cld::set_error("decompose: %s", persistent ? "persistent kernel ended early"
                                               : "host-driven job ended without its done flag");
    return CLDIAM_EHIP;
  }
  if (!persistent) blocks = 0;
  const GState *st = (const GState *)back;
  const int32_t *lg = (const int32_t *)(back + ((char *)L.log - L.zero));
  float kernel_ms = 0.f;
  CLD_HIP(hipEventElapsedTime(&kernel_ms, ev0, ev1));
  rc = CLDIAM_OK;
  for (int g = 0; g < G; ++g) {
    if (st[g].status != CLDIAM_OK && rc == CLDIAM_OK) {
      rc = st[g].status;
      cld::set_error("decompose: graph %d failed: %s", g, cldiam_strerror(rc));
    }
    if (!stats) continue;
    fill_stats(desc[g], st[g], lg + (size_t)g * CLDIAM_STAGE_LOG * 4, &stats[g]);
    stats[g].arcs_scanned = one ? st[g].arcs : 0;
    stats[g].grid_blocks = blocks;
    stats[g].kernel_ms = kernel_ms;
    stats[g].iterations = (int32_t)hc->iterations;
  }
  if (rc == CLDIAM_OK && hc->error) {
    rc = -(int)hc->error;
    cld::set_error("decompose: device reported %s", cldiam_strerror(rc));
  }
  return rc;
}

extern "C" int cldiam_decompose(const cldiam_graph *g, cldiam_stats *stats, int driver, const cldiam_tuning *tuning,
                                void *ws, size_t ws_bytes, void *stream) {
  return cldiam_decompose_batch(1, g, stats, driver, tuning, ws, ws_bytes, stream);
}

// ----------------------------------------------------------- server job --
// A long-lived decomposition job with graph slots: requests are queued by
// cldiam_server_submit, admitted between sweeps when a slot and a node range
// of the workspace are free, advanced together with every other active graph,
// and released as soon as they finish.

struct cldiam_server {
  Layout L;
  Job job;
  int64_t ncap;
  int32_t gcap;
  cldiam_tuning tuning;
  hipStream_t stream;
  int blocks;
  std::vector<GDesc> desc;
  std::vector<uint64_t> tag;
  std::vector<char> active;
  std::vector<std::pair<int64_t, int64_t>> free_ranges;  // (offset, length), sorted by offset
  struct Pending {
    GDesc d;
    uint64_t tag;
  };
  std::vector<Pending> queue;
  size_t qhead = 0;
  struct Done {
    uint64_t tag;
    cldiam_stats st;
  };
  std::vector<Done> done;
  // pinned copy of the device's states (all slots) and Ctl, as they lie in the workspace
  char *back = nullptr;
  size_t back_bytes = 0;
  const GState *st_host() const { return (const GState *)back; }
  const Ctl *hc() const { return (const Ctl *)(back + ((char *)L.ctl - L.zero)); }
};

namespace {

bool take_range(cldiam_server *s, int64_t n, int64_t *off) {
  for (size_t i = 0; i < s->free_ranges.size(); ++i) {
    auto &r = s->free_ranges[i];
    if (r.second >= n) {
      *off = r.first;
      r.first += n;
      r.second -= n;
      if (r.second == 0) s->free_ranges.erase(s->free_ranges.begin() + i);
      return true;
    }
  }
  return false;
}

void give_range(cldiam_server *s, int64_t off, int64_t n) {
  auto &fr = s->free_ranges;
  auto it = std::lower_bound(fr.begin(), fr.end(), std::make_pair(off, (int64_t)0));
  it = fr.insert(it, {off, n});
  size_t i = it - fr.begin();
  if (i + 1 < fr.size() && fr[i].first + fr[i].second == fr[i + 1].first) {
    fr[i].second += fr[i + 1].second;
    fr.erase(fr.begin() + i + 1);
  }
  if (i > 0 && fr[i - 1].first + fr[i - 1].second == fr[i].first) {
    fr[i - 1].second += fr[i].second;
    fr.erase(fr.begin() + i);
  }
}

}  // namespace

extern "C" size_t cldiam_server_workspace_size(int64_t node_capacity, int32_t max_graphs) {
  return cldiam_decompose_workspace_size(node_capacity, max_graphs);
}

extern "C" int cldiam_server_create(cldiam_server **out, int64_t node_capacity, int32_t max_graphs,
                                    const cldiam_tuning *tuning, void *ws, size_t ws_bytes, void *stream) {
  if (!out || node_capacity < 1 || node_capacity >= ((int64_t)1 << 31) || max_graphs < 1 || max_graphs > 65536) {
    cld::set_error("server: invalid capacity");
    return CLDIAM_EINVAL;
  }
  *out = nullptr;
  cldiam_server *s = new cldiam_server();
  PtrArena pa(ws, ws_bytes);
  // room for every set of graphs of node_capacity nodes in all, each aligned
  const int64_t slots = aligned_nodes(node_capacity + (int64_t)(max_graphs - 1) * (kNodeAlign - 1));
  if (!carve(pa, slots, max_graphs, &s->L) || pa.a.used > ws_bytes) {
    delete s;
    cld::set_error("server: workspace of %zu bytes, %zu needed", ws_bytes,
                   cldiam_decompose_workspace_size(node_capacity, max_graphs));
    return CLDIAM_ENOMEM;
  }
  s->ncap = node_capacity;
  s->gcap = max_graphs;
  s->tuning = tuning ? *tuning : cldiam_tuning{-1, 0, 0.f, 0, 0, 0, 0, 0, 0, 0};
  s->stream = (hipStream_t)stream;
  const Layout &L = s->L;
  s->job = make_job(L, max_graphs);
  Job &job = s->job;
  int rc = grid_blocks(CLDIAM_DRIVER_HOST, tuning ? tuning->grid_blocks : 0, &s->blocks);
  if (rc) { delete s; return rc; }
  if (s->blocks <= 0) s->blocks = 256;
  job.nblocks = s->blocks;
  job.cutoff = local_cutoff(tuning, s->blocks);
  s->desc.assign(max_graphs, GDesc{});
  s->tag.assign(max_graphs, 0);
  s->active.assign(max_graphs, 0);
  s->free_ranges.push_back({0, slots});
  s->back_bytes = (size_t)((char *)L.log - L.zero);
  std::vector<GState> idle(max_graphs, GState{});
  for (auto &g : idle) g.phase = PH_IDLE;
  void *p = nullptr;
  if (hipHostMalloc(&p, s->back_bytes, hipHostMallocDefault) != hipSuccess) {
    delete s;
    cld::set_error("server: pinned host buffer allocation failed");
    return CLDIAM_EHIP;
  }
  s->back = (char *)p;
  unsigned long long limit = 0;
  rc = read_wall_limit(&limit);
  if (rc) { cldiam_server_destroy(s); return rc; }
  hipStream_t st = s->stream;
  if (hipMemsetAsync(L.zero, 0, L.zero_bytes, st) != hipSuccess ||
      hipMemcpyAsync(L.desc, s->desc.data(), sizeof(GDesc) * max_graphs, hipMemcpyHostToDevice, st) != hipSuccess ||
      hipMemcpyAsync(L.st, idle.data(), sizeof(GState) * max_graphs, hipMemcpyHostToDevice, st) != hipSuccess ||
      hipMemcpyAsync(&L.ctl->t_limit, &limit, sizeof limit, hipMemcpyHostToDevice, st) != hipSuccess ||
      hipStreamSynchronize(st) != hipSuccess) {
    cldiam_server_destroy(s);
    cld::set_error("server: initialisation failed");
    return CLDIAM_EHIP;
  }
  *out = s;
  return CLDIAM_OK;
}

extern "C" void cldiam_server_destroy(cldiam_server *s) {
  if (!s) return;
  if (s->back) (void)hipHostFree(s->back);
  delete s;
}

extern "C" int cldiam_server_submit(cldiam_server *s, const cldiam_graph *g, uint64_t tag) {
  if (!s || !g) { cld::set_error("server: null argument"); return CLDIAM_EINVAL; }
  if (g->n > s->ncap) { cld::set_error("server: graph of %d nodes above the capacity %lld", g->n, (long long)s->ncap); return CLDIAM_ENOMEM; }
  cldiam_server::Pending p;
  int rc = make_desc(*g, 0, &s->tuning, &p.d);
  if (rc) return rc;
  p.tag = tag;
  s->queue.push_back(p);
  return CLDIAM_OK;
}

extern "C" int cldiam_server_step(cldiam_server *s, int32_t max_sweeps, int32_t *h_active, int32_t *h_queued) {
  if (!s || max_sweeps < 0) { cld::set_error("server: invalid step"); return CLDIAM_EINVAL; }
  hipStream_t stream = s->stream;
  Job &job = s->job;
  bool admitted = false;
  // admit queued graphs in arrival order while a slot and a node range are free
  while (s->qhead < s->queue.size()) {
    int slot = -1;
    for (int g = 0; g < s->gcap; ++g)
      if (!s->active[g]) { slot = g; break; }
    if (slot < 0) break;
    cldiam_server::Pending &p = s->queue[s->qhead];
    int64_t off = 0;
    if (!take_range(s, aligned_nodes(p.d.n), &off)) break;
    p.d.off = off;
    s->desc[slot] = p.d;
    s->tag[slot] = p.tag;
    s->active[slot] = 1;
    k_admit<<<init_grid(p.d.n, 1), 256, 0, stream>>>(job, slot, p.d);
    CLD_LAUNCH_CHECK("k_admit");
    admitted = true;
    s->qhead++;
  }
  if (s->qhead > 1024 && s->qhead * 2 > s->queue.size()) {
    s->queue.erase(s->queue.begin(), s->queue.begin() + s->qhead);
    s->qhead = 0;
  }
  int nactive = 0;
  for (int g = 0; g < s->gcap; ++g) nactive += s->active[g];
  if (nactive > 0 && max_sweeps > 0) {
    for (int i = 0; i < max_sweeps; ++i) launch_step(job, nullptr, 0, stream, i == 0);
    CLD_LAUNCH_CHECK("k_sweep");
    CLD_HIP(hipMemcpyAsync(s->back, s->L.zero, s->back_bytes, hipMemcpyDeviceToHost, stream));
    CLD_HIP(hipStreamSynchronize(stream));
    const GState *st = s->st_host();
    if (s->hc()->error) {
      cld::set_error("server: device reported %s", cldiam_strerror(-(int)s->hc()->error));
      return -(int)s->hc()->error;
    }
    // the stage logs of the slots that are done, in one copy
    int first = -1, last = -1;
    for (int g = 0; g < s->gcap; ++g) {
      if (!s->active[g] || st[g].phase != PH_DONE) continue;
      if (first < 0) first = g;
      last = g;
    }
    std::vector<int32_t> lg;
    constexpr size_t kLog = CLDIAM_STAGE_LOG * 4;
    if (first >= 0) {
      lg.resize((size_t)(last - first + 1) * kLog);
      CLD_HIP(hipMemcpyAsync(lg.data(), job.log + (size_t)first * kLog, sizeof(int32_t) * lg.size(),
                             hipMemcpyDeviceToHost, stream));
      CLD_HIP(hipStreamSynchronize(stream));
    }
    for (int g = first; g >= 0 && g <= last; ++g) {
      if (!s->active[g] || st[g].phase != PH_DONE) continue;
      cldiam_server::Done dn;
      dn.tag = s->tag[g];
      fill_stats(s->desc[g], st[g], lg.data() + (size_t)(g - first) * kLog, &dn.st);
      s->done.push_back(dn);
      s->active[g] = 0;
      give_range(s, s->desc[g].off, aligned_nodes(s->desc[g].n));
      --nactive;
    }
  } else if (admitted) {
    CLD_HIP(hipStreamSynchronize(stream));
  }
  if (h_active) *h_active = nactive;
  if (h_queued) *h_queued = (int32_t)(s->queue.size() - s->qhead);
  return CLDIAM_OK;
}

extern "C" int cldiam_server_poll(cldiam_server *s, uint64_t *h_tags, cldiam_stats *h_stats, int32_t max_done,
                                  int32_t *h_ndone) {
  if (!s || !h_ndone || max_done < 0) { cld::set_error("server: invalid poll"); return CLDIAM_EINVAL; }
  int32_t k = 0;
  while (k < max_done && k < (int32_t)s->done.size()) {
    if (h_tags) h_tags[k] = s->done[k].tag;
    if (h_stats) h_stats[k] = s->done[k].st;
    ++k;
  }
  s->done.erase(s->done.begin(), s->done.begin() + k);
  *h_ndone = k;
  return CLDIAM_OK;
}
