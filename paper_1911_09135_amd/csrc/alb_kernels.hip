// Device side of the adaptive load balancer (ALB) for gfx950 (wave64).
//
// One BSP round of a data-driven push traversal (paper Section 2) is two
// phases over the active worklist F:
//
//   phase 1  inspection + TWC (Algorithm 1, Section 3 "TWC").  Each workgroup
//            takes up to B entries of F at a time (see Order).  A vertex
//            whose out-degree is >= threshold is appended to the huge list;
//            its degree is added to prefixWork in the same wave-aggregated 64-bit atomic, so the
//            exclusive prefix of the huge degrees (Section 4.1 "Search") is
//            known once the phase ends.  Every other vertex is processed at
//            once by the workgroup, wavefront or thread bin of its degree.
//   phase 2  execution (Algorithm 2), only when the huge list is non-empty
//            (Section 4.3).  Huge edge k goes to thread k mod T (the cyclic
//            distribution, Section 4.1), so the 64 lanes of a wavefront take
//            64 consecutive edges and read consecutive col / weight entries.
//            The source of edge k is the last prefixWork entry <= k.  The
//            search starts from a chunk index written when the huge list is
//            reserved (the slot owning the first edge of every 2^s-edge
//            chunk), so it costs one or two probes instead of log2(v) levels.
//
// Each lane keeps kU edges in flight: loads of all of them are issued before
// any operator decision, which hides the random-access latency of the
// destination labels.  The operator (BFS, SSSP, CC, PageRank, or a recorder
// for tests) is a template parameter.  Pushes to the next worklist are
// staged per wavefront in LDS and reserved in batches.
//
// Rounds are driven either from the host (one launch per phase) or inside one
// persistent launch whose phases are separated by a grid-wide barrier.

#include <type_traits>

#include "alb_internal.h"

namespace alb {
namespace {

constexpr int kWave = 64;
constexpr int kU = kEdgesPerLanePass;  // edges in flight per lane
// Per-wavefront LDS staging of next-worklist pushes, in bytes: 1,024 vertex
// ids or 512 (query, vertex) pairs.  Reservations on the worklist's size
// counter are what it saves: atomics on one address complete one every 12 ns
// whoever issues them, so their number, not their latency, bounds a phase.
constexpr uint32_t kPushBytes = 4096;

__device__ __forceinline__ uint32_t lane_id() {
  return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}
// Inclusive sum over the wavefront's lanes (all of them active), with lane
// moves inside the vector unit: a shuffle goes through LDS, 64 cycles or more
// each, and six of them in a row were a tenth of a short round's phase.
__device__ __forceinline__ uint32_t wave_inclusive(uint32_t x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1, 2, 4, 8
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
  return x;
}
// number of set bits of m below this lane
__device__ __forceinline__ uint32_t bits_below(unsigned long long m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// The XCD (accelerator complex die, one L2) the calling wave runs on: the
// XCC_ID hardware register, bits [3:0].
__device__ __forceinline__ uint32_t xcd_id() {
  return __builtin_amdgcn_s_getreg((3 << 11) | (0 << 6) | 20) & (uint32_t)(kBarXcds - 1);
}

template <class T>
__device__ __forceinline__ T ld_relaxed(T *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ __forceinline__ void st_relaxed(T *p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ __forceinline__ T add_relaxed(T *p, T v) {
  return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Records written in one phase and read in the next go through agent-scope
// accesses, so that the grid barrier between the phases needs no cache
// maintenance (see grid_barrier).
__device__ __forceinline__ void st_hint(int2 *p, int2 h) {
  st_relaxed((unsigned long long *)p, ((unsigned long long)(uint32_t)h.y << 32) | (uint32_t)h.x);
}
__device__ __forceinline__ int2 ld_hint(const int2 *p) {
  const unsigned long long x = ld_relaxed((const unsigned long long *)p);
  return make_int2((int32_t)(uint32_t)x, (int32_t)(x >> 32));
}
__device__ __forceinline__ void st_rec(int4 *p, int4 r) {
  st_hint((int2 *)p, make_int2(r.x, r.y));
  st_hint((int2 *)p + 1, make_int2(r.z, r.w));
}
__device__ __forceinline__ int4 ld_rec(const int4 *p) {
  const int2 lo = ld_hint((const int2 *)p), hi = ld_hint((const int2 *)p + 1);
  return make_int4(lo.x, lo.y, hi.x, hi.y);
}

// Overflow is recorded as the first round in which it happened; a workgroup
// stops at the start of a later round, so every workgroup decides alike.
__device__ __forceinline__ void flag_overflow(Ctl *c, int round) {
  __hip_atomic_fetch_min(&c->overflow, (uint32_t)round, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// fp32 value -> 64-bit fixed point (round to nearest)
__device__ __forceinline__ unsigned long long to_fix(float x) { return __double2ull_rn((double)x * kFixScale); }

template <class V>
__device__ __forceinline__ int32_t to_bits(V x) {
  return __builtin_bit_cast(int32_t, x);
}
template <class V>
__device__ __forceinline__ V from_bits(int32_t x) {
  return __builtin_bit_cast(V, x);
}

// ---------------------------------------------------------------------------
// Operators.  The work along one edge is split into prepare() (issue the loads
// it needs) and commit() (decide, update the destination, and say whether the
// destination goes to the next worklist), so that a lane can have kU edges'
// loads in flight before the first decision.
// ---------------------------------------------------------------------------

// Label indices (long long) address the label arrays: the vertex id for a
// single query; query offset + vertex id for a batch of queries sharing one
// launch.  Graph indices (CSR positions, vertex ids) are separate.

// BFS: level[dst] = level[src] + 1 on first visit (compare-and-swap from INF).
// Every active vertex of round r has level r, so no source level is read.
struct OpBFS {
  using val_t = int32_t;
  static constexpr int kKind = OP_BFS;
  struct pre_t {
    int32_t cur;
  };
  static constexpr bool kPush = true, kNeedSrc = false, kRecord = false, kPR = false, kBatch = true, kHot = false;
  int32_t *level;
  __device__ __forceinline__ val_t load_src(long long, int32_t, uint32_t tag, bool &) const {
    return (int32_t)tag - 1;
  }
  __device__ __forceinline__ pre_t prepare(int32_t, long long dl, val_t, int32_t) const {
    return {ld_relaxed(&level[dl])};
  }
  __device__ __forceinline__ bool commit(const pre_t &p, int32_t, long long dl, val_t sv, int32_t, int32_t,
                                         uint32_t) const {
    if (p.cur != kInf) return false;
    int32_t expected = kInf;
    return __hip_atomic_compare_exchange_strong(&level[dl], &expected, sv + 1, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
  }
};

// BFS once the persistent launch has built the reached-vertex bitmap: a
// destination whose bit is set has been reached and its level is not read
// (a clear bit says nothing: the level decides).  A type of its own, so that
// the rounds before the bitmap exists run the plain operator's code.
struct OpBFSFilter : OpBFS {
  const uint32_t *vbits;
  __device__ __forceinline__ pre_t prepare(int32_t, long long dl, val_t, int32_t) const {
    if ((vbits[dl >> 5] >> (dl & 31)) & 1u) return {0};
    return {ld_relaxed(&level[dl])};
  }
};

// SSSP and CC keep one 64-bit word per vertex: (label << 32) | tag, where tag
// is 1 + the round that last lowered the label.  A relaxation in round r
// offers (candidate << 32) | (r + 1) to an atomic minimum: it lowers the word
// exactly when the candidate is smaller (an equal candidate never changes the
// word, its tag being no smaller), and the old word says both whether the
// label dropped and whether it had already dropped this round, in which case
// the vertex is already on the next worklist.  One random atomic per
// relaxation serves as both the update and the push deduplication.
__device__ __forceinline__ bool lower_word(unsigned long long *word, int32_t cand, unsigned long long cur,
                                           uint32_t tag, int32_t dedup) {
  if (cand >= (int32_t)(cur >> 32)) return false;  // a stale (larger) cached word only costs an atomic
  const unsigned long long old = __hip_atomic_fetch_min(word, ((unsigned long long)(uint32_t)cand << 32) | tag,
                                                        __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return cand < (int32_t)(old >> 32) && (!dedup || (uint32_t)old != tag);
}

// The label of an active vertex.  If its tag shows that it was lowered again
// during the current round, it is already on the next worklist and will be
// processed there with the newer label, so relaxing its edges now (with the
// older, larger label) is skipped.
__device__ __forceinline__ int32_t label_of_active(unsigned long long w, uint32_t tag, bool &skip) {
  skip = (uint32_t)w == tag;
  return (int32_t)(w >> 32);
}

struct OpSSSP {  // relaxation: dist[dst] = min(dist[dst], dist[src] + w)
  using val_t = int32_t;
  static constexpr int kKind = OP_SSSP;
  struct pre_t {
    int32_t cand;
    unsigned long long cur;
  };
  static constexpr bool kPush = true, kNeedSrc = false, kRecord = false, kPR = false, kBatch = true, kHot = false;
  unsigned long long *word;
  const int32_t *w;
  int32_t dedup;
  __device__ __forceinline__ val_t load_src(long long sl, int32_t, uint32_t tag, bool &skip) const {
    return label_of_active(ld_relaxed(&word[sl]), tag, skip);
  }
  // The candidate sv + w saturates at INT32_MAX (the unreached label), which it
  // then cannot lower.  Both terms are in [0, INT32_MAX], so their sum fits in
  // 32 unsigned bits.  A sum beyond INT32_MAX - 1 is never a shortest
  // distance (graph creation bounds those by max(w) * (n - 1)), so dropping
  // it changes no result.
  __device__ __forceinline__ pre_t prepare(int32_t pos, long long dl, val_t sv, int32_t) const {
    const uint32_t c = (uint32_t)sv + (uint32_t)w[pos];
    return {(int32_t)min(c, (uint32_t)kInf), ld_relaxed(&word[dl])};
  }
  __device__ __forceinline__ bool commit(const pre_t &p, int32_t, long long dl, val_t, int32_t, int32_t,
                                         uint32_t tag) const {
    return lower_word(&word[dl], p.cand, p.cur, tag, dedup);
  }
};

// Continuous serving: BFS and SSSP queries in one launch.  A query slot
// flagged unit relaxes every edge with weight 1, so its distances are BFS
// levels; the others use the graph's weights.
struct OpServe : OpSSSP {
  const int32_t *unit;  // per query slot
  __device__ __forceinline__ pre_t prepare(int32_t pos, long long dl, val_t sv, int32_t q) const {
    const uint32_t c = (uint32_t)sv + (unit[q] ? 1u : (uint32_t)w[pos]);
    return {(int32_t)min(c, (uint32_t)kInf), ld_relaxed(&word[dl])};
  }
};

struct OpCC {  // min-label propagation
  using val_t = int32_t;
  static constexpr int kKind = OP_CC;
  struct pre_t {
    unsigned long long cur;
  };
  static constexpr bool kPush = true, kNeedSrc = false, kRecord = false, kPR = false, kBatch = false, kHot = false;
  unsigned long long *word;
  int32_t dedup;
  __device__ __forceinline__ val_t load_src(long long sl, int32_t, uint32_t tag, bool &skip) const {
    return label_of_active(ld_relaxed(&word[sl]), tag, skip);
  }
  __device__ __forceinline__ pre_t prepare(int32_t, long long dl, val_t, int32_t) const {
    return {ld_relaxed(&word[dl])};
  }
  __device__ __forceinline__ bool commit(const pre_t &p, int32_t, long long dl, val_t sv, int32_t, int32_t,
                                         uint32_t tag) const {
    return lower_word(&word[dl], sv, p.cur, tag, dedup);
  }
};

// CC with the filter: a set bit says the destination's label is already 0,
// the smallest vertex id, which no relaxation can lower; its word is not
// read (a clear bit says nothing).
struct OpCCFilter : OpCC {
  const uint32_t *vbits;
  __device__ __forceinline__ pre_t prepare(int32_t, long long dl, val_t, int32_t) const {
    if ((vbits[dl >> 5] >> (dl & 31)) & 1u) return {0ull};
    return {ld_relaxed(&word[dl])};
  }
};

// The filtering operator of BFS and CC, and the property its bitmap records.
template <class Op>
struct Filtered;
template <>
struct Filtered<OpBFS> {
  using type = OpBFSFilter;
  __device__ static type make(const OpBFS &op, const Args &a) {
    type f;
    f.level = op.level;
    f.vbits = a.vbits;
    return f;
  }
  __device__ static bool bit(const Args &a, uint32_t v) { return a.level[v] != kInf; }  // reached
};
template <>
struct Filtered<OpCC> {
  using type = OpCCFilter;
  __device__ static type make(const OpCC &op, const Args &a) {
    type f;
    f.word = op.word;
    f.dedup = op.dedup;
    f.vbits = a.vbits;
    return f;
  }
  __device__ static bool bit(const Args &a, uint32_t v) { return (a.word[v] >> 32) == 0ull; }  // label 0
};

// k-core (peeling): an active vertex has left the core; each of its edges
// lowers the neighbour's remaining degree, and the neighbour whose degree
// falls from k to k - 1 leaves in the next round, so every vertex is pushed
// at most once.  Round 0 inspects every vertex (no worklist) and takes those
// with fewer than k edges, judged by the CSR degree rather than the
// remaining degree that other lanes are already lowering.
//
// Decrements of one hub complete one every 12 ns, whoever issues them (Zipf
// graph of 1M vertices, k = 16: round 0's 4.9M decrements took 0.75 ms, the
// 60,000 of the largest hub alone 0.72).  Neighbours of at least kHotDegree
// edges, marked in a bitmap at set-up, are therefore counted in a table in
// LDS and lowered once per workgroup at the end of its phase; a vertex whose
// slot another holds takes the plain path.  Below that degree a hub costs a
// round 12 us at most, and marking more would only fill the table.  A graph
// without any has one clear word for a bitmap (hot_shift), which stays in the
// L1 (uniform graph of 2^20 vertices and 8.4M edges, k = 12, 16 workgroups: 2,620
// us with a whole one, 2,315 so; a branch around the look-up was slower on graphs
// with hubs, RMAT-20 253 us against 243).
// Workgroups of 64 threads have 128 slots: with 1,024, their 14.5 KB of LDS let
// 11 of them onto a CU instead of 20 (undirected Zipf graph of 2^19 vertices,
// k = 16, automatic grid: 437 us with 1,024 slots, 386 with 128).  So few fill up,
// and a vertex looks in four of them (Zipf graph of 2^20 vertices, k = 32: 1,585 us
// with 1,024 slots, 2,730 with 128, 1,610 with 128 and four looks).
constexpr uint32_t kHotNone = 0xffffffffu;
constexpr uint32_t hot_slots(int B) { return B == kWave ? 128 : 1024; }  // a power of two and a multiple of B
template <uint32_t kSlots>
struct HotTable {
  uint32_t key[kSlots], cnt[kSlots];
};
template <uint32_t kSlots>
__device__ __forceinline__ HotTable<kSlots> &hot_table() {
  __shared__ HotTable<kSlots> t;
  return t;
}
template <int B>
__device__ __forceinline__ void hot_clear() {
  HotTable<hot_slots(B)> &t = hot_table<hot_slots(B)>();
  for (uint32_t i = threadIdx.x; i < hot_slots(B); i += B) {
    t.key[i] = kHotNone;
    t.cnt[i] = 0;
  }
  __syncthreads();
}

template <uint32_t kSlots>
struct OpKCore {
  using val_t = int32_t;
  static constexpr int kKind = OP_KCORE;
  struct pre_t {
    uint32_t hot;
  };
  static constexpr bool kPush = true, kNeedSrc = false, kRecord = false, kPR = false, kBatch = false, kHot = true;
  int32_t *rem;
  int32_t k;
  const uint32_t *hot;
  uint32_t shift;
  __device__ __forceinline__ val_t load_src(long long, int32_t deg, uint32_t tag, bool &skip) const {
    if (tag == 1u) skip = deg >= k;
    return 0;
  }
  __device__ __forceinline__ pre_t prepare(int32_t, long long dl, val_t, int32_t) const {
    return {(hot[(uint32_t)dl >> shift] >> (dl & 31)) & 1u};
  }
  __device__ __forceinline__ bool commit(const pre_t &p, int32_t, long long dl, val_t, int32_t, int32_t,
                                         uint32_t) const {
    if (p.hot) {
      HotTable<kSlots> &t = hot_table<kSlots>();
      const uint32_t v = (uint32_t)dl, home = (v * 2654435761u) / (uint32_t)((1ull << 32) / kSlots);
#pragma unroll 1
      for (uint32_t probe = 0; probe < (kSlots < 1024 ? 4u : 1u); ++probe) {
        const uint32_t i = home ^ probe;
        uint32_t owner = __hip_atomic_load(&t.key[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (owner == kHotNone) {
          const uint32_t was = atomicCAS(&t.key[i], kHotNone, v);
          owner = was == kHotNone ? v : was;
        }
        if (owner == v) {
          atomicAdd(&t.cnt[i], 1u);
          return false;
        }
      }
    }
    return __hip_atomic_fetch_add(&rem[dl], -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == k;
  }
  // slot i's count (at a phase's end): does its vertex leave the core?
  __device__ __forceinline__ bool settle(uint32_t i, int32_t &v) const {
    HotTable<kSlots> &t = hot_table<kSlots>();
    const int32_t c = (int32_t)t.cnt[i];
    v = (int32_t)t.key[i];
    t.key[i] = kHotNone;
    if (c == 0) return false;
    t.cnt[i] = 0;
    const int32_t old = __hip_atomic_fetch_add(&rem[v], -c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return old >= k && old - c < k;
  }
};

// k-core with the filter: a set bit says the destination has already left
// the core (remaining degree below k), so decrementing it changes nothing
// (its degree stays below k and it is never pushed again); the atomic is
// skipped.
template <uint32_t kSlots>
struct OpKCoreFilter : OpKCore<kSlots> {
  using Core = OpKCore<kSlots>;
  using val_t = typename Core::val_t;
  const uint32_t *vbits;
  struct pre_t {
    typename Core::pre_t core;
    bool gone;
  };
  __device__ __forceinline__ pre_t prepare(int32_t pos, long long dl, val_t sv, int32_t src) const {
    return {Core::prepare(pos, dl, sv, src), ((vbits[dl >> 5] >> (dl & 31)) & 1u) != 0u};
  }
  __device__ __forceinline__ bool commit(const pre_t &p, int32_t pos, long long dl, val_t sv, int32_t src, int32_t gt,
                                         uint32_t tag) const {
    return !p.gone && Core::commit(p.core, pos, dl, sv, src, gt, tag);
  }
};
template <uint32_t kSlots>
struct Filtered<OpKCore<kSlots>> {
  using type = OpKCoreFilter<kSlots>;
  __device__ static type make(const OpKCore<kSlots> &op, const Args &a) {
    type f;
    f.rem = op.rem;
    f.k = op.k;
    f.hot = op.hot;
    f.shift = op.shift;
    f.vbits = a.vbits;
    return f;
  }
  __device__ static bool bit(const Args &a, uint32_t v) { return a.level[v] < a.kcore_k; }  // left the core
};

struct OpPR {  // acc[dst] += rank[src] / outdeg(src): fp32 contribution, exact fixed-point sum
  using val_t = float;
  static constexpr int kKind = OP_PR;
  struct pre_t {};
  static constexpr bool kPush = false, kNeedSrc = false, kRecord = false, kPR = true, kBatch = false, kHot = false;
  const float *rank;
  unsigned long long *acc;
  __device__ __forceinline__ val_t load_src(long long sl, int32_t deg, uint32_t, bool &) const {
    return rank[sl] / (float)deg;
  }
  __device__ __forceinline__ pre_t prepare(int32_t, long long, val_t, int32_t) const { return {}; }
  __device__ __forceinline__ bool commit(const pre_t &, int32_t, long long dl, val_t sv, int32_t, int32_t,
                                         uint32_t) const {
    add_relaxed(&acc[dl], to_fix(sv));
    return false;
  }
};

struct OpRecord {  // counts each processed edge and the thread that took it; pushes every destination
  using val_t = int32_t;
  static constexpr int kKind = OP_RECORD;
  struct pre_t {};
  static constexpr bool kPush = true, kNeedSrc = true, kRecord = true, kPR = false, kBatch = false, kHot = false;
  int32_t *hits;
  int32_t *thread_of;
  __device__ __forceinline__ val_t load_src(long long, int32_t, uint32_t, bool &) const { return 0; }
  __device__ __forceinline__ pre_t prepare(int32_t, long long, val_t, int32_t) const { return {}; }
  __device__ __forceinline__ bool commit(const pre_t &, int32_t pos, long long, val_t, int32_t, int32_t gt,
                                         uint32_t) const {
    add_relaxed(&hits[pos], 1);
    thread_of[pos] = gt;
    return true;
  }
};

template <class Op>
Op make_op(const Args &a);
template <>
OpBFS make_op<OpBFS>(const Args &a) { return OpBFS{a.level}; }
template <>
OpSSSP make_op<OpSSSP>(const Args &a) { return OpSSSP{a.word, a.w, a.dedup}; }
template <>
OpServe make_op<OpServe>(const Args &a) {
  OpServe o;
  o.word = a.word;
  o.w = a.w;
  o.dedup = a.dedup;
  o.unit = a.q_unit;
  return o;
}
template <>
OpCC make_op<OpCC>(const Args &a) { return OpCC{a.word, a.dedup}; }
template <>
OpPR make_op<OpPR>(const Args &a) { return OpPR{a.rank, a.acc}; }
template <>
OpRecord make_op<OpRecord>(const Args &a) { return OpRecord{a.hits, a.thread_of}; }
template <>
OpKCore<hot_slots(64)> make_op<OpKCore<hot_slots(64)>>(const Args &a) {
  return {a.level, a.kcore_k, a.hot, a.hot_shift};
}
template <>
OpKCore<hot_slots(256)> make_op<OpKCore<hot_slots(256)>>(const Args &a) {
  return {a.level, a.kcore_k, a.hot, a.hot_shift};
}

// ---------------------------------------------------------------------------
// Per-thread statistics, shared memory, work-distribution grid, push staging.
// ---------------------------------------------------------------------------

struct Acc {
  unsigned long long frontier = 0, edges_twc = 0, edges_lb = 0, huge_v = 0, pushes = 0;
  unsigned long long dangling = 0;  // fixed point
  unsigned long long prof[kProfParts] = {0, 0, 0, 0, 0, 0};
};

// Profiling aid: thread 0 of each workgroup adds the ticks since *t to part k.
__device__ __forceinline__ void prof_mark(const Args &a, Acc &acc, int k, uint64_t &t) {
  if (a.profile && threadIdx.x == 0) {
    const uint64_t now = (uint64_t)wall_clock64();
    acc.prof[k] += now - t;
    t = now;
  }
}

// Profiling aid: the edges this workgroup processed in round r (each wave
// adds its lanes' counts since the last call).
__device__ __forceinline__ void prof_round_edges(const Args &a, const Acc &acc, unsigned long long &last, uint32_t id,
                                                 int r) {
  const unsigned long long now = acc.edges_twc + acc.edges_lb;
  unsigned long long d = now - last;
  last = now;
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) d += __shfl_xor(d, o);
  if (lane_id() == 0 && d && r < kTimeline && id < (uint32_t)kProfMembers)
    add_relaxed(&a.prof_wg[(size_t)r * kProfMembers + id], (uint32_t)d);
}

// Worklist entries: a vertex id for one query; (query << 32) | vertex for a batch.
template <bool M>
using Entry = typename std::conditional<M, unsigned long long, int32_t>::type;

template <int B, class Op, bool M = false>
struct Smem {
  using V = typename Op::val_t;
  int32_t pos[kU * B];  // thread-bin gather: CSR position, source value and source (batch: query) of each edge
  V sv[kU * B];
  int32_t src[(Op::kNeedSrc || M) ? kU * B : 1];
  int32_t wsum[B / kWave];
  unsigned long long ured[B / kWave][kStats];
  unsigned long long dred[B / kWave];
  int32_t wcand[B / kWave];  // workgroup bin: a thread of each wavefront that holds a list for it, or -1
  int32_t owner, obeg, odeg, ov;
  V osv;
  int32_t flag;
  uint32_t ticket, members;  // persistent launch: this workgroup's ticket and the member count
  uint32_t xcd, xcd_n, n_xcd;  // its XCD, the members on that XCD, the XCDs holding members
  unsigned long long cbase;  // phase 1: first worklist entry of the current claim
  uint32_t clen;             // and its length
  Entry<M> pbuf[B / kWave][kPushBytes / sizeof(Entry<M>)];  // per-wavefront push staging
  // end of a phase: entries staged per wavefront, the workgroup's reservation
  alignas(16) uint32_t pcnt[B / kWave];
  uint32_t pbase;
};

// The workgroup's index and the workgroup count used for work distribution:
// the hardware ones for one-phase launches, the membership ticket and the
// member count inside the persistent launch.
struct Grid {
  uint32_t id;
  uint32_t n;
  uint32_t xcd = 0, xcd_n = 1, n_xcd = 1;  // persistent launch: barrier topology (see grid_barrier)
};

// Next-worklist pushes of one wavefront, staged in LDS and written out in
// batches: one global reservation per batch instead of one per ballot.
template <class E>
struct Pusher {
  E *buf;            // this wavefront's LDS staging area
  uint32_t cnt;      // entries staged (wave-uniform)
  E *qn;             // next worklist
  uint32_t *qn_cnt;  // its size counter
};

template <int B, class Op, bool M>
__device__ void flush_stats(Acc &acc, Smem<B, Op, M> &sm, Ctl *c) {
  const uint32_t lane = lane_id();
  const int w = threadIdx.x / kWave;
  unsigned long long v[kStats] = {acc.frontier, acc.edges_twc, acc.edges_lb, acc.huge_v, acc.pushes};
#pragma unroll
  for (int k = 0; k < kStats; ++k) {
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) v[k] += __shfl_xor(v[k], d);
    if (lane == 0) sm.ured[w][k] = v[k];
  }
  __syncthreads();
  if (threadIdx.x < kStats) {
    unsigned long long t = 0;
    for (int j = 0; j < B / kWave; ++j) t += sm.ured[j][threadIdx.x];
    if (t) add_relaxed(&c->stat[xcd_id() % kStatXcds][threadIdx.x].v, t);
  }
  if (threadIdx.x == 0) {
    for (int k = 0; k < kProfParts; ++k)
      if (acc.prof[k]) add_relaxed(&c->prof[k], acc.prof[k]);
  }
  __syncthreads();
  acc = Acc();
}

template <int B, class Op, bool M>
__device__ void flush_dangling(Acc &acc, Smem<B, Op, M> &sm, unsigned long long *dst) {
  unsigned long long x = acc.dangling;
#pragma unroll
  for (int d = kWave / 2; d > 0; d >>= 1) x += __shfl_xor(x, d);
  if (lane_id() == 0) sm.dred[threadIdx.x / kWave] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long t = 0;
    for (int j = 0; j < B / kWave; ++j) t += sm.dred[j];
    if (t != 0) add_relaxed(dst, t);
  }
  __syncthreads();
  acc.dangling = 0;
}

// Write this wavefront's staged entries to the next worklist from `base` on
// (all its lanes call this).
template <class E>
__device__ __forceinline__ void write_pushes(const Args &a, int round, Pusher<E> &pu, uint32_t base) {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  for (uint32_t j = lane_id(); j < pu.cnt; j += kWave) {
    const uint32_t idx = base + j;
    if (idx < a.qcap)
      st_relaxed(&pu.qn[idx], pu.buf[j]);
    else
      flag_overflow(a.ctl, round);
  }
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  pu.cnt = 0;
}

// Stage v for every lane with pred (all lanes of the wavefront call this).  A
// full staging area is written out with a reservation of its own.
template <class E>
__device__ __forceinline__ void push_wave(bool pred, E v, const Args &a, int round, Pusher<E> &pu, Acc &acc) {
  const unsigned long long m = __ballot(pred);
  if (m == 0ull) return;
  const uint32_t total = (uint32_t)__popcll(m);
  if (pu.cnt + total > kPushBytes / sizeof(E)) {
    uint32_t base = 0;
    if (lane_id() == 0) base = add_relaxed(pu.qn_cnt, pu.cnt);
    write_pushes(a, round, pu, (uint32_t)__shfl(base, 0));
  }
  if (pred) pu.buf[pu.cnt + bits_below(m)] = v;
  pu.cnt += total;
  if (lane_id() == 0) acc.pushes += total;
}

// The end of a phase: the whole workgroup writes out what its wavefronts have
// staged with ONE reservation.  One per wavefront made the phase ends of a
// launch of 800 to 1,024 workgroups cost 40 to 50 us each (12 ns per atomic on
// the one counter).  All threads call this; a workgroup barrier separates it
// from the next call.
template <int B, class S, class E>
__device__ __forceinline__ void flush_phase(const Args &a, S &sm, int round, Pusher<E> &pu) {
  const int w = threadIdx.x / kWave;
  if (lane_id() == 0) sm.pcnt[w] = pu.cnt;
  __syncthreads();
  uint32_t total = 0, before = 0;
#pragma unroll
  for (int j = 0; j < B / kWave; ++j) {
    const uint32_t c = sm.pcnt[j];
    before += j < w ? c : 0u;
    total += c;
  }
  if (total == 0) return;
  if (threadIdx.x == 0) sm.pbase = add_relaxed(pu.qn_cnt, total);
  __syncthreads();
  if (pu.cnt) write_pushes(a, round, pu, sm.pbase + before);
}

// A phase's end, before flush_phase: the hot counts become decrements and pushes.
template <int B, class Op, class E>
__device__ __forceinline__ void settle_hot(const Args &a, const Op &op, int round, Pusher<E> &pu, Acc &acc) {
  if constexpr (Op::kHot) {
    if (op.shift != 5) return;
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < hot_slots(B); i += B) {
      int32_t v;
      const bool p = op.settle(i, v);
      push_wave<E>(p, (E)v, a, round, pu, acc);
    }
  }
}

// log2 of the chunk size of the huge-edge index for a threshold t: the
// largest power of two not above t, clamped, so that a chunk holds at most
// two segment starts when t >= 2^Args::hint_min.  A short worklist (nF entries)
// has few lists, for which coarse chunks do, and perhaps a long one, whose
// fine chunks one wavefront would have to write (a hub of 1.8M edges: 13 us).
__device__ __forceinline__ uint32_t hint_shift(const Args &a, int64_t t, uint32_t nF) {
  const int least = nF < 256u ? max(a.hint_min, kHintCoarse) : a.hint_min;
  if (t < (1ll << least)) return (uint32_t)least;
  if (t >= (1ll << kHintMaxShift)) return kHintMaxShift;
  return 63u - (uint32_t)__builtin_clzll((unsigned long long)t);
}

// Algorithm 1, "work.push(src)": append every huge lane's vertex to the huge
// list and its degree to the running edge total with ONE 64-bit atomic per
// wavefront on (count << 32 | edges).  Slot j receives the edges of all
// earlier slots as its prefixWork entry, i.e. the exclusive scan of the huge
// degrees in list order, with the vertex's CSR start, the vertex (batch: its
// query) and the source value.  The
// wavefront then writes the chunk index for every chunk whose first edge
// falls in one of its new segments.  All lanes of the wavefront call this.
__device__ __forceinline__ void reserve_huge(bool huge, int32_t v_or_q, int32_t beg, int32_t deg, int32_t sv_bits,
                                             const Args &a, int round, unsigned long long *ctr, uint32_t hs,
                                             Acc &acc) {
  const unsigned long long hm = __ballot(huge);
  if (hm == 0ull) return;
  const uint32_t lane = lane_id();
  const unsigned long long mine = huge ? (unsigned long long)(uint32_t)deg : 0ull;
  unsigned long long incl = mine;
  if (__ballot(mine >> 25) == 0ull) {  // the 64 lanes' sum fits in 32 bits
    incl = wave_inclusive((uint32_t)mine);
  } else {
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      const unsigned long long y = __shfl_up(incl, d);
      if ((int)lane >= d) incl += y;
    }
  }
  const unsigned long long tot_e = __shfl(incl, kWave - 1);
  const uint32_t tot_c = (uint32_t)__popcll(hm);
  unsigned long long base = 0;
  int bad = 0;
  if (lane == kWave - 1) {
    if (tot_e >> 32) {
      bad = 1;
    } else {
      base = add_relaxed(ctr, ((unsigned long long)tot_c << 32) | tot_e);
      if ((unsigned long long)(uint32_t)base + tot_e > 0xffffffffull) bad = 1;
      acc.huge_v += tot_c;
    }
    if (bad) flag_overflow(a.ctl, round);
  }
  base = __shfl(base, kWave - 1);
  bad = __shfl(bad, kWave - 1);
  if (bad) return;  // the round is abandoned; nothing below may be trusted
  uint32_t j = 0, p = 0;
  if (huge) {
    j = (uint32_t)(base >> 32) + bits_below(hm);
    p = (uint32_t)base + (uint32_t)(incl - mine);
    if (j < a.qcap)
      st_rec(&a.huge_rec[j], make_int4((int32_t)p, beg, v_or_q, sv_bits));
    else
      flag_overflow(a.ctl, round);
  }
  // chunk index: chunk c's first edge c << hs lies in [p, p + deg).  A lane
  // writes up to two entries itself; longer runs are shared by the wavefront.
  const uint64_t my_lo = ((uint64_t)p + (1ull << hs) - 1) >> hs;
  const uint64_t my_hi = huge ? (((uint64_t)p + (uint32_t)deg - 1) >> hs) + 1 : 0;  // one past the last
  const bool few = my_hi <= my_lo + 2;
  if (few) {
    for (uint64_t c = my_lo; c < my_hi; ++c) {
      if (c < a.hint_cap)
        st_hint(&a.hint[c], make_int2((int32_t)j, (int32_t)(p + (uint32_t)deg)));
      else
        flag_overflow(a.ctl, round);
    }
  }
  unsigned long long rem = __ballot(huge && !few);
  while (rem) {
    const int l = __ffsll(rem) - 1;
    rem &= rem - 1;
    const uint32_t jj = __shfl(j, l), pp = __shfl(p, l);
    const uint32_t dd = (uint32_t)__shfl(deg, l);
    const uint64_t c_lo = ((uint64_t)pp + (1ull << hs) - 1) >> hs;
    const uint64_t c_hi = ((uint64_t)pp + dd - 1) >> hs;
    for (uint64_t c = c_lo + lane; c <= c_hi; c += kWave) {
      if (c < a.hint_cap)
        st_hint(&a.hint[c], make_int2((int32_t)jj, (int32_t)(pp + dd)));
      else
        flag_overflow(a.ctl, round);
    }
  }
}

// Apply the operator along up to kU edges per lane and push; every lane of
// the wavefront calls this (act[u] false for empty slots).  src[u] is the
// source vertex (recorder) or, for a batch, the query of slot u.
template <class Op, bool M>
__device__ __forceinline__ void edges(const bool (&act)[kU], const int32_t (&pos)[kU],
                                      const typename Op::val_t (&sv)[kU], const int32_t (&src)[kU], const Op &op,
                                      const Args &a, uint32_t tag, int round, Pusher<Entry<M>> &pu, Acc &acc,
                                      int32_t gt) {
  int32_t dst[kU];
  long long dl[kU];
  typename Op::pre_t pre[kU];
#pragma unroll
  for (int u = 0; u < kU; ++u) dst[u] = a.col[act[u] ? pos[u] : 0];
  // an empty slot addresses label 0, which always exists (a batch's query
  // offsets can be negative, so no other index is safe for every query)
#pragma unroll
  for (int u = 0; u < kU; ++u) {
    if constexpr (M)
      dl[u] = act[u] ? dst[u] + a.qoff[src[u]] : 0;
    else
      dl[u] = act[u] ? dst[u] : 0;
  }
#pragma unroll
  for (int u = 0; u < kU; ++u) pre[u] = op.prepare(act[u] ? pos[u] : 0, dl[u], sv[u], src[u]);
  bool p[kU];
#pragma unroll
  for (int u = 0; u < kU; ++u) p[u] = act[u] && op.commit(pre[u], pos[u], dl[u], sv[u], src[u], gt, tag);
  if constexpr (Op::kPush) {
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      if constexpr (M)
        push_wave<Entry<M>>(p[u], ((unsigned long long)(uint32_t)src[u] << 32) | (uint32_t)dst[u], a, round, pu,
                            acc);
      else
        push_wave<Entry<M>>(p[u], dst[u], a, round, pu, acc);
    }
  }
}

// Exclusive sum over the workgroup.  A workgroup barrier separates it from the
// next use of wsum.
template <int B>
__device__ __forceinline__ void block_exscan(int32_t x, int32_t &excl, int32_t &total, int32_t *wsum) {
  const uint32_t lane = lane_id();
  const int w = threadIdx.x / kWave;
  const int32_t incl = (int32_t)wave_inclusive((uint32_t)x);
  if (lane == kWave - 1) wsum[w] = incl;
  __syncthreads();
  int32_t before = 0, tot = 0;
#pragma unroll
  for (int j = 0; j < B / kWave; ++j) {
    const int32_t s = wsum[j];
    before += (j < w) ? s : 0;
    tot += s;
  }
  excl = before + incl - x;
  total = tot;
}

// Waves per SIMD the persistent kernel's register budget is sized for: the
// traversal is bound by the latency of dependent random loads, so more
// resident waves keep more of them in flight.
#ifndef ALB_WAVES_PER_EU
#define ALB_WAVES_PER_EU 4
#endif

// ---------------------------------------------------------------------------
// Phase 1: inspection (Algorithm 1) fused with the TWC bins.
// ---------------------------------------------------------------------------

// Worklist entries per claim: B, unless the worklist would give a workgroup
// fewer than two claims; then whole wavefronts' worth, just enough for two
// claims per workgroup, so that a short worklist still reaches every
// workgroup instead of leaving most of them idle for the phase.
__device__ __forceinline__ uint32_t twc_chunk(uint32_t nF, uint32_t wgs, int B) {
  const uint32_t per = nF ? (nF - 1u) / (2u * wgs) + 1u : 0u;  // rounded up, without a sum that could wrap
  return min(max((per + kWave - 1u) / kWave * kWave, (uint32_t)kWave), (uint32_t)B);
}

// Workgroups take runs of consecutive positions one at a time (which worklist
// entry a position stands for, Order says), so a run that takes long does not
// hold up work queued behind it.  The first run of workgroup g is fixed
// (positions [g * C0, (g + 1) * C0)) and needs no atomic; later runs are
// claimed from a counter over the positions beyond those, each sized from the
// remainder the previous claim's atomic returned (guided self-scheduling): B
// while plenty remain, then fewer whole wavefronts, so that the phase ends with short runs and the workgroups
// reach the barrier together.  The counter is only ever touched by the
// atomic (a plain load of a contended counter is slow).  Thread 0 of the
// workgroup holds the state; the caller's workgroup barriers separate one
// claim's reads of the published run from the next claim's writes.
struct Claims {
  uint32_t C0, len;
  unsigned long long S, nxt, seen;  // end of the fixed runs; the current run (at first the fixed one)
  __device__ Claims(Grid gr, uint32_t run)
      : C0(run), len(C0), S((unsigned long long)gr.n * C0), nxt((unsigned long long)gr.id * C0), seen(S) {}
  // Publish the next run as (*base, *n); *base >= nF means no more work.
  __device__ void next(unsigned long long *claim, uint32_t nF, Grid gr, int B, unsigned long long &base,
                       uint32_t &n) {
    if (S >= (unsigned long long)nF) {
      nxt = ~0ull;  // the fixed runs covered the worklist
    } else {
      len = twc_chunk(seen < nF ? nF - (uint32_t)seen : 0u, gr.n, B);
      nxt = S + add_relaxed(claim, (unsigned long long)len);
      seen = nxt + len;
    }
    base = nxt;
    n = len;
  }
};


// The order in which a phase's runs take the worklist's entries.  Neighbouring
// entries have alike degrees (the hubs of an RMAT graph sit at its lowest ids,
// and lists push their destinations in ascending order), so runs of consecutive
// entries differ by far more than one run should (RMAT-20 CC, round 0: the
// busiest workgroup had 4.8 times the mean edges, half of all workgroup time
// went by at barriers).  Runs therefore take entries from all over the
// list, in groups of kGroup from 256 / kGroup places, or singly where one run
// per workgroup covers it.  Except there on low-degree graphs (fill_log above
// 6): they have little skew, and neighbours in the list share the lines of their
// edges and labels (1,001 x 777 grid SSSP: 12.6 ms consecutive, 15.2 spread).
// The recorded round of alb_trace_round keeps consecutive runs of whole
// wavefronts' entries, so that its record shows the claims.
// Groups of 16, 4 and 1 (us): RMAT-20 CC 1,105, 1,050, 1,012; 64-query batch
// 2,542, 2,484, 2,485; Zipf 8.4M BFS 1,815, 1,829, 1,868.
constexpr uint32_t kGroup = 4, kPlaces = 256 / kGroup;
//
// The first run's length: a worklist that fits in one run of 2^fill_log entries
// per workgroup (the entries whose edges, at the graph's mean degree, fill one
// pass of the workgroup) is split over as many workgroups as it fills, and
// over 96 if it fills fewer.  A run's time is a chain of dependent loads, about
// the same for 2 entries as for one full pass, while every pass beyond the
// first and every long list in the same run adds to it (RMAT-14 BFS: 2,498
// entries in runs of 64 took 18.8 us, in runs of 27 14.7); but each workgroup
// with pushes also costs its 12 ns at the worklist counter, so a low-degree
// graph's runs are long (a grid of mean degree 4: 256 entries).
struct Order {
  uint32_t run;    // length of the first run
  uint32_t total;  // positions, a few of them beyond the list
  uint32_t used;   // single entries: from one to the next; 0: groups or consecutive
  uint32_t step;   // groups: from one place to the next; 0: consecutive
  __device__ Order(uint32_t nF, uint32_t wgs, int B, uint32_t fill, bool consecutive) {
    const uint32_t fill_log = fill & ~kFlat;
    used = step = 0;
    total = nF;
    if ((uint64_t)nF <= (uint64_t)wgs << fill_log && !consecutive) {
      const uint32_t w = max((nF + (1u << fill_log) - 1u) >> fill_log, min(wgs, 96u));
      run = (nF + w - 1u) / w;
      if (fill_log <= 6) {
        used = w;
        total = w * run;
      }
    } else {
      run = twc_chunk(nF, wgs, B);
      // A list of many runs per workgroup evens out by the claims alone, and
      // ascending ids then spread CC's labels faster within the round (Zipf of
      // 2^24 vertices: 13.9 ms consecutive, 14.5 spread; RMAT-21, within the
      // limit, 2.4 and 1.1).  The last positions have to fit in 32 bits.
      // Nor do flat graphs (kFlat) gain: there is no skew, and neighbours
      // share lines (undirected grid of 900 x 900, PageRank in bins, 10
      // iterations: 819 us spread, 685 consecutive; CC 56.9 and 53.6 ms).
      if (!consecutive && !(fill & kFlat) && (uint64_t)nF <= 32ull * (uint32_t)B * wgs && nF <= 0xffffff00u) {
        step = (uint32_t)(((uint64_t)nF + 255) / 256);
        total = step * 256u;
      }
    }
  }
  // entry of position base + j of workgroup id's run (may lie beyond the list)
  __device__ uint32_t entry(uint32_t base, uint32_t j, uint32_t id, bool ids) const {
    if (used) return j * used + id;
    const uint32_t p = base + j;
    if (!step) return p;
    const uint32_t place = p / kGroup % kPlaces;
    uint32_t row = p / 256u;
    if (ids) {
      // a round over every vertex: each place starts elsewhere.  Equal offsets
      // gave one run the ids that are alike in their low bits, and an RMAT id's
      // bits make its degree (RMAT-20 CC: 1,050 us so, 680 with this).
      row += __umulhi(place * 0x9E3779B1u, step);
      if (row >= step) row -= step;
    }
    return (place * step + row) * kGroup + p % kGroup;
  }
};

template <int B, class Op, bool M, class S>
__device__ void phase_twc(const Args &a, const Op &op, S &sm, Grid gr, int round,
                          const Entry<M> *F, uint32_t nF, Entry<M> *qn, uint32_t *qn_cnt, unsigned long long *hctr,
                          int64_t threshold, uint32_t hs, Acc &acc) {
  using V = typename Op::val_t;
  const int tid = threadIdx.x;
  const uint32_t lane = lane_id();
  const int32_t gt = (int32_t)(gr.id * B + tid);
  const uint32_t tag = (uint32_t)round + 1u;
  unsigned long long *claim = &a.ctl->chunk[round % 3].v;
  Pusher<Entry<M>> pu{sm.pbuf[tid / kWave], 0u, qn, qn_cnt};
  uint64_t pt = a.profile ? (uint64_t)wall_clock64() : 0;
  const Order order(nF, gr.n, B, a.fill, Op::kRecord);
  Claims cl(gr, order.run);
  unsigned long long base = cl.nxt;
  uint32_t C = cl.len;
  for (bool more = base < order.total; more;) {
    const uint32_t i = order.entry((uint32_t)base, (uint32_t)tid, gr.id, F == nullptr);
    const bool mine = tid < (int)C && base + (uint32_t)tid < order.total && i < nF;
    int32_t v = -1, beg = 0, deg = 0, q = 0;  // q: the entry's query (batch)
    int64_t thr = threshold;
    int32_t c_wave = a.c_wave, c_wg = a.c_wg;  // TWC cutoffs (a batch's queries may have their own)
    if (mine) {
      if constexpr (M) {
        const unsigned long long e = ld_relaxed(&F[i]);
        v = (int32_t)(uint32_t)e;
        q = (int32_t)(e >> 32);
        if (a.qthr) thr = a.qthr[q];
        if (a.qcut) {
          c_wave = a.qcut[2 * q];
          c_wg = a.qcut[2 * q + 1];
        }
      } else {
        v = F ? ld_relaxed(&F[i]) : (int32_t)i;
      }
      beg = a.off[v];
      deg = a.off[v + 1] - beg;
    }
    if constexpr (M) {
      // continuous serving: this round had an entry of query slot q.  One
      // plain store per run of equal slots in the wavefront, skipped once
      // the mark already reads this round (the grid barrier publishes it).
      // A store from every wavefront, all to the one address of a lone
      // query's slot, serialised the round: writing through to memory they
      // tripled the inspection phase.
      if (a.q_last) {
        const int32_t qq = mine ? q : -1;
        const int32_t prev = __shfl_up(qq, 1);
        if (mine && (lane == 0 || prev != qq) && a.q_last[qq] != (int32_t)round) a.q_last[qq] = (int32_t)round;
      }
    }
    V sv = V(0);
    if (deg > 0) {
      bool skip = false;
      long long sl = v;
      if constexpr (M) sl += a.qoff[q];
      sv = op.load_src(sl, deg, tag, skip);
      if (skip) deg = 0;
    }
    // inspection: degree >= THRESHOLD goes to the huge list
    const bool huge = v >= 0 && deg > 0 && (int64_t)deg >= thr;
    reserve_huge(huge, M ? q : v, beg, deg, to_bits(sv), a, round, hctr, hs, acc);
    if constexpr (Op::kRecord) {
      if (mine) a.bins[i] = (int8_t)(huge ? 3 : deg >= c_wg ? 2 : deg >= c_wave ? 1 : 0);
    }
    if constexpr (Op::kPR) {
      if (v >= 0 && deg == 0) acc.dangling += to_fix(a.rank[v]);
    }
    if (huge) deg = 0;
    acc.frontier += (v >= 0);
    acc.edges_twc += (unsigned long long)deg;
    prof_mark(a, acc, kProfInspect, pt);

    // workgroup bin: the whole workgroup strides one vertex's edges
    for (;;) {
      const unsigned long long cand = __ballot(deg > 0 && deg >= c_wg);
      if (lane == 0) sm.wcand[tid / kWave] = cand ? tid + __ffsll(cand) - 1 : -1;
      __syncthreads();
      int32_t o = -1;
#pragma unroll
      for (int w = 0; w < B / kWave; ++w) o = max(o, sm.wcand[w]);
      if (o < 0) break;
      if (tid == o) {
        sm.obeg = beg;
        sm.odeg = deg;
        sm.osv = sv;
        sm.ov = M ? q : v;
        deg = 0;
      }
      __syncthreads();
      const int32_t ob = sm.obeg, od = sm.odeg, ov = sm.ov;
      const V os = sm.osv;
      for (int32_t j0 = 0; j0 < od; j0 += kU * B) {
        bool act[kU];
        int32_t pos[kU], src[kU];
        V s[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          const int32_t j = j0 + u * B + tid;
          act[u] = j < od;
          pos[u] = ob + j;
          s[u] = os;
          src[u] = ov;
        }
        edges<Op, M>(act, pos, s, src, op, a, tag, round, pu, acc, gt);
      }
    }

    prof_mark(a, acc, kProfWgBin, pt);
    // wavefront bin: one wavefront strides one vertex's edges
    for (;;) {
      const unsigned long long mm = __ballot(deg > 0 && deg >= c_wave);
      if (mm == 0ull) break;
      const int ld = __ffsll(mm) - 1;
      const int32_t ob = __shfl(beg, ld), od = __shfl(deg, ld), ov = __shfl(M ? q : v, ld);
      const V os = __shfl(sv, ld);
      if ((int)lane == ld) deg = 0;
      for (int32_t j0 = 0; j0 < od; j0 += kU * kWave) {
        bool act[kU];
        int32_t pos[kU], src[kU];
        V s[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          const int32_t j = j0 + u * kWave + (int32_t)lane;
          act[u] = j < od;
          pos[u] = ob + j;
          s[u] = os;
          src[u] = ov;
        }
        edges<Op, M>(act, pos, s, src, op, a, tag, round, pu, acc, gt);
      }
    }

    prof_mark(a, acc, kProfWaveBin, pt);
    // thread bin: fine-grained gather of the remaining short lists through LDS,
    // kU * B edges at a time, so that the workgroup's lanes stay busy
    int32_t rank, total;
    block_exscan<B>(deg, rank, total, sm.wsum);
    for (int32_t done = 0; done < total; done += kU * B) {
      const int32_t lo = max(rank, done), hi = min(rank + deg, done + kU * B);
      for (int32_t e = lo; e < hi; ++e) {
        sm.pos[e - done] = beg + (e - rank);
        sm.sv[e - done] = sv;
        if constexpr (Op::kNeedSrc || M) sm.src[e - done] = M ? q : v;
      }
      __syncthreads();
      const int32_t cnt = min(kU * B, total - done);
      bool act[kU];
      int32_t pos[kU], src[kU];
      V s[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int32_t idx = u * B + tid;
        act[u] = idx < cnt;
        pos[u] = act[u] ? sm.pos[idx] : 0;
        s[u] = act[u] ? sm.sv[idx] : V(0);
        src[u] = 0;
        if constexpr (Op::kNeedSrc || M) src[u] = act[u] ? sm.src[idx] : 0;
      }
      edges<Op, M>(act, pos, s, src, op, a, tag, round, pu, acc, gt);
      __syncthreads();
    }
    prof_mark(a, acc, kProfThreadBin, pt);
    more = cl.S < (unsigned long long)order.total;  // else the fixed runs covered the worklist
    if (more) {
      if (tid == 0) cl.next(claim, order.total, gr, B, sm.cbase, sm.clen);
      __syncthreads();
      base = sm.cbase;
      C = sm.clen;
      more = base < order.total;
    }
  }
  settle_hot<B>(a, op, round, pu, acc);
  if constexpr (Op::kPush) flush_phase<B>(a, sm, round, pu);
  prof_mark(a, acc, kProfThreadBin, pt);
}

// The huge-list slot whose edge range holds huge edge k: the last slot j with
// prefixWork[j] <= k.  The chunk index gives the slot j0 that owns the first
// edge of k's chunk and where j0's edges end; k before that end is j0's,
// otherwise an exponential search forward from j0 + 1, then bisection, finds
// the answer (one probe when every huge degree is at least the chunk size).
__device__ __forceinline__ uint32_t owner_of(const Args &a, uint32_t vh, uint32_t hs, uint32_t k) {
  const int2 h = ld_hint(&a.hint[k >> hs]);
  if (k < (uint32_t)h.y) return (uint32_t)h.x;  // inside the segment that holds the chunk's first edge
  uint64_t lo = (uint32_t)h.x + 1u, step = 1, hi = lo + 1;
  while (hi < vh && (uint32_t)ld_relaxed(&a.huge_rec[hi].x) <= k) {
    lo = hi;
    step <<= 1;
    hi = lo + step;
  }
  if (hi > vh) hi = vh;
  while (hi - lo > 1) {
    const uint64_t mid = lo + ((hi - lo) >> 1);
    if ((uint32_t)ld_relaxed(&a.huge_rec[mid].x) <= k)
      lo = mid;
    else
      hi = mid;
  }
  return (uint32_t)lo;
}

// ---------------------------------------------------------------------------
// Phase 2: execution (Algorithm 2) with the cyclic distribution.
// ---------------------------------------------------------------------------
template <int B, class Op, bool M, class S>
__device__ void phase_lb(const Args &a, const Op &op, S &sm, Grid gr, int round, unsigned long long hc,
                         Entry<M> *qn, uint32_t *qn_cnt, uint32_t hs, Acc &acc) {
  using V = typename Op::val_t;
  const uint32_t vh = (uint32_t)(hc >> 32);
  const uint32_t e = (uint32_t)hc;
  if (vh == 0) return;
  // an overflowed reservation leaves the huge list inconsistent: skip (one
  // thread looks, so that the workgroup's waves agree: this phase's own pushes
  // may overflow meanwhile)
  if (threadIdx.x == 0) sm.owner = ld_relaxed(&a.ctl->overflow) <= (uint32_t)round;
  __syncthreads();
  if (sm.owner) return;
  const uint64_t T = (uint64_t)gr.n * B;
  const uint32_t lane = lane_id();
  const uint64_t g = (uint64_t)gr.id * B + threadIdx.x;
  const uint32_t tag = (uint32_t)round + 1u;
  Pusher<Entry<M>> pu{sm.pbuf[threadIdx.x / kWave], 0u, qn, qn_cnt};
  uint64_t pt = a.profile ? (uint64_t)wall_clock64() : 0;
  // slot u of a pass: huge edge k (if active) -> CSR position, source, source value
  auto take = [&](uint64_t k, bool on, bool &act, int32_t &pos, int32_t &src, V &sv) {
    act = on;
    pos = 0;
    src = 0;
    sv = V(0);
    if (on) {
      const int4 r = ld_rec(&a.huge_rec[owner_of(a, vh, hs, (uint32_t)k)]);
      pos = r.y + (int32_t)((uint32_t)k - (uint32_t)r.x);
      src = r.z;
      sv = from_bits<V>(r.w);
    }
    acc.edges_lb += on;
  };
  bool act[kU];
  int32_t pos[kU], src[kU];
  V s[kU];
  if (!a.blocked) {
    // cyclic: thread g takes huge edges g, g + T, g + 2T, ...; kU of them per
    // pass, so a wavefront's lanes read consecutive CSR entries
    for (uint64_t k0 = g - lane; k0 < e; k0 += kU * T) {
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const uint64_t k = k0 + lane + (uint64_t)u * T;
        take(k, k < e, act[u], pos[u], src[u], s[u]);
      }
      edges<Op, M>(act, pos, s, src, op, a, tag, round, pu, acc, (int32_t)g);
    }
  } else {
    // blocked (the alternative of Section 4.1): thread g takes the run
    // [g * c, (g + 1) * c) of c = ceil(e / T) consecutive huge edges
    const uint64_t c = (e + T - 1) / T;
    for (uint64_t j0 = 0; j0 < c; j0 += kU) {
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const uint64_t j = j0 + (uint64_t)u, k = g * c + j;
        take(k, j < c && k < e, act[u], pos[u], src[u], s[u]);
      }
      edges<Op, M>(act, pos, s, src, op, a, tag, round, pu, acc, (int32_t)g);
    }
  }
  settle_hot<B>(a, op, round, pu, acc);
  if constexpr (Op::kPush) flush_phase<B>(a, sm, round, pu);
  prof_mark(a, acc, kProfLb, pt);
}

// PageRank update: r'(v) = (1-d)/n + d * (acc(v) + D/n), rounded to fp32; acc cleared.
template <int B>
__device__ void phase_pr_update(const Args &a, Grid gr, unsigned long long dangling_fix) {
  const double d = (double)a.damping;
  const double N = (double)a.n;
  const double base = (1.0 - d) / N + d * ((double)dangling_fix * kFixInv) / N;
  for (uint32_t v = gr.id * B + threadIdx.x; v < (uint32_t)a.n; v += gr.n * B) {
    const double x = (double)a.acc[v] * kFixInv;
    a.rank[v] = (float)(base + d * x);
    a.acc[v] = 0ull;
  }
}

// Wait until every memory operation this wave issued has completed; also a
// compiler barrier, so no load or store moves across it.
__device__ __forceinline__ void wait_memory() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory"); }

// Bounded wait of thread 0 until *w reaches target.  Returns false if the
// launch was aborted or this wait outlasted timeout_ticks (which then
// aborts it: every workgroup leaves at its next barrier).
__device__ __forceinline__ bool bar_wait(const Args &a, unsigned long long *w, unsigned long long target, int round) {
  Ctl *c = a.ctl;
  const uint64_t t0 = (uint64_t)wall_clock64();
  unsigned long long seen;
  for (uint32_t look = 0; (seen = ld_relaxed(w)) < target; ++look) {
    __builtin_amdgcn_s_sleep(1);
    if (look % 16 != 15) continue;  // the rest costs another round trip
    if (ld_relaxed(&c->abort)) return false;
    if ((uint64_t)wall_clock64() - t0 > a.timeout_ticks) {
      st_relaxed(&c->diag_seen, seen);
      st_relaxed(&c->diag_target, target);
      st_relaxed(&c->diag_round, (uint32_t)round);
      st_relaxed(&c->abort, 1u);
      return false;
    }
  }
  return true;
}

// Grid-wide barrier among the members of the persistent launch.  Every wave
// first waits until its own memory operations have completed; thread 0 then
// arrives on its XCD's counter, the XCD's last arrival on the root counter,
// the last of those opens the generation word, which everybody watches.
// Counters only grow, so nothing is reset between barriers.
//
// Two kinds.  Light: no cache maintenance.  For data that one phase writes
// and a later one reads through agent-scope accesses only: worklists, huge
// records, chunk index, counters, and label words (updated by atomics).  Such
// an access is performed at the level the XCDs share, so once the writer has
// waited for it and arrived, a reader past the barrier sees it.  Plain loads
// of a label may still return a value from an earlier round, which is why
// operators read labels with agent-scope loads (they cost what plain loads
// do: 248-250 G random 8-byte reads/s from a table that the L2 holds, either
// way).  Two plain readers across light barriers do with such an old value:
// k-core's bitmap of hubs, which only chooses between two ways to count a
// decrement, and the build of a filter bitmap, whose labels change in one
// direction, so that an old one leaves a bit clear and the label is read.
// (Values from before the launch are never seen: a kernel starts with the
// caches invalidated.)  Full: with an agent-scope release by each XCD's last
// arrival (the L2 write-back covers every line of that L2 whichever CU wrote it) and an
// agent-scope acquire by every workgroup, for phases that exchange data by
// plain loads and stores (PageRank, filter bitmaps, serving).  The acquires
// of the workgroups of one XCD run one after the other: with them the barrier
// took 3.5 us among 128 workgroups, 6.7 among 512 and 11.3 among 1,024, without
// 2.3, 3.0 and 3.9.
template <bool kFull, class S>
__device__ bool grid_barrier(const Args &a, S &sm, Grid gr, unsigned long long &epoch, int round,
                             bool sys = false) {
  wait_memory();
  __syncthreads();
  if constexpr (!kFull) {
    if (gr.n == 1) return true;  // a lone workgroup
  }
  if (threadIdx.x == 0) {
    unsigned long long *b = a.bar;
    const unsigned long long target = epoch + 1;
    // few members (and no release to share) arrive on one counter directly
    // (its own: a launch may use both kinds of barrier): 32 of them meet in 1.6
    // us so, in 2.1 by way of the XCDs' counters, 64 in 2.0 and 2.2, 128 in 2.8
    // and 2.3
    if (!kFull && gr.n <= 48) {
      if ((add_relaxed(&b[kBarFlat], 1ull) + 1) % gr.n == 0) st_relaxed(&b[kBarGen], target);
    } else if ((add_relaxed(&b[kBarXcdArrive + (size_t)kBarStride * gr.xcd], 1ull) + 1) % gr.xcd_n == 0) {
      // the XCD's last arrival releases every store its members made before
      // arriving; `sys`: to the host as well (stores into host memory)
      if constexpr (kFull) {
        if (sys)
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");
        else
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      }
      const unsigned long long o2 = add_relaxed(&b[kBarRoot], 1ull);
      if ((o2 + 1) % gr.n_xcd == 0) st_relaxed(&b[kBarGen], target);
    }
    const bool ok = bar_wait(a, &b[kBarGen], target, round);
    if constexpr (kFull) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    sm.flag = ok ? 1 : 0;
  }
  __syncthreads();
  ++epoch;
  return sm.flag != 0;
}

template <bool M>
__device__ __forceinline__ const Entry<M> *round_frontier(const Args &a, int r) {
  if (a.all_rounds || (r == 0 && a.identity_first)) return nullptr;
  return (const Entry<M> *)((r & 1) ? a.q1 : a.q0);
}
template <bool M>
__device__ __forceinline__ Entry<M> *round_next(const Args &a, int r) {
  return (Entry<M> *)((r & 1) ? a.q0 : a.q1);
}

__device__ __forceinline__ uint32_t round_size(const Args &a, int r) {
  if (a.all_rounds) return (uint32_t)a.n;
  if (r == 0) return a.nfront0;
  const uint32_t c = ld_relaxed(&a.ctl->qcount[r % 3].v);
  return c < a.qcap ? c : a.qcap;
}

// The huge threshold of a round: the configured one, or with the small-round
// rule small_threshold while the worklist has fewer entries than launched
// threads.
__device__ __forceinline__ int64_t round_threshold(const Args &a, uint32_t nF, uint64_t T) {
  if (a.adaptive && (uint64_t)nF < T) return a.small_threshold;
  return a.threshold;
}

// Clear the counters ahead (nobody reads or writes them this round).
__device__ __forceinline__ void clear_ahead(const Args &a, int r) {
  st_relaxed(&a.ctl->chunk[(r + 1) % 3].v, 0ull);
  st_relaxed(&a.ctl->qcount[(r + 2) % 3].v, 0u);
  st_relaxed(&a.ctl->huge[(r + 1) & 1].v, 0ull);
  st_relaxed(&a.ctl->dangling[(r + 1) & 1].v, 0ull);
}

// Membership of the persistent launch.  The grid may be larger than what the
// device can hold at once, so co-residency is not assumed: every workgroup
// takes a ticket from its XCD's counter when it starts (one counter for all
// would take 12 ns per workgroup, 10 us for 800).  The XCDs' first ticket
// holders elect a leader, which closes membership (sets the counters' top
// bits) once all workgroups have joined or no new one has joined for
// join_window_ticks, and publishes the member counts.  A workgroup whose
// ticket shows the closed bit is not a member and leaves at once.  Members are
// running when they join and never leave before the end, so every barrier
// among them completes.  Returns false for a non-member; *gr gets (index,
// member count, XCD, members on that XCD, XCDs in use).  Indices go round the
// XCDs from the last to the first: all first tickets, then all second ones, and
// so on.  Index 0 has the lowest vertices in a phase over all of them, often the
// longest lists, and a chain of loads takes 4 to 5 % longer on XCD 0 than
// elsewhere (pull PageRank in bins, TWC only, 20 iterations: RMAT-20 16.3 ms with
// index 0 there, 15.8 with it on XCD 7; a star of 200,001 vertices 2,530 and 2,420
// us).
template <class S>
__device__ bool join_members(const Args &a, S &sm, Grid *gr) {
  constexpr unsigned long long kClosed = 1ull << 63;
  if (threadIdx.x < kWave) {  // the first wavefront; lane k looks after XCD k's counter
    Ctl *c = a.ctl;
    const uint32_t lane = lane_id();
    const uint32_t x = xcd_id();
    unsigned long long t = 0;
    if (lane == 0) t = add_relaxed(&a.bar[kBarXcdMembers + (size_t)kBarStride * x], 1ull);
    t = __shfl(t, 0);
    const bool member = (t & kClosed) == 0;
    uint32_t lead = 1;
    if (lane == 0 && member && t == 0) lead = add_relaxed(&c->leader, 1u);
    lead = __shfl(lead, 0);
    if (member && lead == 0) {
      unsigned long long *mine = &a.bar[kBarXcdMembers + (size_t)kBarStride * (lane % kBarXcds)];
      unsigned long long seen = 0, cnt = 0;
      uint64_t t_last = (uint64_t)wall_clock64();
      if (lane == 0) st_relaxed(&c->t_begin, (unsigned long long)t_last);
      for (;;) {
        cnt = lane < (uint32_t)kBarXcds ? ld_relaxed(mine) : 0ull;
        unsigned long long tot = cnt;
#pragma unroll
        for (int d = kBarXcds / 2; d > 0; d >>= 1) tot += __shfl_xor(tot, d);
        tot = __shfl(tot, 0);
        if (tot >= (unsigned long long)gridDim.x) break;
        const uint64_t now = (uint64_t)__shfl((unsigned long long)wall_clock64(), 0);
        if (tot != seen) {
          seen = tot;
          t_last = now;
        } else if (now - t_last > a.join_window_ticks) {
          if (lane < (uint32_t)kBarXcds)
            cnt = __hip_atomic_fetch_or(mine, kClosed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
      uint32_t n = (uint32_t)cnt;
      if (lane < (uint32_t)kBarXcds) st_relaxed(&c->xcd_members[lane], n);
#pragma unroll
      for (int d = kBarXcds / 2; d > 0; d >>= 1) n += __shfl_xor(n, d);
      wait_memory();  // the counts are in memory before the total announces them
      if (lane == 0) st_relaxed(&c->n_members, n);
    }
    uint32_t n = 0, cnt = 0;
    if (member) {
      while ((n = ld_relaxed(&c->n_members)) == 0) __builtin_amdgcn_s_sleep(1);
      cnt = lane < (uint32_t)kBarXcds ? ld_relaxed(&c->xcd_members[lane]) : 0u;
    }
    // members before this one: those with smaller tickets, and equal ones on later XCDs
    const uint32_t tk = (uint32_t)t;
    uint32_t before = min(cnt, tk) + (lane > x && cnt > tk ? 1u : 0u);
#pragma unroll
    for (int d = kBarXcds / 2; d > 0; d >>= 1) before += __shfl_xor(before, d);
    const uint32_t used = (uint32_t)__popcll(__ballot(cnt != 0));
    const uint32_t xn = __shfl(cnt, (int)x);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    if (lane == 0) {
      sm.flag = member ? 1 : 0;
      sm.ticket = before;
      sm.members = n;
      sm.xcd = x;
      sm.xcd_n = xn;
      sm.n_xcd = used;
    }
  }
  __syncthreads();
  const bool member = sm.flag != 0;
  gr->id = sm.ticket;
  gr->n = sm.members;
  gr->xcd = sm.xcd;
  gr->xcd_n = sm.xcd_n;
  gr->n_xcd = sm.n_xcd;
  __syncthreads();
  return member;
}

// ---------------------------------------------------------------------------
// Kernels.
// ---------------------------------------------------------------------------

// The control block before a launch (one thread).
__device__ void reset_ctl(Ctl *c) {
  for (int k = 0; k < 3; ++k) {
    c->qcount[k].v = 0;
    c->chunk[k].v = 0;
  }
  for (int k = 0; k < 3; ++k)
    for (int x = 0; x < kStatXcds; ++x) c->tile_dangling[k][x].v = 0;
  for (int k = 0; k < 2; ++k) {
    c->huge[k].v = 0;
    c->dangling[k].v = 0;
    c->filt_count[k].v = 0;
  }
  c->overflow = 0xffffffffu;
  c->abort = 0;
  c->rounds = 0;
  for (int x = 0; x < kStatXcds; ++x)
    for (int k = 0; k < kStats; ++k) c->stat[x][k].v = 0;
  c->leader = 0;
  c->n_members = 0;
  c->diag_seen = c->diag_target = 0;
  c->diag_round = 0;
  c->threshold_used = 0;
  for (int k = 0; k < kProfParts; ++k) c->prof[k] = 0;
  c->t_init = c->t_begin = c->t_rounds = c->t_end = 0;
}

// Vertex v's label before a traversal.
template <class T>
__device__ __forceinline__ void init_label(const Args &a, int op, T v) {
  if (op == OP_BFS) st_relaxed(&a.level[v], (int32_t)v == a.source ? 0 : kInf);
  if (op == OP_SSSP)
    st_relaxed(&a.word[v], (unsigned long long)(uint32_t)((int32_t)v == a.source ? 0 : kInf) << 32);
  if (op == OP_CC) st_relaxed(&a.word[v], (unsigned long long)v << 32);
  if (op == OP_KCORE) {  // the wavefront's lanes hold 64 consecutive vertices from a multiple of 64 on
    const int32_t deg = a.off[v + 1] - a.off[v];
    st_relaxed(&a.level[v], deg);
    const unsigned long long hot = __ballot(deg >= kHotDegree);
    const uint32_t lane = lane_id(), x = (uint32_t)v / kWave * 2u + lane;
    if (lane < 2 && (a.hot_shift == 5 || x == 0) && x < ((uint32_t)a.n + 31u) / 32u)
      st_relaxed(&a.hot[x], (uint32_t)(hot >> (32 * lane)));
  }
  if (op == OP_PR) {
    a.rank[v] = 1.0f / (float)a.n;
    a.acc[v] = 0ull;
  }
}

__global__ void k_clear(Args a) {
  const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  for (size_t i = t; i < kBarWords; i += gridDim.x * blockDim.x) a.bar[i] = 0ull;
  if (t == 0) reset_ctl(a.ctl);
}

__global__ void k_init(Args a, int op) {
  const uint32_t stride = gridDim.x * blockDim.x;
  const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t == 0) {
    const unsigned long long now = (unsigned long long)wall_clock64();
    reset_ctl(a.ctl);
    a.ctl->t_init = now;
  }
  for (uint32_t v = t; v < (uint32_t)a.n; v += stride) init_label(a, op, v);
  for (size_t i = t; i < kBarWords; i += stride) a.bar[i] = 0ull;
  if (t == 0) {
    if (a.source >= 0 && op != OP_RECORD) ((int32_t *)a.q0)[0] = a.source;
  }
}

__global__ void k_finish(Args a, int op) {
  const uint32_t stride = gridDim.x * blockDim.x;
  for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < (uint32_t)a.n; v += stride)
    a.out[v] = op == OP_KCORE ? (int32_t)(a.level[v] >= a.kcore_k) : (int32_t)(a.word[v] >> 32);
}

// Batch set-up: every label of every query to INF, the first worklist (query
// q's source is entry q; the launch gives it label 0), barrier words and
// control block.
__global__ void k_init_batch(Args a, int op) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t == 0) {
    const unsigned long long now = (unsigned long long)wall_clock64();
    reset_ctl(a.ctl);
    a.ctl->t_init = now;
  }
  for (size_t i = t; i < (size_t)a.nlabels; i += stride) {
    if (op == OP_BFS) a.level[i] = kInf;
    if (op == OP_SSSP) a.word[i] = (unsigned long long)(uint32_t)kInf << 32;
  }
  for (size_t q = t; q < (size_t)a.nq; q += stride)
    ((unsigned long long *)a.q0)[q] = ((unsigned long long)q << 32) | (uint32_t)a.qsrc[q];
  for (size_t i = t; i < kBarWords; i += stride) a.bar[i] = 0ull;
}

// Batch outputs: query blockIdx.y, its vertices strided over blockIdx.x.  After
// a launch that was abandoned or did not converge, which the call reports as
// an error, none: host arrays keep what they held.
__global__ void k_finish_batch(Args a, int op) {
  const Ctl *c = a.ctl;
  if (c->abort || c->overflow != 0xffffffffu || c->qcount[c->rounds % 3].v != 0) return;
  const int32_t q = blockIdx.y;
  const int32_t n = a.qn[q];
  const long long base = a.qlbase[q];
  int32_t *out = a.qout[q];
  for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x)
    out[v] = op == OP_BFS ? a.level[base + v] : (int32_t)(a.word[base + v] >> 32);
}

// The set-up a persistent launch does itself, followed by a grid barrier.
template <int B, class Op, bool M>
__device__ __forceinline__ void set_up(const Args &a, Grid gr) {
  const uint32_t t = gr.id * B + threadIdx.x, stride = gr.n * B;
  if constexpr (M) {
    for (uint32_t q = t; q < (uint32_t)a.nq; q += stride) {
      const long long l = a.qoff[q] + a.qsrc[q];
      if constexpr (std::is_same<Op, OpBFS>::value)
        st_relaxed(&a.level[l], 0);
      else
        st_relaxed(&a.word[l], 0ull);
    }
  } else if (!a.apart) {
    if (t == 0 && a.source >= 0) st_relaxed((int32_t *)a.q0, a.source);
    for (uint32_t v = t; v < (uint32_t)a.n; v += stride) init_label(a, (int)Op::kKind, v);
  }
  if (a.clear_ctl) {
    for (size_t i = t; i < kBarWords; i += stride) a.clear_bar[i] = 0ull;
    if (t == B - 1) reset_ctl(a.clear_ctl);
  }
}

// The labels of a converged single-query launch as int32 outputs.
template <int B, class Op>
__device__ __forceinline__ void write_out(const Args &a, Grid gr) {
  if constexpr (std::is_same<Op, OpBFS>::value) {
    if (a.out)  // the caller's output is host memory
      for (uint32_t v = gr.id * B + threadIdx.x; v < (uint32_t)a.n; v += gr.n * B) a.out[v] = ld_relaxed(&a.level[v]);
  } else if constexpr (std::is_same<Op, OpSSSP>::value || std::is_same<Op, OpCC>::value) {
    for (uint32_t v = gr.id * B + threadIdx.x; v < (uint32_t)a.n; v += gr.n * B)
      a.out[v] = (int32_t)(ld_relaxed(&a.word[v]) >> 32);
  } else if constexpr (Op::kKind == OP_KCORE) {
    for (uint32_t v = gr.id * B + threadIdx.x; v < (uint32_t)a.n; v += gr.n * B)
      a.out[v] = (int32_t)(ld_relaxed(&a.level[v]) >= a.kcore_k);
  }
}

// The end of a persistent launch, after the workgroup's statistics: the last
// workgroup to leave sums them up and writes the result block (a copy of the
// control block by the host took 8 to 10 us of a call).
template <class S>
__device__ __forceinline__ void leave(const Args &a, S &sm, Grid gr) {
  wait_memory();
  __syncthreads();
  if (threadIdx.x < kWave) {
    uint32_t last = 0;
    if (threadIdx.x == 0) {
      const unsigned long long o1 = add_relaxed(&a.bar[kBarXcdOut + (size_t)kBarStride * gr.xcd], 1ull);
      if (o1 + 1 == gr.xcd_n) last = add_relaxed(&a.bar[kBarRootOut], 1ull) + 1 == gr.n_xcd;
    }
    last = __shfl(last, 0);
    if (last) {
      Ctl *c = a.ctl;
      Result *o = a.result;
      const uint32_t lane = lane_id();
      if (lane < kStats) {
        unsigned long long t = 0;
#pragma unroll
        for (int x = 0; x < kStatXcds; ++x) t += ld_relaxed(&c->stat[x][lane].v);
        o->stat[lane] = t;
      }
      if (lane == 0) {
        const uint32_t rounds = ld_relaxed(&c->rounds);
        o->overflow = ld_relaxed(&c->overflow);
        o->abort = ld_relaxed(&c->abort);
        o->diag_round = ld_relaxed(&c->diag_round);
        o->diag_seen = ld_relaxed(&c->diag_seen);
        o->diag_target = ld_relaxed(&c->diag_target);
        o->rounds = rounds;
        o->n_members = gr.n;
        o->left = ld_relaxed(&c->qcount[rounds % 3].v);
        o->threshold_used = ld_relaxed(&c->threshold_used);
        o->t_init = ld_relaxed(&c->t_init);
        o->t_begin = ld_relaxed(&c->t_begin);
        o->t_rounds = ld_relaxed(&c->t_rounds);
        o->t_end = (unsigned long long)wall_clock64();
        o->done = 1;
      }
    }
  }
}

template <int B, class Op>
__global__ __launch_bounds__(B) void k_twc(Args a, Op op) {
  __shared__ Smem<B, Op> sm;
  if constexpr (Op::kHot) hot_clear<B>();
  Acc acc;
  const int r = a.round;
  const uint32_t nF = round_size(a, r);
  if (blockIdx.x == 0 && threadIdx.x == 0) clear_ahead(a, r);
  const Grid gr{blockIdx.x, gridDim.x};
  const int64_t thr = round_threshold(a, nF, (uint64_t)gr.n * B);
  phase_twc<B, Op, false>(a, op, sm, gr, r, round_frontier<false>(a, r), nF, round_next<false>(a, r),
                          &a.ctl->qcount[(r + 1) % 3].v,
                   &a.ctl->huge[r & 1].v, thr, hint_shift(a, thr, nF), acc);
  if constexpr (Op::kPR) flush_dangling<B, Op>(acc, sm, &a.ctl->dangling[r & 1].v);
  flush_stats<B, Op>(acc, sm, a.ctl);
}

template <int B, class Op>
__global__ __launch_bounds__(B) void k_lb(Args a, Op op) {
  __shared__ Smem<B, Op> sm;
  if constexpr (Op::kHot) hot_clear<B>();
  Acc acc;
  const int r = a.round;
  const unsigned long long hc = ld_relaxed(&a.ctl->huge[r & 1].v);
  const int64_t thr = round_threshold(a, round_size(a, r), (uint64_t)gridDim.x * B);
  phase_lb<B, Op, false>(a, op, sm, Grid{blockIdx.x, gridDim.x}, r, hc, round_next<false>(a, r),
                         &a.ctl->qcount[(r + 1) % 3].v,
                  hint_shift(a, thr, round_size(a, r)), acc);
  flush_stats<B, Op>(acc, sm, a.ctl);
}

template <int B>
__global__ __launch_bounds__(B) void k_pr_update(Args a) {
  phase_pr_update<B>(a, Grid{blockIdx.x, gridDim.x}, ld_relaxed(&a.ctl->dangling[a.round & 1].v));
  if (blockIdx.x == 0 && threadIdx.x == 0) st_relaxed(&a.ctl->rounds, (uint32_t)a.round + 1u);
}

// The filter bitmap (BFS: reached; CC: label 0): word x holds vertices
// [32x, 32x + 32).  Each wavefront of the members tests 64 consecutive
// vertices (coalesced loads), two of its lanes store the ballot's halves,
// and lane 0 adds the set bits to *count.
template <int B, class Op>
__device__ __forceinline__ void build_filter(const Args &a, Grid gr, unsigned long long *count) {
  const uint32_t n = (uint32_t)a.n;
  const uint32_t words = (n + 31u) / 32u;
  const uint32_t lane = lane_id();
  const uint32_t nwaves = (uint32_t)gr.n * (B / kWave);
  unsigned long long set = 0;
  for (uint32_t base = ((uint32_t)gr.id * (B / kWave) + threadIdx.x / kWave) * kWave; base < n;
       base += nwaves * kWave) {
    const uint32_t v = base + lane;
    const unsigned long long m = __ballot(v < n && Filtered<Op>::bit(a, v));
    const uint32_t x = base / 32u + lane;
    if (lane < 2 && x < words) a.vbits[x] = (uint32_t)(m >> (32 * lane));
    set += (unsigned long long)__popcll(m);
  }
  if (lane == 0 && set) add_relaxed(count, set);
}

// Waves per SIMD of k_persistent: k-core in workgroups of 64 keeps five (20
// workgroups per CU, of which grids up to 5,120 are accepted).
template <int B, class Op, bool F>
constexpr int waves_wanted() {
  return Op::kHot && B == kWave && !F && ALB_WAVES_PER_EU < 5 ? 5 : ALB_WAVES_PER_EU;
}

// F: BFS or CC with the filter bitmap (a kernel of its own, so that every
// other launch runs code without it).
template <int B, class Op, bool M, bool F = false>
__global__ __launch_bounds__(B) __attribute__((amdgpu_waves_per_eu(waves_wanted<B, Op, F>()))) void k_persistent(
    Args a, Op op) {
  __shared__ Smem<B, Op, M> sm;
  Acc acc;
  Grid gr;
  bool joined;
  if constexpr (F) {  // the filtering kernel has two operator types' phases: everything inlined
    [[clang::always_inline]] joined = join_members(a, sm, &gr);
  } else {
    joined = join_members(a, sm, &gr);
  }
  if (!joined) return;
  if (a.threshold < 0) a.threshold = (int64_t)gr.n * B;  // the launched thread count (the paper's rule)
  unsigned long long epoch = 0, prof_last = 0;
  set_up<B, Op, M>(a, gr);
  if constexpr (Op::kHot) hot_clear<B>();
  bool ok;
  if constexpr (F) {
    [[clang::always_inline]] ok = grid_barrier<Op::kPR>(a, sm, gr, epoch, 0);
  } else {
    ok = grid_barrier<Op::kPR>(a, sm, gr, epoch, 0);
  }
  if (gr.id == 0 && threadIdx.x == 0) st_relaxed(&a.ctl->t_rounds, (unsigned long long)wall_clock64());
  uint64_t reached = 0;  // BFS: vertices in the worklists so far (each is in exactly one round's)
  bool filtered = false;  // the filter bitmap is in use
  int r = 0;
  for (; ok && r < a.max_rounds; ++r) {
    const uint32_t over = ld_relaxed(&a.ctl->overflow);  // (both loads in flight together)
    const uint32_t nF = round_size(a, r);
    if (over < (uint32_t)r) {  // set in an earlier round: seen by all alike
      ok = false;
      break;
    }
    if (nF == 0) break;
    if constexpr (F) {
      // BFS: once half of the vertices have been reached (every member
      // decides alike from the worklist sizes), most edges lead to reached
      // vertices: build the bitmap once and filter from this round on.
      // CC: from round 1 on, rebuild the bitmap of label-0 vertices at each
      // round's start and filter once they are at least half of all.
      // k-core: the same from round 0 on, with the vertices below k.
      bool build = false;
      if constexpr (std::is_same<Op, OpBFS>::value) {
        reached += nF;
        build = !filtered && 2 * reached >= (uint64_t)a.n;
      } else if constexpr (std::is_same<Op, OpCC>::value) {
        build = r >= 1;
      } else {
        build = true;
      }
      // the next round's count: nobody reads it before then (this round's
      // members read [r & 1] right after the build's barrier)
      if (gr.id == 0 && threadIdx.x == 0) st_relaxed(&a.ctl->filt_count[(r + 1) & 1].v, 0ull);
      if (build) {
        build_filter<B, Op>(a, gr, &a.ctl->filt_count[r & 1].v);
        [[clang::always_inline]] ok = grid_barrier<true>(a, sm, gr, epoch, r);
        if (!ok) break;
        if constexpr (std::is_same<Op, OpBFS>::value)
          filtered = true;
        else
          filtered = 2 * ld_relaxed(&a.ctl->filt_count[r & 1].v) >= (unsigned long long)a.n;
      }
    }
    const bool tl = gr.id == 0 && threadIdx.x == 0 && r < kTimeline;
    if (gr.id == 0 && threadIdx.x == 0) clear_ahead(a, r);
    if (tl) a.ctl->tl[4 * r] = (unsigned long long)wall_clock64();
    Entry<M> *qn = round_next<M>(a, r);
    uint32_t *qn_cnt = &a.ctl->qcount[(r + 1) % 3].v;
    const int64_t thr = round_threshold(a, nF, (uint64_t)gr.n * B);
    // batch with per-query thresholds: chunk index sized for the smallest one
    const uint32_t hs = hint_shift(a, M && a.qthr ? a.qthr_min : thr, nF);
    if constexpr (F) {  // two operator types here: both phases inlined
      if (filtered) {
        using FOp = typename Filtered<Op>::type;
        const FOp fop = Filtered<Op>::make(op, a);
        [[clang::always_inline]] phase_twc<B, FOp, M>(a, fop, sm, gr, r, round_frontier<M>(a, r), nF, qn, qn_cnt,
                                                      &a.ctl->huge[r & 1].v, thr, hs, acc);
      } else {
        [[clang::always_inline]] phase_twc<B, Op, M>(a, op, sm, gr, r, round_frontier<M>(a, r), nF, qn, qn_cnt,
                                                     &a.ctl->huge[r & 1].v, thr, hs, acc);
      }
    } else {
      phase_twc<B, Op, M>(a, op, sm, gr, r, round_frontier<M>(a, r), nF, qn, qn_cnt, &a.ctl->huge[r & 1].v, thr, hs,
                          acc);
    }
    if constexpr (Op::kPR) flush_dangling<B, Op>(acc, sm, &a.ctl->dangling[r & 1].v);
    uint64_t pb = a.profile ? (uint64_t)wall_clock64() : 0;
    if constexpr (F) {
      [[clang::always_inline]] ok = grid_barrier<Op::kPR>(a, sm, gr, epoch, r);
    } else {
      ok = grid_barrier<Op::kPR>(a, sm, gr, epoch, r);
    }
    if (!ok) break;
    prof_mark(a, acc, kProfBarrier, pb);
    const unsigned long long hc = ld_relaxed(&a.ctl->huge[r & 1].v);
    if (tl) {
      a.ctl->tl[4 * r + 1] = (unsigned long long)wall_clock64();
      a.ctl->tl[4 * r + 3] = (unsigned long long)nF | ((hc >> 32) << 32);
    }
    if ((hc >> 32) != 0) {  // the execution phase runs only when there is imbalance to fix
      if constexpr (F) {
        if (filtered) {
          using FOp = typename Filtered<Op>::type;
          const FOp fop = Filtered<Op>::make(op, a);
          [[clang::always_inline]] phase_lb<B, FOp, M>(a, fop, sm, gr, r, hc, qn, qn_cnt, hs, acc);
        } else {
          [[clang::always_inline]] phase_lb<B, Op, M>(a, op, sm, gr, r, hc, qn, qn_cnt, hs, acc);
        }
      } else {
        phase_lb<B, Op, M>(a, op, sm, gr, r, hc, qn, qn_cnt, hs, acc);
      }
      pb = a.profile ? (uint64_t)wall_clock64() : 0;
      if constexpr (F) {
        [[clang::always_inline]] ok = grid_barrier<Op::kPR>(a, sm, gr, epoch, r);
      } else {
        ok = grid_barrier<Op::kPR>(a, sm, gr, epoch, r);
      }
      if (!ok) break;
      prof_mark(a, acc, kProfBarrier, pb);
    }
    if (tl) a.ctl->tl[4 * r + 2] = (unsigned long long)wall_clock64();
    if (a.prof_wg) prof_round_edges(a, acc, prof_last, gr.id, r);
    if constexpr (Op::kPR) {
      phase_pr_update<B>(a, gr, ld_relaxed(&a.ctl->dangling[r & 1].v));
      if (!grid_barrier<true>(a, sm, gr, epoch, r)) break;
    }
  }
  if (gr.id == 0 && threadIdx.x == 0) {
    st_relaxed(&a.ctl->rounds, (uint32_t)r);
    st_relaxed(&a.ctl->threshold_used, (long long)a.threshold);
    st_relaxed(&a.ctl->t_end, (unsigned long long)wall_clock64());
  }
  if constexpr (!M) {
    // (not after the last round allowed, if it left work: the call returns an error then)
    if (ok && !a.apart &&
        (r < a.max_rounds || (ld_relaxed(&a.ctl->overflow) == 0xffffffffu && round_size(a, r) == 0)))
      write_out<B, Op>(a, gr);
  }
  if constexpr (F) {
    [[clang::always_inline]] flush_stats<B, Op>(acc, sm, a.ctl);
  } else {
    flush_stats<B, Op>(acc, sm, a.ctl);
  }
  leave(a, sm, gr);
}

// ---------------------------------------------------------------------------
// Continuous serving: one persistent batch launch that queries join between
// rounds.  Round r is two phases, as a batch's:
//   phase 1  inspection and TWC over round r's worklist (recording, per
//            slot, that it had an entry this round); workgroup 0 then takes
//            the requests the host has published into their slots (tables
//            only) and decides whether the launch ends;
//   -------- grid barrier
//   phase 2  workgroup 0 marks the active slots without an entry this round
//            as finished (their labels have been final since round r - 1);
//            every member initialises the newly admitted slots' labels and
//            writes the labels of the slots finished in round r - 1 to
//            open_out as int32; workgroup 0 appends the new sources to round
//            r + 1's worklist; then the cyclic phase of round r;
//   -------- grid barrier
//   workgroup 0 publishes the slots converted this round to the host.
// A request published while others are on the device thus starts at the
// next round boundary, beside them.  Everything member 0 decides for round r
// (admissions, exit) sits in [r & 1] entries: with only two barriers per
// round a slow member may still read round r's entry while member 0 already
// writes round r + 1's.
// ---------------------------------------------------------------------------
template <class T>
__device__ __forceinline__ T ld_sys(T *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
template <class T>
__device__ __forceinline__ void st_sys(T *p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Workgroup 0, thread 0, at the end of round r's phase 1: take the published
// requests (at most the ring's size; the host bounds them by its free slots)
// into their slots' tables, list them for phase 2 (admit_n[r & 1]), and
// decide whether the launch ends after this round's first barrier.
__device__ void open_admit(const Args &a, int r, uint32_t nF) {
  Ctl *c = a.ctl;
  OpenShared *sh = a.open;
  const unsigned long long tail = ld_sys(&sh->tail);
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "");  // the entries below were written before the tail
  const unsigned long long head = c->open_head;
  int32_t *admit = a.q_admit + (size_t)(r & 1) * kOpenRing;
  uint32_t k = 0;
  for (unsigned long long i = head; i < tail && k < (uint32_t)kOpenRing; ++i, ++k) {
    OpenReq *q = &sh->req[i % kOpenRing];
    const int32_t slot = ld_sys(&q->slot);
    if (slot < 0 || slot >= a.nslots) {  // cannot happen with a well-formed ring: stop taking requests
      flag_overflow(c, r);
      break;
    }
    admit[k] = slot;
    ((long long *)a.qoff)[slot] = ld_sys(&q->qoff);
    ((long long *)a.qlbase)[slot] = ld_sys(&q->lbase);
    ((int32_t *)a.qsrc)[slot] = ld_sys(&q->src);
    ((int32_t *)a.qn)[slot] = ld_sys(&q->n);
    a.q_unit[slot] = ld_sys(&q->unit);
    a.q_out[slot] = (int32_t *)ld_sys(&q->out);
    a.q_last[slot] = r;  // not finished in this round's phase 2: its source is in round r + 1's worklist
    a.q_active[slot] = 1;
  }
  c->open_head = head + k;
  st_sys(&sh->head, head + k);
  c->admit_n[r & 1] = k;
  c->open_active += k;
  uint32_t ex = 0;
  const bool idle = k == 0 && nF == 0 && c->open_active == 0 && c->conv_n[r & 1] == 0;
  if (!idle) {
    c->idle_since = 0;
  } else {
    const uint64_t now = (uint64_t)wall_clock64();
    if (ld_sys(&sh->stop)) ex = 1;
    if (c->idle_since == 0) c->idle_since = now;
    else if (now - c->idle_since > a.idle_ticks) ex = 1;
    __builtin_amdgcn_s_sleep(8);  // idle: poll the ring less often
  }
  c->open_exit[r & 1] = ex;
}

// Workgroup 0 after round r's first barrier: an active slot without an
// entry in round r's worklist has finished.  It is listed for round r + 1's
// conversion (q_conv[(r + 1) & 1], conv_n[(r + 1) & 1]).
template <int B>
__device__ void open_complete(const Args &a, int r, uint32_t *s_cnt) {
  Ctl *c = a.ctl;
  int32_t *list = a.q_conv + (size_t)((r + 1) & 1) * kOpenRing;
  if (threadIdx.x == 0) *s_cnt = 0;
  __syncthreads();
  for (int32_t q = threadIdx.x; q < a.nslots; q += B) {
    if (a.q_active[q] && ld_relaxed(&a.q_last[q]) != r) {
      a.q_active[q] = 0;
      list[atomicAdd(s_cnt, 1u)] = q;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    c->conv_n[(r + 1) & 1] = *s_cnt;
    c->open_active -= *s_cnt;
  }
  __syncthreads();
}

// Every member in round r's phase 2: the slots admitted in round r get their
// labels (INF, the source 0); the slots finished in round r - 1 get theirs
// written as int32 (SSSP: the distance half of the label word; BFS: the
// level) into the caller's pinned output, or into open_out.  Workgroup 0 then appends the new sources to round
// r + 1's worklist.
template <class Op>
__device__ void open_prepare(const Args &a, Grid gr, int B, int r, uint32_t k, uint32_t nc) {
  const int32_t *admit = a.q_admit + (size_t)(r & 1) * kOpenRing;
  for (uint32_t i = 0; i < k; ++i) {
    const int32_t slot = admit[i];
    const long long base = a.qlbase[slot];
    const long long sl = a.qoff[slot] + a.qsrc[slot];
    const int32_t n = a.qn[slot];
    for (int32_t v = (int32_t)(gr.id * B + threadIdx.x); v < n; v += (int32_t)(gr.n * B)) {
      const long long l = base + v;
      if constexpr (std::is_same<Op, OpBFS>::value)
        a.level[l] = l == sl ? 0 : kInf;
      else
        a.word[l] = l == sl ? 0ull : (unsigned long long)(uint32_t)kInf << 32;
    }
  }
  const int32_t *conv = a.q_conv + (size_t)(r & 1) * kOpenRing;
  for (uint32_t i = 0; i < nc; ++i) {
    const int32_t slot = conv[i];
    const long long base = a.qlbase[slot];
    const int32_t n = a.qn[slot];
    int32_t *dst = a.q_out[slot];  // the caller's pinned array, else the lane's output area
    if (!dst) dst = a.open_out + base;
    for (int32_t v = (int32_t)(gr.id * B + threadIdx.x); v < n; v += (int32_t)(gr.n * B)) {
      if constexpr (std::is_same<Op, OpBFS>::value)
        dst[v] = a.level[base + v];
      else
        dst[v] = (int32_t)(a.word[base + v] >> 32);
    }
  }
  if (k && gr.id == 0 && threadIdx.x == 0) {
    unsigned long long *F = (unsigned long long *)(((r + 1) & 1) ? a.q1 : a.q0);
    const uint32_t at = add_relaxed(&a.ctl->qcount[(r + 1) % 3].v, k);  // beside the cyclic phase's pushes
    for (uint32_t i = 0; i < k; ++i) {
      const int32_t slot = admit[i];
      if (at + i < a.qcap)
        F[at + i] = ((unsigned long long)(uint32_t)slot << 32) | (uint32_t)a.qsrc[slot];
      else
        flag_overflow(a.ctl, r);
    }
  }
}

// Workgroup 0, thread 0, after round r's second barrier: the slots converted
// in round r go to the completion ring after a system-scope release, so
// that their int32 labels are in memory when the host copies them.
__device__ void open_publish(const Args &a, int r, uint32_t nc) {
  Ctl *c = a.ctl;
  OpenShared *sh = a.open;
  const int32_t *list = a.q_conv + (size_t)(r & 1) * kOpenRing;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");
  for (uint32_t j = 0; j < nc; ++j) st_sys(&sh->fin[(c->open_done + j) % kOpenRing], list[j]);
  c->open_done += nc;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");
  st_sys(&sh->done, c->open_done);
}

template <int B, class Op>
__global__ __launch_bounds__(B) __attribute__((amdgpu_waves_per_eu(ALB_WAVES_PER_EU))) void k_open(Args a, Op op) {
  __shared__ Smem<B, Op, true> sm;
  __shared__ uint32_t s_cnt;
  Acc acc;
  Grid gr;
  if (!join_members(a, sm, &gr)) return;
  if (a.threshold < 0) a.threshold = (int64_t)gr.n * B;
  if (gr.id == 0 && threadIdx.x == 0) st_sys(&a.open->live, 1u);
  unsigned long long epoch = 0;
  int r = 0;
  for (;; ++r) {
    if (ld_relaxed(&a.ctl->overflow) < (uint32_t)r) break;
    const uint32_t nF = round_size(a, r);
    const bool tl = gr.id == 0 && threadIdx.x == 0 && r < kTimeline;
    if (gr.id == 0 && threadIdx.x == 0) clear_ahead(a, r);
    if (tl) a.ctl->tl[4 * r] = (unsigned long long)wall_clock64();
    Entry<true> *qn = round_next<true>(a, r);
    uint32_t *qn_cnt = &a.ctl->qcount[(r + 1) % 3].v;
    const int64_t thr = round_threshold(a, nF, (uint64_t)gr.n * B);
    const uint32_t hs = hint_shift(a, thr, nF);
    if (nF)
      phase_twc<B, Op, true>(a, op, sm, gr, r, round_frontier<true>(a, r), nF, qn, qn_cnt, &a.ctl->huge[r & 1].v,
                             thr, hs, acc);
    if (gr.id == 0 && threadIdx.x == 0) open_admit(a, r, nF);
    if (!grid_barrier<true>(a, sm, gr, epoch, r)) break;
    if (ld_relaxed(&a.ctl->open_exit[r & 1])) break;
    if (gr.id == 0) open_complete<B>(a, r, &s_cnt);
    const uint32_t k = ld_relaxed(&a.ctl->admit_n[r & 1]);
    const uint32_t nc = ld_relaxed(&a.ctl->conv_n[r & 1]);
    open_prepare<Op>(a, gr, B, r, k, nc);
    const unsigned long long hc = nF ? ld_relaxed(&a.ctl->huge[r & 1].v) : 0ull;
    if (tl) {
      a.ctl->tl[4 * r + 1] = (unsigned long long)wall_clock64();
      a.ctl->tl[4 * r + 3] = (unsigned long long)nF | ((hc >> 32) << 32);
    }
    if ((hc >> 32) != 0) phase_lb<B, Op, true>(a, op, sm, gr, r, hc, qn, qn_cnt, hs, acc);
    // a round that wrote finished labels into host memory releases them at
    // system scope on every XCD before workgroup 0 publishes the slots
    if (!grid_barrier<true>(a, sm, gr, epoch, r, nc != 0)) break;
    if (tl) a.ctl->tl[4 * r + 2] = (unsigned long long)wall_clock64();
    if (nc && gr.id == 0 && threadIdx.x == 0) open_publish(a, r, nc);
  }
  if (gr.id == 0 && threadIdx.x == 0) {
    st_relaxed(&a.ctl->rounds, (uint32_t)r);
    st_relaxed(&a.ctl->threshold_used, (long long)a.threshold);
    st_relaxed(&a.ctl->t_end, (unsigned long long)wall_clock64());
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");
    st_sys(&a.open->live, 0u);
  }
  flush_stats<B, Op>(acc, sm, a.ctl);
}

// Continuous serving set-up: control block, barrier words, slot flags.
__global__ void k_init_open(Args a) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (size_t i = t; i < kBarWords; i += stride) a.bar[i] = 0ull;
  for (size_t i = t; i < (size_t)a.nslots; i += stride) {
    a.q_active[i] = 0;
    a.q_last[i] = -1;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    Ctl *c = a.ctl;
    reset_ctl(c);
    c->open_head = 0;
    c->admit_n[0] = c->admit_n[1] = 0;
    c->open_done = 0;
    c->open_active = 0;
    c->open_exit[0] = c->open_exit[1] = 0;
    c->conv_n[0] = c->conv_n[1] = 0;
    c->idle_since = 0;
  }
}

// ---------------------------------------------------------------------------
// Pull PageRank (the paper's pr, Section 5): each vertex v sums its
// in-neighbours' contributions c(u) = rank(u) / outdeg(u) over the transposed
// graph, so no atomic touches a destination label except for the edges of
// huge in-degree vertices.  Inspection and bins work on in-degrees: the TWC
// bins reduce each vertex's sum inside one workgroup, wavefront or lane and
// store it once; the huge vertices' in-edges take the cyclic distribution of
// Algorithm 2, each wavefront adds its lanes' contributions per vertex
// (segmented by the owning vertex) with one atomic per segment.  The sums use
// the same exact 64-bit fixed point as the push version, so both give
// bitwise the same ranks.
// ---------------------------------------------------------------------------
struct OpPRPull {  // type facts for Smem only; the pull phases do the work
  using val_t = float;
  static constexpr int kKind = OP_PR;
  struct pre_t {};
  static constexpr bool kPush = false, kNeedSrc = false, kRecord = false, kPR = true, kBatch = false, kHot = false;
};

// Fixed-point contributions of up to kU in-edges per lane, loads issued first.
__device__ __forceinline__ unsigned long long pull_edges(const Args &a, const bool (&act)[kU],
                                                         const int32_t (&pos)[kU]) {
  int32_t u[kU];
#pragma unroll
  for (int i = 0; i < kU; ++i) u[i] = a.tcol[act[i] ? pos[i] : 0];
  float c[kU];
#pragma unroll
  for (int i = 0; i < kU; ++i) c[i] = a.contrib[u[i]];
  unsigned long long x = 0;
#pragma unroll
  for (int i = 0; i < kU; ++i) x += act[i] ? to_fix(c[i]) : 0ull;
  return x;
}

template <int B>
__device__ unsigned long long block_sum(unsigned long long x, Smem<B, OpPRPull> &sm) {
#pragma unroll
  for (int d = kWave / 2; d > 0; d >>= 1) x += __shfl_xor(x, d);
  if (lane_id() == 0) sm.dred[threadIdx.x / kWave] = x;
  __syncthreads();
  unsigned long long t = 0;
#pragma unroll
  for (int j = 0; j < B / kWave; ++j) t += sm.dred[j];
  __syncthreads();
  return t;
}

template <int B>
__device__ void pull_gather(const Args &a, Smem<B, OpPRPull> &sm, Grid gr, int it, int64_t thr, uint32_t hs,
                            Acc &acc) {
  const int tid = threadIdx.x;
  const uint32_t lane = lane_id();
  const uint32_t nF = (uint32_t)a.n;
  Claims cl(gr, twc_chunk(nF, gr.n, B));
  for (bool first = true;; first = false) {
    if (!first && tid == 0) cl.next(&a.ctl->chunk[it % 3].v, nF, gr, B, sm.cbase, sm.clen);
    __syncthreads();
    const unsigned long long base = first ? cl.nxt : sm.cbase;
    const uint32_t C = first ? cl.len : sm.clen;
    if (base >= nF) break;
    const uint32_t i = (uint32_t)base + tid;
    const bool mine = tid < (int)C && i < nF;
    int32_t v = -1, beg = 0, deg = 0;
    if (mine) {
      v = (int32_t)i;
      beg = a.toff[v];
      deg = a.toff[v + 1] - beg;
    }
    // inspection by in-degree (Algorithm 1); huge vertices wait for phase 2
    const bool huge = deg > 0 && (int64_t)deg >= thr;
    reserve_huge(huge, v, beg, deg, 0, a, it, &a.ctl->huge[it & 1].v, hs, acc);
    if (huge) deg = 0;
    acc.frontier += mine;
    acc.edges_twc += (unsigned long long)deg;

    // workgroup bin: the workgroup sums one vertex's in-edges, then stores
    for (;;) {
      if (tid == 0) sm.owner = -1;
      __syncthreads();
      if (deg >= a.c_wg) sm.owner = tid;
      __syncthreads();
      const int32_t o = sm.owner;
      if (o < 0) break;
      if (tid == o) {
        sm.obeg = beg;
        sm.odeg = deg;
        sm.ov = v;
        deg = 0;
      }
      __syncthreads();
      const int32_t ob = sm.obeg, od = sm.odeg, ov = sm.ov;
      unsigned long long x = 0;
      for (int32_t j0 = 0; j0 < od; j0 += kU * B) {
        bool act[kU];
        int32_t pos[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          act[u] = j0 + u * B + tid < od;
          pos[u] = ob + j0 + u * B + tid;
        }
        x += pull_edges(a, act, pos);
      }
      x = block_sum<B>(x, sm);
      if (tid == 0) a.acc[ov] = x;
    }
    // wavefront bin: one wavefront sums one vertex's in-edges
    for (;;) {
      const unsigned long long mm = __ballot(deg >= a.c_wave && deg > 0);
      if (mm == 0ull) break;
      const int ld = __ffsll(mm) - 1;
      const int32_t ob = __shfl(beg, ld), od = __shfl(deg, ld), ov = __shfl(v, ld);
      if ((int)lane == ld) deg = 0;
      unsigned long long x = 0;
      for (int32_t j0 = 0; j0 < od; j0 += kU * kWave) {
        bool act[kU];
        int32_t pos[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          act[u] = j0 + u * kWave + (int32_t)lane < od;
          pos[u] = ob + j0 + u * kWave + (int32_t)lane;
        }
        x += pull_edges(a, act, pos);
      }
#pragma unroll
      for (int d = kWave / 2; d > 0; d >>= 1) x += __shfl_xor(x, d);
      if ((int)lane == ld) a.acc[ov] = x;
    }
    // thread bin: each lane sums its own short list (fewer than c_wave edges)
    if (deg > 0) {
      unsigned long long x = 0;
      for (int32_t j0 = 0; j0 < deg; j0 += kU) {
        bool act[kU];
        int32_t pos[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          act[u] = j0 + u < deg;
          pos[u] = beg + j0 + u;
        }
        x += pull_edges(a, act, pos);
      }
      a.acc[v] = x;
    }
    // vertices without in-edges keep the 0 the update phase left
  }
}

template <int B>
__device__ void pull_lb(const Args &a, Grid gr, unsigned long long hc, uint32_t hs, Acc &acc) {
  const uint32_t vh = (uint32_t)(hc >> 32);
  const uint32_t e = (uint32_t)hc;
  if (vh == 0 || ld_relaxed(&a.ctl->overflow) != 0xffffffffu) return;
  const uint64_t T = (uint64_t)gr.n * B;
  const uint32_t lane = lane_id();
  const uint64_t g = (uint64_t)gr.id * B + threadIdx.x;
  for (uint64_t k0 = g - lane; k0 < e; k0 += kU * T) {
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const uint64_t k = k0 + lane + (uint64_t)u * T;
      const bool act = k < e;
      int32_t v = -1;
      unsigned long long x = 0;
      if (act) {
        const int4 r = ld_rec(&a.huge_rec[owner_of(a, vh, hs, (uint32_t)k)]);
        v = r.z;
        x = to_fix(a.contrib[a.tcol[r.y + (int32_t)((uint32_t)k - (uint32_t)r.x)]]);
      }
      acc.edges_lb += act;
      // consecutive lanes hold consecutive huge edges, so lanes of one vertex
      // form one run: add each run with one atomic from its last lane
      unsigned long long incl = x;
#pragma unroll
      for (int d = 1; d < kWave; d <<= 1) {
        const unsigned long long y = __shfl_up(incl, d);
        if ((int)lane >= d) incl += y;
      }
      const int32_t vprev = __shfl_up(v, 1), vnext = __shfl_down(v, 1);
      const unsigned long long heads = __ballot(lane == 0 || v != vprev);
      const int start = 63 - __builtin_clzll(heads & ((2ull << lane) - 1ull));
      const unsigned long long before = __shfl(incl, start > 0 ? start - 1 : 0);
      const bool tail = lane == kWave - 1 || v != vnext;
      if (act && tail) add_relaxed(&a.acc[v], incl - (start > 0 ? before : 0ull));
    }
  }
}

// rank(v) from the sums, the next contributions, the next dangling mass.
template <int B>
__device__ void pull_update(const Args &a, Smem<B, OpPRPull> &sm, Grid gr, int it, Acc &acc) {
  const double d = (double)a.damping;
  const double N = (double)a.n;
  const unsigned long long dfix = ld_relaxed(&a.ctl->dangling[it & 1].v);
  const double base = (1.0 - d) / N + d * ((double)dfix * kFixInv) / N;
  for (uint32_t v = gr.id * B + threadIdx.x; v < (uint32_t)a.n; v += gr.n * B) {
    const float r = (float)(base + d * ((double)a.acc[v] * kFixInv));
    a.rank[v] = r;
    a.acc[v] = 0ull;  // huge vertices' sums start from 0 in the next phase 2
    const int32_t od = a.off[v + 1] - a.off[v];
    a.contrib[v] = od > 0 ? r / (float)od : 0.0f;
    if (od == 0) acc.dangling += to_fix(r);
  }
  flush_dangling<B, OpPRPull>(acc, sm, &a.ctl->dangling[(it + 1) & 1].v);
}

template <int B>
__global__ __launch_bounds__(B) __attribute__((amdgpu_waves_per_eu(ALB_WAVES_PER_EU))) void k_pull_pr(Args a) {
  __shared__ Smem<B, OpPRPull> sm;
  Acc acc;
  Grid gr;
  if (!join_members(a, sm, &gr)) return;
  if (a.threshold < 0) a.threshold = (int64_t)gr.n * B;
  const uint32_t hs = hint_shift(a, a.threshold, (uint32_t)a.n);
  unsigned long long epoch = 0;
  // set-up: ranks, sums, the first contributions and the first dangling mass
  set_up<B, OpPRPull, false>(a, gr);
  for (uint32_t v = gr.id * B + threadIdx.x; v < (uint32_t)a.n; v += gr.n * B) {
    const float r0 = 1.0f / (float)a.n;
    const int32_t od = a.off[v + 1] - a.off[v];
    a.contrib[v] = od > 0 ? r0 / (float)od : 0.0f;
    if (od == 0) acc.dangling += to_fix(r0);
  }
  flush_dangling<B, OpPRPull>(acc, sm, &a.ctl->dangling[0].v);
  const bool ok = grid_barrier<true>(a, sm, gr, epoch, 0);
  if (gr.id == 0 && threadIdx.x == 0) st_relaxed(&a.ctl->t_rounds, (unsigned long long)wall_clock64());
  int it = 0;
  for (; ok && it < a.max_rounds; ++it) {
    if (gr.id == 0 && threadIdx.x == 0) {
      st_relaxed(&a.ctl->chunk[(it + 1) % 3].v, 0ull);
      st_relaxed(&a.ctl->huge[(it + 1) & 1].v, 0ull);
      st_relaxed(&a.ctl->dangling[(it + 1) & 1].v, 0ull);
    }
    pull_gather<B>(a, sm, gr, it, a.threshold, hs, acc);
    if (!grid_barrier<true>(a, sm, gr, epoch, it)) break;
    const unsigned long long hc = ld_relaxed(&a.ctl->huge[it & 1].v);
    if ((hc >> 32) != 0) {
      pull_lb<B>(a, gr, hc, hs, acc);
      if (!grid_barrier<true>(a, sm, gr, epoch, it)) break;
    }
    pull_update<B>(a, sm, gr, it, acc);
    if (!grid_barrier<true>(a, sm, gr, epoch, it)) break;
  }
  if (gr.id == 0 && threadIdx.x == 0) {
    st_relaxed(&a.ctl->rounds, (uint32_t)it);
    st_relaxed(&a.ctl->threshold_used, (long long)a.threshold);
  }
  flush_stats<B, OpPRPull>(acc, sm, a.ctl);
  leave(a, sm, gr);
}

// ---------------------------------------------------------------------------
// Transposing a graph on the device, for push PageRank in tiles: edges go to
// bins of destinations, and each bin is sorted by counting in LDS.  Global
// atomics are one per workgroup and bin (a scatter with one per edge would
// take 15M / 23.5 G/s = 0.65 ms on a graph of 1M vertices, as much as a push
// iteration; this takes 0.32 ms; RMAT scale 20, whose heaviest bin holds 6 % of
// the edges, 1.5).
// ---------------------------------------------------------------------------
constexpr int kTrWg = 256, kTrSortWg = 1024;
constexpr uint32_t kTrStep = 4096;  // edges whose sources are expanded together

__device__ __forceinline__ uint32_t tr_edge(const Transpose &t, uint32_t w) {
  return (uint32_t)((uint64_t)t.m * w / kTransposeWgs);
}

// Edges per bin, of each workgroup's share and in all.
__global__ __launch_bounds__(kTrWg) void k_tr_count(Transpose t) {
  extern __shared__ uint32_t bin[];
  const uint32_t e0 = tr_edge(t, blockIdx.x), e1 = tr_edge(t, blockIdx.x + 1);
  for (uint32_t b = threadIdx.x; b < t.bins; b += kTrWg) bin[b] = 0;
  __syncthreads();
  for (uint32_t e = e0 + threadIdx.x; e < e1; e += 4 * kTrWg) {
    uint32_t v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = e + k * kTrWg < e1 ? (uint32_t)t.col[e + k * kTrWg] : 0u;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (e + k * kTrWg < e1) atomicAdd(&bin[v[k] >> t.bits], 1u);
  }
  __syncthreads();
  for (uint32_t b = threadIdx.x; b < t.bins; b += kTrWg) {
    const uint32_t c = bin[b];
    t.hist[(size_t)blockIdx.x * t.bins + b] = c;
    if (c) add_relaxed(&t.cursor[b], c);
  }
}

// Exclusive prefix sum over len entries of LDS by the whole workgroup of B
// threads; returns the total.
template <int B>
__device__ __forceinline__ uint32_t lds_exscan(uint32_t *x, uint32_t len, uint32_t *wsum) {
  const uint32_t per = (len + B - 1) / B, i0 = threadIdx.x * per;
  uint32_t sum = 0;
  for (uint32_t k = 0; k < per && i0 + k < len; ++k) sum += x[i0 + k];
  int32_t excl, total;
  block_exscan<B>((int32_t)sum, excl, total, (int32_t *)wsum);
  uint32_t at = (uint32_t)excl;
  for (uint32_t k = 0; k < per && i0 + k < len; ++k) {
    const uint32_t c = x[i0 + k];
    x[i0 + k] = at;
    at += c;
  }
  __syncthreads();
  return (uint32_t)total;
}

// Totals per bin -> start of each bin (one workgroup).
__global__ __launch_bounds__(kTrSortWg) void k_tr_start(Transpose t) {
  __shared__ uint32_t x[kBinsMax], wsum[kTrSortWg / kWave];
  for (uint32_t b = threadIdx.x; b < t.bins; b += kTrSortWg) x[b] = t.cursor[b];
  __syncthreads();
  lds_exscan<kTrSortWg>(x, t.bins, wsum);
  for (uint32_t b = threadIdx.x; b < t.bins; b += kTrSortWg) t.start[b] = t.cursor[b] = x[b];
  if (threadIdx.x == 0) t.start[t.bins] = t.m;
}

// The last row that begins at or before edge e and has edges (e < m).
__device__ __forceinline__ uint32_t row_of_edge(const int32_t *off, uint32_t n, uint32_t e) {
  uint32_t lo = 0, hi = n;  // off[lo] <= e < off[hi]
  while (hi - lo > 1) {
    const uint32_t mid = lo + ((hi - lo) >> 1);
    if ((uint32_t)off[mid] <= e)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

// Every edge into its bin.
__global__ __launch_bounds__(kTrWg) void k_tr_scatter(Transpose t) {
  extern __shared__ uint32_t bin[];  // next place of this workgroup's edges per bin
  constexpr uint32_t kRun = kTrStep / kTrWg;
  __shared__ uint32_t row[kTrStep], wmax[kTrWg / kWave], first[kTrWg + 1];
  const uint32_t tid = threadIdx.x, lane = lane_id();
  const uint32_t e0 = tr_edge(t, blockIdx.x), e1 = tr_edge(t, blockIdx.x + 1);
  if (e0 == e1) return;
  for (uint32_t b = tid; b < t.bins; b += kTrWg) {
    const uint32_t c = t.hist[(size_t)blockIdx.x * t.bins + b];
    bin[b] = c ? add_relaxed(&t.cursor[b], c) : 0u;
  }
  for (uint32_t g0 = e0; g0 < e1; g0 += kTrStep * kTrWg) {  // first rows of up to kTrWg steps at a time
    if (g0 + (uint64_t)tid * kTrStep < e1) first[tid] = row_of_edge(t.off, (uint32_t)t.n, g0 + tid * kTrStep);
    if (tid == 0) {
      const uint32_t end = (uint32_t)min((uint64_t)g0 + (uint64_t)kTrStep * kTrWg, (uint64_t)e1);
      first[(end - g0 + kTrStep - 1) / kTrStep] = row_of_edge(t.off, (uint32_t)t.n, end - 1);
    }
    __syncthreads();
    for (uint32_t s = 0; s < (uint32_t)kTrWg; ++s) {
      const uint64_t s0 = (uint64_t)g0 + (uint64_t)s * kTrStep;
      if (s0 >= e1) break;
      const uint32_t b0 = (uint32_t)s0, ne = min(kTrStep, e1 - b0);
      // the source of each edge: mark every row's first edge, then a running maximum
      for (uint32_t i = tid; i < kTrStep; i += kTrWg) row[i] = 0;
      __syncthreads();
      for (uint32_t r = first[s] + tid; r <= first[s + 1]; r += kTrWg) {
        const uint32_t p0 = (uint32_t)t.off[r], p1 = (uint32_t)t.off[r + 1], p = max(p0, b0);
        if (p < p1 && p < b0 + ne) row[p - b0] = r;
      }
      __syncthreads();
      uint32_t x[kRun], top = 0;
#pragma unroll
      for (uint32_t k = 0; k < kRun; ++k) {
        top = max(top, row[tid * kRun + k]);
        x[k] = top;
      }
      uint32_t incl = top;
#pragma unroll
      for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t y = __shfl_up(incl, d);
        if ((int)lane >= d) incl = max(incl, y);
      }
      if (lane == kWave - 1) wmax[tid / kWave] = incl;
      __syncthreads();
      uint32_t before = __shfl_up(incl, 1);
      if (lane == 0) before = 0;
      for (uint32_t j = 0; j < tid / kWave; ++j) before = max(before, wmax[j]);
#pragma unroll
      for (uint32_t k = 0; k < kRun; ++k) row[tid * kRun + k] = max(before, x[k]);
      __syncthreads();
      for (uint32_t i = tid; i < ne; i += kTrWg) {
        const uint32_t v = (uint32_t)t.col[b0 + i];
        const uint32_t at = atomicAdd(&bin[v >> t.bits], 1u);
        t.pairs[at] = make_uint2(row[i], v);
      }
      __syncthreads();
    }
  }
}

// One bin: count its destinations, offsets, sources in place.
__global__ __launch_bounds__(kTrSortWg) void k_tr_sort(Transpose t) {
  extern __shared__ uint32_t cnt[];  // 1 << bits
  __shared__ uint32_t wsum[kTrSortWg / kWave];
  const uint32_t b = blockIdx.x, width = 1u << t.bits;
  const uint32_t s0 = t.start[b], s1 = t.start[b + 1];
  const uint32_t v0 = b << t.bits;
  for (uint32_t i = threadIdx.x; i < width; i += kTrSortWg) cnt[i] = 0;
  __syncthreads();
  for (uint32_t p = s0 + threadIdx.x; p < s1; p += 4 * kTrSortWg) {
    uint32_t v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = p + k * kTrSortWg < s1 ? t.pairs[p + k * kTrSortWg].y : v0;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (p + k * kTrSortWg < s1) atomicAdd(&cnt[v[k] - v0], 1u);
  }
  __syncthreads();
  lds_exscan<kTrSortWg>(cnt, width, wsum);
  for (uint32_t i = threadIdx.x; i < width; i += kTrSortWg) {
    if (v0 + i < (uint32_t)t.n) t.toff[v0 + i] = (int32_t)(s0 + cnt[i]);
  }
  if (b == t.bins - 1 && threadIdx.x == 0) t.toff[t.n] = (int32_t)t.m;
  __syncthreads();
  for (uint32_t p = s0 + threadIdx.x; p < s1; p += 4 * kTrSortWg) {
    uint2 x[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = p + k * kTrSortWg < s1 ? t.pairs[p + k * kTrSortWg] : make_uint2(0u, v0);
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (p + k * kTrSortWg < s1) t.tcol[s0 + atomicAdd(&cnt[x[k].y - v0], 1u)] = (int32_t)x[k].x;
  }
}

__global__ void k_tr_zero(Transpose t) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *t.t_init = (unsigned long long)wall_clock64();
  for (uint32_t b = blockIdx.x * blockDim.x + threadIdx.x; b < t.bins; b += gridDim.x * blockDim.x) t.cursor[b] = 0;
}

// ---------------------------------------------------------------------------
// PageRank in tiles, for the balancer's default settings.  The rows and
// in-edges of the transposed graph, merged in order (each row's edges, then
// its end), are cut into tiles of tile_items, so that every tile costs the
// same whatever the in-degrees; each workgroup keeps its run of tiles
// through all iterations.  A tile's edges are read in order, four and two
// bytes each (source, and row relative to the tile's first, laid out once per
// call), and their contributions gathered from an array that the L2s hold up
// to a few million vertices; sums are exact 64-bit integers added in LDS,
// where the order does not matter and neighbouring lanes of one row only
// serialise within the CU.  A row that ends in the tile is updated at once: its
// new contribution goes to a second array, its sum never to memory.  Only rows
// cut by a workgroup boundary meet in memory, between the two barriers of an
// iteration.  The bin kernels above spent their time in chains of dependent
// loads per vertex, skew and full barriers (RMAT scale 20, 16M edges: 291 us an
// iteration against 96 here, 104 with tiles of 4,096; scale 22 862 and 406; Zipf
// 1M, 17.7M edges, 121 and 101; the gathers alone take 64 at the L2s' 250 G/s for
// 16M edges).  The sums, and so the ranks, are
// bit for bit the same.  Cutting rows and entries, merged, into equal parts is
// the merge-path decomposition of sparse matrix-vector products (Merrill and
// Garland, 2016).
// ---------------------------------------------------------------------------
constexpr int kTileLoads = 4;  // edges in flight per lane

template <int B>
struct SmemTiles {
  union {
    unsigned long long acc[kTileItems + 1];  // sums of the tile's rows
    uint16_t row[kTileItems];                // set-up: rows of the tile's edges
  };
  unsigned long long carry, defer;  // sums: of the row the last tile left open; of the row shared with earlier workgroups
  unsigned long long part[B / kWave];
  uint32_t wmax[B / kWave];
  int32_t flag;
  uint32_t ticket, members, xcd, xcd_n, n_xcd;
};

// Rows that end within the first d merged items.
__device__ __forceinline__ uint32_t rows_within(const int32_t *off, uint32_t n, uint64_t m, uint64_t d) {
  uint64_t lo = d > m ? d - m : 0, hi = d < n ? d : n;
  while (lo < hi) {
    const uint64_t mid = (lo + hi) >> 1;
    if ((uint64_t)(uint32_t)off[mid + 1] + mid + 1 <= d)
      lo = mid + 1;
    else
      hi = mid;
  }
  return (uint32_t)lo;
}

struct Tile {
  uint32_t row, rows;  // first row and rows that end in it
  uint32_t edge, edges;
};
__device__ __forceinline__ Tile tile_at(const Args &a, uint64_t items, uint32_t t) {
  const uint64_t d0 = (uint64_t)t * a.tile_items, d1 = min(d0 + a.tile_items, items);
  const uint32_t r0 = a.tile_row[t], r1 = a.tile_row[t + 1];
  const uint32_t e0 = (uint32_t)(d0 - r0);
  return {r0, r1 - r0, e0, (uint32_t)(d1 - r1) - e0};
}

// Lay the workgroup's tiles [t0, t1) out: first rows, and each edge's row.
template <int B>
__device__ void lay_out_tiles(const Args &a, SmemTiles<B> &sm, uint64_t m, uint32_t t0, uint32_t t1) {
  static_assert(kTileItems % B == 0, "whole runs per thread");
  constexpr uint32_t kRun = kTileItems / B;
  const uint32_t tid = threadIdx.x, lane = lane_id();
  const uint32_t n = (uint32_t)a.n;
  const uint64_t items = (uint64_t)n + m;
  if (t0 < t1)
    for (uint32_t t = t0 + tid; t <= t1; t += B)
      a.tile_row[t] = rows_within(a.toff, n, m, min((uint64_t)t * a.tile_items, items));
  __syncthreads();
  for (uint32_t t = t0; t < t1; ++t) {
    const Tile tl = tile_at(a, items, t);
    for (uint32_t i = tid; i < kTileItems; i += B) sm.row[i] = 0;
    __syncthreads();
    // the first edge of every row that has one here
    for (uint32_t l = tid; l <= tl.rows && tl.row + l < n; l += B) {
      const uint32_t s0 = (uint32_t)a.toff[tl.row + l], s1 = (uint32_t)a.toff[tl.row + l + 1];
      const uint32_t s = max(s0, tl.edge);
      if (s < s1 && s < tl.edge + tl.edges) sm.row[s - tl.edge] = (uint16_t)l;
    }
    __syncthreads();
    // running maximum: kRun consecutive entries per thread, then over the threads
    uint32_t x[kRun], top = 0;
#pragma unroll
    for (uint32_t k = 0; k < kRun; ++k) {
      top = max(top, (uint32_t)sm.row[tid * kRun + k]);
      x[k] = top;
    }
    uint32_t incl = top;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      const uint32_t y = __shfl_up(incl, d);
      if ((int)lane >= d) incl = max(incl, y);
    }
    if (lane == kWave - 1) sm.wmax[tid / kWave] = incl;
    __syncthreads();
    uint32_t before = __shfl_up(incl, 1);
    if (lane == 0) before = 0;
    for (uint32_t j = 0; j < tid / kWave; ++j) before = max(before, sm.wmax[j]);
#pragma unroll
    for (uint32_t k = 0; k < kRun; ++k) {
      const uint32_t i = tid * kRun + k;
      if (i < tl.edges) a.tile_lrow[tl.edge + i] = (uint16_t)max(before, x[k]);
    }
    __syncthreads();
  }
}

template <int B>
__global__ __launch_bounds__(B) __attribute__((amdgpu_waves_per_eu(4))) void k_pr_tiles(Args a) {
  __shared__ SmemTiles<B> sm;
  Acc acc;
  Grid gr;
  if (!join_members(a, sm, &gr)) return;
  const uint32_t tid = threadIdx.x;
  const uint32_t n = (uint32_t)a.n;
  const uint64_t m = (uint64_t)(uint32_t)a.toff[n];
  const uint64_t items = (uint64_t)n + m;
  const uint32_t t0 = (uint32_t)((uint64_t)a.n_tiles * gr.id / gr.n);
  const uint32_t t1 = (uint32_t)((uint64_t)a.n_tiles * (gr.id + 1) / gr.n);
  const uint32_t stripe = xcd_id() % kStatXcds;
  unsigned long long epoch = 0, dangling = 0;
  // add the workgroup's dangling mass to iteration it's
  auto flush = [&](int it) {
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) dangling += __shfl_xor(dangling, d);
    if (lane_id() == 0) sm.part[tid / kWave] = dangling;
    __syncthreads();
    if (tid == 0) {
      unsigned long long t = 0;
      for (int j = 0; j < B / kWave; ++j) t += sm.part[j];
      if (t) add_relaxed(&a.ctl->tile_dangling[it % 3][stripe].v, t);
    }
    dangling = 0;
  };

  // set-up: the inspection's counts (every iteration works on every vertex),
  // first contributions, dangling mass, cleared meeting sums, the tiles
  if (a.clear_ctl) {
    for (size_t i = gr.id * B + tid; i < kBarWords; i += (size_t)gr.n * B) a.clear_bar[i] = 0ull;
    if (gr.id == 0 && tid == B - 1) reset_ctl(a.clear_ctl);
  }
  const float r0 = 1.0f / (float)a.n;
  for (uint32_t v = gr.id * B + tid; v < n; v += gr.n * B) {
    const int32_t deg = a.insp_off[v + 1] - a.insp_off[v];
    const bool huge = deg > 0 && (int64_t)deg >= a.insp_threshold;
    acc.frontier += (unsigned long long)a.max_rounds;
    acc.huge_v += huge ? (unsigned long long)a.max_rounds : 0ull;
    const unsigned long long e = (unsigned long long)deg * (unsigned long long)a.max_rounds;
    acc.edges_lb += huge ? e : 0ull;
    acc.edges_twc += huge ? 0ull : e;
    const int32_t od = a.off[v + 1] - a.off[v];
    st_relaxed(&a.contrib[v], od > 0 ? r0 / (float)od : 0.0f);
    if (od == 0) dangling += to_fix(r0);
    st_relaxed(&a.acc[v], 0ull);
  }
  flush(0);
  lay_out_tiles(a, sm, m, t0, t1);
  for (uint32_t i = tid; i <= kTileItems; i += B) sm.acc[i] = 0;
  // the row open at this workgroup's start has edges in earlier workgroups
  const uint32_t first = t0 < t1 ? a.tile_row[t0] : n;
  const bool shared_first = first < n && (uint64_t)(uint32_t)a.toff[first] + first < (uint64_t)t0 * a.tile_items;
  bool ok = grid_barrier<false>(a, sm, gr, epoch, 0);
  if (gr.id == 0 && tid == 0) st_relaxed(&a.ctl->t_rounds, (unsigned long long)wall_clock64());

  const double d = (double)a.damping, N = (double)a.n;
  int it = 0;
  for (; ok && it < a.max_rounds; ++it) {
    if (gr.id == 0 && tid < (uint32_t)kStatXcds) st_relaxed(&a.ctl->tile_dangling[(it + 2) % 3][tid].v, 0ull);
    unsigned long long mass = 0;
#pragma unroll
    for (int x = 0; x < kStatXcds; ++x) mass += ld_relaxed(&a.ctl->tile_dangling[it % 3][x].v);
    const double base = (1.0 - d) / N + d * ((double)mass * kFixInv) / N;
    const float *cin = it & 1 ? a.contrib2 : a.contrib;
    float *cout = it & 1 ? a.contrib : a.contrib2;
    const bool last = it + 1 == a.max_rounds;
    auto update = [&](uint32_t v, unsigned long long sum) {
      const float r = (float)(base + d * ((double)sum * kFixInv));
      if (last) a.rank[v] = r;
      const int32_t od = a.off[v + 1] - a.off[v];
      st_relaxed(&cout[v], od > 0 ? r / (float)od : 0.0f);
      if (od == 0) dangling += to_fix(r);
    };
    bool deferred = false;  // thread 0: the shared first row ends in this workgroup
    unsigned long long carry = 0;  // thread 0: sum of the open row
    uint32_t open = first;
    for (uint32_t t = t0; t < t1; ++t) {
      const Tile tl = tile_at(a, items, t);
      const int32_t *col = a.tcol + tl.edge;
      const uint16_t *lrow = a.tile_lrow + tl.edge;
      for (uint32_t i0 = tid; i0 < tl.edges; i0 += kTileLoads * B) {
        int32_t u[kTileLoads];
        uint32_t l[kTileLoads];
        float c[kTileLoads];
#pragma unroll
        for (int k = 0; k < kTileLoads; ++k) {
          const uint32_t i = i0 + k * B;
          u[k] = i < tl.edges ? col[i] : -1;
          l[k] = i < tl.edges ? lrow[i] : 0u;
        }
#pragma unroll
        for (int k = 0; k < kTileLoads; ++k) c[k] = u[k] >= 0 ? ld_relaxed(&cin[u[k]]) : 0.0f;
#pragma unroll
        for (int k = 0; k < kTileLoads; ++k)
          if (u[k] >= 0) atomicAdd(&sm.acc[l[k]], to_fix(c[k]));
      }
      __syncthreads();
      for (uint32_t l = tid; l < tl.rows; l += B) {
        unsigned long long sum = sm.acc[l];
        sm.acc[l] = 0;
        if (l == 0) {  // thread 0: the row open before this tile
          sum += carry;
          carry = 0;
          if (tl.row == first && shared_first) {
            sm.defer = sum;
            deferred = true;
            continue;
          }
        }
        update(tl.row + l, sum);
      }
      if (tid == 0) {
        carry += sm.acc[tl.rows];
        sm.acc[tl.rows] = 0;
        open = tl.row + tl.rows;
      }
      __syncthreads();
    }
    if (tid == 0 && carry) add_relaxed(&a.acc[open], carry);  // the rest of the open row is a later workgroup's
    flush(it + 1);
    ok = grid_barrier<false>(a, sm, gr, epoch, it);
    if (!ok) break;
    if (tid == 0 && deferred) {
      const unsigned long long sum = sm.defer + ld_relaxed(&a.acc[first]);
      st_relaxed(&a.acc[first], 0ull);
      update(first, sum);
      if (dangling) add_relaxed(&a.ctl->tile_dangling[(it + 1) % 3][stripe].v, dangling);
      dangling = 0;
    }
    ok = grid_barrier<false>(a, sm, gr, epoch, it);
  }
  if (gr.id == 0 && tid == 0) {
    st_relaxed(&a.ctl->rounds, (uint32_t)it);
    st_relaxed(&a.ctl->threshold_used, (long long)a.threshold);
  }
  // statistics: the workgroups' sums
  unsigned long long v[kStats] = {acc.frontier, acc.edges_twc, acc.edges_lb, acc.huge_v, 0ull};
#pragma unroll
  for (int k = 0; k < kStats; ++k) {
#pragma unroll
    for (int x = kWave / 2; x > 0; x >>= 1) v[k] += __shfl_xor(v[k], x);
    if (lane_id() == 0 && v[k]) add_relaxed(&a.ctl->stat[stripe][k].v, v[k]);
  }
  leave(a, sm, gr);
}

// ---------------------------------------------------------------------------
// Dispatch over workgroup size and operator.
// ---------------------------------------------------------------------------

template <int B, class Op>
struct TwcF {
  static hipError_t run(int grid, const Args *a, hipStream_t s) {
    hipLaunchKernelGGL((k_twc<B, Op>), dim3(grid), dim3(B), 0, s, *a, make_op<Op>(*a));
    return hipGetLastError();
  }
};
template <int B, class Op>
struct LbF {
  static hipError_t run(int grid, const Args *a, hipStream_t s) {
    hipLaunchKernelGGL((k_lb<B, Op>), dim3(grid), dim3(B), 0, s, *a, make_op<Op>(*a));
    return hipGetLastError();
  }
};
template <int B, class Op>
struct PersistentF {
  static hipError_t run(int grid, const Args *a, hipStream_t s) {
    if constexpr (std::is_same<Op, OpBFS>::value || std::is_same<Op, OpCC>::value ||
                  (Op::kKind == OP_KCORE)) {
      if (a->vbits) {  // with the filter bitmap
        hipLaunchKernelGGL((k_persistent<B, Op, false, true>), dim3(grid), dim3(B), 0, s, *a, make_op<Op>(*a));
        return hipGetLastError();
      }
    }
    hipLaunchKernelGGL((k_persistent<B, Op, false>), dim3(grid), dim3(B), 0, s, *a, make_op<Op>(*a));
    return hipGetLastError();
  }
};
template <int B, class Op>
struct OccF {
  static hipError_t run(int *blocks) {
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, (const void *)k_persistent<B, Op, false>, B, 0);
  }
};
// batches: BFS and SSSP only
template <int B, class Op>
struct BatchF {
  static hipError_t run(int grid, const Args *a, hipStream_t s) {
    if constexpr (Op::kBatch) {
      hipLaunchKernelGGL((k_persistent<B, Op, true>), dim3(grid), dim3(B), 0, s, *a, make_op<Op>(*a));
      return hipGetLastError();
    } else {
      return hipErrorInvalidValue;
    }
  }
};
template <int B, class Op>
struct BatchOccF {
  static hipError_t run(int *blocks) {
    if constexpr (Op::kBatch)
      return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, (const void *)k_persistent<B, Op, true>, B, 0);
    else
      return hipErrorInvalidValue;
  }
};

// continuous serving: one operator for BFS and SSSP queries (OP_SSSP)
template <int B, class Op>
struct OpenF {
  static hipError_t run(int grid, const Args *a, hipStream_t s) {
    if constexpr (std::is_same<Op, OpSSSP>::value) {
      hipLaunchKernelGGL((k_open<B, OpServe>), dim3(grid), dim3(B), 0, s, *a, make_op<OpServe>(*a));
      return hipGetLastError();
    } else {
      return hipErrorInvalidValue;
    }
  }
};
template <int B, class Op>
struct OpenOccF {
  static hipError_t run(int *blocks) {
    if constexpr (std::is_same<Op, OpSSSP>::value)
      return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, (const void *)k_open<B, OpServe>, B, 0);
    else
      return hipErrorInvalidValue;
  }
};

template <template <int, class> class F, int B, typename... Xs>
hipError_t by_op(OpKind op, Xs... xs) {
  switch (op) {
    case OP_BFS: return F<B, OpBFS>::run(xs...);
    case OP_SSSP: return F<B, OpSSSP>::run(xs...);
    case OP_CC: return F<B, OpCC>::run(xs...);
    case OP_PR: return F<B, OpPR>::run(xs...);
    case OP_RECORD: return F<B, OpRecord>::run(xs...);
    case OP_KCORE: return F<B, OpKCore<hot_slots(B)>>::run(xs...);
  }
  return hipErrorInvalidValue;
}

template <template <int, class> class F, typename... Xs>
hipError_t by_wg(OpKind op, int wg, Xs... xs) {
  switch (wg) {
    case 64: return by_op<F, 64>(op, xs...);
    case 256: return by_op<F, 256>(op, xs...);
    case 1024: return by_op<F, 1024>(op, xs...);
  }
  return hipErrorInvalidValue;
}

}  // namespace

bool supported_wg(int wg) { return wg == 64 || wg == 256 || wg == 1024; }

hipError_t launch_init(OpKind op, const Args &a, hipStream_t s) {
  const int threads = 256;
  int blocks = (int)(((int64_t)a.n + threads - 1) / threads);
  if (blocks > 4096) blocks = 4096;
  if (blocks < 128) blocks = 128;
  hipLaunchKernelGGL(k_init, dim3(blocks), dim3(threads), 0, s, a, (int)op);
  return hipGetLastError();
}

hipError_t launch_clear(const Args &a, hipStream_t s) {
  hipLaunchKernelGGL(k_clear, dim3(8), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_finish(OpKind op, const Args &a, hipStream_t s) {
  const int threads = 256;
  int blocks = (int)(((int64_t)a.n + threads - 1) / threads);
  if (blocks > 4096) blocks = 4096;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_finish, dim3(blocks), dim3(threads), 0, s, a, (int)op);
  return hipGetLastError();
}

hipError_t launch_twc(OpKind op, int wg, int grid, const Args &a, hipStream_t s) {
  return by_wg<TwcF>(op, wg, grid, &a, s);
}
hipError_t launch_lb(OpKind op, int wg, int grid, const Args &a, hipStream_t s) {
  return by_wg<LbF>(op, wg, grid, &a, s);
}
hipError_t launch_persistent(OpKind op, int wg, int grid, const Args &a, hipStream_t s) {
  return by_wg<PersistentF>(op, wg, grid, &a, s);
}
hipError_t persistent_occupancy(OpKind op, int wg, int *blocks_per_cu) {
  return by_wg<OccF>(op, wg, blocks_per_cu);
}
hipError_t batch_occupancy(OpKind op, int wg, int *blocks_per_cu) { return by_wg<BatchOccF>(op, wg, blocks_per_cu); }
hipError_t launch_batch(OpKind op, int wg, int grid, const Args &a, hipStream_t s) {
  return by_wg<BatchF>(op, wg, grid, &a, s);
}

hipError_t launch_init_batch(OpKind op, const Args &a, hipStream_t s) {
  const int threads = 256;
  long long blocks = (a.nlabels + threads - 1) / threads;
  if (blocks > 8192) blocks = 8192;
  if (blocks < 128) blocks = 128;
  hipLaunchKernelGGL(k_init_batch, dim3((unsigned)blocks), dim3(threads), 0, s, a, (int)op);
  return hipGetLastError();
}

hipError_t launch_finish_batch(OpKind op, const Args &a, int32_t max_n, hipStream_t s) {
  const int threads = 256;
  int bx = (max_n + threads - 1) / threads;
  if (bx > 64) bx = 64;
  if (bx < 1) bx = 1;
  hipLaunchKernelGGL(k_finish_batch, dim3(bx, a.nq), dim3(threads), 0, s, a, (int)op);
  return hipGetLastError();
}

hipError_t pull_occupancy(int wg, int *blocks_per_cu) {
  switch (wg) {
    case 64: return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, (const void *)k_pull_pr<64>, 64, 0);
    case 256: return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, (const void *)k_pull_pr<256>, 256, 0);
    case 1024:
      return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, (const void *)k_pull_pr<1024>, 1024, 0);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_pr_tiles(int grid, const Args &a, hipStream_t s) {
  hipLaunchKernelGGL(k_pr_tiles<kTileWg>, dim3(grid), dim3(kTileWg), 0, s, a);
  return hipGetLastError();
}
hipError_t pr_tiles_occupancy(int *blocks_per_cu) {
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, (const void *)k_pr_tiles<kTileWg>, kTileWg, 0);
}

hipError_t launch_transpose(const Transpose &t, hipStream_t s) {
  const size_t bin_bytes = sizeof(uint32_t) * t.bins;
  hipLaunchKernelGGL(k_tr_zero, dim3(8), dim3(kTrWg), 0, s, t);
  hipLaunchKernelGGL(k_tr_count, dim3(kTransposeWgs), dim3(kTrWg), bin_bytes, s, t);
  hipLaunchKernelGGL(k_tr_start, dim3(1), dim3(kTrSortWg), 0, s, t);
  hipLaunchKernelGGL(k_tr_scatter, dim3(kTransposeWgs), dim3(kTrWg), bin_bytes, s, t);
  hipLaunchKernelGGL(k_tr_sort, dim3(t.bins), dim3(kTrSortWg), sizeof(uint32_t) << t.bits, s, t);
  return hipGetLastError();
}

hipError_t launch_init_open(const Args &a, hipStream_t s) {
  hipLaunchKernelGGL(k_init_open, dim3(64), dim3(256), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_open(OpKind op, int wg, int grid, const Args &a, hipStream_t s) {
  return by_wg<OpenF>(op, wg, grid, &a, s);
}
hipError_t open_occupancy(OpKind op, int wg, int *blocks_per_cu) { return by_wg<OpenOccF>(op, wg, blocks_per_cu); }

hipError_t launch_pull_pr(int wg, int grid, const Args &a, hipStream_t s) {
  switch (wg) {
    case 64: hipLaunchKernelGGL(k_pull_pr<64>, dim3(grid), dim3(64), 0, s, a); break;
    case 256: hipLaunchKernelGGL(k_pull_pr<256>, dim3(grid), dim3(256), 0, s, a); break;
    case 1024: hipLaunchKernelGGL(k_pull_pr<1024>, dim3(grid), dim3(1024), 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_pr_update(int wg, int grid, const Args &a, hipStream_t s) {
  switch (wg) {
    case 64: hipLaunchKernelGGL(k_pr_update<64>, dim3(grid), dim3(64), 0, s, a); break;
    case 256: hipLaunchKernelGGL(k_pr_update<256>, dim3(grid), dim3(256), 0, s, a); break;
    case 1024: hipLaunchKernelGGL(k_pr_update<1024>, dim3(grid), dim3(1024), 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace alb
