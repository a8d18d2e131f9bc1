// Internal definitions of the gfx950 Jet library: device context layout and the host-side launch
// wrappers of every kernel.  Not part of the public ABI (see include/jet.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <string>
#include <vector>

#include "../../include/jet.h"
#include "ahead.h"

namespace jet {

constexpr int kMaxK = 128;
constexpr int kSmallNet = 64;      // nets up to this size are processed by one wave, several per wave
constexpr int kChunkNets = 32;     // nets of one chunk at most (64 pins hold more only with single-pin nets)
constexpr int kMediumNet = 1024;   // nets up to this size: one 64-thread workgroup, candidates in LDS
constexpr int kMediumSmall = 256;  // medium nets up to this size use a smaller LDS list (more per CU)
constexpr int kLaneDegree = 32;    // moves with more incident nets are applied by many threads
constexpr int kBigCap = 4096;      // larger nets: one 256-thread workgroup, up to kBigCap candidates in LDS
constexpr int kMaxSortedDegree = 8192;  // longer incidence lists are radix-sorted in global scratch
constexpr int kHubDegree = 256;        // vertices with more incident nets take whole workgroups (k_hub.hip)

// Device status block, read back by the host after each phase that needs a decision.
constexpr int kKm1Slots = 64;
// Counters that every workgroup of a pass adds to, spread over slots a cache line apart.  Atomics on one
// address are served one after the other, about 10 ns each: the three counters of a gain pass over
// 2,048 workgroups, all on one line, took 50 us; over 64 lines they take less than one.
struct alignas(128) CtrSlot {
  long long km1;      // metric changes since the last fold
  long long n_cand;   // |M| of the candidate pass
  long long inc_low, inc_hub;  // incidences scanned by the candidate pass (non-hub / hub vertices)
  long long ab_inc;   // incidences of candidates scanned by the graph afterburner
  long long rb_inc;   // incidences scanned by the rebalancing gain pass
  long long rb_elig;  // vertices it examined in full
  long long rb_ent;   // order-key entries it wrote
};
// A union context refines many hypergraphs with the same k at once (the batch): vertices and nets
// are concatenated, and every per-block quantity is kept per segment hg * k + b.
constexpr int kMaxH = 4096;    // hypergraphs in one union context
constexpr int kMaxSeg = 16384; // segments (hypergraph, block) of one context

struct DevStatus {
  CtrSlot slot[kKm1Slots];
  int64_t km1;            // current metric, maintained incrementally: km1 + sum over the slots
  int32_t n_moves;        // entries in the move list
  int32_t n_ovf;          // large nets handed to the global-scratch afterburner this iteration
  int32_t n_bigmv;        // listed moves with more than kLaneDegree incident nets
  int64_t mv_inc;         // incident nets of the listed moves (sum of their degrees)
  int32_t rb_nlist;       // vertices on the rebalancing candidate list of the round
  int32_t rb_nhub;        // hub vertices on the hub candidate list of the round
  int32_t rb_nseg;        // union: overloaded segments of the round (listed in rb_seg)
  int32_t err;            // nonzero: a kernel met an input it cannot handle (see kErr*)
  int32_t err_arg;        // detail for err
  int64_t bw[kMaxSeg];    // block weights per segment (the host reads the first H * k)
  // not read back by the host:
  int32_t bcnt[kMaxSeg];     // vertices per segment
  int32_t rb_count[kMaxSeg];   // rebalancing: eligible entries per segment
  int64_t rb_off[kMaxSeg + 1]; // rebalancing: list offsets per segment
  int64_t rb_need[kMaxSeg];    // rebalancing: weight that must leave the segment's block
  int32_t rb_kept[kMaxSeg];    // rebalancing: entries the grid-wide first selection pass kept per block
  int64_t hkm1[kMaxH];    // union: metric change per hypergraph since the last fold
  int32_t hmoves[kMaxH];  // union: moves listed per hypergraph in the current phase
  int32_t rb_seg[kMaxSeg];   // union: the overloaded segments of the round
};

struct LoopCtl {
  int32_t phase;
  int32_t phase_mask;     // bit p set iff a hypergraph of the record is in phase p (1 << phase for one)
  int32_t stamp;          // iteration stamp: v is locked iff lockstamp[v] == stamp - 1
  int32_t tau_q;          // quantised temperature of the current round
  int32_t tau_r;          // index of the current temperature round
  int32_t round;          // consecutive iterations without strict improvement
  int32_t it;             // iterations of the current round
  int32_t lock_any;       // the last Jet phase moved a vertex (some vertex is locked)
  int32_t lock_was_any;   // lock_any as it was when the current iteration began
  int32_t n_cand, n_moved;          // the current iteration's Jet phase
  int32_t rb_rounds, rb_moved;      // the current iteration's rebalancing rounds
  int32_t improved;       // the current partition is the round's best and not in `best` yet: the next
                          // candidate pass copies it, a rollback has nothing to undo
  uint32_t seq;           // control kernels run in this call
  int32_t ntrace;         // iteration records written (counted beyond the capacity too)
  int32_t iterations, rebalance_rounds, moves_executed;  // totals of the call
  int64_t km1;            // exact metric of the current partition
  int64_t best_ovl, best_km1;
  int64_t km1_in;
  // parameters of the call
  int32_t limit, max_iters, num_tau, max_rb;
  int32_t tau_qs[8];
  int32_t rb_only;        // rebalancing rounds only (jet_rebalance)
  int32_t rb_unw;         // rebalancing order, jet_params.rb_unweighted: 0, 1 or 2
  int32_t trace_cap;
  int64_t lmax, dz, A;    // balance limit, deadzone threshold, ceil(W/k) of the hypergraph
};

// A launch of a phase returns at once unless some hypergraph of the gate record is in it.
#define JET_GATE(lc, want)                                                      \
  do {                                                                          \
    if ((lc) != nullptr && (want) >= 0 && !(((lc)->phase_mask >> (want)) & 1)) \
      return;                                                                   \
  } while (0)

__device__ __forceinline__ void set_phase(LoopCtl &r, int32_t p) {
  r.phase = p;
  r.phase_mask = 1 << p;
}

// The hypergraphs of one phase in a union context, in index order, with prefix sums of their
// vertex tiles (kUnionTile vertices; every hypergraph's vertices start on a tile) and of their
// chunks of small nets (no chunk holds nets of two hypergraphs).  The control kernels rebuild the
// lists after every change of phase; kernels of a phase walk only the listed hypergraphs' tiles.
constexpr int kUnionTile = 256;
struct ActList {
  int32_t cnt;
  int32_t hg[kMaxH + 1];
  int32_t tpref[kMaxH + 2];
  int32_t cpref[kMaxH + 2];
};
enum : int { kActJet = 0, kActRb = 1, kActRoll = 2, kActLists = 3 };

// The hypergraphs of a union context as the kernels see them; lcs == nullptr for a context of one
// hypergraph (its record is the gate record, segments are blocks).
struct Union {
  const LoopCtl *lcs;    // per-hypergraph loop records
  const uint16_t *vhg;   // hypergraph of every vertex (padding vertices: the pseudo-hypergraph H)
  const uint16_t *nhg;   // hypergraph of every net
  const ActList *act;    // [kActLists]
  const int32_t *ht0;    // [H + 1] first tile of every hypergraph
  const int32_t *hch0;   // [H + 1] first chunk of every hypergraph
};

// Last list position i with pref[i] <= x (pref[0] = 0 <= x < pref[cnt]), found by the 64 lanes of
// a wave together: each round every lane tests one sample position and a ballot keeps the last
// one that passed, so at most two rounds (dependent loads) for the 4,096 list entries a union
// holds.  Every lane of the wave must call it with the same x.
__device__ __forceinline__ int32_t act_find(const int32_t *pref, int32_t cnt, int32_t x) {
  const int lane = __lane_id();
  int32_t lo = 0, span = cnt;  // the answer lies in [lo, lo + span)
  while (span > 1) {
    const int32_t stride = (span + 63) >> 6;
    const int32_t pos = lo + lane * stride;
    const bool ok = lane * stride < span && pref[pos] <= x;
    const unsigned long long m = __ballot(ok);
    const int32_t top = 63 - __clzll(m);  // lane 0 always passes (pref[lo] <= x)
    lo += top * stride;
    span = stride < span - top * stride ? stride : span - top * stride;
  }
  return lo;
}

// Virtual tile t of a list -> its first vertex and its hypergraph (wave-uniform t).
__device__ __forceinline__ int64_t act_tile_base(const ActList &L, const int32_t *ht0, int32_t t,
                                                 int32_t *hg_out = nullptr) {
  const int32_t i = act_find(L.tpref, L.cnt, t);
  const int32_t hg = L.hg[i];
  if (hg_out) *hg_out = hg;
  return ((int64_t)ht0[hg] + (t - L.tpref[i])) * kUnionTile;
}
// Virtual chunk c of a list -> the chunk index (wave-uniform c).
__device__ __forceinline__ int32_t act_chunk(const ActList &L, const int32_t *hch0, int32_t c) {
  const int32_t i = act_find(L.cpref, L.cnt, c);
  return hch0[L.hg[i]] + (c - L.cpref[i]);
}

// Per-family timing and algorithmic bytes accumulated on the device: a mark kernel before the
// family's launches records the wall clock, one after it adds the elapsed ticks and the bytes.
struct DevProf {
  unsigned long long t0[8];
  unsigned long long ticks[8];
  unsigned long long launches[8];
  double bytes[8];
};

// Destination of the afterburner's recomputed-gain contributions.  On small levels (few
// vertices, many incident nets each) the contributions would pile onto a few cache lines, so they
// go to `copies` private copies of the array (chosen by the contributing wave or block), summed
// into rg afterwards; otherwise copies == 1 and base is rg itself.
struct RgSink {
  int32_t *base;
  int32_t n;
  int32_t copies;
};
__device__ __forceinline__ void rg_add(const RgSink &s, uint32_t slot, int32_t v, int32_t d) {
  atomicAdd(&s.base[(size_t)(slot % (uint32_t)s.copies) * (size_t)s.n + (size_t)v], d);
}

// adds to a counter of one of the slots (chosen by the caller, e.g. from the block index)
__device__ __forceinline__ void count_add(DevStatus *st, uint32_t slot, long long CtrSlot::*field, long long d) {
  if (d != 0) atomicAdd((unsigned long long *)&(st->slot[slot % kKm1Slots].*field), (unsigned long long)d);
}
__device__ __forceinline__ void add_km1(DevStatus *st, uint32_t slot, int64_t d) {
  count_add(st, slot, &CtrSlot::km1, d);
}
// union: the metric change of hypergraph hg
__device__ __forceinline__ void add_km1_hg(DevStatus *st, int32_t hg, int64_t d) {
  if (d != 0) atomicAdd((unsigned long long *)&st->hkm1[hg], (unsigned long long)d);
}

enum : int32_t {
  kErrNone = 0,
  kErrPartRange = 1,      // part[v] outside [0,k)
  kErrPinRange = 2,       // pin outside [0,n)
  kErrDupPin = 3,         // a vertex twice in one net
  kErrDegree = 4,         // vertex degree above kMaxSortedDegree
  kErrMixedOverflow = 5,  // afterburner: too many ordered events in one huge net
  kErrWeight = 6,         // weight < 1
  kErrOverflow = 7,       // a vertex's incident weight sum >= 2^31
  kErrTarget = 8,         // inspection input: candidate target outside [0,k) or equal to its block
  kErrHandOver = 9,       // a workgroup waited for another one's sums in vain
};

// kernel families timed by the optional instrumentation
enum ProfFamily : int {
  kProfCandidates = 0,   // k_candidates or k_candidates_bits (hubs too where they are beside the others)
  kProfCandidatesHub,    // k_hub where hubs are not beside the others
  kProfAfterburner,      // k_ab_chunks + k_ab_nets + k_ab_overflow + k_rg_reduce, or k_ab_graph
  kProfSelect,           // k_select_moves
  kProfApply,            // k_apply
  kProfRbGain,           // k_rb_list(_union) + k_rb_gain(_bits) + k_rb_hub_list + k_rb_hub
  kProfRbSelect,         // k_rb_sel_hist + k_rb_sel_split + k_rb_select
  kProfFamilies
};

// Synchronous clustering of the coarsening phase (Section 6, Algorithm 4): one rating-table slot
struct CoSlot {
  int32_t key;               // cluster label, -1 empty
  int32_t mark;              // last net that added to val
  unsigned long long val;    // heavy-edge rating, 32.32 fixed point
};

// Clustering state, allocated at the first clustering call of a context.  Between sub-rounds the
// per-vertex arrays hold -1 (tp, tt, gslot, newlab) or 0 (jw, gcnt).
struct CoState {
  bool ready = false;
  uint64_t *qnet = nullptr;          // [m] floor(w(e) 2^32 / (|e| - 1)), 0 for single-pin nets
  int64_t *deg = nullptr;            // [n] sum over incident nets of (|e| - 1)
  std::vector<int64_t> hdeg;         // host copy
  int64_t max_deg = 0;               // largest of them
  int64_t *cw = nullptr;             // [n] cluster weights of jet_coarsen's own clustering
  int32_t *tp = nullptr, *tt = nullptr;  // [n] proposals, targets after swap prevention
  int32_t *gcnt = nullptr, *gslot = nullptr, *newlab = nullptr, *flag = nullptr;  // [n]
  unsigned long long *jw = nullptr;  // [n] proposal weight per target
  int64_t cap = 0;                   // entries of the per-sub-round arrays below
  int32_t *gpos = nullptr, *gtarget = nullptr, *members = nullptr;  // [cap]
  int64_t *goff = nullptr, *gmoved = nullptr;                       // [cap + 1], [cap]
  int64_t ptab_len = 0;
  int64_t *ptab = nullptr;           // [ptab_len] rating-table offsets over list positions
  int64_t tab_slots = 0;
  CoSlot *tab = nullptr;             // [tab_slots] rating tables of one launch
  int32_t *ctr = nullptr;            // [4] device counters: groups, bad entries, clusters, members placed
  int32_t *ngroups = nullptr;        // == ctr
};

// Flow-based refinement of one block pair (Section 5), allocated at the first flow call of a
// context; the network arrays grow to the largest pair seen.  The Lawler network of the pair's
// induced subhypergraph: node 0 the contracted source terminals, node 1 the contracted sink
// terminals, nodes 2 .. NV-1 the region vertices in increasing ID, then per relevant net (two or
// more distinct endpoints) e_in = NV + 2 r and e_out = e_in + 1.  Net r owns the arc block
// [rbase[r], rbase[r] + 2 + 4 ends): e_in -> e_out and its reverse, then per endpoint j the arcs
// x -> e_in, e_in -> x, e_out -> x, x -> e_out; arc a's reverse is a ^ 1.
struct FlowState {
  // per net / per vertex, sized at first use
  int32_t *cnt_a = nullptr, *cnt_b = nullptr;  // [m] pins in block a / b
  int32_t *nexp = nullptr;      // [m] net expanded by the region search
  int32_t *ends = nullptr;      // [m] distinct endpoints
  int32_t *asize = nullptr;     // [m] arc block size (0 if not relevant)
  int32_t *rel = nullptr;       // [m] relevant
  int64_t *nbase = nullptr;     // [m + 1] arc block offsets
  int64_t *nrid = nullptr;      // [m + 1] relevant index
  int32_t *lvl = nullptr;       // [n] region search level (-1 unseen)
  int8_t *rmark = nullptr;      // [n] 1: region of a, 2: region of b
  int32_t *wtmp = nullptr;      // [n] scan input
  int64_t *wscan = nullptr;     // [n + 1] scan output
  int32_t *vnode = nullptr;     // [n] network node of a vertex of the pair, -1 otherwise
  int32_t *nvert = nullptr;     // [n] vertex of region node 2 + i
  int32_t *vcnt = nullptr;      // [n + 2] arcs per vertex node, then fill cursors
  int64_t *voffn = nullptr;     // [n + 3] vertex node adjacency offsets
  int64_t *sc = nullptr;        // [16] scalars
  int64_t *hsc = nullptr;       // [16] pinned host mirror
  // per relevant net
  int32_t *rnet = nullptr, *rends = nullptr;  // [m]
  int64_t *rbase = nullptr;                   // [m]
  // network, grown on demand
  int64_t node_cap = 0, arc_cap = 0, vadj_cap = 0;
  int32_t *head = nullptr, *tail = nullptr;   // [arcs]
  int64_t *res = nullptr;                     // [arcs] residual capacity
  int64_t *vadj = nullptr;                    // [vertex-node arc entries] first arc of each endpoint
  int32_t *h = nullptr;                       // [nodes] height
  int64_t *ex = nullptr;                      // [nodes] excess (net inflow)
  uint8_t *term = nullptr;                    // [nodes] 0 free, 1 source, 2 sink
  uint8_t *rs = nullptr, *rt = nullptr;       // [nodes] reaches from the sources / reaches the sinks
  int32_t *front[3] = {nullptr, nullptr, nullptr};  // [nodes] breadth-first frontiers (rotating)
  int32_t *fcnt = nullptr;                    // [6] their sizes, then what k_fl_deep left
  int32_t *hfront = nullptr;                  // [3] pinned host copy of the latter
};

// The pieces of an iteration: what the host launches for a phase.
enum TickKind : int { kTickJet = 0, kTickRb = 1, kTickRoll = 2 };
constexpr int kTickPieces = 3;
constexpr int kSides = 3;
// Rounds of a union's rebalancing piece: an iteration of one hypergraph takes two to three, and while some
// of them finish theirs the next Jet launches cover the others only.  96 hypergraphs with 1 / 2 / 3 / 4
// rounds: 168 / 142 / 126 / 139 ms.
constexpr int32_t kUnionRounds = 3;
// Pins from which the afterburner's kernels run beside each other.  It pays on smaller levels too (beside /
// after each other, row-net k = 64: 10,000 rows 46 / 55 ms, 40,000 15.7 / 18.8, 250,000 8.5 / 10.5; SAT-like
// k = 32: 10,000 40.5 / 42.9, 100,000 104 / 117); the line spares small contexts the three streams.
constexpr int64_t kForkPins = 1 << 19;

constexpr int32_t kLaneDegreeDefault = 24;  // JET_OPT_CAND_LANE_DEGREE unless set

struct Ctx {
  hipStream_t stream = nullptr;
  int32_t n = 0, m = 0, k = 0, nw_words = 1;  // nw_words = ceil(k/64) words per mask
  int64_t p = 0;
  double eps = 0.0;
  int64_t W = 0, A = 0, lmax = 0;
  bool unit_nw = true, unit_vw = true;
  int32_t stamp = 0;  // iteration stamp for locks
  // move application: net-centric when (incident nets of the moves) * apply_divisor >= p,
  // vertex-centric otherwise (0 = always vertex-centric); environment JET_APPLY_DIVISOR overrides
  // (16 against 32 on one card: row-net 1M 11.07 / 10.92 ms, rebalancing 1M 1.24 / 1.20, a V-cycle 513 /
  // 504, SAT-like 300k 127.7 / 128.4; 64 is slower than 32 on all four)
  int32_t apply_divisor = 32;
  // the path the device took at the last application of each kind (Jet moves, rebalancing moves),
  // used to size the next launch of that kind
  bool wide_hint[2] = {false, false};
  bool wide_enabled = false;  // JET_OPT_APPLY_WIDE
  int32_t lane_degree = kLaneDegreeDefault;  // JET_OPT_CAND_LANE_DEGREE
  int32_t cand_xcd = 1;       // JET_OPT_CAND_XCD: contiguous vertex ranges per XCD in the candidate kernels
  int32_t rb_xcd = 1;         // JET_OPT_RB_XCD: contiguous list ranges per XCD in the rebalancing gain pass
  int32_t apply_xcd = 0;      // JET_OPT_APPLY_XCD: contiguous move and chunk ranges per XCD in the application
  int32_t graph_kernels = 1;  // JET_OPT_GRAPH_KERNELS: graph-specialised afterburner when every net has two pins
  int32_t flow_workers = 4;   // JET_OPT_FLOW_WORKERS: block pairs of a matching refined at once
  int32_t sel_split_min = 1 << 18;  // JET_OPT_SEL_SPLIT_MIN
  int32_t sel_slices = 0;     // most workgroups per block in the split pass; 0 = by the number of blocks
  int64_t grid_cap = 2048;    // JET_OPT_GRID: workgroups of the persistent (grid-stride) kernels

  // hypergraph
  int64_t *off = nullptr;    // [m+1]
  int32_t *pins = nullptr;   // [p]
  int32_t *nw = nullptr;     // [m] or null
  int32_t *vw = nullptr;     // [n] or null
  int64_t *voff = nullptr;   // [n+1] incidence offsets
  int32_t *inc = nullptr;    // [p] incident nets, ascending per vertex
  int32_t *sumw = nullptr;   // [n] omega(I(v))
  int32_t *adj = nullptr;    // [p] graphs only (every net of two pins): the other pin of net inc[q]

  // net scheduling (built once at init)
  int4 *chunks = nullptr;    // [nchunks] (first net, nets, pins, first pin) of runs of consecutive small nets
  uint8_t *pnet = nullptr;   // [p] index of the pin's net inside its chunk (chunked nets only)
  int32_t nchunks = 0;
  int32_t *mid_nets = nullptr;  // nets with kSmallNet < |e| <= kMediumNet, largest first
  int32_t nmid = 0;
  int32_t nmid_large = 0;       // leading entries of mid_nets with |e| > kMediumSmall
  int32_t *big_nets = nullptr;  // nets with |e| > kMediumNet, largest first
  int32_t nbig = 0;
  int32_t nbig_over = 0;        // leading entries of big_nets with |e| > kBigCap
  int32_t *hubs = nullptr;      // vertices with more than kHubDegree incident nets
  int32_t nhubs = 0;
  int2 *ovf_list = nullptr;     // [nbig_over] (index into big_nets, net) needing the scratch path
  int64_t *ovf_off = nullptr;   // [nbig_over + 1] scratch offsets: 2 |e| event slots per net
  unsigned long long *ovf_ka = nullptr, *ovf_kb = nullptr;  // event keys (ping-pong)
  uint32_t *ovf_ma = nullptr, *ovf_mb = nullptr;            // event block | kind<<8

  // partition state
  int32_t *phi = nullptr;     // [m*k] pin counts (when some net has more than 65,535 pins)
  uint16_t *phi16 = nullptr;  // [m*k] pin counts, 16-bit (otherwise); exactly one is allocated
  uint64_t *ns = nullptr;     // [m * 2 * nw_words]: connectivity mask words, then "exactly one pin" words
  uint64_t *rec = nullptr;    // [n] candidate record: gain (low 32), target (bits 32-39), source (40-47)
  uint32_t *inm = nullptr;    // candidate bitmask, padded to a multiple of 256 vertices
  int32_t *rg = nullptr;      // [n] recomputed gains
  int32_t rg_copies = 1;      // private copies of rg the afterburner accumulates into (small levels)
  int32_t *rgx = nullptr;     // [rg_copies * n] those copies, zero between calls
  int32_t *lockstamp = nullptr;  // [n] stamp of the iteration that last moved v
  int32_t *best = nullptr;    // [n] rollback snapshot
  int4 *moves = nullptr;      // [n] move list (v, from, to, weight)
  uint8_t *mvfrom = nullptr;  // [n] block a listed move left, 0xff otherwise (vertices the listing pass walked)
  int32_t *bigmv = nullptr;   // [n] positions in the move list of the moves counted by n_bigmv
  int32_t *rb_list = nullptr; // [n] non-hub vertices that may move in the current rebalancing round
  int32_t *rb_slot = nullptr; // [n] the entry slot of each listed vertex (its block's region)
  int32_t *rb_hlist = nullptr; // [nhubs] hubs (indices into hubs) that may move in the current rebalancing round
  unsigned long long *hub_words = nullptr; // [kHubGrid / 2 * (k + 1)] sums of shared hubs in the running hub pass
  int64_t *lstat = nullptr;   // [5] level statistics scratch
  float *tau_io = nullptr;    // [17] learned temperature: features in, temperature out

  // rebalancing
  uint32_t *rb_keys = nullptr;   // [n * 8] entries: 5 key words, v, target, weight
  uint32_t *rb_keys2 = nullptr;  // [n * 8] entries kept by the grid-wide first selection pass
  unsigned long long *rb_gw = nullptr;  // [kMaxK * 256] first-byte histogram per block: weights (zero between rounds)
  uint32_t *rb_gc = nullptr;            // [kMaxK * 256] and entry counts
  int32_t *rb_target = nullptr;  // [n] selected target for inspection (-1)

  // union context (batch): H hypergraphs with the same k; H == 1 otherwise
  int32_t H = 1;
  uint16_t *vhg = nullptr;       // [n] hypergraph of each vertex (union only)
  uint16_t *nhg = nullptr;       // [m] hypergraph of each net (union only)
  LoopCtl *lcs = nullptr;        // [H] per-hypergraph loop records (== lc when H == 1)
  LoopCtl *hlcs = nullptr;       // [H] pinned host mirror (== hlc when H == 1)
  std::vector<int32_t> hg_v0;    // [H+1] first vertex of each hypergraph (multiples of kUnionTile)
  std::vector<int32_t> hg_n;     // [H] its vertex count (the rest up to the next start is padding)
  std::vector<int32_t> hg_e0;    // [H+1] first net of each hypergraph
  ActList *act = nullptr;        // [kActLists] device lists of the hypergraphs per phase
  int32_t *ht0 = nullptr;        // [H+1] device: first tile of each hypergraph
  int32_t *hch0 = nullptr;       // [H+1] device: first chunk of each hypergraph
  std::vector<int64_t> hg_lmax, hg_A;  // [H] balance limit and ceil(W/k) per hypergraph
  std::vector<double> hg_eps;    // [H]
  std::vector<int64_t> hg_W;     // [H]
  // device-resident loop
  LoopCtl *lc = nullptr;         // device loop record (the gate record of a union)
  LoopCtl *hlc = nullptr;        // pinned host mirror
  unsigned long long *mail = nullptr;  // [1] pinned host memory the control kernel writes (read_mail)
  int32_t *cpart = nullptr;      // [n] the partition the loop works on (copied in and out per call)
  jet_trace *dtrace = nullptr;   // device iteration records
  int32_t dtrace_cap = 0;
  hipStream_t gstream = nullptr; // stream the iteration graph is captured on
  hipStream_t side[kSides] = {};  // branches of the afterburner beside `stream`
  hipEvent_t fork = nullptr, join[kSides] = {};
  // captured pieces of the loop (TickKind): Jet phase, rb_slots rebalancing rounds, rollback, each with
  // its control kernel
  hipGraph_t graph[kTickPieces] = {};
  hipGraphExec_t gexec[kTickPieces] = {};
  bool use_graph = true;         // JET_OPT_GRAPH
  int32_t rb_slots = 1;          // JET_OPT_RB_SLOTS: rounds of one rebalancing piece (a union: kUnionRounds)
  int32_t replays = 2;           // JET_OPT_REPLAYS: control kernels in flight while another piece is launched ahead
  int64_t polls = 0;             // host polls of the last call (diagnostic)
  int64_t replays_done = 0;      // graph replays or eager ticks of the last call
  DevProf *dprof = nullptr;      // device timing accumulators
  CoState *co = nullptr;         // clustering of the coarsening phase (allocated on first use)
  FlowState *fl = nullptr;       // flow-based refinement (allocated on first use)
  int64_t co_slots = (int64_t)1 << 28;  // JET_OPT_CO_TABLE_SLOTS: rating-table slots of one launch
  DevStatus *st = nullptr;       // device status
  DevStatus *hst = nullptr;      // pinned host mirror
  int64_t *scan_tmp = nullptr;   // scan scratch
  int64_t scan_tmp_len = 0;

  // instrumentation
  bool prof = false;
  int64_t n_low = 0, p_low = 0;  // vertices / incidences handled by the non-hub candidate kernel
  int64_t max_low_degree = 0;    // largest degree among them
  uint32_t prof_mask = 0xffffffffu;       // families marked while profiling is on
  double wall_khz = 100000.0;             // device wall clock rate

  std::string last_error;
};

// Workgroups of kernel K that the card holds at once, a multiple of its eight XCDs.  A grid-stride
// kernel launched with more leaves the rest for a second, mostly empty wave: 2,048 workgroups of a
// kernel that fits 1,536 take as long as two rounds.
template <auto K>
int64_t resident_grid(int block) {
  static const int64_t g = [](int b) {
    int per_cu = 0, dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, K, b, 0) != hipSuccess || per_cu < 1)
      return (int64_t)2048;
    return std::max<int64_t>(8, (int64_t)per_cu * cus / 8 * 8);
  }(block);
  return g;
}
template <auto K>
struct KernelTag {  // a kernel as a type
  static constexpr auto value = K;
};
// Launches K with one workgroup per `blocks`, at most as many as are resident and c.grid_cap allows.
template <auto K, typename... A>
void launch_resident(Ctx &c, int64_t blocks, int block, A... args) {
  const int64_t g = std::max<int64_t>(1, std::min<int64_t>({blocks, c.grid_cap, resident_grid<K>(block)}));
  hipLaunchKernelGGL(K, dim3((unsigned)g), dim3((unsigned)block), 0, c.stream, args...);
}

// Unit net weights: one lane per vertex (the candidate and rebalancing gain passes) instead of eight.
// One lane is right while the vertices are light (mean degree below lane_degree) and more than a few:
// 2,000 to 30,000 vertices are 32 to 500 waves of one-lane vertices on 1,024 SIMDs, and their refinement
// took 2 to 8% longer than with eight lanes; from 65,000 on local hypergraphs are 1% (260,000: 18%) faster
// with one.  A lane degree other than the default decides at every size.
constexpr int32_t kFewVertices = 1 << 15;
inline bool light_lanes(const Ctx &c) {
  return (c.n > kFewVertices || c.lane_degree != kLaneDegreeDefault) && c.p_low < (int64_t)c.lane_degree * c.n_low;
}

// Workgroups of a move application: those that fit (at most kApplyGrid), more for `groups` groups of chunks,
// and never fewer than the kWeightBlocks that sum the block weights of a list (a card partition of 32
// CUs may fit fewer).
constexpr int kApplyGrid = 2048;
constexpr unsigned kWeightBlocks = 64;
inline int64_t apply_grid(int64_t fits, int64_t groups) {
  const int64_t g = std::min<int64_t>(kApplyGrid, fits);
  return std::max<int64_t>({g, std::min<int64_t>(groups, 1 << 20), (int64_t)kWeightBlocks});
}

// the union view of a context for the kernels
inline Union union_of(const Ctx &c) {
  return c.H > 1 ? Union{c.lcs, c.vhg, c.nhg, c.act, c.ht0, c.hch0}
                 : Union{nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};
}

// Mark a family's launches for the device timing when instrumentation is on (no-ops otherwise);
// the marks are gated like the family (want = its loop phase, or kPhAny outside the loop).
// bytes: static algorithmic bytes; per_inc: bytes per scanned incidence (families whose byte count
// depends on device counters add those on the device).
int prof_begin(Ctx &c, int fam, const LoopCtl *lc, int32_t want);
void prof_end(Ctx &c, int token, const LoopCtl *lc, int32_t want, double bytes, double per_inc);

// ------------------------------------------------------------------ launch wrappers
// All launch on c.stream; they return hipSuccess or the launch error.

// setup (k_setup.hip)
hipError_t launch_check_pins(Ctx &c);
hipError_t launch_degrees(Ctx &c, int32_t *deg);
hipError_t launch_exclusive_scan_i32_to_i64(Ctx &c, const int32_t *in, int64_t *out, int64_t len);
hipError_t launch_fill_incidence(Ctx &c, int64_t *cursor);
hipError_t launch_sort_incidence(Ctx &c);
hipError_t launch_check_weights(Ctx &c);

// state (k_state.hip)
hipError_t launch_check_part(Ctx &c, const int32_t *part);
hipError_t launch_build_phi(Ctx &c, const int32_t *part, int32_t *phi);
// the context's counts and connectivity words
hipError_t launch_build_counts(Ctx &c, const int32_t *part);
hipError_t launch_block_weights(Ctx &c, const int32_t *part);
hipError_t launch_km1_from_ns(Ctx &c);
// one network evaluation on the network's stream: raw features x (device [16]) -> *tau (host);
// y is device scratch for the output
int mlp_infer_one(jet_mlp *net, const float *x, float *y, float *tau);

// cut nets, their weight, net weight total, largest net, boundary vertices (device int64[5])
hipError_t launch_level_stats(Ctx &c, int64_t *out5);

// iteration (k_iter.hip)
// Launches of the iteration's phases.  lc == nullptr: a launch outside the loop (never gated, the
// scalar arguments are used); otherwise every kernel returns at once unless lc->phase is the phase
// the launch belongs to, and the stamp, temperature and deadzone are read from lc.
hipError_t launch_candidates(Ctx &c, const int32_t *part, int32_t locked_stamp, const uint8_t *lock_bytes,
                             int32_t tau_q, const LoopCtl *lc = nullptr);
hipError_t launch_export_candidates(Ctx &c, int32_t *t, int32_t *g, uint8_t *in_m);
hipError_t launch_import_candidates(Ctx &c, const int32_t *part, const int32_t *t, const int32_t *g,
                                    const uint8_t *in_m);
// expects n_ovf == 0 (cleared by launch_candidates or launch_reset_counters)
hipError_t launch_afterburner(Ctx &c, const int32_t *part, const LoopCtl *lc = nullptr);
enum : int32_t { kResetCandidates = 1, kResetMoves = 2 };
hipError_t launch_reset_counters(Ctx &c, int32_t what);
hipError_t launch_afterburner_overflow(Ctx &c, RgSink sink, const LoopCtl *lc);  // k_ab_large.hip
bool ab_branches(const Ctx &c);
hipError_t launch_select_moves(Ctx &c, int32_t *part, const LoopCtl *lc);
// wide: size the net-centric grids for that path (a performance hint; the device decides the path)
hipError_t launch_apply_moves(Ctx &c, int32_t *part, bool wide, const LoopCtl *lc = nullptr, int32_t want = kPhAny);
hipError_t launch_diff_moves(Ctx &c, int32_t *part, const int32_t *target, const LoopCtl *lc);

// rebalancing (k_rebal.hip)
hipError_t launch_rebalance_round(Ctx &c, int32_t *part, int64_t dz, int32_t *sel_target,
                                  const LoopCtl *lc = nullptr);

// the device-resident loop (k_loop.hip)
// the launches of one piece of an iteration, gated by c.lc
hipError_t launch_tick(Ctx &c, int kind);
// loop records for a call: the host wrote each hypergraph's parameters into c.lcs; this completes
// them from the status block (metric, overload, first phase) and sets the gate record
hipError_t launch_loop_init(Ctx &c);
// zeroes the candidate bits where the candidate kernel of this context only sets them
hipError_t launch_clear_candidate_bits(Ctx &c);
hipError_t launch_fill_u32(Ctx &c, uint32_t *p, int64_t count, uint32_t value, const LoopCtl *lc, int32_t want);

// k_hub.hip: vertices with more than kHubDegree incident nets
constexpr int kHubGrid = 2048;  // workgroups of a hub pass at most
hipError_t launch_candidates_hub(Ctx &c, const int32_t *part, int32_t locked_stamp, const uint8_t *lock_bytes,
                                 int32_t tau_q, const LoopCtl *lc);
hipError_t launch_rb_hubs(Ctx &c, const int32_t *part, int64_t dz, const LoopCtl *lc);

// k_graph.hip: graph-specialised afterburner (every net of two pins)
hipError_t launch_build_adj(Ctx &c);
bool graph_afterburner(const Ctx &c);
hipError_t launch_ab_graph(Ctx &c, const int32_t *part, const LoopCtl *lc, int32_t want);

constexpr int kCoLdsTable = 512;  // largest rating table (slots) that needs no global scratch
// Rating-table slots of a vertex with d = sum of (|e| - 1) over its nets: a power of two at least twice the
// number of clusters it can meet (at most min(d, n)), so probing stays short.  The host lays out the
// tables above kCoLdsTable by it, the rating kernel finds its own by it.
__host__ __device__ inline int64_t co_table(int64_t d, int64_t n) {
  if (d <= 0) return 0;
  const int64_t want = 2 * (d < n ? d : n);
  return want <= 16 ? 16 : (int64_t)1 << (64 - __builtin_clzll((unsigned long long)(want - 1)));
}
// k_coarsen.hip: synchronous clustering (Section 6, Algorithm 4)
hipError_t launch_co_prepare(Ctx &c);
hipError_t launch_co_init(Ctx &c, int32_t *label, int64_t *cw);
hipError_t launch_co_check(Ctx &c, const int32_t *list, int64_t len, int32_t *bad);
hipError_t launch_co_rate(Ctx &c, const int32_t *verts, int64_t a, int64_t b, int64_t base, const int32_t *label,
                          const int64_t *cw, int64_t wmax);
hipError_t launch_co_settle(Ctx &c, const int32_t *verts, int64_t len, int32_t *label, int64_t *cw, int64_t wmax,
                            int32_t *t_out);
hipError_t launch_co_count(Ctx &c, const int32_t *label, int32_t *count);

// flow-based refinement (k_flow.hip); each returns a JET_* code and sets c.last_error on failure
struct FlowPairResult {
  int64_t old_cut = 0, new_cut = 0;
  int64_t arcs = 0;  // sum over the maximum-flow iterations of the network's arcs
  int32_t iterations = 0, region_a = 0, region_b = 0, moved = 0, replaced = 0;
};
int flow_region(Ctx &c, const int32_t *part, int32_t a, int32_t b, int32_t alpha, int8_t *region);
int flow_mincut(Ctx &c, const int32_t *part, int32_t a, int32_t b, const int8_t *term, int64_t *flow,
                uint8_t *in_sr, uint8_t *in_tr);
int flow_pair(Ctx &c, int32_t *part, int32_t a, int32_t b, int32_t alpha, FlowPairResult *r);
struct FlowRefineResult {
  int64_t km1_in = 0, km1_out = 0;
  int64_t arcs = 0;
  int32_t rounds = 0, matchings = 0, pairs = 0, accepted = 0, flow_calls = 0, moved = 0;
};
int flow_refine(Ctx &c, int32_t *part, int32_t alpha, int32_t max_rounds, FlowRefineResult *r);
void flow_free(Ctx &c);

}  // namespace jet
