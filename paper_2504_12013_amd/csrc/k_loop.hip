// The Jet loop of Algorithm 1 kept on the device.  The decisions of the loop (rebalance or not,
// strict improvement of the key (overload, metric), snapshot, iteration limit, fixed point, end of a
// temperature round and rollback to its best partition) are taken by one small control kernel after
// each phase on a loop record (LoopCtl); every kernel of the iteration returns at once unless the
// record is in the phase it belongs to.  The Jet phase, a rebalancing round and the rollback, each
// followed by its control kernel, are the pieces of an iteration; the host captures each in a HIP
// graph once per context and launches them by what the control kernel last reported in pinned memory.
// A union's hypergraphs may be in several phases at once: a piece then works on those in its phase.
// Pieces after the loop finished do nothing.  The sequence of states is exactly that of the host loop it replaces (one Jet phase, then rebalancing rounds while a
// block is overloaded, a round moved something and the cap allows, then the key), so results and
// per-iteration records do not depend on which pieces were launched ahead.
//
// The control kernel that leaves a phase also enters the next one (iteration stamp, counters, the
// round's needs and list regions), and the next Jet phase's candidate pass, which reads every
// vertex's block anyway, takes the snapshot of an improving iteration.  A launch costs 2 to 5 us here
// even when its gate is closed, so a rebalancing round of 2,000 vertices went from 15 launches to 5.
#include <algorithm>

#include "dev_util.h"
#include "jet_internal.h"

namespace jet {

namespace {

// ------------------------------------------------------------------ the loop's decisions

// Start of a Jet phase: a new iteration stamp, so the vertices moved by the previous iteration's
// Jet phase (stamped stamp - 1) are the locked ones.
__device__ __forceinline__ void begin_jet(LoopCtl &r) {
  r.stamp += 1;
  r.lock_was_any = r.lock_any;
  set_phase(r, kPhJet);
}

// Completes the record the host wrote (parameters, limits, stamp) from the state build_state left
// (metric, block weights): the first round's key and the first phase.
__device__ __forceinline__ void first_phase(LoopCtl &r, int64_t ovl, int64_t km1) {
  r.km1 = km1;
  r.km1_in = km1;
  r.best_ovl = ovl;
  r.best_km1 = km1;
  r.improved = 1;  // the start is the first round's best: the first candidate pass takes the snapshot
  if (r.rb_only) set_phase(r, (ovl > 0 && r.max_rb > 0) ? kPhRb : kPhDone);  // jet_rebalance
  else begin_jet(r);
}

// End of an iteration: the key (overload, metric) against the round's best (strict, lexicographic),
// the iteration record, the limit of non-improving iterations, the round's cap and the fixed point.
__device__ __forceinline__ void end_iteration(LoopCtl &r, int64_t ovl, jet_trace *trace) {
  const int64_t km1 = r.km1;
  r.it += 1;
  r.round += 1;
  if (ovl < r.best_ovl || (ovl == r.best_ovl && km1 < r.best_km1)) {
    r.best_ovl = ovl;
    r.best_km1 = km1;
    r.improved = 1;
    r.round = 0;
  }
  r.iterations += 1;
  r.rebalance_rounds += r.rb_rounds;
  if (trace && r.ntrace < r.trace_cap) {
    jet_trace t;
    t.km1 = km1;
    t.overload = ovl;
    t.n_cand = r.n_cand;
    t.n_moved = r.n_moved;
    t.rb_rounds = r.rb_rounds;
    t.rb_moved = r.rb_moved;
    trace[r.ntrace] = t;
  }
  r.ntrace += 1;
  // nothing moved, nothing rebalanced and nothing was locked: the next iteration would repeat it
  const bool fixed = r.n_moved == 0 && r.rb_moved == 0 && r.lock_was_any == 0;
  if (r.round >= r.limit || r.it >= r.max_iters || fixed) set_phase(r, kPhRoll);
  else begin_jet(r);
}

// After the Jet phase's moves are applied: its counts, the locks it leaves, and whether a
// rebalancing round follows (Algorithm 1: rebalance while a block is overloaded).  The candidate
// pass has taken the previous improvement's snapshot.
__device__ __forceinline__ void after_jet(LoopCtl &r, int64_t ovl, int64_t km1, int32_t moved, int32_t cand,
                                          jet_trace *trace) {
  r.km1 = km1;
  r.improved = 0;
  r.n_cand = cand;
  r.n_moved = moved;
  r.lock_any = moved > 0 ? 1 : 0;
  r.moves_executed += moved;
  r.rb_rounds = 0;
  r.rb_moved = 0;
  if (ovl > 0 && r.max_rb > 0) set_phase(r, kPhRb);
  else end_iteration(r, ovl, trace);
}

// After a rebalancing round's moves are applied: another round while a block is still overloaded,
// the round moved a vertex and the cap allows (Section 4.3).
__device__ __forceinline__ void after_rb(LoopCtl &r, int64_t ovl, int64_t km1, int32_t moved, jet_trace *trace) {
  r.km1 = km1;
  r.rb_rounds += 1;
  r.rb_moved += moved;
  if (ovl != 0 && r.rb_rounds < r.max_rb && moved != 0) return;
  if (r.rb_only) {
    r.rebalance_rounds += r.rb_rounds;
    set_phase(r, kPhDone);
  } else {
    end_iteration(r, ovl, trace);
  }
}

// After the rollback's moves are applied: the next temperature round starts from the round's
// best partition with no locks, or the loop is done.
__device__ __forceinline__ void after_roll(LoopCtl &r, int64_t ovl, int64_t km1) {
  r.km1 = km1;
  r.tau_r += 1;
  if (r.tau_r >= r.num_tau) {
    set_phase(r, kPhDone);
    return;
  }
  r.tau_q = r.tau_qs[r.tau_r];
  r.stamp += 2;  // the round's first iteration sees no lock
  r.round = 0;
  r.it = 0;
  r.lock_any = 0;
  r.best_ovl = ovl;
  r.best_km1 = km1;
  begin_jet(r);
}

// want: the phase just executed, kPhAny at the start of a call
__device__ __forceinline__ void advance(LoopCtl &r, int32_t want, int64_t ovl, int64_t km1, int32_t moved,
                                        int32_t cand, jet_trace *trace) {
  if (want == kPhJet) after_jet(r, ovl, km1, moved, cand, trace);
  else if (want == kPhRb) after_rb(r, ovl, km1, moved, trace);
  else if (want == kPhRoll) after_roll(r, ovl, km1);
  else first_phase(r, ovl, km1);
}

// ------------------------------------------------------------------ control kernels

// The counters of a phase start at zero.
__device__ __forceinline__ void clear_counters(DevStatus *st) {
  st->n_moves = 0;
  st->n_ovf = 0;
  st->n_bigmv = 0;
  st->mv_inc = 0;
  st->rb_nlist = 0;
  st->rb_nhub = 0;
}

// Tells the host where the loop is (one store to pinned memory).
__device__ __forceinline__ void post(unsigned long long *mail, uint32_t seq, int32_t mask, int32_t rb_rounds,
                                     bool last, int32_t err) {
  const unsigned long long rb = (unsigned long long)min(rb_rounds, (1 << kMailRbBits) - 1);
  __hip_atomic_store(mail,
                     (unsigned long long)(seq & kMailSeqMask) | ((unsigned long long)mask << kMailMaskSh) |
                         (rb << kMailRbSh) | ((last ? 1ull : 0ull) << kMailLastSh) |
                         ((err != 0 ? 1ull : 0ull) << kMailErrSh),
                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ void post(unsigned long long *mail, uint32_t seq, const LoopCtl &r, int32_t err) {
  post(mail, seq, r.phase_mask, r.rb_rounds, r.round + 1 >= r.limit || r.it + 1 >= r.max_iters, err);
}

// One hypergraph: one thread per block.  Record, block weights and metric slots are loaded at
// once and the decision runs on the copy in LDS: a single thread walking them in global memory took
// 7 us at k = 64 and 12 us at k = 128, this takes 3 us.  When a rebalancing round follows, its needs
// (bw - Lmax) and list regions are set here.
constexpr int kCtlOne = 128;
static_assert(kCtlOne >= kMaxK && kCtlOne >= kKm1Slots && kKm1Slots == kWave, "one thread per block and slot");
__global__ __launch_bounds__(kCtlOne) void k_control(LoopCtl *lc, DevStatus *st, int32_t k, int64_t lmax,
                                                     int32_t want, jet_trace *trace, unsigned long long *mail) {
  __shared__ LoopCtl r;
  __shared__ int64_t s_ovl[kCtlOne / kWave], s_cnt[kCtlOne / kWave], s_km1;
  const int b = threadIdx.x, w = b / kWave;
  for (int i = b; i < (int)(sizeof(LoopCtl) / 4); i += kCtlOne)
    reinterpret_cast<int32_t *>(&r)[i] = reinterpret_cast<const int32_t *>(lc)[i];
  const int64_t bw = b < k ? st->bw[b] : 0;
  const int32_t bc = b < k ? st->bcnt[b] : 0;
  int64_t slot = b < kKm1Slots ? st->slot[b].km1 : 0;
  int32_t cand = b < kKm1Slots ? (int32_t)st->slot[b].n_cand : 0;
  const int64_t km1_base = st->km1;
  const int32_t moved = st->n_moves, err = st->err;
  const int64_t over = b < k ? max(bw - lmax, (int64_t)0) : 0;
  int64_t mx = over;
#pragma unroll
  for (int o = kWave / 2; o >= 1; o >>= 1) mx = max(mx, (int64_t)__shfl_xor(mx, o, kWave));
  slot = wave_sum(slot);
  cand = wave_sum(cand);  // the first wave's counts
  const int64_t cnt = over > 0 ? bc : 0, incl = wave_incl_scan(cnt);
  if (lane_id() == kWave - 1) {
    s_ovl[w] = mx;
    s_cnt[w] = incl;
    if (w == 0) s_km1 = km1_base + slot;
  }
  __syncthreads();
  const uint32_t seq = r.seq + 1;
  if (want != kPhAny && r.phase != want) {  // block-uniform
    if (b == 0) {
      lc->seq = seq;
      post(mail, seq, r, err);
    }
    return;
  }
  __syncthreads();  // every thread has read the phase
  if (b == 0) {
    advance(r, want, max(s_ovl[0], s_ovl[1]), s_km1, moved, cand, trace);
    r.seq = seq;
    post(mail, seq, r, err);
    st->km1 = s_km1;
    clear_counters(st);
  }
  if (b < kKm1Slots) st->slot[b] = CtrSlot{};
  __syncthreads();
  if (r.phase == kPhRb && b < k) {
    st->rb_need[b] = over;
    st->rb_count[b] = 0;
    st->rb_kept[b] = 0;
    st->rb_off[b] = incl - cnt + (w ? s_cnt[0] : 0);
    if (b == 0) st->rb_off[k] = s_cnt[0] + s_cnt[1];
  }
  for (int i = b; i < (int)(sizeof(LoopCtl) / 4); i += kCtlOne)
    reinterpret_cast<int32_t *>(lc)[i] = reinterpret_cast<const int32_t *>(&r)[i];
}

constexpr int kCtlThreads = 256;

// Union: the lists of hypergraphs per phase, with the prefix sums of their tiles and chunks, in
// hypergraph order (one workgroup; hypergraphs, tiles and chunks packed into one block scan: at most
// 4,096 hypergraphs, 2^23 tiles of 256 vertices and 2^27 chunks).
__device__ __forceinline__ void build_lists(const LoopCtl *lcs, int32_t H, ActList *act, const int32_t *ht0,
                                            const int32_t *hch0) {
  __shared__ unsigned long long sm[kCtlThreads / kWave + 1];
  const int tid = threadIdx.x;
  unsigned long long run[kActLists] = {};
  constexpr int kTileSh = 13, kChunkSh = 37;
  constexpr unsigned long long kTileMask = (1ull << (kChunkSh - kTileSh)) - 1ull;
  for (int32_t base = 0; base < H; base += kCtlThreads) {  // block-uniform trip count
    const int32_t hg = base + tid;
    int32_t ph = kPhDone;
    unsigned long long one = 0ull;
    if (hg < H) {
      ph = lcs[hg].phase;
      one = 1ull | ((unsigned long long)(uint32_t)(ht0[hg + 1] - ht0[hg]) << kTileSh) |
            ((unsigned long long)(uint32_t)(hch0[hg + 1] - hch0[hg]) << kChunkSh);
    }
#pragma unroll
    for (int L = 0; L < kActLists; ++L) {
      const bool in = hg < H && ph == (L == kActJet ? kPhJet : L == kActRb ? kPhRb : kPhRoll);
      unsigned long long tot;
      const unsigned long long at = run[L] + block_excl_scan<kCtlThreads>(in ? one : 0ull, sm, &tot);
      if (in) {
        const int32_t i = (int32_t)(at & ((1ull << kTileSh) - 1ull));
        act[L].hg[i] = hg;
        act[L].tpref[i] = (int32_t)((at >> kTileSh) & kTileMask);
        act[L].cpref[i] = (int32_t)(at >> kChunkSh);
      }
      run[L] += tot;
    }
  }
  if (tid == 0) {
#pragma unroll
    for (int L = 0; L < kActLists; ++L) {
      const int32_t i = (int32_t)(run[L] & ((1ull << kTileSh) - 1ull));
      act[L].cnt = i;
      act[L].tpref[i] = (int32_t)((run[L] >> kTileSh) & kTileMask);
      act[L].cpref[i] = (int32_t)(run[L] >> kChunkSh);
    }
  }
}

// Union: one thread per hypergraph, then the gate record's phase mask from all records (a union's
// gate is a record of its own) and the lists.  The move counts start at zero for the next phase; the
// rebalancing needs are set by the round's own preparation (one workgroup over all segments).
__global__ __launch_bounds__(kCtlThreads) void k_control_union(LoopCtl *lcs, int32_t H, LoopCtl *gate, DevStatus *st,
                                                               int32_t k, int32_t want, unsigned long long *mail,
                                                               Union u) {
  __shared__ int32_t smask;
  if (threadIdx.x == 0) smask = 0;
  __syncthreads();
  int32_t m = 0;
  for (int32_t hg = threadIdx.x; hg < H; hg += kCtlThreads) {
    int32_t pm = lcs[hg].phase_mask;
    if (want == kPhAny || (pm >> want) & 1) {
      LoopCtl r = lcs[hg];
      const int64_t *bw = st->bw + (int64_t)hg * k;
      int64_t ovl = 0;
      for (int32_t b0 = 0; b0 < k; b0 += 8) {  // eight loads in flight
        int64_t x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = b0 + j < k ? bw[b0 + j] : 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) ovl = max(ovl, x[j] - r.lmax);
      }
      const int64_t km1 = (want == kPhAny ? 0 : r.km1) + st->hkm1[hg];
      st->hkm1[hg] = 0;
      advance(r, want, ovl, km1, st->hmoves[hg], 0, nullptr);
      lcs[hg] = r;
      pm = r.phase_mask;
    }
    st->hmoves[hg] = 0;
    m |= pm;
  }
  if (m) atomicOr(&smask, m);
  __syncthreads();
  if (threadIdx.x == 0) {
    gate->phase_mask = smask;
    gate->seq += 1;
    post(mail, gate->seq, smask, 0, false, st->err);
    clear_counters(st);
  }
  if (threadIdx.x < kKm1Slots) st->slot[threadIdx.x] = CtrSlot{};
  build_lists(lcs, H, const_cast<ActList *>(u.act), u.ht0, u.hch0);
}

__global__ void k_fill_u32(uint32_t *__restrict__ p, int64_t count, uint32_t value, const LoopCtl *lc,
                           int32_t want) {
  JET_GATE(lc, want);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = value;
}

// Device timing marks of a kernel family: `end` == 0 stores the wall clock, `end` == 1 adds the
// elapsed ticks, one launch and the family's algorithmic bytes (static part plus the part the
// device counters give).  Gated like the family.
__global__ void k_prof_mark(DevProf *dp, const DevStatus *st, const LoopCtl *lc, int32_t want, int32_t fam,
                            int32_t end, double bytes, double per_inc) {
  JET_GATE(lc, want);
  const unsigned long long now = wall_clock64();
  if (!end) {
    if (threadIdx.x == 0) dp->t0[fam] = now;
    return;
  }
  const CtrSlot &c = st->slot[threadIdx.x];  // one lane per slot
  auto total = [&](long long x) { return (double)wave_sum(x); };
  double b = bytes;
  switch (fam) {
  case kProfCandidates: b += per_inc * (total(c.inc_low) + total(c.inc_hub)); break;  // hubs: if beside
  case kProfCandidatesHub: b += per_inc * total(c.inc_hub); break;
  case kProfAfterburner:  // per_inc is nonzero for the graph afterburner only
    if (per_inc > 0.0) b += per_inc * total(c.ab_inc) + 24.0 * total(c.n_cand);
    break;
  case kProfApply: b += 5.0 * st->n_moves + 20.0 * (double)st->mv_inc; break;
  case kProfRbGain: b += 4.0 * total(c.rb_elig) + 32.0 * total(c.rb_ent) + per_inc * total(c.rb_inc); break;
  case kProfRbSelect: b += 32.0 * total(c.rb_ent) + 8.0 * st->n_moves; break;
  default: break;
  }
  if (threadIdx.x != 0) return;
  dp->ticks[fam] += now - dp->t0[fam];
  dp->launches[fam] += 1;
  dp->bytes[fam] += b;
}

inline unsigned grid_for(int64_t work, int block, int64_t cap) {
  int64_t g = (work + block - 1) / block;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (unsigned)g;
}

}  // namespace

int prof_begin(Ctx &c, int fam, const LoopCtl *lc, int32_t want) {
  if (!c.prof || !((c.prof_mask >> fam) & 1u) || !c.dprof) return -1;
  hipLaunchKernelGGL(k_prof_mark, dim3(1), dim3(64), 0, c.stream, c.dprof, c.st, lc, want, fam, 0, 0.0, 0.0);
  return fam;
}

void prof_end(Ctx &c, int token, const LoopCtl *lc, int32_t want, double bytes, double per_inc) {
  if (token < 0) return;
  hipLaunchKernelGGL(k_prof_mark, dim3(1), dim3(64), 0, c.stream, c.dprof, c.st, lc, want, token, 1, bytes, per_inc);
}

hipError_t launch_fill_u32(Ctx &c, uint32_t *p, int64_t count, uint32_t value, const LoopCtl *lc, int32_t want) {
  hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(count, 256, 1024)), dim3(256), 0, c.stream, p, count, value, lc, want);
  return hipGetLastError();
}

// The loop's decision after phase `want` (kPhAny: at the start of a call).
static hipError_t launch_control(Ctx &c, int32_t want) {
  if (c.H > 1)
    hipLaunchKernelGGL(k_control_union, dim3(1), dim3(kCtlThreads), 0, c.stream, c.lcs, c.H, c.lc, c.st, c.k, want,
                       c.mail, union_of(c));
  else
    hipLaunchKernelGGL(k_control, dim3(1), dim3(kCtlOne), 0, c.stream, c.lc, c.st, c.k, c.lmax, want, c.dtrace,
                       c.mail);
  return hipGetLastError();
}

hipError_t launch_loop_init(Ctx &c) {
  hipError_t e = launch_clear_candidate_bits(c);
  return e == hipSuccess ? launch_control(c, kPhAny) : e;
}

hipError_t launch_tick(Ctx &c, int kind) {
  const LoopCtl *lc = c.lc;
  hipError_t e = hipSuccess;
  if (kind == kTickJet) {
    // Jet phase: candidates, afterburner, kept moves (locks), their application
    e = launch_candidates(c, c.cpart, 0, nullptr, 0, lc);
    if (e == hipSuccess) e = launch_afterburner(c, c.cpart, lc);
    if (e == hipSuccess) e = launch_select_moves(c, c.cpart, lc);
    if (e == hipSuccess) e = launch_apply_moves(c, c.cpart, false, lc, kPhJet);
    if (e == hipSuccess) e = launch_control(c, kPhJet);
    if (e != hipSuccess) return e;
  }
  if (kind == kTickRb) {
    for (int r = 0; r < c.rb_slots; ++r) {
      e = launch_rebalance_round(c, c.cpart, 0, nullptr, lc);
      if (e == hipSuccess) e = launch_apply_moves(c, c.cpart, false, lc, kPhRb);
      if (e == hipSuccess) e = launch_control(c, kPhRb);
      if (e != hipSuccess) return e;
    }
  }
  if (kind == kTickRoll) {
    // end of a temperature round: back to its best partition
    e = launch_diff_moves(c, c.cpart, c.best, lc);
    if (e == hipSuccess) e = launch_apply_moves(c, c.cpart, false, lc, kPhRoll);
    if (e == hipSuccess) e = launch_control(c, kPhRoll);
  }
  return e;
}

}  // namespace jet
