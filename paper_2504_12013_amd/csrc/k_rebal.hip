// Deterministic rebalancing round (Section 4.3) on the device.
//
//  prepare : per overloaded block the weight that must leave (bw - Lmax) and its list region (in the
//            loop the control kernel that enters the round does this)
//  gain    : per vertex of an overloaded block that passes the heavy-vertex rule, the best valid
//            target (balanced after adding v, not in the deadzone; adjacency not required; lowest
//            block on ties) and an exact 160-bit order key
//  select  : per overloaded block, radix selection of the minimal prefix (in priority order) whose
//            weight reaches the needed amount -- the same set as sort + prefix sum + binary search
//  apply   : shared with the Jet moves (all selected vertices move at once)
//
// Order key, descending = (priority desc, vertex ID asc), priority gain*c for gain >= 0 and gain/c
// for gain < 0.  Words (most significant first):
//   w0      a 32-bit code that never decreases with the priority (bit length + leading 24 bits of
//           an exact integer image of it), so the first passes split the list well;
//   w1..w3  K + 2^95 where K = gain*c for gain >= 0 and K = -ceil(|gain| 2^62 / c) for gain < 0:
//           distinct rationals with c < 2^31 differ by more than 2^-62, so K orders them exactly;
//   w4      0xffffffff - v.
#include <algorithm>
#include <climits>

#include "chunk.h"
#include "conn.h"
#include "dev_util.h"
#include "entry.h"
#include "hub.h"
#include "jet_internal.h"
#include "moves.h"

namespace jet {

namespace {

// Needs and list regions of one round outside the loop (inside it the control kernel sets them).
__global__ void k_rb_prepare(int32_t k, int64_t lmax, DevStatus *st) {
  __shared__ int64_t cnts[kMaxK];
  const int b = threadIdx.x;
  if (b < kKm1Slots) st->slot[b].rb_inc = st->slot[b].rb_elig = st->slot[b].rb_ent = 0;
  if (b < k) {
    const int64_t over = st->bw[b] - lmax;
    st->rb_need[b] = over > 0 ? over : 0;
    st->rb_count[b] = 0;
    st->rb_kept[b] = 0;
    cnts[b] = over > 0 ? st->bcnt[b] : 0;
  }
  __syncthreads();
  if (b == 0) {
    int64_t run = 0;
    for (int i = 0; i < k; ++i) {
      st->rb_off[i] = run;
      run += cnts[i];
    }
    st->rb_off[k] = run;
    st->n_moves = 0;
    st->n_bigmv = 0;
    st->mv_inc = 0;
    st->rb_nlist = 0;
    st->rb_nhub = 0;
  }
}

// Union contexts (many hypergraphs, segments hg * k + b): the need and list region of every
// segment of a hypergraph in the rebalancing phase, its move count cleared, one workgroup scanning
// the segments in order.
constexpr int kPrepThreads = 1024;
__global__ __launch_bounds__(kPrepThreads) void k_rb_prepare_union(int32_t k, int32_t H, DevStatus *st,
                                                                   const LoopCtl *lc, Union u) {
  JET_GATE(lc, kPhRb);
  __shared__ int64_t sm[kPrepThreads / kWave + 1];
  __shared__ int64_t carry, scarry;
  if (threadIdx.x == 0) carry = scarry = 0;
  if (threadIdx.x < kKm1Slots) {
    CtrSlot &c = st->slot[threadIdx.x];
    c.rb_inc = c.rb_elig = c.rb_ent = 0;
  }
  const int32_t nseg = H * k;
  for (int32_t base = 0; base < nseg; base += kPrepThreads) {  // block-uniform trip count
    const int32_t sg = base + threadIdx.x;
    int64_t cnt = 0;
    if (sg < nseg) {
      const int32_t hg = sg / k;
      const LoopCtl &h = u.lcs[hg];
      int64_t need = 0;
      if (h.phase == kPhRb) {
        const int64_t over = st->bw[sg] - h.lmax;
        need = over > 0 ? over : 0;
        if (sg % k == 0) st->hmoves[hg] = 0;
      }
      st->rb_need[sg] = need;
      st->rb_count[sg] = 0;
      st->rb_kept[sg] = 0;
      cnt = need > 0 ? st->bcnt[sg] : 0;
    }
    int64_t tot;
    const int64_t ex = block_excl_scan<kPrepThreads>(cnt, sm, &tot);
    if (sg < nseg) st->rb_off[sg] = carry + ex;
    // the overloaded segments, in order, for the selection
    int64_t ntot;
    const int64_t nex = block_excl_scan<kPrepThreads>((int64_t)(cnt > 0 ? 1 : 0), sm, &ntot);
    if (cnt > 0) st->rb_seg[scarry + nex] = sg;
    __syncthreads();
    if (threadIdx.x == 0) {
      carry += tot;
      scarry += ntot;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    st->rb_off[nseg] = carry;
    st->rb_nseg = (int32_t)scarry;
    st->n_moves = 0;
    st->n_bigmv = 0;
    st->mv_inc = 0;
    st->rb_nlist = 0;
    st->rb_nhub = 0;
  }
}

// Union: movable non-hub vertices of overloaded segments (heavy-vertex rule with the hypergraph's
// own ceil(W/k)), each with an entry slot in its segment's region (order inside a region does not
// matter: entries are selected by exact keys).  A workgroup takes kListPer tiles of the listed
// hypergraphs at a time (each tile one hypergraph's), counts per (tile, block) in LDS and reserves
// list positions and region slots with one atomic per workgroup and per (tile, overloaded block).
__global__ __launch_bounds__(kUnionTile) void k_rb_list_union(const int32_t *__restrict__ part,
                                                              const int32_t *__restrict__ vw,
                                                              const int64_t *__restrict__ voff, int32_t n, int32_t k,
                                                              DevStatus *st, int32_t *__restrict__ list,
                                                              int32_t *__restrict__ slot,
                                                              uint8_t *__restrict__ mvfrom, const LoopCtl *lctl,
                                                              Union u) {
  JET_GATE(lctl, kPhRb);
  constexpr int T = 8;  // tiles per workgroup step
  __shared__ int64_t s_vb[T], s_lmax[T], s_A[T];
  __shared__ int32_t s_hg[T];
  __shared__ int64_t sbw[T][kMaxK];
  __shared__ int32_t lcnt[T][kMaxK], lbase[T][kMaxK];
  __shared__ int32_t sm[kUnionTile / kWave + 1];
  __shared__ int32_t s_base;
  const int tid = threadIdx.x;
  const ActList &L = u.act[kActRb];
  const int32_t nt = L.tpref[L.cnt];
  for (int32_t t0 = blockIdx.x * T; t0 < nt; t0 += gridDim.x * T) {  // block-uniform trip count
    if (tid < kWave)  // the first wave finds every tile's first vertex and hypergraph
      for (int j = 0; j < T; ++j) {
        int32_t hg = 0;
        const int64_t vb = t0 + j < nt ? act_tile_base(L, u.ht0, t0 + j, &hg) : (int64_t)n;
        if (tid == 0) {
          s_vb[j] = vb;
          s_hg[j] = hg;
          s_lmax[j] = u.lcs[hg].lmax;
          s_A[j] = u.lcs[hg].A;
        }
      }
    __syncthreads();
    for (int x = tid; x < T * k; x += kUnionTile) {
      const int j = x / k, b = x % k;
      sbw[j][b] = s_vb[j] < n ? st->bw[(int64_t)s_hg[j] * k + b] : 0;
      lcnt[j][b] = 0;
    }
    __syncthreads();
    uint32_t mask = 0;
    int32_t cnt = 0, sv[T];
    int32_t loc[T];
#pragma unroll
    for (int j = 0; j < T; ++j) {
      sv[j] = 0;
      loc[j] = 0;
      const int64_t v = s_vb[j] + tid;
      if (s_vb[j] >= n || v >= n) continue;
      mvfrom[v] = 0xff;
      const int32_t s = part[v];
      const int64_t bs = sbw[j][s];
      if (bs <= s_lmax[j] || u.vhg[v] != s_hg[j]) continue;  // not overloaded, or a padding vertex
      const int64_t c = vw ? vw[v] : 1;
      if (2 * c <= 3 * (bs - s_A[j]) && voff[v + 1] - voff[v] <= kHubDegree) {
        mask |= 1u << j;
        ++cnt;
        sv[j] = s;
        loc[j] = atomicAdd(&lcnt[j][s], 1);
      }
    }
    int32_t tot;
    const int32_t rk = block_excl_scan<kUnionTile>(cnt, sm, &tot);
    if (tid == 0) s_base = tot ? atomicAdd(&st->rb_nlist, tot) : 0;
    for (int x = tid; x < T * k; x += kUnionTile) {
      const int j = x / k, b = x % k;
      const int32_t c = lcnt[j][b];
      if (c) {
        const int64_t sg = (int64_t)s_hg[j] * k + b;
        lbase[j][b] = (int32_t)(st->rb_off[sg] + atomicAdd(&st->rb_count[sg], c));
      }
    }
    __syncthreads();
    int32_t out = s_base + rk;
#pragma unroll
    for (int j = 0; j < T; ++j) {
      if ((mask >> j) & 1u) {
        list[out] = (int32_t)(s_vb[j] + tid);
        slot[out] = lbase[j][sv[j]] + loc[j];
        ++out;
      }
    }
    __syncthreads();  // LDS is rewritten by the next step
  }
}

// Rebalancing candidates of the round (Section 4.3): movable non-hub vertices of overloaded blocks
// (eligible under the heavy-vertex rule), listed so that the gain pass touches only them, with
// the entry slot each one owns in its block's region of the entry array.  Each workgroup takes
// kListPer vertices per thread (strided, so the loads coalesce), all loads in flight at once:
// it counts per block, one atomic per block reserves the slots (the block's count of listed
// vertices, after which hub entries are appended), and the threads write their vertices from
// registers.  The order inside a region does not matter: entries are selected by exact keys.
constexpr int kListBlock = 256;
constexpr int kListPer = 8;
__global__ __launch_bounds__(kListBlock) void k_rb_list(const int32_t *__restrict__ part,
                                                        const int32_t *__restrict__ vw,
                                                        const int64_t *__restrict__ voff, int32_t n, int32_t k,
                                                        int64_t lmax, int64_t A, DevStatus *st,
                                                        int32_t *__restrict__ list, int32_t *__restrict__ slot,
                                                        uint8_t *__restrict__ mvfrom,
                                                        const int32_t *__restrict__ hubs, int32_t nhubs,
                                                        int32_t *__restrict__ hlist, int32_t list_blocks,
                                                        const LoopCtl *lctl) {
  JET_GATE(lctl, kPhRb);
  __shared__ int64_t bw[kMaxK];
  __shared__ int32_t lc[kMaxK], lbase[kMaxK];
  __shared__ int32_t sm[kListBlock / kWave + 1];
  __shared__ int32_t s_base;
  const int tid = threadIdx.x;
  for (int b = tid; b < k; b += kListBlock) {
    bw[b] = st->bw[b];
    lc[b] = 0;
  }
  __syncthreads();
  if ((int32_t)blockIdx.x >= list_blocks) {  // hub vertices that may move, by their index in the hub list
    const int32_t h = ((int32_t)blockIdx.x - list_blocks) * kListBlock + tid;
    bool e = false;
    if (h < nhubs) {
      const int32_t v = hubs[h];
      const int64_t hb = bw[part[v]], c = vw ? vw[v] : 1;
      e = hb > lmax && 2 * c <= 3 * (hb - A);
    }
    const uint64_t mm = ballot(e);
    if (!mm) return;  // wave-uniform, no barrier follows
    int32_t base = 0;
    if (lane_id() == 0) base = atomicAdd(&st->rb_nhub, __popcll(mm));
    base = __shfl(base, 0, kWave);
    if (e) hlist[base + rank_below(mm)] = h;
    return;
  }
  const int64_t r0 = (int64_t)blockIdx.x * (kListBlock * kListPer) + tid;
  int32_t pv[kListPer];
#pragma unroll
  for (int j = 0; j < kListPer; ++j) {
    const int64_t v = r0 + j * kListBlock;
    pv[j] = v < n ? part[v] : -1;
    if (v < n) mvfrom[v] = 0xff;
  }
  // vertices of overloaded blocks: weight and degree (loaded only for them)
  bool over[kListPer];
  int64_t bs[kListPer], c[kListPer], d0[kListPer], d1[kListPer];
#pragma unroll
  for (int j = 0; j < kListPer; ++j) {
    bs[j] = pv[j] >= 0 ? bw[pv[j]] : 0;
    over[j] = pv[j] >= 0 && bs[j] > lmax;
  }
#pragma unroll
  for (int j = 0; j < kListPer; ++j) {
    c[j] = 1;
    d0[j] = 0;
    d1[j] = 0;
    if (over[j]) {
      const int64_t v = r0 + j * kListBlock;
      if (vw) c[j] = vw[v];
      d0[j] = voff[v];
      d1[j] = voff[v + 1];
    }
  }
  uint32_t mask = 0;
  int32_t cnt = 0;
#pragma unroll
  for (int j = 0; j < kListPer; ++j) {
    if (over[j] && 2 * c[j] <= 3 * (bs[j] - A) && d1[j] - d0[j] <= kHubDegree) {  // hubs: listed separately
      mask |= 1u << j;
      ++cnt;
      atomicAdd(&lc[pv[j]], 1);
    }
  }
  int32_t tot;
  const int32_t rk = block_excl_scan<kListBlock>(cnt, sm, &tot);
  if (tid == 0) s_base = tot ? atomicAdd(&st->rb_nlist, tot) : 0;
  for (int b = tid; b < k; b += kListBlock) {
    const int32_t x = lc[b];
    lbase[b] = x ? (int32_t)st->rb_off[b] + atomicAdd(&st->rb_count[b], x) : 0;
    lc[b] = 0;
  }
  __syncthreads();
  if (tot == 0) return;
  int32_t out = s_base + rk;
#pragma unroll
  for (int j = 0; j < kListPer; ++j) {
    if ((mask >> j) & 1u) {
      list[out] = (int32_t)(r0 + j * kListBlock);
      slot[out] = lbase[pv[j]] + atomicAdd(&lc[pv[j]], 1);
      ++out;
    }
  }
}

// Adds the thread's counts (scanned incidences, examined vertices, written entries) to the status,
// one atomic per workgroup and counter.  Every thread of the block calls it.
template <int NWV>
__device__ __forceinline__ void flush_rb_counters(unsigned long long a, unsigned long long b, unsigned long long c,
                                                  unsigned long long (*wsum)[3], DevStatus *st) {
  a = wave_sum(a);
  b = wave_sum(b);
  c = wave_sum(c);
  const int w = threadIdx.x / kWave;
  if (lane_id() == 0) {
    wsum[w][0] = a;
    wsum[w][1] = b;
    wsum[w][2] = c;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long t0 = 0ull, t1 = 0ull, t2 = 0ull;
    for (int i = 0; i < NWV; ++i) {
      t0 += wsum[i][0];
      t1 += wsum[i][1];
      t2 += wsum[i][2];
    }
    if (t1) {
      count_add(st, blockIdx.x, &CtrSlot::rb_inc, (long long)t0);
      count_add(st, blockIdx.x, &CtrSlot::rb_elig, (long long)t1);
      count_add(st, blockIdx.x, &CtrSlot::rb_ent, (long long)t2);
    }
  }
}

// With net weights.
template <int G>
__global__ __launch_bounds__(G == 16 ? 512 : 256) void k_rb_gain(
    const int32_t *__restrict__ part, const int64_t *__restrict__ voff, const int32_t *__restrict__ inc,
    const int32_t *__restrict__ nw, const uint64_t *__restrict__ ns, const int32_t *__restrict__ sumw,
    const int32_t *__restrict__ vw, const int32_t *__restrict__ list, const int32_t *__restrict__ slot, int32_t k,
    int64_t lmax, int64_t dz, DevStatus *st, uint32_t *__restrict__ entries, const LoopCtl *lc, Union u,
    int32_t xcd) {
  JET_GATE(lc, kPhRb);
  if (lc && !u.lcs) dz = lc->dz;
  constexpr int BLOCK = (G == 16) ? 512 : 256;
  constexpr int VPB = BLOCK / G;
  __shared__ int64_t bw[kMaxK];
  __shared__ unsigned long long wsum[BLOCK / kWave][3];
  for (int b = threadIdx.x; b < k; b += BLOCK) bw[b] = st->bw[b];
  __syncthreads();
  const int lg = threadIdx.x % G;
  const int64_t nl = st->rb_nlist;  // listed by k_rb_list: every entry is eligible
  const int64_t ntiles = (nl + VPB - 1) / VPB;
  unsigned long long scanned = 0ull, examined = 0ull, emitted = 0ull;
  // with xcd set, the workgroups of one XCD (round robin by workgroup) take one contiguous eighth of
  // the list, whose vertices are neighbours: their nets' words are fetched into one L2
  int64_t t0 = blockIdx.x, tend = ntiles, tstep = gridDim.x;
  if (xcd && !u.lcs && gridDim.x % 8 == 0) {
    const int64_t per = (ntiles + 7) / 8, x = blockIdx.x % 8;
    t0 = x * per + blockIdx.x / 8;
    tend = min(ntiles, (x + 1) * per);
    tstep = gridDim.x / 8;
  }
  for (int64_t tile = t0; tile < tend; tile += tstep) {  // no barriers: each vertex owns its slot
    const int64_t i = tile * VPB + threadIdx.x / G;
    const bool elig = i < nl;
    int64_t v = 0;
    int32_t s = 0, c = 1;
    int64_t q0 = 0, q1 = 0;
    int64_t lm = lmax, dzz = dz, sg0 = 0;  // union: the vertex's hypergraph's limits and segments
    int32_t unw = (lc && !u.lcs) ? lc->rb_unw : 0;
    if (elig) {
      v = list[i];
      s = part[v];
      c = vw ? vw[v] : 1;
      q0 = voff[v];
      q1 = voff[v + 1];
      if (u.lcs) {
        const int32_t hg = u.vhg[v];
        lm = u.lcs[hg].lmax;
        dzz = u.lcs[hg].dz;
        sg0 = (int64_t)hg * k;
        unw = u.lcs[hg].rb_unw;
      }
    }
    int32_t conn[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) conn[j] = 0;
    int32_t benefit = 0;
    if (elig) vertex_conn<G>(inc, q0, q1, G, nw, ns, lg, s, conn, benefit);
    // best valid target by conn (gain = conn - aff), lowest block on ties; -1 = none
    int32_t bestc = -1, bestb = INT32_MAX;
    if (elig) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int32_t b = lg * 8 + j;
        if (b >= k) continue;
        const int64_t bwb = u.lcs ? st->bw[sg0 + b] : bw[b];
        if (b != s && bwb + c <= lm && bwb < dzz && conn[j] > bestc) {
          bestc = conn[j];
          bestb = b;
        }
      }
    }
#pragma unroll
    for (int o = 1; o < G; o <<= 1) {
      const int32_t oc = __shfl_xor(bestc, o, G);
      const int32_t ob = __shfl_xor(bestb, o, G);
      if (oc > bestc || (oc == bestc && ob < bestb)) {
        bestc = oc;
        bestb = ob;
      }
    }
    if (elig && lg == 0) {
      uint32_t *ent = entries + (int64_t)slot[i] * kEntryWords;
      write_entry(ent, bestc >= 0, bestc - (sumw[v] - benefit), c, (int32_t)v, bestb, unw);
      scanned += (unsigned long long)(q1 - q0);
      examined += 1ull;
      emitted += bestc >= 0 ? 1ull : 0ull;
    }
  }
  flush_rb_counters<BLOCK / kWave>(scanned, examined, emitted, wsum, st);
}

// Unit net weights: G lanes per listed vertex (G = 1 on light levels), the block counts conn(v, b)
// bit-sliced as in the candidate pass (conn.h).  The valid targets form a mask (b != s, room for v's
// weight, outside the deadzone); the best is the lowest block of largest count in it (counts of zero
// included, as for the lane-group kernel).  k = 128 took 16 lanes per vertex with six exchanges and 24
// instructions per net on each: 85 us per pass on 300,000 SAT-like vertices against 30 us now.
template <int G, int HW, int N, bool HUBS>
__global__ __launch_bounds__(256) void k_rb_gain_bits(
    const int32_t *__restrict__ part, const int64_t *__restrict__ voff, const int32_t *__restrict__ inc,
    const uint64_t *__restrict__ ns, const int32_t *__restrict__ sumw, const int32_t *__restrict__ vw,
    const int32_t *__restrict__ list, const int32_t *__restrict__ slot, int32_t k, int64_t lmax, int64_t dz,
    DevStatus *st, uint32_t *__restrict__ entries, const LoopCtl *lc, Union u, int32_t xcd, HubArgs hubs,
    int32_t hub_blocks) {
  JET_GATE(lc, kPhRb);
  if (HUBS && (int32_t)blockIdx.x < hub_blocks) {
    hub_work<1, HW, true, true>(hubs, (int32_t)blockIdx.x, hub_blocks);
    return;
  }
  const int32_t bid = (int32_t)blockIdx.x - hub_blocks, nblk = (int32_t)gridDim.x - hub_blocks;
  const bool un = u.lcs != nullptr;
  if (lc && !un) dz = lc->dz;
  const int32_t unw0 = lc && !un ? lc->rb_unw : 0;
  constexpr int VPW = kWave / G;
  __shared__ int64_t slack[32 * HW];
  __shared__ uint32_t s_ok[HW];  // one hypergraph: blocks outside the deadzone
  __shared__ long long s_minslack;
  __shared__ unsigned long long wsum[4][3];
  if (threadIdx.x < HW) s_ok[threadIdx.x] = 0u;
  if (threadIdx.x == 0) s_minslack = LLONG_MAX;
  __syncthreads();
  if (!un)
    for (int b = threadIdx.x; b < k; b += 256) {
      const int64_t bwb = st->bw[b];
      slack[b] = lmax - bwb;
      if (bwb < dz) {
        atomicOr(&s_ok[b >> 5], 1u << (b & 31));
        atomicMin(&s_minslack, (long long)(lmax - bwb));
      }
    }
  __syncthreads();
  const int64_t minslack = s_minslack;
  const int64_t nl = st->rb_nlist;
  const int l = lane_id(), lg = l % G;
  unsigned long long scanned = 0ull, examined = 0ull, emitted = 0ull;
  // with xcd set, the workgroups of one XCD take one contiguous eighth of the list (as k_rb_gain)
  int64_t bstart = ((int64_t)bid * 4 + threadIdx.x / kWave) * VPW, bend = nl;
  int64_t bstep = (int64_t)nblk * 4 * VPW;
  if (xcd && !un && nblk % 8 == 0) {
    const int64_t span = 4 * VPW, steps = (nl + span - 1) / span, per = (steps + 7) / 8, x = bid % 8;
    bstart = (x * per + bid / 8) * span + (threadIdx.x / kWave) * VPW;
    bend = min(nl, (x + 1) * per * span);
    bstep = (int64_t)(nblk / 8) * span;
  }
  for (int64_t base = bstart; base < bend; base += bstep) {  // wave-uniform trip count
    const int64_t i = base + l / G;
    const bool elig = i < nl;
    int32_t v = 0, s = 0, c = 1, unw = unw0;
    int64_t q0 = 0, q1 = 0, lm = lmax, dzz = dz, sg0 = 0;  // union: the vertex's hypergraph's limits and segments
    if (elig) {
      v = list[i];
      s = part[v];
      c = vw ? vw[v] : 1;
      q0 = voff[v];
      q1 = voff[v + 1];
      if (un) {
        const int32_t hg = u.vhg[v];
        lm = u.lcs[hg].lmax;
        dzz = u.lcs[hg].dz;
        sg0 = (int64_t)hg * k;
        unw = u.lcs[hg].rb_unw;
      }
    }
    uint32_t pl[HW][N] = {};
    int32_t benefit = 0;
    if (elig) planes_accumulate<HW, N>(inc, q0 + lg, q1, G, ns, s, pl, benefit);
    // valid targets of a word: room for c (every block outside the deadzone has it when c <= the
    // smallest slack there), outside the deadzone, not s
    int32_t bestb;
    const int32_t bestc = planes_target<G, HW, N>(pl, benefit, l, bestb, [&](int x, const uint32_t (&)[N]) {
      uint32_t ok = 0u;
      if (un) {
#pragma unroll 1
        for (int b0 = 0; b0 < 32 && 32 * x + b0 < k; b0 += 8) {  // eight loads in flight
          int64_t w8[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const int b = 32 * x + b0 + j;
            w8[j] = b < k ? st->bw[sg0 + b] : LLONG_MAX / 2;
          }
#pragma unroll
          for (int j = 0; j < 8; ++j)
            if (w8[j] + c <= lm && w8[j] < dzz) ok |= 1u << (b0 + j);
        }
      } else {
        ok = s_ok[x];
        if ((int64_t)c > minslack) {
          uint32_t room = 0u;
#pragma unroll 1
          for (int b = 0; b < 32 && 32 * x + b < k; ++b)
            if (slack[32 * x + b] >= (int64_t)c) room |= 1u << b;
          ok &= room;
        }
      }
      return ok & ~(x == (s >> 5) ? 1u << (s & 31) : 0u);
    });
    if (!elig || lg != 0) continue;
    write_entry(entries + (int64_t)slot[i] * kEntryWords, bestc >= 0, bestc - (sumw[v] - benefit), c, v, bestb,
                unw);
    scanned += (unsigned long long)(q1 - q0);
    examined += 1ull;
    emitted += bestc >= 0 ? 1ull : 0ull;
  }
  flush_rb_counters<4>(scanned, examined, emitted, wsum, st);
}

constexpr int kSelThreads = 1024;
constexpr int kSelPer = 2;    // list entries in flight per thread of the selection in memory (4: spills)
constexpr int kSplitPer = 4;  // and of the grid-wide first pass

// Writes one selected entry as a move of vertex ent[5] from block `from` to ent[6], and the vertex's
// new block.
__device__ __forceinline__ void put_move(const uint32_t *ent, int32_t from, int32_t pos, int4 *moves,
                                         int32_t *sel_target, int32_t *part, uint8_t *mvfrom) {
  moves[pos] = make_int4((int32_t)ent[5], from, (int32_t)ent[6], (int32_t)ent[7]);
  part[ent[5]] = (int32_t)ent[6];
  mvfrom[ent[5]] = (uint8_t)from;
  if (sel_target) sel_target[ent[5]] = (int32_t)ent[6];
}

// Threshold of one radix pass, computed by the 64 lanes of one wave: the largest digit dg whose
// weight at or above it, sum_{j >= dg} hw[j], reaches the remaining need nr.  Lane l holds the four
// bins of group 63 - l, so an inclusive scan over the lanes gives each group's suffix sum; the
// first lane whose suffix reaches the need owns the threshold.  When the whole weight is at most
// the need (only possible before the first selection), every entry with a weight is emitted:
// thr 0, done.  Otherwise done when the threshold digit's weight is exactly the rest of the need
// or a single entry holds it.  One lane writes the results.
__device__ __forceinline__ void pass_threshold(const unsigned long long *hw, const int32_t *hc, int64_t nr,
                                               int32_t *s_thr, int64_t *s_need, int32_t *s_done) {
  const int lane = lane_id();
  const int g = kWave - 1 - lane;
  int64_t h[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) h[j] = (int64_t)hw[4 * g + j];
  const int64_t sg = h[0] + h[1] + h[2] + h[3];
  const int64_t suf = wave_incl_scan(sg);
  const int64_t total = __shfl(suf, kWave - 1, kWave);
  const uint64_t reach = ballot(suf >= nr);
  if (total <= nr) {
    if (lane == 0) {
      *s_thr = 0;
      *s_done = 1;
    }
  } else if (lane == (int)__builtin_ctzll(reach)) {
    int64_t cum = suf - sg;
    int thr = 4 * g;
#pragma unroll
    for (int j = 3; j >= 0; --j) {
      if (cum + h[j] >= nr) {
        thr = 4 * g + j;
        break;
      }
      cum += h[j];
    }
    const int64_t rem = nr - cum;
    *s_thr = thr;
    *s_need = rem;
    *s_done = ((int64_t)hw[thr] == rem || hc[thr] == 1) ? 1 : 0;
  }
}

// ---- the first pass over all CUs (large levels) ----
// The first pass of the selection over an overloaded block's entries runs on up to S workgroups per
// block (grid S x k, a workgroup has a tile of entries at least; blocks without need exit at once):
// k_rb_sel_hist adds the histogram of the entries' split digit into hist[b]; k_rb_sel_split derives the
// same threshold from it in every workgroup, emits the entries above the threshold digit (and on
// it, when that completes the selection) and compacts the entries on the threshold digit into the
// block's region of keep2.  The single-workgroup selection then continues over the kept entries, which
// still differ anywhere in the key; it clears hist[b] again.
// A block that holds half of 300,000 vertices took 140 us on the two slices that suit an average block, now
// 27 us, and a round's histogram and split 15 us on average (34).
constexpr int kSplitThreads = 256;  // one thread per histogram bin

constexpr int kSplitTile = kSplitThreads * kSplitPer;

// The slice of a list of len entries for workgroup s of S: S only as far as slices hold `least` entries.
__device__ __forceinline__ void slice_range(int32_t len, int s, int S, int32_t least, int32_t &lo, int32_t &hi) {
  S = min(S, (len + least - 1) / least);
  if (s >= S) {
    lo = hi = 0;
    return;
  }
  lo = (int32_t)((int64_t)len * s / S);
  hi = (int32_t)((int64_t)len * (s + 1) / S);
}

// Split digit of an entry's first key word: monotone in it, and finer than its first byte (sign and bit
// length of the priority, the same for nearly all moves) where priorities lie: three bits of mantissa for
// losses per weight from 2^-7 up to 2^8 and for gains times weight below 2^15.
// order 2 (buckets): the byte that holds the bucket.
__device__ __forceinline__ uint32_t split_digit(uint32_t w0, int32_t order) {
  if (order == 2) return w0 >> 24;
  if (w0 >> 31) return 128u + min((w0 & 0x7fffffffu) >> 21, 127u);
  const int32_t e = (int32_t)((0x7fffffffu - w0) >> 21) - 56 * 8;  // bit length 63: a loss of 1 per weight
  return 127u - (uint32_t)min(max(e, 0), 127);
}

__global__ __launch_bounds__(kSplitThreads) void k_rb_sel_hist(const uint32_t *__restrict__ entries,
                                                               const DevStatus *st, unsigned long long *__restrict__ gw,
                                                               uint32_t *__restrict__ gc, int32_t least, const LoopCtl *lc) {
  JET_GATE(lc, kPhRb);
  __shared__ unsigned long long hw[256];
  __shared__ uint32_t hc[256];
  const int b = blockIdx.y, tid = threadIdx.x;
  if (st->rb_need[b] <= 0) return;
  int32_t lo, hi;
  slice_range(st->rb_count[b], blockIdx.x, gridDim.x, least, lo, hi);
  if (lo >= hi) return;
  const uint32_t *list = entries + st->rb_off[b] * kEntryWords;
  const int32_t order = lc ? lc->rb_unw : 0;
  hw[tid] = 0ull;
  hc[tid] = 0u;
  __syncthreads();
  for (int32_t ib = lo + tid; ib < hi; ib += kSplitThreads * 4) {  // four entries' loads in flight
    uint32_t wt[4], k0[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int32_t i = ib + u * kSplitThreads;
      wt[u] = 0u;
      k0[u] = 0u;
      if (i < hi) {
        wt[u] = list[(int64_t)i * kEntryWords + 7];
        k0[u] = list[(int64_t)i * kEntryWords];
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (wt[u] == 0u) continue;  // a vertex without a valid target (or past the slice)
      const uint32_t dg = split_digit(k0[u], order);
      atomicAdd(&hw[dg], (unsigned long long)wt[u]);
      atomicAdd(&hc[dg], 1u);
    }
  }
  __syncthreads();
  if (hc[tid]) {
    atomicAdd(&gw[(int64_t)b * 256 + tid], hw[tid]);
    atomicAdd(&gc[(int64_t)b * 256 + tid], hc[tid]);
  }
}

__global__ __launch_bounds__(kSplitThreads) void k_rb_sel_split(
    const uint32_t *__restrict__ entries, uint32_t *__restrict__ keep2, DevStatus *st,
    const unsigned long long *__restrict__ gw, const uint32_t *__restrict__ gc, int4 *__restrict__ moves,
    int32_t *__restrict__ sel_target, int32_t *__restrict__ part, uint8_t *__restrict__ mvfrom,
    const int64_t *__restrict__ voff, int32_t *__restrict__ bigmv, int32_t least, const LoopCtl *lc) {
  JET_GATE(lc, kPhRb);
  __shared__ unsigned long long hw[256];
  __shared__ int32_t hc[256];
  __shared__ int32_t s_thr, s_done, s_ebase, s_kbase;
  __shared__ int64_t s_need;
  __shared__ int32_t sm[kSplitThreads / kWave + 1];
  __shared__ unsigned long long s_deg;
  const int b = blockIdx.y, tid = threadIdx.x;
  const int64_t need = st->rb_need[b];
  if (need <= 0) return;
  int32_t lo, hi;
  slice_range(st->rb_count[b], blockIdx.x, gridDim.x, least, lo, hi);
  if (lo >= hi) return;
  const uint32_t *list = entries + st->rb_off[b] * kEntryWords;
  uint32_t *kept = keep2 + st->rb_off[b] * kEntryWords;
  hw[tid] = gw[(int64_t)b * 256 + tid];
  hc[tid] = (int32_t)gc[(int64_t)b * 256 + tid];
  if (tid == 0) s_deg = 0ull;
  __syncthreads();
  if (tid < kWave) pass_threshold(hw, hc, need, &s_thr, &s_need, &s_done);
  __syncthreads();
  const uint32_t thr = (uint32_t)s_thr;
  const bool done = s_done != 0;
  const int32_t order = lc ? lc->rb_unw : 0;
  unsigned long long deg = 0ull;
  for (int32_t tb = lo; tb < hi; tb += kSplitThreads * kSplitPer) {  // block-uniform trip count
    uint32_t ent[kSplitPer][kEntryWords];
    uint32_t emit = 0u, keep = 0u;
#pragma unroll
    for (int j = 0; j < kSplitPer; ++j) {
      const int32_t i = tb + j * kSplitThreads + tid;
      if (i < hi) {
        load_entry(list + (int64_t)i * kEntryWords, ent[j]);
        if (ent[j][7] == 0u) continue;  // a vertex without a valid target: dropped
        const uint32_t dg = split_digit(ent[j][0], order);
        if (dg > thr || (dg == thr && done)) emit |= 1u << j;
        else if (dg == thr) keep |= 1u << j;
      }
    }
    int32_t tot;
    const int32_t rk =
        block_excl_scan<kSplitThreads>((int32_t)(__popc(emit) | (__popc(keep) << 16)), sm, &tot);
    const int32_t etot = tot & 0xffff, ktot = tot >> 16;
    if (tid == 0) {
      s_ebase = etot ? atomicAdd(&st->n_moves, etot) : 0;
      s_kbase = ktot ? atomicAdd(&st->rb_kept[b], ktot) : 0;
    }
    __syncthreads();
    int32_t pos = s_ebase + (rk & 0xffff), kp = s_kbase + (rk >> 16);
#pragma unroll
    for (int j = 0; j < kSplitPer; ++j) {
      const bool e = (emit >> j) & 1u;
      int64_t d = 0;
      if (e) {
        d = voff[ent[j][5] + 1] - voff[ent[j][5]];
        put_move(ent[j], b, pos, moves, sel_target, part, mvfrom);
      }
      push_big_move(d > kLaneDegree, pos, st, bigmv);
      pos += e ? 1 : 0;
      deg += (unsigned long long)d;
      if ((keep >> j) & 1u) {
        store_entry(kept + (int64_t)kp * kEntryWords, ent[j]);
        ++kp;
      }
    }
    __syncthreads();  // s_ebase and s_kbase are rewritten by the next tile
  }
  deg = wave_sum(deg);
  if (lane_id() == 0 && deg) atomicAdd(&s_deg, deg);
  __syncthreads();
  if (tid == 0 && s_deg) atomicAdd((unsigned long long *)&st->mv_inc, s_deg);
}

constexpr int kRegPer = 4;    // entries per thread of the selection in registers
constexpr int kFinish = 64;   // entries a wave orders by comparing all pairs

// Threshold of a histogram whose bins hold weight << 16 | count (at most kSelThreads * kRegPer entries,
// so the counts never carry): as pass_threshold, and the number of entries on the threshold digit.
__device__ __forceinline__ void packed_threshold(const unsigned long long *h, int64_t nr, int32_t *s_thr,
                                                 int64_t *s_need, int32_t *s_done, int32_t *s_left) {
  const int lane = lane_id();
  const int g = kWave - 1 - lane;
  int64_t v[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = (int64_t)h[4 * g + j];
  const int64_t sg = v[0] + v[1] + v[2] + v[3];
  const int64_t suf = wave_incl_scan(sg);
  const int64_t total = __shfl(suf, kWave - 1, kWave);
  const uint64_t reach = ballot((suf >> 16) >= nr);
  if ((total >> 16) <= nr) {
    if (lane == 0) {
      *s_thr = 0;
      *s_done = 1;
    }
  } else if (lane == (int)__builtin_ctzll(reach)) {
    int64_t cum = suf - sg, on = 0;
    int thr = 4 * g;
#pragma unroll
    for (int j = 3; j >= 0; --j) {
      on = v[j];
      if (((cum + on) >> 16) >= nr) {
        thr = 4 * g + j;
        break;
      }
      cum += on;
    }
    const int64_t rem = nr - (cum >> 16);
    *s_thr = thr;
    *s_need = rem;
    *s_left = (int32_t)(on & 0xffff);
    *s_done = (on >> 16) == rem || (on & 0xffff) == 1 ? 1 : 0;
  }
}

// The selection of at most kSelThreads * kRegPer entries: every thread keeps its entries in
// registers, an entry above the threshold digit of a pass is marked selected, one below it is
// dropped, and the moves are written once at the end, with one reservation.  Nothing is compacted
// or read again.  A pass takes the highest eight of the bits in which the remaining entries differ
// (their AND and OR over the workgroup); words 1..3 are skipped at once when they share them, and the
// last kFinish entries are ordered by one wave, each lane summing the weight of the keys above its
// own.  What bounds it is the chain of steps, about 1.5 us each: byte by byte through the key it took
// 20 us for 500 entries, now 16.
// Every thread of the block calls it, with the weight to select.
__device__ __forceinline__ void select_registers(const uint32_t *list, int32_t len, int64_t need,
                                                 int32_t b, DevStatus *st, int4 *__restrict__ moves,
                                                 int32_t *__restrict__ sel_target, int32_t *__restrict__ part,
                                                 uint8_t *__restrict__ mvfrom,
                                                 const int64_t *__restrict__ voff, int32_t *__restrict__ bigmv,
                                                 int32_t *hmoves) {
  __shared__ unsigned long long hist[2][256];
  __shared__ uint32_t s_and[5], s_or[5], f_bits[kSelThreads * kRegPer / 32];
  __shared__ int32_t r_thr, r_done, r_left, r_base, r_ref, r_differ, f_n, f_idx[kFinish];
  __shared__ int64_t r_need;
  __shared__ int32_t r_sm[kSelThreads / kWave + 1];
  __shared__ unsigned long long r_deg;
  const int tid = threadIdx.x;
  // the first and last key word and the weight stay in registers; words 1..3 (the exact rational)
  // are read again in the rare rounds that reach them, vertex and target only for selected entries
  uint32_t k0[kRegPer], k4[kRegPer], wt[kRegPer];
  uint32_t alive = 0u, sel = 0u;
#pragma unroll
  for (int j = 0; j < kRegPer; ++j) {
    const int32_t i = j * kSelThreads + tid;
    k0[j] = k4[j] = wt[j] = 0u;
    if (i < len) {
      const uint32_t *p = list + (int64_t)i * kEntryWords;
      k0[j] = p[0];
      k4[j] = p[4];
      wt[j] = p[7];
    }
    if (wt[j] != 0u) alive |= 1u << j;  // a vertex without a valid target: dropped
  }
  if (tid < 256) hist[0][tid] = hist[1][tid] = 0ull;
  if (tid < kSelThreads * kRegPer / 32) f_bits[tid] = 0u;
  if (tid < 5) {
    s_and[tid] = 0xffffffffu;
    s_or[tid] = 0u;
  }
  if (tid == 0) {
    r_need = need;
    r_done = 0;
    r_left = len;
    r_differ = 0;
    f_n = 0;
    r_deg = 0ull;
  }
  __syncthreads();
  int buf = 0;
  bool done = false;
#pragma unroll 1
  for (int x = 0; x < 5 && !done && r_left > kFinish; ++x) {  // block-uniform
    if (x == 1) {  // do the remaining entries share words 1..3?
      if (alive) r_ref = tid + kSelThreads * __builtin_ctz(alive);  // any of them
      __syncthreads();
      const uint32_t *q = list + (int64_t)r_ref * kEntryWords;
      const uint32_t q1 = q[1], q2 = q[2], q3 = q[3];
      bool differ = false;
#pragma unroll
      for (int j = 0; j < kRegPer; ++j) {
        if (!((alive >> j) & 1u)) continue;
        const uint32_t *p = list + (int64_t)(j * kSelThreads + tid) * kEntryWords;
        differ = differ || p[1] != q1 || p[2] != q2 || p[3] != q3;
      }
      if (ballot(differ) && lane_id() == 0) r_differ = 1;
      __syncthreads();
      if (!r_differ) x = 4;
    }
    uint32_t cur[kRegPer];
    uint32_t an = 0xffffffffu, orr = 0u;
#pragma unroll
    for (int j = 0; j < kRegPer; ++j) {
      cur[j] = x == 0 ? k0[j] : k4[j];
      if ((alive >> j) & 1u) {
        if (x >= 1 && x <= 3) cur[j] = list[(int64_t)(j * kSelThreads + tid) * kEntryWords + x];
        an &= cur[j];
        orr |= cur[j];
      }
    }
    if (ballot(alive != 0u)) {
#pragma unroll
      for (int o = kWave / 2; o >= 1; o >>= 1) {
        an &= (uint32_t)__shfl_xor((int)an, o, kWave);
        orr |= (uint32_t)__shfl_xor((int)orr, o, kWave);
      }
      if (lane_id() == 0) {
        atomicAnd(&s_and[x], an);
        atomicOr(&s_or[x], orr);
      }
    }
    __syncthreads();
    uint32_t diff = s_and[x] ^ s_or[x];  // bits in which the remaining entries differ
    while (diff != 0u) {  // block-uniform
      const int sh = max(0, 24 - __clz((int)diff));
#pragma unroll
      for (int j = 0; j < kRegPer; ++j)
        if ((alive >> j) & 1u)
          atomicAdd(&hist[buf][(cur[j] >> sh) & 0xffu], ((unsigned long long)wt[j] << 16) | 1ull);
      if (tid < 256) hist[buf ^ 1][tid] = 0ull;  // the next pass's histogram
      __syncthreads();
      if (tid < kWave) packed_threshold(hist[buf], r_need, &r_thr, &r_need, &r_done, &r_left);
      __syncthreads();
      const uint32_t thr = (uint32_t)r_thr;
      done = r_done != 0;
#pragma unroll
      for (int j = 0; j < kRegPer; ++j) {
        if (!((alive >> j) & 1u)) continue;
        const uint32_t dg = (cur[j] >> sh) & 0xffu;
        if (dg > thr || (dg == thr && done)) sel |= 1u << j;
        if (dg != thr || done) alive &= ~(1u << j);
      }
      buf ^= 1;
      if (done || r_left <= kFinish) break;
      diff &= (1u << sh) - 1u;
    }
  }
  // r_done and r_left stay as they are from here on.  The last entries (distinct keys, so at most one is
  // left otherwise): the first wave orders them
  if (!done) {  // block-uniform
#pragma unroll
    for (int j = 0; j < kRegPer; ++j)
      if ((alive >> j) & 1u) f_idx[atomicAdd(&f_n, 1)] = j * kSelThreads + tid;
    __syncthreads();
    if (tid < kWave) {
      const int n = f_n;
      uint32_t ent[kEntryWords] = {};
      if (tid < n) load_entry(list + (int64_t)f_idx[tid] * kEntryWords, ent);
      const uint64_t hi = ((uint64_t)ent[0] << 32) | ent[1], lo = ((uint64_t)ent[2] << 32) | ent[3];
      int64_t above = 0;  // weight of the entries with larger keys
      for (int i = 0; i < n; ++i) {
        const uint32_t e0 = (uint32_t)__builtin_amdgcn_readlane((int)ent[0], i);
        const uint32_t e1 = (uint32_t)__builtin_amdgcn_readlane((int)ent[1], i);
        const uint32_t e2 = (uint32_t)__builtin_amdgcn_readlane((int)ent[2], i);
        const uint32_t e3 = (uint32_t)__builtin_amdgcn_readlane((int)ent[3], i);
        const uint32_t e4 = (uint32_t)__builtin_amdgcn_readlane((int)ent[4], i);
        const uint32_t ew = (uint32_t)__builtin_amdgcn_readlane((int)ent[7], i);
        const uint64_t ehi = ((uint64_t)e0 << 32) | e1, elo = ((uint64_t)e2 << 32) | e3;
        const bool gt = ehi > hi || (ehi == hi && (elo > lo || (elo == lo && e4 > ent[4])));
        above += gt ? (int64_t)ew : 0;
      }
      if (tid < n && above < r_need) atomicOr(&f_bits[f_idx[tid] >> 5], 1u << (f_idx[tid] & 31));
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kRegPer; ++j) {
      const int32_t i = j * kSelThreads + tid;
      if (((alive >> j) & 1u) && ((f_bits[i >> 5] >> (i & 31)) & 1u)) sel |= 1u << j;
    }
  }
  // vertices and degrees are read before the reservation, beside the scan
  int32_t vtx[kRegPer], deg[kRegPer];
#pragma unroll
  for (int j = 0; j < kRegPer; ++j) {
    vtx[j] = deg[j] = 0;
    if (!((sel >> j) & 1u)) continue;
    vtx[j] = (int32_t)list[(int64_t)(j * kSelThreads + tid) * kEntryWords + 5];
    deg[j] = (int32_t)(voff[vtx[j] + 1] - voff[vtx[j]]);
  }
  int32_t tot;
  const int32_t rk = block_excl_scan<kSelThreads>((int32_t)__popc(sel), r_sm, &tot);
  if (tot == 0) return;  // block-uniform
  if (tid == 0) {
    r_base = atomicAdd(&st->n_moves, tot);
    if (hmoves) atomicAdd(hmoves, tot);
  }
  __syncthreads();
  int32_t pos = r_base + rk;
  int64_t dsum = 0;
#pragma unroll
  for (int j = 0; j < kRegPer; ++j) {
    const bool e = (sel >> j) & 1u;
    if (e) {
      const uint32_t t = list[(int64_t)(j * kSelThreads + tid) * kEntryWords + 6];
      const uint32_t ent[kEntryWords] = {0u, 0u, 0u, 0u, 0u, (uint32_t)vtx[j], t, wt[j]};
      put_move(ent, b, pos, moves, sel_target, part, mvfrom);
    }
    push_big_move(deg[j] > kLaneDegree, pos, st, bigmv);
    pos += e ? 1 : 0;
    dsum += deg[j];
  }
  dsum = wave_sum(dsum);
  if (lane_id() == 0 && dsum) atomicAdd(&r_deg, (unsigned long long)dsum);
  __syncthreads();
  if (tid == 0 && r_deg) atomicAdd((unsigned long long *)&st->mv_inc, r_deg);
}

// The selection of one segment by a workgroup.  Lists of more than kSelThreads * kRegPer entries are
// cut down in memory first: the highest eight of the bits in which the entries differ (AND and OR of all
// key words) make the digit of a pass; it emits the entries above the threshold digit and keeps those on
// it, in the other of the two entry regions.  The counts of the histogram give the moves' reservation, so
// the waves place their entries with LDS counters and meet at no barrier inside a scan.  What bounds it is
// one CU reading the list three times per pass; byte by byte, with barriers per tile of 2,048 entries, it
// took 94 to 168 us on 1M SAT-like vertices, now 30 to 60.  With gw / gc (the histograms of the
// grid-wide first pass) the first pass has already run: the kernel rederives its threshold, clears the
// histogram, and continues over the entries that pass kept in keep2 (nothing is left to do when it
// completed the selection).
__device__ __forceinline__ void select_segment(const int32_t sgm, uint32_t *entries, DevStatus *st,
                                               int4 *__restrict__ moves, int32_t *__restrict__ sel_target,
                                               int32_t *__restrict__ part, uint8_t *__restrict__ mvfrom,
                                               const int64_t *__restrict__ voff,
                                               int32_t *__restrict__ bigmv, unsigned long long *__restrict__ gw,
                                               uint32_t *__restrict__ gc, uint32_t *keep2, int32_t k,
                                               const Union &u) {
  __shared__ unsigned long long hw[256];
  __shared__ int32_t hc[256];
  __shared__ uint32_t s_and[5], s_or[5];
  __shared__ int32_t s_thr, s_done, s_emit, s_keep;
  __shared__ int64_t s_need;
  __shared__ unsigned long long s_deg;
  const int32_t b = sgm % k;        // the block the selected vertices leave
  const int tid = threadIdx.x;
  const int64_t need = st->rb_need[sgm];
  if (need <= 0) return;
  int32_t *hmoves = u.lcs ? &st->hmoves[sgm / k] : nullptr;  // union: per hypergraph
  const int64_t at = st->rb_off[sgm] * kEntryWords;
  const uint32_t *list = entries + at;
  uint32_t *other = keep2 + at;
  int32_t len = st->rb_count[sgm];
  if (tid == 0) {
    s_need = need;
    s_deg = 0ull;
  }
  if (gw) {  // the first pass ran over all CUs: continue over the kept entries
    for (int i = tid; i < 256; i += kSelThreads) {
      hw[i] = gw[(int64_t)b * 256 + i];
      hc[i] = (int32_t)gc[(int64_t)b * 256 + i];
      gw[(int64_t)b * 256 + i] = 0ull;
      gc[(int64_t)b * 256 + i] = 0u;
    }
    __syncthreads();
    if (tid < kWave) pass_threshold(hw, hc, need, &s_thr, &s_need, &s_done);
    __syncthreads();
    if (s_done) return;  // the split pass emitted the whole selection
    list = keep2 + at;
    other = entries + at;
    len = st->rb_kept[sgm];
  }
  __syncthreads();
  while (len > kSelThreads * kRegPer) {  // block-uniform
    if (tid < 5) {
      s_and[tid] = 0xffffffffu;
      s_or[tid] = 0u;
    }
    if (tid < 256) {
      hw[tid] = 0ull;
      hc[tid] = 0;
    }
    if (tid == 0) s_emit = s_keep = 0;
    uint32_t an[5], orr[5];
#pragma unroll
    for (int x = 0; x < 5; ++x) {
      an[x] = 0xffffffffu;
      orr[x] = 0u;
    }
    for (int32_t i0 = tid; i0 < len; i0 += kSelThreads * kSelPer) {
#pragma unroll
      for (int j = 0; j < kSelPer; ++j) {
        const int32_t i = i0 + j * kSelThreads;
        uint32_t ent[kEntryWords] = {};
        if (i < len) load_entry(list + (int64_t)i * kEntryWords, ent);
        const bool valid = ent[7] != 0u;  // else a vertex without a valid target
#pragma unroll
        for (int x = 0; x < 5; ++x) {
          an[x] &= valid ? ent[x] : 0xffffffffu;
          orr[x] |= valid ? ent[x] : 0u;
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int x = 0; x < 5; ++x) {
#pragma unroll
      for (int o = kWave / 2; o >= 1; o >>= 1) {
        an[x] &= (uint32_t)__shfl_xor((int)an[x], o, kWave);
        orr[x] |= (uint32_t)__shfl_xor((int)orr[x], o, kWave);
      }
      if (lane_id() == 0) {
        atomicAnd(&s_and[x], an[x]);
        atomicOr(&s_or[x], orr[x]);
      }
    }
    __syncthreads();
    int x = 0;
    while (x < 4 && (s_and[x] & s_or[x]) == s_or[x]) ++x;  // the first word in which entries differ
    const uint32_t diff = s_or[x] & ~s_and[x];
    const int sh = diff ? max(0, 24 - __clz((int)diff)) : 0;  // one valid entry or none: any digit will do
    for (int32_t i0 = tid; i0 < len; i0 += kSelThreads * 4) {  // four entries' loads in flight
      uint32_t wt[4], key[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int32_t i = i0 + j * kSelThreads;
        wt[j] = key[j] = 0u;
        if (i < len) {
          wt[j] = list[(int64_t)i * kEntryWords + 7];
          key[j] = list[(int64_t)i * kEntryWords + x];
        }
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (wt[j] == 0u) continue;
        atomicAdd(&hw[(key[j] >> sh) & 0xffu], (unsigned long long)wt[j]);
        atomicAdd(&hc[(key[j] >> sh) & 0xffu], 1);
      }
    }
    __syncthreads();
    if (tid < kWave) pass_threshold(hw, hc, s_need, &s_thr, &s_need, &s_done);
    __syncthreads();
    const int thr = s_thr;
    const bool done = s_done != 0;
    if (tid < 256 && hc[tid] && (tid > thr || (tid == thr && done))) atomicAdd(&s_emit, hc[tid]);
    __syncthreads();
    if (tid == 0 && s_emit) {  // from here on the next position of the move list
      const int32_t n = s_emit;
      s_emit = atomicAdd(&st->n_moves, n);
      if (hmoves) atomicAdd(hmoves, n);
    }
    __syncthreads();
    int64_t dsum = 0;
    for (int32_t i0 = tid - lane_id(); i0 < len; i0 += kSelThreads * kSelPer) {  // wave-uniform
      uint32_t ent[kSelPer][kEntryWords];
#pragma unroll
      for (int j = 0; j < kSelPer; ++j) {
        const int32_t i = i0 + j * kSelThreads + lane_id();
        ent[j][7] = 0u;
        if (i < len) load_entry(list + (int64_t)i * kEntryWords, ent[j]);
      }
#pragma unroll
      for (int j = 0; j < kSelPer; ++j) {
        uint32_t key = ent[j][0];
#pragma unroll
        for (int y = 1; y < 5; ++y) key = x == y ? ent[j][y] : key;
        const int dg = (int)((key >> sh) & 0xffu);
        const bool valid = ent[j][7] != 0u;
        const bool e = valid && (dg > thr || (dg == thr && done)), kp = valid && dg == thr && !done;
        const uint64_t me = ballot(e), mk = ballot(kp);
        int32_t eb = 0, kb = 0;
        if (lane_id() == 0) {
          eb = me ? atomicAdd(&s_emit, __popcll(me)) : 0;
          kb = mk ? atomicAdd(&s_keep, __popcll(mk)) : 0;
        }
        const int32_t pos = __shfl(eb, 0, kWave) + rank_below(me), kpos = __shfl(kb, 0, kWave) + rank_below(mk);
        int64_t d = 0;
        if (e) {
          d = voff[ent[j][5] + 1] - voff[ent[j][5]];
          put_move(ent[j], b, pos, moves, sel_target, part, mvfrom);
        }
        push_big_move(d > kLaneDegree, pos, st, bigmv);
        dsum += d;
        if (kp) store_entry(other + (int64_t)kpos * kEntryWords, ent[j]);
      }
    }
    dsum = wave_sum(dsum);
    if (lane_id() == 0 && dsum) atomicAdd(&s_deg, (unsigned long long)dsum);
    __syncthreads();  // the kept entries are written, also for the other waves of the workgroup
    len = done ? 0 : s_keep;
    uint32_t *t = const_cast<uint32_t *>(list);
    list = other;
    other = t;
    __syncthreads();  // every thread has read the counters
  }
  if (tid == 0 && s_deg) atomicAdd((unsigned long long *)&st->mv_inc, s_deg);
  if (len > 0) select_registers(list, len, s_need, b, st, moves, sel_target, part, mvfrom, voff, bigmv, hmoves);
}

// One workgroup per overloaded block: the block's segment (one hypergraph).  A union's workgroups
// walk the segments of the hypergraphs in their rebalancing phase.
__global__ __launch_bounds__(kSelThreads) void k_rb_select(uint32_t *entries, DevStatus *st,
                                                           int4 *__restrict__ moves, int32_t *__restrict__ sel_target,
                                                           int32_t *__restrict__ part,
                                                           uint8_t *__restrict__ mvfrom,
                                                           const int64_t *__restrict__ voff,
                                                           int32_t *__restrict__ bigmv,
                                                           unsigned long long *__restrict__ gw,
                                                           uint32_t *__restrict__ gc, uint32_t *keep2,
                                                           const LoopCtl *lc, int32_t k, Union u) {
  JET_GATE(lc, kPhRb);
  const int32_t nseg = u.lcs ? st->rb_nseg : k;  // union: the overloaded segments the preparation listed
  for (int32_t x = blockIdx.x; x < nseg; x += gridDim.x) {  // block-uniform trip count
    select_segment(u.lcs ? st->rb_seg[x] : x, entries, st, moves, sel_target, part, mvfrom, voff, bigmv, gw, gc,
                   keep2, k, u);
    __syncthreads();  // shared state is reused by the next segment
  }
}

inline unsigned grid_for(int64_t work, int block, int64_t cap) {
  int64_t g = (work + block - 1) / block;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (unsigned)g;
}

template <int G>
hipError_t gain_launch(Ctx &c, const int32_t *part, int64_t dz, const LoopCtl *lc) {
  constexpr int BLOCK = (G == 16) ? 512 : 256;
  constexpr int VPB = BLOCK / G;
  const Union u = union_of(c);
  if (c.H > 1)
    hipLaunchKernelGGL(k_rb_list_union, dim3(grid_for(c.n, 8 * kUnionTile, c.grid_cap)), dim3(kUnionTile), 0, c.stream, part, c.vw, c.voff,
                       c.n, c.k, c.st, c.rb_list, c.rb_slot, c.mvfrom, lc, u);
  else {
    // the first workgroups take the vertices, the others the hubs
    const int32_t lb = (int32_t)(((int64_t)c.n + kListBlock * kListPer - 1) / (kListBlock * kListPer));
    hipLaunchKernelGGL(k_rb_list, dim3((unsigned)(lb + (c.nhubs + kListBlock - 1) / kListBlock)), dim3(kListBlock), 0,
                       c.stream, part, c.vw, c.voff, c.n, c.k, c.lmax, c.A, c.st, c.rb_list, c.rb_slot, c.mvfrom,
                       c.hubs, c.nhubs, c.rb_hlist, lb, lc);
  }
  // the list length is known on the device only: a persistent grid walks it; unit net weights take the
  // bit-sliced kernel (one lane per vertex on light levels, eight otherwise)
  if (c.unit_nw) {
    const bool few = c.max_low_degree < 32;
    const int hw = c.k <= 32 ? 1 : c.k <= 64 ? 2 : 4;
    const bool hubs = hubs_beside_gains(c);
    HubArgs ha{};
    if (hubs) {
      ha = hub_args(c, part, lc);
      ha.dz = dz;
    }
    const int32_t hb = hubs ? hub_blocks(c) : 0;
    auto go = [&](auto tag, int64_t per) {
      constexpr auto K = decltype(tag)::value;
      const int64_t g = std::max<int64_t>(
          1, std::min<int64_t>({((int64_t)c.n + per - 1) / per, c.grid_cap, resident_grid<K>(256)}));
      hipLaunchKernelGGL(K, dim3((unsigned)(hb + g)), dim3(256), 0, c.stream, part, c.voff, c.inc, c.ns, c.sumw, c.vw,
                         c.rb_list, c.rb_slot, c.k, c.lmax, dz, c.st, c.rb_keys, lc, u, c.rb_xcd, ha, hb);
    };
#define JET_GAIN(GG, HW, N)                                                                     \
  (hubs ? go(KernelTag<k_rb_gain_bits<GG, HW, N, true>>{}, 256 / GG)                            \
        : go(KernelTag<k_rb_gain_bits<GG, HW, N, false>>{}, 256 / GG))
    if (light_lanes(c)) {
      if (hw == 1) few ? JET_GAIN(1, 1, 5) : JET_GAIN(1, 1, 9);
      else if (hw == 2) few ? JET_GAIN(1, 2, 5) : JET_GAIN(1, 2, 9);
      else few ? JET_GAIN(1, 4, 5) : JET_GAIN(1, 4, 9);
    } else {
      if (hw == 1) few ? JET_GAIN(8, 1, 5) : JET_GAIN(8, 1, 9);
      else if (hw == 2) few ? JET_GAIN(8, 2, 5) : JET_GAIN(8, 2, 9);
      else few ? JET_GAIN(8, 4, 5) : JET_GAIN(8, 4, 9);
    }
#undef JET_GAIN
  } else {
    const unsigned grid = (unsigned)std::min<int64_t>(c.grid_cap, (c.n + VPB - 1) / VPB);
    hipLaunchKernelGGL((k_rb_gain<G>), dim3(grid), dim3(BLOCK), 0, c.stream, part, c.voff, c.inc, c.nw, c.ns,
                       c.sumw, c.vw, c.rb_list, c.rb_slot, c.k, c.lmax, dz, c.st, c.rb_keys, lc, u, c.rb_xcd);
  }
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? launch_rb_hubs(c, part, dz, lc) : e;
}

hipError_t gain_dispatch(Ctx &c, const int32_t *part, int64_t dz, const LoopCtl *lc) {
  if (c.k <= 8) return gain_launch<1>(c, part, dz, lc);
  if (c.k <= 16) return gain_launch<2>(c, part, dz, lc);
  if (c.k <= 32) return gain_launch<4>(c, part, dz, lc);
  if (c.k <= 64) return gain_launch<8>(c, part, dz, lc);
  return gain_launch<16>(c, part, dz, lc);
}

}  // namespace

hipError_t launch_rebalance_round(Ctx &c, int32_t *part, int64_t dz, int32_t *sel_target,
                                  const LoopCtl *lc) {
  const int32_t want = lc ? (int32_t)kPhRb : (int32_t)kPhAny;
  if (c.H > 1)
    hipLaunchKernelGGL(k_rb_prepare_union, dim3(1), dim3(kPrepThreads), 0, c.stream, c.k, c.H, c.st, lc,
                       union_of(c));
  else if (!lc)
    hipLaunchKernelGGL(k_rb_prepare, dim3(1), dim3(kMaxK), 0, c.stream, c.k, c.lmax, c.st);
  hipError_t e = hipGetLastError();
  // the preparation (in the loop: the control kernel) cleared the move list and the counters
  if (e != hipSuccess) return e;
  int tok = prof_begin(c, kProfRbGain, lc, want);
  e = gain_dispatch(c, part, dz, lc);
  // 12 B per vertex, plus on the device: examined vertices, written entries, scanned incidences
  prof_end(c, tok, lc, want, 12.0 * c.n, 8.0 + (c.k + 7) / 8 + (c.unit_nw ? 0.0 : 4.0));
  if (e != hipSuccess) return e;
  tok = prof_begin(c, kProfRbSelect, lc, want);
  const bool split = c.H == 1 && c.n >= c.sel_split_min;
  if (split) {
    // as many slices as some 2,048 workgroups allow (or the set count, 1..64): one block may list most
    // of the vertices, and a workgroup without a full tile exits at once
    const unsigned S = c.sel_slices > 0 ? (unsigned)c.sel_slices
                                        : (unsigned)std::max<int64_t>(1, std::min<int64_t>(64, 2048 / c.k));
    const int32_t least = c.sel_slices > 0 ? 1 : kSplitTile;
    hipLaunchKernelGGL(k_rb_sel_hist, dim3(S, (unsigned)c.k), dim3(kSplitThreads), 0, c.stream, c.rb_keys, c.st,
                       c.rb_gw, c.rb_gc, least, lc);
    hipLaunchKernelGGL(k_rb_sel_split, dim3(S, (unsigned)c.k), dim3(kSplitThreads), 0, c.stream, c.rb_keys,
                       c.rb_keys2, c.st, c.rb_gw, c.rb_gc, c.moves, sel_target, part, c.mvfrom, c.voff, c.bigmv, least,
                       lc);
  }
  hipLaunchKernelGGL(k_rb_select, dim3(c.H > 1 ? (unsigned)std::min<int64_t>(512, (int64_t)c.H * c.k) : (unsigned)c.k),
                     dim3(kSelThreads), 0, c.stream, c.rb_keys, c.st,
                     c.moves, sel_target, part, c.mvfrom, c.voff, c.bigmv, split ? c.rb_gw : nullptr,
                     split ? c.rb_gc : nullptr, c.rb_keys2, lc, c.k, union_of(c));
  prof_end(c, tok, lc, want, 0.0, 0.0);  // bytes from the entry and move counts (device)
  return hipGetLastError();
}

}  // namespace jet
