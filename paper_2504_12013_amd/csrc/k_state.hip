// Partition state from scratch (start of every call): pin counts phi_e[b] = |e intersect V_b| and
// the connectivity set Lambda(e) (Section 2; tracked per net as in Section 4.2), block weights
// c(V_b), and the (lambda - 1) metric.  All sums are integer and commutative, so the result does
// not depend on scheduling.
#include <stddef.h>

#include "chunk.h"
#include "dev_util.h"
#include "jet_internal.h"
#include "phi.h"

namespace jet {

namespace {

// Block of v; out of range is reported and counts as block 0.
__device__ __forceinline__ int32_t checked_block(const int32_t *__restrict__ part, int64_t v, int32_t k,
                                                 DevStatus *st) {
  const int32_t b = part[v];
  if ((uint32_t)b < (uint32_t)k) return b;
  if (atomicCAS(&st->err, 0, kErrPartRange) == 0) st->err_arg = (int32_t)v;
  return 0;
}

__global__ void k_check_part(const int32_t *__restrict__ part, int32_t n, int32_t k, DevStatus *st) {
  for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x)
    (void)checked_block(part, v, k, st);
}

// A block read before the check of the partition has been looked at: out of range counts as block 0.
__device__ __forceinline__ int32_t safe_block(int32_t b, int32_t k) { return (uint32_t)b < (uint32_t)k ? b : 0; }

// Four byte counters as four counts.
__device__ __forceinline__ void store_counts(uint16_t *p, uint32_t c) {
  *reinterpret_cast<uint2 *>(p) =
      make_uint2((c & 0xffu) | ((c & 0xff00u) << 8), ((c >> 16) & 0xffu) | ((c >> 8) & 0xff0000u));
}
__device__ __forceinline__ void store_counts(int32_t *p, uint32_t c) {
  *reinterpret_cast<int4 *>(p) =
      make_int4((int)(c & 0xffu), (int)((c >> 8) & 0xffu), (int)((c >> 16) & 0xffu), (int)(c >> 24));
}

// Small nets, one wave per chunk, one pin per lane: byte counters of (net of the chunk, block) in LDS, from
// which the wave writes the nets' rows of counts (consecutive nets: one run of memory, four counts per
// lane where rows allow it) and, with ns, their connectivity words.  Bound by writing m x k counts once;
// clearing the table, an atomic per pin and reading it back for the words took 2.75 ms on the 12.6M
// edges of a mesh at k = 64, now 0.46 ms.
template <int NW, typename T>
__global__ __launch_bounds__(256) void k_state_chunks(const int32_t *__restrict__ pins, const int4 *__restrict__ chunks,
                                                      const uint8_t *__restrict__ pnet, int32_t nchunks,
                                                      const int32_t *__restrict__ part, int32_t k, T *__restrict__ phi,
                                                      uint64_t *__restrict__ ns, int32_t vec) {
  __shared__ uint32_t cnt[4][kChunkNets][16 * NW];
  __shared__ unsigned long long some[4][kChunkNets][NW], one[4][kChunkNets][NW];
  const int w = threadIdx.x / kWave, l = lane_id();
  uint32_t(*C)[16 * NW] = cnt[w];
  for (int x = l; x < kChunkNets * 16 * NW; x += kWave) (&C[0][0])[x] = 0u;
  const int32_t nwv = gridDim.x * 4, per = vec ? k / 4 : k;  // stores per net
  const uint32_t inv = (1u << 20) / (uint32_t)per + 1u;  // x / per == (x * inv) >> 20 for x < 4,096, per <= 128
  auto fetch = [&](int32_t c, int4 &d, int32_t &p, int32_t &j) {
    d = c < nchunks ? chunks[c] : make_int4(0, 0, 0, 0);
    p = j = 0;
    if (l < d.z) {
      j = pnet[(int64_t)d.w + l];
      p = pins[(int64_t)d.w + l];
    }
  };
  int4 cd;
  int32_t pin, j;
  fetch(blockIdx.x * 4 + w, cd, pin, j);
  for (int32_t c = blockIdx.x * 4 + w; c < nchunks; c += nwv) {  // wave-uniform
    const bool act = l < cd.z;
    const int32_t b = act ? safe_block(part[pin], k) : 0;
    int4 ncd;
    int32_t npin, nj;
    fetch(c + nwv, ncd, npin, nj);  // the next chunk's loads overlap this chunk's work
    if (l < kChunkNets) {
#pragma unroll
      for (int x = 0; x < NW; ++x) some[w][l][x] = one[w][l][x] = 0ull;
    }
    if (act) atomicAdd(&C[j][b >> 2], 1u << (8 * (b & 3)));
    wave_lds_sync();
    if (act && ns) {
      const uint32_t mine = (C[j][b >> 2] >> (8 * (b & 3))) & 0xffu;
      atomicOr(&some[w][j][b >> 6], 1ull << (b & 63));
      if (mine == 1u) atomicOr(&one[w][j][b >> 6], 1ull << (b & 63));
    }
    T *row = phi + (int64_t)cd.x * k;
    const int32_t total = cd.y * per;
    for (int32_t i = l; i < total; i += kWave) {
      const int32_t e = (int32_t)(((uint32_t)i * inv) >> 20), x = i - e * per;
      if (vec) store_counts(row + 4 * (int64_t)i, C[e][x]);
      else row[i] = (T)((C[e][x >> 2] >> (8 * (x & 3))) & 0xffu);
    }
    wave_lds_sync();
    if (ns && l < cd.y) {
      uint64_t *nse = ns + (int64_t)(cd.x + l) * (2 * NW);
#pragma unroll
      for (int x = 0; x < NW; ++x) {
        nse[x] = some[w][l][x];
        nse[NW + x] = one[w][l][x];
      }
    }
    if (act) C[j][b >> 2] = 0u;  // every nonzero counter word has a pin here
    wave_lds_sync();
    cd = ncd;
    pin = npin;
    j = nj;
  }
}

// Larger nets: one block per net (the big ones first), histogram in LDS, then the block writes the row it
// owns and the words.
template <int NW, typename T>
__global__ __launch_bounds__(256) void k_state_large(const int64_t *__restrict__ off, const int32_t *__restrict__ pins,
                                                     const int32_t *__restrict__ big, int32_t nbig,
                                                     const int32_t *__restrict__ mid, const int32_t *__restrict__ part,
                                                     int32_t k, T *__restrict__ phi, uint64_t *__restrict__ ns) {
  __shared__ int32_t hist[kMaxK];
  const int32_t e = (int32_t)blockIdx.x < nbig ? big[blockIdx.x] : mid[blockIdx.x - nbig];
  const int64_t q0 = off[e], q1 = off[e + 1];
  for (int b = threadIdx.x; b < k; b += blockDim.x) hist[b] = 0;
  __syncthreads();
  for (int64_t qb = q0 + threadIdx.x; qb < q1; qb += 4 * blockDim.x) {  // four pins' loads in flight
    int32_t v[4], b[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = qb + u * blockDim.x < q1 ? pins[qb + u * blockDim.x] : -1;
#pragma unroll
    for (int u = 0; u < 4; ++u) b[u] = v[u] >= 0 ? safe_block(part[v[u]], k) : -1;
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (b[u] >= 0) atomicAdd(&hist[b[u]], 1);
  }
  __syncthreads();
  const int b = threadIdx.x, x = threadIdx.x / kWave;
  const int32_t h = b < k ? hist[b] : 0;
  if (b < k) phi[(int64_t)e * k + b] = (T)h;
  if (!ns || x >= NW) return;
  const uint64_t some = ballot(h > 0), one = ballot(h == 1);
  if (lane_id() == 0) {
    ns[(int64_t)e * (2 * NW) + x] = some;
    ns[(int64_t)e * (2 * NW) + NW + x] = one;
  }
}

// Block weights and sizes, and the check of the partition (every vertex is read here).
__global__ __launch_bounds__(256) void k_block_weights(const int32_t *__restrict__ part,
                                                       const int32_t *__restrict__ vw, int32_t n, int32_t k,
                                                       DevStatus *st, Union u) {
  __shared__ unsigned long long sw[kMaxK];
  __shared__ int32_t sc[kMaxK];
  for (int b = threadIdx.x; b < k; b += blockDim.x) {
    sw[b] = 0;
    sc[b] = 0;
  }
  __syncthreads();
  if (u.vhg) {
    // union: a workgroup takes a contiguous range of tiles (every tile holds one hypergraph's
    // vertices) and adds its sums to the segments where the range crosses into the next hypergraph
    // (an atomic per vertex on the few segments took 540 us for 96 hypergraphs)
    const int64_t nt = (n + kUnionTile - 1) / kUnionTile, per = (nt + gridDim.x - 1) / gridDim.x;
    const int64_t t0 = (int64_t)blockIdx.x * per, t1 = min(nt, t0 + per);
    for (int64_t t = t0; t < t1; ++t) {  // block-uniform trip count
      const int64_t v = t * kUnionTile + threadIdx.x;
      const int32_t hg = u.vhg[t * kUnionTile];
      const bool mine = v < n && u.vhg[v] == hg;
      if (mine) {
        const int32_t b = checked_block(part, v, k, st);
        atomicAdd(&sw[b], (unsigned long long)(vw ? vw[v] : 1));
        atomicAdd(&sc[b], 1);
      } else if (v < n) {  // padding: the pseudo-hypergraph's segments
        const int64_t sg = (int64_t)u.vhg[v] * k + checked_block(part, v, k, st);
        atomicAdd((unsigned long long *)&st->bw[sg], (unsigned long long)(vw ? vw[v] : 1));
        atomicAdd(&st->bcnt[sg], 1);
      }
      if (t + 1 < t1 && u.vhg[(t + 1) * kUnionTile] == hg) continue;
      __syncthreads();
      for (int b = threadIdx.x; b < k; b += blockDim.x) {
        const int64_t sg = (int64_t)hg * k + b;
        if (sw[b]) atomicAdd((unsigned long long *)&st->bw[sg], sw[b]);
        if (sc[b]) atomicAdd(&st->bcnt[sg], sc[b]);
        sw[b] = 0;
        sc[b] = 0;
      }
      __syncthreads();
    }
    return;
  }
  for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
    const int32_t b = checked_block(part, v, k, st);
    atomicAdd(&sw[b], (unsigned long long)(vw ? vw[v] : 1));
    atomicAdd(&sc[b], 1);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < k; b += blockDim.x) {
    if (sw[b]) atomicAdd((unsigned long long *)&st->bw[b], sw[b]);
    if (sc[b]) atomicAdd(&st->bcnt[b], sc[b]);
  }
}

template <int NW>
__global__ __launch_bounds__(256) void k_km1(const uint64_t *__restrict__ ns, const int32_t *__restrict__ nw,
                                             int32_t m, DevStatus *st, Union u) {
  int64_t s = 0;
  if (u.nhg) {
    // union: a wave takes a contiguous range of nets (nets are numbered by hypergraph) and adds its
    // sum where the range crosses into the next hypergraph; a step of 64 nets that spans two adds
    // per net (an atomic per net on the few addresses took 2.1 ms for 96 hypergraphs)
    const int64_t nwv = (int64_t)gridDim.x * (blockDim.x / kWave);
    const int64_t per = ((m + nwv - 1) / nwv + kWave - 1) / kWave * kWave;
    const int64_t e0 = ((int64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave) * per;
    const int64_t e1 = min((int64_t)m, e0 + per);
    int32_t hg = -1;
    for (int64_t eb = e0; eb < e1; eb += kWave) {  // wave-uniform trip count
      const int64_t e = eb + lane_id();
      const int32_t h0 = u.nhg[eb], h1 = u.nhg[min(e1, eb + kWave) - 1];
      int64_t d = 0;
      if (e < e1) {
        int lam = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) lam += __popcll(ns[e * 2 * NW + w]);
        d = (int64_t)(lam - 1) * (nw ? nw[e] : 1);
      }
      if (h0 != hg || h0 != h1) {
        s = wave_sum(s);
        if (lane_id() == 0 && hg >= 0) add_km1_hg(st, hg, s);
        s = 0;
        hg = h0;
      }
      if (h0 == h1) s += d;
      else if (e < e1) add_km1_hg(st, u.nhg[e], d);
    }
    s = wave_sum(s);
    if (lane_id() == 0 && hg >= 0) add_km1_hg(st, hg, s);
    return;
  }
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m; e += (int64_t)gridDim.x * blockDim.x) {
    int lam = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) lam += __popcll(ns[e * 2 * NW + w]);
    s += (int64_t)(lam - 1) * (nw ? nw[e] : 1);
  }
  s = wave_sum(s);
  if (lane_id() == 0) add_km1(st, blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave, s);
}

// Level statistics for the learned temperature: over nets, the number and weight of cut nets
// (lambda >= 2), the net weight total and the largest net; over vertices, those with an incident
// cut net.  Integer sums, one atomic per block and counter.
template <int NW>
__global__ __launch_bounds__(256) void k_stats_nets(const int64_t *__restrict__ off, const uint64_t *__restrict__ ns,
                                                    const int32_t *__restrict__ nw, int32_t m,
                                                    int64_t *__restrict__ out) {
  int64_t cut = 0, cutw = 0, sw = 0, mx = 0;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m; e += (int64_t)gridDim.x * blockDim.x) {
    int lam = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) lam += __popcll(ns[e * 2 * NW + w]);
    const int64_t w = nw ? nw[e] : 1;
    sw += w;
    if (lam >= 2) {
      cut += 1;
      cutw += w;
    }
    const int64_t sz = off[e + 1] - off[e];
    mx = sz > mx ? sz : mx;
  }
  cut = wave_sum(cut);
  cutw = wave_sum(cutw);
  sw = wave_sum(sw);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const int64_t y = __shfl_xor(mx, o, kWave);
    mx = y > mx ? y : mx;
  }
  if (lane_id() == 0) {
    if (cut) atomicAdd((unsigned long long *)&out[0], (unsigned long long)cut);
    if (cutw) atomicAdd((unsigned long long *)&out[1], (unsigned long long)cutw);
    if (sw) atomicAdd((unsigned long long *)&out[2], (unsigned long long)sw);
    atomicMax((unsigned long long *)&out[3], (unsigned long long)mx);
  }
}

template <int NW>
__global__ __launch_bounds__(256) void k_stats_boundary(const int64_t *__restrict__ voff, const int32_t *__restrict__ inc,
                                                        const uint64_t *__restrict__ ns, int32_t n,
                                                        int64_t *__restrict__ out) {
  int64_t cnt = 0;
  for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
    for (int64_t q = voff[v]; q < voff[v + 1]; ++q) {
      const int64_t e = inc[q];
      int lam = 0;
#pragma unroll
      for (int w = 0; w < NW; ++w) lam += __popcll(ns[e * 2 * NW + w]);
      if (lam >= 2) {
        cnt += 1;
        break;
      }
    }
  }
  cnt = wave_sum(cnt);
  if (lane_id() == 0 && cnt) atomicAdd((unsigned long long *)&out[4], (unsigned long long)cnt);
}

inline unsigned grid_for(int64_t work, int block, int64_t cap) {
  int64_t g = (work + block - 1) / block;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (unsigned)g;
}

}  // namespace

hipError_t launch_check_part(Ctx &c, const int32_t *part) {
  hipLaunchKernelGGL(k_check_part, dim3(grid_for(c.n, 256, 16384)), dim3(256), 0, c.stream, part, c.n, c.k, c.st);
  return hipGetLastError();
}

namespace {

// Counts of every net, and with ns the connectivity words.  Every row is written whole.
template <int NW, typename T>
hipError_t build_counts(Ctx &c, const int32_t *part, T *phi, uint64_t *ns) {
  // four counts per store where rows begin on a multiple of it (a caller's table may begin anywhere)
  const int32_t vec = c.k % 4 == 0 && reinterpret_cast<uintptr_t>(phi) % (4 * sizeof(T)) == 0 ? 1 : 0;
  if (c.nchunks > 0)
    launch_resident<k_state_chunks<NW, T>>(c, ((int64_t)c.nchunks + 3) / 4, 256, c.pins, c.chunks, c.pnet, c.nchunks,
                                           part, c.k, phi, ns, vec);
  if (c.nmid + c.nbig > 0)
    hipLaunchKernelGGL((k_state_large<NW, T>), dim3((unsigned)(c.nmid + c.nbig)), dim3(256), 0, c.stream, c.off,
                       c.pins, c.big_nets, c.nbig, c.mid_nets, part, c.k, phi, ns);
  return hipGetLastError();
}

template <typename T>
hipError_t build_counts(Ctx &c, const int32_t *part, T *phi, uint64_t *ns) {
  return c.nw_words == 1 ? build_counts<1>(c, part, phi, ns) : build_counts<2>(c, part, phi, ns);
}

}  // namespace

hipError_t launch_build_phi(Ctx &c, const int32_t *part, int32_t *phi) {
  return build_counts(c, part, phi, (uint64_t *)nullptr);
}

hipError_t launch_build_counts(Ctx &c, const int32_t *part) {
  return c.phi16 ? build_counts(c, part, c.phi16, c.ns) : build_counts(c, part, c.phi, c.ns);
}

hipError_t launch_block_weights(Ctx &c, const int32_t *part) {
  const size_t nseg = (c.H > 1 ? (size_t)c.H + 1 : 1) * (size_t)c.k;  // a union's padding has its own segments
  hipError_t e = hipMemsetAsync(c.st->bw, 0, sizeof(int64_t) * nseg, c.stream);
  if (e == hipSuccess) e = hipMemsetAsync(c.st->bcnt, 0, sizeof(int32_t) * nseg, c.stream);
  if (e != hipSuccess) return e;
  // few workgroups: each adds up to k weights and counts to the same addresses
  hipLaunchKernelGGL(k_block_weights, dim3(grid_for(c.n, 256, c.H > 1 ? 2048 : 256)), dim3(256), 0, c.stream, part, c.vw, c.n, c.k,
                     c.st, union_of(c));
  return hipGetLastError();
}

hipError_t launch_km1_from_ns(Ctx &c) {
  hipError_t e = hipMemsetAsync(c.st->slot, 0, offsetof(DevStatus, km1) + sizeof(int64_t), c.stream);
  if (e == hipSuccess && c.H > 1) e = hipMemsetAsync(c.st->hkm1, 0, sizeof(int64_t) * (size_t)c.H, c.stream);
  if (e != hipSuccess) return e;
  const unsigned g = grid_for(c.m, 256, c.H > 1 ? 4096 : 1024);
  if (c.nw_words == 1)
    hipLaunchKernelGGL(k_km1<1>, dim3(g), dim3(256), 0, c.stream, c.ns, c.nw, c.m, c.st, union_of(c));
  else
    hipLaunchKernelGGL(k_km1<2>, dim3(g), dim3(256), 0, c.stream, c.ns, c.nw, c.m, c.st, union_of(c));
  return hipGetLastError();
}

hipError_t launch_level_stats(Ctx &c, int64_t *out5) {
  hipError_t e = hipMemsetAsync(out5, 0, 5 * sizeof(int64_t), c.stream);
  if (e != hipSuccess) return e;
  const unsigned gm = grid_for(c.m, 256, 4096), gn = grid_for(c.n, 256, 4096);
  if (c.nw_words == 1) {
    hipLaunchKernelGGL(k_stats_nets<1>, dim3(gm), dim3(256), 0, c.stream, c.off, c.ns, c.nw, c.m, out5);
    hipLaunchKernelGGL(k_stats_boundary<1>, dim3(gn), dim3(256), 0, c.stream, c.voff, c.inc, c.ns, c.n, out5);
  } else {
    hipLaunchKernelGGL(k_stats_nets<2>, dim3(gm), dim3(256), 0, c.stream, c.off, c.ns, c.nw, c.m, out5);
    hipLaunchKernelGGL(k_stats_boundary<2>, dim3(gn), dim3(256), 0, c.stream, c.voff, c.inc, c.ns, c.n, out5);
  }
  return hipGetLastError();
}

}  // namespace jet
