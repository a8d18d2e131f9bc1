// Per-vertex block connectivity, shared by the candidate and rebalancing kernels: with net weights first,
// with unit weights (bit-sliced) below.
//
// G lanes cooperate on one vertex v; lane j of the group owns blocks 8j .. 8j+7 and accumulates
//     conn[b] = sum of w(e) over incident nets e that have a pin in block b
// from the nets' connectivity words; every lane also accumulates
//     benefit  = sum of w(e) over incident nets where v is the only pin in s.
// With aff = w(I(v)) - benefit (incident nets with at least two pins in s):
//     gain(v, b) = conn[b] - aff        for b != s
// (Section 2 metric; a net gains b when it had no pin there, loses s when v was its last pin there).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace jet {

// Group-parallel form: lane lg of the group loads incident net (base + lg) of each batch of G
// consecutive incidences, so the group keeps G independent load chains in flight; the batch is
// then exchanged inside the group with cross-lane shuffles (each lane takes the 32-bit half of
// the mask word holding its byte).  Batches start at q0, q0 + stride, ... below q1.  The
// arguments are equal for the G lanes of a group, so the shuffles only ever read lanes of the
// same group that run the same iteration.
template <int G>
__device__ __forceinline__ void conn_accumulate(const int32_t *__restrict__ inc, int64_t q0, int64_t q1,
                                                int64_t stride, const int32_t *__restrict__ nw,
                                                const uint64_t *__restrict__ ns, int lg, int32_t s,
                                                int32_t conn[8], int32_t &benefit) {
  constexpr int NW = (G == 16) ? 2 : 1;
  constexpr int U = 4;               // batches whose loads are issued before any is consumed
  const int word = lg >> 3;          // mask word holding this lane's blocks
  const int half = (lg & 7) >> 2;    // 32-bit half of that word
  const int shift = (lg & 3) * 8;    // byte inside the half
  const int sw = s >> 6;
  const uint64_t sbit = 1ull << (s & 63);
  for (int64_t b0 = q0; b0 < q1; b0 += U * stride) {
    int32_t e[U], w[U], own[U];
    uint32_t lo[U][NW], hi[U][NW];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t q = b0 + u * stride + lg;
      e[u] = q < q1 ? inc[q] : -1;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      w[u] = 0;
      own[u] = 0;
#pragma unroll
      for (int x = 0; x < NW; ++x) {
        lo[u][x] = 0u;
        hi[u][x] = 0u;
      }
      if (e[u] >= 0) {
        w[u] = nw[e[u]];
        const uint64_t *nse = ns + (int64_t)e[u] * (2 * NW);
        uint64_t one;
        if (NW == 1) {  // mask and "one pin" word in one access
          const ulonglong2 q = *reinterpret_cast<const ulonglong2 *>(nse);
          lo[u][0] = (uint32_t)q.x;
          hi[u][0] = (uint32_t)(q.x >> 32);
          one = q.y;
        } else {
#pragma unroll
          for (int x = 0; x < NW; ++x) {
            const uint64_t m = nse[x];
            lo[u][x] = (uint32_t)m;
            hi[u][x] = (uint32_t)(m >> 32);
          }
          one = nse[NW + sw];
        }
        own[u] = (one & sbit) ? w[u] : 0;  // v is this net's only pin in s
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (b0 + u * stride >= q1) break;  // uniform over the group
#pragma unroll
      for (int j = 0; j < G; ++j) {
        const int32_t wj = __shfl(w[u], j, G);
        const int32_t oj = __shfl(own[u], j, G);
        uint32_t mine = 0u;
#pragma unroll
        for (int x = 0; x < NW; ++x) {
          const uint32_t l32 = (uint32_t)__shfl((int)lo[u][x], j, G);
          const uint32_t h32 = (uint32_t)__shfl((int)hi[u][x], j, G);
          if (x == word) mine = half ? h32 : l32;
        }
        const uint32_t byte = (mine >> shift) & 0xffu;
#pragma unroll
        for (int b = 0; b < 8; ++b) conn[b] += ((byte >> b) & 1u) ? wj : 0;
        benefit += oj;
      }
    }
  }
}

// Sequential form for one lane per vertex (G = 1): four incident nets per step.
__device__ __forceinline__ void conn_accumulate_lane(const int32_t *__restrict__ inc, int64_t q0, int64_t q1,
                                                     const int32_t *__restrict__ nw,
                                                     const uint64_t *__restrict__ ns, int32_t s, int32_t conn[8],
                                                     int32_t &benefit) {
  const uint64_t sbit = 1ull << (s & 63);
  auto add = [&](uint64_t mw, uint64_t ow, int32_t w) {
    const uint32_t byte = (uint32_t)mw & 0xffu;
#pragma unroll
    for (int j = 0; j < 8; ++j) conn[j] += ((byte >> j) & 1u) ? w : 0;
    if (ow & sbit) benefit += w;
  };
  int64_t q = q0;
  for (; q + 3 < q1; q += 4) {
    const int32_t e0 = inc[q], e1 = inc[q + 1], e2 = inc[q + 2], e3 = inc[q + 3];
    const uint64_t *n0 = ns + (int64_t)e0 * 2, *n1 = ns + (int64_t)e1 * 2;
    const uint64_t *n2 = ns + (int64_t)e2 * 2, *n3 = ns + (int64_t)e3 * 2;
    const uint64_t m0 = n0[0], m1 = n1[0], m2 = n2[0], m3 = n3[0];
    const uint64_t o0 = n0[1], o1 = n1[1], o2 = n2[1], o3 = n3[1];
    const int32_t w0 = nw[e0], w1 = nw[e1], w2 = nw[e2], w3 = nw[e3];
    add(m0, o0, w0);
    add(m1, o1, w1);
    add(m2, o2, w2);
    add(m3, o3, w3);
  }
  for (; q < q1; ++q) {
    const int32_t e = inc[q];
    add(ns[(int64_t)e * 2], ns[(int64_t)e * 2 + 1], nw[e]);
  }
}

// Strided form: each lane of the group walks q0, q0 + step, ... itself (all lanes of the group load
// the same incident net); four nets per step.  Used by the workgroup-per-vertex kernels with G = 1.
template <int G>
__device__ __forceinline__ void conn_accumulate_strided(const int32_t *__restrict__ inc, int64_t q0, int64_t q1,
                                                        int64_t step, const int32_t *__restrict__ nw,
                                                        const uint64_t *__restrict__ ns, int lg, int32_t s,
                                                        int32_t conn[8], int32_t &benefit) {
  constexpr int NW = (G == 16) ? 2 : 1;
  const int word = lg >> 3;
  const int shift = (lg & 7) * 8;
  const int sw = s >> 6;
  const uint64_t sbit = 1ull << (s & 63);
  auto add = [&](uint64_t mw, uint64_t ow, int32_t w) {
    const uint32_t byte = (uint32_t)(mw >> shift) & 0xffu;
#pragma unroll
    for (int j = 0; j < 8; ++j) conn[j] += ((byte >> j) & 1u) ? w : 0;
    if (ow & sbit) benefit += w;
  };
  int64_t q = q0;
  for (; q + 3 * step < q1; q += 4 * step) {
    const int32_t e0 = inc[q], e1 = inc[q + step], e2 = inc[q + 2 * step], e3 = inc[q + 3 * step];
    const uint64_t *n0 = ns + (int64_t)e0 * (2 * NW), *n1 = ns + (int64_t)e1 * (2 * NW);
    const uint64_t *n2 = ns + (int64_t)e2 * (2 * NW), *n3 = ns + (int64_t)e3 * (2 * NW);
    const uint64_t m0 = n0[word], m1 = n1[word], m2 = n2[word], m3 = n3[word];
    const uint64_t o0 = n0[NW + sw], o1 = n1[NW + sw], o2 = n2[NW + sw], o3 = n3[NW + sw];
    const int32_t w0 = nw[e0], w1 = nw[e1], w2 = nw[e2], w3 = nw[e3];
    add(m0, o0, w0);
    add(m1, o1, w1);
    add(m2, o2, w2);
    add(m3, o3, w3);
  }
  for (; q < q1; q += step) {
    const int32_t e = inc[q];
    const uint64_t *nse = ns + (int64_t)e * (2 * NW);
    add(nse[word], nse[NW + sw], nw[e]);
  }
}

// Dispatch: conn[] and benefit of v over the incidences [q0, q1) walked in batches (see above).
template <int G>
__device__ __forceinline__ void vertex_conn(const int32_t *__restrict__ inc, int64_t q0, int64_t q1, int64_t stride,
                                            const int32_t *__restrict__ nw, const uint64_t *__restrict__ ns, int lg,
                                            int32_t s, int32_t conn[8], int32_t &benefit) {
  if (G == 1) conn_accumulate_lane(inc, q0, q1, nw, ns, s, conn, benefit);
  else conn_accumulate<G>(inc, q0, q1, stride, nw, ns, lg, s, conn, benefit);
}

// ---- bit-sliced counts (unit net weights) ----
// conn(v, b) for all blocks is kept in N bit planes of HW 32-bit words (HW = 1, 2, 4 for k <= 32, 64,
// 128): bit b of plane p is bit p of block b's count.  These passes are bound by vector instructions
// (four cycles each) before the gathers, so the masks of four nets enter through a tree of full adders
// (three instructions on a word: two XORs and a bit select), which is 23 instructions per word and four
// nets with nine planes; rippling each mask through the planes took 72.

// p + a + b: the sum bit stays in p, the carry is returned
__device__ __forceinline__ uint32_t full_add(uint32_t &p, uint32_t a, uint32_t b) {
  const uint32_t x = p ^ a, c = (x & b) | (~x & p);
  p = x ^ b;
  return c;
}

template <int N>
__device__ __forceinline__ void planes_add4(uint32_t (&pl)[N], uint32_t m0, uint32_t m1, uint32_t m2, uint32_t m3) {
  const uint32_t c0 = full_add(pl[0], m0, m1), c1 = full_add(pl[0], m2, m3);
  uint32_t d = full_add(pl[1], c0, c1);
#pragma unroll
  for (int p = 2; p < N; ++p) {
    const uint32_t t = pl[p] & d;
    pl[p] ^= d;
    d = t;
  }
}

// Incidences q, q + step, ... below q1 of one lane (four in flight, at most 2^N - 1 in all): the nets'
// masks into the planes; benefit counts the nets where s is marked as holding one pin.
template <int HW, int N>
__device__ __forceinline__ void planes_accumulate(const int32_t *__restrict__ inc, int64_t q, int64_t q1, int64_t step,
                                                  const uint64_t *__restrict__ ns, int32_t s, uint32_t (&pl)[HW][N],
                                                  int32_t &benefit) {
  const uint4 *words = reinterpret_cast<const uint4 *>(ns);  // HW <= 2: mask, one; HW == 4: mask, then one
  const uint32_t sbit = 1u << (s & 31);
  const int sw = s >> 5;
  for (; q < q1; q += 4 * step) {
    int32_t e[4];
    uint4 a[4], b[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) e[u] = q + u * step < q1 ? inc[q + u * step] : -1;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      a[u] = make_uint4(0u, 0u, 0u, 0u);
      b[u] = make_uint4(0u, 0u, 0u, 0u);
      if (e[u] >= 0) {
        if (HW == 4) {
          a[u] = words[(int64_t)e[u] * 2];
          b[u] = words[(int64_t)e[u] * 2 + 1];
        } else {
          a[u] = words[e[u]];
        }
      }
    }
    planes_add4(pl[0], a[0].x, a[1].x, a[2].x, a[3].x);
    if (HW >= 2) planes_add4(pl[HW >= 2 ? 1 : 0], a[0].y, a[1].y, a[2].y, a[3].y);
    if (HW == 4) {
      planes_add4(pl[HW == 4 ? 2 : 0], a[0].z, a[1].z, a[2].z, a[3].z);
      planes_add4(pl[HW == 4 ? 3 : 0], a[0].w, a[1].w, a[2].w, a[3].w);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t o = HW == 1   ? a[u].z
                         : HW == 2 ? (sw ? a[u].w : a[u].z)
                                   : (sw & 2 ? (sw & 1 ? b[u].w : b[u].z) : (sw & 1 ? b[u].y : b[u].x));
      benefit += (o & sbit) != 0u;
    }
  }
}

// The same for a graph (every net has two pins, adj holds the other one): the neighbours' blocks instead of
// the nets' words.  Only blocks other than s are added; benefit counts the neighbours outside s.  Inside
// a block nothing is (wave-uniformly: nothing that any lane needs).
template <int HW, int N>
__device__ __forceinline__ void planes_accumulate_graph(const int32_t *__restrict__ adj, int64_t q, int64_t q1,
                                                        const int32_t *__restrict__ part, int32_t s,
                                                        uint32_t (&pl)[HW][N], int32_t &benefit) {
  for (; q < q1; q += 8) {
    int32_t v[8], b[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = q + u < q1 ? adj[q + u] : -1;
#pragma unroll
    for (int u = 0; u < 8; ++u) b[u] = v[u] >= 0 ? part[v[u]] : s;
    int32_t out = 0;
#pragma unroll
    for (int u = 0; u < 8; ++u) out += b[u] != s;
    benefit += out;
    if (!ballot(out != 0)) continue;
    uint32_t m[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) m[u] = b[u] != s ? 1u << (b[u] & 31) : 0u;
#pragma unroll
    for (int x = 0; x < HW; ++x) {
#pragma unroll
      for (int h = 0; h < 8; h += 4)
        planes_add4(pl[x], (b[h] >> 5) == x ? m[h] : 0u, (b[h + 1] >> 5) == x ? m[h + 1] : 0u,
                    (b[h + 2] >> 5) == x ? m[h + 2] : 0u, (b[h + 3] >> 5) == x ? m[h + 3] : 0u);
    }
  }
}

// a += b over N planes, the last carry dropped (the caller's counts fit)
template <int N>
__device__ __forceinline__ void planes_sum(uint32_t (&a)[N], const uint32_t (&b)[N]) {
  uint32_t c = 0u;
#pragma unroll
  for (int p = 0; p < N; ++p) {
    uint32_t x = a[p];
    c = full_add(x, b[p], c);
    a[p] = x;
  }
}

// Sums the planes of the lanes of each aligned group of GL lanes.  Every lane ends with one word of the
// group's sums, out: lane bits 0.. choose it (bit 0 the upper or lower half of the words, bit 1 the
// half of that half), so each of the first log2(HW) exchanges moves only the words the partner keeps.
// Returns the word's index.  benefit is summed too.  M >= N planes hold the sums.
template <int GL, int HW, int N, int M>
__device__ __forceinline__ int planes_combine(uint32_t (&pl)[HW][N], uint32_t (&out)[M], int32_t &benefit, int lane) {
  uint32_t w[HW][M];
#pragma unroll
  for (int x = 0; x < HW; ++x)
#pragma unroll
    for (int p = 0; p < M; ++p) w[x][p] = p < N ? pl[x][p] : 0u;
  int word = 0, o = 1;
  int have = HW;  // words still held (compile-time after unrolling)
#pragma unroll
  for (int step = 0; step < 2; ++step) {
    if (have == 1 || o >= GL) break;
    const int half = have / 2;
    const bool up = (lane & o) != 0;  // keeps the upper half
#pragma unroll
    for (int x = 0; x < HW / 2; ++x) {
      if (x >= half) break;
      uint32_t mine[M], theirs[M];
#pragma unroll
      for (int p = 0; p < M; ++p) {
        const uint32_t lo = w[x][p], hi = w[x + half < HW ? x + half : 0][p];
        mine[p] = up ? hi : lo;
        theirs[p] = (uint32_t)__shfl_xor((int)(up ? lo : hi), o, GL);
      }
      planes_sum<M>(mine, theirs);
#pragma unroll
      for (int p = 0; p < M; ++p) w[x][p] = mine[p];
    }
    word = 2 * word + (up ? 1 : 0);
    benefit += __shfl_xor(benefit, o, GL);
    have = half;
    o <<= 1;
  }
#pragma unroll
  for (int r = 0; r < 6; ++r) {
    if (o >= GL) break;
    uint32_t theirs[M];
#pragma unroll
    for (int p = 0; p < M; ++p) theirs[p] = (uint32_t)__shfl_xor((int)w[0][p], o, GL);
    planes_sum<M>(w[0], theirs);
    benefit += __shfl_xor(benefit, o, GL);
    o <<= 1;
  }
#pragma unroll
  for (int p = 0; p < M; ++p) out[p] = w[0][p];
  return word;
}

// Lowest block of largest count among the blocks of mask in one word (counts of zero included): the
// mask is narrowed from the top plane down.  Returns the count, -1 when the mask is empty.
template <int M>
__device__ __forceinline__ int32_t planes_best(const uint32_t (&pl)[M], uint32_t mask, int32_t &bit) {
  bit = 0;
  if (!mask) return -1;
  int32_t c = 0;
#pragma unroll
  for (int p = M - 1; p >= 0; --p) {
    const uint32_t x = mask & pl[p];
    mask = x ? x : mask;
    c |= x ? 1 << p : 0;
  }
  bit = __ffs((int)mask) - 1;
  return c;
}

// blocks with a nonzero count
template <int M>
__device__ __forceinline__ uint32_t planes_any(const uint32_t (&pl)[M]) {
  uint32_t any = 0u;
#pragma unroll
  for (int p = 0; p < M; ++p) any |= pl[p];
  return any;
}

// The best block of a vertex whose counts a group of G lanes holds in pl: valid(word index, counts) is
// the mask of allowed blocks of a word.  Every lane of the group returns the count (-1: none) and block
// (lowest on ties); benefit becomes the group's sum.
template <int G, int HW, int N, typename Valid>
__device__ __forceinline__ int32_t planes_target(uint32_t (&pl)[HW][N], int32_t &benefit, int lane, int32_t &block,
                                                 Valid valid) {
  int32_t bestc = -1, bestb = 0;
  if (G == 1) {
#pragma unroll
    for (int x = 0; x < HW; ++x) {
      int32_t b;
      const int32_t c = planes_best<N>(pl[x], valid(x, pl[x]), b);
      if (c > bestc) {
        bestc = c;
        bestb = 32 * x + b;
      }
    }
  } else {
    static_assert(G == 1 || G >= HW, "a lane for every word");
    uint32_t w[N];
    const int x = planes_combine<G, HW, N, N>(pl, w, benefit, lane);
    bestc = planes_best<N>(w, valid(x, w), bestb);
    bestb += 32 * x;
#pragma unroll
    for (int o = 1; o < HW; o <<= 1) {  // the lanes that hold the other words
      const int32_t oc = __shfl_xor(bestc, o, G), ob = __shfl_xor(bestb, o, G);
      if (oc > bestc || (oc == bestc && ob < bestb)) {
        bestc = oc;
        bestb = ob;
      }
    }
  }
  block = bestb;
  return bestc;
}

}  // namespace jet
