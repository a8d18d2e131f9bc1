// One node's turn of a push-relabel sweep on the network of FlowState (kernel k_fl_sweep), apart from the
// kernel so that a host build can run it under other orders of memory operations.  Include after
// hip/hip_runtime.h.
//
// The turns of a sweep run at once with relaxed atomics only, so a node may see the excess of a push before
// the residual of the arc that brought it, on every load of its turn.  Then it finds no residual arc, or
// not the lowest one, and relabels too far (past 2N at worst).  Nothing is lost by that: the sums are exact
// once the sweep has ended.  A node without a residual arc waits for the next sweep, nodes at 2N get
// exact heights from a global relabel, and a flow that ends with the sinks in the sources' reach
// (an arc stayed steep) goes on from its saturated sources; max_flow and flow_pair see to both.
#pragma once
#include <stdint.h>

namespace jet {

constexpr int kPushCycles = 64;  // push or relabel steps of one node per sweep
constexpr int kSweepU = 8;       // arcs whose loads are in flight together

template <typename T>
__device__ __forceinline__ T ld(const T *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void push(int64_t a, int32_t u, int32_t v, int64_t d, int64_t *res, int64_t *ex) {
  atomicAdd((unsigned long long *)&res[a], (unsigned long long)(-d));
  atomicAdd((unsigned long long *)&res[a ^ 1], (unsigned long long)d);
  atomicAdd((unsigned long long *)&ex[u], (unsigned long long)(-d));
  atomicAdd((unsigned long long *)&ex[v], (unsigned long long)d);
}

// Out-arcs of node u by index: vertex nodes (u < nv) have two per adjacency entry (x -> e_in, and x -> e_out
// as the reverse of e_out -> x), net nodes one to their partner node and one per endpoint.
struct OutArcs {
  int64_t base;  // first adjacency entry of a vertex node, arc block of a net node
  int32_t count;
  bool vertex, out;
};
__device__ __forceinline__ OutArcs out_arcs(int64_t u, int32_t nv, const int64_t *voffn, const int64_t *rbase,
                                            const int32_t *rends) {
  if (u < nv) {
    const int64_t lo = voffn[u];
    return OutArcs{lo, (int32_t)(2 * (voffn[u + 1] - lo)), true, false};
  }
  const int64_t r = (u - nv) >> 1;
  return OutArcs{rbase[r], 1 + rends[r], false, ((u - nv) & 1) != 0};
}
__device__ __forceinline__ int64_t out_arc(const OutArcs &o, const int64_t *vadj, int32_t i) {
  if (o.vertex) return vadj[o.base + (i >> 1)] + (i & 1 ? 3 : 0);
  if (i == 0) return o.base + (o.out ? 1 : 0);
  return o.base + 2 + 4 * (int64_t)(i - 1) + (o.out ? 2 : 1);
}

// An active node (free, positive excess, height below 2N) pushes to its lowest residual neighbour if that is
// lower, else relabels to one above it.  Only u's thread lowers u's excess and the residuals of u's arcs,
// so a push never takes more than is there.  A step is a chain of loads past the caches (residual, head,
// height), issued for kSweepU arcs at a time.
__device__ __forceinline__ void sweep_node(int64_t u, int64_t N, int32_t nv, const uint8_t *term, int32_t *h,
                                           int64_t *ex, int64_t *res, const int32_t *head, const int64_t *voffn,
                                           const int64_t *vadj, const int64_t *rbase, const int32_t *rends) {
  const int32_t h2n = (int32_t)(2 * N);
  const uint8_t tu = term[u];
  int64_t e = ld(&ex[u]);
  int32_t hu = h[u];
  if (tu != 0 || e <= 0 || hu >= h2n) return;
  const OutArcs o = out_arcs(u, nv, voffn, rbase, rends);
  for (int c = 0; c < kPushCycles; ++c) {
    int64_t best_a = -1, best_r = 0;
    int32_t best_h = INT32_MAX, best_v = 0;
    for (int32_t i0 = 0; i0 < o.count; i0 += kSweepU) {
      int64_t a[kSweepU], r[kSweepU];
      int32_t v[kSweepU], hv[kSweepU];
#pragma unroll
      for (int i = 0; i < kSweepU; ++i) a[i] = i0 + i < o.count ? out_arc(o, vadj, i0 + i) : -1;
#pragma unroll
      for (int i = 0; i < kSweepU; ++i) {
        r[i] = a[i] >= 0 ? ld(&res[a[i]]) : 0;
        v[i] = a[i] >= 0 ? head[a[i]] : 0;
      }
#pragma unroll
      for (int i = 0; i < kSweepU; ++i) hv[i] = r[i] > 0 ? ld(&h[v[i]]) : INT32_MAX;
#pragma unroll
      for (int i = 0; i < kSweepU; ++i)
        if (r[i] > 0 && hv[i] < best_h) {
          best_h = hv[i];
          best_a = a[i];
          best_r = r[i];
          best_v = v[i];
        }
    }
    if (best_a < 0) return;  // the residual that came with the excess is not visible yet
    if (hu > best_h) {
      const int64_t d = e < best_r ? e : best_r;  // the residual can only have grown since it was read
      push(best_a, (int32_t)u, best_v, d, res, ex);
    } else {
      hu = best_h + 1 < h2n ? best_h + 1 : h2n;
      __hip_atomic_store(&h[u], hu, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    e = ld(&ex[u]);
    if (e <= 0 || hu >= h2n) return;
  }
}

}  // namespace jet
