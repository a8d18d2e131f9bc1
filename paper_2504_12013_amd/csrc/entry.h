// Rebalancing entries (Section 4.3): the exact order key of a move, shared by the kernels that write
// entries (gain passes) and the selection.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace jet {

__device__ __forceinline__ uint32_t mono_code(unsigned __int128 x) {
  if (x == 0) return 0u;
  const uint64_t hi = (uint64_t)(x >> 64), lo = (uint64_t)x;
  const int L = hi ? 128 - __clzll(hi) : 64 - __clzll(lo);  // bit length, 1..128
  uint32_t mant;
  if (L - 1 >= 24) mant = (uint32_t)(x >> (L - 1 - 24)) & 0xffffffu;
  else mant = (uint32_t)(x << (24 - (L - 1))) & 0xffffffu;
  return ((uint32_t)L << 24) | mant;
}

__device__ __forceinline__ void priority_key(int32_t g, int32_t c, int32_t v, uint32_t key[5]) {
  const unsigned __int128 bias = (unsigned __int128)1 << 95;
  unsigned __int128 U;
  if (g >= 0) {
    const unsigned __int128 gc = (unsigned __int128)((uint64_t)(uint32_t)g * (uint64_t)(uint32_t)c);
    U = bias + gc;
    key[0] = 0x80000000u | mono_code(gc);
  } else {
    const uint64_t a = (uint64_t)(-(int64_t)g), cc = (uint64_t)(uint32_t)c;
    const uint64_t q0 = a / cc, r0 = a % cc;
    const uint64_t x1 = r0 << 31, f1 = x1 / cc, r1 = x1 % cc;
    const uint64_t x2 = r1 << 31, f2 = x2 / cc, r2 = x2 % cc;
    const unsigned __int128 ce =
        ((unsigned __int128)q0 << 62) + ((unsigned __int128)f1 << 31) + (unsigned __int128)f2 + (r2 != 0 ? 1 : 0);
    U = bias - ce;
    key[0] = 0x7fffffffu - mono_code(ce);
  }
  key[1] = (uint32_t)(U >> 64);
  key[2] = (uint32_t)(U >> 32);
  key[3] = (uint32_t)U;
  key[4] = 0xffffffffu - (uint32_t)v;
}

// The key of an entry in the order jet_params.rb_unweighted names: 0 the priority of Section 4.3,
// 1 the gain alone (the original Jet's priority), 2 the original's bucket order of the loss
// (Section 4.3 contrasts it with the sort): a move that does not lose goes to bucket 0, a loss
// L >= 1 to bucket 1 + floor(log2 L); lower buckets first, and inside a bucket vertex-ID order
// stands in for the original's arrival order.  Bucket words: w0 = (255 - bucket) << 24,
// w1..w3 = 0 (so the selection skips their passes), w4 = 0xffffffff - v as for the priorities.
// The bucket words replace the others by selects, so the key stays in registers.
__device__ __forceinline__ void entry_key(int32_t g, int32_t c, int32_t v, int32_t order, uint32_t key[5]) {
  priority_key(g, order ? 1 : c, v, key);
  const bool bk = order == 2;
  const int32_t bucket = g >= 0 ? 0 : 64 - __clzll((unsigned long long)(-(int64_t)g));
  key[0] = bk ? (uint32_t)(255 - bucket) << 24 : key[0];
  key[1] = bk ? 0u : key[1];
  key[2] = bk ? 0u : key[2];
  key[3] = bk ? 0u : key[3];
}

// entry layout: 8 words = key[0..4], v, target, weight
constexpr int kEntryWords = 8;

// Entries are 32 bytes on a 32-byte boundary: two 16-byte accesses each.
__device__ __forceinline__ void load_entry(const uint32_t *__restrict__ p, uint32_t ent[kEntryWords]) {
  const uint4 a = reinterpret_cast<const uint4 *>(p)[0], b = reinterpret_cast<const uint4 *>(p)[1];
  ent[0] = a.x;
  ent[1] = a.y;
  ent[2] = a.z;
  ent[3] = a.w;
  ent[4] = b.x;
  ent[5] = b.y;
  ent[6] = b.z;
  ent[7] = b.w;
}
__device__ __forceinline__ void store_entry(uint32_t *__restrict__ p, const uint32_t ent[kEntryWords]) {
  reinterpret_cast<uint4 *>(p)[0] = make_uint4(ent[0], ent[1], ent[2], ent[3]);
  reinterpret_cast<uint4 *>(p)[1] = make_uint4(ent[4], ent[5], ent[6], ent[7]);
}

// One rebalancing entry: the exact order key, vertex, target and weight; a vertex without a valid
// target leaves weight 0 (the selection skips such entries).
// order: jet_params.rb_unweighted (entry_key); the entry keeps the real weight c
__device__ __forceinline__ void write_entry(uint32_t *p, bool ok, int32_t g, int32_t c, int32_t v, int32_t t,
                                            int32_t order) {
  uint32_t ent[kEntryWords] = {0u, 0u, 0u, 0u, 0u, (uint32_t)v, ok ? (uint32_t)t : 0xffu, ok ? (uint32_t)c : 0u};
  if (ok) entry_key(g, c, v, order, ent);
  store_entry(p, ent);
}

}  // namespace jet
