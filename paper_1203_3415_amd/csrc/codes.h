// Adjacency codes of the census kernels (device side): bit layout, code bits
// of a labelled member and of an edge, and small wave helpers.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "internal.h"

namespace motif {

using u64 = unsigned long long;

// Whether an earlier step of the call failed, an in-CSR check beside the
// censuses included: for the last steps, which run after it on the stream.
__device__ __forceinline__ bool failed(const int32_t* st) { return st[kStatus] != 0 || st[kBeside] != 0; }

// Bit of the arc i -> j (i != j) in the adjacency codes that index the
// device class tables.  Row-major with the diagonal left out, except for
// k = 5, where the two arcs between slots 3 and 4 (the members of a pair in
// the closed forms) are moved to bits 0 and 1 and the rest keep their order
// above them: a code without that edge and its three variants with it are
// then four consecutive entries of the 2 MB table, one aligned 8-byte read
// (lut_quad) instead of two.  (For k = 4 the table sits in LDS, and the same
// order measured slightly slower.)  The host table keeps row-major order;
// device_lut_order writes the device copy in this one.
template <int K>
__host__ __device__ constexpr int cbit(int i, int j) {
  const int n = i * (K - 1) + (j < i ? j : j - 1);
  if (K != 5) return n;
  const int a = (K - 2) * K, b = (K - 1) * (K - 1) + K - 2;  // row-major bits of (3, 4) and (4, 3)
  return n == a ? 0 : n == b ? 1 : n < a ? n + 2 : n < b ? n + 1 : n;
}
static_assert(cbit<5>(3, 4) == 0 && cbit<5>(4, 3) == 1 && cbit<5>(0, 1) == 2 && cbit<5>(4, 2) == 19 &&
                  cbit<5>(3, 2) == 16 && cbit<5>(4, 0) == 17,
              "k = 5 order");

// Code bits of a neighbour placed in slot S whose types towards the anchor
// vertices 0..K-3 are packed 2 bits each in L (1 = arc anchor->x, 2 = arc
// x->anchor, 3 = both).
template <int K, int S>
__device__ __forceinline__ uint32_t slot_code(uint32_t L) {
  uint32_t c = 0;
#pragma unroll
  for (int i = 0; i < K - 2; ++i) {
    const uint32_t t = (L >> (2 * i)) & 3u;
    c |= (t & 1u) ? (1u << cbit<K>(i, S)) : 0u;
    c |= (t & 2u) ? (1u << cbit<K>(S, i)) : 0u;
  }
  return c;
}

// Code bits of the edge between slot K-2 (x) and slot K-1 (y); t = type of y
// relative to x.
template <int K>
__device__ __forceinline__ uint32_t rel_code(uint32_t t) {
  return ((t & 1u) ? (1u << cbit<K>(K - 2, K - 1)) : 0u) | ((t & 2u) ? (1u << cbit<K>(K - 1, K - 2)) : 0u);
}

// Code bits of the edge between slots i and j; t = type of j relative to i.
template <int K>
__host__ __device__ __forceinline__ constexpr uint32_t edge_code(int i, int j, uint32_t t) {
  return ((t & 1u) ? 1u << cbit<K>(i, j) : 0u) | ((t & 2u) ? 1u << cbit<K>(j, i) : 0u);
}

// The type of an edge seen from its other end.
__device__ __forceinline__ uint32_t flip(uint32_t t) { return ((t & 1u) << 1) | ((t & 2u) >> 1); }

constexpr int num_classes(int k) { return k == 3 ? 13 : k == 4 ? 199 : 9364; }

// Ordering point for LDS traffic inside one wave: LDS operations of a wave
// complete in issue order, so only the compiler has to be kept from moving
// accesses across it.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace motif
