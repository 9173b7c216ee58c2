// What the censuses by subgraph copies share (counts.hip, copies5.hip): the
// lists of vertices by work and small device helpers.
#pragma once
#include <hip/hip_runtime.h>

#include "codes.h"
#include "internal.h"

namespace motif {

constexpr uint32_t kNone = 0xFFFFFFFFu;

// Lists of vertices by the work they bring, counted in the zeroed queue words
// of a census (64 int32).  Units are dealt out by position, not pulled from a
// counter: a pull is an atomic on one address, about 25 ns each however many
// waves wait for it, which was most of these kernels' time on 10^4 vertices.
enum ListId : int { kTri16 = 0, kTri64 = 1, kTri128 = 2, kTriBig = 3, kWedge16 = 4, kWedge64 = 5, kWedge256 = 6,
                    kWedgeTop = 7, kWedgeHuge = 8, kWedgeFar7 = 9, kWedgeFar11 = 10, kLists = 11 };
struct Lists {
  int32_t* v[kLists];
};
constexpr int kHugeD = 1000;  // lower neighbours from which a vertex's wedges are cut by row entries too
// On graphs of many ids (kFarBlocks): visits and lower neighbours up to which a
// vertex's wedges are hashed in parts instead of counted block by block.
constexpr int kFarVisits = 65536, kFarD = 1024, kFarBlocks = 32;
constexpr int kCap16 = 96, kCap64 = 384, kCap256 = 3072;  // visits of a vertex in the three wedge hashes

__device__ __forceinline__ uint32_t hash_mul(uint32_t x, int bits) { return (x * 2654435761u) >> (32 - bits); }

__device__ __forceinline__ void gadd(uint64_t* a, u64 v) {
  if (v) atomicAdd(reinterpret_cast<u64*>(a), v);
}

__device__ __forceinline__ uint32_t typ(const uint4& d, uint32_t t) { return t == 1u ? d.x : t == 2u ? d.y : d.z; }

// body(i, p[i]) for i = r, r + step, r + 2 step, r + 3 step below m, the four
// loads issued together.
template <class F>
__device__ __forceinline__ void each4(const uint32_t* p, int32_t r, int32_t step, int32_t m, F&& body) {
  uint32_t f[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) f[k] = p[min(r + k * step, m - 1)];
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (r + k * step < m) body(r + k * step, f[k]);
}

__device__ __forceinline__ bool ranked_below(const DevGraph& G, uint32_t dw, int32_t w, uint32_t du, int32_t u) {
  return dw < du || (dw == du && w < u);
}

// A word of packed counters that holds one single wedge: one bit set, at the
// foot of a field (ones: the feet).
template <class W>
__device__ __forceinline__ bool one_wedge(W c, W ones) {
  return (c & (c - 1)) == 0 && (c & ones) != 0;
}
constexpr u64 kOnes7 = 1ull | 1ull << 7 | 1ull << 14 | 1ull << 21 | 1ull << 28 | 1ull << 35 | 1ull << 42 | 1ull << 49 |
                       1ull << 56;

// Side streams of a pipeline (default priority), made on first use; when one
// cannot be had its work stays on the caller's stream.
struct Chains {
  Pipeline& p;
  hipStream_t s;
  bool used[Pipeline::kChains] = {};
  Chains(Pipeline& pl, hipStream_t st) : p(pl), s(st) {}
  hipStream_t on(int i) const { return used[i] ? p.chain[i] : s; }
  void fork(int i) {  // chain i goes on from here
    if (!p.may_fork) return;
    if (!p.ev_chain && hipEventCreateWithFlags(&p.ev_chain, hipEventDisableTiming) != hipSuccess) p.ev_chain = nullptr;
    if (!p.chain[i] && hipStreamCreateWithFlags(&p.chain[i], hipStreamNonBlocking) != hipSuccess) p.chain[i] = nullptr;
    if (!p.ev_end[i] && hipEventCreateWithFlags(&p.ev_end[i], hipEventDisableTiming) != hipSuccess) p.ev_end[i] = nullptr;
    if (p.chain[i] && p.ev_end[i] && p.ev_chain && hipEventRecord(p.ev_chain, s) == hipSuccess &&
        hipStreamWaitEvent(p.chain[i], p.ev_chain, 0) == hipSuccess)
      used[i] = true;
  }
  void join() {
    for (int i = 0; i < Pipeline::kChains; ++i)
      if (used[i] && (hipEventRecord(p.ev_end[i], p.chain[i]) != hipSuccess ||
                      hipStreamWaitEvent(s, p.ev_end[i], 0) != hipSuccess))
        (void)hipStreamSynchronize(p.chain[i]);
  }
};

}  // namespace motif
