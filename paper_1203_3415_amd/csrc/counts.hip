// k = 3 and k = 4 censuses by counting typed subgraph copies (gfx950, wave64).
//
// The paper's anchors see a k-set once per anchor and correct the closed forms
// of the pairs of neighbours by the edges inside the neighbourhood (Theorem
// "teo3", Theorem "lema4d").  The same totals follow from fewer visits: for
// every class c, count the copies N(c) of c as a subgraph, that is the vertex
// sets with a subset of their edges (types kept) forming c, whatever the other
// pairs look like.  Each N has a closed form over small local counts,
//   k = 3  wedge     typed degrees;                triangle  listed
//   k = 4  claw      typed degrees;                P4        typed degrees of an edge's ends, less its triangles
//          paw       typed degrees of a triangle's corners
//          diamond   pairs of the typed triangles T of an edge
//          C4        pairs of the typed wedges W between two opposite vertices
//          K4        listed
// and a set of class c holds a fixed number of copies of each class, so the
// induced counts are a fixed integer combination of the N (inclusion and
// exclusion over the edges left out; subgraph_inverse in classes.cpp), taken
// once per graph by k_solve.  All sums are modulo 2^64 and the final counts
// exact.
//
// Work: the triangles and K4s from the oriented rows N+ (sum over edges x -> y
// of d+(y) visits), the wedges of every C4 from its vertex u of highest rank
// (sum over edges v -> u of d(v)).  On the n = 10^5, m = 10^6 power-law graph
// that is 3.0e7 and 4.6e7 visits, against 1.3e9 for the per-core scan of the
// anchors' neighbourhoods that this replaced.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "codes.h"
#include "internal.h"

namespace motif {

namespace {

constexpr uint32_t kNone = 0xFFFFFFFFu;
constexpr u64 kNeg = ~0ull;

// Counters in the zeroed queue words of a census (64 int32).
enum QueueSlot : int { kQTri = 0, kQTriBig = 1, kQWedge = 2, kQWedgeMid = 3, kQWedgeTop = 4, kQEdges = 6,
                       kNTriBig = 8, kNWedgeMid = 9, kNWedgeTop = 10 };

// Chunks of vertices handed out in batches: a workgroup works on one graph at
// a time, so that its LDS counters can be added to that graph's totals.
constexpr int kBatchChunk = 256;

__device__ __forceinline__ uint32_t hash_mul(uint32_t x, int bits) { return (x * 2654435761u) >> (32 - bits); }

__device__ __forceinline__ void gadd(uint64_t* a, u64 v) {
  if (v) atomicAdd(reinterpret_cast<u64*>(a), v);
}

__device__ __forceinline__ uint32_t typ(const uint4& d, uint32_t t) { return t == 1u ? d.x : t == 2u ? d.y : d.z; }

// ============================================================ triangles ==
//
// Every triangle x < y < z (rank order) once, from x: N+(x) in a wave-private
// hash, the N+ rows of its members streamed against it.  Per triangle: one
// count per typed triangle (27), and for k = 4 the typed degrees of its three
// corners (paws), the typed triangle counts T of its three edges (T[e][3 p +
// q], p, q the types of the third vertex seen from the lower and the higher
// end, less one) and one bit per type in a 64 x 64 adjacency of N+(x), from
// which the K4s above x are read off as the common bits of two rows.
// One wave per x with at most kTriD higher neighbours (sixteen lanes per row);
// the others go to k_tri_big.
constexpr int kTriD = 64;
constexpr int kTriHB = 8;
constexpr int kTriH = 1 << kTriHB;

// Workgroup counters of the triangle kernels and their flush to one graph.
template <bool K4>
struct TriBins {
  u64* tri;   // [27] typed triangles (xy, xz, yz)
  u64* paw;   // [27][3 corners][3 types] sums of the corner's typed degree
  u64* kh;    // [199] K4 classes
  __device__ __forceinline__ void clear(int t, int nt) const {
    for (int i = t; i < 27; i += nt) tri[i] = 0;
    if constexpr (K4) {
      for (int i = t; i < 243; i += nt) paw[i] = 0;
      for (int i = t; i < 199; i += nt) kh[i] = 0;
    }
  }
  // Adds everything to graph g's totals and clears (between barriers).
  __device__ __forceinline__ void flush(int32_t g, const uint16_t* lut3, const uint16_t* lut4, uint64_t* a3,
                                        uint64_t* a4, int t, int nt) const {
    for (int i = t; i < 27; i += nt) {
      const u64 c = tri[i];
      if (!c) continue;
      const uint32_t xy = (uint32_t)i / 9 + 1, xz = ((uint32_t)i / 3) % 3 + 1, yz = (uint32_t)i % 3 + 1;
      if (a3) gadd(&a3[(int64_t)g * 13 + lut3[edge_code<3>(0, 1, xy) | edge_code<3>(0, 2, xz) | edge_code<3>(1, 2, yz)]], c);
      if constexpr (K4) {
        // the paths of three edges whose ends are one vertex
        uint64_t* a = a4 + (int64_t)g * 199;
        auto p4 = [&](uint32_t mid, uint32_t p, uint32_t q) {
          gadd(&a[lut4[edge_code<4>(0, 1, mid) | edge_code<4>(0, 2, p) | edge_code<4>(1, 3, q)]], 0 - c);
        };
        p4(xy, xz, yz);
        p4(xz, xy, flip(yz));
        p4(yz, flip(xy), flip(xz));
      }
    }
    if constexpr (K4) {
      uint64_t* a = a4 + (int64_t)g * 199;
      for (int i = t; i < 243; i += nt) {
        const int tau = i / 9, corner = (i / 3) % 3;
        const u64 c = tri[tau];
        if (!c) continue;
        const uint32_t xy = (uint32_t)tau / 9 + 1, xz = ((uint32_t)tau / 3) % 3 + 1, yz = (uint32_t)tau % 3 + 1;
        const uint32_t s = (uint32_t)i % 3 + 1;
        // the corner's own two triangle neighbours are no pendants
        const uint32_t t1 = corner == 0 ? xy : corner == 1 ? flip(xy) : flip(xz);
        const uint32_t t2 = corner == 0 ? xz : corner == 1 ? yz : flip(yz);
        const u64 w = paw[i] - c * (u64)((t1 == s) + (t2 == s));
        gadd(&a[lut4[edge_code<4>(0, 1, xy) | edge_code<4>(0, 2, xz) | edge_code<4>(1, 2, yz) |
                     edge_code<4>(corner, 3, s)]], w);
      }
      for (int i = t; i < 199; i += nt) gadd(&a[i], kh[i]);
    }
  }
};

// One triangle: typed count and the corners' typed degrees.
template <bool K4>
__device__ __forceinline__ void tri_add(const TriBins<K4>& b, uint32_t tau, const uint4& dx, const uint4& dy,
                                        const uint4& dz) {
  atomicAdd(&b.tri[tau], 1ull);
  if constexpr (K4) {
    u64* p = b.paw + tau * 9;
    atomicAdd(&p[0], (u64)dx.x); atomicAdd(&p[1], (u64)dx.y); atomicAdd(&p[2], (u64)dx.z);
    atomicAdd(&p[3], (u64)dy.x); atomicAdd(&p[4], (u64)dy.y); atomicAdd(&p[5], (u64)dy.z);
    atomicAdd(&p[6], (u64)dz.x); atomicAdd(&p[7], (u64)dz.y); atomicAdd(&p[8], (u64)dz.z);
  }
}

template <bool K4>
__global__ __launch_bounds__(256) void k_tri(DevGraph G, const uint16_t* __restrict__ lut3,
                                             const uint16_t* __restrict__ lut4, uint64_t* __restrict__ a3,
                                             uint64_t* __restrict__ a4, uint32_t* __restrict__ T, const int32_t* st,
                                             int32_t* __restrict__ queue, int32_t chunk, int32_t* __restrict__ big) {
  constexpr int NW = 4;
  __shared__ u64 s_tri[27], s_paw[K4 ? 243 : 1], s_kh[K4 ? 199 : 1];
  __shared__ uint16_t lut[K4 ? 4096 : 1];
  __shared__ uint32_t s_key[NW][kTriH];
  __shared__ uint8_t s_at[NW][kTriH];
  __shared__ uint32_t s_list[NW][kTriD];
  __shared__ u64 s_T[K4 ? NW : 1][kTriD];                          // nine 7-bit counters per member of N+(x)
  __shared__ u64 s_a1[K4 ? NW : 1][kTriD], s_a2[K4 ? NW : 1][kTriD];  // adjacency of N+(x), a bit plane per arc
  __shared__ int32_t sh_v;
  if (st[kStatus] != 0) return;
  const TriBins<K4> bins{s_tri, s_paw, s_kh};
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  bins.clear(threadIdx.x, 256);
  if (K4)
    for (int i = threadIdx.x; i < 4096; i += 256) lut[i] = lut4[i];
  for (int i = lane; i < kTriH; i += 64) s_key[wv][i] = kNone;
  if (K4) {
    s_T[wv][lane] = 0;
    s_a1[wv][lane] = 0;
    s_a2[wv][lane] = 0;
  }
  __syncthreads();
  uint32_t* key = s_key[wv];
  uint8_t* at = s_at[wv];
  uint32_t* list = s_list[wv];
  u64 *Tl = s_T[K4 ? wv : 0], *A1 = s_a1[K4 ? wv : 0], *A2 = s_a2[K4 ? wv : 0];
  const int32_t n = G.n;

  auto one = [&](int32_t x) {  // uniform over the wave
    const int32_t xa = G.np_off[x], d = G.np_off[x + 1] - xa;
    if (d < 2) return;
    if (d > kTriD) {
      if (lane == 0) big[atomicAdd(&queue[kNTriBig], 1)] = x;
      return;
    }
    // member `lane` of N+(x): entry, hash slot, row
    uint32_t e = 0, hs = 0;
    int32_t ra = 0, len = 0;
    uint4 dy = make_uint4(0, 0, 0, 0);
    if (lane < d) {
      e = G.np_idx[xa + lane];
      const uint32_t y = e & kIdMask;
      list[lane] = e;
      hs = hash_mul(y, kTriHB);
      while (atomicCAS(&key[hs], kNone, y) != kNone) hs = (hs + 1) & (kTriH - 1);
      at[hs] = (uint8_t)lane;
      ra = G.np_off[y];
      len = G.np_off[y + 1] - ra;
      if (K4) dy = G.dt[y];
    }
    const uint4 dx = K4 ? G.dt[x] : make_uint4(0, 0, 0, 0);
    wave_sync();
    const int32_t sub = lane >> 4, l16 = lane & 15;
    for (int32_t j0 = 0; j0 < d; j0 += 4) {
      const int32_t j = j0 + sub;
      const int32_t a = __shfl(ra, j), mj = __shfl(len, j), m = j < d ? mj : 0;
      for (int32_t t = l16; t < m; t += 16) {
        const uint32_t f = G.np_idx[a + t], z = f & kIdMask;
        uint32_t h = hash_mul(z, kTriHB), kk;
        while ((kk = key[h]) != z && kk != kNone) h = (h + 1) & (kTriH - 1);
        if (kk != z) continue;
        const int32_t k = at[h];
        const uint32_t ey = list[j], ez = list[k];
        const uint32_t xy = ey >> kTypeShift, xz = ez >> kTypeShift, yz = f >> kTypeShift;
        const uint32_t tau = (xy - 1) * 9 + (xz - 1) * 3 + (yz - 1);
        if constexpr (K4) {
          tri_add<true>(bins, tau, dx, G.dt[ey & kIdMask], G.dt[z]);
          atomicAdd(&Tl[j], 1ull << (7 * ((xz - 1) * 3 + (yz - 1))));
          atomicAdd(&Tl[k], 1ull << (7 * ((xy - 1) * 3 + (flip(yz) - 1))));
          atomicAdd(&T[(int64_t)(a + t) * 9 + (flip(xy) - 1) * 3 + (flip(xz) - 1)], 1u);
          if (yz & 1u) atomicOr(&A1[j], 1ull << k);
          if (yz & 2u) atomicOr(&A2[j], 1ull << k);
        } else {
          atomicAdd(&bins.tri[tau], 1ull);
        }
      }
    }
    wave_sync();
    if constexpr (K4) {
      if (lane < d) {
        const u64 p1 = A1[lane], p2 = A2[lane];
        const uint32_t bx = edge_code<4>(0, 1, e >> kTypeShift);
        for (u64 r = p1 | p2; r; r &= r - 1ull) {  // edge lane -> k above x
          const int k = __builtin_ctzll(r);
          const u64 q1 = A1[k], q2 = A2[k];
          u64 com = (p1 | p2) & (q1 | q2);
          if (!com) continue;
          const uint32_t bk = bx | edge_code<4>(0, 2, list[k] >> kTypeShift) |
                              edge_code<4>(1, 2, (uint32_t)((p1 >> k) & 1) | (uint32_t)((p2 >> k) & 1) << 1);
          for (; com; com &= com - 1ull) {
            const int l = __builtin_ctzll(com);
            const uint32_t code = bk | edge_code<4>(0, 3, list[l] >> kTypeShift) |
                                  edge_code<4>(1, 3, (uint32_t)((p1 >> l) & 1) | (uint32_t)((p2 >> l) & 1) << 1) |
                                  edge_code<4>(2, 3, (uint32_t)((q1 >> l) & 1) | (uint32_t)((q2 >> l) & 1) << 1);
            atomicAdd(&bins.kh[lut[code]], 1ull);
          }
        }
        const u64 c = Tl[lane];
        if (c)
          for (int i = 0; i < 9; ++i) {
            const uint32_t v = (uint32_t)(c >> (7 * i)) & 127u;
            if (v) atomicAdd(&T[(int64_t)(xa + lane) * 9 + i], v);
          }
      }
      wave_sync();
      if (lane < d) {
        Tl[lane] = 0;
        A1[lane] = 0;
        A2[lane] = 0;
      }
    }
    if (lane < d) key[hs] = kNone;
    wave_sync();
  };

  if (!G.gid) {
    for (;;) {
      int32_t v0 = 0;
      if (lane == 0) v0 = atomicAdd(&queue[kQTri], chunk);
      v0 = __shfl(v0, 0);
      if (v0 >= n) break;
      const int32_t v1 = min(n, v0 + chunk);
      for (int32_t x = v0; x < v1; ++x) one(x);
    }
    __syncthreads();
    bins.flush(0, lut3, K4 ? lut : lut4, a3, a4, threadIdx.x, 256);
    return;
  }
  int32_t cur = -1;
  for (;;) {
    __syncthreads();
    if (threadIdx.x == 0) sh_v = atomicAdd(&queue[kQTri], kBatchChunk);
    __syncthreads();
    const int32_t v0 = sh_v;
    if (v0 >= n) break;
    const int32_t v1 = min(n, v0 + kBatchChunk);
    for (int32_t a = v0; a < v1;) {
      const int32_t g = G.gid[a];
      const int32_t b = (int32_t)min((int64_t)v1, G.voff[g + 1]);
      if (g != cur) {
        __syncthreads();
        if (cur >= 0) bins.flush(cur, lut3, K4 ? lut : lut4, a3, a4, threadIdx.x, 256);
        __syncthreads();
        bins.clear(threadIdx.x, 256);
        __syncthreads();
        cur = g;
      }
      for (int32_t x = a + wv; x < b; x += NW) one(x);
      a = b;
    }
  }
  if (cur >= 0) bins.flush(cur, lut3, K4 ? lut : lut4, a3, a4, threadIdx.x, 256);
}

// The x with more than kTriD higher neighbours, one workgroup each: N+(x) in
// an LDS hash of up to kBigH / 2 members (beyond that a binary search in the
// id-sorted row), T by global atomics, and for k = 4 the two adjacency bit
// planes of N+(x) in the workgroup's slice of global memory (2 D rows of
// `words` words, D >= any d+).  d+ is at most sqrt(2 m), so a slice is a few
// hundred KB on 10^6 arcs; few x are here on sparse graphs (553 of 96,632 on
// the n = 10^5 graph).
constexpr int kBigHB = 13;
constexpr int kBigH = 1 << kBigHB;

template <bool K4>
__global__ __launch_bounds__(512) void k_tri_big(DevGraph G, const uint16_t* __restrict__ lut3,
                                                 const uint16_t* __restrict__ lut4, uint64_t* __restrict__ a3,
                                                 uint64_t* __restrict__ a4, uint32_t* __restrict__ T,
                                                 const int32_t* st, int32_t* __restrict__ queue,
                                                 const int32_t* __restrict__ big, u64* __restrict__ planes, int64_t D,
                                                 int64_t words) {
  constexpr int NT = 512, NW = NT / 64;
  __shared__ u64 s_tri[27], s_paw[K4 ? 243 : 1], s_kh[K4 ? 199 : 1];
  __shared__ uint32_t key[kBigH];
  __shared__ uint16_t at[kBigH];
  __shared__ int32_t sh_i;
  if (st[kStatus] != 0) return;
  const int32_t nbig = queue[kNTriBig];
  if (nbig == 0) return;
  const TriBins<K4> bins{s_tri, s_paw, s_kh};
  bins.clear(threadIdx.x, NT);
  for (int i = threadIdx.x; i < kBigH; i += NT) key[i] = kNone;
  u64* P1 = K4 ? planes + (int64_t)blockIdx.x * 2 * D * words : nullptr;
  u64* P2 = K4 ? P1 + D * words : nullptr;
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int32_t cur = -1;
  for (;;) {
    __syncthreads();
    if (threadIdx.x == 0) sh_i = atomicAdd(&queue[kQTriBig], 1);
    __syncthreads();
    if (sh_i >= nbig) break;
    const int32_t x = big[sh_i];
    const int32_t g = G.gid ? G.gid[x] : 0;
    if (g != cur) {
      if (cur >= 0) bins.flush(cur, lut3, lut4, a3, a4, threadIdx.x, NT);
      __syncthreads();
      bins.clear(threadIdx.x, NT);
      cur = g;
    }
    const int32_t xa = G.np_off[x], d = G.np_off[x + 1] - xa;
    const int32_t W = (d + 63) / 64;  // <= words: d <= D
    const bool hashed = d <= kBigH / 2;
    if (hashed)
      for (int32_t i = threadIdx.x; i < d; i += NT) {
        const uint32_t y = G.np_idx[xa + i] & kIdMask;
        uint32_t h = hash_mul(y, kBigHB);
        while (atomicCAS(&key[h], kNone, y) != kNone) h = (h + 1) & (kBigH - 1);
        at[h] = (uint16_t)i;
      }
    if (K4)
      for (int64_t i = threadIdx.x; i < (int64_t)d * W; i += NT) {
        __hip_atomic_store(&P1[i], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&P2[i], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    const uint4 dx = K4 ? G.dt[x] : make_uint4(0, 0, 0, 0);
    for (int32_t j = wv; j < d; j += NW) {
      const uint32_t ey = G.np_idx[xa + j], y = ey & kIdMask, xy = ey >> kTypeShift;
      const int32_t ra = G.np_off[y], rb = G.np_off[y + 1];
      const uint4 dy = K4 ? G.dt[y] : make_uint4(0, 0, 0, 0);
      for (int32_t t = ra + lane; t < rb; t += 64) {
        const uint32_t f = G.np_idx[t], z = f & kIdMask;
        int32_t k = -1;
        if (hashed) {
          uint32_t h = hash_mul(z, kBigHB), kk;
          while ((kk = key[h]) != z && kk != kNone) h = (h + 1) & (kBigH - 1);
          if (kk == z) k = at[h];
        } else {
          int32_t lo = 0, hi = d;
          while (lo < hi) {
            const int32_t mid = (lo + hi) >> 1;
            if ((G.np_idx[xa + mid] & kIdMask) < z) lo = mid + 1; else hi = mid;
          }
          if (lo < d && (G.np_idx[xa + lo] & kIdMask) == z) k = lo;
        }
        if (k < 0) continue;
        const uint32_t xz = G.np_idx[xa + k] >> kTypeShift, yz = f >> kTypeShift;
        const uint32_t tau = (xy - 1) * 9 + (xz - 1) * 3 + (yz - 1);
        if constexpr (K4) {
          tri_add<true>(bins, tau, dx, dy, G.dt[z]);
          atomicAdd(&T[(int64_t)(xa + j) * 9 + (xz - 1) * 3 + (yz - 1)], 1u);
          atomicAdd(&T[(int64_t)(xa + k) * 9 + (xy - 1) * 3 + (flip(yz) - 1)], 1u);
          atomicAdd(&T[(int64_t)t * 9 + (flip(xy) - 1) * 3 + (flip(xz) - 1)], 1u);
          const int64_t w = (int64_t)j * W + (k >> 6);
          if (yz & 1u) atomicOr(&P1[w], 1ull << (k & 63));
          if (yz & 2u) atomicOr(&P2[w], 1ull << (k & 63));
        } else {
          atomicAdd(&bins.tri[tau], 1ull);
        }
      }
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if constexpr (K4) {
      auto word = [&](const u64* p, int64_t i) {  // set by atomics in L2
        return __hip_atomic_load(p + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      };
      for (int32_t j = wv; j < d; j += NW) {
        const uint32_t bx = edge_code<4>(0, 1, G.np_idx[xa + j] >> kTypeShift);
        for (int32_t kw = 0; kw < W; ++kw) {
          const u64 p1 = word(P1, (int64_t)j * W + kw), p2 = word(P2, (int64_t)j * W + kw);
          for (u64 r = p1 | p2; r; r &= r - 1ull) {  // the same on every lane
            const int b = __builtin_ctzll(r);
            const int32_t k = kw * 64 + b;
            const uint32_t bk = bx | edge_code<4>(0, 2, G.np_idx[xa + k] >> kTypeShift) |
                                edge_code<4>(1, 2, (uint32_t)((p1 >> b) & 1) | (uint32_t)((p2 >> b) & 1) << 1);
            for (int32_t lw = lane; lw < W; lw += 64) {
              const u64 r1 = word(P1, (int64_t)j * W + lw), r2 = word(P2, (int64_t)j * W + lw);
              const u64 q1 = word(P1, (int64_t)k * W + lw), q2 = word(P2, (int64_t)k * W + lw);
              for (u64 com = (r1 | r2) & (q1 | q2); com; com &= com - 1ull) {
                const int l = __builtin_ctzll(com);
                const uint32_t code = bk | edge_code<4>(0, 3, G.np_idx[xa + lw * 64 + l] >> kTypeShift) |
                                      edge_code<4>(1, 3, (uint32_t)((r1 >> l) & 1) | (uint32_t)((r2 >> l) & 1) << 1) |
                                      edge_code<4>(2, 3, (uint32_t)((q1 >> l) & 1) | (uint32_t)((q2 >> l) & 1) << 1);
                atomicAdd(&bins.kh[lut4[code]], 1ull);
              }
            }
          }
        }
      }
      __syncthreads();
    }
    if (hashed)
      for (int i = threadIdx.x; i < kBigH; i += NT) key[i] = kNone;
  }
  __syncthreads();
  if (cur >= 0) bins.flush(cur, lut3, lut4, a3, a4, threadIdx.x, NT);
}

// ================================================================ wedges ==
//
// C4s, each from its vertex u of highest rank: W[w][3 p + q] = wedges u - v -
// w with v of lower rank than u, p and q (less one) the types of v seen from u
// and of w seen from v.  Two wedges to the same w of lower rank are a C4
// u - v - w - v'.  A count is at most min(d-(u), d(w)), which bounds the width
// of its field: nine fields of 7 bits share one 64-bit word while d-(u) <= 127.
//   k_wedge<64, 8>    one wave per u with at most 192 visits (a hash of w)
//   k_wedge<256, 12>  one workgroup per u with at most 3,072 visits
//   k_wedge_top       the rest: a direct table over one block of vertex ids at
//                     a time, the work unit being (u, block)
__device__ __forceinline__ bool ranked_below(const DevGraph& G, uint32_t dw, int32_t w, uint32_t du, int32_t u) {
  return dw < du || (dw == du && w < u);
}

// Pairs of wedges to one w, by the types of both, into bins[9 i + j], i <= j.
__device__ __forceinline__ void c4_pairs(const uint32_t (&c)[9], u64* bins) {
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    if (!c[i]) continue;
#pragma unroll
    for (int j = i; j < 9; ++j) {
      const u64 w = j == i ? (u64)c[i] * (c[i] - 1u) / 2u : (u64)c[i] * c[j];
      if (w) atomicAdd(&bins[9 * i + j], w);
    }
  }
}

__device__ __forceinline__ void c4_flush(const u64* bins, const uint16_t* lut4, uint64_t* a, int t, int nt) {
  // slots u = 0, w = 1, the two middle vertices 2 and 3
  for (int k = t; k < 81; k += nt) {
    const int i = k / 9, j = k % 9;
    if (i > j || !bins[k]) continue;
    const uint32_t pi = (uint32_t)i / 3 + 1, qi = (uint32_t)i % 3 + 1, pj = (uint32_t)j / 3 + 1, qj = (uint32_t)j % 3 + 1;
    gadd(&a[lut4[edge_code<4>(0, 2, pi) | edge_code<4>(2, 1, qi) | edge_code<4>(0, 3, pj) | edge_code<4>(3, 1, qj)]],
         bins[k]);
  }
}

constexpr int kMidVisits = 3072;

// NT threads per u, a hash of 2^HB slots (at most 3/4 full).  NT = 64: every
// vertex, those with more visits go to `mid`; NT = 256: the vertices of `mid`.
template <int NT, int HB>
__global__ __launch_bounds__(256) void k_wedge(DevGraph G, const uint16_t* __restrict__ lut4,
                                               uint64_t* __restrict__ a4, const int32_t* st,
                                               int32_t* __restrict__ queue, int32_t chunk, int32_t* __restrict__ mid,
                                               int32_t* __restrict__ top) {
  constexpr int NU = 256 / NT, H = 1 << HB;
  constexpr bool WAVE = NT == 64;
  constexpr int kCap = WAVE ? 192 : kMidVisits;
  static_assert(kCap <= H * 3 / 4, "hash load");
  __shared__ uint32_t s_key[NU][H];
  __shared__ u64 s_cnt[NU][H];
  __shared__ u64 bins[81];
  __shared__ int32_t sh_v;
  if (st[kStatus] != 0) return;
  const int un = threadIdx.x / NT, t = threadIdx.x % NT, lane = threadIdx.x & 63;
  uint32_t* key = s_key[un];
  u64* cnt = s_cnt[un];
  for (int i = t; i < H; i += NT) {
    key[i] = kNone;
    cnt[i] = 0;
  }
  for (int i = threadIdx.x; i < 81; i += 256) bins[i] = 0;
  __syncthreads();
  auto sync = [] {
    if constexpr (WAVE) wave_sync();
    else __syncthreads();
  };
  auto one = [&](int32_t u) {  // uniform over the NT threads
    const int32_t ma = G.gs_off[u] - G.np_off[u];
    const int32_t dm = G.gs_off[u + 1] - G.np_off[u + 1] - ma;
    if (dm < 2) return;
    if constexpr (WAVE) {
      int32_t vis = kMidVisits + 1;
      if (dm <= 127) {
        vis = 0;
        for (int32_t i = lane; i < dm; i += 64) {
          const uint32_t v = G.nm_idx[ma + i] & kIdMask;
          vis += min(G.gs_off[v + 1] - G.gs_off[v], kMidVisits + 1);
        }
#pragma unroll
        for (int o = 32; o; o >>= 1) vis += __shfl_xor(vis, o);
      }
      if (vis > kCap) {
        if (lane == 0) {
          if (vis <= kMidVisits) mid[atomicAdd(&queue[kNWedgeMid], 1)] = u;
          else top[atomicAdd(&queue[kNWedgeTop], 1)] = u;
        }
        return;
      }
    }
    for (int32_t i = t >> 3; i < dm; i += NT / 8) {  // eight lanes per row
      const uint32_t ev = G.nm_idx[ma + i], v = ev & kIdMask;
      const int32_t ra = G.gs_off[v], rb = G.gs_off[v + 1];
      const int p7 = 21 * (int)((ev >> kTypeShift) - 1u);
      for (int32_t r = ra + (t & 7); r < rb; r += 8) {
        const uint32_t f = G.gs_idx[r], w = f & kIdMask;
        if ((int32_t)w == u) continue;
        uint32_t h = hash_mul(w, HB);
        for (;;) {
          const uint32_t old = atomicCAS(&key[h], kNone, w);
          if (old == kNone || old == w) break;
          h = (h + 1) & (H - 1);
        }
        atomicAdd(&cnt[h], 1ull << (p7 + 7 * (int)((f >> kTypeShift) - 1u)));
      }
    }
    sync();
    const uint32_t du = (uint32_t)(G.gs_off[u + 1] - G.gs_off[u]);
    for (int i = t; i < H; i += NT) {
      const u64 c = cnt[i];
      if (!c) continue;
      cnt[i] = 0;
      const uint32_t w = key[i];
      key[i] = kNone;
      // a single wedge: one field, equal to one
      constexpr u64 kOnes = 1ull | 1ull << 7 | 1ull << 14 | 1ull << 21 | 1ull << 28 | 1ull << 35 | 1ull << 42 |
                            1ull << 49 | 1ull << 56;
      if ((c & (c - 1ull)) == 0 && (c & kOnes)) continue;
      if (!ranked_below(G, (uint32_t)(G.gs_off[w + 1] - G.gs_off[w]), (int32_t)w, du, u)) continue;
      uint32_t f[9];
#pragma unroll
      for (int k = 0; k < 9; ++k) f[k] = (uint32_t)(c >> (7 * k)) & 127u;
      c4_pairs(f, bins);
    }
    sync();
  };
  const int32_t n = G.n;
  if constexpr (!WAVE) {
    const int32_t nmid = queue[kNWedgeMid];
    int32_t cur = -1;
    for (;;) {
      if (threadIdx.x == 0) sh_v = atomicAdd(&queue[kQWedgeMid], 1);
      __syncthreads();
      const int32_t i = sh_v;
      __syncthreads();
      if (i >= nmid) break;
      const int32_t u = mid[i], g = G.gid ? G.gid[u] : 0;
      if (g != cur) {
        if (cur >= 0) c4_flush(bins, lut4, a4 + (int64_t)cur * 199, threadIdx.x, 256);
        __syncthreads();
        if (threadIdx.x < 81) bins[threadIdx.x] = 0;
        __syncthreads();
        cur = g;
      }
      one(u);
    }
    if (cur >= 0) c4_flush(bins, lut4, a4 + (int64_t)cur * 199, threadIdx.x, 256);
  } else if (!G.gid) {
    for (;;) {
      int32_t v0 = 0;
      if (lane == 0) v0 = atomicAdd(&queue[kQWedge], chunk);
      v0 = __shfl(v0, 0);
      if (v0 >= n) break;
      const int32_t v1 = min(n, v0 + chunk);
      for (int32_t u = v0; u < v1; ++u) one(u);
    }
    __syncthreads();
    c4_flush(bins, lut4, a4, threadIdx.x, 256);
  } else {
    int32_t cur = -1;
    for (;;) {
      __syncthreads();
      if (threadIdx.x == 0) sh_v = atomicAdd(&queue[kQWedge], kBatchChunk);
      __syncthreads();
      const int32_t v0 = sh_v;
      if (v0 >= n) break;
      const int32_t v1 = min(n, v0 + kBatchChunk);
      for (int32_t a = v0; a < v1;) {
        const int32_t g = G.gid[a];
        const int32_t b = (int32_t)min((int64_t)v1, G.voff[g + 1]);
        if (g != cur) {
          __syncthreads();
          if (cur >= 0) c4_flush(bins, lut4, a4 + (int64_t)cur * 199, threadIdx.x, 256);
          __syncthreads();
          if (threadIdx.x < 81) bins[threadIdx.x] = 0;
          __syncthreads();
          cur = g;
        }
        for (int32_t u = a + un; u < b; u += NU) one(u);
        a = b;
      }
    }
    if (cur >= 0) c4_flush(bins, lut4, a4 + (int64_t)cur * 199, threadIdx.x, 256);
  }
}

// Vertex u of many visits: (u, block of w) is a work unit of one workgroup.
// The wedge counts of the block's vertices sit in a direct LDS table, the
// widest block that the bound of u allows: nine 7-bit fields in 8 bytes for
// d-(u) <= 127, 3 x three 10-bit fields in 12 for d-(u) <= 1,023, else 3 x
// three 21-bit fields in 24 (WIDE, for graphs with degrees of 2^21 and more:
// nine words of 36 bytes).  split holds the start of every granule of ids in
// every row, so a unit reads just its part of each row N(v) (null: binary
// search).  Parts of more than kLongPart entries are listed and taken by whole
// waves, the others by eight lanes.
constexpr int kTopTable = 147456;  // bytes: 6,144 vertices of 24 bytes, 4,096 of 36
constexpr int kLongPart = 64;
constexpr int kLongCap = 128;
constexpr int kTopThreads = 1024;

template <bool WIDE>
constexpr int top_granule() { return WIDE ? 4096 : 6144; }

template <bool WIDE>
__global__ __launch_bounds__(kTopThreads) void k_wedge_top(DevGraph G, const uint16_t* __restrict__ lut4,
                                                           uint64_t* __restrict__ a4, const int32_t* st,
                                                           int32_t* __restrict__ queue,
                                                           const int32_t* __restrict__ top,
                                                           const int32_t* __restrict__ split, int32_t ngran) {
  constexpr int NT = kTopThreads, GR = top_granule<WIDE>();
  constexpr int kMaxBlock = WIDE ? 4096 : 18432;
  __shared__ __align__(16) uint32_t tab[kTopTable / 4];
  __shared__ u64 bins[81];
  __shared__ int32_t l_a[kLongCap], l_b[kLongCap], l_p[kLongCap], nlong;
  __shared__ u64 sh_i;
  __shared__ uint16_t act[4096];  // vertices with two wedges or more
  __shared__ int32_t nact;
  if (st[kStatus] != 0) return;
  const int32_t ntop = queue[kNWedgeTop];
  if (ntop == 0) return;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int i = threadIdx.x; i < 81; i += NT) bins[i] = 0;
  u64* const t64 = reinterpret_cast<u64*>(tab);
  const int64_t units = (int64_t)ntop * ngran;
  int32_t cur = -1;
  for (;;) {
    __syncthreads();
    if (threadIdx.x == 0) {
      sh_i = atomicAdd(reinterpret_cast<u64*>(&queue[kQWedgeTop]), 1ull);  // two words: units may pass 2^31
      nlong = 0;
      nact = 0;
    }
    __syncthreads();
    const int64_t unit = (int64_t)sh_i;
    if (unit >= units) break;
    const int32_t u = top[unit / ngran];
    const int32_t g = G.gid ? G.gid[u] : 0;
    const int32_t base = G.voff ? (int32_t)G.voff[g] : 0;
    const int32_t ng = G.voff ? (int32_t)(G.voff[g + 1] - G.voff[g]) : G.n;
    const int32_t ma = G.gs_off[u] - G.np_off[u];
    const int32_t dm = G.gs_off[u + 1] - G.np_off[u + 1] - ma;
    // format: 0 = 8 bytes, 1 = 12, 2 = 24, 3 = 36; granules per block
    const int fmt = WIDE ? 3 : dm <= 127 ? 0 : dm <= 1023 ? 1 : 2;
    const int32_t per = WIDE ? 1 : fmt == 0 ? 3 : fmt == 1 ? 2 : 1;
    const int32_t blk = (int32_t)(unit % ngran);
    const int32_t g0 = blk * per;                 // first granule
    if ((int64_t)g0 * GR >= ng) continue;         // uniform over the workgroup
    const int32_t g1 = min(g0 + per, (ng + GR - 1) / GR);
    const int32_t w0 = base + g0 * GR, w1 = min(base + ng, base + g1 * GR);
    const int32_t nw = w1 - w0;                   // <= kMaxBlock
    const int32_t BS = per * GR;                  // table stride of the formats with three or nine arrays
    if (g != cur) {
      if (cur >= 0) c4_flush(bins, lut4, a4 + (int64_t)cur * 199, threadIdx.x, NT);
      __syncthreads();
      for (int i = threadIdx.x; i < 81; i += NT) bins[i] = 0;
      cur = g;
    }
    for (int i = threadIdx.x; i < kTopTable / 16; i += NT) reinterpret_cast<uint4*>(tab)[i] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    auto add = [&](uint32_t p, uint32_t f) {  // p, type less one
      const int32_t w = (int32_t)(f & kIdMask) - w0;
      const uint32_t q = (f >> kTypeShift) - 1u;
      if (fmt == 0) atomicAdd(&t64[w], 1ull << (21 * p + 7 * q));
      else if (fmt == 1) atomicAdd(&tab[p * BS + w], 1u << (10 * q));
      else if (fmt == 2) atomicAdd(&t64[p * BS + w], 1ull << (21 * q));
      else atomicAdd(&tab[(3 * p + q) * BS + w], 1u);
    };
    for (int32_t i = threadIdx.x >> 3; i < dm; i += NT / 8) {
      const uint32_t ev = G.nm_idx[ma + i], p = (ev >> kTypeShift) - 1u;
      const int32_t v = (int32_t)(ev & kIdMask);
      int32_t a, b;
      if (split) {
        const int32_t* sp = split + (int64_t)v * (ngran + 1);
        a = sp[g0];
        b = sp[g1];
      } else {
        auto first = [&](int32_t id) {
          int32_t lo = G.gs_off[v], hi = G.gs_off[v + 1];
          while (lo < hi) {
            const int32_t mid = (lo + hi) >> 1;
            if ((int32_t)(G.gs_idx[mid] & kIdMask) < id) lo = mid + 1; else hi = mid;
          }
          return lo;
        };
        a = first(w0);
        b = first(w1);
      }
      if (b - a > kLongPart) {
        int32_t s = kLongCap;
        if ((threadIdx.x & 7) == 0) s = atomicAdd(&nlong, 1);
        s = __shfl(s, lane & 56);
        if (s < kLongCap) {
          if ((threadIdx.x & 7) == 0) {
            l_a[s] = a;
            l_b[s] = b;
            l_p[s] = (int32_t)p;
          }
          continue;
        }
      }
      for (int32_t r = a + (threadIdx.x & 7); r < b; r += 8) add(p, G.gs_idx[r]);
    }
    __syncthreads();
    const int32_t nl = min(nlong, kLongCap);
    for (int32_t i = wv; i < nl; i += NT / 64) {
      const int32_t b = l_b[i];
      const uint32_t p = (uint32_t)l_p[i];
      for (int32_t r = l_a[i] + lane; r < b; r += 64) add(p, G.gs_idx[r]);
    }
    __syncthreads();
    // u itself is in every row N(v): its counts are no wedges
    const uint32_t du = (uint32_t)(G.gs_off[u + 1] - G.gs_off[u]);
    auto fields = [&](int32_t w, uint32_t (&c)[9]) {
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        const int p = k / 3, q = k % 3;
        c[k] = fmt == 0 ? (uint32_t)(t64[w] >> (7 * k)) & 127u
             : fmt == 1 ? (tab[p * BS + w] >> (10 * q)) & 1023u
             : fmt == 2 ? (uint32_t)(t64[p * BS + w] >> (21 * q)) & 0x1FFFFFu
                        : tab[k * BS + w];
      }
    };
    auto many = [&](int32_t w) {  // two wedges or more
      uint32_t c[9], s = 0;
      fields(w, c);
#pragma unroll
      for (int k = 0; k < 9; ++k) s |= c[k] > 1u ? 2u : s ? (c[k] ? 2u : 0u) : c[k];
      return s >= 2u;
    };
    // the vertices that count are listed first: few of a block do, and the
    // pair loop then runs on full waves
    for (int32_t b0 = 0; b0 < nw; b0 += 4096) {
      for (int32_t w = b0 + (int32_t)threadIdx.x; w < min(nw, b0 + 4096); w += NT) {
        if (!many(w)) continue;
        const int32_t id = w0 + w;
        if (id == u || !ranked_below(G, (uint32_t)(G.gs_off[id + 1] - G.gs_off[id]), id, du, u)) continue;
        act[atomicAdd(&nact, 1)] = (uint16_t)w;
      }
      __syncthreads();
      const int32_t na = nact;
      for (int32_t i = threadIdx.x; i < na; i += NT) {
        uint32_t c[9];
        fields((int32_t)act[i], c);
        c4_pairs(c, bins);
      }
      __syncthreads();
      if (threadIdx.x == 0) nact = 0;
      __syncthreads();
    }
  }
  __syncthreads();
  if (cur >= 0) c4_flush(bins, lut4, a4 + (int64_t)cur * 199, threadIdx.x, NT);
}

// split[v * (ngran + 1) + i] = first entry of row v with id >= the start of
// granule i of its graph (i = ngran: the row's end).
__global__ void k_split(DevGraph G, int32_t gran, int32_t ngran, int32_t* __restrict__ split, const int32_t* st) {
  if (st[kStatus] != 0) return;
  const int64_t cols = ngran + 1, total = (int64_t)G.n * cols;
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < total; k += (int64_t)gridDim.x * blockDim.x) {
    const int32_t v = (int32_t)(k / cols), i = (int32_t)(k % cols);
    const int64_t id = (G.voff ? G.voff[G.gid[v]] : 0) + (int64_t)i * gran;
    int32_t lo = G.gs_off[v], hi = G.gs_off[v + 1];
    if (i == ngran) {
      lo = hi;
    } else {
      while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        if ((int64_t)(G.gs_idx[mid] & kIdMask) < id) lo = mid + 1; else hi = mid;
      }
    }
    split[k] = lo;
  }
}

// ==================================================== vertices and edges ==
//
// Wedges and claws from the typed degrees of each vertex; P4s from those of
// each edge's ends (the paths whose two ends coincide are taken off with the
// triangles); diamonds from each edge's typed triangle counts.
template <bool K3, bool K4>
__global__ __launch_bounds__(256) void k_local(DevGraph G, const uint16_t* __restrict__ lut3,
                                               const uint16_t* __restrict__ lut4, uint64_t* __restrict__ a3,
                                               uint64_t* __restrict__ a4, const uint32_t* __restrict__ T,
                                               const int32_t* st, int32_t* __restrict__ queue, int32_t chunk) {
  __shared__ u64 w3[6], w4[10], p4[27], h4[K4 ? 199 : 1];
  __shared__ uint16_t lut[K4 ? 4096 : 1];
  __shared__ int32_t sh_v;
  if (st[kStatus] != 0) return;
  const int nt = 256;
  auto clear = [&] {
    for (int i = threadIdx.x; i < 27; i += nt) {
      p4[i] = 0;
      if (i < 6) w3[i] = 0;
      if (i < 10) w4[i] = 0;
    }
    if (K4)
      for (int i = threadIdx.x; i < 199; i += nt) h4[i] = 0;
  };
  clear();
  if (K4)
    for (int i = threadIdx.x; i < 4096; i += nt) lut[i] = lut4[i];
  __syncthreads();
  auto flush = [&](int32_t g) {
    if (K3 && threadIdx.x < 6) {
      // pairs (a, b), a <= b, row-major
      const int i = threadIdx.x, a = i < 3 ? 1 : i < 5 ? 2 : 3, b = i < 3 ? i + 1 : i < 5 ? i - 1 : 3;
      gadd(&a3[(int64_t)g * 13 + lut3[edge_code<3>(0, 1, a) | edge_code<3>(0, 2, b)]], w3[i]);
    }
    if constexpr (K4) {
      uint64_t* A = a4 + (int64_t)g * 199;
      if (threadIdx.x < 10) {
        int k = threadIdx.x, a = 1, b = 1, c = 1;
        for (; k; --k) {  // the k-th triple a <= b <= c
          if (c < 3) ++c;
          else if (b < 3) c = ++b;
          else a = b = c = a + 1;
        }
        gadd(&A[lut[edge_code<4>(0, 1, a) | edge_code<4>(0, 2, b) | edge_code<4>(0, 3, c)]], w4[threadIdx.x]);
      }
      for (int i = threadIdx.x; i < 27; i += nt)
        gadd(&A[lut[edge_code<4>(0, 1, i / 9 + 1) | edge_code<4>(0, 2, (i / 3) % 3 + 1) |
                    edge_code<4>(1, 3, i % 3 + 1)]], p4[i]);
      for (int i = threadIdx.x; i < 199; i += nt) gadd(&A[i], h4[i]);
    }
  };
  auto vertex = [&](int32_t v) {
    const uint4 D = G.dt[v];
    const u64 d[4] = {0, D.x, D.y, D.z};
    if constexpr (K3) {
      int k = 0;
#pragma unroll
      for (int a = 1; a <= 3; ++a)
#pragma unroll
        for (int b = a; b <= 3; ++b, ++k) {
          const u64 w = a == b ? d[a] * (d[a] - (d[a] > 0)) / 2 : d[a] * d[b];
          if (w) atomicAdd(&w3[k], w);
        }
    }
    if constexpr (K4) {
      auto c2 = [](u64 x) { return x * (x - (x > 0)) / 2; };
      auto c3 = [](u64 x) {  // x (x - 1) (x - 2) / 6, x < 2^30: the division comes before the last product
        if (x < 3) return (u64)0;
        const u64 y = x * (x - 1) / 2;
        return y % 3 == 0 ? y / 3 * (x - 2) : y * ((x - 2) / 3);
      };
      int k = 0;
#pragma unroll
      for (int a = 1; a <= 3; ++a)
#pragma unroll
        for (int b = a; b <= 3; ++b)
#pragma unroll
          for (int c = b; c <= 3; ++c, ++k) {
            const u64 w = a == b && b == c ? c3(d[a]) : a == b ? c2(d[a]) * d[c] : b == c ? d[a] * c2(d[b])
                                                                                         : d[a] * d[b] * d[c];
            if (w) atomicAdd(&w4[k], w);
          }
    }
  };
  auto edge = [&](int64_t e) {
    const uint32_t f = G.np_idx[e], t = f >> kTypeShift, tf = flip(t);
    const uint4 X = G.dt[G.np_row[e]], Y = G.dt[f & kIdMask];
#pragma unroll
    for (uint32_t p = 1; p <= 3; ++p) {
      const u64 dx = typ(X, p) - (p == t);
#pragma unroll
      for (uint32_t q = 1; q <= 3; ++q) {
        const u64 w = dx * (u64)(typ(Y, q) - (q == tf));
        if (w) atomicAdd(&p4[(t - 1) * 9 + (p - 1) * 3 + (q - 1)], w);
      }
    }
    uint32_t c[9], s = 0;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      c[i] = T[e * 9 + i];
      s += c[i];
    }
    if (s < 2) return;
    const uint32_t base = edge_code<4>(0, 1, t);
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      if (!c[i]) continue;
      const uint32_t ci = base | edge_code<4>(0, 2, i / 3 + 1) | edge_code<4>(1, 2, i % 3 + 1);
#pragma unroll
      for (int j = i; j < 9; ++j) {
        const u64 w = j == i ? (u64)c[i] * (c[i] - 1u) / 2u : (u64)c[i] * c[j];
        if (w) atomicAdd(&h4[lut[ci | edge_code<4>(0, 3, j / 3 + 1) | edge_code<4>(1, 3, j % 3 + 1)]], w);
      }
    }
  };
  const int32_t n = G.n;
  const int64_t items = (int64_t)n + (K4 ? G.np_off[n] : 0);
  int32_t cur = G.gid ? -1 : 0;
  for (;;) {
    __syncthreads();
    if (threadIdx.x == 0) sh_v = atomicAdd(&queue[kQEdges], 1);
    __syncthreads();
    const int64_t i0 = (int64_t)sh_v * chunk;
    if (i0 >= items) break;
    const int64_t i1 = min(items, i0 + chunk);
    for (int64_t a = i0; a < i1;) {
      int64_t b = i1;
      if (a < n && b > n) b = n;
      if (G.gid) {  // up to the end of the graph
        const int32_t g = G.gid[a < n ? a : (int64_t)G.np_row[a - n]];
        const int64_t end = a < n ? G.voff[g + 1] : (int64_t)n + G.np_off[G.voff[g + 1]];
        b = min(b, end);
        if (g != cur) {
          __syncthreads();
          if (cur >= 0) flush(cur);
          __syncthreads();
          clear();
          __syncthreads();
          cur = g;
        }
      }
      for (int64_t i = a + threadIdx.x; i < b; i += nt) {
        if (i < n) vertex((int32_t)i);
        else if constexpr (K4) edge(i - n);
      }
      a = b;
    }
  }
  __syncthreads();
  if (cur >= 0) flush(cur);
}

// ================================================================= solve ==
// out[c] = sum of coef * N over row c of the inverse (in CSR form), one
// workgroup per graph and block of classes.  A negative count is a failed
// self-check; nothing is written by k_solve_write then.
__global__ __launch_bounds__(256) void k_solve(const uint64_t* __restrict__ acc, const SubInverse M,
                                               uint64_t* __restrict__ out, int32_t C, int64_t total, int32_t* st) {
  if (st[kStatus] != 0) return;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    const int32_t c = (int32_t)(i % C);
    const uint64_t* a = acc + (i - c);
    int64_t s = 0;
    for (int32_t k = M.off[c], e = M.off[c + 1]; k < e; ++k) s += (int64_t)M.coef[k] * (int64_t)a[M.cls[k]];
    if (s < 0) atomicMin(&st[kStatus], MOTIF_EINTERNAL);
    out[i] = (uint64_t)s;
  }
}

__global__ void k_solve_write(const uint64_t* __restrict__ in, uint64_t* __restrict__ out, int64_t total,
                              const int32_t* st) {
  if (st[kStatus] != 0) return;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x)
    out[i] = in[i];
}

unsigned grid_of(int64_t items, int per, int64_t most) {
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>(most, (items + per - 1) / per));
}

// ------------------------------------------------------------------ sizes --

constexpr int64_t kSplitCap = int64_t(64) << 20;  // entries of the row-split table (256 MB), beyond that binary searches
constexpr size_t kPlaneBytes = size_t(64) << 20;  // adjacency slices of k_tri_big

struct CountPlan {
  bool wide;                 // degrees may reach 2^21
  int32_t gran, ngran;
  bool split;
  int64_t D, words;          // bound on d+ and the words of an adjacency row
  int slices;                // workgroups of k_tri_big
  bool top;                  // some u may have more visits than a wave takes
};

CountPlan count_plan(int64_t n, int64_t m, int64_t maxn) {
  CountPlan c{};
  const int64_t mg = maxn > 0 ? maxn : n;
  c.wide = std::min(mg - 1, m) >= (int64_t(1) << 21);
  c.gran = c.wide ? top_granule<true>() : top_granule<false>();
  c.ngran = (int32_t)std::max<int64_t>(1, (mg + c.gran - 1) / c.gran);
  c.split = n * (c.ngran + 1) <= kSplitCap;
  // N+(x) has at most sqrt(2 m*) entries: its members all have degree d(x) or more
  int64_t r = 1;
  while (r * r <= 2 * m) ++r;
  c.D = std::max<int64_t>(1, std::min(mg, r));
  c.words = (c.D + 63) / 64;
  const size_t per = (size_t)c.D * (size_t)c.words * 16;
  c.slices = c.D > kTriD ? (int)std::max<size_t>(1, std::min<size_t>(256, kPlaneBytes / per)) : 0;
  c.top = 2 * m > 192;
  return c;
}

}  // namespace

size_t count_bytes(int64_t n, int64_t m, int64_t maxn, bool k4) {
  auto al = [](size_t b) { return (b + 255) & ~size_t(255); };
  if (!k4) return 0;
  const CountPlan c = count_plan(n, m, maxn);
  size_t b = al(sizeof(uint32_t) * 9 * (size_t)(m + 1)) + 2 * al(sizeof(int32_t) * (size_t)(n + 1));
  if (c.split) b += al(sizeof(int32_t) * (size_t)n * (c.ngran + 1));
  b += al((size_t)c.slices * (size_t)c.D * (size_t)c.words * 16 + 16);
  return b;
}

void enqueue_counts(Pipeline& p, const DevGraph& g, uint64_t* a3, uint64_t* a4, int32_t* queue, hipStream_t s) {
  // (the accumulators and the queue words are zeroed by the caller)
  const DevTables& T = dev_tables();
  const int64_t n = g.n, m = (g.gs_cap - 1) / 2;
  if (n == 0) return;
  const int cus = p.num_cus;
  int32_t* big = g.tmp_n;
  // enough chunks that every wave of the chip gets several, at most 16 vertices
  const int32_t chunk = (int32_t)std::max<int64_t>(1, std::min<int64_t>(16, n / (cus * 32)));
  const unsigned tri_grid = grid_of(n, g.gid ? kBatchChunk : 4 * chunk, cus * 6);
  if (!a4) {
    hipLaunchKernelGGL((k_tri<false>), dim3(grid_of(n, g.gid ? kBatchChunk : 4 * chunk, cus * 8)), dim3(256), 0, s, g,
                       T.lut[3], T.lut[4], a3, nullptr, nullptr, p.status, queue, chunk, big);
    hipLaunchKernelGGL((k_tri_big<false>), dim3(cus), dim3(512), 0, s, g, T.lut[3], T.lut[4], a3, nullptr, nullptr,
                       p.status, queue, big, nullptr, 0, 0);
    hipLaunchKernelGGL((k_local<true, false>), dim3(grid_of(n, 256, cus * 4)), dim3(256), 0, s, g, T.lut[3], T.lut[4],
                       a3, nullptr, nullptr, p.status, queue, 256);
    return;
  }
  const CountPlan c = count_plan(n, m, g.max_graph_n);
  uint32_t* Te = p.arena.take<uint32_t>(9 * (size_t)(m + 1));
  int32_t* mid = p.arena.take<int32_t>((size_t)n + 1);
  int32_t* top = p.arena.take<int32_t>((size_t)n + 1);
  int32_t* split = c.split ? p.arena.take<int32_t>((size_t)n * (c.ngran + 1)) : nullptr;
  u64* planes = p.arena.take<u64>((size_t)c.slices * (size_t)c.D * (size_t)c.words * 2 + 1);
  enqueue_zero(Te, sizeof(uint32_t) * 9 * (size_t)(m + 1), s);
  hipLaunchKernelGGL((k_tri<true>), dim3(tri_grid), dim3(256), 0, s, g, T.lut[3], T.lut[4], a3, a4, Te, p.status,
                     queue, chunk, big);
  if (c.slices > 0)
    hipLaunchKernelGGL((k_tri_big<true>), dim3(std::min(c.slices, cus)), dim3(512), 0, s, g, T.lut[3], T.lut[4], a3,
                       a4, Te, p.status, queue, big, planes, c.D, c.words);
  hipLaunchKernelGGL((k_wedge<64, 8>), dim3(grid_of(n, g.gid ? kBatchChunk : 4 * chunk, cus * 8)), dim3(256), 0, s, g,
                     T.lut[4], a4, p.status, queue, chunk, mid, top);
  if (c.top) {
    hipLaunchKernelGGL((k_wedge<256, 12>), dim3(cus * 3), dim3(256), 0, s, g, T.lut[4], a4, p.status, queue, 1, mid,
                       top);
    if (split)
      hipLaunchKernelGGL(k_split, dim3(grid_of(n * (c.ngran + 1), 256, 65536)), dim3(256), 0, s, g, c.gran, c.ngran,
                         split, p.status);
    if (c.wide)
      hipLaunchKernelGGL((k_wedge_top<true>), dim3(cus), dim3(kTopThreads), 0, s, g, T.lut[4], a4, p.status, queue,
                         top, split, c.ngran);
    else
      hipLaunchKernelGGL((k_wedge_top<false>), dim3(cus), dim3(kTopThreads), 0, s, g, T.lut[4], a4, p.status, queue,
                         top, split, c.ngran);
  }
  const int32_t lchunk = 1024;
  const dim3 lgrid(grid_of(n + m, lchunk, cus * 8));
  if (a3)
    hipLaunchKernelGGL((k_local<true, true>), lgrid, dim3(256), 0, s, g, T.lut[3], T.lut[4], a3, a4, Te, p.status,
                       queue, lchunk);
  else
    hipLaunchKernelGGL((k_local<false, true>), lgrid, dim3(256), 0, s, g, T.lut[3], T.lut[4], a3, a4, Te, p.status,
                       queue, lchunk);
}

void enqueue_solve(int k, const uint64_t* acc, uint64_t* tmp, uint64_t* out, int64_t ngraphs, int32_t* status,
                   hipStream_t s) {
  const int C = num_classes(k);
  const int64_t total = ngraphs * C;
  hipLaunchKernelGGL(k_solve, dim3(grid_of(total, 256, 65536)), dim3(256), 0, s, acc, dev_tables().inv[k], tmp, C,
                     total, status);
  hipLaunchKernelGGL(k_solve_write, dim3(grid_of(total, 256, 65536)), dim3(256), 0, s, tmp, out, total, status);
}

}  // namespace motif
