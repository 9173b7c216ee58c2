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
#include <type_traits>

#include "codes.h"
#include "counts.h"
#include "internal.h"

namespace motif {

namespace {

// The totals of graph g that this workgroup adds to.  A single graph has R
// copies of its totals, summed by k_solve_one: additions to one address (and
// one 128-byte line) queue up, and a thousand workgroups ending together on
// the same 199 counters took longer than their counting.
template <int C, int R>
__device__ __forceinline__ uint64_t* totals(const DevGraph& G, uint64_t* a, int32_t g) {
  return a + (int64_t)(G.gid ? g : (int32_t)blockIdx.x & (R - 1)) * C;
}

// ============================================================ triangles ==
//
// Every triangle x < y < z (rank order) once, from x: N+(x) in a wave-private
// hash, the N+ rows of its members streamed against it.  Per triangle: one
// count per typed triangle (27), and for k = 4 the typed degrees of its three
// corners (paws), the typed triangle counts T of its three edges (T[e][3 p +
// q], p, q the types of the third vertex seen from the lower and the higher
// end, less one) and one bit per type in an adjacency matrix of N+(x), from
// which the K4s above x are read off as the common bits of two rows.
// Sixteen lanes per x with at most 16 higher neighbours (four x per wave: the
// chain of loads before the first row is the bulk of a small x), one wave up
// to 64 and up to 128 (k_tri), one workgroup beyond (k_tri_big).

// Workgroup counters of the triangle kernels and their flush to one graph: by
// class in LDS first, so that a workgroup makes one global addition per class.
template <bool K4>
struct TriBins {
  u64* tri;   // [27] typed triangles (xy, xz, yz)
  u64* paw;   // [27][3 corners][3 types] sums of the corner's typed degree
  u64* kh;    // [199] classes (K4s while counting)
  u64* h3;    // [13] k = 3 classes, zero outside flush
  __device__ __forceinline__ void clear(int t, int nt) const {
    for (int i = t; i < 27; i += nt) tri[i] = 0;
    for (int i = t; i < 13; i += nt) h3[i] = 0;
    if constexpr (K4) {
      for (int i = t; i < 243; i += nt) paw[i] = 0;
      for (int i = t; i < 199; i += nt) kh[i] = 0;
    }
  }
  // Adds everything to one graph's totals and clears (every thread; the
  // counters are settled before and usable after).
  __device__ __forceinline__ void flush(const uint16_t* lut3, const uint16_t* lut4, uint64_t* a3, uint64_t* a4, int t,
                                        int nt) const {
    for (int i = t; i < 27; i += nt) {
      const u64 c = tri[i];
      if (!c) continue;
      const uint32_t xy = (uint32_t)i / 9 + 1, xz = ((uint32_t)i / 3) % 3 + 1, yz = (uint32_t)i % 3 + 1;
      atomicAdd(&h3[lut3[edge_code<3>(0, 1, xy) | edge_code<3>(0, 2, xz) | edge_code<3>(1, 2, yz)]], c);
      if constexpr (K4) {
        // the paths of three edges whose ends are one vertex
        auto p4 = [&](uint32_t mid, uint32_t p, uint32_t q) {
          atomicAdd(&kh[lut4[edge_code<4>(0, 1, mid) | edge_code<4>(0, 2, p) | edge_code<4>(1, 3, q)]], 0 - c);
        };
        p4(xy, xz, yz);
        p4(xz, xy, flip(yz));
        p4(yz, flip(xy), flip(xz));
      }
    }
    if constexpr (K4) {
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
        atomicAdd(&kh[lut4[edge_code<4>(0, 1, xy) | edge_code<4>(0, 2, xz) | edge_code<4>(1, 2, yz) |
                           edge_code<4>(corner, 3, s)]], w);
      }
    }
    __syncthreads();
    if (a3)
      for (int i = t; i < 13; i += nt) gadd(&a3[i], h3[i]);
    if constexpr (K4)
      for (int i = t; i < 199; i += nt) gadd(&a4[i], kh[i]);
    __syncthreads();
    clear(t, nt);
    __syncthreads();
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

// Calls one(v) for the listed vertices, `groups` of them at a time per
// workgroup (this thread's group: `my`), and flush(g) with every thread of the
// workgroup, between barriers, when all of a graph's vertices that this
// workgroup takes are done and at the end.  A single graph's list is dealt out
// entry by entry; a batch's in one segment per workgroup, cut into runs of one
// graph, so that a flush comes once per graph and segment or so.  WHOLE: a wave
// holds several groups and one() needs all of it: groups past the end of the
// list join in with one(-1).
template <int NT, bool WHOLE, class One, class Flush>
__device__ __forceinline__ void for_listed(const DevGraph& G, const int32_t* list, int32_t count, int groups, int my,
                                           One&& one, Flush&& flush) {
  if (!G.gid) {
    const int32_t step = (int32_t)gridDim.x * groups;
    for (int32_t i = (int32_t)blockIdx.x * groups + my; WHOLE ? __ballot(i < count) != 0ull : i < count; i += step)
      one(!WHOLE || i < count ? list[i] : -1);
    __syncthreads();
    flush(0);
    return;
  }
  __shared__ int32_t sh_run;
  const int32_t nb = min((int32_t)gridDim.x, count);  // (the callers leave workgroups from `count` on out)
  const int32_t s1 = (int32_t)((int64_t)count * (blockIdx.x + 1) / nb);
  int32_t cur = -1;
  for (int32_t s0 = (int32_t)((int64_t)count * blockIdx.x / nb); s0 < s1;) {
    const int32_t g = G.gid[list[s0]];
    __syncthreads();
    if (threadIdx.x == 0) sh_run = NT;
    __syncthreads();
    const int32_t i = s0 + (int32_t)threadIdx.x;
    if (i >= s1 || G.gid[list[i]] != g) atomicMin(&sh_run, (int32_t)threadIdx.x);
    __syncthreads();
    const int32_t e = s0 + sh_run;  // at least one entry
    if (g != cur) {
      if (cur >= 0) flush(cur);
      __syncthreads();
      cur = g;
    }
    for (int32_t k = s0 + my; WHOLE ? __ballot(k < e) != 0ull : k < e; k += groups)
      one(!WHOLE || k < e ? list[k] : -1);
    s0 = e;
  }
  __syncthreads();
  if (cur >= 0) flush(cur);
}

// Sorts the vertices into the lists: higher neighbours for the triangles,
// lower neighbours and visits for the wedges (k = 4).  Eight lanes per vertex;
// one counter update per list and workgroup.
// big: higher neighbours from which a vertex has a workgroup to itself; far: the
// graph has many ids.
constexpr int kClassify = 2048;  // most vertices of a workgroup (places fit in 12 bits)
template <bool K4>
__global__ __launch_bounds__(256) void k_classify(DevGraph G, Lists L, int32_t* __restrict__ nlist, int32_t big,
                                                  int32_t far, const int32_t* st) {
  __shared__ int32_t cnt[kLists], base[kLists];
  __shared__ uint32_t where[kClassify];
  if (st[kStatus] != 0) return;
  const int l8 = threadIdx.x & 7;
  const int64_t per = ((int64_t)G.n + gridDim.x - 1) / gridDim.x;  // vertices of this workgroup, at most kClassify
  const int64_t v0 = (int64_t)blockIdx.x * per, v1 = min((int64_t)G.n, v0 + per);
  if (v0 >= v1) return;
  if (threadIdx.x < kLists) cnt[threadIdx.x] = 0;
  __syncthreads();
  for (int64_t v = v0 + (threadIdx.x >> 3); v < v1; v += 32) {
    int lt = 15, lw = 15;
    const int32_t pa = G.np_off[v], pb = G.np_off[v + 1], d = pb - pa;
    if (d >= 2) lt = d <= 16 ? kTri16 : d >= big ? kTriBig : d <= 64 ? kTri64 : kTri128;
    if (K4) {
      const int32_t ma = G.gs_off[v] - pa, dm = G.gs_off[v + 1] - pb - ma;
      if (dm > (far ? kFarD : 127)) {
        lw = dm > kHugeD ? kWedgeHuge : kWedgeTop;
      } else if (dm >= 2) {
        int32_t vis = 0;
        const int32_t cap = far ? kFarVisits + 1 : kCap256 + 1;
        for (int32_t i = l8; i < dm; i += 32) {  // (past the end: the last one, not counted)
          uint32_t w[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) w[k] = G.nm_idx[ma + min(i + 8 * k, dm - 1)] & kIdMask;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int32_t dw = min(G.deg[w[k]], cap);
            vis += i + 8 * k < dm ? dw : 0;
          }
        }
#pragma unroll
        for (int o = 4; o; o >>= 1) vis += __shfl_xor(vis, o);
        if (dm > 127) lw = vis <= kFarVisits ? kWedgeFar11 : dm > kHugeD ? kWedgeHuge : kWedgeTop;
        else lw = vis <= kCap16 ? kWedge16 : vis <= kCap64 ? kWedge64 : vis <= kCap256 ? kWedge256 : kWedgeTop;
        if (far && lw == kWedgeTop && dm <= 127 && vis <= kFarVisits) lw = kWedgeFar7;
      }
    }
    if (l8 == 0) {  // lists of v (15: none) and its places in this workgroup's parts of them
      const int at = lt < kLists ? atomicAdd(&cnt[lt], 1) : 0, aw = lw < kLists ? atomicAdd(&cnt[lw], 1) : 0;
      where[v - v0] = (uint32_t)lt | (uint32_t)lw << 4 | (uint32_t)at << 8 | (uint32_t)aw << 20;
    }
  }
  __syncthreads();
  if (threadIdx.x < kLists && cnt[threadIdx.x]) base[threadIdx.x] = atomicAdd(&nlist[threadIdx.x], cnt[threadIdx.x]);
  __syncthreads();
  for (int64_t v = v0 + threadIdx.x; v < v1; v += 256) {
    const uint32_t w = where[v - v0], lt = w & 15u, lw = (w >> 4) & 15u;
    if (lt < kLists) L.v[lt][base[lt] + (int32_t)((w >> 8) & 4095u)] = (int32_t)v;
    if (lw < kLists) L.v[lw][base[lw] + (int32_t)(w >> 20)] = (int32_t)v;
  }
}

// GS lanes per x of at most D higher neighbours.  The triangles found are
// queued per wave and worked off by full waves: a pass over 64 entries finds
// one or two, and counting those on the spot kept 62 lanes waiting each time
// (n = 10^5 graph, k = 4: 343 us for the x of at most 64 neighbours).
template <int GS, int D, bool K4>
__global__ __launch_bounds__(256) void k_tri(DevGraph G, const uint16_t* __restrict__ lut3,
                                             const uint16_t* __restrict__ lut4, uint64_t* __restrict__ a3,
                                             uint64_t* __restrict__ a4, uint32_t* __restrict__ T, const int32_t* st,
                                             const int32_t* __restrict__ nlist, const int32_t* __restrict__ vlist) {
  constexpr int NGR = 256 / GS, HB = D == 16 ? 6 : D == 64 ? 8 : 9, H = 1 << HB, LPR = GS / 4;  // groups, hash, lanes per row
  constexpr int DM = (D + GS - 1) / GS, W = (D + 63) / 64;  // members per lane, words of an adjacency row
  constexpr int QC = 192;                                   // queued triangles per wave
  static_assert(H == 4 * D && D <= 128, "hash load; seven bits per count");
  __shared__ u64 s_tri[27], s_paw[K4 ? 243 : 1], s_kh[K4 ? 199 : 1], s_h3[13];
  __shared__ uint16_t lut[K4 ? 4096 : 1];
  __shared__ uint32_t s_key[NGR][H];
  __shared__ uint8_t s_at[NGR][H];
  __shared__ uint32_t s_list[NGR][D];
  __shared__ u64 s_T[K4 ? NGR : 1][D];                                     // nine 7-bit counters per member of N+(x)
  __shared__ u64 s_a1[K4 ? NGR : 1][D * W], s_a2[K4 ? NGR : 1][D * W];     // adjacency of N+(x), a bit plane per arc
  __shared__ int32_t s_x[NGR];
  __shared__ uint32_t s_q[K4 ? 4 : 1][QC];
  __shared__ int32_t s_qt[K4 ? 4 : 1][QC];
  if (st[kStatus] != 0) return;
  const int32_t count = nlist[D == 16 ? kTri16 : D == 64 ? kTri64 : kTri128];
  if ((int64_t)blockIdx.x * (G.gid ? 1 : NGR) >= count) return;
  const TriBins<K4> bins{s_tri, s_paw, s_kh, s_h3};
  const int wv = threadIdx.x >> 6, wl = threadIdx.x & 63;
  const int gr = threadIdx.x / GS, lane = threadIdx.x % GS, lane0 = wl - lane;
  bins.clear(threadIdx.x, 256);
  if (K4)
    for (int i = threadIdx.x; i < 4096; i += 256) lut[i] = lut4[i];
  for (int i = lane; i < H; i += GS) s_key[gr][i] = kNone;
  if (K4)
    for (int i = lane; i < D; i += GS) {
      s_T[gr][i] = 0;
      for (int w = 0; w < W; ++w) s_a1[gr][i * W + w] = s_a2[gr][i * W + w] = 0;
    }
  __syncthreads();
  uint32_t* key = s_key[gr];
  uint8_t* at = s_at[gr];
  uint32_t* list = s_list[gr];
  u64 *Tl = s_T[K4 ? gr : 0], *A1 = s_a1[K4 ? gr : 0], *A2 = s_a2[K4 ? gr : 0];
  int qn = 0;  // the same on every lane of the wave
  // queue entry: group of the wave, j, k (members y and z), type of z seen
  // from y; and the place of z in N+(y)
  auto drain = [&] {
    if constexpr (K4) {
      wave_sync();
      for (int i = wl; i < qn; i += 64) {
        const uint32_t q = s_q[wv][i];
        const int g = wv * (64 / GS) + (int)(q >> 16), j = (int)(q & 127u), k = (int)((q >> 7) & 127u);
        const uint32_t yz = (q >> 14) & 3u, ey = s_list[g][j], ez = s_list[g][k];
        const uint32_t xy = ey >> kTypeShift, xz = ez >> kTypeShift;
        atomicAdd(&T[(int64_t)s_qt[wv][i] * 9 + (flip(xy) - 1) * 3 + (flip(xz) - 1)], 1u);
        tri_add<true>(bins, (xy - 1) * 9 + (xz - 1) * 3 + (yz - 1), G.dt[s_x[g]], G.dt[ey & kIdMask],
                      G.dt[ez & kIdMask]);
        atomicAdd(&s_T[g][j], 1ull << (7 * ((xz - 1) * 3 + (yz - 1))));
        atomicAdd(&s_T[g][k], 1ull << (7 * ((xy - 1) * 3 + (flip(yz) - 1))));
        if (yz & 1u) atomicOr(&s_a1[g][j * W + (k >> 6)], 1ull << (k & 63));
        if (yz & 2u) atomicOr(&s_a2[g][j * W + (k >> 6)], 1ull << (k & 63));
      }
      wave_sync();
    }
    qn = 0;
  };

  auto one = [&](int32_t x) {  // the same x on the GS lanes of a group; x < 0: none.  Called by whole waves.
    int32_t xa = 0, d = 0;
    if (x >= 0) {
      xa = G.np_off[x];
      d = G.np_off[x + 1] - xa;  // 2 .. D
      if (K4 && lane == 0) s_x[gr] = x;
    }
    // members lane, lane + GS .. of N+(x): entry, hash slot, row
    uint32_t e[DM], hs[DM];
    int32_t ra[DM], len[DM];
#pragma unroll
    for (int u = 0; u < DM; ++u) {
      const int32_t i = lane + u * GS;
      e[u] = hs[u] = 0;
      ra[u] = len[u] = 0;
      if (i < d) {
        e[u] = G.np_idx[xa + i];
        const uint32_t y = e[u] & kIdMask;
        list[i] = e[u];
        hs[u] = hash_mul(y, HB);
        while (atomicCAS(&key[hs[u]], kNone, y) != kNone) hs[u] = (hs[u] + 1) & (H - 1);
        at[hs[u]] = (uint8_t)i;
        ra[u] = G.np_off[y];
        len[u] = G.np_off[y + 1] - ra[u];
      }
    }
    wave_sync();
    const int32_t sub = lane / LPR, lr = lane % LPR;
    for (int32_t j0 = 0; __ballot(j0 < d) != 0ull; j0 += 4) {
      const int32_t j = j0 + sub;
      int32_t a = __shfl(ra[0], lane0 + (j & (GS - 1))), m = __shfl(len[0], lane0 + (j & (GS - 1)));
      if constexpr (DM > 1) {
        const int32_t a1 = __shfl(ra[DM - 1], lane0 + (j & (GS - 1))), m1 = __shfl(len[DM - 1], lane0 + (j & (GS - 1)));
        if (j >= GS) {
          a = a1;
          m = m1;
        }
      }
      if (j >= d) m = 0;
      for (int32_t t0 = 0; __ballot(t0 + lr < m) != 0ull; t0 += 4 * LPR) {
        uint32_t f[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) f[u] = m > 0 ? G.np_idx[a + min(t0 + lr + u * LPR, m - 1)] : 0u;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int32_t t = t0 + lr + u * LPR;
          int32_t k = -1;
          if (t < m) {
            const uint32_t z = f[u] & kIdMask;
            uint32_t h = hash_mul(z, HB), kk;
            while ((kk = key[h]) != z && kk != kNone) h = (h + 1) & (H - 1);
            if (kk == z) k = at[h];
          }
          if constexpr (K4) {
            const u64 hit = __ballot(k >= 0);
            if (!hit) continue;
            if (k >= 0) {
              const int s = qn + __popcll(hit & ((1ull << wl) - 1ull));
              s_q[wv][s] = (uint32_t)(gr % (64 / GS)) << 16 | (f[u] >> kTypeShift) << 14 | (uint32_t)k << 7 | (uint32_t)j;
              s_qt[wv][s] = a + t;
            }
            qn += __popcll(hit);
            if (qn > QC - 64) drain();
          } else if (k >= 0) {
            atomicAdd(&bins.tri[((list[j] >> kTypeShift) - 1) * 9 + ((list[k] >> kTypeShift) - 1) * 3 +
                                ((f[u] >> kTypeShift) - 1)], 1ull);
          }
        }
      }
    }
    if (K4 && qn) drain();
    wave_sync();
    if constexpr (K4) {
#pragma unroll
      for (int u = 0; u < DM; ++u) {
        const int32_t i = lane + u * GS;
        if (i >= d) continue;
        const uint32_t bx = edge_code<4>(0, 1, e[u] >> kTypeShift);
        for (int w = 0; w < W; ++w) {
          const u64 p1 = A1[i * W + w], p2 = A2[i * W + w];
          for (u64 r = p1 | p2; r; r &= r - 1ull) {  // edge i -> k above x
            const int b = __builtin_ctzll(r), k = w * 64 + b;
            uint32_t bk = 0;
            for (int v = 0; v < W; ++v) {
              const u64 r1 = A1[i * W + v], r2 = A2[i * W + v], q1 = A1[k * W + v], q2 = A2[k * W + v];
              u64 com = (r1 | r2) & (q1 | q2);
              if (!com) continue;
              if (!bk)
                bk = bx | edge_code<4>(0, 2, list[k] >> kTypeShift) |
                     edge_code<4>(1, 2, (uint32_t)((p1 >> b) & 1) | (uint32_t)((p2 >> b) & 1) << 1);
              for (; com; com &= com - 1ull) {
                const int l = __builtin_ctzll(com);
                const uint32_t code = bk | edge_code<4>(0, 3, list[v * 64 + l] >> kTypeShift) |
                                      edge_code<4>(1, 3, (uint32_t)((r1 >> l) & 1) | (uint32_t)((r2 >> l) & 1) << 1) |
                                      edge_code<4>(2, 3, (uint32_t)((q1 >> l) & 1) | (uint32_t)((q2 >> l) & 1) << 1);
                atomicAdd(&bins.kh[lut[code]], 1ull);
              }
            }
          }
        }
        const u64 c = Tl[i];
        if (c)
          for (int f = 0; f < 9; ++f) {
            const uint32_t v = (uint32_t)(c >> (7 * f)) & 127u;
            if (v) atomicAdd(&T[(int64_t)(xa + i) * 9 + f], v);
          }
      }
      wave_sync();
#pragma unroll
      for (int u = 0; u < DM; ++u) {
        const int32_t i = lane + u * GS;
        if (i >= d) continue;
        Tl[i] = 0;
        for (int w = 0; w < W; ++w) A1[i * W + w] = A2[i * W + w] = 0;
      }
    }
#pragma unroll
    for (int u = 0; u < DM; ++u)
      if (lane + u * GS < d) key[hs[u]] = kNone;
    wave_sync();
  };
  for_listed<256, GS < 64>(G, vlist, count, NGR, gr, one, [&](int32_t g) {
    bins.flush(lut3, K4 ? lut : lut4, a3 ? totals<13, kRep3>(G, a3, g) : nullptr,
               K4 ? totals<199, kRep4>(G, a4, g) : nullptr, threadIdx.x, 256);
  });
}

// The x with more than 128 higher neighbours, one workgroup each: N+(x) in an
// LDS hash of up to kBigH / 2 members (beyond that a binary search in the
// id-sorted row), T by global atomics, and for k = 4 the two adjacency bit
// planes of N+(x), in LDS up to kPlaneD members and else in the workgroup's
// slice of global memory (2 D rows of `words` words, D >= any d+).  A launch
// takes the x of above < d+ <= most.  d+ is at most sqrt(2 m), so only large dense graphs have any (98 at most on the n =
// 10^5, m = 10^6 graph).
constexpr int kBigHB = 13;
constexpr int kBigH = 1 << kBigHB;
constexpr int kPlaneD = 256;
// Common bits of a word up to which they are taken one by one (n = 800 with 15 %
// of the arcs: 1,247 us a call, 1,390 with 4; n = 400 with 75 %: 9.2 and 7.5 ms).
constexpr int kFewBits = 8;

template <bool K4>
__global__ __launch_bounds__(512) void k_tri_big(DevGraph G, const uint16_t* __restrict__ lut3,
                                                 const uint16_t* __restrict__ lut4, uint64_t* __restrict__ a3,
                                                 uint64_t* __restrict__ a4, uint32_t* __restrict__ T,
                                                 const int32_t* st, const int32_t* __restrict__ nlist,
                                                 const int32_t* __restrict__ vlist, u64* __restrict__ planes, int64_t D,
                                                 int64_t words, int32_t above, int32_t most) {
  constexpr int NT = 512, NW = NT / 64;
  __shared__ u64 s_tri[27], s_paw[K4 ? 243 : 1], s_kh[K4 ? 199 : 1], s_h3[13];
  __shared__ uint32_t key[kBigH];
  __shared__ uint16_t at[kBigH];
  __shared__ u64 xt1[K4 ? kBigH / 128 : 1], xt2[K4 ? kBigH / 128 : 1];  // types of N+(x), a bit plane per arc
  __shared__ u64 lplane[K4 ? 2 * kPlaneD * kPlaneD / 64 : 1];
  __shared__ uint16_t lut[K4 ? 4096 : 1];
  if (st[kStatus] != 0) return;
  const int32_t count = nlist[kTriBig];
  if ((int32_t)blockIdx.x >= count) return;
  const TriBins<K4> bins{s_tri, s_paw, s_kh, s_h3};
  bins.clear(threadIdx.x, NT);
  for (int i = threadIdx.x; i < kBigH; i += NT) key[i] = kNone;
  if (K4)
    for (int i = threadIdx.x; i < 4096; i += NT) lut[i] = lut4[i];
  __syncthreads();
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  // rows of the adjacency: LDS planes plainly, global ones by accesses in L2
  // (where their bits are set by atomics)
  auto work = [&](int32_t x, auto in_lds, u64* P1, u64* P2) {
    constexpr bool L = decltype(in_lds)::value;
    auto put = [&](u64* p, u64 v) {
      if constexpr (L) *p = v;
      else __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    auto word = [&](const u64* p, int64_t i) {
      if constexpr (L) return p[i];
      else return __hip_atomic_load(p + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
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
    if (K4 && hashed)
      for (int32_t i = threadIdx.x; i < W * 64; i += NT) {
        const uint32_t t = i < d ? G.np_idx[xa + i] >> kTypeShift : 0u;
        const u64 b1 = __ballot(t & 1u), b2 = __ballot(t & 2u);
        if (lane == 0) {
          xt1[i >> 6] = b1;
          xt2[i >> 6] = b2;
        }
      }
    if (K4)
      for (int64_t i = threadIdx.x; i < (int64_t)d * W; i += NT) {
        put(&P1[i], 0ull);
        put(&P2[i], 0ull);
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
      // The K4s of an edge j -> k: the common bits of their rows, one by one
      // where a word has few of them, else counted by their types towards x, j
      // and k, 27 intersections a word (n = 300, three quarters of the arcs:
      // the call 34.2 -> 2.8 ms, with the lanes' choice below).
      auto edge = [&](int32_t j, int32_t k, uint32_t bx, uint32_t yz, int32_t l0, int32_t ls) {
        const uint32_t bk = bx | edge_code<4>(0, 2, G.np_idx[xa + k] >> kTypeShift) | edge_code<4>(1, 2, yz);
        auto code = [&](uint32_t x, uint32_t r, uint32_t q) {
          return bk | edge_code<4>(0, 3, x) | edge_code<4>(1, 3, r) | edge_code<4>(2, 3, q);
        };
        uint32_t n[14];  // two counts a word: at most d, 4,096
        bool many = false;
#pragma unroll
        for (int i = 0; i < 14; ++i) n[i] = 0;
        for (int32_t lw = l0; lw < W; lw += ls) {
          const u64 r1 = word(P1, (int64_t)j * W + lw), r2 = word(P2, (int64_t)j * W + lw);
          const u64 q1 = word(P1, (int64_t)k * W + lw), q2 = word(P2, (int64_t)k * W + lw);
          u64 com = (r1 | r2) & (q1 | q2);
          if (hashed && __popcll(com) > kFewBits) {
            many = true;
            const u64 x1 = xt1[lw], x2 = xt2[lw];
            const u64 r[3] = {r1 & ~r2, r2 & ~r1, r1 & r2}, q[3] = {q1 & ~q2, q2 & ~q1, q1 & q2};
            const u64 x[3] = {x1 & ~x2, x2 & ~x1, x1 & x2};
#pragma unroll
            for (int i = 0; i < 27; ++i)
              n[i >> 1] += (uint32_t)__popcll(x[i / 9] & r[(i / 3) % 3] & q[i % 3]) << (16 * (i & 1));
            continue;
          }
          for (; com; com &= com - 1ull) {
            const int l = __builtin_ctzll(com);
            atomicAdd(&bins.kh[lut[code(G.np_idx[xa + lw * 64 + l] >> kTypeShift,
                                        (uint32_t)((r1 >> l) & 1) | (uint32_t)((r2 >> l) & 1) << 1,
                                        (uint32_t)((q1 >> l) & 1) | (uint32_t)((q2 >> l) & 1) << 1)]], 1ull);
          }
        }
        if (many)
#pragma unroll
          for (int i = 0; i < 27; ++i) {
            const uint32_t c = (n[i >> 1] >> (16 * (i & 1))) & 0xFFFFu;
            if (c) atomicAdd(&bins.kh[lut[code(i / 9 + 1, (i / 3) % 3 + 1, i % 3 + 1)]], (u64)c);
          }
      };
      // a lane per k of row j, or per word of the rows, whichever takes fewer steps
      for (int32_t j = wv; j < d; j += NW) {
        const uint32_t bx = edge_code<4>(0, 1, G.np_idx[xa + j] >> kTypeShift);
        for (int32_t kw = 0; kw < W; ++kw) {
          const u64 p1 = word(P1, (int64_t)j * W + kw), p2 = word(P2, (int64_t)j * W + kw);
          if (L || (hashed && __popcll(p1 | p2) > W)) {
            const uint32_t yz = (uint32_t)((p1 >> lane) & 1) | (uint32_t)((p2 >> lane) & 1) << 1;
            if (yz) edge(j, kw * 64 + lane, bx, yz, 0, 1);
          } else {
            for (u64 r = p1 | p2; r; r &= r - 1ull) {  // the same on every lane
              const int b = __builtin_ctzll(r);
              edge(j, kw * 64 + b, bx, (uint32_t)((p1 >> b) & 1) | (uint32_t)((p2 >> b) & 1) << 1, lane, 64);
            }
          }
        }
      }
      __syncthreads();
    }
    if (hashed)
      for (int i = threadIdx.x; i < kBigH; i += NT) key[i] = kNone;
    __syncthreads();
  };
  u64* const gp = K4 ? planes + (int64_t)blockIdx.x * 2 * D * words : nullptr;
  for_listed<NT, false>(
      G, vlist, count, 1, 0,
      [&](int32_t x) {
        const int32_t d = G.np_off[x + 1] - G.np_off[x];
        if (d <= above || d > most) return;  // another launch's
        if (!K4 || d <= kPlaneD) work(x, std::true_type{}, lplane, lplane + kPlaneD * kPlaneD / 64);
        else work(x, std::false_type{}, gp, gp + D * words);
      },
      [&](int32_t g) {
        bins.flush(lut3, K4 ? lut : lut4, a3 ? totals<13, kRep3>(G, a3, g) : nullptr,
                   K4 ? totals<199, kRep4>(G, a4, g) : nullptr, threadIdx.x, NT);
      });
}

// ================================================================ wedges ==
//
// C4s, each from its vertex u of highest rank: W[w][3 p + q] = wedges u - v -
// w with v of lower rank than u, p and q (less one) the types of v seen from u
// and of w seen from v.  Two wedges to the same w of lower rank are a C4
// u - v - w - v'.  A count is at most min(d-(u), d(w)), which bounds the width
// of its field: nine fields of 7 bits share one 64-bit word while d-(u) <= 127.
//   k_wedge<16, 7>, <64, 9>, <256, 12>   that many threads per u and a hash of
//                    w, for u with at most 96, 384 and 3,072 visits
//   k_wedge_top      the rest: a direct table over one block of vertex ids at a
//                    time, the work unit being (u, block)

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

template <int NT, int HB>
__global__ __launch_bounds__(256) void k_wedge(DevGraph G, const uint16_t* __restrict__ lut4,
                                               uint64_t* __restrict__ a4, const int32_t* st,
                                               const int32_t* __restrict__ nlist, const int32_t* __restrict__ vlist) {
  constexpr int NU = 256 / NT, H = 1 << HB;
  constexpr int LPR = NT == 16 ? 4 : 8;  // lanes per row
  static_assert((NT == 16 ? kCap16 : NT == 64 ? kCap64 : kCap256) <= H * 3 / 4, "hash load");
  __shared__ uint32_t s_key[NU][H];
  __shared__ u64 s_cnt[NU][H];
  __shared__ uint16_t s_act[NU][H];  // slots with two wedges or more
  __shared__ int32_t s_nact[NU];
  __shared__ u64 bins[81];
  if (st[kStatus] != 0) return;
  const int32_t count = nlist[NT == 16 ? kWedge16 : NT == 64 ? kWedge64 : kWedge256];
  if ((int64_t)blockIdx.x * (G.gid ? 1 : NU) >= count) return;
  const int un = threadIdx.x / NT, t = threadIdx.x % NT;
  uint32_t* key = s_key[un];
  u64* cnt = s_cnt[un];
  for (int i = t; i < H; i += NT) {
    key[i] = kNone;
    cnt[i] = 0;
  }
  for (int i = threadIdx.x; i < 81; i += 256) bins[i] = 0;
  if (t == 0) s_nact[un] = 0;
  __syncthreads();
  uint16_t* act = s_act[un];
  auto sync = [] {
    if constexpr (NT <= 64) wave_sync();
    else __syncthreads();
  };
  auto one = [&](int32_t u) {  // the same u on the NT threads
    const int32_t ua = G.gs_off[u], ub = G.gs_off[u + 1];
    const int32_t ma = ua - G.np_off[u], dm = ub - G.np_off[u + 1] - ma;
    for (int32_t i = t / LPR; i < dm; i += NT / LPR) {
      const uint32_t ev = G.nm_idx[ma + i], v = ev & kIdMask;
      const int32_t ra = G.gs_off[v], rb = G.gs_off[v + 1];
      const int p7 = 21 * (int)((ev >> kTypeShift) - 1u);
      auto entry = [&](int32_t, uint32_t f) {
        const uint32_t w = f & kIdMask;
        if ((int32_t)w == u) return;
        uint32_t h = hash_mul(w, HB);
        for (;;) {
          const uint32_t old = atomicCAS(&key[h], kNone, w);
          if (old == kNone || old == w) break;
          h = (h + 1) & (H - 1);
        }
        atomicAdd(&cnt[h], 1ull << (p7 + 7 * (int)((f >> kTypeShift) - 1u)));
      };
      for (int32_t r = t % LPR; r < rb - ra; r += 4 * LPR) each4(G.gs_idx + ra, r, LPR, rb - ra, entry);
    }
    sync();
    const uint32_t du = (uint32_t)(ub - ua);
    // listed first: the ranks of all of them are then one load away
    for (int i = t; i < H; i += NT) {
      const u64 c = cnt[i];
      if (!c) continue;
      if (one_wedge(c, kOnes7)) {
        cnt[i] = 0;
        key[i] = kNone;
      } else {
        act[atomicAdd(&s_nact[un], 1)] = (uint16_t)i;
      }
    }
    sync();
    const int32_t na = s_nact[un];
    for (int k = t; k < na; k += NT) {
      const int i = act[k];
      const u64 c = cnt[i];
      cnt[i] = 0;
      const uint32_t w = key[i];
      key[i] = kNone;
      if (!ranked_below(G, (uint32_t)G.deg[w], (int32_t)w, du, u)) continue;
      uint32_t f[9];
#pragma unroll
      for (int j = 0; j < 9; ++j) f[j] = (uint32_t)(c >> (7 * j)) & 127u;
      c4_pairs(f, bins);
    }
    sync();
    if (t == 0) s_nact[un] = 0;
    sync();
  };
  for_listed<256, false>(G, vlist, count, NU, un, one, [&](int32_t g) {
    c4_flush(bins, lut4, totals<199, kRep4>(G, a4, g), threadIdx.x, 256);
    __syncthreads();
    if (threadIdx.x < 81) bins[threadIdx.x] = 0;
  });
}

// Vertices of k_wedge_top on graphs of many ids, where nearly every block would
// have a handful of a vertex's entries: the w of u in parts by their mixed ids,
// as many as keep a part within the hash (H / 2 vertices; a part with more is
// halved until it fits), one workgroup per u.  Rows in pieces of 64 entries,
// sixteen lanes each, listed once.  FB bits per count: 7 in one word for u with
// at most 127 lower neighbours, 11 in two.  k = 4 of power laws, m = 6 * 10^6
// arcs: n = 3 * 10^6 (exponent 2.5) 65.7 ms by blocks and 10.5 so, n = 6 * 10^6
// (2.2) 244 and 65; n = 10^6 of 10^7 arcs 53.4 and 26.9.
__device__ __forceinline__ uint32_t mix32(uint32_t h) {  // finaliser of MurmurHash3 (A. Appleby), a bijection
  h ^= h >> 16;
  h *= 0x85EBCA6Bu;
  h ^= h >> 13;
  h *= 0xC2B2AE35u;
  return h ^ h >> 16;
}
template <int HB, int FB>
__global__ __launch_bounds__(1024) void k_wedge_far(DevGraph G, const uint16_t* __restrict__ lut4,
                                                    uint64_t* __restrict__ a4, const int32_t* st,
                                                    const int32_t* __restrict__ nlist, const int32_t* __restrict__ vlist) {
  constexpr int NT = 1024, H = 1 << HB, NWORD = FB == 7 ? 1 : 2, MAXP = kFarVisits / 64 + kFarD;
  static_assert(H / 2 + NT < H, "probes end: a part stops at H / 2 vertices, with one more per thread on the way");
  static_assert(FB == 7 || kFarD < 2048, "11-bit counts");
  __shared__ uint32_t key[H], piece[MAXP];  // piece: row << 16 | place in it
  __shared__ u64 cnt[NWORD][H], bins[81];
  __shared__ int32_t row[kFarD], len[kFarD];  // len: entries << 2 | type less one
  __shared__ int32_t npiece, visits, used, over;
  if (st[kStatus] != 0) return;
  const int32_t count = nlist[FB == 7 ? kWedgeFar7 : kWedgeFar11];
  if ((int32_t)blockIdx.x >= count) return;
  const int t = threadIdx.x;
  for (int i = t; i < H; i += NT) {
    key[i] = kNone;
    for (int w = 0; w < NWORD; ++w) cnt[w][i] = 0;
  }
  if (t < 81) bins[t] = 0;
  if (t == 0) npiece = visits = used = over = 0;
  __syncthreads();
  auto one = [&](int32_t u) {  // the same u on every thread
    const int32_t ua = G.gs_off[u], ub = G.gs_off[u + 1];
    const int32_t ma = ua - G.np_off[u], dm = ub - G.np_off[u + 1] - ma;  // dm <= kFarD
    const uint32_t du = (uint32_t)(ub - ua);
    if (t < dm) {
      const uint32_t ev = G.nm_idx[ma + t], v = ev & kIdMask;
      const int32_t ra = G.gs_off[v], m = G.gs_off[v + 1] - ra, q = (m + 63) >> 6;
      row[t] = ra;
      len[t] = m << 2 | (int32_t)((ev >> kTypeShift) - 1u);
      atomicAdd(&visits, m);
      const int32_t at = atomicAdd(&npiece, q);
      for (int32_t j = 0; j < q; ++j) piece[at + j] = (uint32_t)t << 16 | (uint32_t)j;
    }
    __syncthreads();
    const int32_t np = npiece, vis = visits;
    uint32_t parts = 1;
    while ((uint32_t)vis > parts * (H * 3 / 8)) parts *= 2;
    __syncthreads();
    if (t == 0) npiece = visits = 0;
    for (uint32_t first = 0; first < parts; ++first)
      for (uint32_t mod = parts, res = first;;) {  // w with mix32(w) = res modulo mod, a power of two
        for (int32_t x = t >> 4; x < np; x += NT / 16) {
          const uint32_t pc = piece[x];
          const int32_t i = (int32_t)(pc >> 16), off = (int32_t)(pc & 0xFFFFu) * 64, p = len[i] & 3;
          each4(G.gs_idx + row[i] + off, t & 15, 16, min(64, (len[i] >> 2) - off), [&](int32_t, uint32_t f) {
            const uint32_t w = f & kIdMask;
            if ((mix32(w) & (mod - 1u)) != res || (int32_t)w == u) return;
            if (__hip_atomic_load(&over, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) return;
            uint32_t h = hash_mul(w, HB);
            for (;;) {
              const uint32_t old = atomicCAS(&key[h], kNone, w);
              if (old == kNone && atomicAdd(&used, 1) >= H / 2) over = 1;
              if (old == kNone || old == w) break;
              h = (h + 1) & (H - 1);
            }
            const int k = 3 * p + (int)(f >> kTypeShift) - 1;
            if constexpr (NWORD == 1) atomicAdd(&cnt[0][h], 1ull << (7 * k));
            else atomicAdd(&cnt[k / 5][h], 1ull << (11 * (k % 5)));
          });
        }
        __syncthreads();
        const bool full = over != 0;
        for (int i = t; i < H; i += NT) {
          const uint32_t w = key[i];
          if (w == kNone) continue;
          uint32_t c[9], sum = 0;
#pragma unroll
          for (int k = 0; k < 9; ++k) {
            c[k] = NWORD == 1 ? (uint32_t)(cnt[0][i] >> (7 * k)) & 127u
                              : (uint32_t)(cnt[NWORD == 1 ? 0 : k / 5][i] >> (11 * (k % 5))) & 2047u;
            sum += c[k];
          }
          if (!full && sum > 1 && ranked_below(G, (uint32_t)G.deg[w], (int32_t)w, du, u)) c4_pairs(c, bins);
          key[i] = kNone;
          for (int k = 0; k < NWORD; ++k) cnt[k][i] = 0;
        }
        __syncthreads();
        if (t == 0) used = over = 0;
        __syncthreads();
        if (full) {  // the same on every thread
          mod *= 2;
          continue;
        }
        while (mod > parts && res >= mod / 2) {  // both halves of the part above are done
          mod /= 2;
          res -= mod;
        }
        if (mod == parts) break;
        res += mod / 2;
      }
  };
  for_listed<NT, false>(G, vlist, count, 1, 0, one, [&](int32_t g) {
    c4_flush(bins, lut4, totals<199, kRep4>(G, a4, g), t, NT);
    __syncthreads();
    if (t < 81) bins[t] = 0;
  });
}

// Vertex u of many visits: (u, block of kBlock ids) is a work unit of one
// workgroup.  The sum over w of the products of two of its nine wedge counts is
// a 9 x 9 Gram matrix, taken by the matrix cores: the counts sit in LDS as
// bytes, one row of the block per field, so that a lane reads sixteen of its
// field's counts at once, and 64 w are one v_mfma_i32_16x16x64_i8 with the same
// register as both operands (row 9 holds ones: the plain sums, for the pairs
// within a field).  Counts stay below 128 where d-(u) or d(w) does; the w of
// degree over 127 (hubs), when d-(u) is too, have 32-bit counts instead, kHubs
// of them at a time, multiplied digit by digit (ND digits of 7 bits).  The
// pairs as 45 products per w summed in LDS took 1,300 us on the n = 10^5 graph,
// where every wave's 45 additions meet on the same 45 words.
//
// The blocks of a single graph: ids 0, kBlock, 2 kBlock, .. and, for the
// vertices of more than kHugeD lower neighbours, kCuts equal shares of the G*
// entries besides (a power-law graph's first ids are its hubs: of 1.7e7
// entries that a first block took, 4.4e5 were one unit's, and the workgroups
// with such units had three times the mean work).  split holds the first entry
// of every block in every row, so that a unit reads its part of each row N(v)
// only (null: binary search).  The parts are
// listed in LDS first, empty ones left out, kParts rows at a time, so that the
// loads that find them are one short chain for many rows; 4, 16 or 64 lanes
// then read a part, by its length.
constexpr int kBlock = 12288;
constexpr int kByteRow = kBlock + 64;  // bytes of a field's row: four fields on distinct banks
constexpr int kCuts = 24;
constexpr int64_t kCutsM = 32768;  // arcs from which the shares are cut
constexpr int kHubs = 1024;
constexpr int kShortPart = 16, kLongPart = 64, kLongs = 128;
constexpr int kTopThreads = 1024;
constexpr int kParts = 1024;
constexpr int kGramRun = 1024;  // products of 64 w between flushes: 64 * 127^2 * 1024 < 2^31

typedef int v4i __attribute__((ext_vector_type(4)));

// Gram sums of one wave over ND digits: acc[a (a + 1) / 2 + b] = digit a
// (rows) by digit b <= a (columns), 16 x 16 spread over the lanes: register r
// of lane l is row (l / 16) * 4 + r, column l % 16.
template <int ND>
struct Gram {
  static constexpr int N = ND * (ND + 1) / 2;
  v4i acc[N];
  int run = 0;
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int i = 0; i < N; ++i) acc[i] = v4i{0, 0, 0, 0};
    run = 0;
  }
  // Into bins[9 i + j], i <= j: sums of n_i n_j; bins[81 + i]: sums of n_i.
  __device__ __forceinline__ void flush(u64* bins) {
    if (run == 0) return;
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));  // (else the 24 addresses below live in registers through the caller's loop)
    const int j = lane & 15;
#pragma unroll
    for (int a = 0; a < ND; ++a)
#pragma unroll
      for (int b = 0; b <= a; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = (lane >> 4) * 4 + r;
          const u64 v = (u64)(uint32_t)acc[a * (a + 1) / 2 + b][r] << (7 * (a + b));
          if (!v || i > 8 || j > 9) continue;
          if (j == 9) {
            if (b == 0) atomicAdd(&bins[81 + i], v);
          } else if (a == b) {
            if (i <= j) atomicAdd(&bins[9 * i + j], v);
          } else {
            atomicAdd(&bins[9 * min(i, j) + max(i, j)], i == j ? 2 * v : v);
          }
        }
    clear();
  }
};

template <int ND, bool SPLIT>
__global__ __launch_bounds__(kTopThreads) void k_wedge_top(DevGraph G, const uint16_t* __restrict__ lut4,
                                                           uint64_t* __restrict__ a4, const int32_t* st,
                                                           const int32_t* __restrict__ nlist,
                                                           const int32_t* __restrict__ top,
                                                           const int32_t* __restrict__ huge,
                                                           const int32_t* __restrict__ split, int32_t nblk,
                                                           int32_t nfine, const int32_t* __restrict__ bnd) {
  // bnd: ids of the nfine + 1 boundaries, then the places among them of the
  // nblk + 1 multiples of kBlock (null: these alone, within each graph)
  constexpr int NT = kTopThreads, NW = NT / 64, NQ = kBlock / 64;
  __shared__ __align__(16) uint32_t bytes[9 * kByteRow / 4];
  __shared__ __align__(16) uint32_t wide[9 * kHubs];
  __shared__ int32_t pt_a[kParts + kLongs], pt_n[kParts + kLongs];
  __shared__ u64 mlow[NQ], mhub[NQ];  // of the block's ids: of lower rank than u, of degree over 127
  __shared__ uint16_t hpre[NQ];       // hubs before each word of mhub
  __shared__ u64 bins[90];
  __shared__ int32_t nshort, nmid, nlong, nhub;
  if (st[kStatus] != 0) return;
  const int64_t uhuge = (int64_t)nlist[kWedgeHuge] * nfine, units = uhuge + (int64_t)nlist[kWedgeTop] * nblk;
  if ((int64_t)blockIdx.x >= units) return;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int i = threadIdx.x; i < 90; i += NT) bins[i] = 0;
  if (threadIdx.x == 0) nshort = nmid = nlong = nhub = 0;
  Gram<1> low;   // byte counts
  Gram<ND> hub;  // hub counts
  low.clear();
  hub.clear();
  int32_t cur = -1;
  auto give = [&](int32_t g) {  // every wave's sums to graph g
    low.flush(bins);
    hub.flush(bins);
    __syncthreads();
    if (threadIdx.x < 9) {  // pairs within a field: (sum of squares - sum) / 2
      u64& d = bins[10 * threadIdx.x];
      d = (d - bins[81 + threadIdx.x]) / 2;
    }
    __syncthreads();
    c4_flush(bins, lut4, totals<199, kRep4>(G, a4, g), threadIdx.x, NT);
    __syncthreads();
    for (int i = threadIdx.x; i < 90; i += NT) bins[i] = 0;
    __syncthreads();
  };
  const v4i ones = v4i{0x01010101, 0x01010101, 0x01010101, 0x01010101}, none = v4i{0, 0, 0, 0};
  const int fld = lane & 15, kb = lane >> 4;
  // A unit: its vertex, the vertex's N- row, its ids [w0, w0 + nw).
  struct Unit {
    int32_t u = 0, du = 0, ma = 0, dm = 0, f0 = 0, f1 = 0, g = 0, base = 0, w0 = 0, nw = 0;
  };
  auto scalar = [](int32_t v) { return __builtin_amdgcn_readfirstlane(v); };  // the same on every lane
  auto vertex_of = [&](int64_t unit, Unit& X) {
    const bool h = unit < uhuge;
    const int64_t i = h ? unit : unit - uhuge;
    const int32_t per = h ? nfine : nblk;
    const int64_t at = i < (int64_t(1) << 31) ? (int64_t)((uint32_t)i / (uint32_t)per) : i / per;
    const int32_t blk = (int32_t)(i - at * per);
    X.u = scalar((h ? huge : top)[at]);
    X.f0 = scalar(h || !bnd ? blk : bnd[nfine + 1 + blk]);
    X.f1 = scalar(h || !bnd ? blk + 1 : bnd[nfine + 2 + blk]);
  };
  auto id_of = [&](int32_t f) { return bnd ? (int64_t)scalar(bnd[f]) : (int64_t)f * kBlock; };  // within the graph
  auto rows_of = [&](Unit& X) {
    const int32_t ua = scalar(G.gs_off[X.u]), ub = scalar(G.gs_off[X.u + 1]);
    const int32_t pa = scalar(G.np_off[X.u]), pb = scalar(G.np_off[X.u + 1]);
    X.du = ub - ua;
    X.ma = ua - pa;
    X.dm = ub - pb - X.ma;
    X.g = G.gid ? scalar(G.gid[X.u]) : 0;
    X.base = G.voff ? scalar((int32_t)G.voff[X.g]) : 0;
    const int64_t ng = G.voff ? scalar((int32_t)G.voff[X.g + 1]) - X.base : (int64_t)G.n;
    const int64_t i0 = min(ng, id_of(X.f0)), i1 = min(ng, id_of(X.f1));
    X.w0 = X.base + (int32_t)i0;
    X.nw = (int32_t)(i1 - i0);  // at most kBlock
  };
  // part of row v among the unit's ids
  auto part_of = [&](const Unit& X, int32_t v, int32_t& a, int32_t& b) {
    if constexpr (SPLIT) {
      const int32_t* sp = split + (int64_t)v * (nfine + 1);
      a = sp[X.f0];
      b = sp[X.f1];
    } else {
      auto first = [&](int64_t id) {
        int32_t lo = G.gs_off[v], hi = G.gs_off[v + 1];
        while (lo < hi) {
          const int32_t mid = (lo + hi) >> 1;
          if ((int64_t)(G.gs_idx[mid] & kIdMask) < id) lo = mid + 1; else hi = mid;
        }
        return lo;
      };
      a = first(X.base + id_of(X.f0));
      b = first(X.base + id_of(X.f1));
    }
  };
  constexpr int PER = NQ / NW;  // words of the masks per wave
  static_assert(NQ % NW == 0, "whole words per wave");
  auto degrees = [&](const Unit& X, int32_t (&d)[PER]) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int32_t w = (wv + i * NW) * 64 + lane;
      d[i] = w < X.nw ? G.deg[X.w0 + w] : 0;
    }
  };
  // What the next unit starts with (vertex, row, first parts, degrees of its
  // ids) is loaded a step at a time between the phases of the current one, so
  // that those chains of loads run beside it; and the counters are cleared as
  // they are read, so that a unit finds them zero.
  Unit U, V;
  uint32_t ev = 0;
  int32_t pa = 0, pb = 0, dg[PER];
  vertex_of(blockIdx.x, U);
  rows_of(U);
  if (threadIdx.x < kParts && (int32_t)threadIdx.x < U.dm) {
    ev = G.nm_idx[U.ma + threadIdx.x];
    part_of(U, (int32_t)(ev & kIdMask), pa, pb);
  }
  degrees(U, dg);
  for (int i = threadIdx.x; i < 9 * kByteRow / 16; i += NT) reinterpret_cast<uint4*>(bytes)[i] = make_uint4(0, 0, 0, 0);
  for (int i = threadIdx.x; i < 9 * kHubs / 4; i += NT) reinterpret_cast<uint4*>(wide)[i] = make_uint4(0, 0, 0, 0);
  __syncthreads();
  for (int64_t unit = blockIdx.x; unit < units; unit += gridDim.x) {
    vertex_of(unit + gridDim.x < units ? unit + gridDim.x : unit, V);
    const int32_t u = U.u, du = U.du, dm = U.dm, w0 = U.w0, nw = U.nw, nq = (nw + 63) / 64;
    const bool divert = dm > 127;
    if (U.g != cur) {
      if (cur >= 0) give(cur);
      cur = U.g;
    }
    // parts by length: short ones from the front of the list, middle ones from
    // its back, the long ones in a list of their own while it has room
    auto list_part = [&](uint32_t e, int32_t a, int32_t b) {
      const int32_t m = b - a;
      if (m <= 0) return;
      int32_t s = kLongs;
      if (m > kLongPart) s = atomicAdd(&nlong, 1);
      if (s < kLongs) s += kParts;
      else s = m > kShortPart ? kParts - 1 - atomicAdd(&nmid, 1) : atomicAdd(&nshort, 1);
      pt_a[s] = a;
      pt_n[s] = m << 2 | (int32_t)((e >> kTypeShift) - 1u);  // m < 2^28: a row has at most kBlock of a block's ids
    };
    if (threadIdx.x < kParts && (int32_t)threadIdx.x < dm) list_part(ev, pa, pb);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int32_t q = wv + i * NW, w = q * 64 + lane, id = w0 + w, d = dg[i];
      const u64 lo = __ballot(w < nw && (d < du || (d == du && id < u))), hb = __ballot(d > 127);
      if (lane == 0) {
        mlow[q] = lo;
        mhub[q] = hb;
      }
    }
    __syncthreads();
    rows_of(V);
    int32_t nh = 0;
    if (divert) {
      if (wv == 0) {
        int32_t run = 0;
        for (int32_t q0 = 0; q0 < nq; q0 += 64) {
          const int32_t q = q0 + lane, c = q < nq ? __popcll(mhub[q]) : 0;
          int32_t inc = c;
#pragma unroll
          for (int o = 1; o < 64; o <<= 1) {
            const int32_t y = __shfl_up(inc, o);
            if (lane >= o) inc += y;
          }
          if (q < nq) hpre[q] = (uint16_t)(run + inc - c);
          run += __shfl(inc, 63);
        }
        if (lane == 0) nhub = run;
      }
      __syncthreads();
      nh = nhub;
    }
    const bool have = threadIdx.x < kParts && (int32_t)threadIdx.x < V.dm;
    if (have) ev = G.nm_idx[V.ma + threadIdx.x];
    degrees(V, dg);
    for (int32_t h0 = 0; h0 == 0 || h0 < nh; h0 += kHubs) {
      const int32_t nhc = min(kHubs, nh - h0);  // hubs of this pass
      auto hub_at = [&](int32_t w) {  // index of hub w in this pass (any value of kHubs or more: not in it)
        const u64 m = mhub[w >> 6];
        return (uint32_t)((int32_t)hpre[w >> 6] + __popcll(m & ((1ull << (w & 63)) - 1ull)) - h0);
      };
      auto add = [&](uint32_t p, uint32_t f) {  // p, type less one
        const int32_t w = (int32_t)(f & kIdMask) - w0;
        const uint32_t k = 3 * p + (f >> kTypeShift) - 1u;
        if (divert) {
          if ((mhub[w >> 6] >> (w & 63)) & 1ull) {
            const uint32_t h = hub_at(w);
            if (h < (uint32_t)kHubs) atomicAdd(&wide[k * kHubs + h], 1u);
            return;
          }
          if (h0) return;
        }
        atomicAdd(&bytes[(k * kByteRow + (uint32_t)w) >> 2], 1u << (8 * (w & 3)));
      };
      // part s by L lanes, of which this is l, four entries of each at a time;
      // rows start with the same few hubs, so each part is read from another
      // place of it
      auto take = [&](int32_t s, int32_t l, int32_t L) {
        const int32_t a = pt_a[s], mp = pt_n[s], m = mp >> 2, rot = (s * 5) % m;
#pragma unroll 1
        for (int32_t r = l; r < m; r += 4 * L) {
          uint32_t f[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int32_t q = min(r + L * i, m - 1) + rot;
            f[i] = G.gs_idx[a + (q >= m ? q - m : q)];
          }
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (r + L * i < m) add((uint32_t)mp & 3u, f[i]);
        }
      };
      for (int32_t i0 = 0; i0 < dm; i0 += kParts) {
        if (i0 > 0 || h0 > 0) {  // (the first rows were listed ahead)
          const int32_t i = i0 + (int32_t)threadIdx.x;
          if (threadIdx.x < kParts && i < dm) {
            const uint32_t e = G.nm_idx[U.ma + i];
            int32_t a, b;
            part_of(U, (int32_t)(e & kIdMask), a, b);
            list_part(e, a, b);
          }
          __syncthreads();
        }
        const int32_t ns = nshort, nm = nmid, nl = min(nlong, kLongs);
#pragma unroll 1
        for (int32_t k = wv; k < nl; k += NW) take(kParts + k, lane, 64);
#pragma unroll 1
        for (int32_t k = threadIdx.x >> 4; k < nm; k += NT / 16) take(kParts - 1 - k, threadIdx.x & 15, 16);
#pragma unroll 1
        for (int32_t k = threadIdx.x >> 2; k < ns; k += NT / 4) take(k, threadIdx.x & 3, 4);
        __syncthreads();
        if (threadIdx.x == 0) nshort = nmid = nlong = 0;
        if (i0 + kParts < dm || h0 + kHubs < nh) __syncthreads();
      }
      if (h0 == 0 && have) part_of(V, (int32_t)(ev & kIdMask), pa, pb);
      // w of higher rank, and u itself (in every row N(v)), do not count:
      // masked in the byte rows below, cleared among the hubs
      if (nhc > 0) {
#pragma unroll 1
        for (int32_t q = threadIdx.x; q < nq; q += NT)
          for (u64 m = mhub[q] & ~mlow[q]; m; m &= m - 1ull) {
            const uint32_t h = hub_at(q * 64 + __builtin_ctzll(m));
            if (h < (uint32_t)kHubs)
              for (int k = 0; k < 9; ++k) wide[k * kHubs + h] = 0u;
          }
        __syncthreads();
      }
      if (h0 == 0) {
#pragma unroll 2
        for (int32_t q = wv; q < nq; q += NW) {
          v4i x = fld == 9 ? ones : none, y = none;
          if (fld < 9) {
            v4i* p = reinterpret_cast<v4i*>(bytes + (fld * kByteRow + q * 64 + kb * 16) / 4);
            x = *p;
            *p = none;
            const uint32_t m = (uint32_t)(mlow[q] >> (kb * 16)) & 0xFFFFu;
#pragma unroll
            for (int k = 0; k < 4; ++k)  // four mask bits to four mask bytes
              y[k] = x[k] & (int)((((m >> (4 * k)) & 15u) * 0x00204081u & 0x01010101u) * 255u);
          }
          low.acc[0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(y, x, low.acc[0], 0, 0, 0);
        }
        if ((low.run += PER) >= kGramRun) low.flush(bins);
      }
#pragma unroll 1
      for (int32_t q = wv; q < (nhc + 63) / 64; q += NW) {
        v4i x[ND];
#pragma unroll
        for (int a = 0; a < ND; ++a) x[a] = fld == 9 && a == 0 ? ones : none;
        if (fld < 9) {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            uint4* p = reinterpret_cast<uint4*>(wide + fld * kHubs + q * 64 + kb * 16 + 4 * k);
            const uint4 c = *p;
            *p = make_uint4(0, 0, 0, 0);
#pragma unroll
            for (int a = 0; a < ND; ++a)
              x[a][k] = (int)(((c.x >> (7 * a)) & 127u) | ((c.y >> (7 * a)) & 127u) << 8 |
                              ((c.z >> (7 * a)) & 127u) << 16 | ((c.w >> (7 * a)) & 127u) << 24);
          }
        }
#pragma unroll
        for (int a = 0; a < ND; ++a)
#pragma unroll
          for (int b = 0; b <= a; ++b)
            hub.acc[a * (a + 1) / 2 + b] =
                __builtin_amdgcn_mfma_i32_16x16x64_i8(x[a], x[b], hub.acc[a * (a + 1) / 2 + b], 0, 0, 0);
        if (++hub.run >= kGramRun) hub.flush(bins);
      }
      __syncthreads();
    }
    U = V;
  }
  __syncthreads();
  if (cur >= 0) give(cur);
}

// Boundaries of the blocks of a single graph: the multiples of kBlock (nblk + 1
// of them) and the kCuts - 1 inner ends of equal shares of the G* entries,
// merged in order; then the places of the multiples.  One workgroup.
__global__ void k_bounds(DevGraph G, int32_t nblk, int32_t* __restrict__ bnd, const int32_t* st) {
  __shared__ int32_t cut[kCuts];
  if (st[kStatus] != 0) return;
  const int32_t total = G.gs_off[G.n];
  for (int32_t i = threadIdx.x + 1; i < kCuts; i += blockDim.x) {  // cut i: first id with its share of entries before it
    const int64_t key = (int64_t)total * i / kCuts;
    int32_t lo = 0, hi = G.n;
    while (lo < hi) {
      const int32_t mid = (lo + hi) >> 1;
      if (G.gs_off[mid] < key) lo = mid + 1; else hi = mid;
    }
    cut[i] = lo;
  }
  __syncthreads();
  const int32_t nfine = nblk + kCuts - 1;
  auto mult = [&](int32_t j) { return min(G.n, j * kBlock); };
  for (int32_t i = threadIdx.x + 1; i < kCuts; i += blockDim.x) {
    int32_t at = i - 1;  // cuts before it, then the multiples not above it
    for (int32_t j = 0; j <= nblk && mult(j) <= cut[i]; ++j) ++at;
    bnd[at] = cut[i];
  }
  for (int32_t j = threadIdx.x; j <= nblk; j += blockDim.x) {
    int32_t at = j;
    for (int32_t i = 1; i < kCuts && cut[i] < mult(j); ++i) ++at;
    bnd[at] = mult(j);
    bnd[nfine + 1 + j] = at;
  }
}

// split[v * (nfine + 1) + i] = first entry of row v with id >= boundary i of
// its graph.
__global__ void k_split(DevGraph G, int32_t nfine, const int32_t* __restrict__ bnd, int32_t* __restrict__ split,
                        const int32_t* st) {
  if (st[kStatus] != 0) return;
  const int64_t cols = nfine + 1, total = (int64_t)G.n * cols;
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < total; k += (int64_t)gridDim.x * blockDim.x) {
    const int32_t v = (int32_t)(k / cols), i = (int32_t)(k % cols);
    const int64_t id = (G.voff ? G.voff[G.gid[v]] : 0) + (bnd ? (int64_t)bnd[i] : (int64_t)i * kBlock);
    int32_t lo = G.gs_off[v], hi = G.gs_off[v + 1];
    while (lo < hi) {
      const int32_t mid = (lo + hi) >> 1;
      if ((int64_t)(G.gs_idx[mid] & kIdMask) < id) lo = mid + 1; else hi = mid;
    }
    split[k] = lo;
  }
}

// ==================================================== vertices and edges ==
//
// Wedges and claws from the typed degrees of each vertex; P4s from those of
// each edge's ends (the paths whose two ends coincide are taken off with the
// triangles); diamonds from each edge's typed triangle counts.
// Sums stay in registers (a wave's LDS atomics would all hit a handful of
// addresses) and are added up at the end of a graph.
template <bool K3, bool K4>
__global__ __launch_bounds__(256) void k_local(DevGraph G, const uint16_t* __restrict__ lut3,
                                               const uint16_t* __restrict__ lut4, uint64_t* __restrict__ a3,
                                               uint64_t* __restrict__ a4, const uint32_t* __restrict__ T,
                                               const int32_t* st) {
  constexpr int NT = 256, NS = (K3 ? 6 : 0) + (K4 ? 37 : 0), O4 = K3 ? 6 : 0;  // wedges, then claws and P4s
  __shared__ u64 sums[NS], h4[K4 ? 199 : 1];
  __shared__ uint16_t lut[K4 ? 4096 : 1];
  if (st[kStatus] != 0) return;
  const int32_t n = G.n;
  const int64_t items = (int64_t)n + (K4 ? G.np_off[n] : 0);
  const int64_t chunk = (items + gridDim.x - 1) / gridDim.x;  // batch: one run of items per workgroup
  if ((G.gid ? (int64_t)blockIdx.x * chunk : (int64_t)blockIdx.x * NT) >= items) return;
  for (int i = threadIdx.x; i < NS; i += NT) sums[i] = 0;
  if (K4) {
    for (int i = threadIdx.x; i < 199; i += NT) h4[i] = 0;
    for (int i = threadIdx.x; i < 4096; i += NT) lut[i] = lut4[i];
  }
  __syncthreads();
  u64 acc[NS];
#pragma unroll
  for (int i = 0; i < NS; ++i) acc[i] = 0;
  auto flush = [&](int32_t g) {  // every thread
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      u64 v = acc[i];
#pragma unroll
      for (int o = 32; o; o >>= 1) v += __shfl_xor(v, o);
      if ((threadIdx.x & 63) == 0 && v) atomicAdd(&sums[i], v);
      acc[i] = 0;
    }
    __syncthreads();
    const int i = threadIdx.x;
    if (K3 && i < 6) {  // pairs (a, b), a <= b, row-major
      const int a = i < 3 ? 1 : i < 5 ? 2 : 3, b = i < 3 ? i + 1 : i < 5 ? i - 1 : 3;
      gadd(&totals<13, kRep3>(G, a3, g)[lut3[edge_code<3>(0, 1, a) | edge_code<3>(0, 2, b)]], sums[i]);
    }
    if constexpr (K4) {
      if (i < 10) {
        int k = i, a = 1, b = 1, c = 1;
        for (; k; --k) {  // the k-th triple a <= b <= c
          if (c < 3) ++c;
          else if (b < 3) c = ++b;
          else a = b = c = a + 1;
        }
        atomicAdd(&h4[lut[edge_code<4>(0, 1, a) | edge_code<4>(0, 2, b) | edge_code<4>(0, 3, c)]], sums[O4 + i]);
      } else if (i < 37) {
        const int e = i - 10;
        atomicAdd(&h4[lut[edge_code<4>(0, 1, e / 9 + 1) | edge_code<4>(0, 2, (e / 3) % 3 + 1) |
                          edge_code<4>(1, 3, e % 3 + 1)]], sums[O4 + i]);
      }
      __syncthreads();
      for (int k = i; k < 199; k += NT) {
        gadd(&totals<199, kRep4>(G, a4, g)[k], h4[k]);
        h4[k] = 0;
      }
    }
    __syncthreads();
    if (i < NS) sums[i] = 0;
    __syncthreads();
  };
  auto vertex = [&](int32_t v) {
    const uint4 D = G.dt[v];
    const u64 d[4] = {0, D.x, D.y, D.z};
    auto c2 = [](u64 x) { return x * (x - (x > 0)) / 2; };
    if constexpr (K3) {
      int k = 0;
#pragma unroll
      for (int a = 1; a <= 3; ++a)
#pragma unroll
        for (int b = a; b <= 3; ++b, ++k) acc[k] += a == b ? c2(d[a]) : d[a] * d[b];
    }
    if constexpr (K4) {
      auto c3 = [](u64 x) {  // x (x - 1) (x - 2) / 6, x < 2^30: divided before the last product
        if (x < 3) return (u64)0;
        const u64 y = x * (x - 1) / 2;
        return y % 3 == 0 ? y / 3 * (x - 2) : y * ((x - 2) / 3);
      };
      int k = O4;
#pragma unroll
      for (int a = 1; a <= 3; ++a)
#pragma unroll
        for (int b = a; b <= 3; ++b)
#pragma unroll
          for (int c = b; c <= 3; ++c, ++k)
            acc[k] += a == b && b == c ? c3(d[a]) : a == b ? c2(d[a]) * d[c] : b == c ? d[a] * c2(d[b])
                                                                                       : d[a] * d[b] * d[c];
    }
  };
  auto edge = [&](int64_t e) {
    const uint32_t f = G.np_idx[e], t = f >> kTypeShift, tf = flip(t);
    const uint4 X = G.dt[G.np_row[e]], Y = G.dt[f & kIdMask];
    uint32_t c[9], s = 0;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      c[i] = T[e * 9 + i];
      s += c[i];
    }
#pragma unroll
    for (uint32_t p = 1; p <= 3; ++p)
#pragma unroll
      for (uint32_t q = 1; q <= 3; ++q) {
        const u64 w = (u64)(typ(X, p) - (p == t)) * (u64)(typ(Y, q) - (q == tf));
#pragma unroll
        for (uint32_t r = 1; r <= 3; ++r) acc[O4 + 10 + (r - 1) * 9 + (p - 1) * 3 + (q - 1)] += r == t ? w : 0ull;
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
  auto item = [&](int64_t i) {
    if (i < n) vertex((int32_t)i);
    else if constexpr (K4) edge(i - n);
  };
  if (!G.gid) {
    for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < items; i += (int64_t)gridDim.x * NT) item(i);
    flush(0);
    return;
  }
  const int64_t i1 = min(items, (int64_t)(blockIdx.x + 1) * chunk);
  int32_t cur = -1;
  for (int64_t a = (int64_t)blockIdx.x * chunk; a < i1;) {  // up to the end of a graph's vertices or edges
    const int32_t g = G.gid[a < n ? a : (int64_t)G.np_row[a - n]];
    const int64_t b = min(i1, a < n ? G.voff[g + 1] : (int64_t)n + G.np_off[G.voff[g + 1]]);
    if (g != cur) {
      if (cur >= 0) flush(cur);
      cur = g;
    }
    for (int64_t i = a + threadIdx.x; i < b; i += NT) item(i);
    a = b;
  }
  flush(cur);
}

// ================================================================= solve ==
// out[c] = sum of coef * N over row c of the inverse (in CSR form), eight lanes
// per class.  A negative count is a failed self-check, and nothing is written
// then.  One graph: one workgroup computes, checks and writes.
constexpr int kSolve1 = 1024;
template <class P>
__device__ __forceinline__ int64_t solve_row(const P* acc, const SubInverse& M, int32_t c, int l8) {
  int64_t s = 0;
  for (int32_t k = M.off[c] + l8, e = M.off[c + 1]; k < e; k += 8) s += (int64_t)M.coef[k] * (int64_t)acc[M.cls[k]];
#pragma unroll
  for (int o = 4; o; o >>= 1) s += __shfl_xor(s, o);
  return s;
}
__global__ __launch_bounds__(kSolve1) void k_solve_one(const uint64_t* __restrict__ acc, int32_t copies,
                                                       const SubInverse M, uint64_t* __restrict__ out, int32_t C,
                                                       int32_t* st) {
  constexpr int kRows = 2;  // classes per eight lanes: C <= kSolve1 / 8 * kRows
  __shared__ u64 sum[256];
  if (failed(st)) return;
  if (threadIdx.x < 256) sum[threadIdx.x] = 0;
  __syncthreads();
  const int32_t c0 = threadIdx.x & 255;
  if (c0 < C) {
    u64 t = 0;
    for (int32_t r = threadIdx.x >> 8; r < copies; r += kSolve1 / 256) t += acc[(int64_t)r * C + c0];
    if (t) atomicAdd(&sum[c0], t);
  }
  __syncthreads();
  const int l8 = threadIdx.x & 7;
  int64_t v[kRows];
  bool bad = false;
#pragma unroll
  for (int i = 0; i < kRows; ++i) {
    const int32_t c = (int32_t)(threadIdx.x >> 3) + i * (kSolve1 / 8);
    v[i] = c < C ? solve_row(sum, M, c, l8) : 0;
    bad |= v[i] < 0;
  }
  if (__syncthreads_or(bad)) {
    if (threadIdx.x == 0) atomicMin(&st[kStatus], MOTIF_EINTERNAL);
    return;
  }
#pragma unroll
  for (int i = 0; i < kRows; ++i) {
    const int32_t c = (int32_t)(threadIdx.x >> 3) + i * (kSolve1 / 8);
    if (c < C && l8 == 0) out[c] = (uint64_t)v[i];
  }
}
__global__ __launch_bounds__(256) void k_solve(const uint64_t* __restrict__ acc, const SubInverse M,
                                               uint64_t* __restrict__ out, int32_t C, int64_t total, int32_t* st) {
  if (failed(st)) return;
  const int64_t stride = (int64_t)gridDim.x * 32;
  for (int64_t i = blockIdx.x * (int64_t)32 + (threadIdx.x >> 3); i < total; i += stride) {
    const int32_t c = (int32_t)(i % C);
    const int64_t s = solve_row(acc + (i - c), M, c, threadIdx.x & 7);
    if ((threadIdx.x & 7) == 0) {
      if (s < 0) atomicMin(&st[kStatus], MOTIF_EINTERNAL);
      out[i] = (uint64_t)s;
    }
  }
}

__global__ void k_solve_write(const uint64_t* __restrict__ in, uint64_t* __restrict__ out, int64_t total,
                              const int32_t* st) {
  if (failed(st)) return;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x)
    out[i] = in[i];
}

unsigned grid_of(int64_t items, int per, int64_t most) {
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>(most, (items + per - 1) / per));
}

// ------------------------------------------------------------------ sizes --

constexpr int64_t kSplitCap = int64_t(64) << 20;  // entries of the row-split table (256 MB), beyond that binary searches
// Adjacency slices of k_tri_big: 64 MB, or 16 bytes an arc (a slice's room is for
// the largest d+ that m allows, 520 KB at m = 10^6 and 5 MB at 10^7).
constexpr size_t kPlaneBytes = size_t(64) << 20, kPlaneArc = 16;

struct CountPlan {
  bool wide;                 // degrees may reach 2^21
  int32_t nblk, nfine;       // blocks of ids of k_wedge_top, and with the shares of entries
  bool split, far;
  int64_t D, words;          // bound on d+ and the words of an adjacency row
  int slices;                // adjacency slices of k_tri_big in global memory (0: none can be needed)
};

CountPlan count_plan(int64_t n, int64_t m, int64_t maxn, bool batch) {
  CountPlan c{};
  const int64_t mg = maxn > 0 ? maxn : n;
  c.wide = std::min(mg - 1, m) >= (int64_t(1) << 21);
  c.nblk = (int32_t)std::max<int64_t>(1, (mg + kBlock - 1) / kBlock);
  c.nfine = c.nblk + (!batch && m >= kCutsM ? kCuts - 1 : 0);
  c.split = n * (c.nfine + 1) <= kSplitCap;
  c.far = c.nblk > kFarBlocks;
  // N+(x) has at most sqrt(2 m*) entries: its members all have degree d(x) or more
  int64_t r = 1;
  while (r * r <= 2 * m) ++r;
  c.D = std::max<int64_t>(1, std::min(mg, r));
  c.words = (c.D + 63) / 64;
  const size_t per = (size_t)c.D * (size_t)c.words * 16;
  c.slices = c.D > kPlaneD ? (int)std::max<size_t>(1, std::min<size_t>(256, std::max(kPlaneBytes, kPlaneArc * (size_t)m) / per)) : 0;
  return c;
}

}  // namespace

size_t count_bytes(int64_t n, int64_t m, int64_t maxn, bool batch, bool k4) {
  auto al = [](size_t b) { return (b + 255) & ~size_t(255); };
  if (!k4) return 0;
  const CountPlan c = count_plan(n, m, maxn, batch);
  size_t b = al(sizeof(uint32_t) * 9 * (size_t)(m + 1)) + (c.far ? 7 : 5) * al(sizeof(int32_t) * (size_t)(n + 1));
  if (c.split) b += al(sizeof(int32_t) * (size_t)n * (c.nfine + 1));
  b += al(sizeof(int32_t) * (size_t)(c.nfine + c.nblk + 2));
  b += al((size_t)c.slices * (size_t)c.D * (size_t)c.words * 16 + 16);
  return b;
}

// The wedges, and (k_local) the vertices and edges, of a k = 4 pass: the latter
// on ts, behind the triangles that they need.
static void enqueue_wedges(Pipeline& p, const DevGraph& g, uint64_t* a3, uint64_t* a4, const int32_t* queue,
                           const CountsOut& o, hipStream_t s, hipStream_t ts) {
  const DevTables& T = dev_tables();
  const int64_t n = g.n, m = (g.gs_cap - 1) / 2;
  const int cus = p.num_cus;
  const CountPlan c = count_plan(n, m, g.max_graph_n, g.gid != nullptr);
  const int64_t n16 = std::min(n, m);
  auto list_grid = [&](int64_t most, int per, int wgs) { return dim3(grid_of(most, per, (int64_t)cus * wgs)); };
  // (the diamonds need the triangles only)
  const dim3 lgrid(grid_of(n + m, 256, cus * 4));
  if (a3)
    hipLaunchKernelGGL((k_local<true, true>), lgrid, dim3(256), 0, ts, g, T.lut[3], T.lut[4], a3, a4, o.T, p.status);
  else
    hipLaunchKernelGGL((k_local<false, true>), lgrid, dim3(256), 0, ts, g, T.lut[3], T.lut[4], a3, a4, o.T, p.status);
  hipLaunchKernelGGL((k_wedge<16, 7>), list_grid(n16, 16, 6), dim3(256), 0, s, g, T.lut[4], a4, p.status, queue,
                     o.wedge[kWedge16]);
  if (2 * m > kCap16)
    hipLaunchKernelGGL((k_wedge<64, 9>), list_grid(n16, 4, 6), dim3(256), 0, s, g, T.lut[4], a4, p.status, queue,
                       o.wedge[kWedge64]);
  if (2 * m > kCap64)
    hipLaunchKernelGGL((k_wedge<256, 12>), list_grid(n16, 1, 3), dim3(256), 0, s, g, T.lut[4], a4, p.status, queue,
                       o.wedge[kWedge256]);
  if (c.far) {
    hipLaunchKernelGGL((k_wedge_far<13, 7>), list_grid(n16, 1, 1), dim3(1024), 0, s, g, T.lut[4], a4, p.status, queue,
                       o.wedge[kWedgeFar7]);
    hipLaunchKernelGGL((k_wedge_far<12, 11>), list_grid(n16, 1, 1), dim3(1024), 0, s, g, T.lut[4], a4, p.status, queue,
                       o.wedge[kWedgeFar11]);
  }
  if (m > 127) {  // over 127 lower neighbours, or over kCap256 visits
    if (o.bnd) hipLaunchKernelGGL(k_bounds, dim3(1), dim3(64), 0, s, g, c.nblk, o.bnd, p.status);
    if (o.split)
      hipLaunchKernelGGL(k_split, dim3(grid_of(n * (c.nfine + 1), 256, 65536)), dim3(256), 0, s, g, c.nfine, o.bnd, o.split,
                         p.status);
    const dim3 tg = list_grid(n * c.nfine, 1, 1);
    auto launch_top = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, tg, dim3(kTopThreads), 0, s, g, T.lut[4], a4, p.status, queue, o.wedge[kWedgeTop],
                         o.wedge[kWedgeHuge], o.split, c.nblk, c.nfine, o.bnd);
    };
    if (c.wide) launch_top(o.split ? k_wedge_top<5, true> : k_wedge_top<5, false>);
    else launch_top(o.split ? k_wedge_top<3, true> : k_wedge_top<3, false>);
  }
}

void enqueue_counts(Pipeline& p, const DevGraph& g, uint64_t* a3, uint64_t* a4, int32_t* queue, hipStream_t s,
                    CountsOut* left) {
  // (the accumulators and the queue words are zeroed by the caller)
  const DevTables& T = dev_tables();
  const int64_t n = g.n, m = (g.gs_cap - 1) / 2;
  if (n == 0) return;
  const int cus = p.num_cus;
  const CountPlan c = count_plan(n, m, g.max_graph_n, g.gid != nullptr);
  // A vertex with more than 128 higher neighbours has a workgroup to itself; on a
  // dense graph of a vertex or two per CU also one with more than 40, where a
  // wave alone would be the whole call (n = 150, three quarters of the arcs:
  // 4,283 us so, 795 us with a workgroup; n = 200, a fifth of the arcs or fewer,
  // has no such vertices to speak of and the further launch costs 10 to 20 us).
  const int32_t big = a4 && !g.gid && n <= 2 * cus && 5 * m > n * (n - 1) ? 41 : 129;
  // lists in words that the build is done with (at most 2 m / 17 vertices have
  // a degree of 17 or more, 2 m / 65 one of 65)
  Lists L{};
  L.v[kTri16] = g.tmp_n;
  L.v[kTri64] = g.tmp_n2;
  L.v[kTri128] = g.tmp_n3;
  L.v[kTriBig] = g.tmp_n3 + m;
  const unsigned cgrid = std::max(grid_of(n, 64, cus * 4), grid_of(n, kClassify, 1 << 20));
  // workgroups for a list of at most `most` vertices, `per` at a time
  auto list_grid = [&](int64_t most, int per, int wgs) { return dim3(grid_of(most, per, (int64_t)cus * wgs)); };
  // a vertex of tier d has at least d higher neighbours of at least its degree
  const int64_t n16 = std::min(n, m), n64 = std::min(n, 2 * m / 17);
  const int64_t n128 = c.D > 64 && big > 65 ? std::min(n, 2 * m / 65) : 0;
  const int64_t nbig = c.D >= big ? std::min(n, 2 * m / big) : 0;
  if (!a4) {
    hipLaunchKernelGGL((k_classify<false>), dim3(cgrid), dim3(256), 0, s, g, L, queue, big, (int32_t)c.far, p.status);
    hipLaunchKernelGGL((k_tri<16, 16, false>), list_grid(n16, 16, 8), dim3(256), 0, s, g, T.lut[3], T.lut[4], a3, nullptr,
                       nullptr, p.status, queue, L.v[kTri16]);
    if (c.D > 16)
      hipLaunchKernelGGL((k_tri<64, 64, false>), list_grid(n64, 4, 8), dim3(256), 0, s, g, T.lut[3], T.lut[4], a3, nullptr,
                         nullptr, p.status, queue, L.v[kTri64]);
    if (n128 > 0)
      hipLaunchKernelGGL((k_tri<64, 128, false>), list_grid(n128, 4, 8), dim3(256), 0, s, g, T.lut[3], T.lut[4], a3,
                         nullptr, nullptr, p.status, queue, L.v[kTri128]);
    if (nbig > 0)
      hipLaunchKernelGGL((k_tri_big<false>), list_grid(nbig, 1, 3), dim3(512), 0, s, g, T.lut[3], T.lut[4], a3,
                         nullptr, nullptr, p.status, queue, L.v[kTriBig], nullptr, 0, 0, 0, INT32_MAX);
    hipLaunchKernelGGL((k_local<true, false>), dim3(grid_of(n, 256, cus * 4)), dim3(256), 0, s, g, T.lut[3], T.lut[4],
                       a3, nullptr, nullptr, p.status);
    return;
  }
  uint32_t* Te = p.arena.take<uint32_t>(9 * (size_t)(m + 1));
  for (int l = kWedge16; l <= (c.far ? kWedgeFar11 : kWedgeHuge); ++l) L.v[l] = p.arena.take<int32_t>((size_t)n + 1);
  int32_t* split = c.split ? p.arena.take<int32_t>((size_t)n * (c.nfine + 1)) : nullptr;
  int32_t* bnd = p.arena.take<int32_t>((size_t)(c.nfine + c.nblk + 2));
  if (c.nfine == c.nblk) bnd = nullptr;  // the multiples of kBlock alone
  u64* planes = p.arena.take<u64>((size_t)c.slices * (size_t)c.D * (size_t)c.words * 2 + 1);
  CountsOut own;
  CountsOut* const out = left ? left : &own;
  out->T = Te;
  out->split = split;
  out->bnd = bnd;
  for (int l = 0; l < kLists; ++l) out->wedge[l] = L.v[l];
  enqueue_zero(Te, sizeof(uint32_t) * 9 * (size_t)(m + 1), s);
  hipLaunchKernelGGL((k_classify<true>), dim3(cgrid), dim3(256), 0, s, g, L, queue, big, (int32_t)c.far, p.status);
  // The triangles beside the wedges where both are long (n = 10^5, m = 10^6: 450
  // and 1,030 us) and the caller's streams allow it.  Beside the hashed wedges,
  // that is: a workgroup of k_wedge_top has a CU to itself (161,440 of 163,840
  // bytes of LDS, 16 waves of 128 registers), and takes each as the triangles
  // leave it.
  Chains ch(p, s);
  if (p.fork_now && m >= kCutsM && !out->later) ch.fork(0);
  const hipStream_t ts = ch.on(0);
  hipLaunchKernelGGL((k_tri<16, 16, true>), list_grid(n16, 16, 6), dim3(256), 0, ts, g, T.lut[3], T.lut[4], a3, a4, Te,
                     p.status, queue, L.v[kTri16]);
  if (c.D > 16)
    hipLaunchKernelGGL((k_tri<64, 64, true>), list_grid(n64, 4, 6), dim3(256), 0, ts, g, T.lut[3], T.lut[4], a3, a4, Te,
                       p.status, queue, L.v[kTri64]);
  if (n128 > 0)
    hipLaunchKernelGGL((k_tri<64, 128, true>), list_grid(n128, 4, 3), dim3(256), 0, ts, g, T.lut[3], T.lut[4], a3, a4,
                       Te, p.status, queue, L.v[kTri128]);
  if (nbig > 0) {
    // A workgroup whose x need a global slice has its own.  With slices for less
    // than a quarter of the workgroups the x that need none are a launch of all of
    // them (m = 10^7 of n = 5 * 10^4, up to 220 higher neighbours: 528 ms by the 12
    // workgroups of the slices, 280 so; at 129 slices of 512 neither gains).
    const unsigned all = grid_of(nbig, 1, cus * 2), few = c.slices ? std::min<unsigned>(c.slices, all) : all;
    auto launch = [&](unsigned grid, int32_t above, int32_t most) {
      hipLaunchKernelGGL((k_tri_big<true>), dim3(grid), dim3(512), 0, ts, g, T.lut[3], T.lut[4], a3, a4, Te, p.status,
                         queue, L.v[kTriBig], planes, c.D, c.words, above, most);
    };
    const bool split = 4 * few < all;
    if (split) launch(all, 0, kPlaneD);
    launch(few, split ? kPlaneD : 0, INT32_MAX);
  }
  if (out->later) return;  // (not forked)
  enqueue_wedges(p, g, a3, a4, queue, *out, s, ts);
  ch.join();
}

void enqueue_counts_rest(Pipeline& p, const DevGraph& g, uint64_t* a3, uint64_t* a4, const int32_t* queue,
                         const CountsOut& left, hipStream_t s) {
  enqueue_wedges(p, g, a3, a4, queue, left, s, s);
}

void enqueue_solve(int k, const uint64_t* acc, uint64_t* tmp, uint64_t* out, int64_t ngraphs, int32_t* status,
                   hipStream_t s) {
  const int C = num_classes(k);
  const int64_t total = ngraphs * C;
  if (ngraphs == 1) {
    hipLaunchKernelGGL(k_solve_one, dim3(1), dim3(kSolve1), 0, s, acc, k == 3 ? kRep3 : kRep4,
                       dev_tables().inv[k], out, C, status);
    return;
  }
  hipLaunchKernelGGL(k_solve, dim3(grid_of(total, 32, 65536)), dim3(256), 0, s, acc, dev_tables().inv[k], tmp, C, total,
                     status);
  hipLaunchKernelGGL(k_solve_write, dim3(grid_of(total, 256, 65536)), dim3(256), 0, s, tmp, out, total, status);
}

}  // namespace motif
