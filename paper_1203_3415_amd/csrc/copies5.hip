// k = 5 census of one graph by counting typed subgraph copies (gfx950, wave64).
//
// As for k = 3 and 4 (counts.hip): the number N(c) of copies of every class c,
// whatever the pairs that are no edges of c look like, has closed forms over
// small local counts, and the induced counts follow from the N by inclusion and
// exclusion over edges.  The 21 graphs on five vertices fall into four groups:
//   trees             typed degrees, and their sums over a vertex's neighbours
//                     (k_vertex5)
//   graphs with a vertex u joined to the other four   pairs, paths, stars,
//                     triangles .. of the edges among N(u), that is of the
//                     triangles at u; with them bull, kite and triangle with a
//                     path, which hang on a triangle too (k_apex5, k_wheel5,
//                     k_butterfly5)
//   graphs on a C4 u v w v'   typed wedges W between u and every w: pairs and
//                     triples of them, weighted with degrees and with the
//                     triangles on their edges (k_pairs5)
//   C5                typed wedges from its vertex u of highest rank to w and
//                     w', the ends of an edge (k_c5)
// A sum may meet a copy several times (Copies5::mult), and some take in
// walks that fold onto four or three vertices; the number of those is a fixed
// combination of the k = 3 and 4 copies and is taken off at the end (k_sum5).
//
// Work: the wedges (sum of d(v)^2), the triangles, pairs of triangles on an
// edge, and for C5 the edges among the vertices that lie two steps below u.  On
// the n = 20,000, m = 100,000 power-law graph these are 2.5e7, 1.9e4, 2.7e5 and
// 5.8e6; the per-core scan (kr_kernel) takes all 1.3e7 connected triples and
// 1.4e8 row visits for them, in 40 ms.
//
// The thirds z of each edge (u, b) are kept as a row of "links" per G* entry,
// six entries per triangle.  Their number is only known once the triangles are
// counted: the host reads it (and the longest row) and leaves graphs with more
// than the room for them to kr_kernel.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "codes.h"
#include "counts.h"
#include "internal.h"
#include "scan.h"

namespace motif {

namespace {

constexpr int kC5 = 9364;
constexpr int kLocalCopies = 256;        // copies written by k_apex5, at most
// Lists of vertices by their wedge table in k_pairs5.
enum PairList : int { kPair9 = 0, kPair10 = 1, kPair11 = 2, kPair12 = 3, kPair13 = 4, kPairBlock = 5, kPairLists = 6 };
constexpr int kPairQueue = 16, kPairCursor = 24;  // queue words of the pair lists, and of the pulls
// visits of a vertex in a hash of 2^HB words
constexpr int pair_cap(int HB) { return (1 << HB) * 3 / 4; }

struct Links {
  const uint32_t* emap;  // per G* entry (u, b): N+ position of the edge << 1 | u is its higher end
  const int32_t* cnt;    // its triangles
  const int32_t* off;    // its first link
  const uint32_t* idx;   // link: place of the third z in u's row | type of z seen from b
  const int32_t* mate;   // G* entry (b, z)
  const int32_t* src;    // G* entry (u, b)
  const uint32_t* T;     // per N+ entry: typed triangle counts (counts.hip)

  // T of G* entry E as t[3 (type of the third seen from u - 1) + (from b) - 1]
  __device__ __forceinline__ void types(int32_t E, uint32_t (&t)[9]) const {
    const uint32_t m = emap[E];
    const uint32_t* p = T + (int64_t)(m >> 1) * 9;
#pragma unroll
    for (int i = 0; i < 9; ++i) t[i] = p[(m & 1u) ? (i % 3) * 3 + i / 3 : i];
  }
};

// Totals that the workgroups share, a few copies of them (a power of two; see
// totals() in counts.hip).
struct Totals5 {
  const uint16_t* lut;
  uint64_t* acc;
  int copies;
  __device__ __forceinline__ void add(uint32_t code, u64 w) const {
    if (w) atomicAdd(reinterpret_cast<u64*>(acc) + (int64_t)((int)blockIdx.x & (copies - 1)) * kC5 + lut[code], w);
  }
  // N of them, the table's entries loaded together
  template <int N>
  __device__ __forceinline__ void add(const uint32_t (&code)[N], const u64 (&w)[N]) const {
    uint32_t c[N];
#pragma unroll
    for (int i = 0; i < N; ++i) c[i] = lut[code[i]];
    u64* a = reinterpret_cast<u64*>(acc) + (int64_t)((int)blockIdx.x & (copies - 1)) * kC5;
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (w[i]) atomicAdd(a + c[i], w[i]);
  }
};

// The totals of one workgroup in LDS, for the kernels that add millions of small
// numbers all over the classes (additions in global memory: 4 per ns on the whole
// chip), and their own copy of the totals in memory, written at the end.
struct Local5 {
  const uint16_t* lut;
  u64* sum;  // [kC5] in LDS
  __device__ __forceinline__ void clear() const {
    for (int i = threadIdx.x; i < kC5; i += blockDim.x) sum[i] = 0;
    __syncthreads();
  }
  __device__ __forceinline__ void add(uint32_t code, u64 w) const {
    if (w) atomicAdd(&sum[lut[code]], w);
  }
  template <int N>
  __device__ __forceinline__ void add(const uint32_t (&code)[N], const u64 (&w)[N]) const {
    uint32_t c[N];
#pragma unroll
    for (int i = 0; i < N; ++i) c[i] = lut[code[i]];
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (w[i]) atomicAdd(&sum[c[i]], w[i]);
  }
  __device__ __forceinline__ void write(uint64_t* copies, int copy) const {
    __syncthreads();
    for (int i = threadIdx.x; i < kC5; i += blockDim.x) copies[(int64_t)copy * kC5 + i] = sum[i];
  }
};

__device__ __forceinline__ uint32_t ec(int i, int j, uint32_t t) { return edge_code<5>(i, j, t); }

__device__ __forceinline__ uint32_t deg_of(const uint4& d, int s) { return s == 0 ? d.x : s == 1 ? d.y : d.z; }

// Neighbours of type s + 1 apart from the ones of types a, b, c (0: none).
__device__ __forceinline__ u64 other(const uint4& d, int s, uint32_t a, uint32_t b, uint32_t c = 0) {
  const uint32_t t = s + 1;
  return (u64)(deg_of(d, s) - (a == t) - (b == t) - (c == t));
}

__device__ __forceinline__ int32_t find_in(const uint32_t* idx, int32_t lo, int32_t hi, uint32_t id) {
  while (lo < hi) {
    const int32_t mid = (lo + hi) >> 1;
    if ((idx[mid] & kIdMask) < id) lo = mid + 1; else hi = mid;
  }
  return lo;
}

// Whether k_c5 starts from w.
__device__ __forceinline__ bool two_lower(const DevGraph& G, int32_t w) {
  return G.deg[w] - (G.np_off[w + 1] - G.np_off[w]) >= 2;
}

// ================================================================= links ==

// Per edge: its two G* entries, its triangles, and the higher neighbours of its
// lower end that lie above its higher end, by type (hi[6 e ..]), and those of
// them that k_c5 starts from, having two lower neighbours or more (hi[6 e + 3
// ..]).  st + 8: sum
// of the triangles over the G* entries (64 bits); st + 10: the most at one; st +
// 11: vertices of k_c5_fill.
__global__ __launch_bounds__(256) void k_edges5(DevGraph G, const uint32_t* __restrict__ T, uint32_t* __restrict__ emap,
                                                int32_t* __restrict__ cnt, int32_t* __restrict__ epos,
                                                uint32_t* __restrict__ hi, const int32_t* __restrict__ queue,
                                                int32_t* st) {
  __shared__ u64 sum;
  __shared__ int32_t most;
  if (st[kStatus] != 0) return;
  if (threadIdx.x == 0) {
    sum = 0;
    most = 0;
    if (blockIdx.x == 0) st[11] = queue[kWedgeTop] + queue[kWedgeHuge];
  }
  __syncthreads();
  const int32_t ne = G.np_off[G.n];
  u64 s = 0;
  int32_t mx = 0;
  for (int32_t e = blockIdx.x * 256 + threadIdx.x; e < ne; e += gridDim.x * 256) {
    const int32_t x = G.np_row[e], y = (int32_t)(G.np_idx[e] & kIdMask);
    int32_t t = 0;
#pragma unroll
    for (int i = 0; i < 9; ++i) t += (int32_t)T[(int64_t)e * 9 + i];
    const int32_t E1 = find_in(G.gs_idx, G.gs_off[x], G.gs_off[x + 1], (uint32_t)y);
    const int32_t E2 = find_in(G.gs_idx, G.gs_off[y], G.gs_off[y + 1], (uint32_t)x);
    emap[E1] = (uint32_t)e << 1;
    emap[E2] = (uint32_t)e << 1 | 1u;
    cnt[E1] = cnt[E2] = t;
    epos[2 * e] = E1;
    epos[2 * e + 1] = E2;
    if (t) {
      s += 2 * (u64)t;
      mx = max(mx, t);
      uint32_t h[6] = {0, 0, 0, 0, 0, 0};
      const uint32_t dy = (uint32_t)G.deg[y];
      for (int32_t j = G.np_off[x], b = G.np_off[x + 1]; j < b; ++j) {
        const uint32_t f = G.np_idx[j];
        const int32_t w = (int32_t)(f & kIdMask);
        if (w != y && ranked_below(G, dy, y, (uint32_t)G.deg[w], w)) {
          const uint32_t ty = f >> kTypeShift;
          const bool two = two_lower(G, w);
#pragma unroll
          for (int i = 0; i < 3; ++i) {
            h[i] += ty == (uint32_t)i + 1;
            h[3 + i] += two && ty == (uint32_t)i + 1;
          }
        }
      }
#pragma unroll
      for (int i = 0; i < 6; ++i) hi[(int64_t)e * 6 + i] = h[i];
    }
  }
  if (s) {
    atomicAdd(&sum, s);
    atomicMax(&most, mx);
  }
  __syncthreads();
  if (threadIdx.x == 0 && sum) {
    atomicAdd(reinterpret_cast<u64*>(st + 8), sum);
    atomicMax(st + 10, most);
  }
}

struct LinkCount {
  const int32_t* cnt;
  const int32_t* gs_off;
  int32_t n;
  __device__ __forceinline__ int32_t operator()(int64_t i) const { return i < gs_off[n] ? cnt[i] : 0; }
};

// Fills the links, one wave per edge with triangles: the shorter end's row
// against the longer one's, in order, so that a link row is sorted.  Each
// triangle is met at its three edges; per edge (x, y) the typed triangle of the
// third vertex is counted, and at the edge opposite its lowest vertex the walks
// that k_c5 takes in with it: five steps from a vertex u above the rest and
// back that pass a vertex twice.
__global__ __launch_bounds__(256) void k_links5(DevGraph G, Totals5 K, Links L, const int32_t* __restrict__ epos,
                                                const uint32_t* __restrict__ hi, const uint4* __restrict__ up,
                                                uint32_t* __restrict__ idx, int32_t* __restrict__ mate,
                                                int32_t* __restrict__ src, uint32_t* __restrict__ tri, const int32_t* st) {
  if (st[kStatus] != 0) return;
  const int lane = threadIdx.x & 63;
  const int32_t ne = G.np_off[G.n], nw = gridDim.x * 4, w0 = blockIdx.x * 4 + (threadIdx.x >> 6);
  for (int64_t base = w0; base < ne; base += (int64_t)nw * 64) {
    const int64_t el = base + (int64_t)lane * nw;
    u64 todo = __ballot(el < ne && L.cnt[epos[2 * (el < ne ? el : 0)]] > 0);
    for (; todo; todo &= todo - 1ull) {
      const int32_t e = (int32_t)(base + (int64_t)__builtin_ctzll(todo) * nw);
      const uint32_t xy = G.np_idx[e] >> kTypeShift;
      const int32_t x = G.np_row[e], y = (int32_t)(G.np_idx[e] & kIdMask);
      const int32_t xa = G.gs_off[x], ya = G.gs_off[y], dx = G.gs_off[x + 1] - xa, dy = G.gs_off[y + 1] - ya;
      const int32_t o1 = L.off[epos[2 * e]], o2 = L.off[epos[2 * e + 1]];
      const bool sx = dx <= dy;  // x's row is streamed
      const int32_t sa = sx ? xa : ya, sd = sx ? dx : dy, oa = sx ? ya : xa, od = sx ? dy : dx;
      int32_t run = 0;
      for (int32_t i0 = 0; i0 < sd; i0 += 64) {
        const int32_t i = i0 + lane;
        int32_t px = -1, py = -1, z = -1;
        if (i < sd) {
          z = (int32_t)(G.gs_idx[sa + i] & kIdMask);
          const int32_t q = find_in(G.gs_idx, oa, oa + od, (uint32_t)z);
          if (q < oa + od && (int32_t)(G.gs_idx[q] & kIdMask) == z) {
            px = sx ? sa + i : q;
            py = sx ? q : sa + i;
          }
        }
        const u64 hit = __ballot(px >= 0);
        if (px >= 0) {
          const int32_t k = run + __popcll(hit & ((1ull << lane) - 1ull));
          const uint32_t tx = G.gs_idx[px] >> kTypeShift, ty = G.gs_idx[py] >> kTypeShift;
          idx[o1 + k] = (uint32_t)(px - xa) | ty << kTypeShift;
          mate[o1 + k] = py;
          src[o1 + k] = epos[2 * e];
          idx[o2 + k] = (uint32_t)(py - ya) | tx << kTypeShift;
          mate[o2 + k] = px;
          src[o2 + k] = epos[2 * e + 1];
          const uint32_t p = flip(tx), q = flip(ty);
          const uint32_t c1 = (p - 1) * 9 + (q - 1) * 3 + (xy - 1), c2 = (q - 1) * 9 + (p - 1) * 3 + (flip(xy) - 1);
          atomicAdd(&tri[(int64_t)z * 27 + min(c1, c2)], 1u);
          if (ranked_below(G, (uint32_t)G.deg[z], z, (uint32_t)dx, x)) {  // z < x < y
            const uint32_t zx = p, zy = q;
            const uint32_t* hzy = hi + 6 * (int64_t)(L.emap[py] >> 1);
            const uint32_t* hxy = hi + 6 * (int64_t)e;
            const uint4 Uy = up[y], Dz = G.dt[z], Dx = G.dt[x];
            uint32_t code[16];
            u64 w[16];
            // u above all three, joined to corner v: u v w w' v
            auto walk_a = [&](int at, uint32_t n, int s, uint32_t vw, uint32_t ww, uint32_t wv) {
              const uint32_t t = s + 1;
              code[at] = ec(0, 1, flip(t)) | ec(1, 2, vw) | ec(2, 3, ww) | ec(3, 4, wv) | ec(4, 0, t);
              w[at] = 0 - (u64)n;
            };
            // u = y: u c w c o, w below u
            auto walk_b = [&](int at, u64 n, int s, uint32_t uc, uint32_t co, uint32_t ou) {
              const uint32_t t = s + 1;
              code[at] = ec(0, 1, uc) | ec(1, 2, t) | ec(2, 3, flip(t)) | ec(3, 4, co) | ec(4, 0, ou);
              w[at] = 0 - n;
            };
#pragma unroll
            for (int s = 0; s < 3; ++s) {
              walk_a(5 * s, hzy[3 + s], s, zx, xy, flip(zy));
              walk_a(5 * s + 1, hxy[3 + s], s, flip(zx), zy, flip(xy));
              walk_a(5 * s + 2, deg_of(Uy, s), s, flip(zy), zx, xy);
              walk_b(5 * s + 3, other(Dz, s, zy, zx) - hzy[s], s, flip(zy), zx, xy);
              walk_b(5 * s + 4, other(Dx, s, xy, flip(zx)) - hxy[s], s, flip(xy), flip(zx), zy);
            }
            code[15] = ec(0, 1, flip(zy)) | ec(1, 2, zx) | ec(2, 3, flip(zx)) | ec(3, 4, zx) | ec(4, 0, xy);
            w[15] = 0 - 1ull;
            K.add(code, w);
          }
        }
        run += __popcll(hit);
      }
    }
  }
}

// ================================================================= trees ==

// The three trees from the typed degrees around each vertex, one wave per
// vertex: S[3 t + s] = sum over its neighbours of type t of their other
// neighbours of type s, Q the same of products.  Also up: its higher neighbours
// by type, those that k_c5 starts from.
__global__ __launch_bounds__(256) void k_vertex5(DevGraph G, Totals5 K, u64* __restrict__ S, uint4* __restrict__ up,
                                                 const int32_t* st) {
  constexpr int kStar = 15, kPath = 45, kFork = 54, NB = kStar + kPath + kFork;
  __shared__ u64 bins[NB], vals[4][27];
  __shared__ uint32_t dv[4][3];
  if (st[kStatus] != 0) return;
  for (int i = threadIdx.x; i < NB; i += 256) bins[i] = 0;
  __syncthreads();
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  u64* val = vals[wv];
  uint32_t* d = dv[wv];
  constexpr int kPair[6][2] = {{0, 0}, {0, 1}, {0, 2}, {1, 1}, {1, 2}, {2, 2}};
  // item -> the types or sums it takes
  auto star_of = [](int i, int (&k)[3]) {
    int j = i;
    for (k[0] = 0; j > 4 - k[0]; ++k[0]) j -= 5 - k[0];
    k[1] = j;
    k[2] = 4 - k[0] - k[1];
  };
  auto path_of = [](int i, int& a, int& b) {
    for (a = 0; i >= 9 - a; ++a) i -= 9 - a;
    b = a + i;
  };
  for (int32_t v = blockIdx.x * 4 + wv; v < G.n; v += gridDim.x * 4) {
    const int32_t a = G.gs_off[v], b = G.gs_off[v + 1];
    u64 acc[27];
#pragma unroll
    for (int i = 0; i < 27; ++i) acc[i] = 0;
    uint32_t hi[3] = {0, 0, 0};
    const uint4 D = G.dt[v];
    for (int32_t j = a + lane; j < b; j += 64) {
      const uint32_t f = G.gs_idx[j], t = f >> kTypeShift, tf = flip(t);
      const int32_t w = (int32_t)(f & kIdMask);
      const uint4 Dw = G.dt[w];
      const bool above = ranked_below(G, D.w, v, Dw.w, w);
      u64 x[3];
#pragma unroll
      for (int s = 0; s < 3; ++s) {
        x[s] = other(Dw, s, tf, 0);
        hi[s] += above && t == (uint32_t)s + 1 && two_lower(G, w);
      }
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (t == (uint32_t)k + 1) {
#pragma unroll
          for (int s = 0; s < 3; ++s) acc[3 * k + s] += x[s];
#pragma unroll
          for (int s = 0; s < 6; ++s) acc[9 + 6 * k + s] += x[kPair[s][0]] * x[kPair[s][1]];
        }
    }
    const int32_t top = b - a >= 64 ? 32 : b - a > 32 ? 32 : b - a > 16 ? 16 : b - a > 8 ? 8 : b - a > 4 ? 4 : b - a > 2 ? 2 : 1;
#pragma unroll
    for (int i = 0; i < 27; ++i) {
      for (int o = top; o; o >>= 1) acc[i] += __shfl_xor(acc[i], o);
      if (lane == 0) val[i] = acc[i];
    }
#pragma unroll
    for (int s = 0; s < 3; ++s)
      for (int o = top; o; o >>= 1) hi[s] += __shfl_xor(hi[s], o);
    if (lane == 0) {
      up[v] = make_uint4(hi[0], hi[1], hi[2], 0u);
      d[0] = D.x;
      d[1] = D.y;
      d[2] = D.z;
    }
    wave_sync();
    if (lane < 9) S[(int64_t)v * 9 + lane] = val[lane];
    for (int i = lane; i < NB; i += 64) {
      u64 w = 1;
      if (i < kStar) {
        int k[3];
        star_of(i, k);
        for (int s = 0; s < 3; ++s) {
          const u64 x = d[s];
          const int c = k[s];
          if ((u64)c > x) w = 0;
          else if (c) w *= c == 1 ? x : c == 2 ? x * (x - 1) / 2 : c == 3 ? x * (x - 1) * (x - 2) / 6 : x * (x - 1) * (x - 2) * (x - 3) / 24;
        }
      } else if (i < kStar + kPath) {
        int p, q;
        path_of(i - kStar, p, q);
        const int t = p / 3, s1 = p % 3, s2 = q % 3;
        w = val[p] * val[q];
        if (q / 3 == t) {
          const int lo = min(s1, s2), hh = max(s1, s2);
          w -= val[9 + 6 * t + (lo == 0 ? hh : lo == 1 ? hh + 2 : 5)];
        }
        if (p == q) w /= 2;
      } else {
        const int k = i - kStar - kPath, p = k / 6, q = k % 6, t = p / 3, s1 = kPair[q][0], s2 = kPair[q][1];
        const u64 x = d[s1] - (s1 == t), y = d[s2] - (s2 == t);
        w = val[p] ? val[p] * (s1 == s2 ? x * (x - 1) / 2 : x * y) : 0ull;
      }
      if (w) atomicAdd(&bins[i], w);
    }
    wave_sync();
  }
  __syncthreads();
  for (int i = threadIdx.x; i < NB; i += 256) {
    uint32_t code = 0;
    if (i < kStar) {
      int k[3], x = 1;
      star_of(i, k);
      for (int s = 0; s < 3; ++s)
        for (int c = 0; c < k[s]; ++c) code |= ec(0, x++, s + 1);
    } else if (i < kStar + kPath) {
      int p, q;
      path_of(i - kStar, p, q);
      code = ec(0, 1, p / 3 + 1) | ec(1, 2, p % 3 + 1) | ec(0, 3, q / 3 + 1) | ec(3, 4, q % 3 + 1);
    } else {
      const int k = i - kStar - kPath, p = k / 6, q = k % 6;
      code = ec(0, 1, p / 3 + 1) | ec(1, 2, p % 3 + 1) | ec(0, 3, kPair[q][0] + 1) | ec(0, 4, kPair[q][1] + 1);
    }
    K.add(code, bins[i]);
  }
}

// Pairs of triangles at a vertex (one shared edge allowed), one wave per vertex.
__global__ __launch_bounds__(256) void k_butterfly5(DevGraph G, Totals5 K, const uint32_t* __restrict__ tri,
                                                    const int32_t* st) {
  if (st[kStatus] != 0) return;
  const int lane = threadIdx.x & 63;
  for (int32_t v = blockIdx.x * 4 + (threadIdx.x >> 6); v < G.n; v += gridDim.x * 4) {
    const uint32_t c = lane < 27 ? tri[(int64_t)v * 27 + lane] : 0u;
    const u64 have = __ballot(c != 0u);
    for (u64 r = have; r; r &= r - 1ull) {
      const int i = __builtin_ctzll(r);
      const u64 ci = __shfl(c, i);
      if (lane < i || !c) continue;  // (lane: the second triangle's type)
      const uint32_t code = ec(0, 1, i / 9 + 1) | ec(0, 2, (i / 3) % 3 + 1) | ec(1, 2, i % 3 + 1) |
                            ec(0, 3, lane / 9 + 1) | ec(0, 4, (lane / 3) % 3 + 1) | ec(3, 4, lane % 3 + 1);
      K.add(code, lane == i ? ci * (ci - 1) / 2 : ci * (u64)c);
    }
  }
}

// ================================================ graphs around a triangle ==
//
constexpr int kApexThreads = 1024;
constexpr int kStaged = 256;  // links of a unit up to which a wave keeps them in LDS
constexpr int kApexParts = 16;  // most waves that share a unit, four thirds each (64 in what a lane does alone)
constexpr int kCommon = 64;     // of the vertices adjacent to u, b and c, those a wave has in one list
constexpr int kWheelT = 8;    // links of a unit up to which its wheels are taken pair by pair

// A unit is a G* entry (u, b) with triangles, its links the vertices c adjacent
// to both.  One wave per unit, a lane per c; the units are dealt out with a
// stride so that a hub's many heavy entries land on different waves.  What a
// lane finds goes to the totals at once: of 1.1e5 links on the 20,000-vertex
// graph most have a handful of non-zero sums.
template <class F>
__device__ __forceinline__ void for_entries(const DevGraph& G, const int32_t* cnt, int32_t least, int32_t turn, F&& f) {
  const int lane = threadIdx.x & 63;
  const int32_t total = G.gs_off[G.n], per = blockDim.x >> 6, nw = gridDim.x * per;
  // (turn: another wave's entries, in parts of nw / kApexParts)
  const int32_t wave = (blockIdx.x * per + (threadIdx.x >> 6) + turn * (nw / kApexParts)) % nw;
  for (int64_t base = wave; base < total; base += (int64_t)nw * 64) {
    const int64_t el = base + (int64_t)lane * nw;
    const int32_t c = el < total ? cnt[el] : 0;
    for (u64 todo = __ballot(c >= least); todo; todo &= todo - 1ull)
      f((int32_t)(base + (int64_t)__builtin_ctzll(todo) * nw));
  }
}

// Place of local vertex d in the sorted links p[0 .. m), or -1.
__device__ __forceinline__ int32_t link_at(const uint32_t* p, int32_t m, uint32_t d) {
  int32_t lo = 0, hi = m;
  while (lo < hi) {
    const int32_t mid = (lo + hi) >> 1;
    if ((p[mid] & kIdMask) < d) lo = mid + 1; else hi = mid;
  }
  return lo < m && (p[lo] & kIdMask) == d ? lo : -1;
}


__global__ __launch_bounds__(kApexThreads) void k_apex5(DevGraph G, const uint16_t* __restrict__ lut,
                                                        uint64_t* __restrict__ copies, Links L,
                                                        const u64* __restrict__ S, const int32_t* st) {
  __shared__ uint32_t s_R[kApexThreads / 64][kStaged], s_com[kApexThreads / 64][4 * kCommon + 27];
  __shared__ u64 sum[kC5];
  if (st[kStatus] != 0) return;
  const Local5 K{lut, sum};
  K.clear();
  const int lane = threadIdx.x & 63;
  uint32_t *sR = s_R[threadIdx.x >> 6], *com = s_com[threadIdx.x >> 6], *hist = com + 4 * kCommon;
  constexpr int nparts = kApexParts;
  for (int part = 0; part < nparts; ++part)
  for_entries(G, L.cnt, 4 * part + 1, part, [&](int32_t E) {
    const int32_t u = G.gs_row[E], ua = G.gs_off[u], t = L.cnt[E];
    const uint32_t bl = (uint32_t)(E - ua), pb = G.gs_idx[E] >> kTypeShift;
    const int32_t b = (int32_t)(G.gs_idx[E] & kIdMask);
    const uint32_t* R = L.idx + L.off[E];
    const uint4 Du = G.dt[u], Db = G.dt[b];
    const int parts = min(nparts, (t + 3) / 4);  // the waves on this unit
    const bool staged = t <= kStaged;  // b's links in LDS: searched for every third of every c
    if (staged)
      for (int32_t k = lane; k < t; k += 64) sR[k] = R[k];
    wave_sync();
    auto at_b = [&](int32_t k) { return staged ? sR[k] : R[k]; };
    auto place_b = [&](uint32_t d) { return staged ? link_at(sR, t, d) : link_at(R, t, d); };
    uint32_t tb[9];
    L.types(E, tb);
    const uint32_t cb = ec(0, 1, pb);
    // pairs and triples of thirds: a pendant at u; a book
    if (t >= 2 && part == 0)
      for (int k = lane; k < 45; k += 64) {
        int i = 0, j = k;
        for (; j >= 9 - i; ++i) j -= 9 - i;
        j += i;
        const uint32_t pi = i / 3 + 1, pj = j / 3 + 1;
        uint32_t ti = 0, tj = 0;  // (the register array has no run-time index)
#pragma unroll
        for (int x = 0; x < 9; ++x) {
          ti = i == x ? tb[x] : ti;
          tj = j == x ? tb[x] : tj;
        }
        const u64 w = i == j ? (u64)ti * (ti - 1u) / 2 : (u64)ti * tj;
        if (!ti || !tj || !w) continue;
        const uint32_t c = cb | ec(0, 2, pi) | ec(1, 2, i % 3 + 1) | ec(0, 3, pj) | ec(1, 3, j % 3 + 1);
        for (int s = 0; s < 3; ++s) K.add(c | ec(0, 4, s + 1), w * other(Du, s, pb, pi, pj));
        if (t >= 3)
#pragma unroll
          for (int x = 0; x < 9; ++x) {
            if (x < j || !tb[x]) continue;
            const u64 n = tb[x];
            const u64 w3 = i == j && j == x ? n * (n - 1) * (n - 2) / 6 : j == x ? ti * (n * (n - 1) / 2) : w * n;
            K.add(c | ec(0, 4, x / 3 + 1) | ec(1, 4, x % 3 + 1), w3);
          }
      }
    for (int32_t k = 64 * part + lane; k < t; k += 64 * nparts) {
      const uint32_t f = at_b(k), cl = f & kIdMask, bc = f >> kTypeShift;
      const uint32_t fc = G.gs_idx[ua + cl], pc = fc >> kTypeShift;
      const int32_t c = (int32_t)(fc & kIdMask), Ec = ua + (int32_t)cl;
      const uint4 Dc = G.dt[c];
      const uint32_t ac = 3 * (pc - 1) + (bc - 1);
      const uint32_t code = cb | ec(0, 2, pc) | ec(1, 2, bc);
      // kite: another third and a pendant at c
      u64 xc[3], xb[3];
      for (int s = 0; s < 3; ++s) {
        xc[s] = other(Dc, s, flip(pc), flip(bc));
        xb[s] = other(Db, s, flip(pb), bc);
      }
      if (t >= 2)
#pragma unroll
        for (int x = 0; x < 9; ++x) {
          const u64 n = tb[x] - (x == (int)ac);
          if (!n) continue;
          uint32_t cs[3];
          u64 ws[3];
#pragma unroll
          for (int s = 0; s < 3; ++s) {
            cs[s] = code | ec(0, 3, x / 3 + 1) | ec(1, 3, x % 3 + 1) | ec(2, 4, s + 1);
            ws[s] = n * xc[s];
          }
          K.add(cs, ws);
        }
      if (cl < bl) continue;  // each triangle u, b, c once from here
      {
        uint32_t cs[24];
        u64 ws[24];
#pragma unroll
        for (int s = 0; s < 3; ++s) {
          const u64 x = other(Du, s, pb, pc);
#pragma unroll
          for (int q = 0; q < 3; ++q) {
            const int at = 8 * s + 2 * q;
            cs[at] = code | ec(1, 3, s + 1) | ec(2, 4, q + 1);  // bull
            ws[at] = xb[s] * xc[q];
            // a path of two edges from u
            cs[at + 1] = code | ec(0, 3, s + 1) | ec(3, 4, q + 1);
            ws[at + 1] = S[(int64_t)u * 9 + 3 * s + q] - (pb == (uint32_t)s + 1 ? other(Db, q, flip(pb), 0) : 0ull) -
                         (pc == (uint32_t)s + 1 ? other(Dc, q, flip(pc), 0) : 0ull);
          }
          // two pendants at u: types s, s and s, s + 1 (the third and the first)
          const int q = (s + 1) % 3;
          cs[8 * s + 6] = code | ec(0, 3, s + 1) | ec(0, 4, s + 1);
          ws[8 * s + 6] = x * (x - 1) / 2;
          cs[8 * s + 7] = code | ec(0, 3, s + 1) | ec(0, 4, q + 1);
          ws[8 * s + 7] = x * other(Du, q, pb, pc);
        }
        K.add(cs, ws);
      }
      if (t < 2 && L.cnt[Ec] < 2) continue;
      uint32_t tc[9];
      L.types(Ec, tc);
      const uint32_t ab = 3 * (pb - 1) + (flip(bc) - 1);  // b among c's thirds
#pragma unroll
      for (int x = 0; x < 9; ++x) {  // gem: a third of (u, b), one of (u, c)
        const u64 n = tb[x] - (x == (int)ac);
        if (!n) continue;
        uint32_t cs[9];
        u64 ws[9];
#pragma unroll
        for (int y = 0; y < 9; ++y) {
          cs[y] = code | ec(0, 3, x / 3 + 1) | ec(1, 3, x % 3 + 1) | ec(0, 4, y / 3 + 1) | ec(2, 4, y % 3 + 1);
          ws[y] = n * (u64)(tc[y] - (y == (int)ab));
        }
        K.add(cs, ws);
      }
    }
    // the vertices d adjacent to u, b and c, c by c: counted by type, for two of
    // them whatever their own pair, and those after c listed, for the K4s and,
    // two by two, the K5s
    if (t >= 2)
      for (int32_t k = part; k < t; k += parts) {
        const uint32_t f = at_b(k), cl = f & kIdMask, bc = f >> kTypeShift;
        const int32_t Ec = ua + (int32_t)cl, mc = L.cnt[Ec];
        if (cl < bl || mc < 2) continue;
        const uint32_t* Rc = L.idx + L.off[Ec];
        const uint32_t pc = G.gs_idx[Ec] >> kTypeShift;
        const uint32_t code = cb | ec(0, 2, pc) | ec(1, 2, bc);
        if (lane < 27) hist[lane] = 0;
        wave_sync();
        // lists from the skip-th on of the d after c into out[0 .. 2 kCommon);
        // the first time, all are counted by type; returns how many there are
        int32_t nall = 0;
        auto list_after = [&](int32_t skip, uint32_t* out, bool count) {
          int32_t nd = 0;
          for (int32_t i0 = 0; i0 < mc; i0 += 64) {
            const int32_t i = i0 + lane;
            const uint32_t fc = i < mc ? Rc[i] : bl, dl = fc & kIdMask;
            const int32_t at = dl == bl || (!count && dl <= cl) ? -1 : place_b(dl);
            if (count) {
              if (at >= 0)
                atomicAdd(&hist[9 * ((G.gs_idx[ua + dl] >> kTypeShift) - 1) + 3 * ((at_b(at) >> kTypeShift) - 1) +
                                (fc >> kTypeShift) - 1], 1u);
              nall += __popcll(__ballot(at >= 0));
            }
            const bool in = at >= 0 && dl > cl;
            const u64 hit = __ballot(in);
            const int32_t x = nd + __popcll(hit & ((1ull << lane) - 1ull)) - skip;
            if (in && x >= 0 && x < kCommon) {
              out[x] = fc;
              out[kCommon + x] = at_b(at);
            }
            nd += __popcll(hit);
          }
          wave_sync();
          return nd;
        };
        const int32_t nd = list_after(0, com, true);
        if (nall >= 2) {
          const uint32_t n = lane < 27 ? hist[lane] : 0u;
          for (u64 have = __ballot(n > 0u); have; have &= have - 1ull) {
            const int i = __builtin_ctzll(have);
            const u64 ni = __shfl(n, i);
            if (lane < i || !n) continue;  // (lane: the second one's type)
            K.add(code | ec(0, 3, i / 9 + 1) | ec(1, 3, (i / 3) % 3 + 1) | ec(2, 3, i % 3 + 1) | ec(0, 4, lane / 9 + 1) |
                      ec(1, 4, (lane / 3) % 3 + 1) | ec(2, 4, lane % 3 + 1),
                  lane == i ? ni * (ni - 1) / 2 : ni * (u64)n);
          }
        }
        // the K5 of d at x0 + x of one list and e at y of another
        auto five = [&](const uint32_t* A, const uint32_t* B, int32_t x, int32_t y) {
          const uint32_t dl = A[x] & kIdMask, el = B[y] & kIdMask;
          const int32_t Ed = ua + (int32_t)dl;
          const int32_t de = link_at(L.idx + L.off[Ed], L.cnt[Ed], el);
          if (de >= 0)
            K.add(code | ec(0, 3, G.gs_idx[Ed] >> kTypeShift) | ec(1, 3, A[kCommon + x] >> kTypeShift) |
                      ec(2, 3, A[x] >> kTypeShift) | ec(0, 4, G.gs_idx[ua + el] >> kTypeShift) |
                      ec(1, 4, B[kCommon + y] >> kTypeShift) | ec(2, 4, B[y] >> kTypeShift) |
                      ec(3, 4, L.idx[L.off[Ed] + de] >> kTypeShift), 1ull);
        };
        for (int32_t x0 = 0; x0 < nd; x0 += kCommon) {  // (one list, but for the largest)
          if (x0 > 0) list_after(x0, com, false);
          const int32_t nx = min(kCommon, nd - x0);
          for (int32_t x = lane; x < nx; x += 64) {  // K4 u, b < c < d
            const uint32_t dl = com[x] & kIdMask, cd = com[x] >> kTypeShift, bd = com[kCommon + x] >> kTypeShift;
            const uint32_t pd = G.gs_idx[ua + dl] >> kTypeShift;
            const uint32_t four = code | ec(0, 3, pd) | ec(1, 3, bd) | ec(2, 3, cd);
            for (int s = 0; s < 3; ++s) K.add(four | ec(0, 4, s + 1), other(Du, s, pb, pc, pd));
            uint32_t tc[9], td[9];
            L.types(Ec, tc);
            L.types(ua + (int32_t)dl, td);
            const int ac = 3 * (int)(pc - 1) + (int)(bc - 1), ab = 3 * (int)(pb - 1) + (int)(flip(bc) - 1);
            const int ad = 3 * (int)(pd - 1) + (int)(bd - 1), acd = 3 * (int)(pd - 1) + (int)(cd - 1);
            const int adb = 3 * (int)(pb - 1) + (int)(flip(bd) - 1), adc = 3 * (int)(pc - 1) + (int)(flip(cd) - 1);
#pragma unroll
            for (int v = 1; v <= 3; ++v) {  // a vertex on u and one of the three
              uint32_t cs[9];
              u64 ws[9];
#pragma unroll
              for (int i = 0; i < 9; ++i) {
                cs[i] = four | ec(0, 4, i / 3 + 1) | ec(v, 4, i % 3 + 1);
                ws[i] = v == 1 ? tb[i] - (i == ac) - (i == ad) : v == 2 ? tc[i] - (i == ab) - (i == acd)
                                                                       : td[i] - (i == adb) - (i == adc);
              }
              K.add(cs, ws);
            }
          }
          for (int32_t q = lane; q < nx * nx; q += 64)
            if (q / nx < q % nx) five(com, com, q / nx, q % nx);
          for (int32_t y0 = x0 + kCommon; y0 < nd; y0 += kCommon) {
            list_after(y0, com + 2 * kCommon, false);
            const int32_t ny = min(kCommon, nd - y0);
            for (int32_t q = lane; q < nx * ny; q += 64) five(com, com + 2 * kCommon, q / ny, q % ny);
            wave_sync();
          }
        }
        wave_sync();
      }
    // wheels with hub u whose rim's first vertex is b: two thirds c < c' of
    // (u, b) and a vertex d adjacent to both
    if (t >= 2 && t <= kWheelT && part == 0)
      for (int32_t k = lane >> 3; k < t * t; k += 8) {  // eight lanes per pair: the shorter row against the longer
        const int32_t i = k / t, j = k % t;
        const uint32_t f1 = at_b(i), f2 = at_b(j);
        if ((f1 & kIdMask) < bl || i >= j) continue;
        const int32_t E1 = ua + (int32_t)(f1 & kIdMask), E2 = ua + (int32_t)(f2 & kIdMask);
        const int32_t m1 = L.cnt[E1], m2 = L.cnt[E2];
        if (m1 < 2 || m2 < 2) continue;
        const uint32_t *R1 = L.idx + L.off[E1], *R2 = L.idx + L.off[E2];
        const uint32_t code = cb | ec(0, 2, G.gs_idx[E1] >> kTypeShift) | ec(0, 3, G.gs_idx[E2] >> kTypeShift) |
                              ec(1, 2, f1 >> kTypeShift) | ec(1, 3, f2 >> kTypeShift);
        const bool first = m1 <= m2;
        const uint32_t *Ra = first ? R1 : R2, *Rb = first ? R2 : R1;
        const int32_t ma = first ? m1 : m2, mb = first ? m2 : m1, sa = first ? 2 : 3;
        for (int32_t x = lane & 7; x < ma; x += 8) {
          const uint32_t dl = Ra[x] & kIdMask;
          if (dl <= bl) continue;
          const int32_t y = link_at(Rb, mb, dl);
          if (y < 0) continue;
          K.add(code | ec(0, 4, G.gs_idx[ua + dl] >> kTypeShift) | ec(sa, 4, Ra[x] >> kTypeShift) |
                    ec(5 - sa, 4, Rb[y] >> kTypeShift), 1ull);
        }
      }
    wave_sync();
  });
  K.write(copies, blockIdx.x);
}

// Wheels of the units with more links, one workgroup each.  The paths b - c - d
// among N(u) are counted per d by their 27 types while the row of u is short
// enough for that table, and the pairs taken in closed form (n = 115, m = 1,380:
// 476 us as single pairs).  Else they are nodes chained by d, each paired with
// the earlier ones of its d; nodes that do not fit are taken in several passes
// over shares of the d.
constexpr int kNodes = 8192, kHeads = 2048;
constexpr int kWheelRow = 1024;      // neighbours of u up to which d has a table entry
constexpr int32_t kMaxThirds = 4096;  // links of a unit (fourteen bits of a node; one d fits in a pass)

__global__ __launch_bounds__(256) void k_wheel5(DevGraph G, Totals5 K, Links L, const int32_t* st) {
  __shared__ uint32_t words[kNodes + kHeads + kNodes / 2];
  static_assert(sizeof(words) >= kWheelRow * 27 * 2, "table of 16-bit counts");
  uint32_t *node = words, *head = words + kNodes;
  uint16_t* next = reinterpret_cast<uint16_t*>(words + kNodes + kHeads);
  __shared__ int32_t list[256], nlist, nnode;
  if (st[kStatus] != 0) return;
  const int32_t total = G.gs_off[G.n];
  for (int64_t base = blockIdx.x; base < total; base += (int64_t)gridDim.x * 256) {
    __syncthreads();
    if (threadIdx.x == 0) nlist = 0;
    __syncthreads();
    const int64_t el = base + (int64_t)threadIdx.x * gridDim.x;
    if (el < total && L.cnt[el] > kWheelT) list[atomicAdd(&nlist, 1)] = (int32_t)el;
    __syncthreads();
    const int32_t nl = nlist;
    for (int32_t q = 0; q < nl; ++q) {
      const int32_t E = list[q], u = G.gs_row[E], ua = G.gs_off[u], t = L.cnt[E];
      const uint32_t bl = (uint32_t)(E - ua);
      const uint32_t* R = L.idx + L.off[E];
      const uint32_t cb = ec(0, 1, G.gs_idx[E] >> kTypeShift);
      const int32_t du = G.gs_off[u + 1] - ua;
      if (du <= kWheelRow) {
        for (int i = threadIdx.x; i < (du * 27 + 1) / 2; i += 256) words[i] = 0;
        __syncthreads();
        for (int32_t i = threadIdx.x >> 3; i < t; i += 32) {
          const uint32_t cl = R[i] & kIdMask;
          if (cl < bl) continue;
          const int32_t Ec = ua + (int32_t)cl, m = L.cnt[Ec];
          const uint32_t* Rc = L.idx + L.off[Ec];
          const uint32_t ty = 9 * ((G.gs_idx[Ec] >> kTypeShift) - 1u) + 3 * ((R[i] >> kTypeShift) - 1u);
          for (int32_t x = threadIdx.x & 7; x < m; x += 8) {
            const uint32_t f = Rc[x], dl = f & kIdMask;
            if (dl <= bl) continue;
            const uint32_t at = dl * 27 + ty + (f >> kTypeShift) - 1u;
            atomicAdd(&words[at >> 1], 1u << (16 * (at & 1u)));
          }
        }
        __syncthreads();
        auto n_at = [&](int32_t i) { return (words[i >> 1] >> (16 * (i & 1))) & 0xFFFFu; };
        for (int32_t x = threadIdx.x; x < du * 27; x += 256) {  // this type with itself and the later ones
          const u64 n = n_at(x);
          if (!n) continue;
          const int32_t dl = x / 27, i = x % 27;
          const uint32_t code = cb | ec(0, 4, G.gs_idx[ua + dl] >> kTypeShift) | ec(0, 2, i / 9 + 1) |
                                ec(1, 2, (i / 3) % 3 + 1) | ec(2, 4, i % 3 + 1);
#pragma unroll 1
          for (int j0 = i - i % 9; j0 < 27; j0 += 9) {
            uint32_t cs[9];
            u64 ws[9], any = 0;
#pragma unroll
            for (int q = 0; q < 9; ++q) {
              const int j = j0 + q;
              const u64 m = j < i ? 0ull : j == i ? n - 1 : n_at(dl * 27 + j);
              cs[q] = code | ec(0, 3, j0 / 9 + 1) | ec(1, 3, q / 3 + 1) | ec(3, 4, q % 3 + 1);
              ws[q] = j == i ? n * m / 2 : n * m;
              any |= ws[q];
            }
            if (any) K.add(cs, ws);
          }
        }
        __syncthreads();
        continue;
      }
      // share of a pass: the d that are res modulo mod (a power of two); halved
      // while it does not fit, down to one d, whose nodes are at most t
      for (uint32_t mod = 1, res = 0; mod;) {
        for (int i = threadIdx.x; i < kHeads; i += 256) head[i] = 0;
        if (threadIdx.x == 0) nnode = 0;
        __syncthreads();
        for (int32_t i = threadIdx.x >> 3; i < t; i += 32) {
          const uint32_t cl = R[i] & kIdMask;
          if (cl < bl) continue;
          const int32_t Ec = ua + (int32_t)cl, m = L.cnt[Ec];
          const uint32_t* Rc = L.idx + L.off[Ec];
          for (int32_t x = threadIdx.x & 7; x < m; x += 8) {
            const uint32_t f = Rc[x], dl = f & kIdMask;
            if (dl <= bl || (dl & (mod - 1u)) != res) continue;
            const int32_t at = atomicAdd(&nnode, 1);
            if (at >= kNodes) continue;
            node[at] = dl | (uint32_t)i << 16 | (f >> kTypeShift) << kTypeShift;
            next[at] = (uint16_t)atomicExch(&head[hash_mul(dl, 11)], (uint32_t)at + 1u);
          }
        }
        __syncthreads();
        const int32_t nn = nnode;
        __syncthreads();
        if (nn > kNodes && mod < 0x10000u) {  // the same on every thread
          mod *= 2;
          continue;
        }
        for (int32_t i = threadIdx.x; i < nn; i += 256) {
          const uint32_t a = node[i], dl = a & 0xFFFFu;
          for (uint32_t j = next[i]; j; j = next[j - 1]) {
            const uint32_t b = node[j - 1];
            if ((b & 0xFFFFu) != dl) continue;
            const uint32_t f1 = R[(a >> 16) & 0x3FFFu], f2 = R[(b >> 16) & 0x3FFFu];
            K.add(cb | ec(0, 2, G.gs_idx[ua + (f1 & kIdMask)] >> kTypeShift) |
                      ec(0, 3, G.gs_idx[ua + (f2 & kIdMask)] >> kTypeShift) | ec(0, 4, G.gs_idx[ua + dl] >> kTypeShift) |
                      ec(1, 2, f1 >> kTypeShift) | ec(1, 3, f2 >> kTypeShift) | ec(2, 4, a >> kTypeShift) |
                      ec(3, 4, b >> kTypeShift), 1ull);
          }
        }
        __syncthreads();
        while (mod > 1u && res >= mod / 2) {  // both halves of the share above are done
          mod /= 2;
          res -= mod;
        }
        if (mod == 1u) mod = 0;
        else res += mod / 2;
      }
    }
  }
}

// =========================================================== graphs on a C4 ==
//
// Typed wedges n[3 p + q](w) from u to every other w (p, q less one the types
// of the middle seen from u and of w seen from the middle).  Pairs of wedges
// with a pendant at u; triples (K2,3); a triangle on the edge u v with the
// other wedges to w of every wedge u - v - w (house); an edge a - b among the
// middles with a third middle.  u is every vertex and w any other, so that all
// but the first meet each copy from both ends.  The tables are those of k_wedge
// (counts.hip) over the whole rows: hashes of 7-bit counters while d(u) <= 127
// and the visits fit, else 16-bit counters over one block of ids at a time.

// Sums shared by the units of a workgroup.
struct PairBins {
  u64* three;  // [405] triples i <= j <= k, nine per pair
  u64* house;  // [729] (p, third's two types, q, j)
  u64* edge;   // [2187] (pa, pb, ab, qa, qb, j)
  __device__ __forceinline__ void clear(int t, int nt) const {
    for (int i = t; i < 405; i += nt) three[i] = 0;
    for (int i = t; i < 729; i += nt) house[i] = 0;
    for (int i = t; i < 2187; i += nt) edge[i] = 0;
  }
  __device__ __forceinline__ void flush(const Totals5& K, int t, int nt) const {
    constexpr int N = 6;  // at a time
    for (int k0 = t; k0 < 3645; k0 += N * nt) {
      uint32_t code[N];
      u64 w[N];
#pragma unroll
      for (int i = 0; i < N; ++i) {
        int k = k0 + i * nt;
        code[i] = 0;
        w[i] = 0;
        if (k < 729) {
          const int a = k / 81, b = (k / 9) % 9, c = k % 9;
          if (a > b || b > c) continue;
          w[i] = three[(a * 9 - a * (a - 1) / 2 + b - a) * 9 + c];
          code[i] = ec(0, 2, a / 3 + 1) | ec(2, 1, a % 3 + 1) | ec(0, 3, b / 3 + 1) | ec(3, 1, b % 3 + 1) |
                    ec(0, 4, c / 3 + 1) | ec(4, 1, c % 3 + 1);
        } else if (k < 1458) {  // u 0, v 1, roof 2, w 3, other middle 4
          k -= 729;
          w[i] = house[k];
          const int p = k / 243, x = (k / 81) % 3, y = (k / 27) % 3, q = (k / 9) % 3, j = k % 9;
          code[i] = ec(0, 1, p + 1) | ec(0, 2, x + 1) | ec(1, 2, y + 1) | ec(1, 3, q + 1) | ec(0, 4, j / 3 + 1) |
                    ec(4, 3, j % 3 + 1);
        } else if (k < 3645) {
          k -= 1458;
          w[i] = edge[k];
          const int j = k % 9, qb = (k / 9) % 3, qa = (k / 27) % 3, ab = (k / 81) % 3, pb = (k / 243) % 3, pa = k / 729;
          code[i] = ec(0, 1, pa + 1) | ec(0, 2, pb + 1) | ec(1, 2, ab + 1) | ec(1, 3, qa + 1) | ec(2, 3, qb + 1) |
                    ec(0, 4, j / 3 + 1) | ec(4, 3, j % 3 + 1);
        }
      }
      K.add(code, w);
    }
  }
};

// Pairs and triples of the wedges to one w, n(i) the counts of its types.  Most
// w have two or three types, so the loops run over those.
template <class N>
__device__ __forceinline__ void pairs_and_triples(N&& n, u64* pair, const PairBins& B) {
  uint32_t have = 0;
#pragma unroll
  for (int i = 0; i < 9; ++i) have |= n(i) ? 1u << i : 0u;
  for (uint32_t r = have; r; r &= r - 1u) {
    const int i = __builtin_ctz(r);
    const u64 a = n(i);
    for (uint32_t q = r; q; q &= q - 1u) {
      const int j = __builtin_ctz(q);
      const u64 b = n(j), ab = i == j ? a * (a - 1) / 2 : a * b;
      if (!ab) continue;
      atomicAdd(&pair[9 * i + j], ab);
      const int at = i * 9 - i * (i - 1) / 2 + j - i;  // of 45 pairs
      for (uint32_t o = q; o; o &= o - 1u) {
        const int k = __builtin_ctz(o);
        const u64 c = n(k), w = i == k ? ab * (a - 2) / 3 : j == k ? a * (b * (b - 1) / 2) : ab * c;
        if (w) atomicAdd(&B.three[at * 9 + k], w);
      }
    }
  }
}

// Triangles on the edge E = (u, v) with the wedges to w next to v's own.
__device__ __forceinline__ void house_add(const uint32_t (&n)[9], const uint32_t (&tv)[9], uint32_t p, uint32_t q,
                                          u64* house) {
#pragma unroll
  for (int x = 0; x < 9; ++x) {
    if (!tv[x]) continue;
    u64* h = house + 243 * p + 27 * x + 9 * q;
#pragma unroll
    for (int j = 0; j < 9; ++j) {
      const u64 m = n[j] - (j == (int)(3 * p + q));
      if (m) atomicAdd(&h[j], m * tv[x]);
    }
  }
}

// The edges (a, b) among N(u) with b after a in u's row: the links of u's
// entries are one run of the link arrays, eight lanes take one and its thirds w.
// n_of(w, n): the wedges u .. w, false when w is not in the table.
template <class F>
__device__ __forceinline__ void edge_add(const DevGraph& G, const Links& L, int32_t u, int32_t ua, int32_t ub, int32_t t,
                                         int32_t nt, const PairBins& B, F&& n_of) {
  const int32_t k1 = L.off[ub];
  for (int32_t k = L.off[ua] + (t >> 3); k < k1; k += nt >> 3) {
    const int32_t E = L.src[k], M = L.mate[k];  // entries (u, a) and (a, b)
    const uint32_t f = L.idx[k], ea = G.gs_idx[E], bl = f & kIdMask, ab = (f >> kTypeShift) - 1u;
    const int32_t mt = L.cnt[M], mo = L.off[M];
    if ((int32_t)bl < E - ua || mt < 2) continue;  // (one third: u)
    const uint32_t pa = (ea >> kTypeShift) - 1u, pb = (G.gs_idx[ua + (int32_t)bl] >> kTypeShift) - 1u;
    const int32_t aa = G.gs_off[(int32_t)(ea & kIdMask)];
    u64* const e0 = B.edge + ((pa * 3 + pb) * 3 + ab) * 81;
    for (int32_t x = t & 7; x < mt; x += 8) {
      const uint32_t g = L.idx[mo + x], fw = G.gs_idx[aa + (int32_t)(g & kIdMask)];
      const uint32_t qa = (fw >> kTypeShift) - 1u, qb = (g >> kTypeShift) - 1u, w = fw & kIdMask;
      uint32_t n[9];
      if ((int32_t)w == u || !n_of(w, n)) continue;
      u64* e = e0 + (qa * 3 + qb) * 9;
#pragma unroll
      for (int j = 0; j < 9; ++j) {
        const uint32_t m = n[j] - (j == (int)(3 * pa + qa)) - (j == (int)(3 * pb + qb));
        if (m) atomicAdd(&e[j], (u64)m);
      }
    }
  }
}

// Lists the vertices with two neighbours or more by their visits.  Eight lanes
// per vertex.
struct PairListsOf {
  int32_t* v[kPairLists];
};
__global__ __launch_bounds__(256) void k_classify5(DevGraph G, PairListsOf L, int32_t* __restrict__ queue,
                                                   const int32_t* st) {
  __shared__ int32_t cnt[kPairLists], base[kPairLists];
  __shared__ uint16_t where[256];  // list and place of each of this workgroup's vertices
  if (st[kStatus] != 0) return;
  if (threadIdx.x < kPairLists) cnt[threadIdx.x] = 0;
  __syncthreads();
  const int l8 = threadIdx.x & 7;
  const int32_t v0 = blockIdx.x * 256, v1 = min(G.n, v0 + 256);
  for (int32_t v = v0 + (int32_t)(threadIdx.x >> 3); v < v1; v += 32) {
    const int32_t a = G.gs_off[v], b = G.gs_off[v + 1], d = b - a;
    int32_t vis = 0;
    if (d <= 127)
      for (int32_t i = a + l8; i < b; i += 8) vis += min(G.deg[G.gs_idx[i] & kIdMask], pair_cap(13) + 1);
#pragma unroll
    for (int o = 4; o; o >>= 1) vis += __shfl_xor(vis, o);
    if (l8 == 0) {
      int l = d < 2 ? 15 : d > 127 ? kPairBlock : kPair9;
      if (l == kPair9)
        while (l < kPairBlock && vis > pair_cap(9 + l)) ++l;
      where[v - v0] = (uint16_t)(l | (l < kPairLists ? atomicAdd(&cnt[l], 1) : 0) << 4);
    }
  }
  __syncthreads();
  if (threadIdx.x < kPairLists && cnt[threadIdx.x])
    base[threadIdx.x] = atomicAdd(&queue[kPairQueue + threadIdx.x], cnt[threadIdx.x]);
  __syncthreads();
  const int32_t v = v0 + (int32_t)threadIdx.x;
  if (v >= v1) return;
  const int l = where[threadIdx.x] & 15, at = where[threadIdx.x] >> 4;
  if (l < kPairLists) L.v[l][base[l] + at] = v;
}

// The next unit of a workgroup: dealt out by position, or pulled from a counter
// where units are long and uneven (a pull is 25 ns, such a unit 20 us and more).
template <bool PULL>
__device__ __forceinline__ int64_t next_unit(int64_t k, int64_t step, int32_t* cursor, int32_t* slot) {
  if constexpr (!PULL) return k + step;
  __syncthreads();
  if (threadIdx.x == 0) *slot = (int32_t)gridDim.x + atomicAdd(cursor, 1);
  __syncthreads();
  return *slot;
}

// NT threads per u, BT per workgroup; a hash of 2^HB vertices.  The rows of N(u)
// are cut into pieces of 64 entries, sixteen lanes each: whole rows kept a wave
// on one hub's row while the others were done (20 us for a unit's 2,000 visits).
template <int NT, int HB, int BT>
__global__ __launch_bounds__(BT) void k_pairs5(DevGraph G, Totals5 K, Links L, int32_t* __restrict__ queue,
                                               const int32_t* __restrict__ list, const int32_t* st) {
  constexpr int NU = BT / NT, H = 1 << HB;
  static_assert(NU == 1 || NT == 64, "a barrier is the unit's own");
  constexpr int CAP = pair_cap(HB), MAXP = CAP / 64 + 128;
  constexpr bool PULL = NT >= 512;
  __shared__ uint32_t s_key[NU][H];
  __shared__ u64 s_cnt[NU][H], s_pair[NU][81];
  __shared__ uint16_t s_act[NU][CAP / 2];  // slots with two wedges or more
  __shared__ uint32_t s_piece[NU][MAXP];   // neighbour << 16 | piece: of rows with triangles from the front, else the back
  __shared__ int32_t s_n[NU][4], s_row[NU][128], s_len[NU][128];
  __shared__ u64 s_three[405], s_house[729], s_edge[2187];
  __shared__ int32_t s_next;
  if (st[kStatus] != 0) return;
  const int32_t count = queue[kPairQueue + HB - 9];
  if ((int32_t)blockIdx.x * NU >= count) return;
  const int un = threadIdx.x / NT, t = threadIdx.x % NT;
  uint32_t* key = s_key[un];
  u64 *cnt = s_cnt[un], *pair = s_pair[un];
  const PairBins B{s_three, s_house, s_edge};
  B.clear(threadIdx.x, BT);
  for (int i = t; i < H; i += NT) {
    key[i] = kNone;
    cnt[i] = 0;
  }
  for (int i = t; i < 81; i += NT) pair[i] = 0;
  int32_t* nn = s_n[un];  // listed slots, pieces at the front, at the back
  if (t < 3) nn[t] = 0;
  __syncthreads();
  auto sync = [] {
    if constexpr (NT <= 64) wave_sync();
    else __syncthreads();
  };
  uint16_t* act = s_act[un];
  uint32_t* piece = s_piece[un];
  int32_t *row = s_row[un], *len = s_len[un];
  // pendants at u: thread t holds the pairs (pi, pj), by the pendant's type
  u64 pend[2][3] = {{0, 0, 0}, {0, 0, 0}};
  for (int64_t k = (int64_t)blockIdx.x * NU + un; k < count;
       k = next_unit<PULL>(k, (int64_t)gridDim.x * NU, &queue[kPairCursor + HB - 9], &s_next)) {
    const int32_t u = list[k], ua = G.gs_off[u], ub = G.gs_off[u + 1], d = ub - ua;
    for (int32_t i = t; i < d; i += NT) {
      const int32_t v = (int32_t)(G.gs_idx[ua + i] & kIdMask), ra = G.gs_off[v], m = G.gs_off[v + 1] - ra;
      row[i] = ra;
      len[i] = m;
      const int32_t q = (m + 63) >> 6;
      if (L.cnt[ua + i]) {
        const int32_t at = atomicAdd(&nn[1], q);
        for (int32_t j = 0; j < q; ++j) piece[at + j] = (uint32_t)i << 16 | (uint32_t)j;
      } else {
        const int32_t at = atomicAdd(&nn[2], q);
        for (int32_t j = 0; j < q; ++j) piece[MAXP - 1 - at - j] = (uint32_t)i << 16 | (uint32_t)j;
      }
    }
    sync();
    const int32_t nf = nn[1], np = nf + nn[2];
    for (int32_t x = t >> 4; x < np; x += NT / 16) {
      const uint32_t pc = piece[x < nf ? x : MAXP - 1 - (x - nf)];
      const int32_t i = (int32_t)(pc >> 16), off = (int32_t)(pc & 0xFFFFu) * 64;
      const int p7 = 21 * (int)((G.gs_idx[ua + i] >> kTypeShift) - 1u);
      each4(G.gs_idx + row[i] + off, t & 15, 16, min(64, len[i] - off), [&](int32_t, uint32_t f) {
        const uint32_t w = f & kIdMask;
        if ((int32_t)w == u) return;
        uint32_t h = hash_mul(w, HB);
        for (;;) {
          const uint32_t old = atomicCAS(&key[h], kNone, w);
          if (old == kNone || old == w) break;
          h = (h + 1) & (H - 1);
        }
        atomicAdd(&cnt[h], 1ull << (p7 + 7 * (int)((f >> kTypeShift) - 1u)));
      });
    }
    sync();
    for (int i = t; i < H; i += NT) {
      const u64 c = cnt[i];
      if (c && !one_wedge(c, kOnes7)) act[atomicAdd(&nn[0], 1)] = (uint16_t)i;
    }
    sync();
    const int32_t na = nn[0];
    for (int x = t; x < na; x += NT) {
      const u64 c = cnt[act[x]];
      pairs_and_triples([c](int i) { return (uint32_t)(c >> (7 * i)) & 127u; }, pair, B);
    }
    sync();
    const uint4 D = G.dt[u];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int i = t + 64 * r;
      if (t < 64 && i < 81 && pair[i]) {
        const u64 w = pair[i];
        pair[i] = 0;
#pragma unroll
        for (int s = 0; s < 3; ++s) pend[r][s] += w * other(D, s, (uint32_t)(i / 27) + 1, (uint32_t)(i % 9) / 3 + 1);
      }
    }
    if (na > 0) {
      auto n_of = [&](uint32_t w, uint32_t (&n)[9]) {
        uint32_t h = hash_mul(w, HB), kk;
        while ((kk = key[h]) != w && kk != kNone) h = (h + 1) & (H - 1);
        const u64 c = cnt[h];
        if (kk != w || one_wedge(c, kOnes7)) return false;
#pragma unroll
        for (int j = 0; j < 9; ++j) n[j] = (uint32_t)(c >> (7 * j)) & 127u;
        return true;
      };
      for (int32_t x = t >> 4; x < nf; x += NT / 16) {
        const uint32_t pc = piece[x];
        const int32_t i = (int32_t)(pc >> 16), off = (int32_t)(pc & 0xFFFFu) * 64;
        const uint32_t p = (G.gs_idx[ua + i] >> kTypeShift) - 1u;
        uint32_t tv[9];
        L.types(ua + i, tv);
        each4(G.gs_idx + row[i] + off, t & 15, 16, min(64, len[i] - off), [&](int32_t, uint32_t f) {
          const uint32_t w = f & kIdMask;
          uint32_t n[9];
          if ((int32_t)w != u && n_of(w, n)) house_add(n, tv, p, (f >> kTypeShift) - 1u, s_house);
        });
      }
      edge_add(G, L, u, ua, ub, t, NT, B, n_of);
    }
    sync();
    for (int i = t; i < H; i += NT) {
      key[i] = kNone;
      cnt[i] = 0;
    }
    if (t < 3) nn[t] = 0;
    sync();
  }
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int k = t + 64 * r, i = k / 9, j = k % 9;
    if (t < 64 && k < 81)
      for (int s = 0; s < 3; ++s)
        K.add(ec(0, 2, i / 3 + 1) | ec(2, 1, i % 3 + 1) | ec(0, 3, j / 3 + 1) | ec(3, 1, j % 3 + 1) | ec(0, 4, s + 1),
              pend[r][s]);
  }
  __syncthreads();
  B.flush(K, threadIdx.x, BT);
}

// (u, block of ids) units, 16-bit counters (n <= 65,536).
constexpr int kPairIds = 6144;
__global__ __launch_bounds__(1024) void k_pairs5_block(DevGraph G, Totals5 K, Links L, int32_t* __restrict__ queue,
                                                       const int32_t* __restrict__ list, const int32_t* st) {
  constexpr int NT = 1024, MAXP = 1536;
  __shared__ uint32_t cnt[9 * kPairIds / 2];
  __shared__ u64 pair[81], s_three[405], s_house[729], s_edge[2187];
  __shared__ int32_t pt_i[MAXP], pt_a[MAXP], npiece, s_next;  // pieces of rows: neighbour | entries << 20, first entry
  if (st[kStatus] != 0) return;
  const int32_t nblk = (G.n + kPairIds - 1) / kPairIds;
  const int64_t units = (int64_t)queue[kPairQueue + kPairBlock] * nblk;
  if ((int64_t)blockIdx.x >= units) return;
  const int t = threadIdx.x;
  const PairBins B{s_three, s_house, s_edge};
  B.clear(t, NT);
  for (int i = t; i < 9 * kPairIds / 2; i += NT) cnt[i] = 0;
  if (t < 81) pair[t] = 0;
  if (t == 0) npiece = 0;
  u64 pend[3] = {0, 0, 0};
  __syncthreads();
  for (int64_t unit = blockIdx.x; unit < units; unit = next_unit<true>(unit, 0, &queue[kPairCursor + kPairBlock], &s_next)) {
    const int32_t u = list[unit / nblk], w0 = (int32_t)(unit % nblk) * kPairIds, w1 = min(G.n, w0 + kPairIds);
    const int32_t ua = G.gs_off[u], ub = G.gs_off[u + 1], d = ub - ua;
    // f(i, first entry, entries, lane of 16) for the pieces of 64 entries of the
    // parts of the rows of N(u) in the block, NT rows at a time
    auto each_piece = [&](bool linked, auto&& f) {
      for (int32_t i0 = 0; i0 < d; i0 += NT) {
        const int32_t i = i0 + t;
        int32_t a = 0, m = 0;
        if (i < d && (!linked || L.cnt[ua + i])) {
          const int32_t v = (int32_t)(G.gs_idx[ua + i] & kIdMask), ra = G.gs_off[v], rb = G.gs_off[v + 1];
          a = find_in(G.gs_idx, ra, rb, (uint32_t)w0);
          m = find_in(G.gs_idx, a, rb, (uint32_t)w1) - a;
        }
        for (;;) {  // until every row's pieces were listed
          while (m > 0) {
            const int32_t at = atomicAdd(&npiece, 1);
            if (at >= MAXP) break;
            pt_i[at] = i - i0 | min(m, 64) << 20;
            pt_a[at] = a;
            a += 64;
            m -= 64;
          }
          const bool more = __syncthreads_or(m > 0);
          const int32_t np = min(npiece, MAXP);
          for (int32_t x = t >> 4; x < np; x += NT / 16) f(i0 + (pt_i[x] & 0xFFFFF), pt_a[x], pt_i[x] >> 20, t & 15);
          __syncthreads();
          if (t == 0) npiece = 0;
          __syncthreads();
          if (!more) break;
        }
      }
    };
    each_piece(false, [&](int32_t i, int32_t a, int32_t m, int32_t l) {
      const uint32_t p = (G.gs_idx[ua + i] >> kTypeShift) - 1u;
      each4(G.gs_idx + a, l, 16, m, [&](int32_t, uint32_t e) {
        const uint32_t at = (3 * p + (e >> kTypeShift) - 1u) * kPairIds + (e & kIdMask) - (uint32_t)w0;
        atomicAdd(&cnt[at >> 1], 1u << (16 * (at & 1u)));
      });
    });
    auto n_of = [&](uint32_t w, uint32_t (&n)[9]) {
      if (w < (uint32_t)w0 || w >= (uint32_t)w1) return false;
      uint32_t sum = 0;
#pragma unroll
      for (int j = 0; j < 9; ++j) {
        const uint32_t at = j * kPairIds + w - (uint32_t)w0;
        n[j] = (cnt[at >> 1] >> (16 * (at & 1u))) & 0xFFFFu;
        sum += n[j];
      }
      return sum > 1;
    };
    for (int32_t w = w0 + t; w < w1; w += NT)
      if (w != u)
        pairs_and_triples([&](int i) {
          const uint32_t at = i * kPairIds + (uint32_t)(w - w0);
          return (cnt[at >> 1] >> (16 * (at & 1u))) & 0xFFFFu;
        }, pair, B);
    __syncthreads();
    if (t < 81 && pair[t]) {
      const u64 w = pair[t];
      const uint4 D = G.dt[u];
      pair[t] = 0;
      for (int s = 0; s < 3; ++s) pend[s] += w * other(D, s, (uint32_t)(t / 27) + 1, (uint32_t)(t % 9) / 3 + 1);
    }
    each_piece(true, [&](int32_t i, int32_t a, int32_t m, int32_t l) {
      const uint32_t p = (G.gs_idx[ua + i] >> kTypeShift) - 1u;
      uint32_t tv[9];
      L.types(ua + i, tv);
      each4(G.gs_idx + a, l, 16, m, [&](int32_t, uint32_t e) {
        const uint32_t w = e & kIdMask;
        uint32_t n[9];
        if ((int32_t)w != u && n_of(w, n)) house_add(n, tv, p, (e >> kTypeShift) - 1u, s_house);
      });
    });
    edge_add(G, L, u, ua, ub, t, NT, B, n_of);
    __syncthreads();
    for (int i = t; i < 9 * kPairIds / 2; i += NT) cnt[i] = 0;
    __syncthreads();
  }
  if (t < 81)
    for (int s = 0; s < 3; ++s)
      K.add(ec(0, 2, t / 27 + 1) | ec(2, 1, (t / 9) % 3 + 1) | ec(0, 3, (t % 9) / 3 + 1) | ec(3, 1, t % 3 + 1) |
                ec(0, 4, s + 1), pend[s]);
  __syncthreads();
  B.flush(K, t, NT);
}

// ==================================================================== C5 ==
//
// From the vertex u of highest rank: n(w) the typed wedges u - v - w with v and
// w of lower rank, and for every edge w - w' among them with w' below w the
// products n(w) n(w').  The tables and lists of u are k_wedge's (counts.hip);
// the u of k_wedge_top have tables in global memory.

// A bit at the foot of every 7-bit field that is not zero.
__device__ __forceinline__ u64 flags7(u64 c) {
  // the low six bits carry into the seventh unless all are zero
  constexpr u64 low = 63ull * kOnes7;
  return ((c | ((c & low) + low)) >> 6) & kOnes7;
}

// A workgroup keeps several copies of its sums, one per some lanes: the
// products of a wave meet on the same few of the 243.
constexpr int kCopies = 4, kTopCopies = 16;
__device__ __forceinline__ void c5_flush(const Totals5& K, const u64* all, int copies, int t, int nt) {
  for (int k = t; k < 243; k += nt) {
    const int i = k / 27, e = (k / 9) % 3, j = k % 9;
    u64 sum = 0;
    for (int r = 0; r < copies; ++r) sum += all[r * 243 + k];
    K.add(ec(0, 1, i / 3 + 1) | ec(1, 2, i % 3 + 1) | ec(2, 3, e + 1) | ec(4, 3, j % 3 + 1) | ec(0, 4, j / 3 + 1),
          sum);
  }
}

template <int NT, int HB, int LIST>
__global__ __launch_bounds__(NT < 256 ? 256 : NT) void k_c5(DevGraph G, Totals5 K, const int32_t* __restrict__ queue,
                                            const int32_t* __restrict__ list, const int32_t* st) {
  constexpr int BT = NT < 256 ? 256 : NT, NU = BT / NT, H = 1 << HB, LPR = NT == 16 ? 4 : 8, LONG = 64;
  __shared__ int32_t s_row[NU][NT], s_len[NU][NT];
  __shared__ uint32_t s_key[NU][H];
  __shared__ u64 s_cnt[NU][H], bins[kCopies * 243];
  __shared__ uint16_t s_act[NU][H];
  __shared__ int32_t s_nact[NU];
  if (st[kStatus] != 0) return;
  const int32_t count = queue[LIST];
  if ((int32_t)blockIdx.x * NU >= count) return;
  const int un = threadIdx.x / NT, t = threadIdx.x % NT;
  uint32_t* key = s_key[un];
  u64* cnt = s_cnt[un];
  uint16_t* act = s_act[un];
  int32_t *row = s_row[un], *len = s_len[un];
  u64* mine = bins + (threadIdx.x & (kCopies - 1)) * 243;
  for (int i = t; i < H; i += NT) {
    key[i] = kNone;
    cnt[i] = 0;
  }
  for (int i = threadIdx.x; i < kCopies * 243; i += BT) bins[i] = 0;
  if (t == 0) s_nact[un] = 0;
  __syncthreads();
  auto sync = [] {
    if constexpr (NT <= 64) wave_sync();
    else __syncthreads();
  };
  for (int32_t k = (int32_t)blockIdx.x * NU + un; k < count; k += (int32_t)gridDim.x * NU) {
    const int32_t u = list[k], ua = G.gs_off[u], ub = G.gs_off[u + 1];
    const int32_t ma = ua - G.np_off[u], dm = ub - G.np_off[u + 1] - ma;
    const uint32_t du = (uint32_t)(ub - ua);
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
    for (int i = t; i < H; i += NT) {
      if (!cnt[i]) continue;
      const int32_t w = (int32_t)key[i];
      if (ranked_below(G, (uint32_t)G.deg[w], w, du, u)) act[atomicAdd(&s_nact[un], 1)] = (uint16_t)i;
      else cnt[i] = 0;
    }
    sync();
    // NT of the listed w at a time: their rows N- first, then four lanes per
    // row, the whole unit for a long one
    const int32_t na = s_nact[un];
    for (int32_t x0 = 0; x0 < na; x0 += NT) {
      if (x0 + t < na) {
        const int32_t w = (int32_t)key[act[x0 + t]], wa = G.gs_off[w] - G.np_off[w];
        row[t] = wa;
        len[t] = G.gs_off[w + 1] - G.np_off[w + 1] - wa;
      }
      sync();
      const int32_t nx = min(NT, na - x0);
      auto take = [&](int32_t x, int32_t l, int32_t step) {
        const u64 c = cnt[act[x0 + x]], fc = flags7(c);
        const int32_t wa = row[x], wm = len[x];
        auto entry = [&](int32_t, uint32_t f) {
          const uint32_t z = f & kIdMask;
          uint32_t h = hash_mul(z, HB), kk;
          while ((kk = key[h]) != z && kk != kNone) h = (h + 1) & (H - 1);
          if (kk != z) return;
          const u64 e = cnt[h];
          if (!e) return;
          // loops over the types that occur, the fields' top bits as flags
          u64* to = mine + 9 * ((int)(f >> kTypeShift) - 1);
          for (u64 x = fc; x; x &= x - 1ull) {
            const int p = __builtin_ctzll(x);
            const u64 a = (c >> p) & 127u;
            for (u64 y = flags7(e); y; y &= y - 1ull) {
              const int q = __builtin_ctzll(y);
              atomicAdd(&to[27 * (p / 7) + q / 7], a * ((e >> q) & 127u));
            }
          }
        };
        for (int32_t r = l; r < wm; r += 4 * step) each4(G.nm_idx + wa, r, step, wm, entry);
      };
      if constexpr (NT > 16)
        for (int32_t x = t >> 6; x < nx; x += NT / 64)
          if (len[x] > LONG) take(x, t & 63, 64);
      for (int32_t x = t / 4; x < nx; x += NT / 4)
        if (NT == 16 || len[x] <= LONG) take(x, t % 4, 4);
      sync();
    }
    sync();
    for (int i = t; i < H; i += NT) {
      key[i] = kNone;
      cnt[i] = 0;
    }
    if (t == 0) s_nact[un] = 0;
    sync();
  }
  __syncthreads();
  c5_flush(K, bins, kCopies, threadIdx.x, BT);
}

__device__ __forceinline__ int32_t top_vertex(const int32_t* queue, const int32_t* top, const int32_t* huge, int32_t k) {
  const int32_t nh = queue[kWedgeHuge];
  return k < nh ? huge[k] : top[k - nh];
}

// The table of the first + blockIdx.y-th listed u in slice blockIdx.y: per vertex
// w nine 16-bit counts and above the ninth their sum; then the w met, and their
// number.  Several workgroups per u, as the rows phase below: the first of the
// 77 such u of the 20,000-vertex graph alone took 1,500 us as one workgroup.
constexpr int kFillParts = 8, kRowParts = 32;
__global__ __launch_bounds__(512) void k_c5_fill(DevGraph G, const int32_t* __restrict__ queue,
                                                 const int32_t* __restrict__ top, const int32_t* __restrict__ huge,
                                                 int32_t first, uint32_t* __restrict__ slices, const int32_t* st) {
  if (st[kStatus] != 0) return;
  const int t = threadIdx.x, lane = t & 63;
  uint32_t* cnt = slices + (int64_t)blockIdx.y * (6 * (int64_t)G.n + 1);
  uint32_t *act = cnt + (int64_t)5 * G.n, *nact = act + G.n;
  const int32_t u = top_vertex(queue, top, huge, first + (int32_t)blockIdx.y), ua = G.gs_off[u], ub = G.gs_off[u + 1];
  const int32_t ma = ua - G.np_off[u], dm = ub - G.np_off[u + 1] - ma;
  const uint32_t du = (uint32_t)(ub - ua);
  const int32_t group = (int32_t)blockIdx.x * 32 + (t >> 4), groups = (int32_t)gridDim.x * 32;
  for (int32_t i0 = 0; i0 < dm; i0 += groups) {
    const int32_t i = i0 + group;
    int32_t ra = 0, m = 0;
    uint32_t p = 0;
    if (i < dm) {
      const uint32_t ev = G.nm_idx[ma + i], v = ev & kIdMask;
      ra = G.gs_off[v];
      m = G.gs_off[v + 1] - ra;
      p = (ev >> kTypeShift) - 1u;
    }
    for (int32_t r = t & 15; __ballot(r < m); r += 64) {
      uint32_t f[4], old[4];
      bool in[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) f[k] = r + 16 * k < m ? G.gs_idx[ra + r + 16 * k] : 0u;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int32_t w = (int32_t)(f[k] & kIdMask);
        in[k] = r + 16 * k < m && w != u && ranked_below(G, (uint32_t)G.deg[w], w, du, u);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t j = 3 * p + (f[k] >> kTypeShift) - 1u;
        uint32_t* c = cnt + (int64_t)(f[k] & kIdMask) * 5;
        old[k] = in[k] ? atomicAdd(&c[4], j == 8 ? 0x10001u : 0x10000u) : ~0u;
        if (in[k] && j < 8) atomicAdd(&c[j >> 1], 1u << (16 * (j & 1u)));
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const u64 met = __ballot(old[k] >> 16 == 0);
        if (!met) continue;
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(nact, (uint32_t)__popcll(met));
        at = __shfl(at, 0);
        if (old[k] >> 16 == 0) act[at + __popcll(met & ((1ull << lane) - 1ull))] = f[k] & kIdMask;
      }
    }
  }
}

__global__ __launch_bounds__(256) void k_c5_rows(DevGraph G, Totals5 K, const uint32_t* __restrict__ slices,
                                                 const int32_t* st) {
  constexpr int NT = 256;
  __shared__ u64 bins[kTopCopies * 243];
  __shared__ int32_t wid[NT], row[NT], len[NT];
  if (st[kStatus] != 0) return;
  const int t = threadIdx.x;
  const uint32_t* cnt = slices + (int64_t)blockIdx.y * (6 * (int64_t)G.n + 1);
  const uint32_t* act = cnt + (int64_t)5 * G.n;
  const int32_t na = (int32_t)act[G.n];
  if ((int32_t)blockIdx.x * NT >= na) return;
  for (int i = t; i < kTopCopies * 243; i += NT) bins[i] = 0;
  u64* mine = bins + (t & (kTopCopies - 1)) * 243;
  for (int32_t x0 = (int32_t)blockIdx.x * NT; x0 < na; x0 += (int32_t)gridDim.x * NT) {
    __syncthreads();
    if (x0 + t < na) {
      const int32_t w = (int32_t)act[x0 + t], wa = G.gs_off[w] - G.np_off[w];
      wid[t] = w;
      row[t] = wa;
      len[t] = G.gs_off[w + 1] - G.np_off[w + 1] - wa;
    }
    __syncthreads();
    const int32_t nx = min(NT, na - x0);
    auto take = [&](int32_t x, int32_t l, int32_t step) {
      const int32_t wa = row[x], wm = len[x];
      uint32_t c[9];
#pragma unroll
      for (int i = 0; i < 5; ++i) {
        const uint32_t h = cnt[(int64_t)wid[x] * 5 + i];
        c[2 * i] = h & 0xFFFFu;
        if (i < 4) c[2 * i + 1] = h >> 16;
      }
      for (int32_t r0 = l; r0 < wm; r0 += 4 * step) {
        uint32_t f[4], last[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) f[k] = G.nm_idx[wa + min(r0 + k * step, wm - 1)];
#pragma unroll
        for (int k = 0; k < 4; ++k) last[k] = r0 + k * step < wm ? cnt[(int64_t)(f[k] & kIdMask) * 5 + 4] : 0u;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if (!last[k]) continue;
          uint32_t e[9];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const uint32_t h = cnt[(int64_t)(f[k] & kIdMask) * 5 + i];
            e[2 * i] = h & 0xFFFFu;
            e[2 * i + 1] = h >> 16;
          }
          e[8] = last[k] & 0xFFFFu;
          u64* to = mine + 9 * ((int)(f[k] >> kTypeShift) - 1);
#pragma unroll
          for (int p = 0; p < 9; ++p) {
            if (!c[p]) continue;
#pragma unroll
            for (int q = 0; q < 9; ++q)
              if (e[q]) atomicAdd(&to[27 * p + q], (u64)c[p] * e[q]);
          }
        }
      }
    };
    for (int32_t x = t >> 6; x < nx; x += NT / 64)
      if (len[x] > 64) take(x, t & 63, 64);
    for (int32_t x = t >> 2; x < nx; x += NT / 4)
      if (len[x] > 0 && len[x] <= 64) take(x, t & 3, 4);
  }
  __syncthreads();
  c5_flush(K, bins, kTopCopies, t, NT);
}

// ============================================================== the counts ==

// Copies of each class: its totals less the folded walks, over the times a copy
// is met.  acc4, acc3: the copies' totals of k = 4 and 3 (kRep4, kRep3 of them).
__global__ __launch_bounds__(256) void k_sum5(const uint64_t* __restrict__ acc, int copies,
                                              const uint64_t* __restrict__ acc4, const uint64_t* __restrict__ acc3,
                                              Tables5 T, uint64_t* __restrict__ P, uint64_t* __restrict__ I, int32_t* st) {
  __shared__ u64 sums[8][32];
  if (st[kStatus] != 0) return;
  const int32_t c = blockIdx.x * 32 + (threadIdx.x & 31);  // eight threads per class
  const int part = threadIdx.x >> 5;
  u64 s = 0;
  if (c < kC5) {
#pragma unroll 12
    for (int r = part; r < copies; r += 8) s += acc[(int64_t)r * kC5 + c];
    const int32_t f0 = T.fold_off[c], f1 = T.fold_off[c + 1];
    for (int32_t k = f0; k < f1; ++k) {
      const int32_t q = T.fold[k] & 0xFFFF;
      u64 n = 0;
      if (q < 199) {
#pragma unroll
        for (int r = 0; r < kRep4 / 8; ++r) n += acc4[(part + 8 * r) * 199 + q];
      } else {
#pragma unroll
        for (int r = 0; r < kRep3 / 8; ++r) n += acc3[(part + 8 * r) * 13 + q - 199];
      }
      s -= (u64)(T.fold[k] >> 16) * n;
    }
  }
  sums[part][threadIdx.x & 31] = s;
  __syncthreads();
  if (part || c >= kC5) return;
  for (int r = 1; r < 8; ++r) s += sums[r][threadIdx.x];
  const u64 m = T.mult[c];
  if (s % m) atomicMin(&st[kStatus], MOTIF_EINTERNAL);
  P[c] = I[c] = s / m;
}

// Inclusion and exclusion, one edge more at a time: P <- the copies with j
// further edges among the same vertices (each set of j met in j orders of its
// last edge), I +- P.
__global__ __launch_bounds__(256) void k_step5(Tables5 T, int j, const uint64_t* __restrict__ P,
                                               uint64_t* __restrict__ Q, uint64_t* __restrict__ I, int32_t* st) {
  if (st[kStatus] != 0) return;
  const int32_t c = blockIdx.x * 32 + (threadIdx.x >> 3), l8 = threadIdx.x & 7;
  u64 s = 0;
  if (c < kC5)
    for (int32_t k = T.up_off[c] + l8, e = T.up_off[c + 1]; k < e; k += 8) s += (u64)(T.up[k] >> 16) * P[T.up[k] & 0xFFFF];
#pragma unroll
  for (int o = 4; o; o >>= 1) s += __shfl_xor(s, o);
  if (c >= kC5 || l8) return;
  s /= (u64)j;
  Q[c] = s;
  const u64 v = j & 1 ? I[c] - s : I[c] + s;
  I[c] = v;
  if (j == 6 && (int64_t)v < 0) atomicMin(&st[kStatus], MOTIF_EINTERNAL);
}

__global__ void k_write5(const uint64_t* __restrict__ in, uint64_t* __restrict__ out, const int32_t* st) {
  if (st[kStatus] != 0) return;
  const int32_t c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c < kC5) out[c] = in[c];
}

size_t al(size_t b) { return (b + 255) & ~size_t(255); }

size_t slice_words(int64_t n) { return 6 * (size_t)n + 1; }
// Wedge tables of k_c5_fill at a time: 2 KB of them per vertex, 96 MB at most.
int c5_slices(int64_t n) {
  const size_t room = std::min<size_t>(size_t(96) << 20, size_t(2048) * (size_t)n);
  return (int)std::max<size_t>(1, std::min<size_t>((size_t)n, room / (4 * slice_words(n))));
}
// Workgroups of k_apex5, each with its copy of the totals.
// (lean: an eighth of them, for a workspace that was sized for the per-core scan.)
int apex_groups(int64_t m, bool lean) {
  const int64_t per = lean ? 128 : 16;
  return (int)std::max<int64_t>(4, std::min<int64_t>(kLocalCopies, (2 * m + per - 1) / per));
}
int shared_copies(int64_t m) { return m < 4096 ? 4 : 16; }

// Room for links: 6 per triangle.  Small dense graphs have the most per arc (n =
// 100, m = 2,000: 36; the power-law ones of 10^4 arcs and more 1 to 8).
int64_t link_room(int64_t m) { return std::max(16 * m, std::min(48 * m, int64_t(1) << 20)) + 4096; }

}  // namespace

// Up to 65,536 vertices (16-bit counts and places) and 2^20 arcs (the room
// below grows with them), and not where a third of all pairs or more are arcs:
// every vertex is then two steps from every other and each edge has thirds by
// the dozen, which the per-core scan takes in one go (n = 100, m = 5,000: 3.8 ms
// by it, 4.4 ms by copies; m = 2,000, a fifth: 1.22 and 1.03).
bool copies5_fits(int64_t n, int64_t m) {
  return n > 0 && n <= 65536 && m <= (int64_t(1) << 20) && 3 * m <= n * (n - 1);
}

size_t copies5_bytes(int64_t n, int64_t m, bool lean) {
  const size_t gs = (size_t)(2 * m + 1);
  return count_bytes(n, m, n, false, true) + 2 * al(64 * 4) + al(sizeof(uint64_t) * 13 * kRep3) +
         al(sizeof(uint64_t) * 199 * kRep4) + al(sizeof(uint64_t) * kC5 * (size_t)(shared_copies(m) + apex_groups(m, lean))) + 4 * al(sizeof(uint64_t) * kC5) +
         3 * al(4 * gs) + al(8 * (size_t)(m + 1)) + al(24 * (size_t)(m + 1)) + scan1_bytes((int64_t)gs) +
         3 * al(4 * (size_t)link_room(m)) + al(72 * (size_t)n) + al(16 * (size_t)n) + al(108 * (size_t)n) +
         kPairLists * al(4 * (size_t)n) + al(4 * slice_words(n) * (size_t)c5_slices(n)) + 8192;
}

constexpr int64_t kFewUnits = 512;
// Arcs below which the wedges of k = 4 wait until the triangles are known to fit.
constexpr int64_t kFewArcs = 32768;

void enqueue_copies5_start(Pipeline& p, const DevGraph& g, uint64_t* a3, uint64_t* a4, Copies5Run* R, hipStream_t s) {
  const int64_t n = g.n, m = (g.gs_cap - 1) / 2;
  if (!copies5_fits(n, m)) throw WorkspaceError();  // (never; the kernels' 16-bit words rest on it)
  Arena& A = p.arena;
  ZeroBatch z;
  R->a3 = a3;
  R->a4 = a4;
  R->queue = A.take<int32_t>(64);
  R->acc = A.take<uint64_t>((size_t)kC5 * (size_t)(shared_copies(m) + apex_groups(m, R->lean)));
  R->emap = A.take<uint32_t>((size_t)g.gs_cap);
  R->cnt = A.take<int32_t>((size_t)g.gs_cap);
  R->off = A.take<int32_t>((size_t)g.gs_cap);
  R->epos = A.take<int32_t>(2 * (size_t)(m + 1));
  R->hi = A.take<uint32_t>(6 * (size_t)(m + 1));
  R->tri = A.take<uint32_t>(27 * (size_t)n);
  const Scan1 sc = scan1_take(A, g.gs_cap, z);
  z.add(R->queue, 64 * sizeof(int32_t));
  z.add(a3, sizeof(uint64_t) * 13 * kRep3);
  z.add(a4, sizeof(uint64_t) * 199 * kRep4);
  z.add(R->acc, sizeof(uint64_t) * kC5 * (size_t)shared_copies(m));
  z.add(R->tri, sizeof(uint32_t) * 27 * (size_t)n);
  enqueue_zero_batch(z, s);
  // (above, the triangles run beside the wedges)
  R->counts.later = m < kFewArcs;
  enqueue_counts(p, g, a3, a4, R->queue, s, &R->counts);
  hipLaunchKernelGGL(k_edges5, dim3((unsigned)std::min<int64_t>(4096, (m + 255) / 256 + 1)), dim3(256), 0, s, g,
                     R->counts.T, R->emap, R->cnt, R->epos, R->hi, R->queue, p.status);
  enqueue_scan1(sc, R->off, LinkCount{R->cnt, g.gs_off, g.n}, p.status, s);
}

bool copies5_go(const Pipeline& p, int64_t m) {
  uint64_t links;
  static_assert(kStatusWords >= 12, "words 8 to 10");
  std::memcpy(&links, p.host_status + 8, sizeof links);
  return links <= (uint64_t)link_room(m) && p.host_status[10] <= kMaxThirds;
}

void enqueue_copies5_finish(Pipeline& p, const DevGraph& g, const Copies5Run& R, uint64_t* out, hipStream_t s) {
  const int64_t n = g.n, m = (g.gs_cap - 1) / 2;
  Arena& A = p.arena;
  const DevTables& T = dev_tables();
  const int cus = p.num_cus;
  uint32_t* idx = A.take<uint32_t>((size_t)link_room(m));
  int32_t* mate = A.take<int32_t>((size_t)link_room(m));
  int32_t* src = A.take<int32_t>((size_t)link_room(m));
  u64* S = A.take<u64>(9 * (size_t)n);
  uint4* up = A.take<uint4>((size_t)n);
  PairListsOf lists{};
  for (auto& l : lists.v) l = A.take<int32_t>((size_t)n);
  int32_t** list = lists.v;
  const int slices = c5_slices(n), tops = p.host_status[11];
  uint32_t* slice = A.take<uint32_t>((size_t)slices * slice_words(n));
  uint64_t* P[2] = {A.take<uint64_t>(kC5), A.take<uint64_t>(kC5)};
  uint64_t* I = A.take<uint64_t>(kC5);
  const int shared = shared_copies(m);
  const Totals5 K{T.lut[5], R.acc, shared};
  const Links L{R.emap, R.cnt, R.off, idx, mate, src, R.counts.T};
  auto grid = [&](int64_t items, int per, int wgs) {
    return dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>((int64_t)cus * wgs, (items + per - 1) / per)));
  };
  // Up to four chains of kernels at a time: on small graphs each lasts as long as
  // its longest unit, on larger ones they fill each other's ends.
  Chains ch(p, s);
  ch.fork(0);
  for (int first = 0; first < tops; first += slices) {
    const unsigned now = (unsigned)std::min(slices, tops - first);
    enqueue_zero(slice, sizeof(uint32_t) * now * slice_words(n), ch.on(0));
    hipLaunchKernelGGL(k_c5_fill, dim3(kFillParts, now), dim3(512), 0, ch.on(0), g, R.queue, R.counts.wedge[kWedgeTop],
                       R.counts.wedge[kWedgeHuge], first, slice, p.status);
    hipLaunchKernelGGL(k_c5_rows, dim3(kRowParts, now), dim3(256), 0, ch.on(0), g, K, slice, p.status);
  }
  hipLaunchKernelGGL((k_c5<512, 12, kWedge256>), grid(n, 1, 2), dim3(512), 0, ch.on(0), g, K, R.queue,
                     R.counts.wedge[kWedge256], p.status);
  hipLaunchKernelGGL((k_c5<256, 9, kWedge64>), grid(n, 1, 8), dim3(256), 0, ch.on(0), g, K, R.queue,
                     R.counts.wedge[kWedge64], p.status);
  hipLaunchKernelGGL((k_c5<64, 7, kWedge16>), grid(n, 4, 8), dim3(256), 0, ch.on(0), g, K, R.queue,
                     R.counts.wedge[kWedge16], p.status);
  hipLaunchKernelGGL(k_vertex5, grid(n, 4, 4), dim3(256), 0, s, g, K, S, up, p.status);
  hipLaunchKernelGGL(k_classify5, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, g, lists, R.queue, p.status);
  hipLaunchKernelGGL(k_links5, grid(m, 4, 8), dim3(256), 0, s, g, K, L, R.epos, R.hi, up, idx, mate, src, R.tri, p.status);
  ch.fork(1);
  ch.fork(2);
  auto pairs = [&](auto kernel, int hb, int units, int threads, int wgs, hipStream_t on) {
    hipLaunchKernelGGL(kernel, grid(n, units, wgs), dim3(threads), 0, on, g, K, L, R.queue, list[hb - 9], p.status);
  };
  // Below kFewUnits vertices no list fills the chip and a unit gets more threads
  // than otherwise pays (n = 115, m = 1,380: 64 to 512 threads 440 us in all).
  const bool few = n <= kFewUnits;
  hipLaunchKernelGGL(k_pairs5_block, grid(n * ((n + kPairIds - 1) / kPairIds), 1, 1), dim3(1024), 0, s, g, K, L, R.queue,
                     list[kPairBlock], p.status);
  pairs(k_pairs5<1024, 13, 1024>, 13, 1, 1024, 1, ch.on(1));
  if (few) pairs(k_pairs5<1024, 12, 1024>, 12, 1, 1024, 1, ch.on(1));
  else pairs(k_pairs5<512, 12, 512>, 12, 1, 512, 2, ch.on(1));
  if (few) pairs(k_pairs5<1024, 11, 1024>, 11, 1, 1024, 2, ch.on(2));
  else pairs(k_pairs5<256, 11, 256>, 11, 1, 256, 3, ch.on(2));
  if (few) pairs(k_pairs5<512, 10, 512>, 10, 1, 512, 4, ch.on(2));
  else pairs(k_pairs5<128, 10, 128>, 10, 1, 128, 4, ch.on(2));
  if (few) pairs(k_pairs5<256, 9, 256>, 9, 1, 256, 4, ch.on(1));
  else pairs(k_pairs5<64, 9, 256>, 9, 4, 256, 2, ch.on(1));
  const dim3 ag((unsigned)apex_groups(m, R.lean));
  hipLaunchKernelGGL(k_apex5, ag, dim3(kApexThreads), 0, s, g, T.lut[5], R.acc + (size_t)shared * kC5, L, S, p.status);
  hipLaunchKernelGGL(k_wheel5, grid(2 * m, 1, 2), dim3(256), 0, s, g, K, L, p.status);
  hipLaunchKernelGGL(k_butterfly5, grid(n, 4, 4), dim3(256), 0, s, g, K, R.tri, p.status);
  ch.join();
  const dim3 cg((kC5 + 255) / 256);
  hipLaunchKernelGGL(k_sum5, dim3((kC5 + 31) / 32), dim3(256), 0, s, R.acc, shared + (int)ag.x, R.a4, R.a3, T.five, P[0], I, p.status);
  for (int j = 1; j <= 6; ++j)
    hipLaunchKernelGGL(k_step5, dim3((kC5 + 31) / 32), dim3(256), 0, s, T.five, j, P[(j + 1) & 1], P[j & 1], I, p.status);
  hipLaunchKernelGGL(k_write5, cg, dim3(256), 0, s, I, out, p.status);
}

void sync_chains(Pipeline& p) {
  for (hipStream_t c : p.chain)
    if (c) (void)hipStreamSynchronize(c);
}

void free_chains(Pipeline& p) {
  sync_chains(p);
  for (int i = 0; i < Pipeline::kChains; ++i) {
    if (p.chain[i]) (void)hipStreamDestroy(p.chain[i]);
    if (p.ev_end[i]) (void)hipEventDestroy(p.ev_end[i]);
    p.chain[i] = nullptr;
    p.ev_end[i] = nullptr;
  }
  if (p.ev_chain) (void)hipEventDestroy(p.ev_chain);
  p.ev_chain = nullptr;
}

}  // namespace motif
