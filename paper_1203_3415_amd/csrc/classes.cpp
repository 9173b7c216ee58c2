// Class tables: the "hard coded" pattern -> histogram-position matrices of the
// paper (Algorithms "Count 3/4/5 Sized Patterns"; the 13x63x63 Delta-Pattern
// matrices of Section "Counting 5-sized patterns in directed graphs") folded
// into one lookup on the full k(k-1)-bit adjacency code of the k-set.
//
// Canonical code = minimum code over all k! relabellings.  The table is built
// by orbit enumeration: codes are visited in ascending order; the first code
// of an orbit not yet labelled is its minimum, so applying every permutation
// to it labels the whole orbit at once (9608 orbits x 120 permutations for
// k = 5).  Class ids are the ranks of the minima of weakly connected orbits.
//
// Multiplicity of a class = number of connected (k-2)-vertex subsets T of one
// occurrence such that both remaining vertices have a neighbour in T: these
// are exactly the anchors (a vertex, an undirected edge, a connected triple)
// whose v-/e-/Delta-Pattern set contains the occurrence (Fact "correction",
// Figure "correction:five").
#include "classes.h"

#include <algorithm>
#include <functional>
#include <map>
#include <mutex>

namespace motif {
namespace {

struct Perm {
  uint8_t to[32];  // bit b of the source code moves to bit to[b]
};

std::vector<Perm> bit_permutations(int k) {
  std::vector<int> p(k);
  for (int i = 0; i < k; ++i) p[i] = i;
  std::vector<Perm> out;
  do {
    Perm q{};
    for (int i = 0; i < k; ++i)
      for (int j = 0; j < k; ++j)
        if (i != j) q.to[code_bit(k, i, j)] = (uint8_t)code_bit(k, p[i], p[j]);
    out.push_back(q);
  } while (std::next_permutation(p.begin(), p.end()));
  return out;
}

uint32_t apply(const Perm& q, uint32_t code) {
  uint32_t out = 0;
  while (code) {
    int b = __builtin_ctz(code);
    code &= code - 1;
    out |= 1u << q.to[b];
  }
  return out;
}

// Undirected adjacency bitmasks of the k vertices.
void skeleton(int k, uint32_t code, uint32_t* nb) {
  for (int i = 0; i < k; ++i) nb[i] = 0;
  for (int i = 0; i < k; ++i)
    for (int j = 0; j < k; ++j)
      if (i != j && (code >> code_bit(k, i, j) & 1u)) {
        nb[i] |= 1u << j;
        nb[j] |= 1u << i;
      }
}

// Is the vertex subset `mask` connected in the skeleton?
bool subset_connected(const uint32_t* nb, uint32_t mask) {
  if (!mask) return false;
  uint32_t reach = mask & (~mask + 1u);
  for (;;) {
    uint32_t grow = reach;
    for (uint32_t r = reach; r; r &= r - 1) grow |= nb[__builtin_ctz(r)] & mask;
    if (grow == reach) break;
    reach = grow;
  }
  return reach == mask;
}

uint8_t anchors_seeing(int k, uint32_t code) {
  uint32_t nb[8];
  skeleton(k, code, nb);
  const uint32_t all = (1u << k) - 1u;
  int count = 0;
  for (uint32_t t = 0; t <= all; ++t) {
    if (__builtin_popcount(t) != k - 2 || !subset_connected(nb, t)) continue;
    bool dominated = true;
    for (uint32_t rest = all & ~t; rest; rest &= rest - 1)
      if (!(nb[__builtin_ctz(rest)] & t)) dominated = false;
    count += dominated;
  }
  return (uint8_t)count;
}

ClassTable build(int k) {
  ClassTable t;
  t.k = k;
  t.nbits = k * (k - 1);
  const uint32_t N = 1u << t.nbits;
  const std::vector<Perm> perms = bit_permutations(k);
  std::vector<uint32_t> orbit_min(N, UINT32_MAX);
  std::vector<uint32_t> mins;
  for (uint32_t x = 0; x < N; ++x) {
    if (orbit_min[x] != UINT32_MAX) continue;
    mins.push_back(x);  // ascending, so this is the minimum of its orbit
    for (const Perm& q : perms) orbit_min[apply(q, x)] = x;
  }
  // class ids: connected orbit minima in ascending order
  std::vector<int32_t> id_of_min_index(mins.size(), -1);
  for (size_t i = 0; i < mins.size(); ++i) {
    uint32_t nb[8];
    skeleton(k, mins[i], nb);
    if (subset_connected(nb, (1u << k) - 1u)) {
      id_of_min_index[i] = (int32_t)t.canon.size();
      t.canon.push_back(mins[i]);
      t.mult.push_back(anchors_seeing(k, mins[i]));
    }
  }
  t.lut.assign(N, 0xFFFF);
  for (uint32_t x = 0; x < N; ++x) {
    size_t i = std::lower_bound(mins.begin(), mins.end(), orbit_min[x]) - mins.begin();
    if (id_of_min_index[i] >= 0) t.lut[x] = (uint16_t)id_of_min_index[i];
  }
  // Undirected classes: the all-reciprocated directed classes.  Undirected
  // code of such a class: edge {i, j} at und_bit(k, i, j); its canonical code
  // is the minimum over all k! relabellings; ids are ranks of the canonical
  // codes, ascending.
  std::vector<int> p(k);
  std::vector<uint32_t> und_code(t.canon.size(), 0);
  std::vector<char> symmetric(t.canon.size(), 0);
  for (size_t c = 0; c < t.canon.size(); ++c) {
    const uint32_t x = t.canon[c];
    bool sym = true;
    for (int i = 0; i < k && sym; ++i)
      for (int j = 0; j < k; ++j)
        if (i != j && ((x >> code_bit(k, i, j)) & 1u) != ((x >> code_bit(k, j, i)) & 1u)) sym = false;
    if (!sym) continue;
    symmetric[c] = 1;
    uint32_t best = UINT32_MAX;
    for (int i = 0; i < k; ++i) p[i] = i;
    do {
      uint32_t u = 0;
      for (int i = 0; i < k; ++i)
        for (int j = i + 1; j < k; ++j)
          if ((x >> code_bit(k, i, j)) & 1u) {
            const int a = std::min(p[i], p[j]), b2 = std::max(p[i], p[j]);
            u |= 1u << und_bit(k, a, b2);
          }
      best = std::min(best, u);
    } while (std::next_permutation(p.begin(), p.end()));
    und_code[c] = best;
    t.und_canon.push_back(best);
  }
  std::sort(t.und_canon.begin(), t.und_canon.end());
  t.und_of.assign(t.canon.size(), -1);
  for (size_t c = 0; c < t.canon.size(); ++c)
    if (symmetric[c])
      t.und_of[c] = (int16_t)(std::lower_bound(t.und_canon.begin(), t.und_canon.end(), und_code[c]) -
                              t.und_canon.begin());
  return t;
}

std::once_flag g_once[3];
ClassTable g_tables[3];

}  // namespace

const ClassTable* class_table(int k) {
  if (k < 3 || k > 5) return nullptr;
  std::call_once(g_once[k - 3], [k] { g_tables[k - 3] = build(k); });
  return &g_tables[k - 3];
}

SubgraphInverse subgraph_inverse(int k) {
  const ClassTable* t = class_table(k);
  const int C = (int)t->canon.size();
  std::vector<std::map<int32_t, int32_t>> rows(C);
  for (int c = 0; c < C; ++c) {
    const uint32_t x = t->canon[c];
    uint32_t pair[10];
    int e = 0;
    for (int i = 0; i < k; ++i)
      for (int j = i + 1; j < k; ++j) {
        const uint32_t bits = x & (1u << code_bit(k, i, j) | 1u << code_bit(k, j, i));
        if (bits) pair[e++] = bits;
      }
    for (uint32_t out = 0; out < 1u << e; ++out) {
      uint32_t y = x;
      for (uint32_t r = out; r; r &= r - 1) y &= ~pair[__builtin_ctz(r)];
      const uint16_t sub = t->lut[y];
      if (sub != 0xFFFF) rows[sub][c] += __builtin_popcount(out) & 1 ? -1 : 1;
    }
  }
  SubgraphInverse m;
  m.off.push_back(0);
  for (int r = 0; r < C; ++r) {
    for (const auto& kv : rows[r]) {
      m.cls.push_back(kv.first);
      m.coef.push_back(kv.second);
    }
    m.off.push_back((int32_t)m.cls.size());
  }
  return m;
}



// A five-vertex sum of copies5.hip that also takes in maps of its skeleton to
// four or three vertices: the vertex pairs that may fall together, and what one
// copy's maps count for (num / den).
namespace {
struct Folded {
  int edges;
  uint8_t edge[7][2];
  int pairs;
  uint8_t pair[4][2];
  bool one;  // at most one of the pairs at a time
  int num, den;
};
const Folded kFolded[] = {
    {4, {{0, 1}, {1, 2}, {0, 3}, {3, 4}}, 3, {{2, 3}, {1, 4}, {2, 4}}, false, 1, 2},                           // path
    {4, {{0, 1}, {1, 2}, {0, 3}, {0, 4}}, 2, {{2, 3}, {2, 4}}, false, 1, 2},                                   // fork
    {5, {{0, 2}, {1, 2}, {0, 3}, {1, 3}, {0, 4}}, 1, {{1, 4}}, false, 1, 2},                                   // C4 and pendant
    {5, {{0, 1}, {0, 2}, {1, 2}, {0, 3}, {3, 4}}, 2, {{1, 4}, {2, 4}}, false, 1, 2},                           // triangle and path
    {5, {{0, 1}, {0, 2}, {1, 2}, {1, 3}, {2, 4}}, 1, {{3, 4}}, false, 1, 2},                                   // bull
    {6, {{0, 1}, {0, 2}, {1, 2}, {1, 3}, {3, 4}, {0, 4}}, 2, {{2, 3}, {2, 4}}, false, 1, 1},                   // house
    {6, {{0, 1}, {0, 2}, {1, 2}, {0, 3}, {1, 3}, {2, 4}}, 1, {{3, 4}}, false, 1, 1},                           // kite
    {6, {{0, 1}, {0, 2}, {1, 2}, {0, 3}, {0, 4}, {3, 4}}, 4, {{1, 3}, {1, 4}, {2, 3}, {2, 4}}, true, 1, 8},    // butterfly
    {7, {{0, 1}, {0, 2}, {1, 2}, {0, 3}, {1, 3}, {0, 4}, {2, 4}}, 1, {{3, 4}}, false, 1, 2},                   // gem
};

// Times a copy is met by the sums, by its skeleton.
int copies5_mult(uint32_t code) {
  uint32_t nb[8];
  skeleton(5, code, nb);
  int d[5], e = 0;
  for (int i = 0; i < 5; ++i) e += d[i] = __builtin_popcount(nb[i]);
  std::sort(d, d + 5, std::greater<int>());
  auto is = [&](int a, int b, int c, int x, int y) { return d[0] == a && d[1] == b && d[2] == c && d[3] == x && d[4] == y; };
  if (is(3, 3, 2, 2, 2) || is(3, 3, 3, 2, 1)) return e == 12 ? 2 : 1;  // house, K2,3, kite
  if (is(4, 4, 2, 2, 2) || is(3, 3, 3, 3, 2) || is(4, 4, 3, 3, 2)) return 2;
  if (e == 18) return 3;
  if (e == 20) return 5;
  return 1;
}
}  // namespace

Copies5 copies5_tables() {
  const ClassTable* t = class_table(5);
  const int C = (int)t->canon.size();
  Copies5 out;
  for (int c = 0; c < C; ++c) out.mult.push_back((uint8_t)copies5_mult(t->canon[c]));
  // one edge left out
  std::vector<std::map<int, int>> up(C);
  for (int c = 0; c < C; ++c)
    for (int i = 0; i < 5; ++i)
      for (int j = i + 1; j < 5; ++j) {
        const uint32_t bits = 1u << code_bit(5, i, j) | 1u << code_bit(5, j, i), x = t->canon[c];
        if (!(x & bits)) continue;
        const uint16_t sub = t->lut[x & ~bits];
        if (sub != 0xFFFF) ++up[sub][c];
      }
  auto csr = [](const std::vector<std::map<int, int>>& rows, std::vector<int32_t>* off, std::vector<int32_t>* ent) {
    off->push_back(0);
    for (const auto& r : rows) {
      for (const auto& kv : r) ent->push_back(kv.first | kv.second << 16);
      off->push_back((int32_t)ent->size());
    }
  };
  csr(up, &out.up_off, &out.up);
  // maps of the folded sums onto the classes of three and four vertices
  std::vector<std::map<int, int>> fold(C);
  for (int k = 3; k <= 4; ++k) {
    const ClassTable* q = class_table(k);
    for (int c = 0; c < (int)q->canon.size(); ++c) {
      uint32_t nb[8];
      skeleton(k, q->canon[c], nb);
      auto type = [&](int i, int j) {
        return (uint32_t)(q->canon[c] >> code_bit(k, i, j) & 1u) | (uint32_t)(q->canon[c] >> code_bit(k, j, i) & 1u) << 1;
      };
      uint32_t all = 0;  // the edges of the class
      for (int i = 0; i < k; ++i)
        for (int j = i + 1; j < k; ++j)
          if (nb[i] >> j & 1u) all |= 1u << (4 * i + j);
      for (const Folded& P : kFolded) {
        std::map<int, int> here;
        int f[5];
        const int total = k == 3 ? 243 : 1024;
        for (int x = 0; x < total; ++x) {
          for (int i = 0, y = x; i < 5; ++i, y /= k) f[i] = y % k;
          uint32_t met = 0, code = 0;
          bool ok = true;
          for (int e = 0; e < P.edges && ok; ++e) {
            const int i = P.edge[e][0], j = P.edge[e][1], a = f[i], b = f[j];
            if (a == b || !(nb[a] >> b & 1u)) { ok = false; break; }
            met |= 1u << (4 * std::min(a, b) + std::max(a, b));
            const uint32_t ty = type(a, b);
            if (ty & 1u) code |= 1u << code_bit(5, i, j);
            if (ty & 2u) code |= 1u << code_bit(5, j, i);
          }
          if (!ok || met != all) continue;
          int folds = 0;
          for (int i = 0; i < 5 && ok; ++i)
            for (int j = i + 1; j < 5; ++j) {
              if (f[i] != f[j]) continue;
              bool may = false;
              for (int p = 0; p < P.pairs; ++p) may |= P.pair[p][0] == i && P.pair[p][1] == j;
              ok = ok && may;
              ++folds;
            }
          if (!ok || folds == 0 || (P.one && folds > 1)) continue;
          here[t->lut[code]] += P.num;
        }
        for (const auto& kv : here) fold[kv.first][k == 3 ? 199 + c : c] += kv.second / P.den;
      }
    }
  }
  csr(fold, &out.fold_off, &out.fold);
  return out;
}

}  // namespace motif
