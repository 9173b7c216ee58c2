// Host-side class tables for the census: code -> class id and per-class
// anchor multiplicities.  See classes.cpp.
#pragma once
#include <cstdint>
#include <vector>

namespace motif {

struct ClassTable {
  int k = 0;
  int nbits = 0;                 // k(k-1)
  std::vector<uint16_t> lut;     // [2^nbits] class id, 0xFFFF = disconnected
  std::vector<uint32_t> canon;   // [C] canonical (minimum) code of each class
  std::vector<uint8_t> mult;     // [C] anchors that see one occurrence
  // Undirected classes (the connected graphs on k vertices): the directed
  // classes whose arcs are all reciprocated, one per undirected graph.
  std::vector<int16_t> und_of;    // [C] undirected class of a directed class, -1 if an arc is one-way
  std::vector<uint32_t> und_canon; // [U] canonical undirected code of each undirected class
};

// Built once per k and cached (thread-safe).  k in {3,4,5}; nullptr otherwise.
const ClassTable* class_table(int k);

// Inclusion and exclusion over the edges left out: induced count of class r =
// sum over its entries of coef * N(cls), N(c) the number of copies of class c
// as a subgraph (a vertex set with a subset of its edges, types kept).  Row r
// holds the classes with a spanning subgraph of class r; coef = (-1)^(edges
// left out) times the number of such subgraphs in one set.
struct SubgraphInverse {
  std::vector<int32_t> off, cls, coef;  // rows in CSR form
};
SubgraphInverse subgraph_inverse(int k);

// Bit of the arc i -> j in a k-vertex code.
inline int code_bit(int k, int i, int j) { return i * (k - 1) + (j < i ? j : j - 1); }

// Bit of the edge {i, j}, i < j, in a k-vertex undirected code (k(k-1)/2 bits).
inline int und_bit(int k, int i, int j) { return i * (2 * k - i - 1) / 2 + (j - i - 1); }

// Host tables of the k = 5 census by subgraph copies (copies5.hip).
struct Copies5 {
  std::vector<uint8_t> mult;             // times each class's copies are met
  std::vector<int32_t> up_off, up;       // row c: classes with one edge more, class | (edges of it that leave c) << 16
  std::vector<int32_t> fold_off, fold;   // row c: classes of four (0 ..) and three (199 ..) vertices whose copies the
                                         // sums of c take in, class | times << 16
};
Copies5 copies5_tables();

}  // namespace motif
