// What the host knows of a trie's size without asking the device: it chooses the kernel and the
// launch shape of an attention call (the kernels read the real size, and take any).
//
// A pure function of the trie's start (td_init_prompt, td_load_state) and of the depth of its
// leaves, which every append moves down by one: each append adds b nodes, all at one new depth,
// and a collection under a window drops whole levels.  What a collection drops of the levels
// that stay is not counted (only the device knows): without a window the bound runs ahead of a
// trie whose beams share most of their path.
#pragma once

#include <algorithm>
#include <cstdint>

namespace td {

struct NodeBound {
  int32_t nodes = 0;  // stored nodes at the start
  int32_t depth = 0;  // depth of the leaves at the start
  int32_t first = 0;  // depth of the first stored node at the start
  int32_t trunk = 0;  // the levels above this depth hold one node of a live path each
};

// A trie's parameters: beams, window (0 = none), collection interval, slots.
struct TrieShape {
  int32_t b, W, G, cap;
};

// Lowest depth that may be stored.  The last G appends hold a collection, which keeps the W levels
// that end at its new leaves.
inline long lowest_depth(const NodeBound& n, const TrieShape& s, int32_t leaf_depth) {
  if (s.W <= 0 || leaf_depth - n.depth < s.G) return n.first;
  return std::max<long>(n.first, (long)leaf_depth - (s.G - 1) - s.W + 1);
}

// At least the nodes stored when the leaves are at leaf_depth.
inline long node_bound(const NodeBound& n, const TrieShape& s, int32_t leaf_depth) {
  long most = n.nodes + (long)s.b * (leaf_depth - n.depth);
  const long low = lowest_depth(n, s, leaf_depth);
  if (low > n.first)  // (collected: one node per level of the trunk, up to b per level past it)
    most = std::min(most, std::max(0l, n.trunk - low) + s.b * (leaf_depth + 1 - std::max<long>(n.trunk, low)));
  return std::max(1l, std::min<long>(most, s.cap));
}

// At least the nodes of any later step: what a call recorded in a graph may find when replayed.
inline long node_limit(const NodeBound& n, const TrieShape& s, int32_t leaf_depth) {
  if (s.W <= 0) return s.cap;
  const long steady = (long)s.b * (s.W + s.G - 1);
  return std::min<long>(s.cap, std::max(node_bound(n, s, leaf_depth) + (long)s.b * s.G, steady));
}

// Estimate of the key range of `queries` nodes that follow one another: their window, at the
// trie's mean number of nodes per level, and themselves.  (No bound: the levels are uneven, and a
// caller may give the nodes in any order.)
inline long window_keys(const NodeBound& n, const TrieShape& s, int32_t leaf_depth, long nodes, int queries) {
  if (s.W <= 0) return nodes;
  const long levels = std::max(1l, leaf_depth + 1 - lowest_depth(n, s, leaf_depth));
  return std::min(nodes, ((long)s.W * nodes + levels - 1) / levels + queries);
}

}  // namespace td
