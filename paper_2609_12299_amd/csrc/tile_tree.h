// tile_tree.h -- the min-tree over the matching tiles' keys (k_resolve.hip).
// k_match writes the leaves.
#pragma once

#include "chain.h"

namespace argus {

constexpr uint32_t kTreeSub = 1024;  // leaves built by one block
constexpr int64_t kTreeInf = 0x7FFFFFFFFFFFFFFFll;

// The levels above `sub` (at most kTreeSub) consecutive nodes of the tree's
// level of sub * nsub nodes, the b-th such share of them, by 256 threads; s
// holds 2 * sub words of LDS.  A heap in LDS (node j has children 2j and
// 2j + 1; the given nodes at sub..2sub-1) whose level of `width` nodes is part
// of the tree's level of width * nsub nodes.  Nodes at or past `valid`
// count as infinite, and are written so (the leaves past the last tile).
ARGUS_DEV void tree_subtree(int64_t* tree, uint32_t sub, uint32_t b, uint32_t nsub, uint64_t valid,
                            int64_t* s) {
  const uint64_t first = (uint64_t)b * sub;
  int64_t* nodes = tree + (uint64_t)sub * nsub + first;
  for (uint32_t i = threadIdx.x; i < sub; i += 256) {
    int64_t v = kTreeInf;
    if (first + i < valid) v = (int64_t)ld_agent((const uint64_t*)&nodes[i]);
    else nodes[i] = v;
    s[sub + i] = v;
  }
  __syncthreads();
  for (uint32_t width = sub / 2; width >= 1; width >>= 1) {
    for (uint32_t k = threadIdx.x; k < width; k += 256) {
      const uint32_t node = width + k;
      const int64_t l = s[2 * node], r = s[2 * node + 1];
      const int64_t m = l < r ? l : r;
      s[node] = m;
      // (the share's root may be read by another block)
      st_agent((uint64_t*)&tree[(uint64_t)width * nsub + (uint64_t)b * width + k], (uint64_t)m);
    }
    __syncthreads();
  }
}

}  // namespace argus
