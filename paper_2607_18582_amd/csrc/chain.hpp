// Image-resident chains: runs of consecutive bf16 nodes that one block
// computes for a few images of one mutant slot with every intermediate
// activation in LDS (k_chain.hip).  This file is the host planner (no HIP
// runtime calls): which nodes can be in a chain, where a suffix is cut into
// chains, and a chain's operations with their LDS placement.
#pragma once

#include <set>
#include <vector>

#include "kernels.hpp"
#include "plan.hpp"

namespace mure {

// One planned chain: nodes a .. b of the graph.
struct ChainSeg {
  int a = 0, b = -1;
  std::vector<ChainOp> ops;        // op.w / op.b: filled per cluster (pointer-table offsets)
  std::vector<int> ins, outs;      // external nodes read; nodes stored for later readers:
                                   // buffer i of the launch is ins[i], then outs
  int arena = 0;                   // LDS bytes per image
  int gmax = 0;                    // most images per block
  double cost = 0;                 // planner's estimate, clocks per image
  bool valid() const { return b >= a; }
};

// Nodes a .. b as one chain.  keep: nodes in it whose output must be stored
// besides those that nodes after b read; a convolution in keep does not fuse
// its ADD.  false: some node cannot be in a chain, or it does not fit.
bool build_chain(const Graph& g, int a, int b, const std::set<int>& keep, ChainSeg& s);

// What planning asks of every node, worked out once per graph.
struct ChainInfo {
  std::vector<int> fam, fused, readers, last;          // family, fused ADD, readers, last reader
  std::vector<char> ok;                                // can be in a chain
  std::vector<std::vector<int>> convs;                 // convolutions reading the node
  explicit ChainInfo(const Graph& g);
};
bool build_chain(const Graph& g, const ChainInfo& f, int a, int b, const std::set<int>& keep, ChainSeg& s);

// For every node v the chain a suffix whose next node is v starts with
// (invalid: v runs by itself), minimising the estimated cost of the whole
// suffix.
std::vector<ChainSeg> plan_chains(const Graph& g);
std::vector<ChainSeg> plan_chains(const Graph& g, const ChainInfo& f);

}  // namespace mure
