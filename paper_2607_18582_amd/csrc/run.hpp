// What one run of a graph's nodes launches, and where their outputs stand
// (host only, no HIP runtime calls).  A run executes nodes first .. out as
// steps in order: a chain of small nodes, a convolution with the ADD in its
// epilogue, or a single node.  Buffer placement and the executor read the same
// steps.
#pragma once

#include <functional>
#include <map>
#include <memory>
#include <set>
#include <vector>

#include "chain.hpp"
#include "plan.hpp"

namespace mure {

struct RunChain {
  std::shared_ptr<const ChainSeg> seg;
  bool own = false;                // built for this run (not one of the model's)
};

struct RunStep {
  int v = 0;                       // its first node
  int add = -1;                    // ADD computed in convolution v's epilogue
  int chain = -1;                  // chain that starts at v: index into Run::chains
};

struct Run {
  std::vector<RunChain> chains;
  std::vector<RunStep> steps;
  std::vector<int> reads(const Graph& g, const RunStep& s) const;    // nodes the step reads
  std::vector<int> writes(const RunStep& s) const;                   // nodes it stores
};

// A graph's chains by the size of the run and their first node (plan_chains),
// and what plan_run needs to build one that stores more of its nodes.
struct Chains {
  ChainInfo info;
  // null: the node runs by itself
  std::vector<std::shared_ptr<const ChainSeg>> best[CHAIN_SIZES], head[CHAIN_SIZES];
  std::vector<ChainOp> ops;        // of every chain (ChainSeg::at)
  explicit Chains(const Graph& g);
};

// Nodes first .. out as steps.  chains: the model's for runs of `size`
// (nullptr: none); a chain is taken where usable, if given, accepts it.  head:
// first - 1 is a first mutated layer.  fuse: convolutions compute their ADD.
// kept: nodes whose own output must be stored.
Run plan_run(const Graph& g, int first, const Chains* chains, int size, bool head, bool fuse, const std::set<int>& kept,
             const std::function<bool(const ChainSeg&)>& usable = {});

// Liveness-based placement of per-row activation buffers: offsets in bytes
// per row; a buffer is reused once every reader of its previous owner ran.
struct Placement {
  std::map<int, int64_t> offset;   // node -> byte offset per row
  int64_t peak = 0;                // bytes per row
};

// external: nodes whose output lives elsewhere; mmi: a node stored before the
// first step (-1: none).
Placement place_buffers(const Graph& g, const Run& run, const std::set<int>& external, int mmi = -1);

}  // namespace mure
