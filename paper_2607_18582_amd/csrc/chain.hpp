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
  std::vector<ChainOp> ops;
  std::vector<int> ins, outs;      // external nodes read; nodes stored for later readers:
                                   // buffer i of the launch is ins[i], then outs
  int arena = 0;                   // LDS bytes per image
  int gmax = 0;                    // most images per block
  bool past = false;               // some convolution leaves steps of its instance empty
  double cost = 0;                 // planner's estimate, clocks per image
  int64_t at = 0;                  // its first operation in its table of operations
  bool valid() const { return b >= a; }
};

// What planning asks of every node, worked out once per graph.
struct ChainInfo {
  std::vector<int> fam, fused, readers, last;          // family, fused ADD, readers, last reader
  std::vector<int> rank;                               // weighted nodes before it
  std::vector<char> ok;                                // can be in a chain
  std::vector<std::vector<int>> convs;                 // convolutions reading the node
  explicit ChainInfo(const Graph& g);
};

// Runs are of four sizes, by their rows (slots x inputs): few rows are bound by
// launches and an operation's latency, many by the work.
constexpr int CHAIN_SIZES = 4;
constexpr int CHAIN_ROWS[CHAIN_SIZES] = {256, 1024, 4096, 32768};   // planned for
inline int chain_size(int64_t rows) { return rows < 512 ? 0 : rows < 2048 ? 1 : rows < 8192 ? 2 : 3; }
// Images per block for a launch of nx images of each of nslots slots: fewer
// than fit while the launch would leave the chip idle.
inline int chain_images(int gmax, int64_t nx, int64_t nslots) {
  int G = gmax;
  while (G > 1 && (nx + G - 1) / G * nslots < 1024) --G;
  return G;
}

// Nodes a .. b as one chain.  keep: nodes in it whose output must be stored
// besides those that nodes after b read; a convolution in keep does not fuse
// its ADD.  false: some node cannot be in a chain, or it does not fit.
bool build_chain(const Graph& g, const ChainInfo& f, int a, int b, const std::set<int>& keep, int size, ChainSeg& s);
bool build_chain(const Graph& g, int a, int b, const std::set<int>& keep, ChainSeg& s);   // size 0, of the most chains

// Estimated clocks per image of nodes a .. b as launches of their own.
double layers_clocks(const Graph& g, const ChainInfo& f, int a, int b, const std::set<int>& keep, int size);

// For runs of each size and every node v the chain a suffix whose next node is
// v starts with (invalid: v runs by itself), minimising the estimated time of
// the whole suffix.  head: the suffix of the first mutated layer v - 1, whose
// output a chain reads through the mutants' channel maps and a layer reads
// from a copy per mutant.
struct ChainPlan {
  std::vector<ChainSeg> best[CHAIN_SIZES], head[CHAIN_SIZES];
};
ChainPlan plan_chains(const Graph& g, const ChainInfo& f);
std::vector<ChainSeg> plan_chains(const Graph& g);                                        // size 0, of the most chains

}  // namespace mure
