// Host plan of a run: steps and buffer placement.
#include "run.hpp"

#include <algorithm>

namespace mure {

std::vector<int> Run::reads(const Graph& g, const RunStep& s) const {
  if (s.chain >= 0) return chains[s.chain].seg.ins;
  const Node& n = g.nodes[s.v];
  std::vector<int> r(n.in, n.in + n.n_in);
  if (s.add >= 0) r.push_back(g.nodes[s.add].in[1]);
  return r;
}

std::vector<int> Run::writes(const RunStep& s) const {
  if (s.chain >= 0) return chains[s.chain].seg.outs;
  return {s.add >= 0 ? s.add : s.v};
}

Run plan_run(const Graph& g, int first, const Chains* chains, bool fuse, const std::set<int>& kept,
             const std::function<bool(const ChainSeg&)>& usable) {
  Run run;
  std::set<int> fused;                                 // ADDs computed by a convolution's launch
  for (int v = first; v <= g.out(); ++v) {
    // a fused ADD is done: no chain starts there (plan_chains)
    if (fused.count(v)) continue;
    RunStep s;
    s.v = v;
    if (chains && chains->best[v].valid() && (!usable || usable(chains->best[v]))) {
      // planned with nothing kept inside; a kept node changes its operations
      ChainSeg seg = chains->best[v];
      const auto k = kept.lower_bound(v);
      if (k == kept.end() || *k > seg.b || build_chain(g, chains->info, v, seg.b, kept, seg)) {
        s.chain = (int)run.chains.size();
        v = seg.b;
        run.chains.push_back({std::move(seg), 0});
        run.steps.push_back(s);
        continue;
      }
    }
    if (fuse && !kept.count(v)) s.add = fused_add_of(g, v);
    if (s.add >= 0) fused.insert(s.add);
    run.steps.push_back(s);
  }
  return run;
}

Placement place_buffers(const Graph& g, const Run& run, const std::set<int>& external, int mmi) {
  const int out = g.out();
  std::map<int, int> last_use;                         // node -> last step that reads it
  for (size_t i = 0; i < run.steps.size(); ++i)
    for (int p : run.reads(g, run.steps[i])) last_use[p] = (int)i;
  struct Blk { int64_t off, size; int owner; };
  std::vector<Blk> blocks;
  Placement pl;
  auto place = [&](int v) {
    if (external.count(v)) return;
    const int64_t need = (g.act_bytes(v) + 255) / 256 * 256;
    int best = -1;
    for (size_t i = 0; i < blocks.size(); ++i)
      if (blocks[i].owner < 0 && blocks[i].size >= need && (best < 0 || blocks[i].size < blocks[best].size))
        best = (int)i;
    if (best < 0) {
      blocks.push_back({pl.peak, need, v});
      pl.peak += need;
      best = (int)blocks.size() - 1;
    } else {
      blocks[best].owner = v;
    }
    pl.offset[v] = blocks[best].off;
  };
  if (mmi >= 0) place(mmi);
  for (size_t i = 0; i < run.steps.size(); ++i) {
    // free the blocks whose owner neither this step nor a later one reads
    for (Blk& b : blocks) {
      if (b.owner < 0 || b.owner == out) continue;
      const auto it = last_use.find(b.owner);
      if (it == last_use.end() || it->second < (int)i) b.owner = -1;
    }
    for (int v : run.writes(run.steps[i])) place(v);
  }
  return pl;
}

}  // namespace mure
