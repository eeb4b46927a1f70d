// Host plan of a run: steps and buffer placement.
#include "run.hpp"

#include <algorithm>
#include <cstring>

namespace mure {

std::vector<int> Run::reads(const Graph& g, const RunStep& s) const {
  if (s.chain >= 0) return chains[s.chain].seg->ins;
  const Node& n = g.nodes[s.v];
  std::vector<int> r(n.in, n.in + n.n_in);
  if (s.add >= 0) r.push_back(g.nodes[s.add].in[1]);
  return r;
}

std::vector<int> Run::writes(const RunStep& s) const {
  if (s.chain >= 0) return chains[s.chain].seg->outs;
  return {s.add >= 0 ? s.add : s.v};
}

Chains::Chains(const Graph& g) : info(g) {
  ChainPlan plan = plan_chains(g, info);
  // one copy of what several sizes, or the two kinds of suffix, have in common
  std::map<int, std::vector<std::shared_ptr<const ChainSeg>>> known;
  auto share = [&](ChainSeg& s) -> std::shared_ptr<const ChainSeg> {
    if (!s.valid()) return nullptr;
    for (const auto& k : known[s.a])
      if (k->b == s.b && k->ops.size() == s.ops.size() &&
          !std::memcmp(k->ops.data(), s.ops.data(), s.ops.size() * sizeof(ChainOp)))
        return k;
    s.at = (int64_t)ops.size();
    ops.insert(ops.end(), s.ops.begin(), s.ops.end());
    known[s.a].push_back(std::make_shared<const ChainSeg>(std::move(s)));
    return known[s.a].back();
  };
  for (int z = 0; z < CHAIN_SIZES; ++z) {
    for (ChainSeg& s : plan.best[z]) best[z].push_back(share(s));
    for (ChainSeg& s : plan.head[z]) head[z].push_back(share(s));
  }
}

Run plan_run(const Graph& g, int first, const Chains* chains, int size, bool head, bool fuse, const std::set<int>& kept,
             const std::function<bool(const ChainSeg&)>& usable) {
  Run run;
  int64_t at = 0;                                      // operations of the run's own chains
  std::set<int> fused;                                 // ADDs computed by a convolution's launch
  int apart = 0;                                       // nodes up to it run by themselves
  for (int v = first; v <= g.out(); ++v) {
    // a fused ADD is done: no chain starts there (plan_chains)
    if (fused.count(v)) continue;
    RunStep s;
    s.v = v;
    const std::shared_ptr<const ChainSeg> seg = !chains ? nullptr : head && v == first ? chains->head[size][v] : chains->best[size][v];
    if (seg && v > apart && (!usable || usable(*seg))) {
      RunChain c{seg, false};
      // planned with nothing kept inside; a kept node is one more store, which
      // its own launch has in any case
      const auto k = kept.lower_bound(v);
      if (k != kept.end() && *k <= c.seg->b) {
        const auto own = std::make_shared<ChainSeg>();
        if (build_chain(g, chains->info, v, c.seg->b, kept, size, *own) &&
            own->cost < layers_clocks(g, chains->info, v, c.seg->b, kept, size)) {
          own->at = at;
          at += (int64_t)own->ops.size();
          c = {own, true};
        } else {
          apart = c.seg->b;
          c.seg.reset();
        }
      }
      if (c.seg) {
        s.chain = (int)run.chains.size();
        v = c.seg->b;
        run.chains.push_back(c);
        run.steps.push_back(s);
        continue;
      }
    }
    if (fuse && !kept.count(v)) s.add = chains ? chains->info.fused[v] : fused_add_of(g, v);
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
