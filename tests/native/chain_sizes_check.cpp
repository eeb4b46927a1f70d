// Host-only check of the chains planned for runs of every size, and behind a
// first mutated layer, built with AddressSanitizer and UndefinedBehaviorSanitizer
// by tests/test_chain_planner_sizes.py: each is executed symbolically
// (chain_check.cpp), over seeded random graphs and layers of every number of k
// steps; a convolution's instance holds its reduction, and chains with empty
// steps are marked.
#define main chain_check_main
#include "chain_check.cpp"
#undef main

#include "../../paper_2607_18582_amd/csrc/run.hpp"

namespace {
int64_t past = 0;

void check_sizes(Build b) {
  Graph g;
  g.nodes = b.g;
  const std::string m = build_graph(g, b.h, b.w, b.c, DT_BF16);
  if (!m.empty()) { ++failures; return; }
  const Chains chains(g);
  std::set<const ChainSeg*> seen;
  for (int z = 0; z < CHAIN_SIZES; ++z)
    for (const auto* l : {&chains.best[z], &chains.head[z]})
      for (const auto& s : *l) {
        if (!s || !seen.insert(s.get()).second) continue;
        ++segs_run;
        past += s->past;
        if (s->gmax < 1 || s->gmax * s->arena + CHAIN_EXTRA > CHAIN_LDS || (int)s->ops.size() > CHAIN_OPS) ++failures;
        Sim{g, *s, {}, {}}.run();
        bool empty = false;
        for (const ChainOp& o : s->ops) {
          if (o.kind != CH_CONV || o.code < 2) continue;
          const int ks = o.code % 1000 / 10;
          if (o.K > 32 * ks) bad("instance too small", *s, o);
          empty = empty || o.K <= 32 * (ks - 1);
        }
        if (empty != s->past) ++failures;
      }
}
}  // namespace

int main(int argc, char** argv) {
  const int n = argc > 1 ? atoi(argv[1]) : 200;
  Rng r{99};
  check_sizes(resnet20());
  check_sizes(mobilenet(nullptr));
  for (int i = 0; i < n; ++i) check_sizes(i % 8 == 0 ? mobilenet(&r) : random_graph(r));
  for (int c = 8; c <= 400; c += 8) {
    Build b = start(4, 8);
    b.head(b.conv(b.conv(b.conv(0, c, 1, 1, 1), 64, 1, 1, 2), c, 1, 1, 0));
    check_sizes(b);
    if (c > 40) continue;
    b = start(8, c);
    b.head(b.conv(b.conv(b.conv(0, c, 1, 1, 1), 48, 3, 1 + c / 8 % 2, 1), 16, 1, 1, 0));
    check_sizes(b);
  }
  printf("chains %lld, with empty steps %lld, operations %lld, failures %lld\n", (long long)segs_run, (long long)past,
         (long long)ops_run, (long long)failures);
  return failures != 0;
}
