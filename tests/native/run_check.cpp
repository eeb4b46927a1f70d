// Host-only check of what a run launches, built with AddressSanitizer and
// UndefinedBehaviorSanitizer by tests/test_run_plan.py: over seeded random
// bf16 graphs whose residual blocks list the shortcut's projection before or
// after the main branch, a convolution is fused with its ADD only where the
// shortcut is computed before the convolution; and the thin convolution kernel
// is chosen where its blocks have enough pixels.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../../paper_2607_18582_amd/csrc/plan.hpp"

using namespace mure;

namespace {
struct Rng {  // splitmix64
  uint64_t s;
  uint64_t next() {
    uint64_t z = (s += 0x9E3779B97F4A7C15ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
  }
  int below(int n) { return n <= 0 ? 0 : (int)(next() % (uint64_t)n); }
};

struct Build {
  std::vector<Node> g;
  int h, c;
  Build(int h_, int c_) : h(h_), c(c_) {
    Node n;
    n.kind = K_INPUT;
    g.push_back(n);
  }
  int chan(int v) const { return v == 0 ? c : g[v].c_out; }
  int add(int kind, int src, int c_out, int k, int stride, int relu) {
    Node n;
    n.kind = kind; n.n_in = 1; n.in[0] = src; n.in[1] = 0;
    n.c_in = chan(src); n.c_out = c_out; n.kh = n.kw = k; n.stride = stride; n.pad = k / 2; n.relu = relu;
    g.push_back(n);
    return (int)g.size() - 1;
  }
  int conv(int src, int c_out, int k, int stride, int relu) { return add(K_CONV, src, c_out, k, stride, relu); }
  int dw(int src, int stride) { return add(K_DWCONV, src, chan(src), 3, stride, 2); }
  int sum(int a, int skip, int shortcut, int relu) {
    Node n;
    n.kind = K_ADD; n.n_in = 2; n.in[0] = a; n.in[1] = skip;
    n.c_in = chan(skip); n.c_out = chan(a); n.relu = relu; n.shortcut = shortcut;
    g.push_back(n);
    return (int)g.size() - 1;
  }
  // residual block; its projection before (0), between (1) or after (2) the
  // main branch's convolutions
  int block(int src, int c_out, int stride, int where) {
    int p = where == 0 ? conv(src, c_out, 1, stride, 0) : -1;
    const int a = conv(src, c_out, 3, stride, 1);
    if (where == 1) p = conv(src, c_out, 1, stride, 0);
    const int b = conv(a, c_out, 3, 1, 0);
    if (where == 2) p = conv(src, c_out, 1, stride, 0);
    return sum(b, p, 0, 1);
  }
  void head(int src) {
    Node n;
    n.kind = K_GAP; n.n_in = 1; n.in[0] = src; n.in[1] = 0; n.c_in = n.c_out = chan(src);
    g.push_back(n);
    Node d;
    d.kind = K_DENSE; d.n_in = 1; d.in[0] = (int)g.size() - 1; d.in[1] = 0; d.c_in = n.c_out; d.c_out = 10;
    d.kh = d.kw = d.stride = 1;
    g.push_back(d);
  }
};

Build random_graph(Rng& r) {
  const int hs[] = {4, 8, 12, 16, 32};
  Build b(hs[r.below(5)], 8 * (1 + r.below(8)));
  int x = 0, h = b.h;
  const int depth = 1 + r.below(8);
  for (int d = 0; d < depth; ++d) {
    const int st = h >= 8 && h % 2 == 0 && r.below(4) == 0 ? 2 : 1;
    switch (r.below(5)) {
      case 0: x = b.conv(x, 8 * (1 + r.below(24)), 1, 1, r.below(3)); break;
      case 1: x = b.conv(x, 8 * (1 + r.below(16)), 3, st, r.below(3)); h = (h - 1) / st + 1; break;
      case 2: x = b.dw(x, st); h = (h - 1) / st + 1; break;
      case 3: {                                        // identity shortcut
        const int a = b.conv(x, 8 * (1 + r.below(16)), 1 + 2 * r.below(2), 1, 1);
        x = b.sum(b.conv(a, b.chan(x), 1 + 2 * r.below(2), 1, 0), x, 0, r.below(3));
        break;
      }
      default: x = b.block(x, 8 * (1 + r.below(16)), st, r.below(3)); h = (h - 1) / st + 1;
    }
  }
  if (x == 0) x = b.conv(0, 16, 3, 1, 1);
  b.head(x);
  return b;
}

int64_t failures = 0, pairs = 0;

void check(const Build& b, int id) {
  Graph g;
  g.nodes = b.g;
  const std::string m = build_graph(g, b.h, b.h, b.c, DT_BF16);
  if (!m.empty()) {
    printf("graph %d: %s\n", id, m.c_str());
    ++failures;
    return;
  }
  for (int v = 1; v < (int)g.nodes.size(); ++v) {
    const int fa = fused_add_of(g, v);
    if (fa < 0) continue;
    ++pairs;
    if (g.nodes[fa].in[1] >= v && failures++ < 20)
      printf("graph %d: convolution %d adds node %d, computed after it\n", id, v, g.nodes[fa].in[1]);
  }
}

// (output height, width, columns, gathered, compact channels, chosen)
void check_thin() {
  const int t[][6] = {{32, 32, 16, 0, 0, 1}, {32, 32, 64, 0, 0, 1}, {8, 8, 48, 0, 0, 1},  {8, 8, 64, 0, 0, 0},
                      {12, 8, 64, 0, 0, 1},  {17, 8, 64, 0, 0, 0},  {17, 8, 32, 0, 0, 1}, {4, 8, 16, 0, 0, 0},
                      {1, 1, 512, 0, 0, 0},  {1, 1, 16, 0, 0, 0},   {8, 8, 12, 1, 2, 1},  {8, 8, 40, 1, 2, 0},
                      {16, 8, 40, 1, 2, 1},  {64, 64, 43, 1, 9, 1}, {64, 64, 43, 1, 0, 0}};
  for (const auto& c : t)
    if (conv_thin_pays(c[0], c[1], c[2], c[3] != 0, c[4]) != (c[5] != 0)) {
      printf("thin convolution of %d x %d, %d columns: wrong kernel\n", c[0], c[1], c[2]);
      ++failures;
    }
}
}  // namespace

int main(int argc, char** argv) {
  const int n = argc > 1 ? atoi(argv[1]) : 200;
  Rng r{77};
  check_thin();
  for (int i = 0; i < n; ++i) check(random_graph(r), i);
  printf("pairs %lld, failures %lld\n", (long long)pairs, (long long)failures);
  return failures != 0;
}
