// Host-only check of the chain planner (paper_2607_18582_amd/csrc/chain.cpp),
// built with AddressSanitizer and UndefinedBehaviorSanitizer by
// tests/test_chain_planner.py.  Every planned chain of the seeded random bf16
// graphs, and of ResNet-20- and MobileNetV2-shaped ones, is executed
// symbolically: each 16-byte LDS slot holds a tag (node, pixel, 8-channel
// group), and every operation checks that the slots it reads hold what its
// node reads -- zeros around the image -- and stay inside the image's arena.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <set>
#include <vector>

#include "../../paper_2607_18582_amd/csrc/chain.hpp"

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
  int h, w, c;
  int add(int kind, int src, int c_out, int k, int stride, int relu) {
    Node n;
    n.kind = kind; n.n_in = 1; n.in[0] = src; n.in[1] = 0;
    n.c_in = chan(src); n.c_out = c_out; n.kh = n.kw = k; n.stride = stride; n.pad = k / 2; n.relu = relu;
    n.C = c_out;
    g.push_back(n);
    return (int)g.size() - 1;
  }
  int chan(int v) { return v == 0 ? c : g[v].c_out; }
  int conv(int src, int c_out, int k, int stride, int relu) { return add(K_CONV, src, c_out, k, stride, relu); }
  int dw(int src, int stride) { return add(K_DWCONV, src, chan(src), 3, stride, 2); }
  int sum(int a, int skip, int shortcut, int relu) {
    Node n;
    n.kind = K_ADD; n.n_in = 2; n.in[0] = a; n.in[1] = skip;
    n.c_in = chan(skip); n.c_out = chan(a); n.relu = relu; n.shortcut = shortcut;
    g.push_back(n);
    return (int)g.size() - 1;
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

Build start(int h, int c) {
  Build b;
  b.h = b.w = h; b.c = c;
  Node n;
  n.kind = K_INPUT;
  b.g.push_back(n);
  return b;
}

Build resnet20() {
  Build b = start(32, 3);
  int x = b.conv(0, 16, 3, 1, 1);
  for (int s = 0; s < 3; ++s)
    for (int k = 0; k < 3; ++k) {
      const int c = 16 << s, st = s && !k ? 2 : 1;
      const int a = b.conv(x, c, 3, st, 1);
      x = b.sum(b.conv(a, c, 3, 1, 0), x, st == 2, 1);
    }
  b.head(x);
  return b;
}

Build mobilenet(Rng* r) {
  Build b = start(32, 3);
  int x = b.conv(0, 16, 3, 1, 2);
  const int t[] = {1, 6, 6, 6, 6}, c[] = {8, 16, 24, 48, 64}, n[] = {1, 2, 3, 3, 2}, st[] = {1, 2, 2, 2, 1};
  for (int i = 0; i < 5; ++i) {
    const int co = r ? 8 * (1 + r->below(9)) : c[i], ex = r ? 1 + r->below(6) : t[i];
    for (int k = 0; k < n[i]; ++k) {
      const int s = k ? 1 : st[i], ci = b.chan(x);
      int y = ex == 1 ? x : b.conv(x, ci * ex, 1, 1, 2);
      y = b.conv(b.dw(y, s), co, 1, 1, 0);
      x = s == 1 && ci == co ? b.sum(y, x, 0, 0) : y;
    }
  }
  x = b.conv(x, 320, 1, 1, 2);
  b.head(x);
  return b;
}

Build random_graph(Rng& r) {
  const int hs[] = {4, 8, 16, 32};
  Build b = start(hs[r.below(4)], 8 * (1 + r.below(8)));
  int x = 0, h = b.h;
  std::vector<int> hw(1, h);
  const int depth = 2 + r.below(10);
  for (int d = 0; d < depth; ++d) {
    const int c = b.chan(x), st = h >= 8 && r.below(4) == 0 ? 2 : 1;
    switch (r.below(5)) {
      case 0: x = b.conv(x, 8 * (1 + r.below(12)), 1, 1, r.below(3)); break;
      case 1: x = b.conv(x, 16 * (1 + r.below(4)), 3, st, r.below(3)); h /= st; break;
      case 2: x = b.dw(x, st); h /= st; break;
      case 3: {                                        // residual block, identity
        const int a = b.conv(x, c, 3, 1, 1);
        x = b.sum(b.conv(a, c, 3, 1, 0), x, 0, r.below(3));
        break;
      }
      default: {                                       // residual block, option A
        if (h < 8) break;
        const int a = b.conv(x, c + 16, 3, 2, 1);
        x = b.sum(b.conv(a, c + 16, 3, 1, 0), x, 1, 1);
        h /= 2;
      }
    }
  }
  if (x == 0) x = b.conv(0, 16, 3, 1, 1);
  b.head(x);
  return b;
}

int64_t failures = 0, ops_run = 0, segs_run = 0;
void bad(const char* what, const ChainSeg& s, const ChainOp& o) {
  if (failures++ < 20)
    fprintf(stderr, "chain %d..%d op kind %d node %d: %s\n", s.a, s.b, o.kind, o.node, what);
}

using Tag = int64_t;
constexpr Tag ZERO = -1, NONE = -2;
Tag tag(int node, int y, int x, int grp) { return (((int64_t)node * 64 + y) * 64 + x) * 4096 + grp; }

struct Sim {
  const Graph& g;
  const ChainSeg& s;
  std::vector<Tag> lds;
  std::map<int, int> at;                               // tensor offset -> node held (by last write)
  int slot(const ChainT& t, int y, int x, int byte, const ChainOp& o) {   // y, x may be -1 or H, W with a border
    const int p = (y + t.bd) * t.pitch + x + t.bd;
    const int ad = t.off + p * t.pxb + (byte ^ (((p >> t.sh) & t.mask) << 4));
    if (p < 0 || ad < 0 || ad % 16 || ad + 16 > s.arena) { bad("address outside the arena", s, o); return 0; }
    if (byte >= t.pxb) { bad("channel outside the pixel", s, o); return 0; }
    return ad / 16;
  }
  void expect(const ChainT& t, int y, int x, int grp, Tag want, const ChainOp& o) {
    if (lds[slot(t, y, x, grp * 16, o)] != want) bad("reads a slot that does not hold its input", s, o);
  }
  void border(const ChainOp& o, const ChainT& t, int H, int W) {
    for (int y = -1; y <= H; ++y)
      for (int x = -1; x <= W; ++x)
        if (y < 0 || x < 0 || y == H || x == W)
          for (int v = 0; v < t.pxb / 16; ++v) {
            const int p = (y + 1) * t.pitch + x + 1;
            lds[(t.off + p * t.pxb + v * 16) / 16] = ZERO;
          }
  }
  // input node, channel slice [n0, n0 + c) of node v's input tensor for slices
  void run() {
    lds.assign(s.arena / 16, NONE);
    std::map<int, int> slice0;                         // E buffer offset -> (node, n0) for sliced expansions
    size_t ins = s.ins.size();
    std::set<int> stored;
    for (size_t k = 0; k < s.ops.size(); ++k) {
      const ChainOp& o = s.ops[k];
      ++ops_run;
      const int H = o.H, W = o.W;
      if (o.kind == CH_LOAD) {
        if (o.zero) border(o, o.out, H, W);
        for (int y = 0; y < H; ++y)
          for (int x = 0; x < W; ++x)
            for (int v = 0; v < o.C / 8; ++v) lds[slot(o.out, y, x, v * 16, o)] = tag(s.ins[o.buf], y, x, v);
        continue;
      }
      if (o.kind == CH_STORE || o.kind == CH_GAP) {
        const int out = s.outs.at(o.buf - ins);
        const int node = o.kind == CH_GAP ? g.nodes[out].in[0] : out;
        stored.insert(out);
        for (int y = 0; y < H; ++y)
          for (int x = 0; x < W; ++x)
            for (int v = 0; v < o.C / 8; ++v) expect(o.in, y, x, v, tag(node, y, x, v), o);
        continue;
      }
      // the node computed and its input
      int v = o.node, src;
      if (o.kind == CH_ADD) {
        v = -1;
        for (int q = s.a; q <= s.b; ++q)               // the ADD whose operands are resident
          if (g.nodes[q].kind == K_ADD && lds[slot(o.in, 0, 0, 0, o)] == tag(g.nodes[q].in[0], 0, 0, 0) &&
              lds[slot(o.skip, 0, 0, o.add == 2 ? 0 : 0, o)] == tag(g.nodes[q].in[1], 0, 0, 0)) v = q;
        if (v < 0) { bad("no such ADD", s, o); continue; }
      }
      const Node& n = g.nodes[v];
      src = n.in[0];
      const int cs = o.kind == CH_DW ? o.n0 / 8 : 0;   // first input group the op's tensor holds
      const bool sliced = o.kind == CH_DW && o.C < n.c_out;
      const int kk = o.kind == CH_ADD ? 1 : n.kh;
      for (int y = 0; y < o.Ho; ++y)
        for (int x = 0; x < o.Wo; ++x)
          for (int dy = 0; dy < kk; ++dy)
            for (int dx = 0; dx < kk; ++dx) {
              const int st = o.kind == CH_ADD ? 1 : o.stride;
              const int iy = y * st + dy - kk / 2, ix = x * st + dx - kk / 2;
              const bool out = iy < 0 || ix < 0 || iy >= n.inH || ix >= n.inW;
              for (int q = 0; q < o.C / 8; ++q)
                expect(o.in, iy, ix, q, out ? ZERO : tag(src, iy, ix, (o.kind == CH_DW ? cs : 0) + q), o);
            }
      (void)sliced;
      int wr = v;
      if (o.add) {
        if (o.kind != CH_ADD) wr = v + 1;
        const Node& an = g.nodes[wr];
        const int f = o.add == 2 ? 2 : 1;
        for (int y = 0; y < o.Ho; ++y)
          for (int x = 0; x < o.Wo; ++x)
            for (int q = 0; q < o.Cs / 8; ++q) expect(o.skip, f * y, f * x, q, tag(an.in[1], f * y, f * x, q), o);
      }
      if (o.zero) border(o, o.out, o.Ho, o.Wo);
      // a sliced expansion writes groups n0/8 .. of its node into a buffer of
      // the slice; everything else writes at channel oc of the whole tensor
      for (int y = 0; y < o.Ho; ++y)
        for (int x = 0; x < o.Wo; ++x)
          for (int q = 0; q < o.Cout / 8; ++q)
            lds[slot(o.out, y, x, 2 * o.oc + q * 16, o)] =
                tag(wr, y, x, o.kind == CH_DW ? o.oc / 8 + q : o.n0 / 8 + q);
    }
    for (int q : s.outs)
      if (!stored.count(q)) { ++failures; fprintf(stderr, "chain %d..%d: node %d not stored\n", s.a, s.b, q); }
  }
};

void check(Build b, Rng& r, bool print) {
  Graph g;
  g.nodes = b.g;
  const std::string m = build_graph(g, b.h, b.w, b.c, DT_BF16);
  if (!m.empty()) return;
  std::vector<ChainSeg> segs = plan_chains(g);
  for (int v = 1; v < (int)g.nodes.size(); ++v) {
    const ChainSeg& s = segs[v];
    if (!s.valid()) continue;
    if (print)
      printf("start %d: nodes %d..%d ops %zu arena %d gmax %d cost %.0f\n", v, s.a, s.b, s.ops.size(), s.arena, s.gmax, s.cost);
    if (s.gmax * s.arena + CHAIN_EXTRA > CHAIN_LDS) ++failures;
    Sim{g, s, {}, {}}.run();
    ++segs_run;
    // the original's run: some nodes kept
    std::set<int> keep;
    for (int q = s.a; q <= s.b; ++q)
      if (r.below(2)) keep.insert(q);
    ChainSeg t;
    if (build_chain(g, s.a, s.b, keep, t)) {
      Sim{g, t, {}, {}}.run();
      ++segs_run;
    }
  }
}
}  // namespace

int main(int argc, char** argv) {
  const int n = argc > 1 ? atoi(argv[1]) : 200;
  Rng r{2024};
  const bool print = argc > 2;
  check(resnet20(), r, print);
  if (print) printf("mobilenet\n");
  check(mobilenet(nullptr), r, print);
  for (int i = 0; i < n; ++i) check(i % 8 == 0 ? mobilenet(&r) : random_graph(r), r, false);
  printf("chains %lld, operations %lld, failures %lld\n", (long long)segs_run, (long long)ops_run, (long long)failures);
  return failures != 0;
}
