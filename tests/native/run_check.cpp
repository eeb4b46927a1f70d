// Host-only check of what a run launches, built with AddressSanitizer and
// UndefinedBehaviorSanitizer by tests/test_run_plan.py: over seeded random
// bf16 graphs whose residual blocks list the shortcut's projection before or
// after the main branch, a convolution is fused with its ADD only where the
// shortcut is computed before the convolution; every launch of a run reads what
// has been computed, stored and not yet overwritten, and every chain is the one
// that the graph alone gives; the blocks of a chain's launches are each taken
// once; and chains, and the thin convolution kernel, are chosen where they are
// the faster ones.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <set>
#include <vector>

#include "../../paper_2607_18582_amd/csrc/run.hpp"

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

int64_t failures = 0, pairs = 0, runs = 0, chains = 0;
const char* name = "";

void bad(int id, int first, int step, int node, const char* what) {
  if (failures++ < 20) printf("%s %d, run from %d, step %d: node %d %s\n", name, id, first, step, node, what);
}

// The steps in order.  mmi >= 0: stored before the first step (unless virt:
// the first chain reads it elsewhere); nodes before `first` are cached;
// `external` nodes have buffers of their own.
void walk(const Graph& g, const Chains& model, int size, const Run& run, int first, int mmi, bool virt,
          const std::set<int>& external, const std::set<int>& kept, int id) {
  ++runs;
  chains += (int64_t)run.chains.size();
  int64_t at = 0;
  for (const RunChain& c : run.chains) {                // as planned from the graph alone, in its table
    const ChainSeg& t = *c.seg;
    ChainSeg s;
    if (!build_chain(g, model.info, t.a, t.b, kept, size, s) || s.ops.size() != t.ops.size() || s.ins != t.ins ||
        s.outs != t.outs || s.arena != t.arena || s.gmax != t.gmax ||
        memcmp(s.ops.data(), t.ops.data(), s.ops.size() * sizeof(ChainOp)))
      bad(id, first, 0, t.a, "starts another chain than build_chain's");
    if (c.own ? t.at != at : t.at + t.ops.size() > model.ops.size() ||
                             memcmp(&model.ops[t.at], t.ops.data(), t.ops.size() * sizeof(ChainOp)))
      bad(id, first, 0, t.a, "starts a chain whose operations are elsewhere");
    if (c.own) at += (int64_t)t.ops.size();
    for (const ChainOp& o : t.ops)                       // two table entries per weighted node before it
      if (o.wbytes > 0) {
        int rank = 0;
        for (int v = 0; v < o.node; ++v) rank += g.nodes[v].weighted();
        if (o.w != rank) bad(id, first, 0, o.node, "has another rank");
      }
  }
  const Placement pl = place_buffers(g, run, external, mmi);
  std::vector<int> owner(pl.peak / 256, -1);            // buffers are whole units of 256 bytes
  std::set<int> computed;
  auto units = [&](int v) { return (g.act_bytes(v) + 255) / 256; };
  auto store = [&](int v, int i) {
    if (external.count(v)) return;
    const auto it = pl.offset.find(v);
    if (it == pl.offset.end()) { bad(id, first, i, v, "is stored and has no buffer"); return; }
    if (it->second % 256 || it->second / 256 + units(v) > (int64_t)owner.size()) { bad(id, first, i, v, "outside the workspace"); return; }
    for (int64_t u = 0; u < units(v); ++u) owner[it->second / 256 + u] = v;
  };
  auto read = [&](int p, int i) {
    if (p < first && p != mmi) return;
    if (p == mmi && virt && run.steps[i].chain >= 0 && i == 0) return;
    if (!computed.count(p)) { bad(id, first, i, p, "is read before it is computed"); return; }
    if (external.count(p)) return;
    const auto it = pl.offset.find(p);
    if (it == pl.offset.end()) { bad(id, first, i, p, "is read and has no buffer"); return; }
    for (int64_t u = 0; u < units(p); ++u)
      if (owner[it->second / 256 + u] != p) { bad(id, first, i, p, "has been overwritten"); return; }
  };
  if (mmi >= 0) {
    computed.insert(mmi);
    store(mmi, -1);
  }
  for (int i = 0; i < (int)run.steps.size(); ++i) {
    const RunStep& s = run.steps[i];
    std::set<int> done;
    if (s.chain >= 0) {
      const ChainSeg& c = *run.chains[s.chain].seg;
      for (int v = c.a; v <= c.b; ++v) done.insert(v);
    } else {
      done.insert(s.v);
      if (s.add >= 0) done.insert(s.add);
      if (s.add >= 0 && kept.count(s.v)) bad(id, first, i, s.v, "is kept and fused");
    }
    // reads come first: an output may not stand where an input still does
    for (int v : done)
      for (int k = 0; k < g.nodes[v].n_in; ++k)
        if (!done.count(g.nodes[v].in[k])) read(g.nodes[v].in[k], i);
    for (int v : run.writes(s)) store(v, i);
    for (int v : done)
      for (int k = 0; k < g.nodes[v].n_in; ++k)
        if (!done.count(g.nodes[v].in[k])) read(g.nodes[v].in[k], i);
    for (int v : done)
      if (!computed.insert(v).second) bad(id, first, i, v, "is computed twice");
    for (int v : kept)
      if (done.count(v)) {
        bool stored = false;
        for (int w : run.writes(s)) stored = stored || w == v;
        if (!stored) bad(id, first, i, v, "is kept and not stored");
      }
  }
  for (int v = first; v <= g.out(); ++v)
    if (!computed.count(v)) bad(id, first, (int)run.steps.size(), v, "is never computed");
}

void check(const Build& b, int id, Rng& r) {
  Graph g;
  g.nodes = b.g;
  const std::string m = build_graph(g, b.h, b.h, b.c, DT_BF16);
  if (!m.empty()) {
    printf("%s %d: %s\n", name, id, m.c_str());
    ++failures;
    return;
  }
  const int L = g.out();
  for (int v = 1; v <= L; ++v) {
    const int fa = fused_add_of(g, v);
    if (fa < 0) continue;
    ++pairs;
    if (g.nodes[fa].in[1] >= v) bad(id, 0, 0, v, "adds a node computed after it");
  }
  const Chains chains(g);
  for (int size = 0; size < CHAIN_SIZES; ++size) {
    auto go = [&](const Run& run, int first, int mmi, bool virt, const std::set<int>& ext, const std::set<int>& kept) {
      walk(g, chains, size, run, first, mmi, virt, ext, kept, id);
    };
    for (int mmi = 1; mmi < L; ++mmi) {
      if (!g.nodes[mmi].weighted()) continue;
      // mmi's output stored; read by the first chain only; and not by a chain
      const Run run = plan_run(g, mmi + 1, &chains, size, true, true, {});
      go(run, mmi + 1, mmi, false, {}, {});
      const ChainSeg* const head = chains.head[size][mmi + 1].get();
      bool only = head != nullptr;
      for (int v = only ? head->b + 1 : L + 1; v <= L && only; ++v)
        for (int k = 0; k < g.nodes[v].n_in; ++k) only = only && g.nodes[v].in[k] != mmi;
      if (only) go(run, mmi + 1, mmi, true, {}, {});
      const Run apart = plan_run(g, mmi + 1, &chains, size, true, true, {}, [&](const ChainSeg& s) {
        for (int p : s.ins)
          if (p == mmi) return false;
        return true;
      });
      go(apart, mmi + 1, mmi, false, {}, {});
      for (const RunStep& s : apart.steps)              // group reads rely on it
        if (s.chain < 0 && s.add < 0 && g.nodes[s.v].kind == K_ADD && g.nodes[s.v].in[1] == mmi &&
            g.nodes[s.v].in[0] > mmi && fused_add_of(g, g.nodes[s.v].in[0]) == s.v)
          bad(id, mmi + 1, 0, s.v, "reads mmi as a shortcut and is not fused");
      go(plan_run(g, mmi + 1, nullptr, 0, false, true, {}), mmi + 1, mmi, false, {}, {});
      go(plan_run(g, mmi + 1, nullptr, 0, false, false, {}), mmi + 1, mmi, false, {}, {});
    }
    for (int t = 0; t < 6; ++t) {                       // the original's run
      std::set<int> kept, ext;
      for (int v = 1; v < L; ++v)
        if (t && r.below(t > 3 ? 8 : 2) == 0) kept.insert(v);
      ext = kept;
      ext.insert(L);
      go(plan_run(g, 1, t % 2 ? &chains : nullptr, size, false, t < 4, kept), 1, -1, false, ext, kept);
      go(plan_run(g, 1, &chains, size, false, true, kept), 1, -1, false, ext, kept);
    }
  }
}

// MobileNetV2 at widths (c) and expansion t, for 32 x 32 images
Build mobilenet(int t, const std::vector<int>& c) {
  const int n[] = {1, 2, 3, 4, 3, 3, 1}, st[] = {1, 1, 2, 2, 1, 2, 1};
  Build b(32, 3);
  int x = b.conv(0, c[0], 3, 1, 2);
  for (int i = 0; i < 7; ++i)
    for (int k = 0; k < n[i]; ++k) {
      const int s = k ? 1 : st[i], ci = b.chan(x);
      int y = i == 0 ? x : b.conv(x, ci * t, 1, 1, 2);
      y = b.conv(b.dw(y, s), c[i + 1], 1, 1, 0);
      x = s == 1 && ci == c[i + 1] ? b.sum(y, x, 0, 0) : y;
    }
  b.head(b.conv(x, c[8], 1, 1, 2));
  return b;
}

// residual blocks of one width, layers behind each sum
Build residual(int h, int c, int mid, int k) {
  Build b(h, 16);
  int x = b.conv(0, c, 3, 1, 1);
  for (int i = 0; i < 2; ++i) {
    x = b.sum(b.conv(b.conv(x, mid, k, 1, 1), c, k, 1, 0), x, 0, 1);
    x = b.dw(x, 1);
    x = b.conv(x, c, 1, 1, 1);
  }
  b.head(x);
  return b;
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
// Large runs take chains where they were measured faster than their layers:
// (plane, channels, filter, layers, with a chain), the last before a GAP.
// Layers' time over the chain's: 2.1 for three 3x3 layers of 16 at 32 x 32; 0.3 for a
// 1x1 layer and its GAP there, 0.9 for 1x1 layers of 384 at 4 x 4.
void check_choice() {
  const int t[][5] = {{32, 16, 3, 8, 1}, {32, 16, 1, 1, 0}, {4, 384, 1, 4, 0}};
  for (const auto& c : t) {
    Build b(c[0], 3);
    int x = b.conv(0, c[1], 3, 1, 1);
    for (int i = 0; i < c[3]; ++i) x = b.conv(x, c[1], c[2], 1, 1);
    b.head(x);
    Graph g;
    g.nodes = b.g;
    if (!build_graph(g, b.h, b.h, b.c, DT_BF16).empty()) { ++failures; continue; }
    const Chains chains(g);
    const Run run = plan_run(g, 2, &chains, CHAIN_SIZES - 1, false, true, {});
    if (run.chains.empty() != (c[4] == 0)) {
      printf("%d x %d, %d channels, %d x %d: wrong launches\n", c[0], c[0], c[1], c[2], c[2]);
      ++failures;
    }
  }
}

// a chain's blocks over launches of CHAIN_GRID: each block once
void check_grid() {
  for (const int64_t blocks : {(int64_t)1, (int64_t)7, (int64_t)4097, (int64_t)CHAIN_GRID, (int64_t)CHAIN_GRID + 5}) {
    std::vector<char> seen((size_t)blocks, 0);
    for (int64_t b0 = 0; b0 < blocks; b0 += CHAIN_GRID) {
      const int first = (int)b0, end = (int)std::min<int64_t>(b0 + CHAIN_GRID, blocks), turns = (end - first + 7) / 8;
      for (int b = 0; b < turns * 8; ++b) {
        const int idx = chain_block(b, first, turns);
        if (idx < end && seen[(size_t)idx]++) ++failures;
      }
    }
    for (char c : seen) failures += !c;
  }
}
}  // namespace

int main(int argc, char** argv) {
  const int n = argc > 1 ? atoi(argv[1]) : 200;
  Rng r{77};
  check_thin();
  check_grid();
  check_choice();
  name = "mobilenet";
  check(mobilenet(6, {32, 16, 24, 32, 64, 96, 160, 320, 1280}), 0, r);
  check(mobilenet(6, {16, 8, 16, 16, 32, 48, 80, 160, 640}), 1, r);
  check(mobilenet(4, {32, 16, 24, 32, 64, 96, 160, 320, 1280}), 2, r);
  name = "residual";
  int id = 0;
  for (int h : {8, 16, 32})
    for (int c : {16, 24, 32, 40, 48, 64, 96, 128})
      for (int mid : {0, 128})
        for (int k : {1, 3}) check(residual(h, c, mid ? mid : c, k), id++, r);
  name = "random";
  for (int i = 0; i < n; ++i) check(random_graph(r), i, r);
  printf("runs %lld, chains %lld, pairs %lld, failures %lld\n", (long long)runs, (long long)chains, (long long)pairs,
         (long long)failures);
  return failures != 0;
}
