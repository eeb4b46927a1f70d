// Host planner of the image-resident chains.
#include "chain.hpp"

#include <algorithm>
#include <functional>

namespace mure {

namespace {

int ilog2(int v) {
  int l = 0;
  while ((1 << (l + 1)) <= v) ++l;
  return l;
}
bool pow2(int v) { return v > 0 && (v & (v - 1)) == 0; }
bool plane_ok(int H, int W) { return pow2(H) && pow2(W) && H >= 4 && W >= 4 && W <= 32 && H <= 32; }

// k steps of 32 that the conv16 instances exist for
constexpr int KS1[] = {1, 2, 3, 5, 9, 12};       // 1 x 1 filters
constexpr int KS3[] = {5, 9};                    // 3 x 3 filters

int ks_of(const Node& n) {
  const int need = (int)((n.fan_in + 31) / 32);
  if (n.kh == 1) {
    for (int k : KS1)
      if (k == need) return k;
  } else {
    for (int k : KS3)
      if (k == need) return k;
  }
  return 0;
}

// Channel tiles of 16 that a wave computes from one pixel fragment: more
// reuse of the fragment for the wide layers, within the registers the
// weights of all k steps take.
int tn_of(const Node& n, int cout) {
  const int t = (cout + 15) / 16;
  if (n.kh == 1 && ks_of(n) <= 2) return t % 3 == 0 || t > 4 ? 3 : t >= 2 ? 2 : 1;
  return ks_of(n) < 9 && t >= 2 ? 2 : 1;
}

bool chainable(const Graph& g, int v) {
  const Node& n = g.nodes[v];
  if (g.dtype != DT_BF16 || v == g.out() || v == 0) return false;
  if (n.kind == K_GAP) return plane_ok(n.inH, n.inW) && n.C % 8 == 0;
  if (!plane_ok(n.inH, n.inW) || !plane_ok(n.H, n.W) || n.C % 8 || n.inC % 8) return false;
  switch (n.kind) {
    case K_ADD: {
      const Node& s = g.nodes[n.in[1]];
      if (n.shortcut == 0) return true;
      return plane_ok(s.H, s.W) && s.H == 2 * n.H && s.W == 2 * n.W && s.C % 8 == 0 && ((n.C - s.C) / 2) % 8 == 0;
    }
    case K_DWCONV:
      return n.kh == 3 && n.kw == 3 && n.pad == 1 && (n.stride == 1 || n.stride == 2);
    case K_CONV: {
      if (n.maxpool || n.kh != n.kw) return false;
      const int fam = node_family(g, v);
      if (fam == FAM_HALO) return n.inC <= 64 && n.c_out <= 64;
      if (fam != FAM_BIG) return false;
      if (n.kh == 1) {
        if (n.stride != 1 || n.pad != 0) return false;
      } else if (n.kh != 3 || n.pad != 1 || n.stride > 2) {
        return false;
      }
      return ks_of(n) > 0 && n.c_out <= 512;
    }
    default:
      return false;
  }
}

// LDS layout of node t's activation for its readers in [a, b].
struct Layout {
  int bd = 0, pxb = 0, sh = 0, mask = 0;
  bool operator==(const Layout& o) const { return bd == o.bd && pxb == o.pxb && sh == o.sh && mask == o.mask; }
};

Layout layout_of(const Graph& g, const ChainInfo& f, int t, int a, int b) {
  Layout l;
  bool halo = false, other = false;
  for (int v : f.convs[t]) {
    if (v < a || v > b) continue;
    if (g.nodes[v].kh == 3) l.bd = 1;
    if (f.fam[v] == FAM_HALO) halo = true;
    else other = true;
  }
  const int C = g.nodes[t].C, slots = C / 8;
  // 32 consecutive pixels of one channel half (conv32) or 16 pixels of two
  // neighbouring slots (conv16) on distinct 16-byte slots modulo 512 bytes
  // (a swizzle only where conv32 is the one convolution that reads it)
  if (halo && !other && (C == 16 || C == 32 || C == 64)) {
    l.pxb = 2 * C;
    l.sh = C == 16 ? 4 : C == 32 ? 3 : 2;
    l.mask = C == 16 ? 1 : C == 32 ? 3 : 7;
  } else {
    l.pxb = 16 * (slots % 4 == 0 ? slots + 2 : slots);
  }
  return l;
}

// one border pixel stands between a row's end and the next row's beginning
int layout_bytes(const Layout& l, int H, int W) { return ((H + 2 * l.bd) * (W + l.bd) + l.bd) * l.pxb; }

// First-fit allocation of LDS ranges.
struct Arena {
  struct Blk { int off, size; };
  std::vector<Blk> live;
  int peak = 0;
  int alloc(int size) {
    size = (size + 127) / 128 * 128;
    std::sort(live.begin(), live.end(), [](const Blk& x, const Blk& y) { return x.off < y.off; });
    int at = 0;
    for (const Blk& b : live) {
      if (at + size <= b.off) break;
      at = std::max(at, b.off + b.size);
    }
    live.push_back({at, size});
    peak = std::max(peak, at + size);
    return at;
  }
  void release(int off) {
    for (size_t i = 0; i < live.size(); ++i)
      if (live[i].off == off) {
        live.erase(live.begin() + i);
        return;
      }
  }
};

ChainT tensor(const Layout& l, int off, int W) {
  ChainT t;
  t.off = off; t.pitch = W + l.bd; t.pxb = l.pxb; t.bd = l.bd; t.sh = l.sh; t.mask = l.mask;
  return t;
}

// dry: the cost and the LDS only, no operations.  `slice`: output channels of an expansion convolution computed at a time for
// the depthwise node after it (0: all).
bool build_with_slice(const Graph& g, const ChainInfo& f, int a, int b, const std::set<int>& keep, int slice, bool dry, ChainSeg& s) {
  s = ChainSeg();
  s.a = a;
  const int N = b + 1;
  std::vector<int> last(N, -1);                       // last reader in [a, b]
  for (int v = a; v <= b; ++v)
    for (int k = 0; k < g.nodes[v].n_in; ++k) {
      const int p = g.nodes[v].in[k];
      last[p] = v;
      if (p < a && std::find(s.ins.begin(), s.ins.end(), p) == s.ins.end()) s.ins.push_back(p);
    }
  std::sort(s.ins.begin(), s.ins.end(), std::greater<int>());   // the newest first: mmi is buffer 0
  auto stored = [&](int v) { return f.last[v] > b || keep.count(v); };
  for (int v = a; v <= b; ++v)
    if (stored(v)) s.outs.push_back(v);
  if ((int)(s.ins.size() + s.outs.size()) > CHAIN_BUFS) return false;
  auto buf_of = [&](int v) {
    for (size_t i = 0; i < s.ins.size(); ++i)
      if (s.ins[i] == v) return (int)i;
    for (size_t i = 0; i < s.outs.size(); ++i)
      if (s.outs[i] == v) return (int)(s.ins.size() + i);
    return -1;
  };
  int nops = 0;
  auto push = [&](const ChainOp& o) {
    ++nops;
    if (!dry) s.ops.push_back(o);
  };
  Arena ar;
  std::vector<Layout> lay(N);
  std::vector<int> off(N, -1);                        // LDS offset, or -1
  auto io = [&](int kind, int t) {
    const Node& n = g.nodes[t];
    ChainOp o;
    o.kind = kind;
    o.H = o.Ho = n.H; o.W = o.Wo = n.W; o.C = o.Cout = n.C;
    o.lw = ilog2(n.W); o.lp = ilog2(n.H * n.W);
    o.buf = buf_of(t);
    o.dcv = make_divu32((uint32_t)(n.C / 8));
    o.in = o.out = tensor(lay[t], off[t], n.W);
    o.zero = kind == CH_LOAD && lay[t].bd;
    push(o);
    s.cost += (double)n.out_elems() * 2 / 9;
  };
  auto release_dead = [&](int v) {                    // tensors no node after v reads
    for (int t = 0; t < N; ++t)
      if (off[t] >= 0 && last[t] <= v) {
        ar.release(off[t]);
        off[t] = -1;
      }
  };
  for (int t : s.ins) {
    const Node& n = g.nodes[t];
    if (n.C % 8 || !plane_ok(n.H, n.W)) return false;
    lay[t] = layout_of(g, f, t, a, b);
    off[t] = ar.alloc(layout_bytes(lay[t], n.H, n.W));
    io(CH_LOAD, t);
  }
  auto conv_op = [&](int v, int n0, int cout) {
    const Node& n = g.nodes[v];
    ChainOp o;
    const bool halo = f.fam[v] == FAM_HALO;
    o.kind = CH_CONV;
    o.H = n.inH; o.W = n.inW; o.C = n.inC; o.Ho = n.H; o.Wo = n.W; o.Cout = cout;
    o.K = (int)n.fan_in; o.stride = n.stride; o.relu = n.relu;
    o.lw = ilog2(n.W); o.lp = ilog2(n.H * n.W);
    o.n0 = n0;
    o.node = v;
    o.wbytes = cout * o.K * 2;
    o.woff = n0 * o.K * 2;
    if (halo) {
      o.code = 1;                                     // 0: swizzled input
      s.cost += (double)n.c_out * n.fan_in * 2 * 4 / 48;
    } else {
      const int ks = ks_of(n), tn = tn_of(n, cout);
      o.code = (n.kh == 3 ? 1000 : 0) + ks * 10 + tn;
      o.groups = (cout + 16 * tn - 1) / (16 * tn);
      o.splits = std::max(1, CHAIN_WAVES / o.groups);
      o.inv = 255 / o.groups + 1;
      s.cost += (double)cout * n.fan_in * 2 * o.splits / 48;
    }
    s.cost += 2000;
    return o;
  };
  auto dw_op = [&](int v, int n0, int c) {
    const Node& n = g.nodes[v];
    ChainOp o;
    o.kind = CH_DW;
    o.H = n.inH; o.W = n.inW; o.C = c; o.Ho = n.H; o.Wo = n.W; o.Cout = c;
    o.stride = n.stride; o.relu = n.relu; o.lw = ilog2(n.W); o.lp = ilog2(n.H * n.W);
    o.n0 = n0; o.oc = n0;
    o.node = v;
    o.wbytes = c * 18;
    o.woff = n0 * 18;
    o.dcv = make_divu32((uint32_t)(c / 4));
    s.cost += 2000;
    return o;
  };
  double per_block = 0;                               // cost shared by a block's images
  for (int v = a; v <= b; ++v) {
    const Node& n = g.nodes[v];
    if (!f.ok[v] || ar.peak + CHAIN_EXTRA > CHAIN_LDS || nops > CHAIN_OPS) return false;
    const double before = s.cost;
    if (n.kind == K_GAP) {
      if (off[n.in[0]] < 0) return false;
      ChainOp o;
      o.kind = CH_GAP;
      o.H = n.inH; o.W = n.inW; o.C = n.C; o.lw = ilog2(n.inW); o.lp = ilog2(n.inH * n.inW);
      o.in = tensor(lay[n.in[0]], off[n.in[0]], n.inW);
      o.buf = buf_of(v);
      if (o.buf < 0) return false;
      push(o);
      s.cost += 400;
      per_block += 400;
      release_dead(v);
      continue;
    }
    // an expansion and the depthwise node that alone reads it, in slices of
    // channels through a buffer of one slice
    if (slice && n.kind == K_CONV && n.kh == 1 && v + 1 <= b && g.nodes[v + 1].kind == K_DWCONV &&
        g.nodes[v + 1].in[0] == v && f.readers[v] == 1 && !stored(v) && n.c_out > slice &&
        f.fam[v] == FAM_BIG && f.ok[v + 1]) {
      const int w = v + 1;
      const Node& d = g.nodes[w];
      Layout le;
      le.bd = 1;
      le.pxb = 2 * slice;
      const int eo = ar.alloc(layout_bytes(le, n.H, n.W));
      lay[w] = layout_of(g, f, w, a, b);
      off[w] = ar.alloc(layout_bytes(lay[w], d.H, d.W));
      if (ar.peak + CHAIN_EXTRA > CHAIN_LDS) return false;
      for (int c0 = 0; c0 < n.c_out; c0 += slice) {
        const int c = std::min(slice, n.c_out - c0);
        ChainOp o = conv_op(v, c0, c);
        o.in = tensor(lay[n.in[0]], off[n.in[0]], n.inW);
        o.out = tensor(le, eo, n.W);
        o.zero = c0 == 0;                              // the slices share their border
        push(o);
        ChainOp q = dw_op(w, c0, c);
        q.in = o.out;
        q.out = tensor(lay[w], off[w], d.W);
        q.zero = c0 == 0 && lay[w].bd;
        push(q);
      }
      ar.release(eo);
      per_block += s.cost - before;
      if (stored(w)) io(CH_STORE, w);
      release_dead(w);
      v = w;
      continue;
    }
    int tgt = v;
    ChainOp o;
    if (n.kind == K_CONV) {
      o = conv_op(v, 0, n.c_out);
      const int fa = f.fused[v];
      if (fa == v + 1 && fa <= b && f.ok[fa] && !stored(v) && g.nodes[fa].in[1] != v && !n.relu) {
        const Node& an = g.nodes[fa];
        const Node& sn = g.nodes[an.in[1]];
        tgt = fa;
        o.add = an.shortcut == 1 ? 2 : 1;
        o.add_relu = an.relu;
        o.Cs = sn.C;
        o.cpad = (an.C - sn.C) / 2;
        o.skip = tensor(lay[an.in[1]], off[an.in[1]], sn.W);
      }
    } else if (n.kind == K_DWCONV) {
      o = dw_op(v, 0, n.c_out);
      o.oc = 0;
    } else {
      const Node& sn = g.nodes[n.in[1]];
      o.kind = CH_ADD;
      o.H = o.Ho = n.H; o.W = o.Wo = n.W; o.C = o.Cout = n.C;
      o.lw = ilog2(n.W); o.lp = ilog2(n.H * n.W);
      o.add = n.shortcut == 1 ? 2 : 1;
      o.add_relu = n.relu;
      o.Cs = sn.C;
      o.cpad = (n.C - sn.C) / 2;
      o.dcv = make_divu32((uint32_t)(n.C / 8));
      o.skip = tensor(lay[n.in[1]], off[n.in[1]], sn.W);
      s.cost += 600;
    }
    per_block += s.cost - before;
    if (off[n.in[0]] < 0) return false;
    o.in = tensor(lay[n.in[0]], off[n.in[0]], n.inW);
    if (o.kind == CH_CONV && f.fam[v] == FAM_HALO && o.in.mask) o.code = 0;
    const Node& tn = g.nodes[tgt];
    lay[tgt] = layout_of(g, f, tgt, a, b);
    // the sum in place of an identity shortcut that nothing reads later
    bool in_place = false;
    if (o.add == 1) {
      const int sk = g.nodes[tgt].in[1];
      const Layout& ls = lay[sk];
      if (last[sk] <= tgt && sk != n.in[0] && ls.pxb == lay[tgt].pxb && ls.sh == lay[tgt].sh &&
          ls.mask == lay[tgt].mask && ls.bd >= lay[tgt].bd) {
        lay[tgt] = ls;
        off[tgt] = off[sk];
        off[sk] = -1;
        in_place = true;
      }
    }
    if (!in_place) off[tgt] = ar.alloc(layout_bytes(lay[tgt], tn.H, tn.W));
    o.out = tensor(lay[tgt], off[tgt], tn.W);
    o.zero = lay[tgt].bd && !in_place;
    o.same = in_place;
    push(o);
    if (stored(tgt)) io(CH_STORE, tgt);
    v = tgt;
    release_dead(v);
  }
  // buffers stored by a GAP or STORE op only
  s.arena = (ar.peak + 127) / 128 * 128;
  if (s.arena + CHAIN_EXTRA > CHAIN_LDS || nops > CHAIN_OPS) return false;
  s.gmax = std::min(8, (CHAIN_LDS - CHAIN_EXTRA) / s.arena);
  s.cost += per_block * (1.0 / s.gmax - 1.0);
  s.b = b;
  return true;
}

}  // namespace

namespace {
// The cheapest way to slice the expansions of a .. b (-1: it does not fit).
double cheapest(const Graph& g, const ChainInfo& f, int a, int b, const std::set<int>& keep, int& slice) {
  bool expands = false;
  for (int v = a; v < b; ++v) expands = expands || (g.nodes[v + 1].kind == K_DWCONV && g.nodes[v].kind == K_CONV);
  double best = -1;
  int fits = 0;
  for (int sl : {0, 96, 48, 32, 16}) {
    ChainSeg t;
    if ((sl && !expands) || fits == 2) break;          // two that fit: finer ones only add operations
    if (!build_with_slice(g, f, a, b, keep, sl, true, t)) continue;
    ++fits;
    if (best >= 0 && t.cost >= best) continue;
    best = t.cost;
    slice = sl;
  }
  return best;
}
}  // namespace

ChainInfo::ChainInfo(const Graph& g) {
  const int n = (int)g.nodes.size();
  fam.resize(n); fused.resize(n); readers.assign(n, 0); last.assign(n, -1); ok.resize(n); convs.resize(n);
  for (int v = 0; v < n; ++v) {
    const Node& nd = g.nodes[v];
    fam[v] = node_family(g, v);
    fused[v] = fused_add_of(g, v);
    ok[v] = chainable(g, v);
    for (int k = 0; k < nd.n_in; ++k) {
      readers[nd.in[k]]++;
      last[nd.in[k]] = v;
    }
    if (nd.kind == K_CONV || nd.kind == K_DWCONV) convs[nd.in[0]].push_back(v);
  }
}

bool build_chain(const Graph& g, const ChainInfo& f, int a, int b, const std::set<int>& keep, ChainSeg& s) {
  int slice = 0;
  return cheapest(g, f, a, b, keep, slice) >= 0 && build_with_slice(g, f, a, b, keep, slice, false, s);
}
bool build_chain(const Graph& g, int a, int b, const std::set<int>& keep, ChainSeg& s) {
  return build_chain(g, ChainInfo(g), a, b, keep, s);
}

std::vector<ChainSeg> plan_chains(const Graph& g) { return plan_chains(g, ChainInfo(g)); }
std::vector<ChainSeg> plan_chains(const Graph& g, const ChainInfo& f) {
  const int n = (int)g.nodes.size();
  std::vector<ChainSeg> best(n);
  if (g.dtype != DT_BF16) return best;
  std::vector<double> cost(n + 1, 0);
  std::vector<int> end(n, 0), sliced(n, 0);
  for (int v = n - 1; v >= 1; --v) {
    const Node& nd = g.nodes[v];
    cost[v] = cost[v + 1] + ((double)nd.out_elems() + (double)nd.inH * nd.inW * nd.inC) * 2 / 9 + 1000;
    int fails = 0;
    for (int b = v; b < n && f.ok[b] && fails < 2; ++b) {
      // two nodes at least, and not between a convolution and the ADD that its
      // launch would fuse
      if (b == v || f.fused[b] == b + 1) continue;
      int slice = 0;
      const double c = cheapest(g, f, v, b, {}, slice);
      if (c < 0) { ++fails; continue; }
      fails = 0;
      if (c + cost[b + 1] < cost[v]) {
        cost[v] = c + cost[b + 1];
        end[v] = b;
        sliced[v] = slice;
      }
    }
  }
  for (int v = 1; v < n; ++v)
    if (end[v] && !build_with_slice(g, f, v, end[v], {}, sliced[v], false, best[v])) best[v] = ChainSeg();
  return best;
}

}  // namespace mure
