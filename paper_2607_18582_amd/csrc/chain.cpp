// Host planner of the image-resident chains.
#include "chain.hpp"

#include <algorithm>
#include <functional>
#include <map>

namespace mure {

namespace {

int ilog2(int v) {
  int l = 0;
  while ((1 << (l + 1)) <= v) ++l;
  return l;
}
bool pow2(int v) { return v > 0 && (v & (v - 1)) == 0; }
bool plane_ok(int H, int W) { return pow2(H) && pow2(W) && H >= 4 && W >= 4 && W <= 32 && H <= 32; }

// Most k steps of 32 of a conv16 instance, of the fewest that hold the node's
// reduction (0: none does): a wave keeps their weights in registers, and the
// offsets of the taps beside them (3 x 3: up to 32 channels).
constexpr int STEPS1[] = {1, 2, 3, 5, 9, 12}, STEPS3[] = {5, 9};

int ks_of(const Node& n) {
  const int64_t need = (n.fan_in + 31) / 32;
  if (n.kh == 1) {
    for (int k : STEPS1)
      if (need <= k) return k;
  } else {
    for (int k : STEPS3)
      if (need <= k) return k;
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

// An operation as far as its time goes: pixels, channels (in, out) of its
// output tensor, and for a convolution its instance and split.
struct ChainWork {
  int kind, px, c, cout;
  int ks, tn, groups, splits;
};

// Clocks of an operation of a block of G images, two blocks on the CU: a least
// squares fit to 860 chains of 2 to 40 operations over some 16,000 images
// (seeded networks, residual and inverted residual ones; planes of 4 to 32, 8
// to 512 channels).  The sums are 0.8 to 1.13 of the measured time from the
// 5th to the 95th percentile.  Per operation what its latency costs, then what
// its turns of a wave, and its bytes, do.
double op_clocks(const ChainWork& w, int G) {
  auto up = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
  const int64_t n = (int64_t)G * w.px;
  constexpr int NT = CHAIN_WAVES * 64;
  switch (w.kind) {
    case CH_LOAD: return 4100 + 0.12 * (double)(n * w.c * 2);
    case CH_STORE: return 6700 + 0.13 * (double)(n * w.c * 2);
    case CH_DW: return 1650 + 1430.0 * up(n * w.cout / 16, NT) + 3050.0 / 16 / NT * (double)(n * w.cout);
    case CH_ADD: return 1900.0 * up(n * w.c / 8, NT);
    case CH_GAP: return 10600 + 86.0 * w.px * up(G * up(w.c, 64), CHAIN_WAVES);
    default: break;
  }
  if (!w.ks) {                                         // conv32: items of 32 pixels x 32 channels
    const int64_t items = up(n, 32) * (w.cout / 32);
    return up(items, CHAIN_WAVES) * (5400 + 49.0 * w.c) + 7.5 * w.c * (double)std::min<int64_t>(items, CHAIN_WAVES);
  }
  const int tp = w.tn * w.ks <= 6 ? 2 : 1;             // conv16: w.c its whole reduction
  const int64_t it = up(up(up(n, 16), tp), w.splits) * up(w.groups, CHAIN_WAVES);
  // weights past the 64 KB that the operation before touches into the cache
  const double cold = std::max(0.0, 2.0 * w.cout * w.c - 65536);
  return 450 + 0.15 * w.cout * w.c * w.splits + 0.05 * cold + it * (1120.0 + 180 * tp * w.tn);
}

// `slice`: output channels of an expansion convolution computed at a time for
// the depthwise node after it (0: all).  work: what the operations do, instead
// of the operations themselves (nullptr: the operations).
bool build_with_slice(const Graph& g, const ChainInfo& f, int a, int b, const std::set<int>& keep, int slice,
                      std::vector<ChainWork>* work, ChainSeg& s) {
  s = ChainSeg();
  if (work) work->clear();
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
    if (!work) {
      s.ops.push_back(o);
      return;
    }
    const bool c16 = o.kind == CH_CONV && o.code > 1;
    const int px = o.kind == CH_GAP ? o.H * o.W : o.Ho * o.Wo;
    work->push_back({o.kind, px, c16 ? o.K : o.C, o.Cout, c16 ? o.code % 1000 / 10 : 0, c16 ? o.code % 10 : 0, o.groups, o.splits});
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
    o.w = f.rank[v];
    o.wbytes = cout * o.K * 2;
    o.woff = n0 * o.K * 2;
    if (halo) {
      o.code = 1;                                     // 0: swizzled input
    } else {
      const int ks = ks_of(n), tn = tn_of(n, cout);
      s.past = s.past || n.fan_in <= 32 * (ks - 1);
      o.code = (n.kh == 3 ? 1000 : 0) + ks * 10 + tn;
      o.groups = (cout + 16 * tn - 1) / (16 * tn);
      o.splits = std::max(1, CHAIN_WAVES / o.groups);
      o.inv = 255 / o.groups + 1;
    }
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
    o.w = f.rank[v];
    o.wbytes = c * 18;
    o.woff = n0 * 18;
    o.dcv = make_divu32((uint32_t)(c / 4));
    return o;
  };
  for (int v = a; v <= b; ++v) {
    const Node& n = g.nodes[v];
    if (!f.ok[v] || ar.peak + CHAIN_EXTRA > CHAIN_LDS || nops > CHAIN_OPS) return false;
    if (n.kind == K_GAP) {
      if (off[n.in[0]] < 0) return false;
      ChainOp o;
      o.kind = CH_GAP;
      o.H = n.inH; o.W = n.inW; o.C = n.C; o.lw = ilog2(n.inW); o.lp = ilog2(n.inH * n.inW);
      o.in = tensor(lay[n.in[0]], off[n.in[0]], n.inW);
      o.buf = buf_of(v);
      if (o.buf < 0) return false;
      push(o);
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
    }
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
  s.b = b;
  return true;
}

}  // namespace

namespace {
// Whole runs of 125 networks layer by layer against their chains, by the size
// of the run (256, 1,024, 4,096, and 16,384 and 65,536 rows): what a launch less
// saves (nothing where launches queue up behind each other), and a chain's
// operations against its layers, both by the estimates here -- few rows leave
// a block its CU alone; in large runs layers wait for the activations that the
// ones before them still write.  Measured 0.73, 0.92, 0.94 and 0.9; a little
// more here, where a last turn of blocks is often nearly empty and against the
// estimates' error.
constexpr double LAUNCH_US[CHAIN_SIZES] = {6, 6, 3.5, 0.5}, CHAIN_SCALE[CHAIN_SIZES] = {0.75, 1, 1, 0.95};
// Estimates per image are in clocks of one of 256 CUs.
double launch_clocks(int size) { return LAUNCH_US[size] * 256 * 2400 / CHAIN_ROWS[size]; }
constexpr double ADD_READ = 0.09;                      // a byte of the shortcut, in a convolution's launch

// Estimated clocks per image of a chain of these operations in runs of each size.
void chain_clocks(const std::vector<ChainWork>& work, int gmax, double (&clocks)[CHAIN_SIZES]) {
  int last = 0;
  double t = 0;
  for (int z = 0; z < CHAIN_SIZES; ++z) {
    const int G = chain_images(gmax, CHAIN_ROWS[z], 1);
    if (G != last) {
      t = 0;
      for (const ChainWork& w : work) t += op_clocks(w, G);
      last = G;
    }
    clocks[z] = CHAIN_SCALE[z] * t / (2 * G) + launch_clocks(z);
  }
}

// The cheapest way to slice the expansions of a .. b for runs of each size:
// clocks per image and the slice.  false: it does not fit.
bool cheapest(const Graph& g, const ChainInfo& f, int a, int b, const std::set<int>& keep, std::vector<ChainWork>& work,
              double (&best)[CHAIN_SIZES], int (&slice)[CHAIN_SIZES]) {
  bool expands = false;
  for (int v = a; v < b; ++v) expands = expands || (g.nodes[v + 1].kind == K_DWCONV && g.nodes[v].kind == K_CONV);
  int fits = 0;
  for (int sl : {0, 96, 48, 32, 16}) {
    ChainSeg t;
    if ((sl && !expands) || fits == 2) break;          // two that fit: finer ones only add operations
    if (!build_with_slice(g, f, a, b, keep, sl, &work, t)) continue;
    double c[CHAIN_SIZES];
    chain_clocks(work, t.gmax, c);
    for (int z = 0; z < CHAIN_SIZES; ++z) {
      if (fits && c[z] >= best[z]) continue;
      best[z] = c[z];
      slice[z] = sl;
    }
    ++fits;
  }
  return fits > 0;
}

// Estimated clocks per image of node v as a launch of its own: its bytes, and
// for a convolution the work of its tiles; a fit to 2,400 layers of the same
// networks, 0.8 to 1.15 of the measured time.
double layer_clocks(const Graph& g, const ChainInfo& f, int v, int size) {
  const Node& n = g.nodes[v];
  auto up = [](int64_t a, int64_t b) { return (double)((a + b - 1) / b * b); };
  const double in = 2.0 * n.inH * n.inW * n.inC, out = 2.0 * n.out_elems(), px = (double)n.Hc * n.Wc;
  const double t = launch_clocks(size);
  if (n.kind == K_ADD) return t + 0.22 * out;
  if (n.kind == K_GAP) return t + 0.1 * in + 1.25 * n.inH * n.inW;
  if (n.kind == K_CONV) {
    const double macs = px * n.c_out * n.fan_in;
    if (f.fam[v] == FAM_HALO) return t + 0.113 * in + 0.19 * out + 0.0005 * macs;
    if (f.fam[v] == FAM_VALU) return t + 0.052 * in + 0.424 * out + 0.008 * macs;
    return t + 0.077 * in + 0.06 * out + px * (0.247 * up(n.c_out, 16) + 0.0008 * up(n.c_out, 64) * up(n.fan_in, 32));
  }
  return t + 0.09 * in + 0.2 * out;
}
}  // namespace

ChainInfo::ChainInfo(const Graph& g) {
  const int n = (int)g.nodes.size();
  fam.resize(n); fused.resize(n); readers.assign(n, 0); last.assign(n, -1); ok.resize(n); convs.resize(n);
  rank.resize(n);
  for (int v = 0, r = 0; v < n; ++v) {
    const Node& nd = g.nodes[v];
    rank[v] = r;
    r += nd.weighted();
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

bool build_chain(const Graph& g, const ChainInfo& f, int a, int b, const std::set<int>& keep, int size, ChainSeg& s) {
  int slice[CHAIN_SIZES];
  double clocks[CHAIN_SIZES];
  std::vector<ChainWork> work;
  if (!cheapest(g, f, a, b, keep, work, clocks, slice) || !build_with_slice(g, f, a, b, keep, slice[size], nullptr, s))
    return false;
  s.cost = clocks[size];
  return true;
}
bool build_chain(const Graph& g, int a, int b, const std::set<int>& keep, ChainSeg& s) {
  return build_chain(g, ChainInfo(g), a, b, keep, 0, s);
}

double layers_clocks(const Graph& g, const ChainInfo& f, int a, int b, const std::set<int>& keep, int size) {
  double t = 0;
  for (int v = a; v <= b; ++v) {
    t += layer_clocks(g, f, v, size);
    if (f.fused[v] != v + 1 || v == b || keep.count(v)) continue;
    ++v;                                               // the ADD in its launch
    t += ADD_READ * 2 * g.nodes[v].out_elems();
  }
  return t;
}

std::vector<ChainSeg> plan_chains(const Graph& g) { return plan_chains(g, ChainInfo(g)).best[0]; }
ChainPlan plan_chains(const Graph& g, const ChainInfo& f) {
  constexpr int S = CHAIN_SIZES;
  const int n = (int)g.nodes.size();
  ChainPlan plan;
  for (auto& l : plan.best) l.resize(n);
  for (auto& l : plan.head) l.resize(n);
  if (g.dtype != DT_BF16) return plan;
  struct Best { double cost = 0, chain = 0; int end = 0, slice = 0; };
  std::vector<Best> at[S], head[S];
  std::vector<ChainWork> work;
  for (auto& l : at) l.resize(n + 1);
  for (auto& l : head) l.resize(n + 1);
  for (int v = n - 1; v >= 1; --v) {
    // by itself, or with the ADD that its launch computes
    const int fa = f.fused[v];
    for (int z = 0; z < S; ++z)
      at[z][v].cost = layer_clocks(g, f, v, z) + (fa == v + 1 ? ADD_READ * 2 * g.nodes[fa].out_elems() + at[z][v + 2].cost
                                                            : at[z][v + 1].cost);
    // the copy of node v - 1's output that the layers need (a halo convolution
    // reads it in channel groups instead); a chain that reads through channel
    // maps saved its launch and 0.08 clocks a byte of the same networks' time
    const Node& m = g.nodes[v - 1];
    const bool copied = m.weighted() && f.fam[v] != FAM_HALO;
    for (int z = 0; z < S; ++z) {
      head[z][v] = at[z][v];
      if (copied) head[z][v].cost += launch_clocks(z) + 0.08 * 2 * m.out_elems();
    }
    int fails = 0;
    for (int b = v; b < n && f.ok[b] && fails < 2; ++b) {
      // two nodes at least, and not between a convolution and the ADD that its
      // launch would fuse
      if (b == v || f.fused[b] == b + 1) continue;
      int slice[S];
      double clocks[S];
      if (!cheapest(g, f, v, b, {}, work, clocks, slice)) { ++fails; continue; }
      fails = 0;
      for (int z = 0; z < S; ++z) {
        const Best c = {clocks[z] + at[z][b + 1].cost, clocks[z], b, slice[z]};
        if (c.cost < at[z][v].cost) at[z][v] = c;
        if (c.cost < head[z][v].cost && f.last[v - 1] <= b) head[z][v] = c;
      }
    }
  }
  std::map<std::pair<int, int>, ChainSeg> built;       // of the node: by end and slice
  auto build = [&](int v, const Best& c, ChainSeg& s) {
    if (!c.end) return;
    const auto k = built.emplace(std::make_pair(c.end, c.slice), ChainSeg());
    ChainSeg& b = k.first->second;
    if (k.second && !build_with_slice(g, f, v, c.end, {}, c.slice, nullptr, b)) b = ChainSeg();
    s = b;
    s.cost = c.chain;
  };
  for (int v = 1; v < n; ++v) {
    built.clear();
    for (int z = 0; z < S; ++z) {
      build(v, at[z][v], plan.best[z][v]);
      if (g.nodes[v - 1].weighted()) build(v, head[z][v].end ? head[z][v] : at[z][v], plan.head[z][v]);
    }
  }
  return plan;
}

}  // namespace mure
