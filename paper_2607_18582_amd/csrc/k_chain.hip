// Image-resident chains: a block takes G images of one mutant slot through a
// run of consecutive bf16 nodes (3x3 and 1x1 convolutions, depthwise 3x3, ADD,
// GAP) with every intermediate activation in LDS.  Per-layer kernels of such
// small layers are bound by the activations' trips through HBM (16 to 64
// channels at 32x32 and below: 2.8 TB/s of a 5.1 TB/s copy rate on ResNet-20);
// a chain reads its first input and writes its last output only, and the
// first mutated node's output is read straight from the prefix cache through
// the mutant's channel map and compact delta rows.
//
// Each node keeps its own family's arithmetic -- the reduction order, the
// MFMA instruction and the rounding points of the per-layer kernels -- so the
// results are theirs bit for bit:
//   conv16: the tiled implicit GEMM's order, k = (tap, channel) in steps of 32
//           on v_mfma_f32_16x16x32_bf16;
//   conv32: the halo convolution's, k = (chunk of 16 channels, tap) in steps of
//           16 on v_mfma_f32_32x32x16_bf16;
//   dw:     taps in (dy, dx) order from 0, then the bias.
// The weights are the MFMA's first operand and the pixels its second (the
// products and their order are the same), so a lane ends with four
// consecutive output channels of one pixel and stores them as one 8-byte LDS
// write.  The weights of a wave's channel tile stay in registers over its
// pixel tiles and come from L2; the blocks of a slot run on one XCD.
//
// Two blocks of eight waves per CU: an operation's waves meet at a barrier, and
// the other block fills the gaps.  What is independent of LDS -- an
// operation's weights and bias -- is fetched before that barrier, and the next
// operation's weights are touched into the cache meanwhile.  What bounds a
// chain is the latency of its operations (about 6,000 clocks each for a
// 1024 x 16 convolution alone on a CU, against 2,600 of LDS reads and 1,300 of
// MFMA) and the vector instructions of the epilogues.
//
// Measured, layer by layer -> chains where chain.cpp finds them faster:
// run_mutants on ResNet-20, 2,500 inputs x 200 mutants, 50.6 -> 41.0 ms (237 ->
// 142 launches); MobileNetV2, 2,500 x 200, 62.7 -> 45.5 ms (705 -> 214); ResNet-20,
// exhaustive, 1,111 x 61, 24.2 -> 14.7 ms, and 10.4 with the stem's own kernel.
#include "dev.hpp"

#include <algorithm>

namespace mure {

namespace {
typedef float v16f __attribute__((ext_vector_type(16)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(1))) const v4u gv4u;
typedef __attribute__((address_space(1))) const v4f gv4f;
typedef __attribute__((address_space(4))) const ChainOp cop;

constexpr int NT = 64 * CHAIN_WAVES;

struct Blk {
  unsigned char* sm;
  int zero;                              // offset of 16 zero bytes; 16 bytes after them nobody reads
  int G, arena, slot, xi0, cnt;          // images xi0 .. xi0 + cnt - 1 (cnt <= G)
  int tid, lane, wave;
};

__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
  return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)v) |
         (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32;
}

__device__ __forceinline__ ChainT T(const __attribute__((address_space(4))) ChainT& t) {
  ChainT r;
  r.off = t.off; r.pitch = t.pitch; r.pxb = t.pxb; r.bd = t.bd; r.sh = t.sh; r.mask = t.mask;
  return r;
}

// padded pixel index of (y, x), its byte offset and the swizzle of its slots
__device__ __forceinline__ int t_px(const ChainT& t, int y, int x) { return (y + t.bd) * t.pitch + x + t.bd; }
__device__ __forceinline__ int t_swz(const ChainT& t, int p) { return ((p >> t.sh) & t.mask) << 4; }

// Clear the border of every image of tensor t (H rows inside it): the rows
// above and below, and the pixel between each row's end and the next row.
__device__ __forceinline__ void zero_border(const Blk& k, const ChainT& t, int H) {
  const v4u z = {0u, 0u, 0u, 0u};
  const int row = t.pitch * t.pxb;
  for (int img = 0; img < k.G; ++img) {
    unsigned char* const im = k.sm + img * k.arena + t.off;
    for (int i = k.tid * 16; i < row + t.pxb; i += NT * 16) {
      *reinterpret_cast<v4u*>(im + i) = z;
      *reinterpret_cast<v4u*>(im + (H + 1) * row + i) = z;
    }
    for (int y = 2 + (k.tid >> 3); y <= H; y += NT / 8)
      for (int i = (k.tid & 7) * 16; i < t.pxb; i += 128) *reinterpret_cast<v4u*>(im + y * row + i) = z;
  }
}

// The operation's first LDS access: the previous operation is complete (what
// needs no LDS comes before it).
__device__ __forceinline__ void begin(const Blk& k, cop* o) {
  __syncthreads();
  if (o->zero) zero_border(k, T(o->out), o->Ho);
}

// Activation in float32: R = 0 none, 1 ReLU or ReLU6 with its upper bound hi
// (infinity for ReLU): med3 is min(max(v, 0), hi), and 0 for a NaN, as act().
template <int R>
__device__ __forceinline__ float act_r(float v, float hi) {
  return R ? __builtin_amdgcn_fmed3f(v, 0.f, hi) : v;
}
__device__ __forceinline__ float act_hi(int relu) { return relu == 2 ? 6.f : __builtin_inff(); }

// A tensor's pixels by the output's linear pixel index p = y W + x of an
// image: the padded index of (st y, st x) is st * (p + y * (pitch - W)), plus
// bd (pitch + 1) where the border counts.  Tiles are aligned runs of 16 or 32
// pixels and the planes' sizes are powers of two.
struct PxMap {
  int extra, bd1;                        // pitch - W, bd (pitch + 1)
  __device__ __forceinline__ PxMap(const ChainT& t, int W) : extra(t.pitch - W), bd1(t.bd * (t.pitch + 1)) {}
  __device__ __forceinline__ int operator()(int p, int y) const { return __umul24(y, extra) + p; }
};

// Epilogue of four consecutive channels of a lane's output pixel.  R: the
// convolution's activation; AR: -1 no ADD, else the ADD's activation.
template <int R, int AR>
struct Epi {
  const ChainT ot, st;
  const int ostride, sstride;            // bytes of a pixel
  PxMap om, sm;
  const int add, same, cpad, Cs, oc2;
  unsigned char* none;
  const float hi, ahi;
  unsigned char* out;                    // pixel's bytes, without the swizzled part
  const unsigned char* skip;
  int osw, ssw;
  __device__ __forceinline__ Epi(const Blk& k, cop* o)
      : ot(T(o->out)), st(AR >= 0 ? T(o->skip) : ChainT()), ostride(o->out.pxb), sstride(AR >= 0 ? o->skip.pxb : 0),
        om(ot, o->Wo), sm(st, o->Wo), add(AR >= 0 ? o->add : 0), same(AR >= 0 ? o->same : 0),
        cpad(AR >= 0 ? o->cpad : 0), Cs(AR >= 0 ? o->Cs : 0), oc2(2 * o->oc), none(k.sm + k.zero + 16),
        hi(act_hi(o->relu)), ahi(AR >= 0 ? act_hi(o->add_relu) : 0.f) {}
  // pixel p = y W + x of the image at im
  __device__ __forceinline__ void pixel(unsigned char* im, int p, int y) {
    const int q = om(p, y) + om.bd1;
    out = im + ot.off + __umul24(q, ostride);
    osw = t_swz(ot, q);
    if constexpr (AR >= 0) {
      if (same) {
        skip = out;
        ssw = osw;
      } else {
        const int r = (add == 2 ? 2 * sm(p, y) : sm(p, y)) + sm.bd1;
        skip = im + st.off + __umul24(r, sstride);
        ssw = t_swz(st, r);
      }
    }
  }
  // ok false: a lane past the last channel, stored where nobody reads
  __device__ __forceinline__ void put4(int ch, const v4f& acc, const v4f& b, bool ok) const {
    uint32_t lo = f2bf2(act_r<R>(acc[0] + b[0], hi), act_r<R>(acc[1] + b[1], hi));
    uint32_t hw = f2bf2(act_r<R>(acc[2] + b[2], hi), act_r<R>(acc[3] + b[3], hi));
    if constexpr (AR >= 0) {
      const int cs = ch - cpad;
      v2u sv = {0u, 0u};
      if (cs >= 0 && cs < Cs) sv = *reinterpret_cast<const v2u*>(skip + ((2 * cs) ^ ssw));
      lo = f2bf2(act_r<AR>(bf2f((bf16_t)lo) + bf2f((bf16_t)sv[0]), ahi),
                 act_r<AR>(bf2f((bf16_t)(lo >> 16)) + bf2f((bf16_t)(sv[0] >> 16)), ahi));
      hw = f2bf2(act_r<AR>(bf2f((bf16_t)hw) + bf2f((bf16_t)sv[1]), ahi),
                 act_r<AR>(bf2f((bf16_t)(hw >> 16)) + bf2f((bf16_t)(sv[1] >> 16)), ahi));
    }
    *reinterpret_cast<v2u*>(ok ? out + ((2 * ch + oc2) ^ osw) : none) = v2u{lo, hw};
  }
};

// Convolution in the tiled implicit GEMM's order: KS k-steps of 32 (k past K
// has zero weights and reads the zero slot), TN channel tiles of 16 per wave,
// K3: 3 x 3 taps (pad 1), else 1 x 1.  The input is not swizzled, so a
// fragment's address is the pixel's plus the step's part.  PAST: some of the
// steps may be empty.
//
// Instances for 1, 2, 3, 5, 9 and 12 steps serve every reduction up to 12; one
// for each number of steps made every chain slower, whatever it runs (the
// kernel 290 -> 390 KB; MobileNetV2, 2,500 x 200: 46.0 -> 49.0 ms with 1 x 1 instances
// only, 54 with the 3 x 3 ones), and so, by 2 %, do the empty steps' conditions:
// chains without any run a kernel without them.
template <int KS, int TN, bool K3, int R, int AR, bool PAST>
__device__ __forceinline__ void conv16(const Blk& k, cop* o, const bf16_t* Wt, const float* bias) {
  constexpr int TP = TN * KS <= 6 ? 2 : 1;               // pixel tiles in flight
  const int l15 = k.lane & 15, g4 = k.lane >> 4;
  const int Cout = o->Cout, K = o->K, n0 = o->n0, lw = o->lw, lp = o->lp;
  const ChainT it = T(o->in);
  // items: a group of TN channel tiles and one of `splits` parts of the pixel
  // tiles; with fewer groups than waves, one item per wave
  const int groups = o->groups, splits = o->splits;
  const int ptiles = (k.G << lp) >> 4;
  const PxMap im(it, 1 << lw);
  const int istride = it.pxb * o->stride;
  // k past K: in the last step, or with PAST from the instance's least number
  // of steps on
  constexpr int LAST = !PAST || KS <= 3 ? KS - 1 : KS == 5 ? 2 : KS == 9 ? 5 : 9;
  auto past = [&](int s) { return s >= LAST && 32 * s + 8 * g4 >= K; };
  int toff[K3 ? KS : 1];
  if constexpr (K3) {
    // vector u of 8 k is channels 8 (u % c8) .. of tap u / c8, c8 = C / 8: 2 or
    // 4 where the steps are full, 1 to 4 otherwise ((u inv) >> 8 is exact for
    // u < 48); pad 1: the border shifts a pixel to its first tap
    const int c8 = PAST ? o->C >> 3 : KS == 5 ? 2 : 4, inv = PAST ? 255 / c8 + 1 : 256 / c8;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int u = 4 * s + g4, t = (u * inv) >> 8, dy = (t * 11) >> 5;
      toff[s] = __umul24(__umul24(dy, it.pitch) + t - 3 * dy, it.pxb) + 16 * (u - t * c8) + it.off;
    }
  } else {
    toff[0] = im.bd1 * it.pxb + it.off + 16 * g4;
  }
  Epi<R, AR> epi(k, o);
  const int sp0 = (k.wave * o->inv) >> 8;                // wave / groups, for fewer groups than waves
  const int cg0 = splits > 1 ? k.wave - sp0 * groups : k.wave;
  const int sp = splits > 1 ? sp0 : 0;
  v8bf w[TN][KS];
  v4f b[TN];
  auto fetch = [&](int cg) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = (cg * TN + j) * 16 + l15;
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        v4u r = {0u, 0u, 0u, 0u};
        if (n < Cout && !past(s)) r = *(gv4u*)(Wt + (n0 + n) * K + 32 * s + 8 * g4);
        w[j][s] = __builtin_bit_cast(v8bf, r);
      }
      const int c = (cg * TN + j) * 16 + 4 * g4;
      b[j] = v4f{0.f, 0.f, 0.f, 0.f};
      if (c < Cout) b[j] = *(gv4f*)(bias + n0 + c);
    }
  };
  fetch(cg0);                                            // under the previous operation's last waves
  begin(k, o);
  if (sp >= splits) return;
  for (int cg = cg0; cg < groups; cg += CHAIN_WAVES) {
    if (cg != cg0) fetch(cg);
    // the next tiles' fragments are read under the current tiles' epilogue
    v8bf f[TP][KS];
    auto read = [&](int t0) {
#pragma unroll
      for (int i = 0; i < TP; ++i) {
        const int p0 = min(t0 + i, ptiles - 1) << 4;
        const int p = (p0 & ((1 << lp) - 1)) + l15;
        const unsigned char* const base = k.sm + (p0 >> lp) * k.arena + __umul24(im(p, p >> lw), istride);
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          const unsigned char* ad = K3 ? base + toff[K3 ? s : 0] : base + toff[0] + 64 * s;
          if (past(s)) ad = k.sm + k.zero;
          f[i][s] = *reinterpret_cast<const v8bf*>(ad);
        }
      }
    };
    int t0 = sp * TP;
    if (t0 < ptiles) read(t0);
    while (t0 < ptiles) {
      __builtin_amdgcn_sched_barrier(0);
      v4f acc[TP][TN];
#pragma unroll
      for (int i = 0; i < TP; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int i = 0; i < TP; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[j][s], f[i][s], acc[i][j], 0, 0, 0);
      const int tc = t0;
      t0 += splits * TP;
      __builtin_amdgcn_sched_barrier(0);
      if (t0 < ptiles) read(t0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < TP; ++i) {
        if (tc + i >= ptiles) continue;
        const int p0 = (tc + i) << 4, p = (p0 & ((1 << lp) - 1)) + l15;
        epi.pixel(k.sm + (p0 >> lp) * k.arena, p, p >> lw);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const int c = (cg * TN + j) * 16 + 4 * g4;
          epi.put4(c, acc[i][j], b[j], c < Cout);
        }
      }
    }
  }
}

// 3x3 stride-1 convolution in the halo kernel's order: per chunk of 16
// channels the nine taps, TP pixel tiles of 32 by 32 channels per
// wave.  A tap's weights for the next chunk are fetched as soon as its MFMAs
// are issued, a whole chunk ahead of their use.  SWZ: swizzled input, whose
// chunks differ by an exclusive or of the address's slot bits.
template <int TP, bool SWZ, int R, int AR>
__device__ __forceinline__ void conv32(const Blk& k, cop* o, const bf16_t* Wt, const float* bias) {
  const int l31 = k.lane & 31, h = k.lane >> 5;
  const int Cout = o->Cout, lw = o->lw, lp = o->lp;
  const ChainT it = T(o->in);
  const PxMap im(it, 1 << lw);
  const int lg = Cout == 64 ? 1 : 0;                     // 32 or 64 channels
  const int ptiles = (k.G << lp) >> 5, strips = (ptiles + TP - 1) / TP;
  const int nch = o->C / 16;
  Epi<R, AR> epi(k, o);
  // a wave's items have one channel tile: the number of waves is even
  const int cg = k.wave & lg;
  const bf16_t* const wl = Wt + (h * Cout + cg * 32 + l31) * 8;
  v8bf w[9];
  v4f b[4];
#pragma unroll
  for (int t = 0; t < 9; ++t) w[t] = __builtin_bit_cast(v8bf, *(gv4u*)(wl + t * 2 * Cout * 8));
#pragma unroll
  for (int q = 0; q < 4; ++q) b[q] = *(gv4f*)(bias + cg * 32 + 8 * q + 4 * h);
  begin(k, o);                                           // the weights under the previous operation's last waves
  for (int item = k.wave; item < strips << lg; item += CHAIN_WAVES) {
    const int t0 = (item >> lg) * TP;
    int ad[TP][9];
    v16f acc[TP];
#pragma unroll
    for (int i = 0; i < TP; ++i) {
      const int p0 = min(t0 + i, ptiles - 1) << 5, p = (p0 & ((1 << lp) - 1)) + l31;
      const int px = im(p, p >> lw), at = (p0 >> lp) * k.arena + it.off + 16 * h;
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        const int q = px + (t / 3) * it.pitch + t % 3;
        ad[i][t] = (at + __umul24(q, it.pxb)) ^ (SWZ ? t_swz(it, q) : 0);
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
    }
    for (int c = 0; c < nch; ++c) {
      const bf16_t* const wn = wl + (c + 1 < nch ? c + 1 : 0) * 18 * Cout * 8;   // (then the next item's first)
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        v8bf f[TP];
#pragma unroll
        for (int i = 0; i < TP; ++i)
          f[i] = *reinterpret_cast<const v8bf*>(k.sm + (SWZ ? ad[i][t] ^ (32 * c) : ad[i][t] + 32 * c));
#pragma unroll
        for (int i = 0; i < TP; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[t], f[i], acc[i], 0, 0, 0);
        w[t] = __builtin_bit_cast(v8bf, *(gv4u*)(wn + t * 2 * Cout * 8));
      }
    }
#pragma unroll
    for (int i = 0; i < TP; ++i) {
      if (t0 + i >= ptiles) continue;
      const int p0 = (t0 + i) << 5, p = (p0 & ((1 << lp) - 1)) + l31;
      epi.pixel(k.sm + (p0 >> lp) * k.arena, p, p >> lw);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const v4f a4 = {acc[i][4 * q], acc[i][4 * q + 1], acc[i][4 * q + 2], acc[i][4 * q + 3]};
        epi.put4(cg * 32 + 8 * q + 4 * h, a4, b[q], true);
      }
    }
  }
}

// Depthwise 3x3, pad 1: a thread computes four output rows of one column of 4
// channels, the three input rows of the current output row widened in
// registers (each vector is widened once, for up to three output rows).
template <int S, int R>
__device__ __forceinline__ void dw(const Blk& k, cop* o, const bf16_t* Wt, const float* bias) {
  constexpr int RO = 4;                                // output rows per thread
  const int lw = o->lw, lp = o->lp, n0 = o->n0, oc2 = 2 * o->oc;
  const int parts = o->Ho / RO;
  const int total = (k.G << lw) * parts * (o->C / 4);
  const ChainT it = T(o->in), ot = T(o->out);
  DivU32 dcv;
  dcv.d = o->dcv.d; dcv.mul = o->dcv.mul; dcv.sh1 = o->dcv.sh1; dcv.sh2 = o->dcv.sh2;
  const float hi = act_hi(o->relu);
  v2u wr[9];
  v4f b;
  auto fetch = [&](int cv) {
    // four filters of nine taps: 72 bytes from an 8-byte aligned address
    const v2u __attribute__((address_space(1)))* const ws =
        (const v2u __attribute__((address_space(1)))*)(Wt + (int64_t)(n0 + cv * 4) * 9);
#pragma unroll
    for (int q = 0; q < 9; ++q) wr[q] = ws[q];
    b = *(gv4f*)(bias + n0 + cv * 4);
  };
  {
    int rest, cv;
    divmodu(dcv, (uint32_t)k.tid, rest, cv);
    fetch(cv);                                           // under the previous operation's last waves
  }
  begin(k, o);
  for (int i = k.tid; i < total; i += NT) {
    int rest, cv;
    divmodu(dcv, (uint32_t)i, rest, cv);
    if (i != k.tid) fetch(cv);
    const int x = rest & ((1 << lw) - 1);
    rest >>= lw;
    const int part = rest & (parts - 1), img = rest >> (lp - lw - 2);
    const unsigned char* const in = k.sm + img * k.arena + it.off + cv * 8;
    float wt[36];
#pragma unroll
    for (int q = 0; q < 36; ++q) {
      const uint32_t u = wr[q >> 2][(q >> 1) & 1];
      wt[q] = __uint_as_float(q & 1 ? u & 0xffff0000u : u << 16);
    }
    const int y0 = part * RO;
    float row[3][3][4];
    auto load = [&](int iy, float (&v)[3][4]) {        // padded row iy, columns x S .. x S + 2
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) {
        const v2u r = *reinterpret_cast<const v2u*>(in + __umul24(__umul24(iy, it.pitch) + x * S + dx, it.pxb));
#pragma unroll
        for (int j = 0; j < 4; ++j)
          v[dx][j] = __uint_as_float(j & 1 ? r[j >> 1] & 0xffff0000u : r[j >> 1] << 16);
      }
    };
    load(y0 * S, row[0]);
    if (S == 1) load(y0 * S + 1, row[1]);
#pragma unroll
    for (int r = 0; r < RO; ++r) {
      // window rows: stride 1 rotates three, stride 2 shares one
      constexpr int T0[4] = {0, 1, 2, 0};
      float (&r0)[3][4] = row[S == 1 ? T0[r] : r % 2 ? 2 : 0];
      float (&r1)[3][4] = row[S == 1 ? (T0[r] + 1) % 3 : 1];
      float (&r2)[3][4] = row[S == 1 ? (T0[r] + 2) % 3 : r % 2 ? 0 : 2];
      const int iy = (y0 + r) * S;
      if (S == 2) load(iy + 1, r1);
      load(iy + 2, r2);
      float acc[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[j] = 0.f;
#pragma unroll
      for (int dx = 0; dx < 3; ++dx)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] = fmaf(r0[dx][j], wt[j * 9 + dx], acc[j]);
#pragma unroll
      for (int dx = 0; dx < 3; ++dx)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] = fmaf(r1[dx][j], wt[j * 9 + 3 + dx], acc[j]);
#pragma unroll
      for (int dx = 0; dx < 3; ++dx)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] = fmaf(r2[dx][j], wt[j * 9 + 6 + dx], acc[j]);
      v2u ov;
#pragma unroll
      for (int j = 0; j < 4; j += 2)
        ov[j >> 1] = f2bf2(act_r<R>(acc[j] + b[j], hi), act_r<R>(acc[j + 1] + b[j + 1], hi));
      const int p = t_px(ot, y0 + r, x);
      *reinterpret_cast<v2u*>(k.sm + img * k.arena + ot.off + __umul24(p, ot.pxb) +
                              ((oc2 + cv * 8) ^ t_swz(ot, p))) = ov;
    }
  }
}

template <int R, int AR, bool PAST>
__device__ __forceinline__ void conv(const Blk& k, cop* o, const bf16_t* Wt, const float* bias) {
  switch (o->code) {
    // two pixel tiles per wave where that leaves every wave some
    case 0:
      if ((k.G << o->lp) * o->Cout >= 2048 * CHAIN_WAVES) conv32<2, true, R, AR>(k, o, Wt, bias);
      else conv32<1, true, R, AR>(k, o, Wt, bias);
      break;
    case 1: conv32<1, false, R, AR>(k, o, Wt, bias); break;
#define MURE_C16(KS, TN, K3) case (K3 ? 1000 : 0) + KS * 10 + TN: conv16<KS, TN, K3, R, AR, PAST>(k, o, Wt, bias); break;
    MURE_C16(1, 1, false) MURE_C16(1, 2, false) MURE_C16(1, 3, false)
    MURE_C16(2, 1, false) MURE_C16(2, 2, false) MURE_C16(2, 3, false)
    MURE_C16(3, 1, false) MURE_C16(3, 2, false)
    MURE_C16(5, 1, false) MURE_C16(5, 2, false)
    MURE_C16(9, 1, false) MURE_C16(12, 1, false)
    MURE_C16(5, 1, true) MURE_C16(5, 2, true) MURE_C16(9, 1, true)
#undef MURE_C16
    default: break;
  }
}

// Tensor rows between global memory ([pixel][C]) and LDS.  Buffer 0 may be
// read through the slot's channel map: its rows come from the prefix cache,
// and then the channels that the map changes are put in, one (pixel, channel)
// per thread, all of them in flight together; `list` (LDS) collects those
// channels.
__device__ __forceinline__ void load_rows(const Blk& k, const ChainOp& o, const ChainArgs& a, const ChainBuf& bf,
                                          int32_t* list) {
  const int cvs = o.C / 8;
  const int total = (k.cnt << o.lp) * cvs;
  const bool virt = o.buf == 0 && a.vin.chmap != nullptr;
  if (virt && k.wave == 0) {
    // (channel, source) of the changed channels, in channel order
    const int32_t* const m = a.vin.chmap + (int64_t)k.slot * o.C;
    int n = 0;
    for (int c0 = 0; c0 < o.C; c0 += 64) {
      const int c = c0 + k.lane, src = c < o.C ? m[c] : c;
      const unsigned long long hit = __ballot(src != c);
      const int at = n + __popcll(hit & ((1ull << k.lane) - 1));
      if (src != c && at < CHAIN_LIST) {
        list[1 + 2 * at] = c;
        list[2 + 2 * at] = src;
      }
      n += __popcll(hit);
    }
    if (k.lane == 0) list[0] = n;
  }
  constexpr int U = 4;                                 // vectors in flight per thread
  const int64_t row0 = row_at(bf.mode, k.slot, k.xi0, a.nx, a.x0);
  const bf16_t* const base = reinterpret_cast<const bf16_t*>(bf.p) + row0 * bf.row_elems;
  for (int i0 = k.tid; i0 < total; i0 += U * NT) {
    v4u v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      // an image's rows are whole: vector i of the group is 16 bytes at 16 i
      const int i = min(i0 + u * NT, total - 1);
      v[u] = *(gv4u*)(base + (int64_t)i * 8);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * NT;
      if (i >= total) continue;
      int q, cv;
      divmodu(o.dcv, (uint32_t)i, q, cv);
      const int img = q >> o.lp, pix = q & ((1 << o.lp) - 1);
      const int p = t_px(o.out, pix >> o.lw, pix & ((1 << o.lw) - 1));
      *reinterpret_cast<v4u*>(k.sm + img * k.arena + o.out.off + __umul24(p, o.out.pxb) +
                              ((cv * 16) ^ t_swz(o.out, p))) = v[u];
    }
  }
  if (!virt) return;
  __syncthreads();
  const int listed = __builtin_amdgcn_readfirstlane(list[0]);
  const int n = listed <= CHAIN_LIST ? listed : o.C;   // more than the list holds: every channel
  const int32_t* const m = a.vin.chmap + (int64_t)k.slot * o.C;
  const bf16_t* const delta =
      reinterpret_cast<const bf16_t*>(a.vin.delta) + (((int64_t)k.slot * a.nx + k.xi0) << o.lp) * a.vin.T;
  for (int img = 0; img < k.cnt; ++img) {
    const int q0 = img << o.lp;
    for (int i0 = k.tid; i0 < n << o.lp; i0 += U * NT) {
      bf16_t v[U];
      int dst[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = min(i0 + u * NT, (n << o.lp) - 1), e = i >> o.lp, pix = i & ((1 << o.lp) - 1);
        int c = e, src;
        if (listed <= CHAIN_LIST) {
          c = list[1 + 2 * e];
          src = list[2 + 2 * e];
        } else {
          src = m[e];
        }
        const bf16_t* const from =
            src < -1 ? delta + (int64_t)(q0 + pix) * a.vin.T + (-2 - src) : base + (int64_t)(q0 + pix) * o.C + max(src, 0);
        v[u] = *(const bf16_t __attribute__((address_space(1)))*)from;
        if (src == -1) v[u] = 0;
        const int p = t_px(o.out, pix >> o.lw, pix & ((1 << o.lw) - 1));
        dst[u] = img * k.arena + o.out.off + __umul24(p, o.out.pxb) + ((2 * c) ^ t_swz(o.out, p));
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (i0 + u * NT < n << o.lp) *reinterpret_cast<bf16_t*>(k.sm + dst[u]) = v[u];
    }
  }
}

__device__ __forceinline__ void store_rows(const Blk& k, const ChainOp& o, const ChainArgs& a, const ChainBuf& bf) {
  const int total = (k.cnt << o.lp) * (o.C / 8);
  for (int i = k.tid; i < total; i += NT) {
    int q, cv;
    divmodu(o.dcv, (uint32_t)i, q, cv);
    const int img = q >> o.lp, pix = q & ((1 << o.lp) - 1);
    const int p = t_px(o.in, pix >> o.lw, pix & ((1 << o.lw) - 1));
    const v4u v = *reinterpret_cast<const v4u*>(k.sm + img * k.arena + o.in.off + p * o.in.pxb +
                                                ((cv * 16) ^ t_swz(o.in, p)));
    const int64_t row = row_at(bf.mode, k.slot, k.xi0 + img, a.nx, a.x0);
    *reinterpret_cast<v4u*>(reinterpret_cast<bf16_t*>(bf.p) + row * bf.row_elems + (int64_t)pix * o.C + cv * 8) = v;
  }
}

__device__ __forceinline__ void add_rows(const Blk& k, const ChainOp& o) {
  const int total = (k.G << o.lp) * (o.C / 8);
  for (int i = k.tid; i < total; i += NT) {
    int q, cv;
    divmodu(o.dcv, (uint32_t)i, q, cv);
    const int img = q >> o.lp, pix = q & ((1 << o.lp) - 1), y = pix >> o.lw, x = pix & ((1 << o.lw) - 1);
    unsigned char* const im = k.sm + img * k.arena;
    const int pi = t_px(o.in, y, x);
    const v4u v = *reinterpret_cast<const v4u*>(im + o.in.off + pi * o.in.pxb + ((cv * 16) ^ t_swz(o.in, pi)));
    const int ps = o.add == 2 ? t_px(o.skip, 2 * y, 2 * x) : t_px(o.skip, y, x), cs = cv * 8 - o.cpad;
    v4u sv = {0u, 0u, 0u, 0u};
    if (cs >= 0 && cs < o.Cs)
      sv = *reinterpret_cast<const v4u*>(im + o.skip.off + ps * o.skip.pxb + ((2 * cs) ^ t_swz(o.skip, ps)));
    v4u r;
#pragma unroll
    for (int w = 0; w < 4; ++w)
      r[w] = f2bf2(act(bf2f((bf16_t)v[w]) + bf2f((bf16_t)sv[w]), o.add_relu),
                   act(bf2f((bf16_t)(v[w] >> 16)) + bf2f((bf16_t)(sv[w] >> 16)), o.add_relu));
    const int p = t_px(o.out, y, x);
    *reinterpret_cast<v4u*>(im + o.out.off + p * o.out.pxb + ((cv * 16) ^ t_swz(o.out, p))) = r;
  }
}

// GAP: the pixels summed in order in float32, then scaled, as gap_kernel does.
// One (image, 64 channels) per wave at a time: image after image in the whole
// block leaves all but a few waves idle where the layer is narrow (14k of a
// chain's clocks for 8 images of 64 channels; a pass of resnet20 47.4 -> 46.3 ms, of
// mobilenetv2 48.0 -> 47.6).
__device__ __forceinline__ void gap_rows(const Blk& k, const ChainOp& o, const ChainArgs& a, const ChainBuf& bf) {
  const int P = 1 << o.lp, cw = (o.C + 63) >> 6;       // waves per image
  int img = 0, c0 = k.wave;
  for (;; c0 += CHAIN_WAVES) {
    while (c0 >= cw) {
      c0 -= cw;
      if (++img >= k.cnt) return;
    }
    const int c = c0 * 64 + k.lane;
    if (c >= o.C) continue;
    const unsigned char* const in = k.sm + img * k.arena + o.in.off;
    float s = 0.f;
#pragma unroll 8
    for (int q = 0; q < P; ++q) {
      const int p = t_px(o.in, q >> o.lw, q & ((1 << o.lw) - 1));
      s += bf2f(*reinterpret_cast<const bf16_t*>(in + p * o.in.pxb + ((2 * c) ^ t_swz(o.in, p))));
    }
    const int64_t row = row_at(bf.mode, k.slot, k.xi0 + img, a.nx, a.x0);
    reinterpret_cast<bf16_t*>(bf.p)[row * bf.row_elems + c] = f2bf(s * (1.0f / (float)P));
  }
}
}  // namespace

__device__ __forceinline__ ChainOp fetch_op(cop* o) {
  ChainOp c;
  __builtin_memcpy(&c, (const void __attribute__((address_space(4)))*)o, sizeof(c));
  return c;
}

template <bool PAST>
__global__ __launch_bounds__(NT, 4) void chain_kernel(ChainArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char chain_sm[];
  // the blocks running together on an XCD share their slot's weights in its L2
  const int idx = chain_block((int)blockIdx.x, a.first, a.turns);
  if (idx >= a.end) return;                             // padding of the order (whole block)
  Blk k;
  k.sm = chain_sm;
  k.G = a.G;
  k.arena = a.arena;
  k.zero = a.G * a.arena;
  k.slot = idx / a.per_slot;
  k.xi0 = (idx - k.slot * a.per_slot) * a.G;
  k.cnt = min(a.G, a.nx - k.xi0);
  k.tid = (int)threadIdx.x;
  k.lane = k.tid & 63;
  k.wave = __builtin_amdgcn_readfirstlane(k.tid >> 6);
  if (k.tid == 0) *reinterpret_cast<v4u*>(k.sm + k.zero) = v4u{0u, 0u, 0u, 0u};
  cop* const ops = (cop*)a.ops;
  // every operation's weight and bias pointers, looked up once
  uint64_t* const ptrs = reinterpret_cast<uint64_t*>(k.sm + k.zero + 32);
  if (k.tid < 2 * a.nops) {
    const ChainOp* const op = a.ops + (k.tid >> 1);
    ptrs[k.tid] = 0;
    if (op->wbytes > 0)
      ptrs[k.tid] = reinterpret_cast<const uint64_t*>(a.tabs)[a.tab0 + (2 * op->w + (k.tid & 1)) * a.tab_stride + k.slot];
  }
  __syncthreads();
  for (int i = 0; i < a.nops; ++i) {
    cop* const o = ops + i;
    const int kind = o->kind;
    asm volatile("" : "+v"(k.lane));                   // lane arithmetic stays inside its operation: hoisted, it spills
    asm volatile("" : "+v"(k.tid));
    const bf16_t* const Wt = reinterpret_cast<const bf16_t*>(uniform64(ptrs[2 * i]));
    const float* const bias = reinterpret_cast<const float*>(uniform64(ptrs[2 * i + 1]));
    // touch the next operation's weights, a 128-byte line per thread
    uint32_t touch = 0;
    if (i + 1 < a.nops) {
      const int nb = ops[i + 1].wbytes;
      if (k.tid * 128 < nb)
        touch = *(const uint32_t __attribute__((address_space(1)))*)(uniform64(ptrs[2 * i + 2]) + ops[i + 1].woff +
                                                                      k.tid * 128);
    }
    if (kind == CH_CONV) {
      // the epilogue's forms: activation or none, or a plain convolution with
      // its ADD
      if (o->add) {
        if (o->add_relu) conv<0, 1, PAST>(k, o, Wt, bias);
        else conv<0, 0, PAST>(k, o, Wt, bias);
      } else if (o->relu) {
        conv<1, -1, PAST>(k, o, Wt, bias);
      } else {
        conv<0, -1, PAST>(k, o, Wt, bias);
      }
    } else if (kind == CH_DW) {
      if (o->stride == 1) {
        if (o->relu) dw<1, 1>(k, o, Wt, bias);
        else dw<1, 0>(k, o, Wt, bias);
      } else {
        if (o->relu) dw<2, 1>(k, o, Wt, bias);
        else dw<2, 0>(k, o, Wt, bias);
      }
    } else {
      begin(k, o);
      const ChainOp c = fetch_op(o);
      if (kind == CH_LOAD) load_rows(k, c, a, a.buf[c.buf], reinterpret_cast<int32_t*>(ptrs + 2 * CHAIN_OPS));
      else if (kind == CH_STORE) store_rows(k, c, a, a.buf[c.buf]);
      else if (kind == CH_ADD) add_rows(k, c);
      else gap_rows(k, c, a, a.buf[c.buf]);
    }
    asm volatile("" ::"v"(touch));                    // the touch's result is used: it has been waited for
  }
}

hipError_t launch_chain(const ChainArgs& a0, hipStream_t s) {
  if (a0.nslots <= 0 || a0.nx <= 0 || a0.nops <= 0) return hipSuccess;
  if (a0.G < 1 || a0.arena <= 0 || a0.G * a0.arena + CHAIN_EXTRA > CHAIN_LDS || a0.nops > CHAIN_OPS) return hipErrorInvalidValue;
  ChainArgs a = a0;
  a.per_slot = (a.nx + a.G - 1) / a.G;
  const int64_t blocks = (int64_t)a.per_slot * a.nslots;
  if (blocks >= (1 << 30)) return hipErrorInvalidValue;
  // a grid holds fewer than 2^32 threads: the blocks of large runs over several
  // launches
  for (int64_t b0 = 0; b0 < blocks; b0 += CHAIN_GRID) {
    a.first = (int)b0;
    a.end = (int)std::min<int64_t>(b0 + CHAIN_GRID, blocks);
    a.turns = (a.end - a.first + 7) / 8;
    const dim3 grid((unsigned)(a.turns * 8));
    const size_t lds = (size_t)(a.G * a.arena + CHAIN_EXTRA);
    if (a.past) hipLaunchKernelGGL(chain_kernel<true>, grid, dim3(NT), lds, s, a);
    else hipLaunchKernelGGL(chain_kernel<false>, grid, dim3(NT), lds, s, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace mure
