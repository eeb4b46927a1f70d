// The general CONV2D kernel (any shape), and the bf16 stems' (C_in = 3) own:
// an implicit GEMM on MFMA with a scalar im2col gather.
//
// GEMM view of one node over a chunk: rows m = (slot, input, output pixel),
// columns n = output channel, reduction k = (dy, dx, c_in) in the weight
// layout [C_out][kh][kw][C_in] (c_in fastest).  The reduction is accumulated
// in float32 by v_mfma_f32_16x16x4_f32 (fp32 models, 4 k per step) or
// v_mfma_f32_16x16x32_bf16 (bf16 models, 32 k per step) in increasing k,
// zero-padded to a whole step -- every kernel that computes a node uses the
// same steps, so a node's value never depends on which kernel or batch
// produced it.  Epilogue in float32: + bias, ReLU, 2x2 max-pool, then the
// node-output rounding (bf16 round-to-nearest-even, or float32).
//
// With pooling, the rows of one input are ordered pool-window-major
// (window q = py*Wp + px, then its 4 pixels), so the 4 accumulators a lane
// holds for one output column are one pooling window.
#include "dev.hpp"
#include "plan.hpp"

#include <algorithm>

namespace mure {

template <typename T> struct Mfma;
template <> struct Mfma<float> { static constexpr int BK = 16, PAD = 1; };
template <> struct Mfma<bf16_t> { static constexpr int BK = 32, PAD = 8; };

template <typename T, int BM, int BN>
__global__ __launch_bounds__(256) void conv_mfma_kernel(ConvArgs a) {
  static_assert(BM == 64 && BN == 64, "tile");
  constexpr int BK = Mfma<T>::BK;
  constexpr int LDA = BK + Mfma<T>::PAD;
  constexpr int EPT = BK / 4;
  __shared__ __attribute__((aligned(16))) T As[BM * LDA];
  __shared__ __attribute__((aligned(16))) T Bs[BN * LDA];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave & 1, wn = wave >> 1;
  const int slot = a.slot0 + (int)blockIdx.y;
  const int64_t Mslot = (int64_t)a.nx * a.P;
  const int64_t m_tile0 = (int64_t)blockIdx.x * BM;
  const int n_tile0 = (int)blockIdx.z * BN;
  const T* __restrict__ Wt = reinterpret_cast<const T*>(a.wtab[slot]);
  const int ncol = a.cols ? a.ncols : a.Cout;

  // the A row this thread gathers (fixed for the block)
  const int m_local = tid & (BM - 1);
  const int kq = tid >> 6;
  const int64_t m = m_tile0 + m_local;
  const bool mvalid = m < Mslot;
  int xi = 0, p = 0;
  if (mvalid) { xi = (int)(m / a.P); p = (int)(m % a.P); }
  int oy, ox;
  if (a.pool) {
    const int q = p >> 2, sub = p & 3;
    oy = 2 * (q / a.Wp) + (sub >> 1);
    ox = 2 * (q % a.Wp) + (sub & 1);
  } else {
    oy = p / a.Wc;
    ox = p % a.Wc;
  }
  const int iy0 = oy * a.stride - a.pad, ix0 = ox * a.stride - a.pad;
  const int64_t r = (int64_t)slot * a.nx + xi;
  const T* __restrict__ inrow =
      reinterpret_cast<const T*>(a.in.p) + row_index(a.in.mode, r, a.nx, a.x0) * a.in.row_elems;
  // the B row (output channel) this thread loads
  const int n_ld = n_tile0 + (tid & 63);
  const bool nvalid = n_ld < ncol;
  const T* __restrict__ wrow = Wt;
  if (nvalid) {
    if (a.cols) {   // a gathered delta column: its own mutant's weight row
      const DeltaCol cd = a.cols[n_ld];
      wrow = reinterpret_cast<const T*>(a.wtab[a.slot0 + cd.slot - a.col_slot0]) + (int64_t)cd.c * a.K;
    } else {
      wrow = Wt + (int64_t)n_ld * a.K;
    }
  }

  v4f acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};

  for (int kc = 0; kc < a.K; kc += BK) {
    {  // A: im2col gather of EPT consecutive k for row m
      int k = kc + kq * EPT;
      int ci = k % a.C, t2 = k / a.C;
      int dx = t2 % a.kw, dy = t2 / a.kw;
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        T v = T(0);
        if (mvalid && k < a.K) {
          const int iy = iy0 + dy, ix = ix0 + dx;
          if (iy >= 0 && iy < a.H && ix >= 0 && ix < a.W) v = inrow[((int64_t)iy * a.W + ix) * a.C + ci];
        }
        As[m_local * LDA + kq * EPT + e] = v;
        ++k;
        if (++ci == a.C) { ci = 0; if (++dx == a.kw) { dx = 0; ++dy; } }
      }
    }
    {  // B: EPT consecutive k of output channel n_ld
      const int k0 = kc + kq * EPT;
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const int k = k0 + e;
        Bs[(tid & 63) * LDA + kq * EPT + e] = (nvalid && k < a.K) ? wrow[k] : T(0);
      }
    }
    __syncthreads();
    if constexpr (sizeof(T) == 4) {
#pragma unroll
      for (int ks = 0; ks < BK / 4; ++ks) {
        float av[2], bv[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          av[t] = As[(wm * 32 + t * 16 + (lane & 15)) * LDA + ks * 4 + (lane >> 4)];
          bv[t] = Bs[(wn * 32 + t * 16 + (lane & 15)) * LDA + ks * 4 + (lane >> 4)];
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i], bv[j], acc[i][j], 0, 0, 0);
      }
    } else {
      v8bf av[2], bv[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        av[t] = *reinterpret_cast<const v8bf*>(&As[(wm * 32 + t * 16 + (lane & 15)) * LDA + (lane >> 4) * 8]);
        bv[t] = *reinterpret_cast<const v8bf*>(&Bs[(wn * 32 + t * 16 + (lane & 15)) * LDA + (lane >> 4) * 8]);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[i], bv[j], acc[i][j], 0, 0, 0);
    }
    __syncthreads();
  }

  // epilogue: lane holds rows mb..mb+3 of column n
  const float* __restrict__ bias = a.btab[slot];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int nc = n_tile0 + wn * 32 + j * 16 + (lane & 15);
      const int64_t mb = m_tile0 + wm * 32 + i * 16 + (lane >> 4) * 4;
      if (nc >= ncol || mb >= Mslot) continue;
      // output slot, channel and channel stride of this column
      int os = slot, n = nc, ostride = a.Cout;
      float bv;
      if (a.cols) {
        const DeltaCol cd = a.cols[nc];
        os = a.slot0 + cd.slot - a.col_slot0;
        bv = a.btab[os][cd.c];
        n = a.delta_T > 0 ? cd.t : cd.c;
        if (a.delta_T > 0) ostride = a.delta_T;
      } else {
        bv = bias[nc];
      }
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] = acc[i][j][e] + bv;
        v[e] = act(v[e], a.relu);
      }
      if (a.pool) {
        const float mx = fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3]));
        const int xo = (int)(mb / a.P);
        const int q = (int)(mb % a.P) >> 2;
        const int64_t ro = row_index(a.out_mode, (int64_t)os * a.nx + xo, a.nx, a.x0);
        store_out<T>(a.out, a.out_f32, ro * a.out_row + (int64_t)q * ostride + n, mx);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int64_t mm = mb + e;
          if (mm >= Mslot) break;
          const int xo = (int)(mm / a.P);
          const int pp = (int)(mm % a.P);
          const int64_t ro = row_index(a.out_mode, (int64_t)os * a.nx + xo, a.nx, a.x0);
          store_out<T>(a.out, a.out_f32, ro * a.out_row + (int64_t)pp * ostride + n, v[e]);
        }
      }
    }
  }
}

// bf16 convolutions whose whole reduction is one MFMA step (kh kw C_in <= 32:
// the 3x3x3 stems), without pooling: the same product as conv_mfma_kernel's,
// with the gather from LDS.  A block stages the input rows of a band of output
// rows of one image once (16-byte loads, zeros around the image) and its four
// waves take tiles of 16 output pixels; a lane gathers its pixel's 8 k as
// eight 2-byte LDS reads at precomputed offsets and uses the fragment for every
// 16-channel tile.  The weights stay in registers.  As the first operand they
// leave a lane four consecutive channels of one pixel, stored as 8 bytes;
// gathered columns take the pixels first and store as conv_mfma_kernel does.
//
// The scalar gather from global memory, with its index arithmetic per element,
// had bound the stems: ResNet-20's over 67,771 images 4.16 -> 0.68 ms (3.3 TB/s
// of input and output), the 43 gathered columns of the wide ResNet's 1.11 -> 0.74.
constexpr int THIN_LEAD = 8;                             // elements before a staged row's data (its left padding)

template <int TN, bool COLS>
__global__ __launch_bounds__(256) void conv_thin_kernel(ConvArgs a, int band_rows, int bands, int rs, int nrows) {
  extern __shared__ __attribute__((aligned(16))) unsigned char thin_sm[];
  bf16_t* const rows = reinterpret_cast<bf16_t*>(thin_sm);   // [nrows][rs]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l15 = lane & 15, g4 = lane >> 4;
  const int xi = (int)blockIdx.x / bands, band = (int)blockIdx.x - xi * bands;
  const int slot = a.slot0 + (int)blockIdx.y;
  const int y0 = band * band_rows, ny = min(band_rows, a.Hc - y0);
  const int iy0 = y0 * a.stride - a.pad;
  const bf16_t* const in = reinterpret_cast<const bf16_t*>(a.in.p) +
                           row_at(a.in.mode, slot, xi, a.nx, a.x0) * a.in.row_elems;
  // stage: the padding of every row, then the rows' data
  const int rowv = a.W * a.C;                            // a multiple of 8, and so is rs
  for (int i = tid; i < nrows * (rs / 8); i += 256) {
    const int r = i / (rs / 8), v = i - r * (rs / 8), iy = iy0 + r;
    const int e = v * 8 - THIN_LEAD;
    v4u x = {0u, 0u, 0u, 0u};
    if (e >= 0 && e < rowv && (unsigned)iy < (unsigned)a.H)
      x = *reinterpret_cast<const v4u*>(in + (int64_t)iy * rowv + e);
    *reinterpret_cast<v4u*>(rows + r * rs + v * 8) = x;
  }
  // this lane's k: offsets of k = 8 g4 + j from the pixel's first tap
  int koff[8];
  v4u kmask = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int k = 8 * g4 + j, dy = k < a.K ? k / (a.kw * a.C) : 0;
    koff[j] = k < a.K ? dy * rs + k - dy * a.kw * a.C : 0;
    if (k < a.K) kmask[j >> 1] |= j & 1 ? 0xffff0000u : 0xffffu;
  }
  const int ncol = COLS ? a.ncols : a.Cout;
  const int n_tile0 = (int)blockIdx.z * 16 * TN;
  v8bf w[TN];
  v4f b[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int n = n_tile0 + j * 16 + l15;
    uint32_t r[4] = {0u, 0u, 0u, 0u};
    if (n < ncol) {
      const bf16_t* wr;
      if constexpr (COLS) {
        const DeltaCol cd = a.cols[n];
        wr = reinterpret_cast<const bf16_t*>(a.wtab[a.slot0 + cd.slot - a.col_slot0]) + (int64_t)cd.c * a.K;
      } else {
        wr = reinterpret_cast<const bf16_t*>(a.wtab[slot]) + (int64_t)n * a.K;
      }
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (8 * g4 + e < a.K) r[e >> 1] |= (uint32_t)wr[8 * g4 + e] << (16 * (e & 1));
    }
    w[j] = __builtin_bit_cast(v8bf, v4u{r[0], r[1], r[2], r[3]});
    const int c = n_tile0 + j * 16 + 4 * g4;
#pragma unroll
    for (int e = 0; e < 4; ++e) b[j][e] = !COLS && c + e < a.Cout ? a.btab[slot][c + e] : 0.f;
  }
  __syncthreads();
  const int npx = ny * a.Wc;
  for (int t = wave; t * 16 < npx; t += 4) {
    int oy, ox;
    divmodu(a.dWc, (uint32_t)min(t * 16 + l15, npx - 1), oy, ox);
    const bf16_t* const px = rows + oy * a.stride * rs + THIN_LEAD + (ox * a.stride - a.pad) * a.C;
    v4u f;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      f[j] = ((uint32_t)px[koff[2 * j]] | (uint32_t)px[koff[2 * j + 1]] << 16) & kmask[j];
    const v8bf fb = __builtin_bit_cast(v8bf, f);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const v4f z = {0.f, 0.f, 0.f, 0.f};
      if constexpr (COLS) {
        // lane: pixels 4 g4 + e of column l15
        const v4f acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb, w[j], z, 0, 0, 0);
        const int nc = n_tile0 + j * 16 + l15;
        if (nc >= ncol) continue;
        const DeltaCol cd = a.cols[nc];
        const int os = a.slot0 + cd.slot - a.col_slot0;
        const float bv = a.btab[os][cd.c];
        const int ostride = a.delta_T > 0 ? a.delta_T : a.Cout, n = a.delta_T > 0 ? cd.t : cd.c;
        bf16_t* const o = reinterpret_cast<bf16_t*>(a.out) + row_at(a.out_mode, os, xi, a.nx, a.x0) * a.out_row;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int p = t * 16 + 4 * g4 + e;
          if (p < npx) o[((int64_t)y0 * a.Wc + p) * ostride + n] = f2bf(act(acc[e] + bv, a.relu));
        }
      } else {
        const v4f acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[j], fb, z, 0, 0, 0);
        const int c = n_tile0 + j * 16 + 4 * g4, p = t * 16 + l15;
        if (c >= a.Cout || p >= npx) continue;
        bf16_t* const o = reinterpret_cast<bf16_t*>(a.out) + row_at(a.out_mode, slot, xi, a.nx, a.x0) * a.out_row +
                          ((int64_t)y0 * a.Wc + p) * a.Cout + c;
        const uint32_t lo = f2bf2(act(acc[0] + b[j][0], a.relu), act(acc[1] + b[j][1], a.relu));
        const uint32_t hi = f2bf2(act(acc[2] + b[j][2], a.relu), act(acc[3] + b[j][3], a.relu));
        *reinterpret_cast<uint2*>(o) = uint2{lo, hi};
      }
    }
  }
}

// Whether conv_thin_kernel computes a launch: one k step, rows of whole
// 16-byte vectors (as the tensors' 256-byte aligned buffers then are), the
// left padding within the staged rows' lead, and 8-byte output vectors; and
// enough pixels per block.
static bool thin_fits(const ConvArgs& a, int dtype) {
  return dtype == 1 && conv_thin_pays(a.Hc, a.Wc, a.cols ? a.ncols : a.Cout, a.cols != nullptr, a.delta_T) && !a.pool && !a.add_mode && !a.out_f32 && !a.vin.chmap && a.K <= 32 && (a.W * a.C) % 8 == 0 &&
         a.in.row_elems == (int64_t)a.H * a.W * a.C && reinterpret_cast<uintptr_t>(a.in.p) % 16 == 0 &&
         reinterpret_cast<uintptr_t>(a.out) % 8 == 0 && a.pad * a.C <= THIN_LEAD && a.Cout % 4 == 0 &&
         a.out_row % 4 == 0 && a.Wc <= 1024 &&
         ((THIN_ROWS - 1) * a.stride + a.kh) * (THIN_LEAD + a.W * a.C + a.kw * a.C + 8) * 2 <= 64 * 1024;
}

static hipError_t launch_thin(const ConvArgs& a0, int nslots, hipStream_t s) {
  ConvArgs a = a0;
  a.dWc = make_divu32((uint32_t)a.Wc);
  const int rows = std::min(THIN_ROWS, a.Hc), bands = (a.Hc + rows - 1) / rows;
  // a staged row: lead, data, and what the last pixel's taps read past it
  const int past = std::max(0, (a.Wc - 1) * a.stride - a.pad + a.kw - a.W) * a.C;
  const int rs = THIN_LEAD + (a.W * a.C + past + 7) / 8 * 8;
  const int nrows = (rows - 1) * a.stride + a.kh;
  const int ncol = a.cols ? a.ncols : a.Cout;
  const int tn = ncol <= 16 ? 1 : ncol <= 32 ? 2 : 4;
  if ((int64_t)a.nx * bands >= INT32_MAX || nslots > 65535) return hipErrorInvalidValue;
  const dim3 grid((unsigned)(a.nx * bands), (unsigned)nslots, (unsigned)((ncol + 16 * tn - 1) / (16 * tn)));
  const size_t lds = (size_t)nrows * rs * 2;
#define MURE_THIN(TN)                                                                                      \
  if (tn == TN) {                                                                                          \
    if (a.cols) hipLaunchKernelGGL((conv_thin_kernel<TN, true>), grid, dim3(256), lds, s, a, rows, bands, rs, nrows); \
    else hipLaunchKernelGGL((conv_thin_kernel<TN, false>), grid, dim3(256), lds, s, a, rows, bands, rs, nrows);       \
  }
  MURE_THIN(1)
  MURE_THIN(2)
  MURE_THIN(4)
#undef MURE_THIN
  return hipGetLastError();
}

hipError_t launch_conv(const ConvArgs& a, int nslots, int dtype, hipStream_t s) {
  if (nslots <= 0 || a.nx <= 0) return hipSuccess;
  if (a.cols && (a.in.mode != MODE_CACHE || a.add_mode || a.ncols <= 0)) return hipErrorInvalidValue;
  if (a.cols) nslots = 1;
  if (thin_fits(a, dtype)) return launch_thin(a, nslots, s);
  const int64_t Mslot = (int64_t)a.nx * a.P;
  const int ncol = a.cols ? a.ncols : a.Cout;
  dim3 grid((unsigned)((Mslot + 63) / 64), (unsigned)nslots, (unsigned)((ncol + 63) / 64));
  if (dtype == 0)
    hipLaunchKernelGGL((conv_mfma_kernel<float, 64, 64>), grid, dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL((conv_mfma_kernel<bf16_t, 64, 64>), grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace mure
