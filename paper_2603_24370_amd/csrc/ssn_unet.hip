// Learned initialiser: a U-Net on BF16 MFMA (gfx950) with FP32 accumulation.
//
// Layout: activations NHWC in BF16 (element (n, y, x, c) at
// ((n * H + y) * W + x) * cs + coff + c, so a concatenation is two channel
// ranges of one buffer); 3x3 weights [co][tap][ci] with tap = 3 * ky + kx for
// offsets (ky - 1, kx - 1). Master weights, Adam moments and gradients are FP32.
//
// Kernels:
//   conv3x3_rows   implicit GEMM for the larger layers, M = out channels, N =
//                  pixels, K = 9 * in channels, v_mfma_f32_32x32x16_bf16, input
//                  patches of 32 channels staged in LDS; forward (bias + SiLU
//                  epilogue) and backward-data (the same GEMM with flipped,
//                  transposed weights; optional SiLU' epilogue);
//   conv3x3_taps   the same GEMM for small grids (few images, deep levels), the
//                  patch of all input channels in LDS, the weights streamed;
//   conv3x3_mfma   the same GEMM with both operands read directly, for image
//                  rows that are no multiple of 32 pixels;
//   conv3x3_wgrad  weight gradient, M = out channels, N = in channels per tap,
//                  K = pixels, operands read from LDS with transposing loads,
//                  split over pixel chunks with a fixed-order reduction
//                  (deterministic); its launch also sums the bias gradient;
//   pool / upsample (their backward passes with SiLU') / head 1x1 with the MSE /
//   Adam (optionally with global-norm gradient clipping) with the packing of the
//   BF16 weights: kernels on 8-channel vectors.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "../../include/ss.h"
#include "../../include/ssn.h"

namespace ssn {

typedef unsigned short bf16_t;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

__device__ __forceinline__ float bf2f(bf16_t x) { return __uint_as_float(((unsigned)x) << 16); }

// round to nearest even (finite inputs; Inf/NaN keep their class)
__device__ __forceinline__ bf16_t f2bf(float f) {
  unsigned u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u) return (bf16_t)((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
  u += 0x7fffu + ((u >> 16) & 1u);
  return (bf16_t)(u >> 16);
}

__device__ __forceinline__ float silu_f(float z) { return z / (1.0f + __expf(-z)); }
__device__ __forceinline__ float silu_grad_f(float z) {
  const float s = 1.0f / (1.0f + __expf(-z));
  return s * (1.0f + z * (1.0f - s));
}

// NHWC view
struct TV {
  bf16_t* p;
  int N, H, W;
  int cs;   // channel stride of the buffer
  int coff; // first channel of this view
  int C;    // channels of this view
};

__device__ __forceinline__ long tv_at(const TV& t, int n, int y, int x) {
  return ((long)(n * t.H + y) * t.W + x) * t.cs + t.coff;
}

struct ConvArgs {
  TV in;             // input, in.C a multiple of 16
  const bf16_t* w;   // weight fragments (frag_index), output rows rounded up to 32
  const float* bias; // [Co] or nullptr
  int Co;
  TV out_z;          // forward: pre-activation (p may be nullptr)
  TV out;            // forward: SiLU(z); backward: gradient w.r.t. the input of the layer
  TV zprev;          // backward: if p != nullptr multiply by SiLU'(zprev)
  int mode;          // 0 forward, 1 backward-data
};

// Weights are kept as the fragments the products read: the 16 x 32 block of
// output channels co0 .. co0 + 31, tap t and input channels 16 c .. 16 c + 15 is
// 1 KB in lane order, so a wave's load of a fragment is contiguous (read from
// [co][tap][ci] rows it touched 32 cache lines of 32 bytes each). Fragments of
// one co0 follow each other in the order (t, c). Row m of a fragment is channel
// conv_row(m): a lane of the product (pixel r, rows 8 (v / 4) + 4 half + v % 4)
// then holds the 16 neighbouring channels co0 + 16 half + v of one pixel.
__host__ __device__ __forceinline__ int conv_row(int m) { return ((m >> 2) & 1) * 16 + (m >> 3) * 4 + (m & 3); }

// element of channel co, tap t, input channel ci (nc = input channels / 16)
__device__ __forceinline__ long frag_index(int co, int t, int ci, int nc) {
  const int cl = co & 31;
  const int m = ((cl >> 2) & 3) * 8 + (cl >> 4) * 4 + (cl & 3);  // conv_row(m) = cl
  return ((((long)(co >> 5) * 9 + t) * nc + (ci >> 4)) * 64 + ((ci >> 3) & 1) * 32 + m) * 8 + (ci & 7);
}

__device__ __forceinline__ u32x4 load_u32x4(const bf16_t* p) { return *reinterpret_cast<const u32x4*>(p); }
__device__ __forceinline__ bf16x8 load_frag(const bf16_t* p) { return *reinterpret_cast<const bf16x8*>(p); }

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;

// two floats rounded to nearest even, the first in the low half
__device__ __forceinline__ unsigned pack2(float lo, float hi) {
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}

// End of a convolution at one pixel: the lane's 16 channels co .. co + 15 as two
// 16-byte vectors per tensor. Forward: z = acc + bias and SiLU(z); backward:
// acc, times SiLU'(zprev) where there is one.
template <int MODE>
__device__ __forceinline__ void conv_store(const ConvArgs& a, const f32x16& acc, const float (&bias)[16], int n, int y,
                                           int x, int co) {
  bf16_t* oo = a.out.p + tv_at(a.out, n, y, x) + co;
  if (MODE == 0) {
    u32x4 zv[2], av[2];
#pragma unroll
    for (int v = 0; v < 16; v += 2) {
      const float z0 = acc[v] + bias[v], z1 = acc[v + 1] + bias[v + 1];
      zv[v >> 3][(v & 7) >> 1] = pack2(z0, z1);
      av[v >> 3][(v & 7) >> 1] = pack2(silu_f(z0), silu_f(z1));
    }
    bf16_t* zo = a.out_z.p + tv_at(a.out_z, n, y, x) + co;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      *reinterpret_cast<u32x4*>(zo + 8 * k) = zv[k];
      *reinterpret_cast<u32x4*>(oo + 8 * k) = av[k];
    }
  } else {
    u32x4 zv[2] = {{0u, 0u, 0u, 0u}, {0u, 0u, 0u, 0u}}, gv[2];
    if (a.zprev.p) {
      const bf16_t* zp = a.zprev.p + tv_at(a.zprev, n, y, x) + co;
#pragma unroll
      for (int k = 0; k < 2; ++k) zv[k] = load_u32x4(zp + 8 * k);
    }
#pragma unroll
    for (int v = 0; v < 16; v += 2) {
      float g0 = acc[v], g1 = acc[v + 1];
      if (a.zprev.p) {
        const unsigned w2 = zv[v >> 3][(v & 7) >> 1];
        g0 *= silu_grad_f(bf2f((bf16_t)(w2 & 0xffffu)));
        g1 *= silu_grad_f(bf2f((bf16_t)(w2 >> 16)));
      }
      gv[v >> 3][(v & 7) >> 1] = pack2(g0, g1);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) *reinterpret_cast<u32x4*>(oo + 8 * k) = gv[k];
  }
}

// the 16 biases of a lane's channels (forward; zero otherwise)
template <int MODE>
__device__ __forceinline__ void conv_bias(const ConvArgs& a, int co, float (&bias)[16]) {
#pragma unroll
  for (int v = 0; v < 16; ++v) bias[v] = MODE == 0 ? a.bias[co + v] : 0.0f;
}

// Each wave: 32 output channels x (32 * WN) pixels; block: WB waves along pixels.
// Products of one output accumulate in the order tap, channel.
template <int WN, int WB, int MODE>
__global__ void __launch_bounds__(64 * WB) conv3x3_mfma(ConvArgs a) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 31, half = lane >> 5;
  const int H = a.in.H, W = a.in.W, Ci = a.in.C, nc = Ci / 16;
  const long P = (long)a.in.N * H * W;
  const long pixbase = ((long)blockIdx.x * WB + wave) * (32 * WN);
  int pn[WN], py[WN], px[WN];
  bool pv[WN];
#pragma unroll
  for (int f = 0; f < WN; ++f) {
    const long pix = pixbase + f * 32 + r;
    pv[f] = pix < P;
    const long pp = pv[f] ? pix : 0;
    pn[f] = (int)(pp / ((long)H * W));
    const int rem = (int)(pp - (long)pn[f] * H * W);
    py[f] = rem / W;
    px[f] = rem - py[f] * W;
  }
  f32x16 acc[WN];
#pragma unroll
  for (int f = 0; f < WN; ++f)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[f][v] = 0.0f;
  const bf16_t* wp = a.w + (long)blockIdx.y * 9 * nc * 512 + lane * 8;
  bf16x8 zero;
#pragma unroll
  for (int j = 0; j < 8; ++j) zero[j] = (__bf16)0.0f;
  for (int t = 0; t < 9; ++t) {
    const int dy = t / 3 - 1, dx = t % 3 - 1;
    long boff[WN];
    bool bv[WN];
#pragma unroll
    for (int f = 0; f < WN; ++f) {
      const int yy = py[f] + dy, xx = px[f] + dx;
      bv[f] = pv[f] && yy >= 0 && yy < H && xx >= 0 && xx < W;
      boff[f] = bv[f] ? tv_at(a.in, pn[f], yy, xx) + half * 8 : 0;
    }
    for (int c = 0; c < nc; ++c) {
      const bf16x8 A = load_frag(wp + (t * nc + c) * 512);
#pragma unroll
      for (int f = 0; f < WN; ++f) {
        const bf16x8 B = bv[f] ? load_frag(a.in.p + boff[f] + c * 16) : zero;
        acc[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A, B, acc[f], 0, 0, 0);
      }
    }
  }
  const int co = blockIdx.y * 32 + half * 16;
  if (co >= a.Co) return;
  float bias[16];
  conv_bias<MODE>(a, co, bias);
#pragma unroll
  for (int f = 0; f < WN; ++f)
    if (pv[f]) conv_store<MODE>(a, acc[f], bias, pn[f], py[f], px[f], co);
}

// The GEMM for small grids: a wave computes 32 output channels x 32 pixels, WCO
// waves of a block share the patch of those pixels, all input channels of it in
// LDS (3 rows x 34 pixels, zero outside the image, kTapPad elements of padding
// per pixel against bank conflicts). The products of one output accumulate in
// the order tap, channel (as conv3x3_mfma's), and the weight fragments are read
// in just that order, a contiguous stream. It is bound by latency: a wave or two
// per CU and one chain of 9 Ci / 16 products. So kTapAhead weight fragments are
// in flight ahead of the product, the next nine input fragments are read from
// LDS during the nine in hand, and the patch is staged kTapStage vectors per
// thread at a time. 256 -> 256 channels on 32^2, one image: 15 us (9 fragments
// ahead and one staging load at a time 27 us; conv3x3_mfma 33 us). Two rows per
// wave were slower everywhere (21 us). Requires W % 32 == 0.
constexpr int kTapPad = 8, kTapAhead = 36, kTapStage = 16;  // kTapAhead: an even multiple of 9

__host__ __device__ constexpr long tap_lds_bytes(int Ci) { return 2L * 3 * 34 * (Ci + kTapPad); }

template <int WCO, int MODE>
__global__ void __launch_bounds__(64 * WCO) __attribute__((amdgpu_waves_per_eu(1, 2))) conv3x3_taps(ConvArgs a) {
  constexpr int NT = 64 * WCO, PW = 34, PR = 3;
  extern __shared__ __align__(16) bf16_t patch[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 31, half = lane >> 5;
  const int H = a.in.H, W = a.in.W, Ci = a.in.C, nc = Ci / 16, pitch = Ci + kTapPad;
  const int xt = W / 32, yt = H;
  const int n = blockIdx.x / (xt * yt);
  const int rem = blockIdx.x - n * xt * yt;
  const int y0 = rem / xt, x0 = (rem - y0 * xt) * 32;
  const int ct = blockIdx.y * WCO + wave;  // channel block of the wave
  const bf16_t* __restrict__ wp = a.w + (long)ct * 9 * nc * 512 + lane * 8;
  const int nf = 9 * nc;
  bf16x8 wa[kTapAhead];
#pragma unroll
  for (int k = 0; k < kTapAhead; ++k)
    if (k < nf) wa[k] = load_frag(wp + k * 512);
  // the patch, kTapStage vectors per thread in flight
  const int nv = Ci / 8, ne = PR * PW * nv;
  const bf16_t* __restrict__ base = a.in.p + a.in.coff + (long)n * H * W * a.in.cs;
  for (int i0 = tid; i0 < ne; i0 += NT * kTapStage) {
    u32x4 val[kTapStage];
    int at[kTapStage];
#pragma unroll
    for (int u = 0; u < kTapStage; ++u) {
      const int it = i0 + u * NT;
      const int e = it / nv, v = it - e * nv;
      const int row = e / PW, px = e - row * PW;
      const int yy = y0 + row - 1, xx = x0 + px - 1;
      at[u] = it < ne ? e * pitch + v * 8 : -1;
      val[u] = u32x4{0u, 0u, 0u, 0u};
      if (it < ne && (unsigned)yy < (unsigned)H && (unsigned)xx < (unsigned)W)
        val[u] = load_u32x4(base + (long)(yy * W + xx) * a.in.cs + v * 8);
    }
#pragma unroll
    for (int u = 0; u < kTapStage; ++u)
      if (at[u] >= 0) *reinterpret_cast<u32x4*>(patch + at[u]) = val[u];
  }
  __syncthreads();
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
  const bf16_t* bp = patch + r * pitch + half * 8;
  int c = 0, dx = 0, row = 0;  // the next input fragment: tap (row, dx), channels 16 c ..
  bf16x8 b[2][9];
  auto load_b = [&](bf16x8 (&bb)[9]) {
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      bb[k] = load_frag(bp + (row * PW + dx) * pitch + c * 16);
      if (++c == nc) {
        c = 0;
        if (++dx == 3) {
          dx = 0;
          ++row;
        }
      }
    }
  };
  load_b(b[0]);
  for (int f0 = 0; f0 < nf; f0 += kTapAhead) {  // nf is a multiple of 9
#pragma unroll
    for (int g = 0; g < kTapAhead / 9; ++g) {
      const int f = f0 + 9 * g;
      if (f >= nf) break;
      if (f + 9 < nf) load_b(b[(g + 1) & 1]);
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa[9 * g + k], b[g & 1][k], acc, 0, 0, 0);
        if (f + k + kTapAhead < nf) wa[9 * g + k] = load_frag(wp + (f + k + kTapAhead) * 512);
      }
    }
  }
  const int co = ct * 32 + half * 16;
  if (co >= a.Co) return;
  float bias[16];
  conv_bias<MODE>(a, co, bias);
  conv_store<MODE>(a, acc, bias, n, y0, x0 + r, co);
}

// LDS-tiled implicit GEMM for the larger layers. Block: WCO x WPX waves over R
// image rows; wave (i, j) computes 32 output channels (co0 + 32 i ..) x 32 pixels
// (x0 + 32 j ..) of each of the rows y0 .. y0 + R - 1, with D = weights x input.
// A block walks `per` tiles (down the image columns) and, per tile, the input
// channels in chunks of 32. The patch of a (tile, chunk) (R + 2 rows x
// (32 WPX + 2) pixels, zero outside the image) is read into registers while the
// one before it is computed, and goes to LDS between two barriers, so that a
// block always has a patch in flight. A wave keeps the 18 weight fragments of its
// chunk in registers (they are loaded once where there is one chunk, and each
// tap row's again as soon as its last row is done where there are more), and
// walks the patch row by row: the six fragments of a patch row (three shifts,
// two channel halves) serve up to three output rows, so LDS is read once per
// three products. Products of one output accumulate in the order chunk, tap,
// channel half. LDS entries are padded to kKP channels so that lanes reading
// neighbouring pixels fall in different banks. Requires W % (32 WPX) == 0,
// H % R == 0, in.C % 16 == 0 (weight fragments exist up to gridDim.y * 32 WCO).
constexpr int kKC = 32, kKP = 40;

template <int WCO, int WPX, int R, int MODE>
__global__ void __launch_bounds__(64 * WCO * WPX) __attribute__((amdgpu_waves_per_eu(2)))
conv3x3_rows(ConvArgs a, int ntiles, int per) {
  constexpr int NT = 64 * WCO * WPX, PX = 32 * WPX, PW = PX + 2, PR = R + 2;
  constexpr int NE = PR * PW * 4, NV = (NE + NT - 1) / NT;  // 16-byte vectors of a patch, and per thread
  __shared__ __align__(16) bf16_t sin_[PR * PW * kKP];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wi = wave / WPX, wj = wave - wi * WPX;
  const int r = lane & 31, half = lane >> 5;
  const int H = a.in.H, W = a.in.W, Ci = a.in.C;
  const int xt = W / PX, yt = H / R;
  const int nchunk = (Ci + kKC - 1) / kKC;
  const int cow = blockIdx.y * (32 * WCO) + wi * 32;
  const int t0 = blockIdx.x * per, t1 = min(ntiles, t0 + per);
  if (t0 >= t1) return;
  // tile t: row block t % yt of column block (t / yt) % xt of image t / (xt yt)
  auto tile_at = [&](int t, int& n, int& x0, int& y0) {
    const int c = t / yt;
    y0 = (t - c * yt) * R;
    n = c / xt;
    x0 = (c - n * xt) * PX;
  };
  const int nc = Ci / 16;
  const bf16_t* __restrict__ wp = a.w + (long)(cow >> 5) * 9 * nc * 512 + lane * 8;
  bf16x8 wa[9][2];
  auto load_w = [&](int dy, int c0) {
    const int c = c0 >> 4, c2 = min(c + 1, nc - 1);  // a lone last half is loaded twice, used once
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) {
      const int t = dy * 3 + dx;
      wa[t][0] = load_frag(wp + (t * nc + c) * 512);
      wa[t][1] = load_frag(wp + (t * nc + c2) * 512);
    }
  };
  // patch of (tile t, chunk c0) into registers
  u32x4 pre[NV];
  auto fetch = [&](int t, int c0) {
    int n, x0, y0;
    tile_at(t, n, x0, y0);
    const bf16_t* __restrict__ base = a.in.p + a.in.coff + c0 + (long)n * H * W * a.in.cs;
    const int nv = min(kKC, Ci - c0) >> 3;
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      const int it = tid + q * NT;
      const int v = it & 3, e = it >> 2;
      const int row = e / PW, px = e - row * PW;
      const int yy = y0 + row - 1, xx = x0 + px - 1;
      u32x4 val = {0u, 0u, 0u, 0u};
      if (it < NE && v < nv && (unsigned)yy < (unsigned)H && (unsigned)xx < (unsigned)W)
        val = *reinterpret_cast<const u32x4*>(base + (long)(yy * W + xx) * a.in.cs + v * 8);
      pre[q] = val;
    }
  };
  fetch(t0, 0);
#pragma unroll
  for (int dy = 0; dy < 3; ++dy) load_w(dy, 0);
  for (int t = t0; t < t1; ++t) {
    f32x16 acc[R];
#pragma unroll
    for (int q = 0; q < R; ++q)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[q][v] = 0.0f;
    for (int ck = 0; ck < nchunk; ++ck) {
      const bool two = ck * kKC + 16 < Ci;
      const int cn = ck + 1 < nchunk ? (ck + 1) * kKC : 0;  // next chunk's first channel
      const int tn = ck + 1 < nchunk ? t : t + 1;
      __syncthreads();
#pragma unroll
      for (int q = 0; q < NV; ++q) {
        const int it = tid + q * NT;
        if (it < NE) *reinterpret_cast<u32x4*>(sin_ + (it >> 2) * kKP + (it & 3) * 8) = pre[q];
      }
      __syncthreads();
      if (tn < t1) fetch(tn, cn);
#pragma unroll
      for (int p = 0; p < PR; ++p) {
        bf16x8 b[3][2];
#pragma unroll
        for (int dx = 0; dx < 3; ++dx)
#pragma unroll
          for (int ks = 0; ks < 2; ++ks)
            b[dx][ks] = *reinterpret_cast<const bf16x8*>(sin_ + (p * PW + wj * 32 + r + dx) * kKP + ks * 16 + half * 8);
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) {
#pragma unroll
          for (int dy = 0; dy < 3; ++dy)
            if (p - dy >= 0 && p - dy < R)
              acc[p - dy] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa[dy * 3 + dx][0], b[dx][0], acc[p - dy], 0, 0, 0);
          if (two) {
#pragma unroll
            for (int dy = 0; dy < 3; ++dy)
              if (p - dy >= 0 && p - dy < R)
                acc[p - dy] =
                    __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa[dy * 3 + dx][1], b[dx][1], acc[p - dy], 0, 0, 0);
          }
        }
        if (nchunk > 1 && p >= R - 1) load_w(p - (R - 1), cn);
      }
    }
    // D[row][col]: lane holds pixel col = r and rows 8 (v / 4) + 4 half + v % 4, i.e.
    // channels cow + 16 half + v
    int n, x0, y0;
    tile_at(t, n, x0, y0);
    const int co = cow + half * 16;
    if (co < a.Co) {
      float bias[16];
      conv_bias<MODE>(a, co, bias);
#pragma unroll
      for (int q = 0; q < R; ++q) conv_store<MODE>(a, acc[q], bias, n, y0 + q, x0 + wj * 32 + r, co);
    }
  }
}

// Weight gradient: part[split][co][t][ci] = sum over this split's pixel chunks of
// gz[pix][co] * x[pix + d_t][ci]. A block takes a tile of 32 co x 32 ci; its waves
// 0 .. 2 one row of taps each (three accumulators), all four stage. A chunk is R
// image rows of CW pixels (R * CW <= kChunk): its gz pixels and the R + 2 x rows
// around them (CW + 2 pixels wide) go to LDS as they lie in memory, 32 channels
// (64 bytes) per pixel, in 16-byte vectors; the next chunk's are read into
// registers meanwhile. The products need both operands with the pixels of a
// channel in a lane, which is what the transposing LDS read gives: four pixels x
// sixteen channels per sixteen lanes, so a tap's shift is an offset of whole
// pixels. The gz fragment of 16 pixels serves a wave's three taps. Every tap sums
// its chunks' rows in 16-pixel steps, in order. Requires channel vectors of 8
// (cs, coff, C multiples of 8), W % CW == 0, H % R == 0, (R + 2)(CW + 2) <= kXPix.
// Bound by LDS reads (8 transposing reads of 512 bytes per 3 products) and by the
// latency of its loads at 1.5 blocks per CU. 96 -> 32 channels on 256^2, batch 8,
// with the bias sums: 68 us; storing every channel of a vector separately to
// transpose, and reading three 16-byte words per product: 105 + 13 us.
constexpr int kChunk = 256;         // pixels per chunk
constexpr int kXPix = 396;          // staged x pixels: (R + 2)(CW + 2)
struct WgradArgs {
  TV gz;        // gradient w.r.t. the layer's pre-activation (C = Co)
  TV x;         // layer input (C = Ci)
  float* part;  // [nsplit][Co][9][Ci]
  int nsplit;
  int R;        // rows per chunk
  float* cpart; // per-block channel sums of gz ([kPartBlocks][Co])
};

typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((address_space(3))) s16x4* lds_s16x4;

// 16 channels x 8 pixels per 16 lanes: p points at the lane's (pixel, four
// channels) of the first four pixels, 64 bytes per pixel
__device__ __forceinline__ bf16x8 load_tr(const bf16_t* p) {
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)p);
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(p + 4 * 32));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

constexpr int kPartBlocks = 256;

__device__ __forceinline__ void unpack8(const u32x4 v, float (&x)[8]);

// Block b of kPartBlocks per 256 channels: channel sums of a bf16 NHWC view into
// fp32 partials [kPartBlocks][C]. Block (b, y) takes channels [256 y, 256 y + Cc),
// Cc = min(C - 256 y, 256), a multiple of 8: thread t sums the 8-channel group
// t % G (G = Cc / 8) over the pixels b0 + t / G, step 256 / G, of the block's pixel
// range; the lane sums of each channel are then added in lane order. red: 2048
// floats of LDS.
__device__ __forceinline__ void channel_sums(const TV& g, int b, int y, float* __restrict__ part, float* red) {
  const int t = threadIdx.x, C = g.C;
  const long npix = (long)g.N * g.H * g.W;
  const int c0 = 256 * y;
  const int Cc = min(C - c0, 256);
  const long per = (npix + kPartBlocks - 1) / kPartBlocks;
  const long b0 = b * per, b1 = std::min(npix, b0 + per);
  const int G = Cc / 8, L = 256 / G;
  const int e = t % G, l = t / G;
  float s[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
  if (l < L) {
    const bf16_t* gp = g.p + g.coff + c0 + 8 * e;
    long p = b0 + l;
    constexpr int U = 8;  // loads in flight
    for (; p + (U - 1) * L < b1; p += U * L) {
      u32x4 raw[U];
#pragma unroll
      for (int u = 0; u < U; ++u) raw[u] = load_u32x4(gp + (p + u * L) * g.cs);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float v[8];
        unpack8(raw[u], v);
#pragma unroll
        for (int j = 0; j < 8; ++j) s[j] += v[j];
      }
    }
    for (; p < b1; p += L) {
      float v[8];
      unpack8(load_u32x4(gp + p * g.cs), v);
#pragma unroll
      for (int j = 0; j < 8; ++j) s[j] += v[j];
    }
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) red[t * 8 + j] = s[j];
  __syncthreads();
  if (t < Cc) {
    float a = 0.0f;
    for (int k = 0; k < L; ++k) a += red[(k * G + t / 8) * 8 + t % 8];
    part[(long)b * C + c0 + t] = a;
  }
}

// Blocks 0 .. tiles * nsplit - 1 form the weight gradient, the rest the channel
// sums of gz (the bias gradient).
template <int CW>
__global__ void __launch_bounds__(256) conv3x3_wgrad(WgradArgs a) {
  __shared__ __align__(16) bf16_t gzs[kChunk * 32];  // [pixel][co]
  __shared__ __align__(16) bf16_t xs[kXPix * 32];    // [row][pixel + 1][ci]
  constexpr int XW = CW + 2;
  constexpr int NG = kChunk * 4 / 256, NX = (kXPix * 4 + 255) / 256;
  const int lane = threadIdx.x & 63, dy = threadIdx.x >> 6;
  const int H = a.x.H, W = a.x.W, Ci = a.x.C, Co = a.gz.C, R = a.R;
  const int tci = (Ci + 31) / 32, tco = (Co + 31) / 32;
  const int nw = tci * tco * a.nsplit;
  if ((int)blockIdx.x >= nw) {
    const int k = blockIdx.x - nw;
    channel_sums(a.gz, k % kPartBlocks, k / kPartBlocks, a.cpart, reinterpret_cast<float*>(gzs));
    return;
  }
  const int tile = blockIdx.x % (tci * tco), split = blockIdx.x / (tci * tco);
  const int ci0 = (tile % tci) * 32, co0 = (tile / tci) * 32;
  const int cpr = W / CW, rpi = H / R;
  const int nchunks = a.x.N * rpi * cpr;
  const int ng = R * CW * 4, nx = (R + 2) * XW * 4;
  u32x4 pg[NG], px[NX];
  auto fetch = [&](int ch) {
    const int n = ch / (rpi * cpr);
    const int rem = ch - n * rpi * cpr;
    const int y0 = (rem / cpr) * R, x0 = (rem - (rem / cpr) * cpr) * CW;
    const bf16_t* __restrict__ gb = a.gz.p + tv_at(a.gz, n, y0, x0) + co0;
    const bf16_t* __restrict__ xb = a.x.p + tv_at(a.x, n, 0, 0) + ci0;
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      const int e = threadIdx.x + q * 256, v = e & 3, p = e >> 2;
      const int py = p / CW, pxx = p - py * CW;
      pg[q] = u32x4{0u, 0u, 0u, 0u};
      if (e < ng && co0 + 8 * v < Co) pg[q] = load_u32x4(gb + (long)(py * W + pxx) * a.gz.cs + 8 * v);
    }
#pragma unroll
    for (int q = 0; q < NX; ++q) {
      const int e = threadIdx.x + q * 256, v = e & 3, k = e >> 2;
      const int rr = k / XW, p = k - rr * XW;
      const int yy = y0 + rr - 1, xx = x0 + p - 1;
      px[q] = u32x4{0u, 0u, 0u, 0u};
      if (e < nx && (unsigned)yy < (unsigned)H && (unsigned)xx < (unsigned)W && ci0 + 8 * v < Ci)
        px[q] = load_u32x4(xb + (long)(yy * W + xx) * a.x.cs + 8 * v);
    }
  };
  f32x16 acc[3];
#pragma unroll
  for (int d = 0; d < 3; ++d)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[d][v] = 0.0f;
  // the lane's place in a transposing read: pixels 8 (lane / 32) + (lane % 16) / 4,
  // channels 16 (lane / 16 % 2) + 4 (lane % 4)
  const int tr = (8 * (lane >> 5) + ((lane & 15) >> 2)) * 32 + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  fetch(split);  // nsplit <= nchunks
  for (int ch = split; ch < nchunks; ch += a.nsplit) {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      const int e = threadIdx.x + q * 256;
      if (e < ng) *reinterpret_cast<u32x4*>(gzs + e * 8) = pg[q];
    }
#pragma unroll
    for (int q = 0; q < NX; ++q) {
      const int e = threadIdx.x + q * 256;
      if (e < nx) *reinterpret_cast<u32x4*>(xs + e * 8) = px[q];
    }
    __syncthreads();
    if (ch + a.nsplit < nchunks) fetch(ch + a.nsplit);
    if (dy < 3)
      for (int rr = 0; rr < R; ++rr) {
        const bf16_t* ap = gzs + rr * CW * 32 + tr;
        const bf16_t* bp = xs + (rr + dy) * XW * 32 + tr;
#pragma unroll
        for (int kk = 0; kk < CW; kk += 16) {
          const bf16x8 A = load_tr(ap + kk * 32);
#pragma unroll
          for (int d = 0; d < 3; ++d)
            acc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A, load_tr(bp + (kk + d) * 32), acc[d], 0, 0, 0);
        }
      }
  }
  if (dy < 3) {
    const int r = lane & 31, half = lane >> 5;
    const int ci = ci0 + r;
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int co = co0 + (v >> 2) * 8 + half * 4 + (v & 3);
        if (co < Co && ci < Ci) a.part[(((long)split * Co + co) * 9 + dy * 3 + d) * Ci + ci] = acc[d][v];
      }
  }
}

// out[k] = sum over s of part[s][k], for two sets of partials in one launch (a
// layer's weight gradient, blocks 0 .. wb - 1, and its bias gradient). A block
// takes 32 outputs; its 8 groups of 32 lanes each sum a contiguous eighth of the
// splits in order, and the eight sums are added in group order (fixed order:
// deterministic). Sixteen loads are in flight per lane.
struct ReduceSet {
  const float* part;
  float* out;
  long n;
  int nsplit;
};

__global__ void __launch_bounds__(256) reduce_splits(ReduceSet w, ReduceSet b, int wb) {
  __shared__ float red[256];
  const bool second = (int)blockIdx.x >= wb;
  const float* __restrict__ part = second ? b.part : w.part;
  float* __restrict__ out = second ? b.out : w.out;
  const long n = second ? b.n : w.n;
  const int nsplit = second ? b.nsplit : w.nsplit;
  const int kl = threadIdx.x & 31, g = threadIdx.x >> 5;
  const long k = (long)((int)blockIdx.x - (second ? wb : 0)) * 32 + kl;
  const int per = (nsplit + 7) / 8;
  const int s0 = min(nsplit, g * per), s1 = min(nsplit, s0 + per);
  float s = 0.0f;
  if (k < n) {
    constexpr int U = 16;
    int i = s0;
    for (; i + U <= s1; i += U) {
      float v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = part[(long)(i + u) * n + k];
#pragma unroll
      for (int u = 0; u < U; ++u) s += v[u];
    }
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = i + u < s1 ? part[(long)(i + u) * n + k] : 0.0f;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i + u < s1) s += v[u];
  }
  red[threadIdx.x] = s;
  __syncthreads();
  if (g == 0 && k < n) {
    float o = 0.0f;
#pragma unroll
    for (int j = 0; j < 8; ++j) o += red[j * 32 + kl];
    out[k] = o;
  }
}

// 8 bf16 channels of a 16-byte vector as floats
__device__ __forceinline__ void unpack8(const u32x4 v, float (&x)[8]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    x[2 * j] = bf2f((bf16_t)(v[j] & 0xffffu));
    x[2 * j + 1] = bf2f((bf16_t)(v[j] >> 16));
  }
}

// Pooling, upsampling and their backward passes (with SiLU' of the layer below)
// on NHWC views, one 16-byte vector of 8 channels per thread (C, cs and coff
// multiples of 8): block (bx, y, b) covers 256 vectors of row y of image b, so a
// thread's place costs one 32-bit division. All are bound by memory: on 256^2 x 32
// channels, batch 8, avgpool2_bwd 25 us (135 MB; with SiLU' in a pass of its own 43).
__device__ __forceinline__ u32x4 pack8(const float (&x)[8]) {
  u32x4 r;
#pragma unroll
  for (int j = 0; j < 4; ++j) r[j] = pack2(x[2 * j], x[2 * j + 1]);
  return r;
}

__device__ __forceinline__ void store_u32x4(bf16_t* p, const u32x4 v) { *reinterpret_cast<u32x4*>(p) = v; }

// body(b, y, x, c) for every vector of view t: image, pixel and first channel
template <class F>
__device__ __forceinline__ void for_vectors(const TV& t, F&& body) {
  const int C8 = t.C / 8, k = blockIdx.x * 256 + threadIdx.x;
  if (k >= t.W * C8) return;
  const int x = k / C8, c = 8 * (k - x * C8);
  for (int b = blockIdx.z; b < t.N; b += gridDim.z)
    for (int y = blockIdx.y; y < t.H; y += gridDim.y) body(b, y, x, c);
}

// sum of the 2x2 block (y, x) of a view, rows first
__device__ __forceinline__ void sum2x2(const TV& t, int b, int y, int x, int c, float (&s)[8]) {
  u32x4 raw[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) raw[j] = load_u32x4(t.p + tv_at(t, b, 2 * y + (j >> 1), 2 * x + (j & 1)) + c);
#pragma unroll
  for (int e = 0; e < 8; ++e) s[e] = 0.0f;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float v[8];
    unpack8(raw[j], v);
#pragma unroll
    for (int e = 0; e < 8; ++e) s[e] += v[e];
  }
}

// g rounded to BF16 (as a gradient tensor holds it), times SiLU'(z)
__device__ __forceinline__ u32x4 times_silu_grad(const float (&g)[8], const u32x4 z) {
  float v[8], zz[8];
  unpack8(pack8(g), v);
  unpack8(z, zz);
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] *= silu_grad_f(zz[e]);
  return pack8(v);
}

__global__ void __launch_bounds__(256) avgpool2_fwd(TV in, TV out) {
  for_vectors(out, [&](int b, int y, int x, int c) {
    float s[8];
    sum2x2(in, b, y, x, c, s);
#pragma unroll
    for (int e = 0; e < 8; ++e) s[e] *= 0.25f;
    store_u32x4(out.p + tv_at(out, b, y, x) + c, pack8(s));
  });
}

// g = (g + gout / 4 spread over each 2x2 block) SiLU'(z)
__global__ void __launch_bounds__(256) avgpool2_bwd(TV gout, TV g, TV z) {
  for_vectors(g, [&](int b, int y, int x, int c) {
    bf16_t* o = g.p + tv_at(g, b, y, x) + c;
    const u32x4 go = load_u32x4(gout.p + tv_at(gout, b, y >> 1, x >> 1) + c), old = load_u32x4(o);
    const u32x4 zz = load_u32x4(z.p + tv_at(z, b, y, x) + c);
    float v[8], w[8];
    unpack8(go, v);
    unpack8(old, w);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = v[e] * 0.25f + w[e];
    store_u32x4(o, times_silu_grad(v, zz));
  });
}

__global__ void __launch_bounds__(256) upsample2_fwd(TV in, TV out) {
  for_vectors(in, [&](int b, int y, int x, int c) {
    const u32x4 v = load_u32x4(in.p + tv_at(in, b, y, x) + c);
#pragma unroll
    for (int j = 0; j < 4; ++j) store_u32x4(out.p + tv_at(out, b, 2 * y + (j >> 1), 2 * x + (j & 1)) + c, v);
  });
}

// g = (sum of gout over each 2x2 block) SiLU'(z)
__global__ void __launch_bounds__(256) upsample2_bwd(TV gout, TV g, TV z) {
  for_vectors(g, [&](int b, int y, int x, int c) {
    const u32x4 zz = load_u32x4(z.p + tv_at(z, b, y, x) + c);
    float s[8];
    sum2x2(gout, b, y, x, c, s);
    store_u32x4(g.p + tv_at(g, b, y, x) + c, times_silu_grad(s, zz));
  });
}

// The 1x1 head (cout <= 8 outputs, C % 8 == 0 input channels): one pixel per
// thread, channels moved as 16-byte vectors of 8 (load_u32x4).

// head: out[pix][o] = b[o] + sum_ci w[o][ci] a[pix][ci] (fp32 out, ci ascending)
__global__ void __launch_bounds__(256) head_fwd(TV a, const float* __restrict__ w, const float* __restrict__ b,
                                                int cout, float* __restrict__ out, long npix) {
  const long p = blockIdx.x * (long)blockDim.x + threadIdx.x;
  if (p >= npix) return;
  const bf16_t* ap = a.p + p * a.cs + a.coff;
  float s[8];
#pragma unroll
  for (int o = 0; o < 8; ++o) s[o] = o < cout ? b[o] : 0.0f;
  for (int c0 = 0; c0 < a.C; c0 += 8) {
    float x[8];
    unpack8(load_u32x4(ap + c0), x);
#pragma unroll
    for (int o = 0; o < 8; ++o)
      if (o < cout) {
#pragma unroll
        for (int j = 0; j < 8; ++j) s[o] += w[o * a.C + c0 + j] * x[j];
      }
  }
  for (int o = 0; o < cout; ++o) out[p * cout + o] = s[o];
}

// The loss is the mean squared error: the gradient at output k is
// 2 (out[k] - tgt[k]) / n, formed where it is used.

// head backward to its input, times SiLU'(z): ga[pix][ci] = SiLU'(z) sum_o gout[pix][o] w[o][ci];
// one 8-channel vector per thread
template <int COUT>
__global__ void __launch_bounds__(256) head_bwd_data(const float* __restrict__ out, const float* __restrict__ tgt,
                                                     float inv, const float* __restrict__ w, TV z, TV ga, long npix) {
  const int C = ga.C, C8 = C / 8;
  const int per = 256 / C8;  // pixels per block
  const int l = threadIdx.x / C8, c0 = 8 * (threadIdx.x - l * C8);
  const long p = (long)blockIdx.x * per + l;
  if (l >= per || p >= npix) return;
  float g[COUT];
#pragma unroll
  for (int o = 0; o < COUT; ++o) g[o] = inv * (out[p * COUT + o] - tgt[p * COUT + o]);
  float zz[8], r[8];
  unpack8(load_u32x4(z.p + p * z.cs + z.coff + c0), zz);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    float s = 0.0f;
#pragma unroll
    for (int o = 0; o < COUT; ++o) s += g[o] * w[o * C + c0 + j];
    r[j] = s * silu_grad_f(zz[j]);
  }
  store_u32x4(ga.p + p * ga.cs + ga.coff + c0, pack8(r));
}

// Per-block partials over a range of pixels of the head's weight gradient
// gw[o][ci] = sum_pix gout[pix][o] a[pix][ci] (wpart, [nblk][cout C], cout C <= 256), its
// bias gradient (bpart, [nblk][cout]) and the squared error (lpart). Thread t takes the
// entries (o, 8 channels) e = t % E, E = cout C / 8, over the pixels b0 + t / E, step
// L = 256 / E, and the bias of output t % cout over the pixels b0 + t / cout, step
// 256 / cout; lane sums are then added in lane order (deterministic). Eight pixels of a
// thread are in flight. One launch reads the outputs for all three; the bias and loss
// loops run over L1 and L2 copies.
__global__ void __launch_bounds__(256) head_sums(const float* __restrict__ out, const float* __restrict__ tgt,
                                                 float inv, TV a, int cout, long npix, float* __restrict__ wpart,
                                                 float* __restrict__ bpart, double* __restrict__ lpart) {
  __shared__ float red[256 * 8];
  __shared__ double dred[256];
  const int t = threadIdx.x;
  const int C = a.C, C8 = C / 8, E = cout * C8, L = 256 / E, K = cout * C;
  const int e = t % E, l = t / E;
  const int o = e / C8, c0 = (e - o * C8) * 8;
  const long per = (npix + gridDim.x - 1) / gridDim.x;
  const long b0 = blockIdx.x * per, b1 = std::min(npix, b0 + per);
  constexpr int U = 8;
  float s[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) s[j] = 0.0f;
  if (l < L) {
    const bf16_t* ap = a.p + a.coff + c0;
    for (long p0 = b0 + l; p0 < b1; p0 += U * L) {
      u32x4 raw[U];
      float ov[U], tv[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const long p = p0 + u * L < b1 ? p0 + u * L : p0;
        raw[u] = load_u32x4(ap + p * a.cs);
        ov[u] = out[p * cout + o];
        tv[u] = tgt[p * cout + o];
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (p0 + u * L < b1) {
          const float g = inv * (ov[u] - tv[u]);
          float x[8];
          unpack8(raw[u], x);
#pragma unroll
          for (int j = 0; j < 8; ++j) s[j] += g * x[j];
        }
    }
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) red[t * 8 + j] = s[j];
  __syncthreads();
  if (t < K) {
    const int oo = t / C, c = t - oo * C;
    const int ee = oo * C8 + c / 8, jj = c % 8;
    float acc = 0.0f;
    for (int q = 0; q < L; ++q) acc += red[(q * E + ee) * 8 + jj];
    wpart[(long)blockIdx.x * K + t] = acc;
  }
  __syncthreads();
  // bias and loss over the same range
  const int Lb = 256 / cout, ob = t % cout, lb = t / cout;
  float sb = 0.0f;
  double sl = 0.0;
  if (lb < Lb)
    for (long p0 = b0 + lb; p0 < b1; p0 += U * Lb) {
      float d[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const long p = p0 + u * Lb;
        d[u] = p < b1 ? out[p * cout + ob] - tgt[p * cout + ob] : 0.0f;
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (p0 + u * Lb < b1) {
#pragma clang fp contract(off)
          sb += inv * d[u];
          sl += (double)d[u] * d[u];
        }
    }
  red[t] = sb;
  dred[t] = sl;
  __syncthreads();
  if (t < cout) {
    float acc = 0.0f;
    for (int k = 0; k < Lb; ++k) acc += red[k * cout + t];
    bpart[(long)blockIdx.x * cout + t] = acc;
  }
  for (int k = 128; k > 0; k >>= 1) {
    if (t < k) dred[t] += dred[t + k];
    __syncthreads();
  }
  if (t == 0) lpart[blockIdx.x] = dred[0];
}

// gradient clipping by global L2 norm: per-block partial sums of g^2 (FP64,
// grid-stride ranges, tree order), then scale = min(1, max_norm / |g|)
__global__ void __launch_bounds__(256) grad_sq_partials(const float* __restrict__ g, long n,
                                                        double* __restrict__ part) {
  __shared__ double red[256];
  double s = 0.0;
  for (long k = blockIdx.x * 256L + threadIdx.x; k < n; k += (long)gridDim.x * 256L) s += (double)g[k] * g[k];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

__global__ void __launch_bounds__(256) grad_clip_scale(const double* __restrict__ part, int nblk, float max_norm,
                                                       float* __restrict__ scale) {
  __shared__ double red[256];
  double s = 0.0;
  for (int k = threadIdx.x; k < nblk; k += 256) s += part[k];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double norm = sqrt(red[0]);
    *scale = norm > (double)max_norm ? (float)((double)max_norm / norm) : 1.0f;
  }
}

// One 3x3 layer's parameters as the update and packing kernel walks them (blockIdx.y
// = layer; the segment after the last layer holds the head's weights and biases).
constexpr int kMaxConv = 22;  // 4 * 6 - 2 levels' layers
struct ParamLayer {
  long off, n;  // first parameter and parameter count (weights, then Co biases)
  int Co, Ci;   // 0 for the head
  bf16_t* wf;
  bf16_t* wb;
};
struct ParamLayers {
  ParamLayer l[kMaxConv + 1];
};

struct AdamArgs {
  float *m, *v;
  const float* g;
  const float* gscale;  // nullable: 1
  float lr, b1, b2, eps, c1, c2;
};

// ADAM: one step of Adam (Kingma and Ba 2015) with bias correction on the gradient
// times *gscale. Then the BF16 weight fragments (frag_index) of the layer: wf of
// w[co][t][ci], and wb of the backward-data weights w[co][8 - t][ci] with ci as the
// output channel. One launch for all layers (14 packing launches took 64 us of a
// step).
template <bool ADAM>
__global__ void __launch_bounds__(256) update_params(ParamLayers ls, float* __restrict__ p, AdamArgs a) {
  const ParamLayer L = ls.l[blockIdx.y];
  const float sc = ADAM && a.gscale ? *a.gscale : 1.0f;
  const int nw = L.Co * 9 * L.Ci;
  for (int q = blockIdx.x * 256 + threadIdx.x; q < (int)L.n; q += gridDim.x * 256) {
    const long k = L.off + q;
    float pk = p[k];
    if (ADAM) {
      const float gk = a.g[k] * sc;
      const float mk = a.b1 * a.m[k] + (1.0f - a.b1) * gk;
      const float vk = a.b2 * a.v[k] + (1.0f - a.b2) * gk * gk;
      a.m[k] = mk;
      a.v[k] = vk;
      pk -= a.lr * (mk / a.c1) / (sqrtf(vk / a.c2) + a.eps);
      p[k] = pk;
    }
    if (q < nw) {
      const int ci = q % L.Ci, w = q / L.Ci;
      const int t = w % 9, co = w / 9;
      const bf16_t b = f2bf(pk);
      L.wf[frag_index(co, t, ci, L.Ci / 16)] = b;
      L.wb[frag_index(ci, 8 - t, co, L.Co / 16)] = b;
    }
  }
}

}  // namespace ssn

// ================================================================ host side

using namespace ssn;

namespace {

thread_local std::string g_ssn_err;

int nfail(int code, const std::string& m) {
  g_ssn_err = m;
  return code;
}

#define SN_HIP(call)                                                                      \
  do {                                                                                    \
    hipError_t e_ = (call);                                                               \
    if (e_ != hipSuccess) return nfail(SS_EHIP, std::string(#call) + ": " + hipGetErrorString(e_)); \
  } while (0)

long rup(long x, long m) { return (x + m - 1) / m * m; }

struct HT {  // host handle of one NHWC bf16 buffer (capacity Ncap)
  bf16_t* p = nullptr;
  int H = 0, W = 0, cs = 0;
  TV view(int n, int coff, int C) const {
    TV t;
    t.p = p;
    t.N = n;
    t.H = H;
    t.W = W;
    t.cs = cs;
    t.coff = coff;
    t.C = C;
    return t;
  }
  TV all(int n) const { return view(n, 0, cs); }
};

struct ConvL {
  int Ci, Ci_real, Co, H, W;
  long w_off, b_off;  // float offsets into the flat parameter arrays
  bf16_t* wf;         // forward fragments, rup(Co, 32) * 9 * Ci elements
  bf16_t* wb;         // backward-data fragments, rup(Ci, 32) * 9 * Co elements
};

constexpr long kWgradPartFloats = 1024L * 9 * 1024;

}  // namespace

struct ssn_net {
  int levels, base, cin, cout, cin_pad, Ncap, H, W, L;
  // forward pass captured as a HIP graph for one (x, nb, out) triple
  hipGraphExec_t fgraph = nullptr;
  hipStream_t fcap = nullptr;
  const float* fx = nullptr;
  float* fout = nullptr;
  int fnb = 0;
  int conv_shape;  // 0: by problem size, 1: large direct blocks, 2: small direct blocks, 3: LDS-tiled
  hipStream_t stream;
  float *P, *G, *M, *V;
  long np;
  std::vector<ConvL> conv;  // enc0a enc0b ... mid.a mid.b dec(L-1)a dec(L-1)b ... dec0a dec0b
  long hw_off, hb_off;
  std::vector<int> ch;      // channels per level
  // activations
  HT X0;
  std::vector<HT> ZA, AA, ZB, CAT, Pin;  // Pin[l]: pooled input of level l (l >= 1), Pin[L]: bottleneck input
  HT ZMa, AMa, ZMb, AMb;
  std::vector<HT> ZDa, ADa, ZDb, ADb;
  // gradients
  std::vector<HT> gCAT, gT1, gT2, gT3, gP;  // gT3[l]: gradient at the pre-activation of dec_a(l)
  HT gM1, gM2;
  float *OUT, *part, *cpart;
  double* lpart;
  double* npart;   // per-block partial sums of the squared gradient
  float* gscale;   // gradient scale of the clipped Adam step (device)
  float clip = 0.0f;  // global L2 clipping norm of the Adam step (0: off)
  int adam_t;
  size_t bytes;
};

namespace {

// Carve (or, with base == nullptr, size) the workspace of a network.
size_t net_carve(ssn_net* n, char* base) {
  size_t off = 0;
  auto take = [&](size_t b) -> char* {
    char* p = base ? base + off : nullptr;
    off += (size_t)rup((long)b, 256);
    return p;
  };
  const int L = n->L, N = n->Ncap;
  auto tensor = [&](HT& t, int H, int W, int cs) {
    t.H = H;
    t.W = W;
    t.cs = cs;
    t.p = (bf16_t*)take((size_t)N * H * W * cs * 2);
  };
  n->P = (float*)take(n->np * 4);
  n->G = (float*)take(n->np * 4);
  n->M = (float*)take(n->np * 4);
  n->V = (float*)take(n->np * 4);
  for (ConvL& c : n->conv) {
    c.wf = (bf16_t*)take((size_t)rup(c.Co, 32) * 9 * c.Ci * 2);
    c.wb = (bf16_t*)take((size_t)rup(c.Ci, 32) * 9 * c.Co * 2);
  }
  tensor(n->X0, n->H, n->W, n->cin_pad);
  n->ZA.assign(L, HT()); n->AA.assign(L, HT()); n->ZB.assign(L, HT()); n->CAT.assign(L, HT());
  n->Pin.assign(L + 1, HT());
  n->ZDa.assign(L, HT()); n->ADa.assign(L, HT()); n->ZDb.assign(L, HT()); n->ADb.assign(L, HT());
  n->gCAT.assign(L, HT()); n->gT1.assign(L, HT()); n->gT2.assign(L, HT()); n->gT3.assign(L, HT());
  n->gP.assign(L + 1, HT());
  for (int l = 0; l < L; ++l) {
    const int H = n->H >> l, W = n->W >> l, c = n->ch[l], cn = n->ch[l + 1];
    tensor(n->ZA[l], H, W, c); tensor(n->AA[l], H, W, c); tensor(n->ZB[l], H, W, c);
    tensor(n->CAT[l], H, W, cn + c);
    tensor(n->ZDa[l], H, W, c); tensor(n->ADa[l], H, W, c); tensor(n->ZDb[l], H, W, c); tensor(n->ADb[l], H, W, c);
    tensor(n->gCAT[l], H, W, cn + c); tensor(n->gT1[l], H, W, c); tensor(n->gT2[l], H, W, c);
    tensor(n->gT3[l], H, W, c);
    if (l >= 1) {
      tensor(n->Pin[l], H, W, n->ch[l - 1]);
      tensor(n->gP[l], H, W, n->ch[l - 1]);
    }
  }
  const int HL = n->H >> L, WL = n->W >> L, cL = n->ch[L];
  tensor(n->Pin[L], HL, WL, n->ch[L - 1]);
  tensor(n->gP[L], HL, WL, n->ch[L - 1]);
  tensor(n->ZMa, HL, WL, cL); tensor(n->AMa, HL, WL, cL); tensor(n->ZMb, HL, WL, cL); tensor(n->AMb, HL, WL, cL);
  tensor(n->gM1, HL, WL, cL); tensor(n->gM2, HL, WL, cL);
  n->OUT = (float*)take((size_t)N * n->H * n->W * n->cout * 4);
  n->part = (float*)take(kWgradPartFloats * 4);
  n->cpart = (float*)take((size_t)kPartBlocks * 1024 * 4);
  n->lpart = (double*)take(256 * 8);
  n->npart = (double*)take(kPartBlocks * 8);
  n->gscale = (float*)take(256);
  return off;
}

// Layer table and parameter offsets (oracle order; layer 0 input padded to 16).
void net_layers(ssn_net* n) {
  n->L = n->levels - 1;
  n->ch.clear();
  for (int l = 0; l < n->levels; ++l) n->ch.push_back(n->base << l);
  n->conv.clear();
  long off = 0;
  auto add = [&](int Ci_real, int Ci, int Co, int H, int W) {
    ConvL c;
    c.Ci = Ci; c.Ci_real = Ci_real; c.Co = Co; c.H = H; c.W = W;
    c.w_off = off; off += (long)Co * 9 * Ci;
    c.b_off = off; off += Co;
    c.wf = c.wb = nullptr;
    n->conv.push_back(c);
  };
  int cprev = n->cin;
  for (int l = 0; l < n->L; ++l) {
    const int H = n->H >> l, W = n->W >> l;
    add(cprev, l == 0 ? n->cin_pad : cprev, n->ch[l], H, W);
    add(n->ch[l], n->ch[l], n->ch[l], H, W);
    cprev = n->ch[l];
  }
  add(cprev, cprev, n->ch[n->L], n->H >> n->L, n->W >> n->L);
  add(n->ch[n->L], n->ch[n->L], n->ch[n->L], n->H >> n->L, n->W >> n->L);
  cprev = n->ch[n->L];
  for (int l = n->L - 1; l >= 0; --l) {
    const int H = n->H >> l, W = n->W >> l;
    add(cprev + n->ch[l], cprev + n->ch[l], n->ch[l], H, W);
    add(n->ch[l], n->ch[l], n->ch[l], H, W);
    cprev = n->ch[l];
  }
  n->hw_off = off; off += (long)n->cout * n->ch[0];
  n->hb_off = off; off += n->cout;
  n->np = off;
}

int enc_a(int l) { return 2 * l; }
int enc_b(int l) { return 2 * l + 1; }
int mid_a(const ssn_net* n) { return 2 * n->L; }
int mid_b(const ssn_net* n) { return 2 * n->L + 1; }
int dec_a(const ssn_net* n, int l) { return 2 * n->L + 2 + 2 * (n->L - 1 - l); }
int dec_b(const ssn_net* n, int l) { return dec_a(n, l) + 1; }

int grid1(long n) { return (int)std::min<long>((n + 255) / 256, 65535); }

template <int WCO, int WPX, int R>
void launch_rows(const ssn_net* n, const ConvArgs& ca, int Co) {
  const TV& in = ca.in;
  const int tiles = in.N * (in.H / R) * (in.W / (32 * WPX));
  const int gy = (Co + 32 * WCO - 1) / (32 * WCO);
  // two blocks of four waves per CU are resident (registers); each walks its
  // share of the tiles
  const int gx = std::min(tiles, std::max(1, 2048 / (WCO * WPX) / gy));
  const int per = (tiles + gx - 1) / gx;
  const dim3 grid((unsigned)((tiles + per - 1) / per), (unsigned)gy);
  if (ca.mode == 0)
    hipLaunchKernelGGL((conv3x3_rows<WCO, WPX, R, 0>), grid, dim3(64 * WCO * WPX), 0, n->stream, ca, tiles, per);
  else
    hipLaunchKernelGGL((conv3x3_rows<WCO, WPX, R, 1>), grid, dim3(64 * WCO * WPX), 0, n->stream, ca, tiles, per);
}

template <int WCO>
void launch_taps(const ssn_net* n, const ConvArgs& ca, int Co) {
  const TV& in = ca.in;
  const dim3 grid((unsigned)(in.N * in.H * (in.W / 32)), (unsigned)((Co + 32 * WCO - 1) / (32 * WCO)));
  const unsigned lds = (unsigned)tap_lds_bytes(in.C);
  if (ca.mode == 0) hipLaunchKernelGGL((conv3x3_taps<WCO, 0>), grid, dim3(64 * WCO), lds, n->stream, ca);
  else hipLaunchKernelGGL((conv3x3_taps<WCO, 1>), grid, dim3(64 * WCO), lds, n->stream, ca);
}

constexpr long kTapLds = 80 * 1024;  // two blocks per CU

// Launch shapes. The order in which an output's products accumulate is the
// network's, not the launch's: results in BF16 move by whole roundings when it
// changes. It is chunk, tap, channel half where the chunked grid below has 256
// workgroups, and tap, channel elsewhere.
//
// Chunked layers run on conv3x3_rows. Measured on a 4-level network of base 32
// on 256^2 images in batches of 8 (us):
//  - a wave serves as many rows R as leave 512 waves (two per CU), since each
//    weight fragment serves R rows: 64 -> 64 channels on 128^2 takes 26.8 with
//    R = 4 and 32.5 with R = 2 (21.0 with R = 4 and contiguous fragments; 62
//    with the tiles before, which read weights and patch between barriers and
//    stored 2 bytes per lane);
//  - where the output channels are a multiple of 64, two waves share a patch
//    (half the staging registers, which is what lets R = 4 fit 256 VGPRs: with
//    one, 28 are spilled and 96 -> 32 on 256^2 takes 95 instead of 88; 74.6 with
//    R = 2 and contiguous fragments, 96 MB of tensors at 2.2 TB/s);
//  - a block is 32 pixels wide: 64 x 4 rows take 60 instead of 48 on
//    64 -> 192 at 128^2, whose patch three channel blocks read again. With one
//    wave on the channels two pixel waves are better (88 against 93 on 96 -> 32).
// The others run on conv3x3_taps where rows are a multiple of 32 pixels and the
// patch fits, and on direct-operand blocks otherwise (4 waves with 64 pixels per
// wave for large grids, one wave with 32 pixels for small ones).
void launch_conv(const ssn_net* n, const ConvArgs& ca, long P, int Co) {
  const unsigned gy = (unsigned)((Co + 31) / 32);
  const int W = ca.in.W, H = ca.in.H;
  const int wpx = W >= 128 ? 4 : W >= 64 ? 2 : 1;
  const int wco = Co % 64 == 0 ? 2 : 1;
  const long chunk_blocks =
      (long)ca.in.N * (H / (wpx == 4 ? 2 : 4)) * (W / (32 * wpx)) * ((Co + 32 * wco - 1) / (32 * wco));
  const bool chunk_ok = W >= 32 && W % (32 * wpx) == 0;
  const long waves1 = P / 32 * gy;  // at one row per wave
  if (chunk_ok && (n->conv_shape == 3 || (n->conv_shape == 0 && chunk_blocks >= 256))) {
    if (wco == 2 && waves1 >= 4 * 512) launch_rows<2, 1, 4>(n, ca, Co);
    else if (wco == 2 && waves1 >= 2 * 512) launch_rows<2, 1, 2>(n, ca, Co);
    else if (waves1 < 2 * 512) launch_rows<1, 1, 1>(n, ca, Co);
    else if (wpx >= 2) launch_rows<1, 2, 2>(n, ca, Co);
    else launch_rows<1, 1, 2>(n, ca, Co);
    return;
  }
  if (n->conv_shape == 0 && W % 32 == 0 && tap_lds_bytes(ca.in.C) <= kTapLds) {
    // waves that share a patch: 4 / 2 / 1 on 256 -> 256 channels (32^2, one image) 15 / 16 / 20 us
    if (gy % 4 == 0) launch_taps<4>(n, ca, Co);
    else if (gy % 2 == 0) launch_taps<2>(n, ca, Co);
    else launch_taps<1>(n, ca, Co);
    return;
  }
  const bool large = n->conv_shape == 1 || (n->conv_shape != 2 && (P + 255) / 256 * gy >= 1024);
  if (large) {
    const dim3 grid((unsigned)((P + 255) / 256), gy);
    if (ca.mode == 0) hipLaunchKernelGGL((conv3x3_mfma<2, 4, 0>), grid, dim3(256), 0, n->stream, ca);
    else hipLaunchKernelGGL((conv3x3_mfma<2, 4, 1>), grid, dim3(256), 0, n->stream, ca);
  } else {
    const dim3 grid((unsigned)((P + 31) / 32), gy);
    if (ca.mode == 0) hipLaunchKernelGGL((conv3x3_mfma<1, 1, 0>), grid, dim3(64), 0, n->stream, ca);
    else hipLaunchKernelGGL((conv3x3_mfma<1, 1, 1>), grid, dim3(64), 0, n->stream, ca);
  }
}

void launch_conv_fwd(const ssn_net* n, const ConvL& c, TV in, TV z, TV a) {
  ConvArgs ca;
  ca.in = in;
  ca.w = c.wf;
  ca.bias = n->P + c.b_off;
  ca.Co = c.Co;
  ca.out_z = z;
  ca.out = a;
  ca.zprev.p = nullptr;
  ca.mode = 0;
  launch_conv(n, ca, (long)in.N * in.H * in.W, c.Co);
}

// gradient w.r.t. the layer input: out = conv(gz, wb) [* SiLU'(zprev)]
void launch_conv_bwd_data(const ssn_net* n, const ConvL& c, TV gz, TV out, const TV* zprev) {
  ConvArgs ca;
  ca.in = gz;
  ca.w = c.wb;
  ca.bias = nullptr;
  ca.Co = c.Ci;
  ca.out_z.p = nullptr;
  ca.out = out;
  if (zprev) ca.zprev = *zprev;
  else ca.zprev.p = nullptr;
  ca.mode = 1;
  launch_conv(n, ca, (long)gz.N * gz.H * gz.W, c.Ci);
}

// Sums of a layer's weight and bias partials (launch of reduce_splits).
void launch_reduce_splits(const ssn_net* n, const ReduceSet& w, const ReduceSet& b) {
  const int wb = (int)((w.n + 31) / 32), bb = (int)((b.n + 31) / 32);
  hipLaunchKernelGGL(reduce_splits, dim3((unsigned)(wb + bb)), dim3(256), 0, n->stream, w, b, wb);
}

// Chunk geometry of the weight gradient for a W x H level: cw is the widest
// multiple of 16 up to 64 that divides W; R the largest power of two with
// R * cw <= kChunk and H % R == 0 (the x pixels then fit kXPix).
void wgrad_chunk(int W, int H, int& cw, int& R) {
  cw = 16;
  for (int c = 64; c >= 16; c -= 16)
    if (W % c == 0) {
      cw = c;
      break;
    }
  R = 1;
  while (2 * R * cw <= kChunk && H % (2 * R) == 0) R *= 2;
}

void launch_wgrad(ssn_net* n, const ConvL& c, TV gz, TV x) {
  int cw = 16, R = 1;
  wgrad_chunk(x.W, x.H, cw, R);
  const long nchunks = (long)x.N * (x.H / R) * (x.W / cw);
  const int tci = (c.Ci + 31) / 32, tco = (c.Co + 31) / 32;
  // about 1.5 workgroups per CU (measured: 256 and 768 were 1-3% slower overall)
  int nsplit = (int)std::max<long>(1, std::min<long>(nchunks, 384 / (tci * tco)));
  while ((long)nsplit * c.Co * 9 * c.Ci > kWgradPartFloats) nsplit /= 2;
  WgradArgs wa;
  wa.gz = gz;
  wa.x = x;
  wa.part = n->part;
  wa.nsplit = nsplit;
  wa.R = R;
  wa.cpart = n->cpart;
  const dim3 grid((unsigned)(tci * tco * nsplit + kPartBlocks * ((c.Co + 255) / 256)));
  if (cw == 64) hipLaunchKernelGGL((conv3x3_wgrad<64>), grid, dim3(256), 0, n->stream, wa);
  else if (cw == 48) hipLaunchKernelGGL((conv3x3_wgrad<48>), grid, dim3(256), 0, n->stream, wa);
  else if (cw == 32) hipLaunchKernelGGL((conv3x3_wgrad<32>), grid, dim3(256), 0, n->stream, wa);
  else hipLaunchKernelGGL((conv3x3_wgrad<16>), grid, dim3(256), 0, n->stream, wa);
  launch_reduce_splits(n, {n->part, n->G + c.w_off, (long)c.Co * 9 * c.Ci, nsplit},
                       {n->cpart, n->G + c.b_off, (long)c.Co, kPartBlocks});
}

// The weight fragments of every layer, after an Adam step if there is one.
void launch_params(ssn_net* n, const AdamArgs* adam) {
  ParamLayers ls;
  std::memset(&ls, 0, sizeof(ls));
  const int nl = (int)n->conv.size();
  for (int k = 0; k < nl; ++k) {
    const ConvL& c = n->conv[k];
    ls.l[k] = {c.w_off, (long)c.Co * 9 * c.Ci + c.Co, c.Co, c.Ci, c.wf, c.wb};
  }
  ls.l[nl] = {n->hw_off, n->np - n->hw_off, 0, 0, nullptr, nullptr};
  const dim3 grid(256, (unsigned)(nl + 1));
  if (adam) hipLaunchKernelGGL((update_params<true>), grid, dim3(256), 0, n->stream, ls, n->P, *adam);
  else hipLaunchKernelGGL((update_params<false>), grid, dim3(256), 0, n->stream, ls, n->P, AdamArgs());
}

__global__ void copy_f32(const float* __restrict__ src, float* __restrict__ dst, long n) {
  for (long k = blockIdx.x * (long)blockDim.x + threadIdx.x; k < n; k += (long)gridDim.x * blockDim.x) dst[k] = src[k];
}

// fp32 images to BF16, the channels padded with zeros to 16: one pixel per thread
__global__ void __launch_bounds__(256) input_to_bf16(const float* __restrict__ x, int cin, long npix, TV X) {
  const long p = blockIdx.x * 256L + threadIdx.x;
  if (p >= npix) return;
  float v[2][8];
#pragma unroll
  for (int c = 0; c < 16; ++c) v[c >> 3][c & 7] = c < cin ? x[p * cin + c] : 0.0f;
  store_u32x4(X.p + p * X.cs + X.coff, pack8(v[0]));
  store_u32x4(X.p + p * X.cs + X.coff + 8, pack8(v[1]));
}

// grid of a for_vectors kernel over view t
dim3 vector_grid(const TV& t) {
  return dim3((unsigned)((t.W * (t.C / 8) + 255) / 256), (unsigned)std::min(t.H, 65535), (unsigned)std::min(t.N, 65535));
}

template <int COUT>
void launch_head_bwd_data(const ssn_net* n, const float* target, float inv, TV z, TV g, long npix) {
  const int per = 256 / (g.C / 8);
  hipLaunchKernelGGL((head_bwd_data<COUT>), dim3((unsigned)((npix + per - 1) / per)), dim3(256), 0, n->stream, n->OUT,
                     target, inv, n->P + n->hw_off, z, g, npix);
}

int net_forward(ssn_net* n, const float* x, int nb) {
  const int L = n->L;
  const long npix = (long)nb * n->H * n->W;
  hipLaunchKernelGGL(input_to_bf16, dim3((unsigned)((npix + 255) / 256)), dim3(256), 0, n->stream, x, n->cin, npix,
                     n->X0.all(nb));
  for (int l = 0; l < L; ++l) {
    const int c = n->ch[l], cn = n->ch[l + 1];
    TV in = l == 0 ? n->X0.all(nb) : n->Pin[l].all(nb);
    launch_conv_fwd(n, n->conv[enc_a(l)], in, n->ZA[l].all(nb), n->AA[l].all(nb));
    TV skip = n->CAT[l].view(nb, cn, c);
    launch_conv_fwd(n, n->conv[enc_b(l)], n->AA[l].all(nb), n->ZB[l].all(nb), skip);
    TV pooled = n->Pin[l + 1].all(nb);
    hipLaunchKernelGGL(avgpool2_fwd, vector_grid(pooled), dim3(256), 0, n->stream, skip, pooled);
  }
  launch_conv_fwd(n, n->conv[mid_a(n)], n->Pin[L].all(nb), n->ZMa.all(nb), n->AMa.all(nb));
  launch_conv_fwd(n, n->conv[mid_b(n)], n->AMa.all(nb), n->ZMb.all(nb), n->AMb.all(nb));
  for (int l = L - 1; l >= 0; --l) {
    const int cn = n->ch[l + 1];
    TV prev = l == L - 1 ? n->AMb.all(nb) : n->ADb[l + 1].all(nb);
    TV up = n->CAT[l].view(nb, 0, cn);
    hipLaunchKernelGGL(upsample2_fwd, vector_grid(prev), dim3(256), 0, n->stream, prev, up);
    launch_conv_fwd(n, n->conv[dec_a(n, l)], n->CAT[l].all(nb), n->ZDa[l].all(nb), n->ADa[l].all(nb));
    launch_conv_fwd(n, n->conv[dec_b(n, l)], n->ADa[l].all(nb), n->ZDb[l].all(nb), n->ADb[l].all(nb));
  }
  hipLaunchKernelGGL(head_fwd, dim3((unsigned)((npix + 255) / 256)), dim3(256), 0, n->stream, n->ADb[0].all(nb),
                     n->P + n->hw_off, n->P + n->hb_off, n->cout, n->OUT, npix);
  SN_HIP(hipGetLastError());
  return SS_OK;
}

int net_backward(ssn_net* n, const float* target, int nb, double* loss) {
  const int L = n->L;
  const long npix = (long)nb * n->H * n->W;
  const long nout = npix * n->cout;
  const float inv = 2.0f / (float)nout;
  // head
  hipLaunchKernelGGL(head_sums, dim3(kPartBlocks), dim3(256), 0, n->stream, n->OUT, target, inv, n->ADb[0].all(nb),
                     n->cout, npix, n->part, n->cpart, n->lpart);
  launch_reduce_splits(n, {n->part, n->G + n->hw_off, (long)n->cout * n->ch[0], kPartBlocks},
                       {n->cpart, n->G + n->hb_off, (long)n->cout, kPartBlocks});
  {
    TV z = n->ZDb[0].all(nb), g = n->gT1[0].all(nb);
    switch (n->cout) {
      case 1: launch_head_bwd_data<1>(n, target, inv, z, g, npix); break;
      case 2: launch_head_bwd_data<2>(n, target, inv, z, g, npix); break;
      case 3: launch_head_bwd_data<3>(n, target, inv, z, g, npix); break;
      case 4: launch_head_bwd_data<4>(n, target, inv, z, g, npix); break;
      case 5: launch_head_bwd_data<5>(n, target, inv, z, g, npix); break;
      case 6: launch_head_bwd_data<6>(n, target, inv, z, g, npix); break;
      case 7: launch_head_bwd_data<7>(n, target, inv, z, g, npix); break;
      default: launch_head_bwd_data<8>(n, target, inv, z, g, npix); break;
    }
  }
  // decoder, top level first
  for (int l = 0; l < L; ++l) {
    const int cn = n->ch[l + 1];
    const ConvL& cb = n->conv[dec_b(n, l)];
    const ConvL& ca = n->conv[dec_a(n, l)];
    launch_wgrad(n, cb, n->gT1[l].all(nb), n->ADa[l].all(nb));
    TV za = n->ZDa[l].all(nb);
    launch_conv_bwd_data(n, cb, n->gT1[l].all(nb), n->gT3[l].all(nb), &za);
    launch_wgrad(n, ca, n->gT3[l].all(nb), n->CAT[l].all(nb));
    launch_conv_bwd_data(n, ca, n->gT3[l].all(nb), n->gCAT[l].all(nb), nullptr);
    // the upsampled half of the concatenation feeds back to the level below
    TV gup = n->gCAT[l].view(nb, 0, cn);
    TV dst = l == L - 1 ? n->gM2.all(nb) : n->gT1[l + 1].all(nb);
    TV zsrc = l == L - 1 ? n->ZMb.all(nb) : n->ZDb[l + 1].all(nb);
    hipLaunchKernelGGL(upsample2_bwd, vector_grid(dst), dim3(256), 0, n->stream, gup, dst, zsrc);
  }
  // bottleneck
  {
    const ConvL& cb = n->conv[mid_b(n)];
    const ConvL& ca = n->conv[mid_a(n)];
    launch_wgrad(n, cb, n->gM2.all(nb), n->AMa.all(nb));
    TV za = n->ZMa.all(nb);
    launch_conv_bwd_data(n, cb, n->gM2.all(nb), n->gM1.all(nb), &za);
    launch_wgrad(n, ca, n->gM1.all(nb), n->Pin[L].all(nb));
    launch_conv_bwd_data(n, ca, n->gM1.all(nb), n->gP[L].all(nb), nullptr);
  }
  // encoder, bottom level first
  for (int l = L - 1; l >= 0; --l) {
    const int c = n->ch[l], cn = n->ch[l + 1];
    TV gS = n->gCAT[l].view(nb, cn, c);
    hipLaunchKernelGGL(avgpool2_bwd, vector_grid(gS), dim3(256), 0, n->stream, n->gP[l + 1].all(nb), gS, n->ZB[l].all(nb));
    const ConvL& cb = n->conv[enc_b(l)];
    const ConvL& ca = n->conv[enc_a(l)];
    launch_wgrad(n, cb, gS, n->AA[l].all(nb));
    TV za = n->ZA[l].all(nb);
    launch_conv_bwd_data(n, cb, gS, n->gT2[l].all(nb), &za);
    TV in = l == 0 ? n->X0.all(nb) : n->Pin[l].all(nb);
    launch_wgrad(n, ca, n->gT2[l].all(nb), in);
    if (l > 0) launch_conv_bwd_data(n, ca, n->gT2[l].all(nb), n->gP[l].all(nb), nullptr);
  }
  SN_HIP(hipGetLastError());
  if (loss) {
    double parts[256];
    SN_HIP(hipMemcpyAsync(parts, n->lpart, sizeof(parts), hipMemcpyDeviceToHost, n->stream));
    SN_HIP(hipStreamSynchronize(n->stream));
    double s = 0.0;
    for (int k = 0; k < 256; ++k) s += parts[k];
    *loss = s / (double)nout;
  }
  return SS_OK;
}

// oracle-order flat index <-> padded layout, for one parameter block
template <class F>
void for_each_param(const ssn_net* n, F&& f) {
  long o = 0;  // oracle offset
  for (const ConvL& c : n->conv) {
    for (int co = 0; co < c.Co; ++co)
      for (int t = 0; t < 9; ++t)
        for (int ci = 0; ci < c.Ci_real; ++ci) f(o++, c.w_off + ((long)co * 9 + t) * c.Ci + ci);
    for (int co = 0; co < c.Co; ++co) f(o++, c.b_off + co);
  }
  for (int k = 0; k < n->cout * n->ch[0]; ++k) f(o++, n->hw_off + k);
  for (int k = 0; k < n->cout; ++k) f(o++, n->hb_off + k);
}

long oracle_count(const ssn_net* n) {
  long c = 0;
  for_each_param(n, [&](long, long) { ++c; });
  return c;
}

int check_shape(int levels, int base, int cin, int cout, int N, int H, int W) {
  if (levels < 2 || levels > 6) return nfail(SS_EINVAL, "levels must lie in [2, 6]");
  if (base < 16 || base % 16 || (base << (levels - 1)) > 1024) return nfail(SS_EINVAL, "base must be a multiple of 16");
  if (cin < 1 || cin > 16) return nfail(SS_EINVAL, "cin must lie in [1, 16]");
  if (cout < 1 || cout > 8 || cout * base > 256) return nfail(SS_EINVAL, "cout must lie in [1, 8] with cout*base <= 256");
  const int m = 16 << (levels - 1);
  if (N < 1 || H < m || W < m || H % m || W % m)
    return nfail(SS_ESHAPE, "H and W must be multiples of 16 * 2^(levels-1)");
  return SS_OK;
}

}  // namespace

namespace ss_detail {
int ctx_shape(const ss_ctx* c, int* Nx, int* Ny, int* theory);
}

extern "C" {

long ssn_param_count(int levels, int base, int cin, int cout) {
  ssn_net n;
  n.levels = levels; n.base = base; n.cin = cin; n.cout = cout; n.cin_pad = 16;
  n.H = n.W = 16 << (levels - 1);
  net_layers(&n);
  return oracle_count(&n);
}

int ssn_workspace_bytes(int levels, int base, int cin, int cout, int N, int H, int W, size_t* bytes) {
  int rc = check_shape(levels, base, cin, cout, N, H, W);
  if (rc) return rc;
  if (!bytes) return nfail(SS_EINVAL, "bytes is NULL");
  ssn_net n;
  n.levels = levels; n.base = base; n.cin = cin; n.cout = cout; n.cin_pad = 16;
  n.Ncap = N; n.H = H; n.W = W;
  net_layers(&n);
  *bytes = net_carve(&n, nullptr);
  return SS_OK;
}

int ssn_create(int levels, int base, int cin, int cout, int N, int H, int W, void* ws, size_t ws_bytes, void* stream,
               ssn_net** out) {
  if (!out) return nfail(SS_EINVAL, "out is NULL");
  *out = nullptr;
  size_t need = 0;
  int rc = ssn_workspace_bytes(levels, base, cin, cout, N, H, W, &need);
  if (rc) return rc;
  if (!ws || ws_bytes < need || ((uintptr_t)ws) % 256) return nfail(SS_EINVAL, "workspace missing, small or misaligned");
  ssn_net* n = new (std::nothrow) ssn_net();
  if (!n) return nfail(SS_EINVAL, "out of host memory");
  n->levels = levels; n->base = base; n->cin = cin; n->cout = cout; n->cin_pad = 16;
  n->Ncap = N; n->H = H; n->W = W;
  n->stream = (hipStream_t)stream;
  n->adam_t = 0;
  n->conv_shape = 0;
  if (const char* env = std::getenv("SSN_CONV_SHAPE")) {
    const int v = std::atoi(env);
    if (v >= 0 && v <= 3) n->conv_shape = v;
  }
  net_layers(n);
  n->bytes = net_carve(n, (char*)ws);
  hipError_t e = hipMemsetAsync(ws, 0, n->bytes, n->stream);
  if (e != hipSuccess) {
    delete n;
    return nfail(SS_EHIP, std::string("hipMemsetAsync: ") + hipGetErrorString(e));
  }
  *out = n;
  return SS_OK;
}

void ssn_destroy(ssn_net* n) {
  if (!n) return;
  if (n->fgraph) (void)hipGraphExecDestroy(n->fgraph);
  if (n->fcap) (void)hipStreamDestroy(n->fcap);
  delete n;
}

long ssn_num_params(ssn_net* n) { return n ? oracle_count(n) : SS_EINVAL; }

int ssn_set_weights(ssn_net* n, const float* host, long count) {
  if (!n || !host || count != oracle_count(n)) return nfail(SS_EINVAL, "weights: wrong count");
  std::vector<float> flat(n->np, 0.0f);
  for_each_param(n, [&](long o, long d) { flat[d] = host[o]; });
  SN_HIP(hipMemcpyAsync(n->P, flat.data(), n->np * 4, hipMemcpyHostToDevice, n->stream));
  SN_HIP(hipMemsetAsync(n->M, 0, n->np * 4, n->stream));
  SN_HIP(hipMemsetAsync(n->V, 0, n->np * 4, n->stream));
  n->adam_t = 0;
  launch_params(n, nullptr);
  SN_HIP(hipGetLastError());
  SN_HIP(hipStreamSynchronize(n->stream));
  return SS_OK;
}

static int copy_out(ssn_net* n, const float* dev, float* host, long count) {
  if (!n || !host || count != oracle_count(n)) return nfail(SS_EINVAL, "wrong count");
  std::vector<float> flat(n->np);
  SN_HIP(hipMemcpyAsync(flat.data(), dev, n->np * 4, hipMemcpyDeviceToHost, n->stream));
  SN_HIP(hipStreamSynchronize(n->stream));
  for_each_param(n, [&](long o, long d) { host[o] = flat[d]; });
  return SS_OK;
}

int ssn_get_weights(ssn_net* n, float* host, long count) { return copy_out(n, n ? n->P : nullptr, host, count); }
int ssn_get_grads(ssn_net* n, float* host, long count) { return copy_out(n, n ? n->G : nullptr, host, count); }

}  // extern "C"

namespace {

// The BF16 tensor of kind `kind` of 3x3 layer k (layer order of the parameter
// exchange), as the last forward and backward passes left it.
bool layer_tensor(const ssn_net* n, int kind, int k, int nb, TV* out) {
  const int L = n->L;
  const int nconv = (int)n->conv.size();
  if (k < 0 || k >= nconv) return false;
  // locate the layer: encoder level l (a/b), bottleneck, or decoder level l (a/b)
  int l = -1, part = 0;  // part: 0 enc, 1 mid, 2 dec
  bool second = (k & 1) != 0;
  if (k < 2 * L) { l = k / 2; part = 0; }
  else if (k < 2 * L + 2) { part = 1; }
  else { l = L - 1 - (k - 2 * L - 2) / 2; part = 2; }
  const int c = l >= 0 ? n->ch[l] : n->ch[L], cn = l >= 0 ? n->ch[l + 1] : 0;
  TV t;
  t.p = nullptr;
  switch (kind) {
    case SSN_T_INPUT:
      if (part == 0) t = second ? n->AA[l].all(nb) : (l == 0 ? n->X0.all(nb) : n->Pin[l].all(nb));
      else if (part == 1) t = second ? n->AMa.all(nb) : n->Pin[L].all(nb);
      else t = second ? n->ADa[l].all(nb) : n->CAT[l].all(nb);
      break;
    case SSN_T_PREACT:
      if (part == 0) t = second ? n->ZB[l].all(nb) : n->ZA[l].all(nb);
      else if (part == 1) t = second ? n->ZMb.all(nb) : n->ZMa.all(nb);
      else t = second ? n->ZDb[l].all(nb) : n->ZDa[l].all(nb);
      break;
    case SSN_T_OUTPUT:
      if (part == 0) t = second ? n->CAT[l].view(nb, cn, c) : n->AA[l].all(nb);
      else if (part == 1) t = second ? n->AMb.all(nb) : n->AMa.all(nb);
      else t = second ? n->ADb[l].all(nb) : n->ADa[l].all(nb);
      break;
    case SSN_T_GRAD_PREACT:
      if (part == 0) t = second ? n->gCAT[l].view(nb, cn, c) : n->gT2[l].all(nb);
      else if (part == 1) t = second ? n->gM2.all(nb) : n->gM1.all(nb);
      else t = second ? n->gT1[l].all(nb) : n->gT3[l].all(nb);
      break;
    case SSN_T_GRAD_DATA:
      if (part == 0) {
        if (second) t = n->gT2[l].all(nb);
        else if (l > 0) t = n->gP[l].all(nb);
        else return false;  // the first layer's input gradient is not formed
      } else if (part == 1) {
        t = second ? n->gM1.all(nb) : n->gP[L].all(nb);
      } else {
        t = second ? n->gT3[l].all(nb) : n->gCAT[l].all(nb);
      }
      break;
    default:
      return false;
  }
  *out = t;
  return t.p != nullptr;
}

}  // namespace

extern "C" {

int ssn_tensor_shape(ssn_net* n, int kind, int layer, int* H, int* W, int* C) {
  if (!n || !H || !W || !C) return nfail(SS_EINVAL, "NULL argument");
  TV t;
  if (!layer_tensor(n, kind, layer, 1, &t)) return nfail(SS_EINVAL, "no such tensor");
  *H = t.H;
  *W = t.W;
  *C = t.C;
  return SS_OK;
}

int ssn_read_tensor(ssn_net* n, int kind, int layer, int nb, float* host, long count) {
  if (!n || !host) return nfail(SS_EINVAL, "NULL argument");
  if (nb < 1 || nb > n->Ncap) return nfail(SS_EINVAL, "image count out of range");
  TV t;
  if (!layer_tensor(n, kind, layer, nb, &t)) return nfail(SS_EINVAL, "no such tensor");
  const long npix = (long)nb * t.H * t.W;
  if (count != npix * t.C) return nfail(SS_EINVAL, "count must be n * H * W * C of the tensor");
  std::vector<bf16_t> raw((size_t)npix * t.cs);
  SN_HIP(hipMemcpyAsync(raw.data(), t.p, raw.size() * sizeof(bf16_t), hipMemcpyDeviceToHost, n->stream));
  SN_HIP(hipStreamSynchronize(n->stream));
  for (long p = 0; p < npix; ++p)
    for (int ch = 0; ch < t.C; ++ch) {
      const unsigned u = ((unsigned)raw[(size_t)p * t.cs + t.coff + ch]) << 16;
      float f;
      std::memcpy(&f, &u, 4);
      host[p * t.C + ch] = f;
    }
  return SS_OK;
}

int ssn_forward(ssn_net* n, const float* x, int nb, float* out) {
  if (!n || !x || nb < 1 || nb > n->Ncap) return nfail(SS_EINVAL, "bad forward arguments");
  int rc = net_forward(n, x, nb);
  if (rc) return rc;
  if (out)
    SN_HIP(hipMemcpyAsync(out, n->OUT, (size_t)nb * n->H * n->W * n->cout * 4, hipMemcpyDeviceToDevice, n->stream));
  return SS_OK;
}

int ssn_forward_graph(ssn_net* n, const float* x, int nb, float* out) {
  if (!n || !x || !out || nb < 1 || nb > n->Ncap) return nfail(SS_EINVAL, "bad forward arguments");
  if (!n->fgraph || n->fx != x || n->fout != out || n->fnb != nb) {
    if (n->fgraph) {
      (void)hipGraphExecDestroy(n->fgraph);
      n->fgraph = nullptr;
    }
    if (!n->fcap) SN_HIP(hipStreamCreateWithFlags(&n->fcap, hipStreamNonBlocking));
    hipStream_t s0 = n->stream;
    n->stream = n->fcap;  // the forward's launches go to the capture stream
    hipError_t e = hipStreamBeginCapture(n->fcap, hipStreamCaptureModeRelaxed);
    int rc = e == hipSuccess ? net_forward(n, x, nb) : SS_EHIP;
    if (rc == SS_OK) {
      hipLaunchKernelGGL(copy_f32, dim3(grid1((long)nb * n->H * n->W * n->cout)), dim3(256), 0, n->fcap, n->OUT, out,
                         (long)nb * n->H * n->W * n->cout);
    }
    hipGraph_t g = nullptr;
    const hipError_t e2 = hipStreamEndCapture(n->fcap, &g);
    n->stream = s0;
    if (e != hipSuccess || e2 != hipSuccess || rc != SS_OK)
      return nfail(SS_EHIP, std::string("forward capture: ") + hipGetErrorString(e != hipSuccess ? e : e2));
    e = hipGraphInstantiate(&n->fgraph, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (e != hipSuccess) {
      n->fgraph = nullptr;
      return nfail(SS_EHIP, std::string("hipGraphInstantiate: ") + hipGetErrorString(e));
    }
    n->fx = x;
    n->fout = out;
    n->fnb = nb;
  }
  SN_HIP(hipGraphLaunch(n->fgraph, n->stream));
  return SS_OK;
}

int ssn_backward(ssn_net* n, const float* target, int nb, double* loss) {
  if (!n || !target || nb < 1 || nb > n->Ncap) return nfail(SS_EINVAL, "bad backward arguments");
  return net_backward(n, target, nb, loss);
}

int ssn_adam_step(ssn_net* n, float lr) {
  if (!n || !(lr > 0.0f)) return nfail(SS_EINVAL, "bad Adam arguments");
  n->adam_t += 1;
  const float b1 = 0.9f, b2 = 0.999f;
  const float c1 = 1.0f - std::pow(b1, (float)n->adam_t), c2 = 1.0f - std::pow(b2, (float)n->adam_t);
  const float* gs = nullptr;
  if (n->clip > 0.0f) {
    hipLaunchKernelGGL(grad_sq_partials, dim3(kPartBlocks), dim3(256), 0, n->stream, n->G, n->np, n->npart);
    hipLaunchKernelGGL(grad_clip_scale, dim3(1), dim3(256), 0, n->stream, n->npart, kPartBlocks, n->clip, n->gscale);
    gs = n->gscale;
  }
  const AdamArgs adam = {n->M, n->V, n->G, gs, lr, b1, b2, 1e-8f, c1, c2};
  launch_params(n, &adam);
  SN_HIP(hipGetLastError());
  return SS_OK;
}

int ssn_set_grad_clip(ssn_net* n, float max_norm) {
  if (!n || !(max_norm >= 0.0f) || !std::isfinite(max_norm)) return nfail(SS_EINVAL, "bad clipping norm");
  n->clip = max_norm;
  return SS_OK;
}

int ssn_train_step(ssn_net* n, const float* x, const float* target, int nb, float lr, double* loss) {
  int rc = ssn_forward(n, x, nb, nullptr);
  if (rc) return rc;
  rc = ssn_backward(n, target, nb, loss);
  if (rc) return rc;
  return ssn_adam_step(n, lr);
}

// Forward and backward multiply-add flops of one sample (2 flops per MAC),
// counting the 3x3 and 1x1 convolutions at their real channel counts.
size_t ssn_init_field_workspace_bytes(ssn_net* n) { return n ? (size_t)n->H * n->W * 2 * sizeof(float) : 0; }

int ssn_init_field(ssn_net* n, ss_ctx* ctx, int nv, const double* xy, const double* w, double kappa, double sigma,
                   double pin, uint64_t seed, double noise_amp, void* work, size_t work_bytes) {
  if (!n || !ctx || !work) return nfail(SS_EINVAL, "net, ctx or work is NULL");
  if (n->cin != 2 || n->cout != 4) return nfail(SS_EINVAL, "the learned start needs a network with 2 inputs and 4 outputs");
  int Nx = 0, Ny = 0, theory = -1;
  if (ss_detail::ctx_shape(ctx, &Nx, &Ny, &theory) != SS_OK) return nfail(SS_EINVAL, "ctx is NULL");
  if (theory != SS_THEORY_AH) return nfail(SS_EINVAL, "the learned start exists for the Abelian Higgs model only");
  if (Nx != n->W || Ny != n->H) return nfail(SS_ESHAPE, "the network's image size differs from the lattice");
  if (work_bytes < ssn_init_field_workspace_bytes(n)) return nfail(SS_EINVAL, "work is too small");
  if ((uintptr_t)work % 256) return nfail(SS_EINVAL, "work must be 256-byte aligned");
  // input image on the context's stream (the call synchronises it)
  int rc = ss_learned_input(ctx, nv, xy, kappa, (float*)work);
  if (rc) return nfail(rc, std::string("input image: ") + ss_last_error());
  rc = ssn_forward(n, (const float*)work, 1, nullptr);
  if (rc) return rc;
  // the corrections are read from the network's own output buffer on the
  // context's stream, so the forward pass must have finished
  SN_HIP(hipStreamSynchronize(n->stream));
  rc = ss_init_learned(ctx, nv, xy, w, n->OUT, sigma, pin, seed, noise_amp);  // synchronises the context's stream
  if (rc) return nfail(rc, std::string("corrected ansatz: ") + ss_last_error());
  return SS_OK;
}

int ssn_flops(ssn_net* n, double* fwd, double* bwd) {
  if (!n) return nfail(SS_EINVAL, "net is NULL");
  double f = 0.0, b = 0.0;
  for (size_t k = 0; k < n->conv.size(); ++k) {
    const ConvL& c = n->conv[k];
    const double mac = (double)c.H * c.W * 9.0 * c.Co * c.Ci_real;
    f += 2.0 * mac;
    b += (k == 0 ? 2.0 : 4.0) * mac;  // weight gradient (+ input gradient except for the first layer)
  }
  const double head = (double)n->H * n->W * n->cout * n->ch[0];
  f += 2.0 * head;
  b += 4.0 * head;
  if (fwd) *fwd = f;
  if (bwd) *bwd = b;
  return SS_OK;
}

const char* ssn_last_error(void) { return g_ssn_err.c_str(); }

}  // extern "C"
