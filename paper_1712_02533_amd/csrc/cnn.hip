// Learned warm start: a 6-layer convolutional encoder-decoder (BF16 weights and activations,
// FP32 accumulation) that maps a pair of level-7 frames (2 x 128 x 128, normalised) to the
// level-7 displacement (2 x 128 x 128, in level-7 cells). Trained on this GPU by the kernels in
// this file (forward, backward, Adam) on pairs registered by the plain method.
//
// Network (3x3 convolutions, padding 1; ReLU after every layer but the last):
//   L1 2->64 stride 2 (64^2)   L2 64->128 stride 2 (32^2)   L3 128->256 stride 2 (16^2)
//   L4 [up2(L3), L2] 384->128 (32^2)   L5 [up2(L4), L1] 192->64 (64^2)
//   L6 [up2(L5), input] 66->2 (128^2, linear)
// Activations are NHWC. Weights are [Cout][Kp] with k = (dy * 3 + dx) * Cin + ci, Kp = 9 Cin
// rounded up to 32 (L1 to 64), padded with zeros. L2-L5 run as fused implicit-GEMM
// convolutions on MFMAs (v_mfma_f32_16x16x32_bf16); L1 (2 input channels) and L6 (2 output
// channels, its upsampled input folded into the weights) as direct FP32 kernels. The weight
// gradients of L2-L5 are contracted over pixels by k_wgrad; L1's goes through im2col and a GEMM.
#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>
#include <ctype.h>
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <string>
#include <vector>

#include "../../include/pprs.h"

typedef __bf16 bf16;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

namespace {

const int kBlock = 256;

int grid1d(long long work, int cap = 16384) {
  long long g = (work + kBlock - 1) / kBlock;
  return (int)(g < 1 ? 1 : (g > cap ? cap : g));
}

// ------------------------------------------------------------------------------------------
// GEMM: C[m][n] = sum_k A(m,k) B(n,k), bf16 operands, fp32 result.
// A(m,k) = A[k * lda + m]; B(n,k) = B[k * ldb + n].
// 64 x 64 tiles, 32-deep K steps, 4 wavefronts each owning a 32 x 32 quarter (2 x 2 MFMA).
// Requires M % 64 == 0, N % 64 == 0, (K range of a split) % 32 == 0, lda, ldb % 8 == 0.
// blockIdx.z selects a K split; split s writes C + s * split_stride.

__global__ void __launch_bounds__(256) k_gemm(const bf16* __restrict__ A, int lda,
                                              const bf16* __restrict__ B, int ldb,
                                              float* __restrict__ C, int ldc, int K,
                                              int k_per_split, long long split_stride) {
  constexpr int PADK = 40;  // LDS row of 32 k plus 8 (keeps 16-byte alignment)
  __shared__ __attribute__((aligned(16))) bf16 sA[64 * PADK];
  __shared__ __attribute__((aligned(16))) bf16 sB[64 * PADK];
  int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  int n0 = blockIdx.x * 64, m0 = blockIdx.y * 64;
  int kb = blockIdx.z * k_per_split, ke = min(K, kb + k_per_split);
  int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  f32x4 acc[2][2];
  for (int i = 0; i < 2; ++i)
    for (int j = 0; j < 2; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
  for (int k0 = kb; k0 < ke; k0 += 32) {
    {
      int kk = tid >> 3, mm = (tid & 7) * 8;
      uint4 v = *(const uint4*)&A[(size_t)(k0 + kk) * lda + m0 + mm];
      const bf16* e = (const bf16*)&v;
#pragma unroll
      for (int i = 0; i < 8; ++i) sA[(mm + i) * PADK + kk] = e[i];
    }
    {
      int kk = tid >> 3, nn = (tid & 7) * 8;
      uint4 v = *(const uint4*)&B[(size_t)(k0 + kk) * ldb + n0 + nn];
      const bf16* e = (const bf16*)&v;
#pragma unroll
      for (int i = 0; i < 8; ++i) sB[(nn + i) * PADK + kk] = e[i];
    }
    __syncthreads();
    bf16x8 a[2], b[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      a[i] = *(const bf16x8*)&sA[(wm + i * 16 + (lane & 15)) * PADK + 8 * (lane >> 4)];
      b[i] = *(const bf16x8*)&sB[(wn + i * 16 + (lane & 15)) * PADK + 8 * (lane >> 4)];
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    __syncthreads();
  }
  float* Co = C + (size_t)blockIdx.z * split_stride;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        int row = m0 + wm + i * 16 + 4 * (lane >> 4) + r;
        int col = n0 + wn + j * 16 + (lane & 15);
        Co[(size_t)row * ldc + col] = acc[i][j][r];
      }
}

// ------------------------------------------------------------------------------------------
// A float from the lane a DPP control names (all lanes have a source).
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}

// Fused 3x3 convolution (implicit GEMM) for layers whose input channels come in multiples of
// 64: out[m][n] = relu(bias[n] + sum_k A(m,k) W[n][k]) as bf16, with m = (b, oy, ox) and
// k = tap * C0 + c. A(m,k) is read straight from the NHWC input (no im2col copy), zero outside
// the frame.
// DGRAD: the same product for the data gradient of a decoder layer (input dZ, weights flipped and
// transposed; no bias or ReLU, FP32). Its first C1 channels belong to the upsampled source, whose
// gradient is the sum over the four pixels of an upsampled one: the pixels of a tile are taken in
// 2x2 quads, m = 4 ((b H/2 + Y) H/2 + X) + (2 dy + dx), a quad's four lanes add up and one stores
// to `out` [H/2][H/2][C1]; the rest go to `out2` [H][H][Cout - C1], the skip connection's. Written
// out whole and summed by another kernel the gradient of 64 samples' two layers took 323 us,
// this way 212 (the product is what is left of it).
// S2: the data gradient of a stride-2 layer (input dZ [H][H][C0], the same flipped weights), added to
// `out` [2H][2H][Cout]: pixel (2Y + py, 2X + px) meets 1, 2, 2 or 4 of the nine taps by its parity,
// m = (b H + Y) H + X within a parity. By a product into columns (0.23 GB for the two layers of
// 64 samples) and another kernel gathering them the two took 175 us, this way 73.
// FOLD: a decoder layer, channels [0, C0) from src0 at half resolution (nearest 2x upsampling),
// channels [C0, C0 + C1) from src1 (the skip connection). The upsampled source is read at its own
// resolution: output pixel (2Y + py, 2X + px) sees through its 3x3 taps only the 2 x 2 source
// pixels (Y - 1 + py + i, X - 1 + px + j), so the taps landing on one source pixel are summed into
// folded weights, one matrix per output parity (k_fold_weights: [4][Cout][Kp'], k' = (2i + j) C0
// + c for the upsampled part, then 4 C0 + tap C1 + c for the skip part, Kp' = 4 C0 + 9 C1).
// The pixels of a tile share one parity: m = ((parity B + b) (H/2) + Y) (H/2) + X.
//
// A workgroup computes 64 MT pixels x BN output channels in 64-deep K chunks (one tap, one source
// per chunk). Each of its four wavefronts owns 16 MT pixels and all BN channels, so a pixel's
// values are used by one wavefront only and go from memory straight into its MFMA operands (a
// lane's 8 consecutive channels of one pixel: one 16-byte load), the next chunk's in flight during
// the current one; the weights, which all four share, go through LDS (double buffer). Row offsets
// are 32-bit and change only with the tap; a pixel outside the frame takes an offset beyond the
// buffer, which reads zero. With both operands through LDS and 64-bit addresses per chunk the
// pass spent more on addresses than on MFMAs (511 pairs, executed
// TFLOP/s: L2 330, L3 260, L4 345, L5 245; now 610, 430, 730, 435: the values' nine reads through
// the first-level cache bound it).
// The product is formed transposed (channels as rows), so that a lane ends with 4 consecutive
// channels of a pixel and stores them together.
// Requires C0 % 64 == 0 (S2: 128), C1 % 64 == 0, BN | Cout (DGRAD: BN | C1), (pixels of a parity) % (64 MT) == 0,
// Kp % 8 == 0, Hin a power of two.

constexpr int CV_BK = 64, CV_LD = CV_BK + 8;

typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

template <int MT, int BN, bool DGRAD, bool FOLD, bool S2>
__global__ void __launch_bounds__(256, 2) k_conv_fwd(
    const bf16* __restrict__ src0, int C0, const bf16* __restrict__ src1, int C1, int Hin,
    int stride, const bf16* __restrict__ Wt, int Kp, const float* __restrict__ bias, int Cout,
    void* __restrict__ out_, float* __restrict__ out2) {
  static_assert(FOLD + DGRAD + S2 <= 1, "one of the three");
  constexpr bool PAR = FOLD || S2;  // the pixels of a tile share an output parity
  constexpr int BM = 64 * MT, TN = BN / 16, B_PIECES = BN * 8 / 256;
  constexpr unsigned OUTSIDE = 0x80000000u;  // beyond every buffer: reads zero
  __shared__ __attribute__((aligned(16))) bf16 sB[2][BN * CV_LD];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int Hout = Hin / stride, Hs0 = FOLD ? Hin / 2 : Hin;
  const int n0 = blockIdx.y * BN;
  const int tiles_per_par = PAR ? gridDim.x / 4 : 1;
  const int quarter = PAR ? blockIdx.x / tiles_per_par : 0;
  const int par = S2 ? 3 - quarter : quarter;  // S2: the parity of four taps first
  const int py = par >> 1, px = par & 1;
  const int nchunks = (FOLD ? 4 * C0 + 9 * C1 : S2 ? (1 + py) * (1 + px) * C0 : 9 * C0) / CV_BK;
  const long long m0 = (long long)(PAR ? blockIdx.x - quarter * tiles_per_par : blockIdx.x) * BM;
  if (FOLD) Wt += (size_t)par * Cout * Kp;
  const int Hm = FOLD ? Hout / 2 : Hout, lh = __builtin_ctz(Hm);
  // the tile's first sample: 64-bit bases here, 32-bit offsets from here on
  const long long bs = m0 >> (2 * lh);
  const bf16* const base0 = src0 + (size_t)bs * Hs0 * Hs0 * C0;
  const bf16* const base1 = FOLD ? src1 + (size_t)bs * Hin * Hin * C1 : base0;
  // this lane's pixels: byte offsets of their centre (FOLD: of (Y, X) in src0 and of the output
  // pixel in src1) plus the lane's channels, and which taps lie inside the frame
  const int row16 = lane & 15, kq = lane >> 4;
  unsigned off0[MT], off1[MT], inside[MT];
  // S2: tap k of this parity, its offset in dZ and its place in the 3x3 window
  auto s2_tap = [&](int k, int& dy, int& dx) {
    const int ky = px ? k >> 1 : k, kx = px ? k & 1 : 0;
    dy = py ? 1 - ky : 0;
    dx = px ? 1 - kx : 0;
    return (py ? 2 * ky : 1) * 3 + (px ? 2 * kx : 1);
  };
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    const long long m = m0 + wave * 16 * MT + 16 * i + row16;
    int ox = (int)m & (Hm - 1), oy = (int)(m >> lh) & (Hm - 1);
    if (DGRAD) {  // quads: X, Y from m / 4
      ox = 2 * ((int)(m >> 2) & (Hm / 2 - 1)) + ((int)m & 1);
      oy = 2 * ((int)(m >> (lh + 1)) & (Hm / 2 - 1)) + ((int)m >> 1 & 1);
    }
    const unsigned rb = (unsigned)((m >> (2 * lh)) - bs);
    const int y0 = FOLD ? oy : oy * stride, x0 = FOLD ? ox : ox * stride;
    off0[i] = (((rb * Hs0 + y0) * Hs0 + x0) * C0 + 8 * kq) * 2;
    off1[i] = 0;
    unsigned in = 0;
    if (FOLD) {
      const int y = 2 * oy + py, x = 2 * ox + px;
      off1[i] = (((rb * Hin + y) * Hin + x) * C1 + 8 * kq) * 2;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int sy = oy - 1 + py + (t >> 1), sx = ox - 1 + px + (t & 1);
        in |= (unsigned)(sy >= 0 && sy < Hs0 && sx >= 0 && sx < Hs0) << t;
      }
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        const int iy = y + t / 3 - 1, ix = x + t % 3 - 1;
        in |= (unsigned)(iy >= 0 && iy < Hin && ix >= 0 && ix < Hin) << (4 + t);
      }
    } else if (S2) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        int dy, dx;
        s2_tap(t, dy, dx);
        in |= (unsigned)(t < (1 + py) * (1 + px) && oy + dy < Hin && ox + dx < Hin) << t;
      }
    } else {
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        const int iy = y0 + t / 3 - 1, ix = x0 + t % 3 - 1;
        in |= (unsigned)(iy >= 0 && iy < Hin && ix >= 0 && ix < Hin) << t;
      }
    }
    inside[i] = in;
  }
  // position of the next chunk to fetch: tap (FOLD: 0-3 source pixels, 4-12 skip taps), channel
  int tap = 0, c = 0;
  int wtap = 0;  // S2: first column of the tap's weights
  unsigned voff[MT];
  auto set_tap = [&] {
    const bool skip = FOLD && tap >= 4;
    int dy, dx, C, H;
    if (FOLD && !skip) {
      dy = (tap >> 1) - 1 + py;
      dx = (tap & 1) - 1 + px;
      C = C0;
      H = Hs0;
    } else if (S2) {
      wtap = (8 - s2_tap(tap, dy, dx)) * C0;
      C = C0;
      H = Hin;
    } else {
      const int t = FOLD ? tap - 4 : tap;
      dy = t / 3 - 1;
      dx = t % 3 - 1;
      C = FOLD ? C1 : C0;
      H = Hin;
    }
    const unsigned d = (unsigned)((dy * H + dx) * C * 2);
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      if (FOLD && tap == 4) off0[i] = off1[i];  // on to the skip taps
      voff[i] = (inside[i] >> tap) & 1u ? off0[i] + d : OUTSIDE;
    }
  };
  set_tap();
  u32x4 a[2][MT][2], rb[B_PIECES];
  int chunk_f = 0;
  auto fetch = [&](u32x4 (&fa)[MT][2]) {
    const bool skip = FOLD && tap >= 4;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(skip ? base1 : base0), 0, 0x7fffffff, 0x00020000);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        fa[i][h] = __builtin_amdgcn_raw_buffer_load_b128(rs, voff[i] + 64 * h, c * 2, 0);
#pragma unroll
    for (int r = 0; r < B_PIECES; ++r) {
      const int e = tid + 256 * r;
      rb[r] = *(const u32x4*)(Wt + (size_t)(n0 + (e >> 3)) * Kp +
                              (S2 ? wtap + c : chunk_f * CV_BK) + (e & 7) * 8);
    }
    ++chunk_f;
    c += CV_BK;
    if (c == (skip ? C1 : C0)) {
      c = 0;
      ++tap;
      set_tap();
    }
  };
  auto stash = [&](int buf) {
#pragma unroll
    for (int r = 0; r < B_PIECES; ++r) {
      const int e = tid + 256 * r;
      *(u32x4*)&sB[buf][(e >> 3) * CV_LD + (e & 7) * 8] = rb[r];
    }
  };
  f32x4 acc[MT][TN];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
  // S2: a tap's products are summed by themselves, the taps' sums then added in order
  f32x4 taps[S2 ? MT : 1][S2 ? TN : 1];
  if (S2)
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) taps[S2 ? i : 0][S2 ? j : 0] = (f32x4){0.f, 0.f, 0.f, 0.f};
  // the weights' operands are read two steps ahead (the barriers keep the compiler from reading a
  // whole chunk's at once, which would not leave registers for the accumulators)
  auto multiply = [&](const u32x4 (&fa)[MT][2], int buf) {
    auto weights = [&](int t) {
      return *(const bf16x8*)&sB[buf][(16 * (t % TN) + row16) * CV_LD + 32 * (t / TN) + 8 * kq];
    };
    bf16x8 b[3];
    b[0] = weights(0);
    b[1] = weights(1);
#pragma unroll
    for (int t = 0; t < 2 * TN; ++t) {
      if (t + 2 < 2 * TN) b[(t + 2) % 3] = weights(t + 2);
#pragma unroll
      for (int i = 0; i < MT; ++i)
        acc[i][t % TN] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            b[t % 3], __builtin_bit_cast(bf16x8, fa[i][t / TN]), acc[i][t % TN], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  fetch(a[0]);
  stash(0);
  __syncthreads();
  // two chunks per round, one operand set each; the last of an odd count follows
  for (int chunk = 0; chunk + 2 <= nchunks; chunk += 2) {
    fetch(a[1]);
    multiply(a[0], 0);
    stash(1);
    __syncthreads();
    if (chunk + 2 < nchunks) fetch(a[0]);
    multiply(a[1], 1);
    if (S2 && (chunk + 2) % (C0 / CV_BK) == 0)
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          taps[S2 ? i : 0][S2 ? j : 0] += acc[i][j];
          acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
        }
    stash(0);  // nothing reads it where no chunk follows
    __syncthreads();
  }
  if (nchunks & 1) multiply(a[0], 0);
  // epilogue: bias, ReLU, bf16 NHWC (forward) or the plain FP32 sums (data gradient); lane: pixel
  // row16 of each 16, channels 4 kq .. 4 kq + 3 of each 16
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    long long row = m0 + wave * 16 * MT + 16 * i + row16;
    if (PAR) {  // (b, Y, X) -> the output pixel (b, 2Y + py, 2X + px)
      const long long X = row & (Hm - 1), Y = (row >> lh) & (Hm - 1), bb = row >> (2 * lh);
      row = (bb * 2 * Hm + 2 * Y + py) * 2 * Hm + 2 * X + px;
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int col = n0 + 16 * j + 4 * kq;
      if (S2) {
        f32x4* d = (f32x4*)((float*)out_ + row * Cout + col);
        *d = *d + taps[S2 ? i : 0][S2 ? j : 0];
      } else if (DGRAD) {
        f32x4 v = acc[i][j];
        if (n0 < C1) {  // uniform: BN divides C1
#pragma unroll
          for (int r = 0; r < 4; ++r)  // the quad's first lane: its four values in order
            v[r] = ((v[r] + dpp_f<0x55>(v[r])) + dpp_f<0xaa>(v[r])) + dpp_f<0xff>(v[r]);
          if ((row16 & 3) == 0) *(f32x4*)((float*)out_ + (row >> 2) * C1 + col) = v;
        } else {
          const long long X = (row >> 2) & (Hm / 2 - 1), Y = (row >> (lh + 1)) & (Hm / 2 - 1);
          const long long q = ((row >> (2 * lh)) * Hm + 2 * Y + (row >> 1 & 1)) * Hm + 2 * X + (row & 1);
          *(f32x4*)(out2 + q * (Cout - C1) + (col - C1)) = v;
        }
      } else {
        const f32x4 bv = *(const f32x4*)(bias + col);
        unsigned int h[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float v = acc[i][j][r] + bv[r];
          h[r] = __builtin_bit_cast(unsigned short, (bf16)(v > 0.f ? v : 0.f));
        }
        *(uint2*)((bf16*)out_ + row * Cout + col) =
            make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
      }
    }
  }
}

// Folded weights of an upsampling layer (see k_conv_fwd's FOLD): Wf[par][co][k'] from the
// layer's W[co][k] (k = tap Cin + c): for the upsampled part the sum, over the taps landing on
// source offset (i, j) for parity par, of W[co][tap Cin + c] (FP32, taps in order, rounded to
// BF16 once); the skip part copied.
__global__ void k_fold_weights(const bf16* __restrict__ W, int Cout, int C0, int C1, int Kp,
                               bf16* __restrict__ Wf) {
  const int Cin = C0 + C1, Kf = 4 * C0 + 9 * C1;
  const long long total = 4LL * Cout * Kf;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    const int k = (int)(e % Kf);
    const long long t = e / Kf;
    const int co = (int)(t % Cout), par = (int)(t / Cout);
    const bf16* w = W + (size_t)co * Kp;
    if (k < 4 * C0) {
      const int ij = k / C0, c = k - ij * C0, i = ij >> 1, j = ij & 1;
      const int py = par >> 1, px = par & 1;
      // tap rows (columns) landing on source row (column) offset i (j) for parity py (px)
      const int r0 = py == 0 ? (i == 0 ? 0 : 1) : (i == 0 ? 0 : 2);
      const int r1 = py == 0 ? (i == 0 ? 0 : 2) : (i == 0 ? 1 : 2);
      const int c0 = px == 0 ? (j == 0 ? 0 : 1) : (j == 0 ? 0 : 2);
      const int c1 = px == 0 ? (j == 0 ? 0 : 2) : (j == 0 ? 1 : 2);
      float acc = 0.f;
      for (int ty = r0; ty <= r1; ++ty)
        for (int tx = c0; tx <= c1; ++tx) acc += (float)w[(ty * 3 + tx) * Cin + c];
      Wf[e] = (bf16)acc;
    } else {
      const int r = k - 4 * C0, tap = r / C1, c = r - tap * C1;
      Wf[e] = w[tap * Cin + C0 + c];
    }
  }
}

// Weights of a stride-1 3x3 layer for its data gradient: W'[ci][tap][co] = W[co][8 - tap][ci]
// (the transposed convolution is the convolution with the taps flipped), BF16.
__global__ void k_flip_weights(const bf16* __restrict__ W, int Cout, int Cin, int Kp,
                               bf16* __restrict__ Wf) {
  long long total = (long long)Cin * 9 * Cout;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x) {
    int co = (int)(i % Cout);
    int tap = (int)((i / Cout) % 9);
    int ci = (int)(i / (9LL * Cout));
    Wf[i] = W[(size_t)co * Kp + (size_t)(8 - tap) * Cin + ci];
  }
}

// Weight gradient of a 3x3 layer (64-channel blocks of input and output):
//   dW[co][tap Cin + c] = sum over output pixels p of dZ[p][co] X[p stride + tap][c],
// X the layer's input: channels [0, C0) from src0 (UP: at half resolution, the decoder's nearest
// 2x upsampling), the rest from src1. A workgroup takes 64 output channels (blockIdx.y), 64 input
// channels (blockIdx.x) and a share of the pixels (blockIdx.z) for all nine taps: dZ and the
// input's halo of 64 output pixels (2^LW wide) are staged in LDS once for the nine products, the
// next 64 pixels' loads in flight meanwhile. The contraction runs over pixels, but both operands
// lie channel-fastest: the LDS transpose reads (ds_read_b64_tr_b16: a 16-lane group reads 4 rows
// of 16 and each lane gets a column's 4) hand the MFMAs 8 pixels of one channel per lane. Each
// wavefront owns 16 input channels: 36 accumulator tiles. Partials [split][Cout][9 Cin], summed in
// split order by k_split_sum. The columns written out (906 MB for L5 of 64 samples), read back and
// transposed into LDS by 2-byte stores took 1.9 ms of the 3.9 ms gradients of 64 samples; the four
// launches of this kernel take 0.23 ms (590 TFLOP/s).
typedef __attribute__((ext_vector_type(4))) short s16x4;
template <int STR, int LW, bool UP>
__global__ void __launch_bounds__(256, 2) k_wgrad(const bf16* __restrict__ dZ, int Cout,
                                                  const bf16* __restrict__ src0, int C0,
                                                  const bf16* __restrict__ src1, int C1, int units,
                                                  int per_split, float* __restrict__ part) {
  constexpr int W = 1 << LW, R = 64 >> LW, H = W * STR;  // output width, rows per unit, input side
  constexpr int HR = (R - 1) * STR + 3, HC = (W - 1) * STR + 3, HP = HR * HC;
  constexpr int LD = 72;  // LDS row of 64 channels plus 8
  constexpr int XP = (HP * 8 + 255) / 256;
  __shared__ __attribute__((aligned(16))) short sX[HP * LD];
  __shared__ __attribute__((aligned(16))) short sZ[64 * LD];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 15, kq = lane >> 4;
  const int Cin = C0 + C1, cb = blockIdx.x * 64, co0 = blockIdx.y * 64;
  const bool first = cb < C0;
  const bool up = UP && first;
  const bf16* src = first ? src0 + cb : src1 + (cb - C0);
  const int Cs = first ? C0 : C1, Hs = up ? H / 2 : H;
  const int u0 = blockIdx.z * per_split, u1 = min(u0 + per_split, units);
  uint4 rx[XP], rz[2];
  auto fetch = [&](int u) {
    const int b = u / (W / R), y0 = (u & (W / R - 1)) * R;
#pragma unroll
    for (int q = 0; q < XP; ++q) {
      const int e = tid + 256 * q, px = e >> 3;
      const int iy = y0 * STR - 1 + px / HC, ix = px % HC - 1;
      uint4 v = make_uint4(0u, 0u, 0u, 0u);
      if (px < HP && iy >= 0 && iy < H && ix >= 0 && ix < H) {
        const int sy = up ? iy >> 1 : iy, sx = up ? ix >> 1 : ix;
        v = *(const uint4*)(src + (((size_t)b * Hs + sy) * Hs + sx) * Cs + (e & 7) * 8);
      }
      rx[q] = v;
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int e = tid + 256 * q;
      rz[q] = *(const uint4*)(dZ + ((size_t)u * 64 + (e >> 3)) * Cout + co0 + (e & 7) * 8);
    }
  };
  auto stash = [&] {
#pragma unroll
    for (int q = 0; q < XP; ++q) {
      const int e = tid + 256 * q;
      if ((e >> 3) < HP) *(uint4*)&sX[(e >> 3) * LD + (e & 7) * 8] = rx[q];
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int e = tid + 256 * q;
      *(uint4*)&sZ[(e >> 3) * LD + (e & 7) * 8] = rz[q];
    }
  };
#define LDS_TR(p) \
  __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p))
  auto operand = [&](s16x4 lo, s16x4 hi) {  // pixels 8 kq .. 8 kq + 7 of the lane's channel
    typedef __attribute__((ext_vector_type(8))) short s16x8;
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  // this lane's share of the transpose reads: rows (pixels) 8 kq + j / 4 and 4 more, 4 channels
  int zoff[2], xoff[2][2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const int p0 = 32 * ks + 8 * kq + (j >> 2);
    zoff[ks] = p0 * LD + 4 * (j & 3);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int p = p0 + 4 * h;
      xoff[ks][h] =
          ((p >> LW) * STR * HC + (p & (W - 1)) * STR) * LD + 16 * wave + 4 * (j & 3);
    }
  }
  f32x4 acc[9][4];
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int m = 0; m < 4; ++m) acc[t][m] = (f32x4){0.f, 0.f, 0.f, 0.f};
  if (u0 < u1) fetch(u0);
  for (int u = u0; u < u1; ++u) {
    __syncthreads();
    stash();
    __syncthreads();
    if (u + 1 < u1) fetch(u + 1);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      bf16x8 a[4];
#pragma unroll
      for (int m = 0; m < 4; ++m)
        a[m] = operand(LDS_TR(sZ + zoff[ks] + 16 * m), LDS_TR(sZ + zoff[ks] + 4 * LD + 16 * m));
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        const int d = (t / 3 * HC + t % 3) * LD;
        const bf16x8 b = operand(LDS_TR(sX + xoff[ks][0] + d), LDS_TR(sX + xoff[ks][1] + d));
#pragma unroll
        for (int m = 0; m < 4; ++m)
          acc[t][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m], b, acc[t][m], 0, 0, 0);
      }
    }
  }
#undef LDS_TR
  float* out = part + (size_t)blockIdx.z * Cout * 9 * Cin;
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        out[(size_t)(co0 + 16 * m + 4 * kq + r) * 9 * Cin + t * Cin + cb + 16 * wave + j] =
            acc[t][m][r];
}

// Sum of `splits` partial results, count a multiple of 64: 64 consecutive results per workgroup, a
// quarter of the splits (each fourth) per wavefront in order, then the quarters in order.
__global__ void __launch_bounds__(256) k_split_sum(const float* __restrict__ part,
                                                   long long stride, int splits,
                                                   float* __restrict__ out) {
  __shared__ float red[4][64];
  const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
  const float* p = part + blockIdx.x * 64LL + lane;
  float s = 0.f;
#pragma unroll 8
  for (int k = q; k < splits; k += 4) s += p[k * stride];
  red[q][lane] = s;
  __syncthreads();
  if (q == 0) out[blockIdx.x * 64LL + lane] = ((s + red[1][lane]) + red[2][lane]) + red[3][lane];
}

// ------------------------------------------------------------------------------------------
// Layout kernels

// Columns of a layer with two input channels: col[(b, oy, ox)][(dy * 3 + dx) * 2 + c] =
// X[b][oy*s + dy - 1][ox*s + dx - 1][c] (0 outside), zero for k >= 18 up to Kp (a multiple of 8).
// A thread takes 8 entries, four taps of 4 bytes, and stores them together: bound by the stores
// (one entry a thread took 60 us for the 34 MB of 64 samples, this 16).
__global__ void k_im2col2(const bf16* __restrict__ X, int Bn, int H, int W, int s, int Kp,
                          bf16* __restrict__ col) {
  const int Ho = H / s, Wo = W / s, G = Kp / 8;
  const long long total = (long long)Bn * Ho * Wo * G;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x) {
    const int g = (int)(i % G);
    const long long p = i / G;
    const int ox = (int)(p % Wo), oy = (int)((p / Wo) % Ho);
    const long long b = p / ((long long)Wo * Ho);
    unsigned int v[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int tap = 4 * g + t, y = oy * s + tap / 3 - 1, x = ox * s + tap % 3 - 1;
      const bool in = tap < 9 && y >= 0 && y < H && x >= 0 && x < W;
      v[t] = in ? *(const unsigned int*)(X + ((b * H + y) * W + x) * 2) : 0u;
    }
    *(uint4*)(col + i * 8) = make_uint4(v[0], v[1], v[2], v[3]);
  }
}

// dZ = dA * (A > 0) as bf16 (A is the layer's ReLU output), [M][N] with N a multiple of 8 that
// divides 2048, and the column sums of dZ (the bias gradient) per workgroup: part[block][N]. A
// thread keeps 8 columns: two 16-byte loads of dA and one of A per row.
__global__ void __launch_bounds__(kBlock) k_relu_bwd(const float* __restrict__ dA,
                                                     const bf16* __restrict__ A, long long M,
                                                     int N, bf16* __restrict__ dZ,
                                                     float* __restrict__ part) {
  __shared__ float red[kBlock][8];
  const int per_row = N / 8, c8 = threadIdx.x % per_row, rows = kBlock / per_row;
  float sum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (long long r = (long long)blockIdx.x * rows + threadIdx.x / per_row; r < M;
       r += (long long)gridDim.x * rows) {
    const long long i = r * N + 8 * c8;
    const f32x4 d0 = *(const f32x4*)(dA + i), d1 = *(const f32x4*)(dA + i + 4);
    const bf16x8 a = *(const bf16x8*)(A + i);
    bf16x8 z;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      z[k] = (bf16)((float)a[k] > 0.f ? (k < 4 ? d0[k & 3] : d1[k & 3]) : 0.f);
      sum[k] += (float)z[k];
    }
    *(bf16x8*)(dZ + i) = z;
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) red[threadIdx.x][k] = sum[k];
  __syncthreads();
  for (int n = threadIdx.x; n < N; n += kBlock) {
    float t = 0.f;
    for (int q = 0; q < rows; ++q) t += red[q * per_row + n / 8][n & 7];
    part[(size_t)blockIdx.x * N + n] = t;
  }
}

// Column sums of per-chunk partials [chunks][N]: one workgroup (kBlock threads) per column;
// thread j sums chunks j, j + kBlock, ... in order, then a fixed tree over the threads.
__global__ void __launch_bounds__(kBlock) k_colsum_final(const float* __restrict__ part, int N,
                                                         int chunks, float* __restrict__ out) {
  __shared__ float red[kBlock];
  int n = blockIdx.x;
  float s = 0.f;
  for (int c = threadIdx.x; c < chunks; c += kBlock) s += part[(size_t)c * N + n];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = kBlock / 2; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[n] = red[0];
}

__global__ void k_f32_to_bf16(const float* __restrict__ x, long long count,
                              bf16* __restrict__ y) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < count;
       i += (long long)gridDim.x * blockDim.x)
    y[i] = (bf16)x[i];
}

// ------------------------------------------------------------------------------------------
// Last layer (66 -> 2 channels, stride 1), FP32 direct kernels. W6 is [2][9][66] fp32 (from the
// bf16 copy), bias b6[2].

// Last layer read straight from its sources. Channels 0..63 are the nearest 2x upsampling of
// the L5 output a5 [B][64][64][64]: output pixel (2Y + py, 2X + px) sees through its 3x3 taps
// only the 2 x 2 source pixels (Y - 1 + py + i, X - 1 + px + j), i, j in {0, 1} (tap rows
// {0} and {1, 2} land on source rows Y - 1 and Y when py = 0, {0, 1} and {2} on Y and Y + 1
// when py = 1; columns alike), so the taps that land on one source pixel are summed into the
// folded weights W6f [parity py px][i][j][output][64] (k_w6_prep): 4 source pixels of 64
// channels instead of 9. Channels 64, 65 are the network input x0 [B][128][128][2] (9 taps,
// weights W6 [2][9][66]). Eight lanes share an output pixel, lane g taking channels 8g .. 8g + 7
// (one 16-byte piece of each source pixel, so a source pixel is one 128-byte line per 8 lanes)
// and x0 tap g (and tap 8 on lane 0); the 8 partial sums are then added across the lanes.
// A workgroup takes one (parity, 32 source pixels of a row) of NB samples at a time: its folded
// weights (2 KB of LDS) are read once per NB samples, and NB samples' source pixels are in flight
// together. Bound by the FP32 ALUs (unpacking and FMAs) and those loads: for 511 pairs one sample
// at a time with the parities' 8 KB took 400 us, NB = 4 takes 328. On MFMAs, the FP32 weights in
// three BF16 parts, the pass took 280; but the predictions' last bits start registrations, which
// amplify them. Lanes add up by DPP moves (pairs, pairs of pairs, the mirrored half row).
template <int NB>
__global__ void __launch_bounds__(256) k_l6_fused(const bf16* __restrict__ a5,
                                                  const bf16* __restrict__ x0,
                                                  const float* __restrict__ W6,
                                                  const float* __restrict__ W6f,
                                                  const float* __restrict__ b6, int Bn,
                                                  float* __restrict__ Y) {
  constexpr int C = 66;
  __shared__ __attribute__((aligned(16))) float wf[2 * 2 * 2 * 64];
  const int g = threadIdx.x & 7;  // channel group
  // the grid is a multiple of 512 workgroups: all samples of a workgroup share parity and row
  const int half = blockIdx.x & 1, ys = (blockIdx.x >> 1) & 63, par = (blockIdx.x >> 7) & 3;
  const int py = par >> 1, px = par & 1;
  for (int e = threadIdx.x; e < 2 * 2 * 2 * 64; e += blockDim.x) wf[e] = W6f[par * 512 + e];
  __syncthreads();
  const int xs = half * 32 + (threadIdx.x >> 3);
  const int y = 2 * ys + py, x = 2 * xs + px;
  const int per = (Bn + NB - 1) / NB;  // samples b, b + per, ... of an iteration
  for (int b0 = blockIdx.x >> 9; b0 < per; b0 += gridDim.x >> 9) {
    float s0[NB], s1[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      s0[q] = g == 0 ? b6[0] : 0.f;
      s1[q] = g == 0 ? b6[1] : 0.f;
    }
    uint4 v[2][2][NB];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int sy = ys - 1 + py + i, sx = xs - 1 + px + j;
        const bool ok = sy >= 0 && sy < 64 && sx >= 0 && sx < 64;
#pragma unroll
        for (int q = 0; q < NB; ++q) {
          const int b = min(b0 + q * per, Bn - 1);
          v[i][j][q] = ok ? *(const uint4*)(a5 + (((size_t)b * 64 + sy) * 64 + sx) * 64 + 8 * g)
                          : make_uint4(0u, 0u, 0u, 0u);
        }
      }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int sy = ys - 1 + py + i;
      if (sy < 0 || sy >= 64) continue;  // uniform over the workgroup (one source row)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const float* w0 = wf + (i * 2 + j) * 2 * 64 + 8 * g;
        const f32x4 wa = *(const f32x4*)w0, wb = *(const f32x4*)(w0 + 4);
        const f32x4 wc = *(const f32x4*)(w0 + 64), wd = *(const f32x4*)(w0 + 68);
#pragma unroll
        for (int q = 0; q < NB; ++q) {
          const unsigned int h[4] = {v[i][j][q].x, v[i][j][q].y, v[i][j][q].z, v[i][j][q].w};
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const float lo = __uint_as_float(h[k] << 16), hi = __uint_as_float(h[k] & 0xffff0000u);
            const float w0lo = k < 2 ? wa[2 * k] : wb[2 * k - 4];
            const float w0hi = k < 2 ? wa[2 * k + 1] : wb[2 * k - 3];
            const float w1lo = k < 2 ? wc[2 * k] : wd[2 * k - 4];
            const float w1hi = k < 2 ? wc[2 * k + 1] : wd[2 * k - 3];
            s0[q] = fmaf(w0lo, lo, s0[q]);
            s1[q] = fmaf(w1lo, lo, s1[q]);
            s0[q] = fmaf(w0hi, hi, s0[q]);
            s1[q] = fmaf(w1hi, hi, s1[q]);
          }
        }
      }
    }
    // x0 channels: lane g takes tap g, lane 0 also tap 8
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int tap = t == 0 ? g : 8;
      if (t == 1 && g != 0) break;
      const int yy = y + tap / 3 - 1, xx = x + tap % 3 - 1;
      if (yy >= 0 && yy < 128 && xx >= 0 && xx < 128) {
        const float wa = W6[tap * C + 64], wb = W6[9 * C + tap * C + 64];
        const float wc = W6[tap * C + 65], wd = W6[9 * C + tap * C + 65];
#pragma unroll
        for (int q = 0; q < NB; ++q) {
          const int b = min(b0 + q * per, Bn - 1);
          const unsigned int u =
              *(const unsigned int*)(x0 + (((size_t)b * 128 + yy) * 128 + xx) * 2);
          const float f0 = __uint_as_float(u << 16), f1 = __uint_as_float(u & 0xffff0000u);
          s0[q] = fmaf(wa, f0, s0[q]);
          s1[q] = fmaf(wb, f0, s1[q]);
          s0[q] = fmaf(wc, f1, s0[q]);
          s1[q] = fmaf(wd, f1, s1[q]);
        }
      }
    }
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      // the 8 channel groups' partial sums (lanes 8p .. 8p + 7), fixed order: lane pairs, pairs
      // of pairs, then the mirrored half row (whose four lanes all hold the other four's sum)
      float t0 = s0[q], t1 = s1[q];
      t0 += dpp_f<0xb1>(t0);  // quad_perm 1, 0, 3, 2
      t1 += dpp_f<0xb1>(t1);
      t0 += dpp_f<0x4e>(t0);  // quad_perm 2, 3, 0, 1
      t1 += dpp_f<0x4e>(t1);
      t0 += dpp_f<0x141>(t0);  // row_half_mirror
      t1 += dpp_f<0x141>(t1);
      const int b = b0 + q * per;
      if (g == 0 && b < Bn)
        *(float2*)(Y + (((size_t)b * 128 + y) * 128 + x) * 2) = make_float2(t0, t1);
    }
  }
}

// FP32 copies of the last layer's weights from the BF16 copy: W6 [2][9][66] (the backward
// pass's) and the folded W6f of k_l6_fused, each entry the sum, in tap order, of the taps that
// land on its source pixel. One workgroup.
__global__ void __launch_bounds__(256) k_w6_prep(const bf16* __restrict__ wb6,
                                                 float* __restrict__ W6,
                                                 float* __restrict__ W6f) {
  constexpr int C = 66;
  for (int k = threadIdx.x; k < 2 * 9 * C; k += blockDim.x) W6[k] = (float)wb6[k];
  __syncthreads();
  for (int e = threadIdx.x; e < 4 * 2 * 2 * 2 * 64; e += blockDim.x) {
    const int c = e & 63, o = (e >> 6) & 1, j = (e >> 7) & 1, i = (e >> 8) & 1, par = e >> 9;
    const int py = par >> 1, px = par & 1;
    // tap rows (columns) landing on source row (column) offset i (j) for parity py (px)
    const int r0 = py == 0 ? (i == 0 ? 0 : 1) : (i == 0 ? 0 : 2);
    const int r1 = py == 0 ? (i == 0 ? 0 : 2) : (i == 0 ? 1 : 2);
    const int c0 = px == 0 ? (j == 0 ? 0 : 1) : (j == 0 ? 0 : 2);
    const int c1 = px == 0 ? (j == 0 ? 0 : 2) : (j == 0 ? 1 : 2);
    float acc = 0.f;
    for (int ty = r0; ty <= r1; ++ty)
      for (int tx = c0; tx <= c1; ++tx) acc += W6[o * 9 * C + (ty * 3 + tx) * C + c];
    W6f[e] = acc;
  }
}

// First layer (2 -> 64 channels, stride 2, 128^2 -> 64^2) straight from the input x0
// [B][128][128][2]: one thread per output pixel holds its 18 inputs (k = tap * 2 + c); the
// weights W1 (k_w1_prep: [channels 4g .. 4g + 3][k][4], FP32) and the bias are the same for every
// lane and come through the scalar cache; FP32 sums in k order, then bias and ReLU; the 64 BF16
// outputs leave as eight 16-byte stores (NHWC). 1,152 products per pixel: bound by the ALUs (511
// pairs: 62 us of products) and the 268 MB it writes. With the weights in LDS the pass waited
// on 288 16-byte LDS reads per wavefront: 276 us, now 135.
__global__ void __launch_bounds__(256) k_l1_direct(const bf16* __restrict__ x0,
                                                   const float* __restrict__ W1,
                                                   const float* __restrict__ bias, int Bn,
                                                   bf16* __restrict__ out) {
  const long long total = (long long)Bn * 64 * 64;
  for (long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x; p < total;
       p += (long long)gridDim.x * blockDim.x) {
    const int ox = (int)(p & 63), oy = (int)((p >> 6) & 63);
    const long long b = p >> 12;
    float in[18];
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      const int iy = 2 * oy + tap / 3 - 1, ix = 2 * ox + tap % 3 - 1;
      const bool ok = iy >= 0 && iy < 128 && ix >= 0 && ix < 128;
      unsigned int v = ok ? *(const unsigned int*)(x0 + ((b * 128 + iy) * 128 + ix) * 2) : 0u;
      in[2 * tap] = __uint_as_float(v << 16);
      in[2 * tap + 1] = __uint_as_float(v & 0xffff0000u);
    }
    uint4* dst = (uint4*)(out + p * 64);
#pragma unroll 1
    for (int g2 = 0; g2 < 8; ++g2) {  // output channels 8 g2 .. 8 g2 + 7
      unsigned int h[8];
#pragma unroll
      for (int gg = 0; gg < 2; ++gg) {
        const float* w = W1 + (2 * g2 + gg) * 72;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < 18; ++k)
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[r] = fmaf(w[4 * k + r], in[k], acc[r]);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float v = acc[r] + bias[8 * g2 + 4 * gg + r];
          h[4 * gg + r] = __builtin_bit_cast(unsigned short, (bf16)(v > 0.f ? v : 0.f));
        }
      }
      dst[g2] = make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16),
                           h[6] | (h[7] << 16));
    }
  }
}

// FP32 copy of the first layer's BF16 weights in k_l1_direct's order.
__global__ void k_w1_prep(const bf16* __restrict__ W, int Kp, float* __restrict__ W1) {
  for (int e = threadIdx.x; e < 18 * 64; e += blockDim.x) {
    const int g = e / 72, k = e % 72 / 4, r = e & 3;
    W1[e] = (float)W[(4 * g + r) * Kp + k];
  }
}

// Data gradient of the last layer for its upsampled input, straight onto the L5 output grid
// (the adjoint of k_l6_fused's folded product, which also sums the four upsampled copies):
// source pixel (Y, X) feeds the outputs (2 Ys + py, 2 Xs + px) with Ys = Y + 1 - py - i and
// Xs = X + 1 - px - j through W6f[py px][i][j][o][c] (the output rows 2Y - 1 .. 2Y + 2 and the
// columns alike, 2 outputs each). One workgroup per 16 x 16 source pixels of a sample: dY staged
// in LDS (34 x 34, zero outside the image), a wavefront's halves walk 32 source pixels each, a lane
// taking two channels with its 64 weights in registers. Bound by the LDS reads of dY: 64 samples
// 24 us; one pixel a wavefront with the weights in LDS took 76.
constexpr int L6T = 16, L6H = 2 * L6T + 2, L6C = 66;
__device__ __forceinline__ void l6_stage_dy(const float* __restrict__ dY, int b, int Y0, int X0,
                                            float2* sY) {
  for (int i = threadIdx.x; i < L6H * L6H; i += 256) {
    const int y = 2 * Y0 - 1 + i / L6H, x = 2 * X0 - 1 + i % L6H;
    float2 v = make_float2(0.f, 0.f);
    if (y >= 0 && y < 128 && x >= 0 && x < 128)
      v = *(const float2*)(dY + (((size_t)b * 128 + y) * 128 + x) * 2);
    sY[i] = v;
  }
}
__global__ void __launch_bounds__(256) k_l6_bwd_a5(const float* __restrict__ dY,
                                                   const float* __restrict__ W6f,
                                                   float* __restrict__ dA5) {
  __shared__ __attribute__((aligned(16))) float2 sY[L6H * L6H];
  const int b = blockIdx.x >> 4, Y0 = (blockIdx.x >> 2 & 3) * L6T, X0 = (blockIdx.x & 3) * L6T;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, half = lane >> 5, ch = 2 * (lane & 31);
  float2 w[4][2][2][2];  // [py px][i][j][output]
#pragma unroll
  for (int k = 0; k < 32; ++k)
    w[k >> 3][k >> 2 & 1][k >> 1 & 1][k & 1] = *(const float2*)(W6f + k * 64 + ch);
  l6_stage_dy(dY, b, Y0, X0, sY);
  __syncthreads();
#pragma unroll 2
  for (int it = 0; it < 32; ++it) {
    const int p = wv * 64 + 2 * it + half, ly = p >> 4, lx = p & 15;
    float2 g[4][4];  // dY at rows 2Y - 1 .. 2Y + 2, columns alike
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const f32x4* row = (const f32x4*)(sY + (2 * ly + r) * L6H + 2 * lx);
      const f32x4 lo = row[0], hi = row[1];
      g[r][0] = make_float2(lo[0], lo[1]);
      g[r][1] = make_float2(lo[2], lo[3]);
      g[r][2] = make_float2(hi[0], hi[1]);
      g[r][3] = make_float2(hi[2], hi[3]);
    }
    float s0 = 0.f, s1 = 0.f;
#pragma unroll
    for (int py = 0; py < 2; ++py)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int px = 0; px < 2; ++px)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const float2 d = g[3 - py - 2 * i][3 - px - 2 * j];
            const float2(&wo)[2] = w[2 * py + px][i][j];
            s0 = fmaf(wo[0].x, d.x, s0);
            s1 = fmaf(wo[0].y, d.x, s1);
            s0 = fmaf(wo[1].x, d.y, s0);
            s1 = fmaf(wo[1].y, d.y, s1);
          }
    *(float2*)(dA5 + (((size_t)b * 64 + Y0 + ly) * 64 + X0 + lx) * 64 + ch) = make_float2(s0, s1);
  }
}

// L6 weight and bias gradients. Channels 0..63 of the layer's input are the 2x upsampling of the
// L5 output a5 [B][64][64][64], so a source pixel s meets a tap only through the sum of dY over
// the four output positions whose tap lands on one of its copies:
//   dW(o, tap, c) = sum_s a5(s, c) G(s, tap, o),
//   G(s, tap, o) = sum_{a, b in {0, 1}} dY(2Y + a + 1 - ty, 2X + b + 1 - tx, o),
// 18 products per source pixel and channel where the upsampled form takes 72. One workgroup per
// 16 x 16 source pixels of a sample: a thread forms the 18 sums of its source pixel from the
// staged dY (34 x 34, zero outside the image) and leaves them in LDS; then a wavefront's halves
// walk 32 source pixels each, a lane adding 18 products for two channels (4 bytes of a5, a pixel
// is one line). The input channels 64, 65 (x0 [B][128][128][2]) and the bias come from the
// thread's own four output positions and the 4 x 4 input pixels around them. FP32 sums
// throughout, in a fixed order; per-workgroup partials [workgroup][2 * 9 * 66 + 2] (weights
// o-major as in the layer, then the two biases), summed over workgroups by k_colsum_final. Bound
// by the LDS reads of the sums and the a5 stream: 64 samples 35 us where staging the
// upsampled input and walking it position by position took 235.
__global__ void __launch_bounds__(256) k_l6_bwd_w(const float* __restrict__ dY,
                                                  const bf16* __restrict__ a5,
                                                  const bf16* __restrict__ x0,
                                                  float* __restrict__ part) {
  constexpr int H = 128, GS = 20;  // floats per source pixel's sums (18, padded to 16 bytes)
  __shared__ float2 sY[L6H * L6H];
  __shared__ __attribute__((aligned(16))) float sG[L6T * L6T * GS];
  __shared__ float sX[4][38];
  const int b = blockIdx.x >> 4, Y0 = (blockIdx.x >> 2 & 3) * L6T, X0 = (blockIdx.x & 3) * L6T;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  l6_stage_dy(dY, b, Y0, X0, sY);
  __syncthreads();
  {
    const int ly = tid >> 4, lx = tid & 15;  // source pixel (Y0 + ly, X0 + lx)
    float2 g[4][4];                          // dY at rows 2Y - 1 .. 2Y + 2, columns alike
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int c = 0; c < 4; ++c) g[r][c] = sY[(2 * ly + r) * L6H + 2 * lx + c];
    // tap (ty, tx) takes rows 2 - ty, 3 - ty and columns 2 - tx, 3 - tx of that block
    float* G = sG + tid * GS;
#pragma unroll
    for (int tx = 0; tx < 3; ++tx) {
      float2 h[4];
#pragma unroll
      for (int r = 0; r < 4; ++r)
        h[r] = make_float2(g[r][2 - tx].x + g[r][3 - tx].x, g[r][2 - tx].y + g[r][3 - tx].y);
#pragma unroll
      for (int ty = 0; ty < 3; ++ty)
        *(float2*)(G + 2 * (3 * ty + tx)) =
            make_float2(h[2 - ty].x + h[3 - ty].x, h[2 - ty].y + h[3 - ty].y);
    }
    // input channels and bias of the output positions (2Y, 2X) .. (2Y + 1, 2X + 1)
    float ax[36], ab[2] = {0.f, 0.f};
#pragma unroll
    for (int k = 0; k < 36; ++k) ax[k] = 0.f;
    unsigned int xv[4][4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int y = 2 * (Y0 + ly) - 1 + r, x = 2 * (X0 + lx) - 1 + c;
        const bool in = y >= 0 && y < H && x >= 0 && x < H;
        xv[r][c] = in ? *(const unsigned int*)(x0 + (((size_t)b * H + y) * H + x) * 2) : 0u;
      }
#pragma unroll
    for (int pa = 0; pa < 2; ++pa)
#pragma unroll
      for (int pb = 0; pb < 2; ++pb) {
        const float2 d = g[1 + pa][1 + pb];
        ab[0] += d.x;
        ab[1] += d.y;
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
          const unsigned int u = xv[pa + tap / 3][pb + tap % 3];
          const float f0 = __uint_as_float(u << 16), f1 = __uint_as_float(u & 0xffff0000u);
          ax[4 * tap + 0] = fmaf(d.x, f0, ax[4 * tap + 0]);
          ax[4 * tap + 1] = fmaf(d.x, f1, ax[4 * tap + 1]);
          ax[4 * tap + 2] = fmaf(d.y, f0, ax[4 * tap + 2]);
          ax[4 * tap + 3] = fmaf(d.y, f1, ax[4 * tap + 3]);
        }
      }
#pragma unroll
    for (int k = 0; k < 38; ++k) {
      float v = k < 36 ? ax[k] : ab[k - 36];
#pragma unroll
      for (int m = 1; m < 64; m *= 2) v += __shfl_xor(v, m);
      if (lane == 0) sX[wv][k] = v;
    }
  }
  __syncthreads();
  float acc[18][2];
#pragma unroll
  for (int k = 0; k < 18; ++k) acc[k][0] = acc[k][1] = 0.f;
  {
    const int half = lane >> 5, ch = 2 * (lane & 31);
#pragma unroll 8
    for (int i = 0; i < 32; ++i) {
      const int s = wv * 64 + 2 * i + half;
      const unsigned int u = *(const unsigned int*)(
          a5 + (((size_t)b * 64 + Y0 + (s >> 4)) * 64 + X0 + (s & 15)) * 64 + ch);
      const float f0 = __uint_as_float(u << 16), f1 = __uint_as_float(u & 0xffff0000u);
      const float* G = sG + s * GS;
#pragma unroll
      for (int k = 0; k < 18; ++k) {
        const float w = G[k];
        acc[k][0] = fmaf(w, f0, acc[k][0]);
        acc[k][1] = fmaf(w, f1, acc[k][1]);
      }
    }
    __syncthreads();  // the sums have been read: their LDS takes the wavefronts' results
#pragma unroll
    for (int k = 0; k < 18; ++k) {
      const float v0 = acc[k][0] + __shfl_xor(acc[k][0], 32);
      const float v1 = acc[k][1] + __shfl_xor(acc[k][1], 32);
      if (half == 0) *(float2*)(sG + (wv * 18 + k) * 64 + ch) = make_float2(v0, v1);
    }
  }
  __syncthreads();
  constexpr int NP = 9 * L6C;  // (tap, c) pairs
  static_assert(4 * 18 * 64 <= L6T * L6T * GS, "the wavefronts' results fit the sums' LDS");
  float* out = part + (size_t)blockIdx.x * (2 * NP + 2);
  for (int e = tid; e < 18 * 64; e += 256) {
    const int k = e >> 6, c = e & 63;  // k = 2 tap + o
    const float v = ((sG[e] + sG[18 * 64 + e]) + sG[2 * 18 * 64 + e]) + sG[3 * 18 * 64 + e];
    out[(k & 1) * NP + (k >> 1) * L6C + c] = v;
  }
  if (tid < 38) {
    const float v = ((sX[0][tid] + sX[1][tid]) + sX[2][tid]) + sX[3][tid];
    const int o = tid >> 1 & 1, tap = tid >> 2;  // entries (tap, o, channel), then the biases
    out[tid < 36 ? o * NP + tap * L6C + 64 + (tid & 1) : 2 * NP + tid - 36] = v;
  }
}

// ------------------------------------------------------------------------------------------
// Loss: mean squared error over the interior (a border of `margin` pixels is left out).
// Writes per-block partial sums of squares and dY = 2 (Y - T) / count (0 in the border).

__global__ void k_mse(const float* __restrict__ Y, const float* __restrict__ T, int Bn, int H,
                      int Wd, int margin, float inv_count, float* __restrict__ dY,
                      double* __restrict__ part) {
  __shared__ double red[kBlock];
  long long total = (long long)Bn * H * Wd * 2;
  double s = 0.0;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x) {
    long long p = i / 2;
    int x = (int)(p % Wd), y = (int)((p / Wd) % H);
    bool in = x >= margin && x < Wd - margin && y >= margin && y < H - margin;
    float d = in ? Y[i] - T[i] : 0.f;
    s += (double)d * d;
    if (dY) dY[i] = 2.f * d * inv_count;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = blockDim.x / 2; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// Adam on FP32 master weights; refreshes the bf16 copy. Gradient g is the full fp32 gradient.
__global__ void k_adam(float* __restrict__ w, float* __restrict__ m, float* __restrict__ v,
                       const float* __restrict__ g, long long count, float lr, float b1,
                       float b2, float eps, float c1, float c2, bf16* __restrict__ wb) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < count;
       i += (long long)gridDim.x * blockDim.x) {
    float gi = g[i];
    float mi = b1 * m[i] + (1.f - b1) * gi;
    float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    float wi = w[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    w[i] = wi;
    if (wb) wb[i] = (bf16)wi;
  }
}

// Pack level-7 normalised frames of pairs into the network input [P][128][128][2] (fp32):
// channel 0 = reference, 1 = template; the 129^2 grid is cropped to 128^2.
__global__ void k_pack_pairs(const float* __restrict__ lvl, int n, const int* __restrict__ ref,
                             const int* __restrict__ tmpl, int P, float* __restrict__ out) {
  int S = n - 1;
  long long total = (long long)P * S * S;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x) {
    int x = (int)(i % S), y = (int)((i / S) % S), p = (int)(i / ((long long)S * S));
    out[i * 2] = lvl[(size_t)ref[p] * n * n + (size_t)y * n + x];
    out[i * 2 + 1] = lvl[(size_t)tmpl[p] * n * n + (size_t)y * n + x];
  }
}

// Level-7 displacement planes [P][2][n][n] (domain units) -> [P][n-1][n-1][2] in cells.
__global__ void k_planes_to_nhwc(const float* __restrict__ src, int n, long long pstride, int P,
                                 float scale, float* __restrict__ out) {
  int S = n - 1;
  long long total = (long long)P * S * S;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x) {
    int x = (int)(i % S), y = (int)((i / S) % S), p = (int)(i / ((long long)S * S));
    const float* s = src + p * pstride;
    out[i * 2] = scale * s[(size_t)y * n + x];
    out[i * 2 + 1] = scale * s[(size_t)n * n + (size_t)y * n + x];
  }
}

// Network output [P][S][S][2] (cells) -> slot planes [2][S+1][S+1] (domain units), replicating
// the last row and column; dst of slot p = base + p * stride.
__global__ void k_nhwc_to_planes(const float* __restrict__ y, int S, int P, float scale,
                                 float* __restrict__ base, long long stride) {
  int n = S + 1;
  long long total = (long long)P * n * n;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x) {
    int x = (int)(i % n), yy = (int)((i / n) % n), p = (int)(i / ((long long)n * n));
    int xs = min(x, S - 1), ys = min(yy, S - 1);
    const float* src = y + (((size_t)p * S + ys) * S + xs) * 2;
    float* d = base + p * stride;
    d[(size_t)yy * n + x] = scale * src[0];
    d[(size_t)n * n + (size_t)yy * n + x] = scale * src[1];
  }
}

// bad[p] = 1 when sample p of y [P][n_per] has a non-finite value or one with |v| > limit.
__global__ void k_check_pred(const float* __restrict__ y, long long n_per, float limit,
                             int* __restrict__ bad) {
  __shared__ int red[kBlock];
  const float* s = y + blockIdx.x * n_per;
  int b = 0;
  for (long long i = threadIdx.x; i < n_per; i += blockDim.x) {
    float v = s[i];
    if (!(fabsf(v) <= limit)) b = 1;
  }
  red[threadIdx.x] = b;
  __syncthreads();
  for (int o = blockDim.x / 2; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] |= red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) bad[blockIdx.x] = red[0];
}

}  // namespace

// ==========================================================================================
// Model

namespace pprs_cnn_impl {

struct Layer {
  int cin, cout, stride, kp;    // kp: padded K (columns of the weight matrix)
  int hin, hout;                // spatial size of input / output (square)
  long long woff, boff;         // offsets into the flat parameter vector
};

struct Model {
  int device = 0;
  hipStream_t stream = nullptr;
  Layer L[6];
  long long n_params = 0;
  float *w = nullptr, *m = nullptr, *v = nullptr, *g = nullptr;  // fp32 master, Adam, grad
  bf16* wb = nullptr;                                            // bf16 copy of w
  bf16* wflip = nullptr;  // flipped, transposed weights of a decoder layer (its data gradient)
  bf16* wfold[2] = {nullptr, nullptr};  // folded weights of the upsampling layers L4, L5
  long long step = 0;
  int cap_b = 0;
  // activations and workspaces (sized for cap_b)
  bf16 *x0 = nullptr, *a[5] = {nullptr}, *col = nullptr, *dzb = nullptr;
  float *y = nullptr, *dy = nullptr,
        *da[5] = {nullptr}, *part = nullptr, *w6 = nullptr, *w6f = nullptr, *w1 = nullptr;
  double* lpart = nullptr;
  size_t part_floats = 0;
};

}  // namespace pprs_cnn_impl

struct pprs_cnn {
  pprs_cnn_impl::Model M;
};

using pprs_cnn_impl::Layer;
using pprs_cnn_impl::Model;

static thread_local std::string g_cnn_err;

static pprs_status cfail(pprs_status s, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_cnn_err = buf;
  return s;
}

#define CHK(expr)                                                                     \
  do {                                                                                \
    hipError_t e_ = (expr);                                                           \
    if (e_ != hipSuccess)                                                             \
      return cfail(PPRS_EHIP, "%s: %s (%s:%d)", #expr, hipGetErrorString(e_), __FILE__, \
                   __LINE__);                                                         \
  } while (0)

static pprs_status gemm(Model& M, const bf16* A, int lda, const bf16* B, int ldb,
                         float* C, int ldc, int Mr, int Nc, int K, int splits) {
  if (Mr % 64 || Nc % 64 || K % 32 || lda % 8 || ldb % 8)
    return cfail(PPRS_EINVAL, "gemm shape %d x %d x %d not tileable", Mr, Nc, K);
  int kps = ((K / 32 + splits - 1) / splits) * 32;
  splits = (K + kps - 1) / kps;
  float* out = C;
  long long stride = (long long)Mr * ldc;
  if (splits > 1) {
    if ((size_t)splits * stride > M.part_floats)
      return cfail(PPRS_EINVAL, "split-K workspace too small");
    out = M.part;
  }
  dim3 grid(Nc / 64, Mr / 64, splits);
  hipLaunchKernelGGL(k_gemm, grid, dim3(256), 0, M.stream, A, lda, B, ldb, out, ldc, K, kps, stride);
  CHK(hipGetLastError());
  if (splits > 1) {
    hipLaunchKernelGGL(k_split_sum, dim3((unsigned)(stride / 64)), dim3(256), 0, M.stream, M.part,
                       stride, splits, C);
    CHK(hipGetLastError());
  }
  return PPRS_OK;
}

static void define_layers(Model& M) {
  const int cin[6] = {2, 64, 128, 384, 192, 66}, cout[6] = {64, 128, 256, 128, 64, 2};
  const int stride[6] = {2, 2, 2, 1, 1, 1}, hin[6] = {128, 64, 32, 32, 64, 128};
  long long off = 0;
  for (int l = 0; l < 6; ++l) {
    Layer& y = M.L[l];
    y.cin = cin[l];
    y.cout = cout[l];
    y.stride = stride[l];
    y.hin = hin[l];
    y.hout = hin[l] / stride[l];
    int k = 9 * cin[l];
    y.kp = l == 0 ? 64 : (l == 5 ? k : ((k + 31) / 32) * 32);
    y.woff = off;
    off += (long long)y.cout * y.kp;
    y.boff = off;
    off += y.cout;
  }
  M.n_params = off;
}

// Floats of the partials' buffer for B samples, one user at a time: k_wgrad's pixel shares (up to
// 512 workgroups of 64 x 64 x 9 results, 19 M floats; wgrad takes no more shares than fit), the
// first layer's GEMM (512 splits of 64 x 64), k_relu_bwd's column sums (1024 x 256) and k_l6_bwd_w's
// (one record per workgroup, the only one that grows with the batch). 64 times the largest weight, 28
// M floats, holds the first three.
static size_t partial_floats(const Model& M, int B) {
  long long wmax = 0;
  for (int l = 0; l < 5; ++l) wmax = std::max(wmax, (long long)M.L[l].cout * M.L[l].kp);
  return (size_t)std::max(64 * wmax, (long long)B * (64 / L6T) * (64 / L6T) * (2 * 9 * L6C + 2));
}

// The buffers that follow from the batch, and their sizes for B samples.
struct BatchBuf {
  void** p;
  size_t bytes;
};
static std::vector<BatchBuf> batch_bufs(Model& M, int B) {
  const long long P128 = (long long)B * 128 * 128, P64 = P128 / 4, P32 = P128 / 16, P16 = P128 / 64;
  long long col_max = 0, z_max = 0, wf = 0;
  for (int l = 0; l < 5; ++l) {
    long long pix = (long long)B * M.L[l].hout * M.L[l].hout;
    if (l == 0) col_max = pix * M.L[l].kp;  // the first layer's weight gradient
    z_max = std::max(z_max, pix * (long long)M.L[l].cout);
  }
  for (int l = 3; l < 5; ++l) wf = std::max(wf, (long long)M.L[l].cin * 9 * M.L[l].cout);
  return {{(void**)&M.x0, sizeof(bf16) * P128 * 2},      {(void**)&M.a[0], sizeof(bf16) * P64 * 64},
          {(void**)&M.a[1], sizeof(bf16) * P32 * 128},   {(void**)&M.a[2], sizeof(bf16) * P16 * 256},
          {(void**)&M.a[3], sizeof(bf16) * P32 * 128},   {(void**)&M.a[4], sizeof(bf16) * P64 * 64},
          {(void**)&M.wflip, sizeof(bf16) * wf},         {(void**)&M.col, sizeof(bf16) * col_max},
          {(void**)&M.dzb, sizeof(bf16) * z_max},        {(void**)&M.y, sizeof(float) * P128 * 2},
          {(void**)&M.dy, sizeof(float) * P128 * 2},     {(void**)&M.da[0], sizeof(float) * P64 * 64},
          {(void**)&M.da[1], sizeof(float) * P32 * 128}, {(void**)&M.da[2], sizeof(float) * P16 * 256},
          {(void**)&M.da[3], sizeof(float) * P32 * 128}, {(void**)&M.da[4], sizeof(float) * P64 * 64},
          {(void**)&M.part, sizeof(float) * partial_floats(M, B)},
          {(void**)&M.lpart, sizeof(double) * 1024}};
}
static void free_batch(Model& M) {
  for (const BatchBuf& x : batch_bufs(M, 0)) {
    if (*x.p) (void)hipFree(*x.p);
    *x.p = nullptr;
  }
  M.cap_b = 0;
}

// Buffers for B samples. Where they cannot be had the network holds none: no pointer to freed
// memory stays behind, and the next call allocates what it needs.
static pprs_status alloc_batch(Model& M, int B) {
  if (B <= M.cap_b) return PPRS_OK;
  free_batch(M);
  for (const BatchBuf& x : batch_bufs(M, B)) {
    hipError_t e = hipMalloc(x.p, x.bytes);
    if (e != hipSuccess) {
      (void)hipGetLastError();
      *x.p = nullptr;
      free_batch(M);
      return cfail(PPRS_EHIP, "hipMalloc(%zu) for %d samples: %s", x.bytes, B, hipGetErrorString(e));
    }
  }
  M.part_floats = partial_floats(M, B);
  M.cap_b = B;
  return PPRS_OK;
}

// Launches k_conv_fwd over `pix` output pixels. The tile is the largest that still gives the 256
// compute units two workgroups each: 256 pixels x 64 channels or 128 x 128 (64 accumulator
// registers a lane; 256 x 128 takes 128 and leaves one wavefront per SIMD: L4 of 511 pairs 435
// us against 401; 128 x 64 for L5 693 us against 668), and fewer pixels where the batch is small
// (one pair: L3 is 256 pixels in all; forward of one pair 97 us with 64 pixels, 202 us before).
template <bool DGRAD, bool FOLD, bool S2>
static pprs_status conv_launch(Model& M, const bf16* s0, int c0, const bf16* s1, int c1, int hin,
                               int stride, const bf16* w, int kp, const float* b, int cout,
                               long long pix, void* out, float* out2 = nullptr) {
  const int bn = cout % 128 == 0 ? 128 : 64;
  const long long unit = FOLD || S2 ? pix / 4 : pix;  // pixels that a tile may not straddle
  if (unit % 64 || c0 % 64 || c1 % 64 || kp % 8 || cout % bn || (hin & (hin - 1)) ||
      (DGRAD && c1 % bn) || (S2 && c0 % 128))
    return cfail(PPRS_EINVAL, "convolution of %d + %d to %d channels does not fit its tiles", c0, c1,
                 cout);
  // S2 keeps a second set of sums in registers, so half the tile
  int mt = (bn == 128 ? 2 : 4) / (S2 ? 2 : 1);
  while (mt > 1 && (unit % (64 * mt) || pix / (64 * mt) * (cout / bn) < 512)) mt /= 2;
  dim3 grid((unsigned)(pix / (64 * mt)), cout / bn);
#define CONV(MT, BN)                                                                           \
  hipLaunchKernelGGL((k_conv_fwd<MT, BN, DGRAD, FOLD, S2>), grid, dim3(256), 0, M.stream, s0, c0, s1, \
                     c1, hin, stride, w, kp, b, cout, out, out2)
  if (bn == 128) {
    if constexpr (!S2)
      if (mt == 2) CONV(2, 128);
    if (mt == 1) CONV(1, 128);
  } else {
    if constexpr (!S2)
      if (mt == 4) CONV(4, 64);
    if (mt == 2) CONV(2, 64);
    else if (mt == 1) CONV(1, 64);
  }
#undef CONV
  CHK(hipGetLastError());
  return PPRS_OK;
}

// Fused convolution of layer l (L2..L5) into M.a[l].
static pprs_status conv_fused(Model& M, int l, int B) {
  const Layer& y = M.L[l];
  const bf16* s0 = l == 1 ? M.a[0] : l == 2 ? M.a[1] : l == 3 ? M.a[2] : M.a[3];
  const bf16* s1 = l == 3 ? M.a[1] : l == 4 ? M.a[0] : nullptr;
  int c0 = l == 1 ? 64 : l == 2 ? 128 : l == 3 ? 256 : 128;
  int c1 = y.cin - c0;
  long long pix = (long long)B * y.hout * y.hout;
  const float* b = M.w + y.boff;
  if (l >= 3)
    // folded upsampling: per output parity, 4 C0 + 9 C1 deep (pixels of one parity per tile)
    return conv_launch<false, true, false>(M, s0, c0, s1, c1, y.hin, y.stride, M.wfold[l - 3],
                                    4 * c0 + 9 * c1, b, y.cout, pix, M.a[l]);
  return conv_launch<false, false, false>(M, s0, c0, s1, c1, y.hin, y.stride, M.wb + y.woff, y.kp, b,
                                   y.cout, pix, M.a[l]);
}

// Forward pass for B samples; input x [B][128][128][2] fp32; output in M.y.
static pprs_status forward(Model& M, const float* x, int B) {
  hipStream_t st = M.stream;
  long long P128 = (long long)B * 128 * 128;
  hipLaunchKernelGGL(k_f32_to_bf16, dim3(grid1d(P128 * 2)), dim3(kBlock), 0, st, x, P128 * 2, M.x0);
  {
    // L1 (2 input channels): a direct kernel (18 products per output channel)
    const Layer& y = M.L[0];
    long long pix = (long long)B * y.hout * y.hout;
    hipLaunchKernelGGL(k_l1_direct, dim3(grid1d(pix)), dim3(kBlock), 0, st, M.x0, M.w1, M.w + y.boff, B, M.a[0]);
  }
  for (int l = 1; l < 5; ++l) {
    pprs_status s = conv_fused(M, l, B);
    if (s != PPRS_OK) return s;
  }
  // L6
  const Layer& y6 = M.L[5];
  // four samples per workgroup where that still leaves 16 workgroups per CU (328 us for 511
  // pairs, 400 one by one); the sums are the same
  if (B >= 32)
    hipLaunchKernelGGL(k_l6_fused<4>, dim3(512 * std::min((B + 3) / 4, 32)), dim3(kBlock), 0, st,
                       M.a[4], M.x0, M.w6, M.w6f, M.w + y6.boff, B, M.y);
  else
    hipLaunchKernelGGL(k_l6_fused<1>, dim3(512 * B), dim3(kBlock), 0, st, M.a[4], M.x0, M.w6,
                       M.w6f, M.w + y6.boff, B, M.y);
  CHK(hipGetLastError());
  return PPRS_OK;
}

// fp32 view of the L6 weights from the bf16 copy (so every layer computes with bf16 weights).
// Weight copies derived from the BF16 weights, remade whenever they change: L1's and L6's FP32 copies
// and the folded weights of the upsampling layers L4 and L5.
static pprs_status refresh_derived(Model& M) {
  const Layer& y6 = M.L[5];
  hipLaunchKernelGGL(k_w6_prep, dim3(1), dim3(kBlock), 0, M.stream, M.wb + y6.woff, M.w6, M.w6f);
  hipLaunchKernelGGL(k_w1_prep, dim3(1), dim3(kBlock), 0, M.stream, M.wb + M.L[0].woff, M.L[0].kp, M.w1);
  for (int l = 3; l < 5; ++l) {
    const Layer& y = M.L[l];
    const int c0 = l == 3 ? 256 : 128, c1 = y.cin - c0;
    hipLaunchKernelGGL(k_fold_weights, dim3(grid1d(4LL * y.cout * (4 * c0 + 9 * c1))), dim3(kBlock), 0, M.stream, M.wb + y.woff, y.cout, c0, c1, y.kp, M.wfold[l - 3]);
  }
  CHK(hipGetLastError());
  return PPRS_OK;
}

// Weight gradient of layer l (L2..L5) into M.g: enough pixel shares for two workgroups per compute
// unit, as far as the partials' workspace and 64-pixel units go round.
static pprs_status wgrad(Model& M, int l, int B) {
  const Layer& y = M.L[l];
  const bf16* s0 = l == 1 ? M.a[0] : l == 2 ? M.a[1] : l == 3 ? M.a[2] : M.a[3];
  const bf16* s1 = l == 3 ? M.a[1] : l == 4 ? M.a[0] : nullptr;
  const int c0 = l == 1 ? 64 : l == 2 ? 128 : l == 3 ? 256 : 128, c1 = y.cin - c0;
  const int units = B * y.hout * y.hout / 64;
  const long long size = (long long)y.cout * 9 * y.cin;
  const int blocks = (y.cin / 64) * (y.cout / 64);
  int splits = std::max(1, std::min({512 / blocks, units, (int)(M.part_floats / size)}));
  const int per = (units + splits - 1) / splits;
  splits = (units + per - 1) / per;
  float* out = splits > 1 ? M.part : M.g + y.woff;
  dim3 grid(y.cin / 64, y.cout / 64, splits);
  if (l == 1) hipLaunchKernelGGL((k_wgrad<2, 5, false>), grid, dim3(256), 0, M.stream, M.dzb, y.cout, s0, c0, s1, c1, units, per, out);
  else if (l == 2) hipLaunchKernelGGL((k_wgrad<2, 4, false>), grid, dim3(256), 0, M.stream, M.dzb, y.cout, s0, c0, s1, c1, units, per, out);
  else if (l == 3) hipLaunchKernelGGL((k_wgrad<1, 5, true>), grid, dim3(256), 0, M.stream, M.dzb, y.cout, s0, c0, s1, c1, units, per, out);
  else hipLaunchKernelGGL((k_wgrad<1, 6, true>), grid, dim3(256), 0, M.stream, M.dzb, y.cout, s0, c0, s1, c1, units, per, out);
  CHK(hipGetLastError());
  if (splits > 1) {
    hipLaunchKernelGGL(k_split_sum, dim3((unsigned)(size / 64)), dim3(256), 0, M.stream, M.part, size, splits, M.g + y.woff);
    CHK(hipGetLastError());
  }
  return PPRS_OK;
}

// Loss and full gradient into M.g (uses M.y from forward). Returns the mean squared error.
static pprs_status backward(Model& M, const float* target, int B, int margin, double* loss) {
  hipStream_t st = M.stream;
  int interior = 128 - 2 * margin;
  float inv_count = 1.f / ((float)B * interior * interior * 2);
  int blocks = 1024;
  hipLaunchKernelGGL(k_mse, dim3(blocks), dim3(kBlock), 0, st, M.y, target, B, 128, 128, margin, inv_count, M.dy, M.lpart);
  std::vector<double> hp(blocks);
  CHK(hipMemcpyAsync(hp.data(), M.lpart, sizeof(double) * blocks, hipMemcpyDeviceToHost, st));
  CHK(hipMemsetAsync(M.g, 0, sizeof(float) * M.n_params, st));
  // L6: dW6, db6, dU6
  const Layer& y6 = M.L[5];
  {
    int nw = 2 * 9 * 66 + 2, chunks = B * (64 / L6T) * (64 / L6T);
    hipLaunchKernelGGL(k_l6_bwd_w, dim3(chunks), dim3(256), 0, st, M.dy, M.a[4], M.x0, M.part);
    // weights [2][9*66] then bias [2] are contiguous at woff: columns 0..nw-1 map to them
    hipLaunchKernelGGL(k_colsum_final, dim3(nw), dim3(kBlock), 0, st, M.part, nw, chunks, M.g + y6.woff);
    // d a[4] through the folded weights (the input part needs no gradient)
    hipLaunchKernelGGL(k_l6_bwd_a5, dim3(chunks), dim3(256), 0, st, M.dy, M.w6f, M.da[4]);
  }
  CHK(hipGetLastError());
  // L5 .. L1
  for (int l = 4; l >= 0; --l) {
    const Layer& y = M.L[l];
    long long pix = (long long)B * y.hout * y.hout;
    // dZ = dA * relu'(A) and the bias gradient
    const int blocks_z = 1024;
    hipLaunchKernelGGL(k_relu_bwd, dim3(blocks_z), dim3(kBlock), 0, st, M.da[l], M.a[l], pix, y.cout, M.dzb, M.part);
    hipLaunchKernelGGL(k_colsum_final, dim3(y.cout), dim3(kBlock), 0, st, M.part, y.cout, blocks_z, M.g + y.boff);
    CHK(hipGetLastError());
    // weight gradient: dW[co][k] = sum_pix dZ[pix][co] col[pix][k]
    pprs_status s;
    if (l > 0) {
      s = wgrad(M, l, B);
    } else {
      hipLaunchKernelGGL(k_im2col2, dim3(grid1d(pix * y.kp / 8)), dim3(kBlock), 0, st, M.x0, B, y.hin, y.hin, y.stride, y.kp, M.col);
      // one 64 x 64 result: the splits alone fill the GPU (64 of them: 129 us for 64 samples)
      int splits = (int)std::max<long long>(1, std::min<long long>(512, pix / 256));
      s = gemm(M, M.dzb, y.cout, M.col, y.kp, M.g + y.woff, y.kp, y.cout, y.kp, (int)pix, splits);
    }
    if (s != PPRS_OK) return s;
    if (l == 0) break;
    if (l == 4 || l == 3) {
      // data gradient of the stride-1 decoder layers as a convolution of dZ with the flipped,
      // transposed weights (implicit GEMM, no materialised columns), straight to its two sources
      hipLaunchKernelGGL(k_flip_weights, dim3(grid1d((long long)y.cin * 9 * y.cout)), dim3(kBlock), 0, st, M.wb + y.woff, y.cout, y.cin, y.kp, M.wflip);
      // input [up2(a[l - 1]), a[4 - l]]: u5 = [a4 128, a1 64] at 64^2, u4 = [a3 256, a2 128] at 32^2
      const int up = M.L[l - 1].cout;
      s = conv_launch<true, false, false>(M, M.dzb, y.cout, nullptr, up, y.hout, 1, M.wflip, 9 * y.cout,
                                   nullptr, y.cin, pix, M.da[l - 1], M.da[4 - l]);
      if (s != PPRS_OK) return s;
      CHK(hipGetLastError());
      continue;
    }
    // data gradient of the stride-2 layers, added to the skip connection's gradient that a[l - 1]'s
    // already holds
    hipLaunchKernelGGL(k_flip_weights, dim3(grid1d((long long)y.cin * 9 * y.cout)), dim3(kBlock), 0, st, M.wb + y.woff, y.cout, y.cin, y.kp, M.wflip);
    s = conv_launch<false, false, true>(M, M.dzb, y.cout, nullptr, 0, y.hout, 1, M.wflip,
                                        9 * y.cout, nullptr, y.cin, 4 * pix, M.da[l - 1]);
    if (s != PPRS_OK) return s;
    CHK(hipGetLastError());
  }
  CHK(hipStreamSynchronize(st));
  double sum = 0.0;
  for (int i = 0; i < blocks; ++i) sum += hp[i];
  if (loss) *loss = sum / ((double)B * interior * interior * 2);
  return PPRS_OK;
}

// ------------------------------------------------------------------------------------------
// Weights-only blob (safetensors layout): u64 little-endian header length, a JSON object
// {"name": {"dtype": ..., "shape": [...], "data_offsets": [begin, end]}, "__metadata__": {...}},
// then the tensor bytes. A small recursive-descent reader of that JSON: it accepts objects,
// arrays, strings, numbers and literals, records each top-level tensor's fields and skips
// everything else. Nothing in the blob is interpreted beyond these fields.

namespace {

struct BlobTensor {
  std::string name, dtype;
  std::vector<long long> shape;
  long long begin = -1, end = -1;
};

struct JsonReader {
  const char* p;
  const char* e;
  int depth = 0;
  bool ok = true;
  void ws() {
    while (p < e && (*p == ' ' || *p == '\n' || *p == '\r' || *p == '\t')) ++p;
  }
  bool eat(char ch) {
    ws();
    if (p < e && *p == ch) {
      ++p;
      return true;
    }
    return false;
  }
  bool str(std::string* out) {
    ws();
    if (p >= e || *p != '"') return ok = false;
    ++p;
    std::string r;
    while (p < e && *p != '"') {
      if (*p == '\\') {
        if (++p >= e) return ok = false;
        char c = *p;
        if (c == 'u') {  // keep the escape's text; names here are plain ASCII
          if (e - p < 5) return ok = false;
          r.append(p - 1, 6);
          p += 5;
          continue;
        }
        r.push_back(c == 'n' ? '\n' : c == 't' ? '\t' : c == 'r' ? '\r' : c == 'b' ? '\b'
                    : c == 'f' ? '\f' : c);
        ++p;
        continue;
      }
      r.push_back(*p++);
    }
    if (p >= e) return ok = false;
    ++p;
    if (out) *out = r;
    return true;
  }
  bool integer(long long* out) {
    ws();
    const char* q = p;
    bool neg = false;
    if (q < e && *q == '-') neg = true, ++q;
    if (q >= e || *q < '0' || *q > '9') return ok = false;
    long long v = 0;
    while (q < e && *q >= '0' && *q <= '9') {
      if (v > (1LL << 50)) return ok = false;
      v = v * 10 + (*q++ - '0');
    }
    if (q < e && (*q == '.' || *q == 'e' || *q == 'E')) return ok = false;
    p = q;
    *out = neg ? -v : v;
    return true;
  }
  bool skip() {  // any value
    ws();
    if (p >= e || ++depth > 64) return ok = false;
    bool r = true;
    if (*p == '"') {
      r = str(nullptr);
    } else if (*p == '{') {
      ++p;
      if (!eat('}')) {
        do {
          r = str(nullptr) && eat(':') && skip();
        } while (r && eat(','));
        r = r && eat('}');
      }
    } else if (*p == '[') {
      ++p;
      if (!eat(']')) {
        do {
          r = skip();
        } while (r && eat(','));
        r = r && eat(']');
      }
    } else {
      const char* q = p;
      while (q < e && (isalnum((unsigned char)*q) || *q == '-' || *q == '+' || *q == '.')) ++q;
      r = q > p;
      p = q;
    }
    --depth;
    if (!r) ok = false;
    return r;
  }
  bool int_list(std::vector<long long>* out) {
    if (!eat('[')) return ok = false;
    out->clear();
    if (eat(']')) return true;
    do {
      long long v;
      if (!integer(&v)) return false;
      out->push_back(v);
    } while (eat(','));
    return eat(']') || (ok = false);
  }
  bool tensor(BlobTensor* t) {
    if (!eat('{')) return ok = false;
    if (eat('}')) return true;
    do {
      std::string key;
      if (!str(&key) || !eat(':')) return ok = false;
      if (key == "dtype") {
        if (!str(&t->dtype)) return false;
      } else if (key == "shape") {
        if (!int_list(&t->shape)) return false;
      } else if (key == "data_offsets") {
        std::vector<long long> o;
        if (!int_list(&o) || o.size() != 2) return ok = false;
        t->begin = o[0];
        t->end = o[1];
      } else if (!skip()) {
        return false;
      }
    } while (eat(','));
    return eat('}') || (ok = false);
  }
};

bool parse_blob_header(const char* h, size_t n, std::vector<BlobTensor>& out) {
  JsonReader r{h, h + n};
  if (!r.eat('{')) return false;
  if (r.eat('}')) return true;
  do {
    std::string key;
    if (!r.str(&key) || !r.eat(':')) return false;
    if (key == "__metadata__") {
      if (!r.skip()) return false;
      continue;
    }
    BlobTensor t;
    t.name = key;
    if (!r.tensor(&t)) return false;
    out.push_back(t);
  } while (r.eat(','));
  return r.eat('}') && r.ok;
}

}  // namespace

// ------------------------------------------------------------------------------------------
// C-ABI

extern "C" {

const char* pprs_cnn_last_error(void) { return g_cnn_err.c_str(); }

pprs_status pprs_cnn_create(pprs_cnn** out, int device, void* stream, unsigned long long seed) {
  if (!out) return cfail(PPRS_EINVAL, "out is NULL");
  *out = nullptr;
  CHK(hipSetDevice(device));
  pprs_cnn* c = new pprs_cnn();
  Model& M = c->M;
  M.device = device;
  M.stream = (hipStream_t)stream;
  define_layers(M);
  // He-normal initialisation from a counter-based hash (SplitMix64) of (seed, index)
  std::vector<float> hw(M.n_params, 0.f);
  auto mix = [](unsigned long long x) {
    x += 0x9E3779B97F4A7C15ULL;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ULL;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBULL;
    return x ^ (x >> 31);
  };
  for (int l = 0; l < 6; ++l) {
    const Layer& y = M.L[l];
    int k = 9 * y.cin;
    double sd = sqrt(2.0 / k) * (l == 5 ? 0.1 : 1.0);
    for (int co = 0; co < y.cout; ++co)
      for (int j = 0; j < k; ++j) {
        long long i = y.woff + (long long)co * y.kp + j;
        unsigned long long r1 = mix(seed * 0x100000001B3ULL + 2 * (unsigned long long)i);
        unsigned long long r2 = mix(seed * 0x100000001B3ULL + 2 * (unsigned long long)i + 1);
        double u1 = ((r1 >> 11) + 0.5) / 9007199254740992.0, u2 = (r2 >> 11) / 9007199254740992.0;
        hw[i] = (float)(sd * sqrt(-2.0 * log(u1)) * cos(6.283185307179586 * u2));
      }
  }
  hipError_t e = hipSuccess;
  e = hipMalloc(&M.w, sizeof(float) * M.n_params);
  if (e == hipSuccess) e = hipMalloc(&M.m, sizeof(float) * M.n_params);
  if (e == hipSuccess) e = hipMalloc(&M.v, sizeof(float) * M.n_params);
  if (e == hipSuccess) e = hipMalloc(&M.g, sizeof(float) * M.n_params);
  if (e == hipSuccess) e = hipMalloc(&M.wb, sizeof(bf16) * M.n_params);
  if (e == hipSuccess) e = hipMalloc(&M.w6, sizeof(float) * M.L[5].cout * M.L[5].kp);
  if (e == hipSuccess) e = hipMalloc(&M.w1, sizeof(float) * 18 * 64);
  if (e == hipSuccess) e = hipMalloc(&M.w6f, sizeof(float) * 4 * 2 * 2 * 2 * 64);
  for (int l = 3; l < 5 && e == hipSuccess; ++l) {
    const int c0 = l == 3 ? 256 : 128, c1 = M.L[l].cin - c0;
    e = hipMalloc(&M.wfold[l - 3], sizeof(bf16) * 4 * M.L[l].cout * (4 * c0 + 9 * c1));
  }
  if (e != hipSuccess) {
    (void)hipGetLastError();
    pprs_cnn_destroy(c);
    return cfail(PPRS_ENOMEM, "cnn allocation failed");
  }
  *out = c;
  pprs_status s = pprs_cnn_set_params(c, hw.data(), (size_t)M.n_params);
  return s;
}

void pprs_cnn_destroy(pprs_cnn* c) {
  if (!c) return;
  Model& M = c->M;
  (void)hipSetDevice(M.device);
  (void)hipStreamSynchronize(M.stream);
  free_batch(M);
  void* ptrs[] = {M.w, M.m, M.v, M.g, M.wb, M.w1, M.w6, M.w6f, M.wfold[0], M.wfold[1]};
  for (void* p : ptrs)
    if (p) (void)hipFree(p);
  delete c;
}

size_t pprs_cnn_param_count(const pprs_cnn* c) { return c ? (size_t)c->M.n_params : 0; }

pprs_status pprs_cnn_set_params(pprs_cnn* c, const float* host, size_t count) {
  if (!c || !host) return cfail(PPRS_EINVAL, "NULL argument");
  Model& M = c->M;
  if (count != (size_t)M.n_params) return cfail(PPRS_EINVAL, "expected %lld parameters", M.n_params);
  CHK(hipSetDevice(M.device));
  CHK(hipMemcpyAsync(M.w, host, sizeof(float) * count, hipMemcpyHostToDevice, M.stream));
  CHK(hipMemsetAsync(M.m, 0, sizeof(float) * count, M.stream));
  CHK(hipMemsetAsync(M.v, 0, sizeof(float) * count, M.stream));
  hipLaunchKernelGGL(k_f32_to_bf16, dim3(grid1d(count)), dim3(kBlock), 0, M.stream, M.w, (long long)count, M.wb);
  CHK(hipGetLastError());
  M.step = 0;
  return refresh_derived(M);
}

pprs_status pprs_cnn_load(pprs_cnn* c, const void* blob, size_t bytes) {
  if (!c || !blob) return cfail(PPRS_EINVAL, "NULL argument");
  const unsigned char* b = (const unsigned char*)blob;
  if (bytes < 8) return cfail(PPRS_EINVAL, "blob shorter than its 8-byte header length");
  unsigned long long hl = 0;
  for (int k = 7; k >= 0; --k) hl = (hl << 8) | b[k];
  if (hl < 2 || hl > bytes - 8) return cfail(PPRS_EINVAL, "header length %llu outside the blob", hl);
  std::vector<BlobTensor> ts;
  if (!parse_blob_header((const char*)b + 8, (size_t)hl, ts))
    return cfail(PPRS_EINVAL, "malformed blob header");
  const BlobTensor* t = nullptr;
  for (const BlobTensor& x : ts)
    if (x.name == "params") t = &x;
  if (!t && ts.size() == 1) t = &ts[0];
  if (!t) return cfail(PPRS_EINVAL, "blob holds no tensor named \"params\"");
  if (t->dtype != "F32") return cfail(PPRS_EINVAL, "tensor dtype %s, expected F32", t->dtype.c_str());
  long long count = 1;
  for (long long d : t->shape) {
    if (d < 0 || d > (1LL << 40)) return cfail(PPRS_EINVAL, "bad tensor shape");
    count *= d;
  }
  Model& M = c->M;
  if (count != M.n_params)
    return cfail(PPRS_EINVAL, "blob holds %lld parameters, the network %lld", count, M.n_params);
  size_t data = 8 + (size_t)hl, avail = bytes - data;
  if (t->begin < 0 || t->end < t->begin || (unsigned long long)t->end > avail ||
      t->end - t->begin != 4 * count)
    return cfail(PPRS_EINVAL, "tensor byte range outside the blob");
  std::vector<float> host((size_t)count);  // aligned copy: the data need not be aligned
  memcpy(host.data(), b + data + t->begin, sizeof(float) * (size_t)count);
  pprs_status s = pprs_cnn_set_params(c, host.data(), (size_t)count);
  if (s != PPRS_OK) return s;
  CHK(hipStreamSynchronize(M.stream));  // the host copy must outlive the upload
  return PPRS_OK;
}

pprs_status pprs_cnn_get_params(pprs_cnn* c, float* host, size_t count) {
  if (!c || !host) return cfail(PPRS_EINVAL, "NULL argument");
  Model& M = c->M;
  if (count != (size_t)M.n_params) return cfail(PPRS_EINVAL, "expected %lld parameters", M.n_params);
  CHK(hipSetDevice(M.device));
  CHK(hipMemcpyAsync(host, M.w, sizeof(float) * count, hipMemcpyDeviceToHost, M.stream));
  CHK(hipStreamSynchronize(M.stream));
  return PPRS_OK;
}

pprs_status pprs_cnn_forward(pprs_cnn* c, const float* x, int B, float* y) {
  if (!c || !x || !y || B < 1) return cfail(PPRS_EINVAL, "bad arguments");
  Model& M = c->M;
  CHK(hipSetDevice(M.device));
  pprs_status s = alloc_batch(M, B);
  if (s != PPRS_OK) return s;
  s = forward(M, x, B);
  if (s != PPRS_OK) return s;
  CHK(hipMemcpyAsync(y, M.y, sizeof(float) * (size_t)B * 128 * 128 * 2, hipMemcpyDeviceToDevice, M.stream));
  CHK(hipStreamSynchronize(M.stream));
  return PPRS_OK;
}

pprs_status pprs_cnn_gradients(pprs_cnn* c, const float* x, const float* target, int B,
                               int margin, double* loss, float* grad_host) {
  if (!c || !x || !target || B < 1 || margin < 0 || margin >= 64)
    return cfail(PPRS_EINVAL, "bad arguments");
  Model& M = c->M;
  CHK(hipSetDevice(M.device));
  pprs_status s = alloc_batch(M, B);
  if (s != PPRS_OK) return s;
  if ((s = forward(M, x, B)) != PPRS_OK) return s;
  if ((s = backward(M, target, B, margin, loss)) != PPRS_OK) return s;
  if (grad_host) {
    CHK(hipMemcpyAsync(grad_host, M.g, sizeof(float) * M.n_params, hipMemcpyDeviceToHost, M.stream));
    CHK(hipStreamSynchronize(M.stream));
  }
  return PPRS_OK;
}

pprs_status pprs_cnn_train_step(pprs_cnn* c, const float* x, const float* target, int B,
                                int margin, float lr, double* loss) {
  pprs_status s = pprs_cnn_gradients(c, x, target, B, margin, loss, nullptr);
  if (s != PPRS_OK) return s;
  Model& M = c->M;
  M.step++;
  const float b1 = 0.9f, b2 = 0.999f;
  float c1 = 1.f - powf(b1, (float)M.step), c2 = 1.f - powf(b2, (float)M.step);
  hipLaunchKernelGGL(k_adam, dim3(grid1d(M.n_params)), dim3(kBlock), 0, M.stream, M.w, M.m, M.v, M.g, M.n_params, lr, b1, b2, 1e-8f, c1, c2, M.wb);
  CHK(hipGetLastError());
  return refresh_derived(M);
}

}  // extern "C"

// Used by the runtime: pack pairs of level-7 frames and run the network.
namespace pprs_cnn_api {
hipError_t pack_pairs(const float* lvl, int n, const int* ref, const int* tmpl, int P,
                      float* out, hipStream_t st) {
  long long work = (long long)P * (n - 1) * (n - 1);
  hipLaunchKernelGGL(k_pack_pairs, dim3(grid1d(work)), dim3(kBlock), 0, st, lvl, n, ref, tmpl, P, out);
  return hipGetLastError();
}
pprs_status forward_into(pprs_cnn* c, const float* x, int B, float* y) {
  return pprs_cnn_forward(c, x, B, y);
}
hipError_t planes_to_nhwc(const float* src, int n, long long pstride, int P, float scale,
                          float* out, hipStream_t st) {
  long long work = (long long)P * (n - 1) * (n - 1);
  hipLaunchKernelGGL(k_planes_to_nhwc, dim3(grid1d(work)), dim3(kBlock), 0, st, src, n, pstride, P, scale, out);
  return hipGetLastError();
}
hipError_t nhwc_to_planes(const float* y, int S, int P, float scale, float* base,
                          long long stride, hipStream_t st) {
  long long work = (long long)P * (S + 1) * (S + 1);
  hipLaunchKernelGGL(k_nhwc_to_planes, dim3(grid1d(work)), dim3(kBlock), 0, st, y, S, P, scale, base, stride);
  return hipGetLastError();
}
int cnn_device(const pprs_cnn* c) { return c->M.device; }
hipError_t check_pred(const float* y, int P, long long n_per, float limit, int* bad,
                      hipStream_t st) {
  hipLaunchKernelGGL(k_check_pred, dim3(P), dim3(kBlock), 0, st, y, n_per, limit, bad);
  return hipGetLastError();
}
}  // namespace pprs_cnn_api
