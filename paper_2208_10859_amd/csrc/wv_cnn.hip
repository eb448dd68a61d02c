// Restoration network on decoded viewports: four 3x3 convolutions (3 -> 32
// -> 32 -> 32 -> 3), ReLU after the first three, residual skip.  Forward,
// backward and the optimiser step are hand-written kernels; the convolutions
// are implicit GEMMs on bfloat16 MFMA (v_mfma_f32_16x16x32_bf16) with fp32
// accumulation.  Images and activations are NHWC; three-channel images are
// stored with a fourth zero channel so that a pixel is 8 bytes.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <cstring>

#include "wv_cnn.h"
#include "wv_ctx.h"
#include "wv_dev.h"

namespace wv {
namespace cnn {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int HID = 32;

// float -> bfloat16, round to nearest, ties to even (finite values)
__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }


// Convolutions are implicit GEMMs on gfx950's v_mfma_f32_16x16x32_bf16: M =
// output channels (16 per MFMA), N = pixels (16 consecutive columns of one
// row), K = 9 taps x input channels, tap-major, padded to a multiple of 32.
// For 32 input channels one K step is one tap; for 4 it is 8 taps.  MFMA
// 16x16x32 operands: lane l supplies A[l % 16][8 (l / 16) + q] and
// B[8 (l / 16) + q][l % 16], q = 0..7 (any pairing of K positions works as long
// as A and B use the same one), and receives D[4 (l / 16) + q][l % 16]: four
// consecutive output channels of one pixel, stored as one 8-byte write.
constexpr int kpad32(int cin) { return (9 * cin + 31) / 32 * 32; }

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ bf8 as_bf8(uint4 v) { return __builtin_bit_cast(bf8, v); }

// Two floats to a packed bfloat16 pair, rounded to nearest even (one
// v_cvt_pk_bf16_f32; the same result as f2bf for finite values).
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef float f2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pk_bf16(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2v{a, b}, bf2));
}

// Backward pass of a layer with 32 input channels: its weight and bias
// gradients, dW[o][tap][i] = sum over pixels of dy[p][o] x[p + tap offset][i], as a
// GEMM with M = output channels, N = taps x input channels, K = pixels; and the
// gradient of its input dx (the convolution of dy with the flipped, transposed
// kernel, masked by the ReLU that made the input x: dx = bf16(x > 0 ? sum : 0)).
// Both need the block of x and of dy with a border, so one kernel stages them
// once; of its eight waves four compute each, one of either kind on every SIMD.
// A workgroup stages 16 x 32 pixel blocks, the next one's global reads under way
// while one is multiplied.  The staged pixels stay as they are in memory,
// [16-channel half][pixel][16].
// Weight gradient: both operands are channels x pixels, the transpose of that,
// and are read with the LDS's transposing read (ds_read_b64_tr_b16: of 16
// lanes, lane s addresses 4 channels of a pixel, pixel s / 4, channels 4 (s % 4)
// .. + 3, and receives channel s of the four pixels), two per operand.  Wave w
// takes input channels 16 (w % 2) .. and eight rows of the block, four at a time,
// and streams down the x rows: an x operand serves the three taps (ky) that
// reach the wave's dy rows, which stay in registers.  The bias gradient is the
// product with a column of ones.  The two waves of a channel half are summed in
// LDS at the end.
// Data gradient: wave w takes rows 4 (w - 4) .. + 3, the whole weight matrix in
// registers (18 operands of 8 bf16), loaded once.
// FIRST (layer 2): dx is only needed for the first layer's weight gradient, so it
// goes to LDS instead of memory, and the wave that computed it takes its products
// with the image: four taps of a pixel's four channels are a transposing read's 16
// columns.
// What bounds it: the latency of its two rounds of global reads, then their
// bytes (16 x 128 x 128, 32 dy channels: 50 MB, 9.6 us at a copy's rate).
// There, 32 dy channels: 21 us; as two kernels 27.8 us (14.9 weights, 12.9
// data), 3 dy channels: 14.2 us against 10.4 + 9.7.  With every wave doing both
// parts in turn the registers ran out (23 and 14.9 us).  FIRST:
// 22 us; with a kernel of its own for the first layer 20.8 + 7.5.  Weight gradients
// from transposed copies written to LDS a word at a time took 19.4 us.
//   DYC: dy channels in memory (32, or 4 of which 3 are real).
//   img, part0, width0: FIRST: the image, rows of the first layer's sums.
constexpr int GH = 16, GW = 32;           // block of pixels
constexpr int GWAVES = 8;
typedef short s4 __attribute__((ext_vector_type(4)));

template <int PITCH = 16>   // values from pixel to pixel
__device__ __forceinline__ bf8 tr_operand(const uint16_t* p) {
  using LP = __attribute__((address_space(3))) s4*;
  const s4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LP)(p));
  const s4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LP)(p + 16 * PITCH));   // 16 pixels on
  return as_bf8(__builtin_bit_cast(uint4, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7)));
}

template <int DYC, bool FIRST>
__global__ __launch_bounds__(64 * GWAVES) __attribute__((amdgpu_waves_per_eu(2)))
void k_back(const uint16_t* __restrict__ x, const uint16_t* __restrict__ dy, const uint16_t* __restrict__ wt,
            uint16_t* __restrict__ dx, float* __restrict__ part, int width, const uint16_t* __restrict__ img,
            float* __restrict__ part0, int width0, int N, int H, int W, int bpw) {
  constexpr int MB = DYC == 32 ? 2 : 1, COUTR = DYC == 32 ? 32 : 3, NW = COUTR * 9 * 32, NT = 64 * GWAVES;
  constexpr int PW = GW + 2, XPX = (GH + 2) * PW;               // staged pixels: the block and its border
  constexpr int NACC = 9 * MB + MB;                             // accumulator tiles of a wave
  constexpr int KP = kpad32(DYC), KS = KP / 32;                 // the data gradient's K steps
  constexpr bool IMG = DYC != 32 || FIRST;                      // a 4-channel image is staged too
  constexpr int DXE = FIRST ? 2 * GH * GW * 16 : 0;             // the block's dx
  constexpr int STAGE = ((2 + MB) * XPX * 16 + DXE) * 2 + (IMG ? XPX * 8 : 0);
  constexpr int REDUCE = 2 * NACC * 64 * 16 + (FIRST ? 3 * 8 * 64 * 16 : 0);
  __shared__ __align__(16) unsigned char lds[STAGE > REDUCE ? STAGE : REDUCE];
  uint16_t* xs = (uint16_t*)lds;               // [2][XPX][16]
  uint16_t* ds = xs + 2 * XPX * 16;            // [MB][XPX][16]
  uint16_t* dxs = ds + MB * XPX * 16;          // FIRST: [2][GH * GW][16]
  uint2* im4 = (uint2*)(dxs + DXE);            // dy (DYC = 4) or the image (FIRST): [XPX][4]
  const int nbx = (W + GW - 1) / GW, nby = (H + GH - 1) / GH, nblocks = nbx * nby * N;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int i16 = lane & 15, g = lane >> 4;
  // this lane's part of an operand's first 16 pixels
  const int tr = (4 * g + (i16 >> 2)) * 16 + 4 * (i16 & 3);

  constexpr int NX = (XPX * 4 + NT - 1) / NT, NI = (XPX + NT - 1) / NT;
  uint4 xv[NX], dv[DYC == 32 ? NX : 1];
  uint2 iv[IMG ? NI : 1];
  const uint16_t* __restrict__ src4 = FIRST ? img : dy;
  auto load = [&](int blk) __attribute__((always_inline)) {
    const int bx = blk % nbx, by = (blk / nbx) % nby, n = blk / (nbx * nby);
#pragma unroll
    for (int it = 0; it < NX; ++it) {
      const int idx = tid + NT * it, px = idx >> 2, r = px / PW, c = px - r * PW;
      const int gy = by * GH + r - 1, gx = bx * GW + c - 1;
      xv[it] = make_uint4(0u, 0u, 0u, 0u);
      if constexpr (DYC == 32) dv[it] = make_uint4(0u, 0u, 0u, 0u);
      if (idx < XPX * 4 && gy >= 0 && gy < H && gx >= 0 && gx < W) {
        const size_t e = ((size_t)(n * H + gy) * W + gx) * 32 + (idx & 3) * 8;
        xv[it] = *(const uint4*)(x + e);
        if constexpr (DYC == 32) dv[it] = *(const uint4*)(dy + e);
      }
    }
    if constexpr (IMG) {
#pragma unroll
      for (int it = 0; it < NI; ++it) {
        const int px = tid + NT * it, r = px / PW, c = px - r * PW;
        const int gy = by * GH + r - 1, gx = bx * GW + c - 1;
        iv[it] = make_uint2(0u, 0u);
        if (px < XPX && gy >= 0 && gy < H && gx >= 0 && gx < W)
          iv[it] = *(const uint2*)(src4 + ((size_t)(n * H + gy) * W + gx) * 4);
      }
    }
  };

  const int blk0 = blockIdx.x * bpw, blk1 = min(blk0 + bpw, nblocks);
  // a block into LDS, and the next one's reads under way
  auto stage = [&](int blk) __attribute__((always_inline)) {
    if (blk > blk0) __syncthreads();   // the previous block's operands are read
#pragma unroll
    for (int it = 0; it < NX; ++it) {
      const int idx = tid + NT * it, at = ((idx & 3) >> 1) * (XPX * 16) + (idx >> 2) * 16 + (idx & 1) * 8;
      if (idx < XPX * 4) {
        *(uint4*)(xs + at) = xv[it];
        if constexpr (DYC == 32) *(uint4*)(ds + at) = dv[it];
      }
    }
    if constexpr (IMG) {
#pragma unroll
      for (int it = 0; it < NI; ++it) {
        const int px = tid + NT * it;
        if (px < XPX) {
          im4[px] = iv[it];
          if constexpr (DYC != 32) {
            *(uint4*)(ds + px * 16) = make_uint4(iv[it].x, iv[it].y & 0xffffu, 0u, 0u);   // three real channels
            *(uint4*)(ds + px * 16 + 8) = make_uint4(0u, 0u, 0u, 0u);
          }
        }
      }
    }
    __syncthreads();
    if (blk + 1 < blk1) load(blk + 1);
  };
  load(blk0);
  const uint32_t one2 = 0x3f803f80u;
  const bf8 ones = as_bf8(make_uint4(one2, one2, one2, one2));
  // The waves' parts have loops of their own (with one loop both parts' registers
  // would be held); their barriers pair up.
  if (wave >= 4) {
    // data gradient
    const int cr = 4 * (wave - 4);   // first row
    bf8 wr[KS][2];   // the weight matrix
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int nb = 0; nb < 2; ++nb) wr[ks][nb] = as_bf8(*(const uint4*)(wt + (nb * 16 + i16) * KP + ks * 32 + 8 * g));
    // FIRST: the first layer's weight gradient of this wave's rows: 9 taps x 4
    // image channels as three column blocks of four taps; the bias by ones
    f4 acc1[2][3], accb1[2];
    const uint16_t* ip[3];   // this lane's part of the three operands, first row
    if constexpr (FIRST) {
#pragma unroll
      for (int nb = 0; nb < 3; ++nb) {
        const int tap = min(nb * 4 + (i16 & 3), 8);
        ip[nb] = (const uint16_t*)(im4 + (cr + tap / 3) * PW + tap % 3 + 4 * g + (i16 >> 2));
      }
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        accb1[m] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int nb = 0; nb < 3; ++nb) acc1[m][nb] = f4{0.f, 0.f, 0.f, 0.f};
      }
    }
    for (int blk = blk0; blk < blk1; ++blk) {
      stage(blk);
      // this wave's four rows, 16 columns at a time
      const int bx = blk % nbx, by = (blk / nbx) % nby, n = blk / (nbx * nby);
#pragma unroll
      for (int cb = 0; cb < 2; ++cb) {
        f4 o[4][2];
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int nb = 0; nb < 2; ++nb) o[r][nb] = f4{0.f, 0.f, 0.f, 0.f};
        const int p0 = cr * PW + cb * 16 + i16;   // the lane's pixel of the first row, tap (0, 0)
        if constexpr (DYC == 32) {
          // an input row's operand serves the three output rows it reaches (per
          // output the taps come in the order (ky, kx))
          const uint16_t* p = ds + ((g >> 1) * XPX + p0) * 16 + (g & 1) * 8;
#pragma unroll
          for (int i = 0; i < 6; ++i)
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) {
              const bf8 b = as_bf8(*(const uint4*)(p + (i * PW + kx) * 16));
#pragma unroll
              for (int ky = 0; ky < 3; ++ky) {
                const int r = i - ky;
                if (r < 0 || r >= 4) continue;
#pragma unroll
                for (int nb = 0; nb < 2; ++nb)
                  o[r][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wr[ky * 3 + kx][nb], b, o[r][nb], 0, 0, 0);
              }
            }
        } else {
#pragma unroll
          for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              // taps t0 = 8 ks + 2 g and t0 + 1, four channels each; taps >= 9 are zero
              const uint2* p8 = im4 + p0 + r * PW;
              const int t0 = ks * 8 + 2 * g, t1 = t0 + 1;
              const int u0 = min(t0, 8), u1 = min(t1, 8);
              uint2 lo = p8[(u0 / 3) * PW + u0 % 3];
              uint2 hi = p8[(u1 / 3) * PW + u1 % 3];
              if (t0 >= 9) lo = make_uint2(0u, 0u);
              if (t1 >= 9) hi = make_uint2(0u, 0u);
              const bf8 b = as_bf8(make_uint4(lo.x, lo.y, hi.x, hi.y));
#pragma unroll
              for (int nb = 0; nb < 2; ++nb)
                o[r][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wr[ks][nb], b, o[r][nb], 0, 0, 0);
            }
        }
        // lane (g, i16) holds channels nb * 16 + 4 g .. + 3 of pixel i16; the
        // mask is the staged activation
        const int gx = bx * GW + cb * 16 + i16;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int gy = by * GH + cr + r;
          if (!FIRST && (gy >= H || gx >= W)) continue;   // FIRST: zeros there (the mask's)
          const size_t px = (size_t)(n * H + gy) * W + gx;
#pragma unroll
          for (int nb = 0; nb < 2; ++nb) {
            const uint2 m = *(const uint2*)(xs + (nb * XPX + p0 + (r + 1) * PW + 1) * 16 + 4 * g);
            const uint16_t mh[4] = {(uint16_t)m.x, (uint16_t)(m.x >> 16), (uint16_t)m.y, (uint16_t)(m.y >> 16)};
            float v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = bf2f(mh[q]) > 0.f ? o[r][nb][q] : 0.f;
            const uint2 pk = make_uint2(pk_bf16(v[0], v[1]), pk_bf16(v[2], v[3]));
            if constexpr (FIRST)
              *(uint2*)(dxs + (nb * GH * GW + (cr + r) * GW + cb * 16 + i16) * 16 + 4 * g) = pk;
            else
              *(uint2*)(dx + px * 32 + nb * 16 + 4 * g) = pk;
          }
        }
      }
      if constexpr (FIRST) {
        wave_lds_sync();   // the transposing reads take pixels that other lanes wrote
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          bf8 a[2];
#pragma unroll
          for (int m = 0; m < 2; ++m) a[m] = tr_operand(dxs + (m * GH * GW + (cr + r) * GW) * 16 + tr);
#pragma unroll
          for (int nb = 0; nb < 3; ++nb) {
            const bf8 b = tr_operand<4>(ip[nb] + r * PW * 4);
#pragma unroll
            for (int m = 0; m < 2; ++m)
              acc1[m][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m], b, acc1[m][nb], 0, 0, 0);
          }
#pragma unroll
          for (int m = 0; m < 2; ++m) accb1[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m], ones, accb1[m], 0, 0, 0);
        }
      }
    }
    // FIRST: the four waves' sums, after the weight waves' part of the buffer
    f4* red1 = (f4*)lds + 2 * NACC * 64 + lane;
    __syncthreads();
    if (FIRST && wave > 4) {
#pragma unroll
      for (int m = 0; m < 2; ++m) {
#pragma unroll
        for (int nb = 0; nb < 3; ++nb) red1[((wave - 5) * 8 + m * 4 + nb) * 64] = acc1[m][nb];
        red1[((wave - 5) * 8 + m * 4 + 3) * 64] = accb1[m];
      }
    }
    __syncthreads();
    if (FIRST && wave == 4) {
      float* row0 = part0 + (size_t)blockIdx.x * width0;
#pragma unroll
      for (int m = 0; m < 2; ++m) {
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) {
          f4 v = nb < 3 ? acc1[m][nb < 3 ? nb : 0] : accb1[m];
#pragma unroll
          for (int k = 0; k < 3; ++k) v += red1[(k * 8 + m * 4 + nb) * 64];
          const int tap = nb * 4 + (i16 >> 2), i = i16 & 3;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int o = m * 16 + 4 * g + q;
            if (nb < 3 && tap < 9 && i < 3) row0[(o * 9 + tap) * 3 + i] = v[q];
            if (nb == 3 && i16 == 0) row0[HID * 27 + o] = v[q];
          }
        }
      }
    }
    return;
  }
  // weight gradient
  const int ib = wave & 1, rh = wave >> 1;   // input channel half, row half
  f4 acc[9][MB], accb[MB];
#pragma unroll
  for (int m = 0; m < MB; ++m) {
    accb[m] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 9; ++t) acc[t][m] = f4{0.f, 0.f, 0.f, 0.f};
  }
  for (int blk = blk0; blk < blk1; ++blk) {
    stage(blk);
    // eight rows of the block, four at a time
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int y4 = 8 * rh + 4 * half;
      bf8 a[4][MB];
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int m = 0; m < MB; ++m) a[r][m] = tr_operand(ds + (m * XPX + (y4 + r + 1) * PW + 1) * 16 + tr);
#pragma unroll
      for (int i = 0; i < 6; ++i)
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) {
          const bf8 b = tr_operand(xs + (ib * XPX + (y4 + i) * PW + kx) * 16 + tr);
#pragma unroll
          for (int ky = 0; ky < 3; ++ky) {
            const int r = i - ky;
            if (r < 0 || r >= 4) continue;
#pragma unroll
            for (int m = 0; m < MB; ++m)
              acc[ky * 3 + kx][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[r][m], b, acc[ky * 3 + kx][m], 0, 0, 0);
          }
        }
      if (ib == 0)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int m = 0; m < MB; ++m)
            accb[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[r][m], ones, accb[m], 0, 0, 0);
    }
  }
  // the two row halves of each input channel half
  f4* red = (f4*)lds + (size_t)ib * NACC * 64 + lane;
  __syncthreads();
  if (rh) {
#pragma unroll
    for (int m = 0; m < MB; ++m) {
#pragma unroll
      for (int t = 0; t < 9; ++t) red[(t * MB + m) * 64] = acc[t][m];
      red[(9 * MB + m) * 64] = accb[m];
    }
  }
  __syncthreads();
  if (rh) return;
#pragma unroll
  for (int m = 0; m < MB; ++m) {
#pragma unroll
    for (int t = 0; t < 9; ++t) acc[t][m] += red[(t * MB + m) * 64];
    accb[m] += red[(9 * MB + m) * 64];
  }
  // this workgroup's row of `part` (width values; dW, then db): lane (g, i16)
  // holds output channels 4 g .. + 3 of input channel i16
  float* row_out = part + (size_t)blockIdx.x * width;
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int o = m * 16 + 4 * g + q;
      if (o >= COUTR) continue;
#pragma unroll
      for (int t = 0; t < 9; ++t) row_out[(o * 9 + t) * 32 + ib * 16 + i16] = acc[t][m][q];
      if (ib == 0 && i16 == 0) row_out[NW + o] = accb[m][q];
    }
}

// Sum of the weight-gradient kernels' per-workgroup rows, every layer at once:
// a workgroup adds 64 parameters, each of its eight waves every eighth row,
// and writes the gradient (and the caller's copy) in a fixed order.
// What bounds it: the rows' bytes.  One launch per
// layer with atomics into a cleared gradient, and a copy of it, took
// 4 x 4.5 + 8 us of a 16 x 128 x 128 step; this one takes 6.2 us (20 MB).
// part: `rows` rows of the `first` parameters of the first layer, then (from
// `rest` on) of the others.
__global__ __launch_bounds__(512) void k_wsum(const float* __restrict__ part, int first,
                                              const float* __restrict__ rest, int rows, int width, float* __restrict__ g, float* __restrict__ g2) {
  __shared__ float red[8][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, j = blockIdx.x * 64 + lane;
  float s = 0.f;
  if (j < width) {
    const int stride = j < first ? first : width - first;
    const float* p = j < first ? part + j : rest + (j - first);
#pragma unroll 8
    for (int r = wave; r < rows; r += 8) s += p[(size_t)r * stride];
  }
  red[wave][lane] = s;
  __syncthreads();
  if (wave || j >= width) return;
#pragma unroll
  for (int w = 1; w < 8; ++w) s += red[w][lane];
  g[j] = s;
  if (g2) g2[j] = s;
}

// The whole forward pass in one kernel (3 -> 32 -> 32 -> 32 -> 3): a
// workgroup computes a 14 x 26 output tile and keeps every intermediate
// activation on chip.  Each layer is computed on the region the next one
// needs -- the tile grown by one pixel per remaining layer (20 x 32, 18 x 30,
// 16 x 28 pixels) -- so that no activation is read back from memory; pixels
// of a region outside the image are zero, the padding every layer applies.
// Activations are rounded to bfloat16 after the ReLU, as the backward pass
// reads them.  KEEP: also write the three ReLU activations of the tile's own
// pixels to memory for the backward pass.
//
// Every region has rows of 32 pixels, two blocks of 16 columns.  A wave takes
// one of them and half of the layer's rows and streams down the input rows:
// an operand (16 pixels, 32 channels) is read from LDS once, a row ahead, and
// multiplied into the three output rows that it reaches, so that a row of
// outputs costs three LDS reads instead of nine; per output the taps still
// come in the order (ky, kx).  The layer's weights stay in registers (18
// operands), loaded from global memory in operand order while the slower waves
// finish the layer before: they are the same for every workgroup, and in LDS
// they took 50 KB and as many reads as the activations.
// Two workgroups of four waves fit a CU (78 KB of LDS) and fill each other's
// barriers; with six waves each, whose thirds do not divide over four SIMDs,
// only one was resident (2048 x 2048: 414 us).
// What bounds it: instruction issue of the matrix cores (busy 0.5 of the time
// at the clock they run at) and of the epilogue's vector work between them.
// 2048 x 2048, inference: 422 -> 269 us; 16 x 128 x 128 with the activations
// kept: 33.5 -> 32.6.  Tiles of 8 / 10 / 12 rows: 305 / 302 / 280 us.
constexpr int FH = 14, FW = 26;                       // output tile
constexpr int FWAVES = 4;                             // waves per workgroup
constexpr int FP = 32;                                // pixels per region row

struct FwdArgs {
  const uint16_t* w[4];    // bf16 weights in operand order, see prep_one
  const float* b[4];       // fp32 biases
  uint16_t* act[3];        // ReLU outputs, [pixels][32] (KEEP)
};

// A layer's weights and biases as a lane holds them.
template <int LI>
struct FwdW {
  static constexpr int CIN = LI == 1 ? 4 : 32, COUT = LI == 4 ? 16 : 32, NB = COUT / 16, KS = kpad32(CIN) / 32;
  bf8 w[KS][NB];
  float b[NB][4];
  __device__ __forceinline__ void load(const FwdArgs& fa, int lane) {
    const uint4* p = (const uint4*)fa.w[LI - 1] + lane;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) w[ks][nb] = as_bf8(p[(ks * NB + nb) * 64]);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int co = nb * 16 + 4 * (lane >> 4) + q;
        b[nb][q] = (LI < 4 || co < 3) ? fa.b[LI - 1][co] : 0.f;
      }
  }
};

// One layer from LDS region `in` to region `out` (LI = 1..3) or to z (LI = 4).
// 32-channel regions are four planes of 8-channel (16-byte) pixels, a multiple
// of 256 bytes apart (an operand read then spreads over all banks); columns
// past a region's width hold values that no needed output reads.
template <int LI, bool KEEP>
__device__ __forceinline__ void fwd_layer(const FwdW<LI>& wt, const void* in, uint4* out, uint16_t* __restrict__ act,
                                          float* __restrict__ z, int n, int H, int W, int y0, int x0, int wave,
                                          int lane) {
  constexpr int NB = FwdW<LI>::NB, GROW = 4 - LI;
  constexpr int HO = FH + 2 * GROW, WO = FW + 2 * GROW, RPG = (HO + FWAVES / 2 - 1) / (FWAVES / 2);
  constexpr int PIN = (HO + 2) * FP, POUT = HO * FP;       // plane strides (32-channel regions)
  const int i16 = lane & 15, g = lane >> 4;
  const int rs = min((wave >> 1) * RPG, HO - RPG), col = (wave & 1) * 16 + i16;
  const int gx = x0 - GROW + col;
  const bool colin = gx >= 0 && gx < W;
  const bool own = col >= GROW && col < GROW + FW;
  // the region reaches over the image's edge (uniform)
  const bool border = y0 < GROW || x0 < GROW || y0 + FH + GROW > H || x0 + FP - GROW > W;
  uint2* obase = (uint2*)out + ((g >> 1) * POUT + rs * FP + col) * 2 + (g & 1);

  auto finish = [&](int r, const f4 (&acc)[NB]) __attribute__((always_inline)) {
    const int oy = rs + r, gy = y0 - GROW + oy;
    const bool rowin = gy >= 0 && gy < H;
    if constexpr (LI == 4) {
      if (g == 0 && rowin && colin && col < WO)
        *(float4*)(z + ((size_t)(n * H + gy) * W + gx) * 4) =
            make_float4(acc[0][0] + wt.b[0][0], acc[0][1] + wt.b[0][1], acc[0][2] + wt.b[0][2], 0.f);
    } else {
      const bool inside = rowin && colin;
      const bool keep = KEEP && inside && own && oy >= GROW && oy < GROW + FH;
      uint2* o = obase + r * FP * 2;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        float v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = fmaxf(acc[nb][q] + wt.b[nb][q], 0.f);
        uint2 p = make_uint2(pk_bf16(v[0], v[1]), pk_bf16(v[2], v[3]));
        if (border && !inside) p = make_uint2(0u, 0u);
        o[2 * nb * POUT * 2] = p;
        if (keep) *(uint2*)(act + ((size_t)(n * H + gy) * W + gx) * 32 + nb * 16 + 4 * g) = p;
      }
    }
  };

  if constexpr (LI == 1) {
    // K step 0: taps 2 g and 2 g + 1 of four channels each; step 1: tap 8
    constexpr int WI = FP + 2;
    const uint2* p0 = (const uint2*)in + rs * WI + col;
    const int ta = 2 * g, tb = 2 * g + 1;
    const uint2* pa = p0 + (ta / 3) * WI + ta % 3;
    const uint2* pb = p0 + (tb / 3) * WI + tb % 3;
    const uint2* pc = p0 + 2 * WI + 2;
    auto read = [&](int r, uint2 (&v)[3]) __attribute__((always_inline)) {
      v[0] = pa[r * WI];
      v[1] = pb[r * WI];
      v[2] = pc[r * WI];
    };
    f4 acc[2][NB];     // output row r in slot r % 2
    uint2 v[2][3];
    read(0, v[0]);
#pragma unroll
    for (int r = 0; r < RPG; ++r) {
      if (r + 1 < RPG) read(r + 1, v[(r + 1) & 1]);
      const uint2 a = v[r & 1][0], b = v[r & 1][1], c = g ? make_uint2(0u, 0u) : v[r & 1][2];
      const bf8 b0 = as_bf8(make_uint4(a.x, a.y, b.x, b.y)), b1 = as_bf8(make_uint4(c.x, c.y, 0u, 0u));
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        acc[r & 1][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wt.w[0][nb], b0, f4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        acc[r & 1][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wt.w[1][nb], b1, acc[r & 1][nb], 0, 0, 0);
      if (r > 0) finish(r - 1, acc[(r - 1) & 1]);
    }
    finish(RPG - 1, acc[(RPG - 1) & 1]);
  } else {
    const uint4* p = (const uint4*)in + g * PIN + rs * FP + col;
    f4 acc[4][NB];     // output row r in slot r % 4
    uint4 b[2][3];
    auto read = [&](int i, uint4 (&v)[3]) __attribute__((always_inline)) {
#pragma unroll
      for (int kx = 0; kx < 3; ++kx) v[kx] = p[i * FP + kx];
    };
    read(0, b[0]);
#pragma unroll
    for (int i = 0; i < RPG + 2; ++i) {
      if (i + 1 < RPG + 2) read(i + 1, b[(i + 1) & 1]);
#pragma unroll
      for (int kx = 0; kx < 3; ++kx)
#pragma unroll
        for (int ky = 0; ky < 3; ++ky) {
          const int r = i - ky;
          if (r < 0 || r >= RPG) continue;
#pragma unroll
          for (int nb = 0; nb < NB; ++nb)
            acc[r & 3][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                wt.w[ky * 3 + kx][nb], as_bf8(b[i & 1][kx]), ky + kx ? acc[r & 3][nb] : f4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        }
      if (i >= 3) finish(i - 3, acc[(i - 3) & 3]);
    }
    finish(RPG - 1, acc[(RPG - 1) & 3]);
  }
}

// Barrier for LDS hand-over: waits for no global access (the next layer's
// weights, the activations kept).
__device__ __forceinline__ void lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <bool KEEP>
__global__ __launch_bounds__(64 * FWAVES) __attribute__((amdgpu_waves_per_eu(2)))
void k_forward(const uint16_t* __restrict__ x, const FwdArgs fa, float* __restrict__ z, int N, int H, int W) {
  constexpr int R0W = FP + 2, R0H = FH + 8, RA = FH + 6, RB = FH + 4;
  // operands of a region's last columns reach two pixels past its last row
  __shared__ __align__(256) uint4 ra[4 * RA * FP + 2];   // layer 1's output, then layer 3's
  __shared__ __align__(256) uint4 rb[4 * RB * FP + 2];   // the image patch, then layer 2's output
  uint2* r0 = (uint2*)rb;
  static_assert(R0H * R0W * sizeof(uint2) <= sizeof rb, "the image patch lies in layer 2's region");
  const int nbx = (W + FW - 1) / FW, nby = (H + FH - 1) / FH;
  const int bx = blockIdx.x % nbx, by = (blockIdx.x / nbx) % nby, n = blockIdx.x / (nbx * nby);
  const int y0 = by * FH, x0 = bx * FW;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  FwdW<1> w1;
  w1.load(fa, lane);
  // the image patch: the tile grown by four pixels, zero outside the image
  for (int p = tid; p < R0H * R0W; p += 64 * FWAVES) {
    const int r = p / R0W, c = p - r * R0W;
    const int gy = y0 - 4 + r, gx = x0 - 4 + c;
    uint2 v = make_uint2(0u, 0u);
    if (gy >= 0 && gy < H && gx >= 0 && gx < W) v = *(const uint2*)(x + ((size_t)(n * H + gy) * W + gx) * 4);
    r0[p] = v;
  }
  lds_sync();
  fwd_layer<1, KEEP>(w1, r0, ra, fa.act[0], z, n, H, W, y0, x0, wave, lane);
  FwdW<2> w2;
  w2.load(fa, lane);
  lds_sync();
  fwd_layer<2, KEEP>(w2, ra, rb, fa.act[1], z, n, H, W, y0, x0, wave, lane);
  FwdW<3> w3;
  w3.load(fa, lane);
  lds_sync();
  fwd_layer<3, KEEP>(w3, rb, ra, fa.act[2], z, n, H, W, y0, x0, wave, lane);
  FwdW<4> w4;
  w4.load(fa, lane);
  lds_sync();
  fwd_layer<4, KEEP>(w4, ra, nullptr, nullptr, z, n, H, W, y0, x0, wave, lane);
}

// MSE of y = x + z against t (three channels): dL/dz = 2 (y - t) / count as
// bfloat16, and the mean squared difference in *loss.  Each workgroup leaves
// its sum in part[]; the last one to finish (counter `done`, zero between
// launches) adds them up in order.  One atomic per 256 pixels on one address,
// with a clearing fill before and a copy after, took 15 + 8 us at
// 16 x 128 x 128; this takes 6 us (12.6 MB; 512 workgroups: 15.7, the atomics
// on one address take 30 ns each).
constexpr int kLossGroups = 64, kLossThreads = 1024;
struct __attribute__((packed, aligned(4))) F4u { float v[4]; };   // 4-byte aligned targets
__global__ __launch_bounds__(kLossThreads) void k_loss(const float4* __restrict__ z, const uint2* __restrict__ x,
                                              const F4u* __restrict__ t, uint2* __restrict__ dz,
                                              float* __restrict__ part, uint32_t* __restrict__ done,
                                              float* __restrict__ loss, int P, float scale, float inv_count) {
  __shared__ float red[kLossThreads / 64];
  __shared__ bool last;
  float s = 0.f;
#pragma unroll 4
  for (int p = blockIdx.x * kLossThreads + threadIdx.x; p < P; p += gridDim.x * kLossThreads) {
    const float4 zv = z[p];
    const uint2 xv = x[p];
    const F4u tv = t[p];
    const float zc[3] = {zv.x, zv.y, zv.z};
    const uint16_t xc[3] = {(uint16_t)xv.x, (uint16_t)(xv.x >> 16), (uint16_t)xv.y};
    uint32_t o[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const float d = bf2f(xc[c]) + zc[c] - tv.v[c];
      s += d * d;
      o[c] = f2bf(scale * d);
    }
    dz[p] = make_uint2(o[0] | (o[1] << 16), o[2]);
  }
  auto block_sum = [&](float v) {
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) v += __shfl_xor(v, m);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    float t = red[0];
#pragma unroll
    for (int w = 1; w < kLossThreads / 64; ++w) t += red[w];
    return t;
  };
  s = block_sum(s);
  if (threadIdx.x == 0) {
    __hip_atomic_store(&part[blockIdx.x], s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    last = __hip_atomic_fetch_add(done, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
  }
  __syncthreads();
  if (!last) return;
  s = 0.f;
  for (int i = threadIdx.x; i < (int)gridDim.x; i += kLossThreads)
    s += __hip_atomic_load(&part[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  s = block_sum(s);
  if (threadIdx.x == 0) {
    *loss = s * inv_count;
    *done = 0u;
  }
}

// Parameter layout (fp32): per layer, W[out][3][3][in] then b[out].
struct Layer {
  int cinr, coutr, cinm, coutp;   // real / memory input channels, real / padded output channels
  int w_off, b_off;               // offsets in the parameter vector
};
constexpr int kLayers = 4;

// bfloat16 weights, zero padded.  Forward convolutions: in the order of the
// MFMA operands, [K step][16-channel block][lane][8], lane l holding output
// channel l % 16 at K positions 8 (l / 16) .. + 7 of the step (K = tap-major
// taps x input channels).  Backward convolutions of layers 1..3: the kernel
// flipped and transposed, W'[i][2-ky][2-kx][o] = W[o][ky][kx][i], as
// [i][kpad32(taps x o)] for a convolution from the layer's output channels to
// its input channels.
__device__ __forceinline__ void prep_one(const float* __restrict__ params, uint16_t* __restrict__ wf,
                                         uint16_t* __restrict__ wb, const Layer& L, bool is_fwd, int idx) {
  if (is_fwd) {
    if (idx >= L.coutp * kpad32(L.cinm)) return;
    const int lane = (idx >> 3) & 63, op = idx >> 9, nbs = L.coutp / 16, ks = op / nbs, nb = op - ks * nbs;
    const int o = nb * 16 + (lane & 15), k = ks * 32 + 8 * (lane >> 4) + (idx & 7);
    const int tap = k / L.cinm, i = k - tap * L.cinm;
    float v = 0.f;
    if (o < L.coutr && tap < 9 && i < L.cinr) v = params[L.w_off + (o * 9 + tap) * L.cinr + i];
    wf[idx] = f2bf(v);
  } else {
    // backward conv: input channels = this layer's outputs (in memory: 4 or 32),
    // output channels = this layer's inputs (32)
    const int cin2 = L.coutr == 3 ? 4 : L.coutr, KP = kpad32(cin2);
    if (idx >= HID * KP) return;
    const int o2 = idx / KP, k = idx - o2 * KP, tap2 = k / cin2, i2 = k - tap2 * cin2;
    float v = 0.f;
    if (tap2 < 9 && i2 < L.coutr && o2 < L.cinr) {
      const int ky = 2 - tap2 / 3, kx = 2 - tap2 % 3;
      v = params[L.w_off + (i2 * 9 + ky * 3 + kx) * L.cinr + o2];
    }
    wb[idx] = f2bf(v);
  }
}

// Every layer's forward and backward matrices in one launch: segment k < 4
// is layer k's forward matrix, segment 4 + k its backward one (empty for
// layer 0); start[] holds each segment's first index.
struct PrepArgs {
  Layer L[kLayers];
  uint16_t* wf[kLayers];
  uint16_t* wb[kLayers];
  int start[2 * kLayers + 1];
};

__global__ void k_prep(const float* __restrict__ params, const PrepArgs a) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= a.start[2 * kLayers]) return;
  int seg = 0;
#pragma unroll
  for (int k = 1; k < 2 * kLayers; ++k)
    if (idx >= a.start[k]) seg = k;
  const int li = seg % kLayers;
  const bool fwd = seg < kLayers;
  prep_one(params, a.wf[li], a.wb[li], a.L[li], fwd, idx - a.start[seg]);
}

// Adam on the fp32 parameters; each thread also rounds its parameter into its
// places in the layer's forward and backward matrices (their padding stays
// zero).  What bounds it: a launch; with the matrices rebuilt by a launch of
// their own it took 4.7 + 4.1 us, now 4.1.
__global__ void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, int n, float lr, float b1, float b2, float eps, float c1,
                       float c2, const PrepArgs a) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float pi = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  p[i] = pi;
  Layer L = a.L[0];
  uint16_t *wf = a.wf[0], *wb = nullptr;
#pragma unroll
  for (int k = 1; k < kLayers; ++k)
    if (i >= a.L[k].w_off) {
      L = a.L[k];
      wf = a.wf[k];
      wb = a.wb[k];
    }
  const int r = i - L.w_off, row = r / L.cinr, ci = r - row * L.cinr, o = row / 9, tap = row - o * 9;
  if (i >= L.b_off) return;   // a bias
  const uint16_t h = f2bf(pi);
  const int k = tap * L.cinm + ci, q = k & 31;
  wf[(((k >> 5) * (L.coutp / 16) + (o >> 4)) * 64 + (q >> 3) * 16 + (o & 15)) * 8 + (q & 7)] = h;
  if (wb) {
    const int cin2 = L.coutr == 3 ? 4 : L.coutr;
    wb[ci * kpad32(cin2) + (8 - tap) * cin2 + o] = h;
  }
}

// Images (tile-planar uint8 RGB viewports, [V][ty*tx][3][T][T]) to network
// tensors: crops (v, y0, x0) of S x S as bfloat16 NHWC4 in [0, 1] (or fp32).
__global__ void k_gather(const uint8_t* __restrict__ img, int T, int tx, int ty,
                         const int* __restrict__ crops, int S, void* __restrict__ out, int as_float) {
  const int b = blockIdx.y;
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= S * S) return;
  const int v = crops[3 * b], y = crops[3 * b + 1] + p / S, xg = crops[3 * b + 2] + p % S;
  const size_t tile = (size_t)v * tx * ty + (y / T) * tx + xg / T;
  const size_t base = tile * 3 * T * T + (size_t)(y % T) * T + xg % T;
  const size_t o = ((size_t)b * S * S + p) * 4;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const float f = c < 3 ? img[base + (size_t)c * T * T] * (1.f / 255.f) : 0.f;
    if (as_float)
      ((float*)out)[o + c] = f;
    else
      ((uint16_t*)out)[o + c] = f2bf(f);
  }
}

// Restoration of a viewport around the forward pass: three kernels that move
// bytes, V pixels of a row per thread (4 where the tile edge allows it).  The
// guard decides on the device, so that the host waits once, at the end.
// 2048 x 2048 (us): to_nhwc 15.9 -> 10.8, guard 20.6 -> 11.4 + 4.8, restore
// 21.6 -> 14.6; the whole call, in which the host used to decide between guard
// and restore: 337 -> 299.
template <int V>
struct __attribute__((packed, aligned(1))) Bytes { uint8_t v[V]; };

// The whole tile-planar viewport (ty x tx tiles of T x T) as one bfloat16
// NHWC4 image in [0, 1]; clears the count of fallback tiles.
template <int V>
__global__ __launch_bounds__(256) void k_to_nhwc(const uint8_t* __restrict__ img, int T, int tx, int ty,
                                                 uint2* __restrict__ out, int* __restrict__ fell) {
  const int W = T * tx;
  const int p = (blockIdx.x * 256 + threadIdx.x) * V;
  if (p == 0) *fell = 0;
  if (p >= W * T * ty) return;
  const int y = p / W, xg = p % W;
  const uint8_t* src = img + ((size_t)(y / T) * tx + xg / T) * 3 * T * T + (size_t)(y % T) * T + xg % T;
  Bytes<V> c[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) c[k] = *(const Bytes<V>*)(src + (size_t)k * T * T);
#pragma unroll
  for (int v = 0; v < V; ++v) {
    uint32_t h[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) h[k] = f2bf(c[k].v[v] * (1.f / 255.f));
    out[p + v] = make_uint2(h[0] | (h[1] << 16), h[2]);
  }
}

// The guard of a restored viewport: per T x T tile the sum of |z| and the
// number of non-finite values.  One workgroup per (tile, band of `rows` rows)
// leaves its sums in part[]; k_guard_decide adds a tile's bands in order.  (The
// last workgroup of a tile deciding instead, behind an agent-scope release,
// took 41 us: every workgroup then writes its caches back.)
struct GuardPart { float s; int bad; };
__device__ __forceinline__ void wave_sum(float& s, int& nb) {
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) {
    s += __shfl_xor(s, m);
    nb += __shfl_xor(nb, m);
  }
}
__global__ __launch_bounds__(256) void k_guard(const float4* __restrict__ z, int T, int tx, int rows,
                                               GuardPart* __restrict__ part) {
  const int W = T * tx;
  const int tile = blockIdx.x, tyi = tile / tx, txi = tile - tyi * tx;
  const int r0 = blockIdx.y * rows, r1 = min(r0 + rows, T);
  float s = 0.f;
  int nb = 0;
#pragma unroll 4
  for (int i = threadIdx.x; i < (r1 - r0) * T; i += 256) {
    const int r = r0 + i / T, c = i - (i / T) * T;
    const float4 v4 = z[(size_t)(tyi * T + r) * W + txi * T + c];
    const float v[3] = {v4.x, v4.y, v4.z};
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
      if (!isfinite(v[ch])) ++nb;
      else s += fabsf(v[ch]);
    }
  }
  wave_sum(s, nb);
  __shared__ float rs[4];
  __shared__ int rn[4];
  if ((threadIdx.x & 63) == 0) {
    rs[threadIdx.x >> 6] = s;
    rn[threadIdx.x >> 6] = nb;
  }
  __syncthreads();
  if (threadIdx.x == 0)
    part[(size_t)tile * gridDim.y + blockIdx.y] = {rs[0] + rs[1] + rs[2] + rs[3], rn[0] + rn[1] + rn[2] + rn[3]};
}

// One wave per tile: use[tile] = 1 if the tile keeps the network's output, that
// is if every value is finite and the mean correction (0..1 scale) stays
// within the guard; *fell counts the others.
__global__ __launch_bounds__(64) void k_guard_decide(const GuardPart* __restrict__ part, int bands, double per_tile,
                                                     float guard, int* __restrict__ use, int* __restrict__ fell) {
  const int tile = blockIdx.x;
  float s = 0.f;
  int nb = 0;
  for (int i = threadIdx.x; i < bands; i += 64) {
    const GuardPart g = part[(size_t)tile * bands + i];
    s += g.s;
    nb += g.bad;
  }
  wave_sum(s, nb);
  if (threadIdx.x) return;
  const int ok = nb == 0 && (double)s / per_tile <= (double)guard;
  use[tile] = ok;
  if (!ok) atomicAdd(fell, 1);
}

// Restored viewport: clip(x + z) in 8 bits, or the decoded tile where the
// guard tripped.
template <int V>
__global__ __launch_bounds__(256) void k_restore(const uint8_t* dec, const float4* __restrict__ z, int T, int tx, int ty,
                                                 const int* __restrict__ use, uint8_t* out) {
  const int W = T * tx;
  const int p = (blockIdx.x * 256 + threadIdx.x) * V;
  if (p >= W * T * ty) return;
  const int y = p / W, xg = p % W;
  const int tile = (y / T) * tx + xg / T;
  const size_t base = (size_t)tile * 3 * T * T + (size_t)(y % T) * T + xg % T;
  Bytes<V> c[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) c[k] = *(const Bytes<V>*)(dec + base + (size_t)k * T * T);
  if (use[tile]) {
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const float4 z4 = z[p + v];
      const float zc[3] = {z4.x, z4.y, z4.z};
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const float f = c[k].v[v] * (1.f / 255.f) + zc[k];
        c[k].v[v] = (uint8_t)fminf(fmaxf(rintf(f * 255.f), 0.f), 255.f);
      }
    }
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) *(Bytes<V>*)(out + base + (size_t)k * T * T) = c[k];
}

}  // namespace cnn
}  // namespace wv

using namespace wv;
using namespace wv::cnn;
using wvp::fail;
using wvp::hip_fail;

// weight gradients: at most this many workgroups (one per CU), each writing one
// row of partial sums
constexpr int kWgradRows = 256;

constexpr int kMaxGuardTiles = 65536;

struct wv_cnn {
  Layer layer[kLayers];
  int n_params = 0;
  int64_t max_pixels = 0;
  float* params = nullptr;     // fp32 masters
  float* grads = nullptr;
  float* adam_m = nullptr;
  float* adam_v = nullptr;
  uint16_t* wf[kLayers] = {};   // forward bfloat16 weights
  uint16_t* wb[kLayers] = {};   // backward bfloat16 weights (layers 1..3)
  uint16_t* x = nullptr;        // [P][4] input buffer (restore writes its viewport here)
  const uint16_t* xin = nullptr;  // input of the last forward, read in place
  float* zout = nullptr;        // output of the last forward
  uint16_t* act[3] = {};        // [P][32]
  uint16_t* dbuf[2] = {};       // [P][32]
  float* z = nullptr;           // [P][4]
  uint16_t* dz = nullptr;       // [P][4]
  float* loss_part = nullptr;   // loss sums, one per workgroup
  uint32_t* loss_done = nullptr;  // workgroups finished (0 between launches)
  GuardPart* guard_part = nullptr;  // guard sums, one per workgroup
  int* guard_use = nullptr;         // per tile: keep the network's output; then the count of the others
  int* crops = nullptr;
  float* wpart = nullptr;       // weight-gradient partial sums: the first layer's rows, then the others'
  int n = 0, h = 0, w = 0;      // shape of the last forward
  bool fwd_valid = false, grad_valid = false;
  bool prepped = false;
};

static void layer_table(Layer* L, int& total) {
  const int cinr[kLayers] = {3, HID, HID, HID}, coutr[kLayers] = {HID, HID, HID, 3};
  int off = 0;
  for (int i = 0; i < kLayers; ++i) {
    L[i].cinr = cinr[i];
    L[i].coutr = coutr[i];
    L[i].cinm = cinr[i] == 3 ? 4 : cinr[i];
    L[i].coutp = coutr[i] == 3 ? 16 : coutr[i];
    L[i].w_off = off;
    off += coutr[i] * 9 * cinr[i];
    L[i].b_off = off;
    off += coutr[i];
  }
  total = off;
}

extern "C" int32_t wv_cnn_param_count(void) {
  Layer L[kLayers];
  int t = 0;
  layer_table(L, t);
  return t;
}

extern "C" wv_status wv_cnn_destroy(wv_cnn* net) {
  if (!net) return WV_OK;
  (void)hipDeviceSynchronize();
  void* ptrs[] = {net->params, net->grads, net->adam_m, net->adam_v, net->x, net->act[0], net->act[1],
                  net->act[2], net->dbuf[0], net->dbuf[1], net->z, net->dz, net->loss_part, net->loss_done, net->guard_part,
                  net->guard_use, net->crops, net->wpart};
  for (void* p : ptrs)
    if (p) (void)hipFree(p);
  for (int i = 0; i < kLayers; ++i) {
    if (net->wf[i]) (void)hipFree(net->wf[i]);
    if (net->wb[i]) (void)hipFree(net->wb[i]);
  }
  delete net;
  return WV_OK;
}

extern "C" wv_status wv_cnn_create(wv_cnn** out, int64_t max_pixels) {
  if (!out || max_pixels < 1 || max_pixels > ((int64_t)1 << 28))
    return fail(WV_EINVAL, "wv_cnn_create: max_pixels must be 1 .. 2^28");
  *out = nullptr;
  wv_cnn* net = new (std::nothrow) wv_cnn();
  if (!net) return fail(WV_ENOMEM, "wv_cnn allocation");
  layer_table(net->layer, net->n_params);
  net->max_pixels = max_pixels;
  const size_t P = (size_t)max_pixels, np = (size_t)net->n_params * sizeof(float);
  hipError_t e = hipSuccess;
  auto alloc = [&](void** p, size_t bytes) {
    if (e == hipSuccess) e = hipMalloc(p, bytes);
    if (e == hipSuccess) e = hipMemset(*p, 0, bytes);
  };
  alloc((void**)&net->params, np);
  alloc((void**)&net->grads, np);
  alloc((void**)&net->adam_m, np);
  alloc((void**)&net->adam_v, np);
  for (int i = 0; i < kLayers; ++i) {
    alloc((void**)&net->wf[i], (size_t)net->layer[i].coutp * kpad32(net->layer[i].cinm) * 2);
    if (i > 0) alloc((void**)&net->wb[i], (size_t)HID * kpad32(net->layer[i].coutr == 3 ? 4 : HID) * 2);
  }
  alloc((void**)&net->x, P * 4 * 2);
  for (int i = 0; i < 3; ++i) alloc((void**)&net->act[i], P * HID * 2);
  for (int i = 0; i < 2; ++i) alloc((void**)&net->dbuf[i], P * HID * 2);
  alloc((void**)&net->z, P * 4 * 4);
  alloc((void**)&net->dz, P * 4 * 2);
  alloc((void**)&net->loss_part, kLossGroups * sizeof(float));
  alloc((void**)&net->loss_done, sizeof(uint32_t));
  // a guard workgroup has at least 2048 pixels, or is a tile's only or last one
  alloc((void**)&net->guard_part, (P / 2048 + kMaxGuardTiles) * sizeof(GuardPart));
  alloc((void**)&net->guard_use, (kMaxGuardTiles + 1) * sizeof(int));
  alloc((void**)&net->crops, 3 * 4096 * sizeof(int));
  // a backward workgroup has at least one pixel; every row is written before it
  // is read
  if (e == hipSuccess)
    e = hipMalloc((void**)&net->wpart, std::min<size_t>(kWgradRows, P) * net->n_params * sizeof(float));
  if (e != hipSuccess) {
    wv_cnn_destroy(net);
    return e == hipErrorOutOfMemory ? fail(WV_ENOMEM, "wv_cnn buffers: %s", hipGetErrorString(e))
                                    : hip_fail(e, "wv_cnn_create");
  }
  *out = net;
  return WV_OK;
}

static PrepArgs prep_args(const wv_cnn* net) {
  PrepArgs a;
  int at = 0;
  for (int i = 0; i < kLayers; ++i) {
    const Layer& L = net->layer[i];
    a.L[i] = L;
    a.wf[i] = net->wf[i];
    a.wb[i] = net->wb[i];
    a.start[i] = at;
    at += L.coutp * kpad32(L.cinm);
  }
  for (int i = 0; i < kLayers; ++i) {
    const Layer& L = net->layer[i];
    a.start[kLayers + i] = at;
    if (i > 0) at += HID * kpad32(L.coutr == 3 ? 4 : HID);
  }
  a.start[2 * kLayers] = at;
  return a;
}

static wv_status prep(wv_cnn* net, hipStream_t s) {
  const PrepArgs a = prep_args(net);
  const int at = a.start[2 * kLayers];
  hipLaunchKernelGGL(k_prep, dim3((at + 255) / 256), dim3(256), 0, s, net->params, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "wv_cnn weight preparation");
  net->prepped = true;
  return WV_OK;
}

extern "C" wv_status wv_cnn_set_params(wv_cnn* net, const float* host_params, hipStream_t s) {
  if (!net || !host_params) return fail(WV_EINVAL, "wv_cnn_set_params: bad argument");
  hipError_t e = hipMemcpyAsync(net->params, host_params, (size_t)net->n_params * 4,
                                hipMemcpyHostToDevice, s);
  if (e == hipSuccess) e = hipMemsetAsync(net->adam_m, 0, (size_t)net->n_params * 4, s);
  if (e == hipSuccess) e = hipMemsetAsync(net->adam_v, 0, (size_t)net->n_params * 4, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return hip_fail(e, "wv_cnn_set_params");
  return prep(net, s);
}

extern "C" wv_status wv_cnn_get_params(wv_cnn* net, float* host_params, hipStream_t s) {
  if (!net || !host_params) return fail(WV_EINVAL, "wv_cnn_get_params: bad argument");
  hipError_t e = hipMemcpyAsync(host_params, net->params, (size_t)net->n_params * 4,
                                hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  return e == hipSuccess ? WV_OK : hip_fail(e, "wv_cnn_get_params");
}

static int fwd_grid(int n, int h, int w) { return n * ((h + FH - 1) / FH) * ((w + FW - 1) / FW); }

// The forward pass in one launch; keep: write the activations the backward
// pass reads.
static wv_status forward(wv_cnn* net, const uint16_t* x, int32_t n, int32_t h, int32_t w, float* z, bool keep,
                         hipStream_t s) {
  const char* fn = keep ? "wv_cnn_forward" : "wv_cnn_infer";
  if (!net || !x || n < 1 || h < 1 || w < 1) return fail(WV_EINVAL, "%s: bad argument", fn);
  if ((int64_t)n * h * w > net->max_pixels)
    return fail(WV_EINVAL, "%s: %lld pixels above the %lld the network was created for", fn,
                (long long)n * h * w, (long long)net->max_pixels);
  if (!net->prepped) return fail(WV_EINVAL, "%s: parameters not set", fn);
  float* zo = z ? z : net->z;
  const Layer* L = net->layer;
  FwdArgs fa;
  for (int i = 0; i < kLayers; ++i) {
    fa.w[i] = net->wf[i];
    fa.b[i] = net->params + L[i].b_off;
  }
  for (int i = 0; i < 3; ++i) fa.act[i] = net->act[i];
  const dim3 g(fwd_grid(n, h, w)), b(64 * FWAVES);
  if (keep)
    hipLaunchKernelGGL(k_forward<true>, g, b, 0, s, x, fa, zo, n, h, w);
  else
    hipLaunchKernelGGL(k_forward<false>, g, b, 0, s, x, fa, zo, n, h, w);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, fn);
  net->xin = x;
  net->zout = zo;
  net->n = n;
  net->h = h;
  net->w = w;
  net->fwd_valid = keep;
  net->grad_valid = false;
  return WV_OK;
}

extern "C" wv_status wv_cnn_forward(wv_cnn* net, const uint16_t* x, int32_t n, int32_t h, int32_t w,
                                    float* z, hipStream_t s) {
  return forward(net, x, n, h, w, z, true, s);
}

extern "C" wv_status wv_cnn_infer(wv_cnn* net, const uint16_t* x, int32_t n, int32_t h, int32_t w, float* z,
                                  hipStream_t s) {
  return forward(net, x, n, h, w, z, false, s);
}

extern "C" wv_status wv_cnn_loss_grad(wv_cnn* net, const float* t, float* loss, hipStream_t s) {
  if (!net || !t || !loss) return fail(WV_EINVAL, "wv_cnn_loss_grad: bad argument");
  if (!net->fwd_valid) return fail(WV_EINVAL, "wv_cnn_loss_grad: no forward pass to differentiate");
  const int P = net->n * net->h * net->w;
  hipLaunchKernelGGL(k_loss, dim3(std::min((P + kLossThreads - 1) / kLossThreads, kLossGroups)),
                     dim3(kLossThreads), 0, s,
                     (const float4*)net->zout, (const uint2*)net->xin, (const F4u*)t, (uint2*)net->dz, net->loss_part,
                     net->loss_done, loss, P, 2.0f / (3.0f * (float)P), 1.0f / (3.0f * (float)P));
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "wv_cnn_loss_grad");
  net->grad_valid = true;
  return WV_OK;
}

extern "C" wv_status wv_cnn_backward(wv_cnn* net, float* grads, hipStream_t s) {
  if (!net) return fail(WV_EINVAL, "wv_cnn_backward: bad argument");
  if (!net->grad_valid) return fail(WV_EINVAL, "wv_cnn_backward: no loss gradient");
  const int n = net->n, h = net->h, w = net->w;
  const Layer* L = net->layer;
  // split over pixels: at most kWgradRows workgroups, each writing a row of
  // partial sums that k_wsum adds up
  const int nb = n * ((h + GH - 1) / GH) * ((w + GW - 1) / GW), bpw = (nb + kWgradRows - 1) / kWgradRows;
  const int rows = (nb + bpw - 1) / bpw;
  const dim3 gw(rows), bw(64 * GWAVES);
  const int np = net->n_params, np0 = L[1].w_off, npr = np - np0;   // parameters of the first layer, of the others
  float* rest = net->wpart + (size_t)rows * np0;
  auto part = [&](int l) { return rest + (L[l].w_off - np0); };
  // layer 4: dW4 from a3 and dz; d3 = (W4' * dz) masked by a3 > 0
  hipLaunchKernelGGL((k_back<4, false>), gw, bw, 0, s, net->act[2], net->dz, net->wb[3], net->dbuf[0], part(3), npr,
                     nullptr, nullptr, 0, n, h, w, bpw);
  // layer 3
  hipLaunchKernelGGL((k_back<HID, false>), gw, bw, 0, s, net->act[1], net->dbuf[0], net->wb[2], net->dbuf[1], part(2),
                     npr, nullptr, nullptr, 0, n, h, w, bpw);
  // layer 2, and the weights of layer 1 from the d1 it computes
  hipLaunchKernelGGL((k_back<HID, true>), gw, bw, 0, s, net->act[0], net->dbuf[1], net->wb[1], nullptr, part(1), npr,
                     net->xin, net->wpart, np0, n, h, w, bpw);
  // every layer's rows into the gradient, and into the caller's copy
  hipLaunchKernelGGL(k_wsum, dim3((np + 63) / 64), dim3(512), 0, s, (const float*)net->wpart, np0,
                     (const float*)rest, rows, np, net->grads,
                     grads == net->grads ? nullptr : grads);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "wv_cnn_backward");
  return WV_OK;
}

extern "C" wv_status wv_cnn_adam(wv_cnn* net, float lr, int32_t step, hipStream_t s) {
  if (!net || step < 1 || !(lr > 0)) return fail(WV_EINVAL, "wv_cnn_adam: bad argument");
  const float b1 = 0.9f, b2 = 0.999f;
  const float c1 = 1.f - std::pow(b1, (float)step), c2 = 1.f - std::pow(b2, (float)step);
  hipLaunchKernelGGL(k_adam, dim3((net->n_params + 255) / 256), dim3(256), 0, s, net->params, net->grads,
                     net->adam_m, net->adam_v, net->n_params, lr, b1, b2, 1e-8f, c1, c2, prep_args(net));
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "wv_cnn_adam");
  return net->prepped ? WV_OK : prep(net, s);   // no parameters were set: the padding too
}

extern "C" wv_status wv_cnn_train_step(wv_cnn* net, const uint16_t* x, const float* t, int32_t n,
                                       int32_t h, int32_t w, float lr, int32_t step, float* loss,
                                       hipStream_t s) {
  wv_status st = wv_cnn_forward(net, x, n, h, w, nullptr, s);
  if (st == WV_OK) st = wv_cnn_loss_grad(net, t, loss, s);
  if (st == WV_OK) st = wv_cnn_backward(net, nullptr, s);
  if (st == WV_OK) st = wv_cnn_adam(net, lr, step, s);
  return st;
}

extern "C" wv_status wv_cnn_gather(wv_cnn* net, const uint8_t* images, int32_t tile, int32_t tiles_x,
                                   int32_t tiles_y, int32_t n_images, const int32_t* crops,
                                   int32_t n_crops, int32_t size, int32_t as_float, void* out,
                                   hipStream_t s) {
  if (!net || !images || !crops || !out || tile < 1 || tiles_x < 1 || tiles_y < 1 || n_crops < 1 ||
      n_crops > 4096 || size < 1)
    return fail(WV_EINVAL, "wv_cnn_gather: bad argument");
  for (int i = 0; i < n_crops; ++i) {
    const int v = crops[3 * i], y0 = crops[3 * i + 1], x0 = crops[3 * i + 2];
    if (v < 0 || v >= n_images || y0 < 0 || x0 < 0 || y0 + size > tile * tiles_y ||
        x0 + size > tile * tiles_x)
      return fail(WV_EINVAL, "wv_cnn_gather: crop %d outside its image", i);
  }
  // the crop table is copied synchronously: the network's table buffer is
  // reused by the next call
  hipError_t e = hipMemcpyAsync(net->crops, crops, (size_t)n_crops * 3 * sizeof(int),
                                hipMemcpyHostToDevice, s);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_gather, dim3((size * size + 255) / 256, n_crops), dim3(256), 0, s, images, tile,
                       tiles_x, tiles_y, (const int*)net->crops, size, out, as_float);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  return e == hipSuccess ? WV_OK : hip_fail(e, "wv_cnn_gather");
}

extern "C" wv_status wv_cnn_restore(wv_cnn* net, const uint8_t* decoded, int32_t tile, int32_t tiles_x,
                                    int32_t tiles_y, float guard, uint8_t* out, int32_t* fallback_tiles,
                                    hipStream_t s) {
  if (!net || !decoded || !out || tile < 1 || tiles_x < 1 || tiles_y < 1 || !(guard > 0))
    return fail(WV_EINVAL, "wv_cnn_restore: bad argument");
  const int nt = tiles_x * tiles_y;
  if (nt > kMaxGuardTiles) return fail(WV_EINVAL, "wv_cnn_restore: at most 65536 tiles");
  const int H = tile * tiles_y, W = tile * tiles_x;
  if ((int64_t)H * W > net->max_pixels) return fail(WV_EINVAL, "wv_cnn_restore: image above max_pixels");
  const int P = H * W, V = tile % 4 == 0 ? 4 : 1, gb = (P / V + 255) / 256;
  int* count = net->guard_use + kMaxGuardTiles;
  // the input goes straight into the network's input buffer
  if (V == 4)
    hipLaunchKernelGGL(k_to_nhwc<4>, dim3(gb), dim3(256), 0, s, decoded, tile, tiles_x, tiles_y, (uint2*)net->x, count);
  else
    hipLaunchKernelGGL(k_to_nhwc<1>, dim3(gb), dim3(256), 0, s, decoded, tile, tiles_x, tiles_y, (uint2*)net->x, count);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "wv_cnn_restore");
  // inference only: the activations are not needed
  wv_status st = forward(net, net->x, 1, H, W, nullptr, false, s);
  if (st != WV_OK) return st;
  const int rows = std::max(1, 4096 / tile);
  const int bands = (tile + rows - 1) / rows;
  hipLaunchKernelGGL(k_guard, dim3(nt, bands), dim3(256), 0, s, (const float4*)net->z, tile, tiles_x, rows,
                     net->guard_part);
  hipLaunchKernelGGL(k_guard_decide, dim3(nt), dim3(64), 0, s, (const GuardPart*)net->guard_part, bands,
                     3.0 * tile * tile, guard, net->guard_use, count);
  if (V == 4)
    hipLaunchKernelGGL(k_restore<4>, dim3(gb), dim3(256), 0, s, decoded, (const float4*)net->z, tile, tiles_x, tiles_y,
                       (const int*)net->guard_use, out);
  else
    hipLaunchKernelGGL(k_restore<1>, dim3(gb), dim3(256), 0, s, decoded, (const float4*)net->z, tile, tiles_x, tiles_y,
                       (const int*)net->guard_use, out);
  e = hipGetLastError();
  int fell = 0;
  if (e == hipSuccess) e = hipMemcpyAsync(&fell, count, sizeof(int), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return hip_fail(e, "wv_cnn_restore");
  if (fallback_tiles) *fallback_tiles = fell;
  return WV_OK;
}
