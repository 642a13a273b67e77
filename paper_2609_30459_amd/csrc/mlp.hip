// Learned-initialisation MLP on gfx950 BF16 MFMA (v_mfma_f32_16x16x32_bf16,
// FP32 accumulation): forward, loss, backward and Adam, plus the C ABI of
// vio_mlp.h.
//
// MFMA operand layout (16x16x32): lane l holds A[l%16][8(l/16) .. +7] (a row
// segment of 8 bf16), B[8(l/16) .. +7][l%16] (a column segment) and returns
// D[4(l/16) + q][l%16], q = 0..3.
//
// Inference (k_mlp_infer): layer 1 is one MFMA per 16 hidden units (K = 32 is one
// step); the ReLU'd bf16 activations go through LDS to become the next layer's A
// operand.
//
// Training: one kernel (k_mlp_grad) takes 32 rows at a time through the
// forward pass, the loss, the data gradients (dH2 = dY W3, dH1 = dH2 W2,
// masked by the ReLUs) and the weight gradients (dW = dH^T H_prev, MFMA with
// the rows as the K dimension; bias gradients against a ones operand), and a
// second one adds the workgroups' partial gradients and, in a training step,
// runs Adam. Every sum has a fixed order: no atomics, deterministic results.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>

#include "fe_common.h"
#include "mfma_ops.h"
#include "vio_mlp.h"
#include "wave_ops.h"

namespace vio {

// An MFMA result tile's four values of a lane (rows 4 g + q, q = 0..3, of its
// column) as bf16, two to a word.
struct Quad {
  uint32_t w[2];
};
__device__ __forceinline__ Quad quad_of(f32x4 v) { return {bf16_pair(v[0], v[1]), bf16_pair(v[2], v[3])}; }
__device__ __forceinline__ Quad quad_relu(f32x4 v, float b) {
  return {bf16_pair(fmaxf(v[0] + b, 0.f), fmaxf(v[1] + b, 0.f)), bf16_pair(fmaxf(v[2] + b, 0.f), fmaxf(v[3] + b, 0.f))};
}
// the values of d where h (never negative: a ReLU's result) is not zero
__device__ __forceinline__ Quad quad_where(Quad d, Quad h) {
  typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const u16x2 one = {1, 1};
    const u16x2 on = __builtin_elementwise_min(__builtin_bit_cast(u16x2, h.w[k]), one);
    d.w[k] &= __builtin_bit_cast(uint32_t, (u16x2)(-on));
  }
  return d;
}
// to column `unit` of rows row .. row + 3 of an LDS tile
__device__ __forceinline__ void store_quad(uint16_t (*rows)[MH + 8], int row, int unit, Quad v) {
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    rows[row + 2 * k][unit] = (uint16_t)v.w[k];
    rows[row + 2 * k + 1][unit] = (uint16_t)(v.w[k] >> 16);
  }
}

// ---------------------------------------------------------------------------
// inference forward, with the MFMA sequence of the training kernel and of the
// frontend's learned stage (so the same results row by row). A workgroup of
// eight waves takes chunks of 32 rows; wave w owns hidden units 16 w .. 16 w + 15
// of both hidden layers and keeps its slices of W1 and W2 in registers for all
// its chunks (a wave per 16 rows, each reading all 42 KB of weights, took 8.7 us
// for 600 rows and 23.8 us for 65,536). The activations pass through LDS by
// rows; the two output tiles of a chunk go to another pair of waves each time.
// Bound by latency at small batches (the weights' loads, two barriers a chunk:
// 4.4 us for 600 rows); 65,536 rows take 12.5 us.
// ---------------------------------------------------------------------------
constexpr int kHidWaves = MH / 16;  // one 16-unit hidden tile per wave
constexpr int kChunk = 32;          // rows per chunk: two MFMA row tiles
// workgroups at most: two per compute unit (65,536 rows: 512 workgroups 12.8 us,
// 768 13.3, 1,024 14.2, one per chunk 19.4: each loads the weights once)
constexpr int kInferGroups = 512;
__global__ __launch_bounds__(64 * kHidWaves) void k_mlp_infer(MlpDev M, const float* __restrict__ X, int K,
                                                              int n_chunks, float* __restrict__ Y) {
  // rows padded by 8 entries: the 16 rows of an operand read start 4 banks apart
  __shared__ __align__(16) uint16_t sH1[kChunk][MH + 8];
  __shared__ __align__(16) uint16_t sH2[kChunk][MH + 8];
  __shared__ uint4 sW3[MH / 32][64];  // W3 as the output tile's B operand (columns 3..15 are zero)
  const int lane = (int)threadIdx.x & 63, wv = (int)threadIdx.x >> 6;
  const int r = lane & 15, g = lane >> 4;
  const int unit = 16 * wv + r;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  F32x8 xr[2];  // a chunk's rows, loaded one chunk ahead (rows past the batch read its last row)
  const auto fetch = [&](int ch) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
      xr[t] = *reinterpret_cast<const F32x8*>(X + (size_t)min(ch * kChunk + 16 * t + r, K - 1) * MI + 8 * g);
  };
  fetch((int)blockIdx.x);
  const bf16x8 w1 = load8(M.W1b + (size_t)unit * MI + 8 * g);
  const float b1 = M.P[OFF_B1 + unit], b2 = M.P[OFF_B2 + unit], b3 = M.P[OFF_B3 + min(r, MO - 1)];
  bf16x8 w2[MH / 32];
#pragma unroll
  for (int kc = 0; kc < MH / 32; ++kc) w2[kc] = load8(M.W2b + (size_t)unit * MH + 32 * kc + 8 * g);
  if (wv < MH / 32) {
    const uint4 w = *reinterpret_cast<const uint4*>(M.W3b + (size_t)min(r, MO - 1) * MH + 32 * wv + 8 * g);
    sW3[wv][lane] = r < MO ? w : make_uint4(0u, 0u, 0u, 0u);
  }
  int turn = 0;  // the pair of waves whose turn the output tiles are
  for (int ch = (int)blockIdx.x; ch < n_chunks; ch += (int)gridDim.x) {
    const int i0 = ch * kChunk;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const f32x4 acc = mfma(pack_f32(xr[t].v, i0 + 16 * t + r < K), w1, zero);
      store_quad(sH1, 16 * t + 4 * g, unit, quad_relu(acc, b1));
    }
    if (ch + (int)gridDim.x < n_chunks) fetch(ch + (int)gridDim.x);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      f32x4 acc = zero;
#pragma unroll
      for (int kc = 0; kc < MH / 32; ++kc) acc = mfma(load8(&sH1[16 * t + r][32 * kc + 8 * g]), w2[kc], acc);
      store_quad(sH2, 16 * t + 4 * g, unit, quad_relu(acc, b2));
    }
    // (the next chunk's h1 is written after this barrier, its h2 after the next
    // one, which the waves that read h2 here reach last)
    __syncthreads();
    if ((wv >> 1) == turn) {
      const int t = wv & 1;
      f32x4 acc = zero;
#pragma unroll
      for (int kc = 0; kc < MH / 32; ++kc)
        acc = mfma(load8(&sH2[16 * t + r][32 * kc + 8 * g]), __builtin_bit_cast(bf16x8, sW3[kc][lane]), acc);
      if (r < MO) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int i = i0 + 16 * t + 4 * g + q;
          if (i < K) Y[(size_t)i * MO + r] = acc[q] + b3;
        }
      }
    }
    turn = (turn + 1) & 3;
  }
}

// ---------------------------------------------------------------------------
// training: loss and partial gradients
//
// A workgroup of eight waves takes chunks of 32 rows (two 16-row MFMA tiles, one
// K step of the weight gradients); wave w owns hidden units 16 w .. 16 w + 15 of both hidden layers, with its
// slices of W1, W2, W2^T and W3 in registers for all its chunks. A chunk's
// activations and gradients never leave the compute unit: a wave holds its own
// units' as MFMA results, and passes them on through LDS, by rows to become the
// next layer's A operand, and packed to become a B operand of the weight
// gradients. Those are MFMAs whose K dimension is the chunk's 32 rows, and the
// order of K is free as long as both operands share it: with row 4 g + e of
// tile 0 at k = 8 g + e and of tile 1 at k = 8 g + 4 + e, what lane (r, g) must
// hold of an operand is exactly what it holds of two MFMA results (row 4 g + q,
// column r), so nothing is transposed. The wave accumulates its 16 x 128 rows of dW2, 16 x 32 of dW1,
// 3 x 16 of dW3 and its biases' over its chunks and writes them once, to the
// workgroup's partial gradient.
//
// Bound by latency: the weights' loads and a chunk's chain (four dependent
// layers, five barriers, about 4.4 us with two waves per SIMD). Measured:
// 1,024 rows 10.9 us and 50,000 rows 33.5 us for this kernel, where the forward
// pass, loss, data gradient and weight gradient as four kernels with transposed
// operands in memory took 59 and 748 us (the weight gradient's 105 waves walked
// the whole batch each, the loss ran in one workgroup).
// ---------------------------------------------------------------------------
// A partial gradient: the parameters in their order, then the loss sum, padded
// to whole 64-float lines.
constexpr int kPartLoss = NP;
constexpr int kPartStride = (NP + 1 + 63) / 64 * 64;

// Workgroups (and partial gradients) of a batch of k rows: one chunk each up
// to 64 (a batch of 1024 rows: 32 compute units, the least time), then up to four
// chunks each, so that the partials' traffic stays below the chunks' work,
// and at most 256, one per compute unit (their accumulators fill its registers).
int grad_groups(int k) {
  const int chunks = (k + kChunk - 1) / kChunk;
  return std::min(chunks, std::max(64, std::min(256, chunks / 4)));
}

// both row tiles' values as one operand (k = 8 g + e: rows 4 g + e of tile 0, then of tile 1)
__device__ __forceinline__ bf16x8 pack_tiles(Quad t0, Quad t1) {
  return __builtin_bit_cast(bf16x8, make_uint4(t0.w[0], t0.w[1], t1.w[0], t1.w[1]));
}

__global__ __launch_bounds__(64 * kHidWaves) void k_mlp_grad(MlpDev M, const float* __restrict__ X,
                                                              const float* __restrict__ T, int K, int n_chunks,
                                                              float* __restrict__ part) {
  // rows padded by 8 entries: the 16 rows of an operand read start 4 banks apart
  __shared__ __align__(16) uint16_t sA[kChunk][MH + 8];  // h1 by rows, then dH2
  __shared__ __align__(16) uint16_t sH2[kChunk][MH + 8];
  __shared__ uint4 sB[kHidWaves][64];  // h1 as B operands, by hidden tile
  __shared__ uint4 sX[MI / 16][64];     // x as B operands, by 16 features
  __shared__ uint4 sW3[MH / 32][64];
  __shared__ float sY[kChunk][4];
  __shared__ __align__(16) uint16_t sdY[4][kChunk];  // dY by output (bf16)
  const int lane = (int)threadIdx.x & 63, wv = (int)threadIdx.x >> 6;
  const int r = lane & 15, g = lane >> 4;
  const int unit = 16 * wv + r;  // this lane's hidden unit, as a column of its wave's tiles
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  const bf16x8 zb = __builtin_bit_cast(bf16x8, make_uint4(0u, 0u, 0u, 0u));
  const bf16x8 ones = __builtin_bit_cast(bf16x8, make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u));

  // the wave's weights, in the order they are needed
  const bf16x8 w1 = load8(M.W1b + (size_t)unit * MI + 8 * g);
  const float b1 = M.P[OFF_B1 + unit], b2 = M.P[OFF_B2 + unit];
  bf16x8 w2[MH / 32], w2t[MH / 32];
#pragma unroll
  for (int kc = 0; kc < MH / 32; ++kc) w2[kc] = load8(M.W2b + (size_t)unit * MH + 32 * kc + 8 * g);
  // W3 as the output tile's B operand, in LDS (columns 3..15 are zero): waves 0
  // and 1 compute the outputs of the two row tiles
  if (wv < MH / 32) sW3[wv][lane] = r < MO ? *reinterpret_cast<const uint4*>(M.W3b + (size_t)r * MH + 32 * wv + 8 * g)
                                          : make_uint4(0u, 0u, 0u, 0u);
  const float b3 = M.P[OFF_B3 + min(r, MO - 1)];
  bf16x8 w3c = zb;  // W3's entries of the lane's unit: B operand of dH2 = dY W3 (K = 3, padded)
  if (g == 0) {
    uint16_t v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int c = 0; c < MO; ++c) v[c] = M.W3b[(size_t)c * MH + unit];
    w3c = pack8(v);
  }
#pragma unroll
  for (int kc = 0; kc < MH / 32; ++kc) w2t[kc] = load8(M.W2tb + (size_t)unit * MH + 32 * kc + 8 * g);

  f32x4 dW2[MH / 16], dW1[MI / 16], dW3 = zero, db1 = zero, db2 = zero, db3 = zero;
#pragma unroll
  for (int t = 0; t < MH / 16; ++t) dW2[t] = zero;
#pragma unroll
  for (int t = 0; t < MI / 16; ++t) dW1[t] = zero;
  float loss = 0.f;
  const float inv = 1.f / (float)K;

  // a chunk's inputs, loaded one chunk ahead (rows past the batch read its last
  // row and count as zero): x by rows, by columns (waves 2 and 3: features
  // 16 (wv - 2) + r of the rows this lane packs) and the targets (row 16 t + r of
  // tile t: waves 0 and 4, 1 and 5)
  F32x8 xr[2];
  float xc[8], tx = 0.f, ty = 0.f;
  const auto fetch = [&](int ch) {
    const int i0 = ch * kChunk;
#pragma unroll
    for (int t = 0; t < 2; ++t)
      xr[t] = *reinterpret_cast<const F32x8*>(X + (size_t)min(i0 + 16 * t + r, K - 1) * MI + 8 * g);
    if ((wv & 2) == 0) {
      const size_t i = (size_t)min(i0 + 16 * (wv & 1) + r, K - 1);
      tx = T[2 * i];
      ty = T[2 * i + 1];
    } else if (wv < 2 + MI / 16) {  // waves 2 and 3
#pragma unroll
      for (int e = 0; e < 8; ++e)
        xc[e] = X[(size_t)min(i0 + 16 * (e >> 2) + 4 * g + (e & 3), K - 1) * MI + 16 * (wv - 2) + r];
    }
  };
  fetch((int)blockIdx.x);
  for (int ch = (int)blockIdx.x; ch < n_chunks; ch += (int)gridDim.x) {
    const int i0 = ch * kChunk;
    // ---- layer 1 ----
    Quad h1[2], h2[2];
    // rows of a batch's ragged last chunk that exist, as masks of the lane's words
    const bool whole = i0 + kChunk <= K;
    Quad rows[2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int row = i0 + 16 * t + 4 * g + 2 * k;
        rows[t].w[k] = (row < K ? 0xFFFFu : 0u) | (row + 1 < K ? 0xFFFF0000u : 0u);
      }
    const auto only_rows = [&](Quad v, int t) {
      if (!whole) v = {v.w[0] & rows[t].w[0], v.w[1] & rows[t].w[1]};
      return v;
    };
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const f32x4 acc = mfma(pack_f32(xr[t].v, i0 + 16 * t + r < K), w1, zero);
      h1[t] = only_rows(quad_relu(acc, b1), t);
      store_quad(sA, 16 * t + 4 * g, unit, h1[t]);
    }
    sB[wv][lane] = __builtin_bit_cast(uint4, pack_tiles(h1[0], h1[1]));
    if (wv >= 2 && wv < 2 + MI / 16) {
      const Quad x0 = only_rows({bf16_pair(xc[0], xc[1]), bf16_pair(xc[2], xc[3])}, 0);
      const Quad x1 = only_rows({bf16_pair(xc[4], xc[5]), bf16_pair(xc[6], xc[7])}, 1);
      sX[wv - 2][lane] = __builtin_bit_cast(uint4, pack_tiles(x0, x1));
    }
    const float gtx = tx, gty = ty;
    if (ch + (int)gridDim.x < n_chunks) fetch(ch + (int)gridDim.x);
    __syncthreads();
    // ---- layer 2 ----
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      f32x4 acc = zero;
#pragma unroll
      for (int kc = 0; kc < MH / 32; ++kc) acc = mfma(load8(&sA[16 * t + r][32 * kc + 8 * g]), w2[kc], acc);
      h2[t] = only_rows(quad_relu(acc, b2), t);
      store_quad(sH2, 16 * t + 4 * g, unit, h2[t]);
    }
    const bf16x8 h2p = pack_tiles(h2[0], h2[1]);
    __syncthreads();
    // ---- layer 3 and the loss: wave t < 2 takes row tile t, lane l < 16 its row l ----
    if (wv < 2) {
      f32x4 acc = zero;
#pragma unroll
      for (int kc = 0; kc < MH / 32; ++kc)
        acc = mfma(load8(&sH2[16 * wv + r][32 * kc + 8 * g]), __builtin_bit_cast(bf16x8, sW3[kc][lane]), acc);
      if (r < MO) {
#pragma unroll
        for (int q = 0; q < 4; ++q) sY[16 * wv + 4 * g + q][r] = acc[q] + b3;
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      if (lane < 16) {
        // gradient of Huber (1 px) on (16 y0, 16 y1) - target plus BCE of y2
        // against [|guess - target| <= 2 px], mean over the batch; the loss
        // itself is left to waves 4 and 5, off this chain
        const int row = 16 * wv + lane;
        float d0 = 0.f, d1 = 0.f, d2 = 0.f;
        if (i0 + row < K) {
          const float ex = 16.f * sY[row][0] - gtx, ey = 16.f * sY[row][1] - gty, z = sY[row][2];
          const float c = sqrtf(ex * ex + ey * ey) <= 2.f ? 1.f : 0.f;
          d0 = 16.f * fmaxf(-1.f, fminf(1.f, ex)) * inv;
          d1 = 16.f * fmaxf(-1.f, fminf(1.f, ey)) * inv;
          d2 = (1.f / (1.f + expf(-z)) - c) * inv;
        }
        sdY[0][row] = bf16_bits(d0);
        sdY[1][row] = bf16_bits(d1);
        sdY[2][row] = bf16_bits(d2);
      }
    }
    __syncthreads();
    // ---- dH2 = (dY W3) * [h2 > 0] ----
    Quad d2[2], d1[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      uint16_t av[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
      for (int c = 0; c < MO; ++c) av[c] = g == 0 ? sdY[c][16 * t + r] : (uint16_t)0;
      d2[t] = quad_where(quad_of(mfma(pack8(av), w3c, zero)), h2[t]);
      store_quad(sA, 16 * t + 4 * g, unit, d2[t]);
    }
    const bf16x8 d2p = pack_tiles(d2[0], d2[1]);
    __syncthreads();
    // ---- dH1 = (dH2 W2) * [h1 > 0] ----
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      f32x4 acc = zero;
#pragma unroll
      for (int kc = 0; kc < MH / 32; ++kc) acc = mfma(load8(&sA[16 * t + r][32 * kc + 8 * g]), w2t[kc], acc);
      d1[t] = quad_where(quad_of(acc), h1[t]);
    }
    const bf16x8 d1p = pack_tiles(d1[0], d1[1]);
    // ---- weight gradients over the chunk's rows ----
#pragma unroll
    for (int t = 0; t < MH / 16; ++t) dW2[t] = mfma(d2p, __builtin_bit_cast(bf16x8, sB[t][lane]), dW2[t]);
#pragma unroll
    for (int t = 0; t < MI / 16; ++t) dW1[t] = mfma(d1p, __builtin_bit_cast(bf16x8, sX[t][lane]), dW1[t]);
    bf16x8 dyp = zb;  // A operand: row r < 3 is output r
    if (r < MO) {
      const uint2 lo = *reinterpret_cast<const uint2*>(&sdY[r][4 * g]);
      const uint2 hi = *reinterpret_cast<const uint2*>(&sdY[r][16 + 4 * g]);
      dyp = __builtin_bit_cast(bf16x8, make_uint4(lo.x, lo.y, hi.x, hi.y));
    }
    dW3 = mfma(dyp, h2p, dW3);
    db1 = mfma(d1p, ones, db1);
    db2 = mfma(d2p, ones, db2);
    db3 = mfma(dyp, ones, db3);
    if ((wv & 6) == 4 && lane < 16 && i0 + 16 * (wv - 4) + lane < K) {
      const float* y = sY[16 * (wv - 4) + lane];
      const float ex = 16.f * y[0] - gtx, ey = 16.f * y[1] - gty, z = y[2];
      const float hx = fabsf(ex) <= 1.f ? 0.5f * ex * ex : fabsf(ex) - 0.5f;
      const float hy = fabsf(ey) <= 1.f ? 0.5f * ey * ey : fabsf(ey) - 0.5f;
      const float c = sqrtf(ex * ex + ey * ey) <= 2.f ? 1.f : 0.f;
      loss += hx + hy + ((z > 0.f ? z : 0.f) + log1pf(expf(-fabsf(z))) - c * z);
    }
    __syncthreads();  // the next chunk overwrites sA, sB, sX
  }

  // ---- the workgroup's partial gradient ----
  float* P = part + (size_t)blockIdx.x * kPartStride;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int m = 16 * wv + 4 * g + q;  // the gradient row this lane holds
#pragma unroll
    for (int t = 0; t < MI / 16; ++t) P[OFF_W1 + m * MI + 16 * t + r] = dW1[t][q];
#pragma unroll
    for (int t = 0; t < MH / 16; ++t) P[OFF_W2 + m * MH + 16 * t + r] = dW2[t][q];
    if (r == 0) {
      P[OFF_B1 + m] = db1[q];
      P[OFF_B2 + m] = db2[q];
    }
    if (4 * g + q < MO) {
      P[OFF_W3 + (4 * g + q) * MH + unit] = dW3[q];
      if (wv == 0 && r == 0) P[OFF_B3 + q] = db3[q];
    }
  }
  if ((wv & 6) == 4) {
    loss = wave_sum(lane < 16 ? loss : 0.f, lane);
    if (lane == 0) sY[wv - 4][0] = loss;
  }
  __syncthreads();
  if (threadIdx.x == 0) P[kPartLoss] = sY[0][0] + sY[1][0];
}

// Master parameter i and its bf16 copies.
__device__ __forceinline__ void store_copies(const MlpDev& M, int i, float p) {
  const uint16_t b = bf16_bits(p);
  if (i < OFF_B1) {
    M.W1b[i] = b;
  } else if (i >= OFF_W2 && i < OFF_B2) {
    const int j = (i - OFF_W2) / MH, k = (i - OFF_W2) % MH;
    M.W2b[j * MH + k] = b;
    M.W2tb[k * MH + j] = b;
  } else if (i >= OFF_W3 && i < OFF_B3) {
    M.W3b[i - OFF_W3] = b;
  }
}

__global__ void k_mlp_pack(MlpDev M) {
  const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (i < NP) store_copies(M, i, M.P[i]);
}

// ---------------------------------------------------------------------------
// The sum of the partial gradients, in a fixed order: 64 parameters per
// workgroup, each wave the partials w, w + 8, ..., then the eight waves' sums.
// With step == 0 the gradient goes to G; with step >= 1 the parameters take an
// Adam step (beta1 b1, beta2 b2, bias corrections c1, c2) and their bf16
// copies are refreshed. The batch loss goes to *loss (mapped host memory) when
// given. Bound by latency at 32 partials (2.7 MB, 3.9 us) and by reading them at
// 256 (21.7 MB, 4.5 us).
// ---------------------------------------------------------------------------
constexpr int kSumWaves = 8;
__global__ __launch_bounds__(64 * kSumWaves) void k_mlp_sum(MlpDev M, const float* __restrict__ part, int groups,
                                                            float* __restrict__ G, float* loss, float inv, int step,
                                                            float lr, float b1, float b2, float eps, float c1,
                                                            float c2) {
  __shared__ float s[kSumWaves][64];
  const int lane = (int)threadIdx.x & 63, wv = (int)threadIdx.x >> 6;
  const int i = (int)blockIdx.x * 64 + lane;  // < kPartStride
  float a = 0.f;
  if (i <= kPartLoss) {
    const float* src = part + (size_t)wv * kPartStride + i;
#pragma unroll 8
    for (int p = wv; p < groups; p += kSumWaves, src += (size_t)kSumWaves * kPartStride) a += *src;
  }
  s[wv][lane] = a;
  __syncthreads();
  if (wv != 0) return;
#pragma unroll
  for (int w = 1; w < kSumWaves; ++w) a += s[w][lane];
  if (i == kPartLoss) {
    if (loss) *loss = a * inv;
  } else if (i < NP) {
    if (step == 0) {
      G[i] = a;
    } else {
      const float m = b1 * M.m[i] + (1.f - b1) * a;
      const float v = b2 * M.v[i] + (1.f - b2) * a * a;
      M.m[i] = m;
      M.v[i] = v;
      const float p = M.P[i] - lr * (m / c1) / (sqrtf(v / c2) + eps);
      M.P[i] = p;
      store_copies(M, i, p);
    }
  }
}

hipError_t mlp_pack_launch(const MlpDev& M, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_pack, dim3((NP + 255) / 256), dim3(256), 0, s, M);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Library-held training scratch of vio_mlp_gradient_noalloc: one array per
// GPU, held until the process ends, for batches of up to
// VIO_MLP_NOALLOC_MAX_ROWS rows. Host code reaches it only through the
// device address hipGetSymbolAddress returns (per device, at the first call on
// that device); the array's name itself is not a device address on the host.
// ---------------------------------------------------------------------------
static_assert(VIO_MLP_NOALLOC_MAX_ROWS <= 64 * 4 * kChunk, "at most 64 partial gradients (grad_groups)");
constexpr size_t kNoallocBytes = sizeof(float) * 64 * kPartStride;

static __device__ __align__(256) unsigned char scratch[kNoallocBytes];

namespace {
std::mutex g_scratch_mu;
constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices] = {};  // per device ordinal

// the current device's scratch address (looked up once per device, with that
// device current); nullptr on a HIP error
void* noalloc_scratch(int* dev_out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  *dev_out = dev;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return nullptr;
    g_scratch_ptr[dev] = p;
  }
  return g_scratch_ptr[dev];
}
}  // namespace

hipError_t mlp_forward_launch(const MlpDev& M, const float* X, int K, float* Y, hipStream_t s) {
  if (K <= 0) return hipSuccess;
  const int chunks = (K + kChunk - 1) / kChunk;
  launch_kernel(k_mlp_infer, dim3(std::min(chunks, kInferGroups)), dim3(64 * kHidWaves), 0, s, M, X, K, chunks, Y);
  return hipGetLastError();
}

}  // namespace vio

// ===========================================================================
// C ABI
// ===========================================================================
using namespace vio;

struct vio_mlp {
  int max_batch = 0;
  void* arena = nullptr;
  MlpDev M{};
  float* d_part = nullptr;   // partial gradients [grad_groups(max_batch)][kPartStride]
  float* h_loss = nullptr;   // pinned; the sum kernel writes it through hm_loss
  float* hm_loss = nullptr;
  int step = 0;
};

namespace {
size_t up256(size_t v) { return (v + 255) / 256 * 256; }
}  // namespace

extern "C" {

int vio_mlp_create(int32_t max_batch, vio_mlp** out) {
  if (!out || max_batch < 1 || max_batch > 65536) return VIO_EINVAL;
  *out = nullptr;
  auto* m = new (std::nothrow) vio_mlp();
  if (!m) return VIO_ENOMEM;
  m->max_batch = max_batch;
  size_t off = 0;
  auto take = [&](size_t b) {
    const size_t o = off;
    off = up256(off + b);
    return o;
  };
  const size_t oP = take(4 * NP), om = take(4 * NP), ov = take(4 * NP), oW1 = take(2 * MH * MI), oW2 = take(2 * MH * MH),
               oW2t = take(2 * MH * MH), oW3 = take(2 * MO * MH),
               opart = take(sizeof(float) * kPartStride * (size_t)grad_groups(max_batch));
  if (hipMalloc(&m->arena, off) != hipSuccess) {
    delete m;
    return VIO_ENOMEM;
  }
  if (hipMemset(m->arena, 0, off) != hipSuccess ||
      hipHostMalloc((void**)&m->h_loss, sizeof(float)) != hipSuccess ||
      hipHostGetDevicePointer((void**)&m->hm_loss, m->h_loss, 0) != hipSuccess) {
    vio_mlp_destroy(m);
    return VIO_EDEVICE;
  }
  char* b = static_cast<char*>(m->arena);
  m->M = {reinterpret_cast<float*>(b + oP), reinterpret_cast<float*>(b + om), reinterpret_cast<float*>(b + ov),
          reinterpret_cast<uint16_t*>(b + oW1), reinterpret_cast<uint16_t*>(b + oW2),
          reinterpret_cast<uint16_t*>(b + oW2t), reinterpret_cast<uint16_t*>(b + oW3)};
  m->d_part = reinterpret_cast<float*>(b + opart);
  *out = m;
  return VIO_OK;
}

void vio_mlp_destroy(vio_mlp* m) {
  if (!m) return;
  (void)hipDeviceSynchronize();
  if (m->arena) (void)hipFree(m->arena);
  if (m->h_loss) (void)hipHostFree(m->h_loss);
  delete m;
}

int vio_mlp_set_params(vio_mlp* m, const float* params, int32_t n) {
  if (!m || !params || n != NP) return VIO_EINVAL;
  if (hipMemcpy(m->M.P, params, 4 * NP, hipMemcpyHostToDevice) != hipSuccess) return VIO_EDEVICE;
  if (hipMemset(m->M.m, 0, 4 * NP) != hipSuccess || hipMemset(m->M.v, 0, 4 * NP) != hipSuccess) return VIO_EDEVICE;
  m->step = 0;
  if (mlp_pack_launch(m->M, nullptr) != hipSuccess || hipDeviceSynchronize() != hipSuccess) return VIO_EDEVICE;
  return VIO_OK;
}

int vio_mlp_get_params(vio_mlp* m, float* params, int32_t n) {
  if (!m || !params || n < NP) return VIO_EINVAL;
  if (hipDeviceSynchronize() != hipSuccess) return VIO_EDEVICE;
  return hipMemcpy(params, m->M.P, 4 * NP, hipMemcpyDeviceToHost) == hipSuccess ? VIO_OK : VIO_EDEVICE;
}

int vio_mlp_forward(vio_mlp* m, const float* d_x, int32_t k, float* d_y, void* hip_stream) {
  if (!m || !d_x || !d_y || k < 0) return VIO_EINVAL;
  return mlp_forward_launch(m->M, d_x, k, d_y, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? VIO_OK
                                                                                                  : VIO_EDEVICE;
}

// The batch's partial gradients in `part`, then their sum: the gradient in
// d_grad (step == 0) or an Adam step on the parameters (step >= 1); the loss in
// the handle's pinned word.
static int train_impl(vio_mlp* m, const float* d_x, const float* d_t, int k, float* part, float* d_grad, int step,
                      float lr, hipStream_t s) {
  const int chunks = (k + kChunk - 1) / kChunk, groups = grad_groups(k);
  const float b1 = 0.9f, b2 = 0.999f;
  const float c1 = 1.f - std::pow(b1, (float)step), c2 = 1.f - std::pow(b2, (float)step);
  hipLaunchKernelGGL(k_mlp_grad, dim3(groups), dim3(64 * kHidWaves), 0, s, m->M, d_x, d_t, k, chunks, part);
  hipLaunchKernelGGL(k_mlp_sum, dim3(kPartStride / 64), dim3(64 * kSumWaves), 0, s, m->M, (const float*)part, groups,
                     d_grad, m->hm_loss, 1.f / (float)k, step, lr, b1, b2, 1e-8f, c1, c2);
  return hipGetLastError() == hipSuccess ? VIO_OK : VIO_EDEVICE;
}

static int gradient_impl(vio_mlp* m, const float* d_x, const float* d_t, int k, float* part, float* d_grad, float* loss,
                         hipStream_t s) {
  const int rc = train_impl(m, d_x, d_t, k, part, d_grad, 0, 0.f, s);
  if (rc != VIO_OK) return rc;
  if (hipStreamSynchronize(s) != hipSuccess) return VIO_EDEVICE;
  if (loss) *loss = *m->h_loss;
  return VIO_OK;
}

int vio_mlp_gradient(vio_mlp* m, const float* d_x, const float* d_targets, int32_t k, float* d_grad, float* loss,
                     void* hip_stream) {
  if (!m || !d_x || !d_targets || !d_grad || k < 1 || k > m->max_batch) return VIO_EINVAL;
  return gradient_impl(m, d_x, d_targets, k, m->d_part, d_grad, loss, static_cast<hipStream_t>(hip_stream));
}

int vio_mlp_gradient_noalloc(vio_mlp* m, const float* d_x, const float* d_targets, int32_t k, float* d_grad,
                             float* loss, void* hip_stream) {
  if (!m || !d_x || !d_targets || !d_grad || k < 1 || k > VIO_MLP_NOALLOC_MAX_ROWS) return VIO_EINVAL;
  int dev = 0;
  void* base = noalloc_scratch(&dev);
  if (!base) return VIO_EDEVICE;
  return gradient_impl(m, d_x, d_targets, k, static_cast<float*>(base), d_grad, loss,
                       static_cast<hipStream_t>(hip_stream));
}

int vio_mlp_train_step(vio_mlp* m, const float* d_x, const float* d_targets, int32_t k, float lr, float* loss,
                       void* hip_stream) {
  if (!m || !d_x || !d_targets || k < 1 || k > m->max_batch || !(lr > 0.f)) return VIO_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  const int rc = train_impl(m, d_x, d_targets, k, m->d_part, nullptr, m->step + 1, lr, s);
  if (rc != VIO_OK) return rc;
  m->step += 1;
  if (loss) {
    if (hipStreamSynchronize(s) != hipSuccess) return VIO_EDEVICE;
    *loss = *m->h_loss;
  }
  return VIO_OK;
}

}  // extern "C"
