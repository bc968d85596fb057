// Learned surrogate of the fire simulator (include/fire_nn.h): bf16 GEMMs on
// MFMA (v_mfma_f32_32x32x16_bf16, fp32 accumulation) for the MLP and the
// decoder's dense layer, banded upsample+3x3-convolution layers on MFMA (the
// last one, of one channel, on VALU) with bf16 cells between them, fused
// losses, Adam with fp32 master weights.

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <cstdarg>
#include <cstdio>
#include <string>
#include <vector>

#include "fire_nn.h"

namespace firenn {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;

// fp32 -> bf16 with round-to-nearest-even (inputs are finite)
__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float bf16_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
__device__ __forceinline__ float bf16_lo(uint32_t d) { return __uint_as_float(d << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t d) { return __uint_as_float(d & 0xFFFF0000u); }
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  return (uint32_t)f2bf(a) | ((uint32_t)f2bf(b) << 16);
}

int blocks_for(int64_t n, int t = 256) {
  int64_t b = (n + t - 1) / t;
  if (b < 1) b = 1;
  if (b > 65535) b = 65535;
  return (int)b;
}

// ---------------------------------------------------------------------------
// GEMM: 64x64 output tile per workgroup of 4 waves, each wave one 32x32 MFMA
// tile; K staged through two LDS buffers 32 or 64 at a time (the next tile's
// global loads are in flight while the current one is multiplied). Both
// operands are stored in LDS as [row][k] (A rows are m, B rows are n), so
// that each lane's 8 consecutive k of a fragment are contiguous. A thread
// moves 8 bf16 of each operand per tile; how depends on the operand's
// strides (LoadMode).
constexpr int kTM = 64, kTN = 64, kTK = 32, kLdt = kTK + 8;

// kAlongK: k is contiguous (stride 1) and rows start on 16-byte boundaries:
//   one 16-byte load per thread, one 16-byte LDS store.
// kAlongRows: rows are contiguous and k-slices start on 16-byte boundaries:
//   one 16-byte load of 8 rows at one k, 8 two-byte LDS stores.
// kElementwise: any strides, 8 two-byte loads.
enum LoadMode { kElementwise = 0, kAlongK = 1, kAlongRows = 2 };

template <int MODE>
__device__ __forceinline__ void tile_load(const uint16_t *base, int64_t sr, int64_t sk, int row0,
                                          int rows, int k0, int kdim, int t, uint16_t v[8]) {
  if (MODE == kAlongK) {
    const int row = row0 + (t >> 2), k = k0 + (t & 3) * 8;
    if (row < rows && k + 8 <= kdim) {
      const uint4 q = *reinterpret_cast<const uint4 *>(base + (int64_t)row * sr + k);
      const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        v[2 * j] = (uint16_t)(w[j] & 0xFFFFu);
        v[2 * j + 1] = (uint16_t)(w[j] >> 16);
      }
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        v[i] = (row < rows && k + i < kdim) ? base[(int64_t)row * sr + k + i] : (uint16_t)0;
    }
  } else if (MODE == kAlongRows) {
    const int k = k0 + (t >> 3), row = row0 + (t & 7) * 8;
    if (k < kdim && row + 8 <= rows) {
      const uint4 q = *reinterpret_cast<const uint4 *>(base + (int64_t)k * sk + row);
      const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        v[2 * j] = (uint16_t)(w[j] & 0xFFFFu);
        v[2 * j + 1] = (uint16_t)(w[j] >> 16);
      }
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        v[i] = (k < kdim && row + i < rows) ? base[(int64_t)k * sk + row + i] : (uint16_t)0;
    }
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int e = t + 256 * i;
      const int row = row0 + (e >> 5), k = k0 + (e & 31);
      v[i] = (row < rows && k < kdim) ? base[(int64_t)row * sr + (int64_t)k * sk] : (uint16_t)0;
    }
  }
}

template <int MODE>
__device__ __forceinline__ void tile_store(uint16_t *S, int t, const uint16_t v[8]) {
  if (MODE == kAlongK) {
    uint4 q;
    q.x = (uint32_t)v[0] | ((uint32_t)v[1] << 16);
    q.y = (uint32_t)v[2] | ((uint32_t)v[3] << 16);
    q.z = (uint32_t)v[4] | ((uint32_t)v[5] << 16);
    q.w = (uint32_t)v[6] | ((uint32_t)v[7] << 16);
    *reinterpret_cast<uint4 *>(&S[(t >> 2) * kLdt + (t & 3) * 8]) = q;
  } else if (MODE == kAlongRows) {
    const int kk = t >> 3, r = (t & 7) * 8;
#pragma unroll
    for (int i = 0; i < 8; ++i) S[(r + i) * kLdt + kk] = v[i];
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int e = t + 256 * i;
      S[(e >> 5) * kLdt + (e & 31)] = v[i];
    }
  }
}

// One problem of a launch: C = op(A) op(B) (+ bias) (+ C), C or Cb may be NULL.
struct GemmArgs {
  int M, N, K;
  const uint16_t *A;
  int64_t sam, sak;
  const uint16_t *B;
  int64_t sbk, sbn;
  float *C;
  int64_t ldc;
  const float *bias;
  int relu, accumulate;
  uint16_t *Cb;
};
// The problems of a launch, which fill the chip together: problem p's tiles
// are blocks first[p] .. first[p + 1] - 1. The five weight gradients over 512
// rows (168 workgroups): 18.6 us, after 81 us for five launches of 4 to 128.
constexpr int kMaxGemms = 5;
struct GemmBatch {
  GemmArgs p[kMaxGemms];
  int first[kMaxGemms + 1];
};

// STAGES tiles of kTK per LDS buffer. With two, their loads are in flight
// together, so a workgroup waits for memory once in 64 k (a weight gradient over
// 512 rows took 16 waits of about 1.1 us with one tile a buffer); but twice the
// LDS leaves 4 workgroups a compute unit in place of 8 (two_stages).
template <int AM, int BM, int STAGES>
__device__ __forceinline__ void gemm_tile(const GemmArgs &q, int m0, int n0) {
  __shared__ __attribute__((aligned(16))) uint16_t As[2][STAGES][kTM * kLdt];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[2][STAGES][kTN * kLdt];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
  f32x16_t acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
  uint16_t va[STAGES][8], vb[STAGES][8];
  auto load = [&](int k0) {
#pragma unroll
    for (int j = 0; j < STAGES; ++j) {
      tile_load<AM>(q.A, q.sam, q.sak, m0, q.M, k0 + j * kTK, q.K, tid, va[j]);
      tile_load<BM>(q.B, q.sbn, q.sbk, n0, q.N, k0 + j * kTK, q.K, tid, vb[j]);
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int j = 0; j < STAGES; ++j) {
      tile_store<AM>(As[buf][j], tid, va[j]);
      tile_store<BM>(Bs[buf][j], tid, vb[j]);
    }
  };
  load(0);
  store(0);
  __syncthreads();
  const int half = lane >> 5, r = lane & 31;
  int buf = 0;
  for (int k0 = 0; k0 < q.K; k0 += STAGES * kTK) {
    const bool more = k0 + STAGES * kTK < q.K;
    if (more) load(k0 + STAGES * kTK);
#pragma unroll
    for (int j = 0; j < STAGES; ++j) {
      if (k0 + j * kTK >= q.K) break;
#pragma unroll
      for (int kk = 0; kk < kTK; kk += 16) {
        const bf16x8_t a =
            *reinterpret_cast<const bf16x8_t *>(&As[buf][j][(wr + r) * kLdt + kk + half * 8]);
        const bf16x8_t b =
            *reinterpret_cast<const bf16x8_t *>(&Bs[buf][j][(wc + r) * kLdt + kk + half * 8]);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
      }
    }
    if (more) store(buf ^ 1);  // last read before the previous barrier
    __syncthreads();
    buf ^= 1;
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int i = wr + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
    const int j = wc + (lane & 31);
    const int m = m0 + i, n = n0 + j;
    if (m < q.M && n < q.N) {
      float val = acc[v];
      if (q.bias) val += q.bias[n];
      if (q.accumulate) val += q.C[(int64_t)m * q.ldc + n];
      if (q.relu) val = fmaxf(val, 0.0f);
      if (q.C) q.C[(int64_t)m * q.ldc + n] = val;
      if (q.Cb) q.Cb[(int64_t)m * q.ldc + n] = f2bf(val);
    }
  }
}

template <int AM, int BM, int STAGES>
__global__ __launch_bounds__(256) void gemm_kernel(GemmArgs q) {
  gemm_tile<AM, BM, STAGES>(q, (int)blockIdx.y * kTM, (int)blockIdx.x * kTN);
}

template <int AM, int BM>
__global__ __launch_bounds__(256) void gemm_batch_kernel(GemmBatch batch) {
  int i = 0;
#pragma unroll
  for (int k = 1; k < kMaxGemms; ++k) i += (int)blockIdx.x >= batch.first[k] ? 1 : 0;
  const GemmArgs &q = batch.p[i];
  const int tile = (int)blockIdx.x - batch.first[i], nt = (q.N + kTN - 1) / kTN;
  gemm_tile<AM, BM, 2>(q, tile / nt * kTM, tile % nt * kTN);
}

int64_t gemm_tiles(const GemmArgs &q) {
  return (int64_t)((q.M + kTM - 1) / kTM) * ((q.N + kTN - 1) / kTN);
}

// n problems in one launch, every operand with load mode AM, BM
template <int AM, int BM>
hipError_t gemm_batch(const GemmArgs *q, int n, hipStream_t s) {
  GemmBatch batch{};
  int at = 0;
  for (int i = 0; i < kMaxGemms; ++i) {
    batch.first[i] = i < n ? at : 0x7FFFFFFF;
    if (i < n) {
      batch.p[i] = q[i];
      at += (int)gemm_tiles(q[i]);
    }
  }
  hipLaunchKernelGGL((gemm_batch_kernel<AM, BM>), dim3(at), dim3(256), 0, s, batch);
  return hipGetLastError();
}

// Whether a product takes two tiles a buffer: where a compute unit has one
// workgroup at most, nothing else hides its waits (512x2048x256, B transposed:
// 6.4 us with two, 6.7 with one), and a long contraction repays the workgroups
// that the LDS takes (2048x2048x2048: 39.8 and 45.1 us). Short contractions
// only pay for the second tile (300x4000x32: 6.0 and 4.9 us), and many tiles hide
// the waits themselves (65536x256x256: 37.1 and 34.2 us, 65536x2048x64: 175 and
// 139 us; at 512 tiles and K = 256 the two are within 3%).
bool two_stages(const GemmArgs &q) { return q.K >= 1024 || (q.K >= 256 && gemm_tiles(q) <= 256); }

// how an operand of `rows` x `kdim` with strides (sr, sk) is loaded
int load_mode(const uint16_t *p, int64_t sr, int64_t sk) {
  if ((reinterpret_cast<uintptr_t>(p) & 15u) != 0) return kElementwise;
  if (sk == 1 && sr % 8 == 0) return kAlongK;
  if (sr == 1 && sk % 8 == 0) return kAlongRows;
  return kElementwise;
}

template <int AM, int STAGES>
hipError_t gemm_b(int bm, const GemmArgs &q, hipStream_t s) {
  const dim3 grid((unsigned)((q.N + kTN - 1) / kTN), (unsigned)((q.M + kTM - 1) / kTM));
  if (bm == kAlongK) hipLaunchKernelGGL((gemm_kernel<AM, kAlongK, STAGES>), grid, dim3(256), 0, s, q);
  else if (bm == kAlongRows) hipLaunchKernelGGL((gemm_kernel<AM, kAlongRows, STAGES>), grid, dim3(256), 0, s, q);
  else hipLaunchKernelGGL((gemm_kernel<AM, kElementwise, STAGES>), grid, dim3(256), 0, s, q);
  return hipGetLastError();
}

template <int STAGES>
hipError_t gemm_a(int am, int bm, const GemmArgs &q, hipStream_t s) {
  if (am == kAlongK) return gemm_b<kAlongK, STAGES>(bm, q, s);
  if (am == kAlongRows) return gemm_b<kAlongRows, STAGES>(bm, q, s);
  return gemm_b<kElementwise, STAGES>(bm, q, s);
}

hipError_t gemm(int M, int N, int K, const uint16_t *A, int64_t sam, int64_t sak,
                const uint16_t *B, int64_t sbk, int64_t sbn, float *C, int64_t ldc,
                const float *bias, int relu, int accumulate, uint16_t *Cb, hipStream_t s) {
  const GemmArgs q{M, N, K, A, sam, sak, B, sbk, sbn, C, ldc, bias, relu, accumulate, Cb};
  const int am = load_mode(A, sam, sak), bm = load_mode(B, sbn, sbk);
  return two_stages(q) ? gemm_a<2>(am, bm, q, s) : gemm_a<1>(am, bm, q, s);
}

// ---------------------------------------------------------------------------
// The MLP's forward pass in one launch: a workgroup of 8 waves takes 32 rows
// through all layers, activations in LDS, wave w computing columns 32 w ..
// 32 w + 31 of each layer with 32x32x16 MFMAs in ascending k (the sums of
// gemm_kernel, bit for bit). The weights are read from their transposed bf16
// copy `wt` (fire_nn), whose rows hold a lane's 8 consecutive k in one 16-byte
// load; all of a layer's loads are in flight before its first MFMA, and a
// layer's begin before the previous one's barrier. What bounds it is that
// chain of three layers (load latency, 16 dependent MFMAs, two barriers) and
// the launch: a scoring call of 498 rows takes 12.5 us, against 39.8 us for
// five launches of 8 to 32 workgroups and a copy.
constexpr int kMlpH = 256, kMlpIn = 16, kMlpRows = 32, kMlpLd = kMlpH + 8;
constexpr int kMlpThreads = 512;
// parts of the contraction over the decoder's 2048 in the error of h3, each its
// own tiles of the launch (four times the 32 workgroups of 512 rows)
constexpr int kDhParts = 4;

// acc += act[32][K] times the wave's 32 columns of w ([256][K] transposed
// weights, w at the wave's first column's row)
template <int K>
__device__ __forceinline__ void mlp_load(const uint16_t *w, int lane, uint4 (&b)[K / 16]) {
#pragma unroll
  for (int s = 0; s < K / 16; ++s)
    b[s] = *reinterpret_cast<const uint4 *>(w + (lane & 31) * K + 16 * s + 8 * (lane >> 5));
}

template <int K>
__device__ __forceinline__ f32x16_t mlp_tile(const uint16_t *act, int lane, const uint4 (&b)[K / 16]) {
  f32x16_t acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
#pragma unroll
  for (int s = 0; s < K / 16; ++s) {
    const bf16x8_t a = *reinterpret_cast<const bf16x8_t *>(&act[(lane & 31) * kMlpLd + 16 * s + 8 * (lane >> 5)]);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, __builtin_bit_cast(bf16x8_t, b[s]), acc, 0, 0, 0);
  }
  return acc;
}

__global__ __launch_bounds__(kMlpThreads) void mlp_forward_kernel(
    const float *x, int B, float inv_w, float inv_h, const uint16_t *w1t, const uint16_t *w2t,
    const uint16_t *w3t, const uint16_t *wf, const float *c1, const float *c2, const float *c3,
    const float *cf, uint16_t *xb, uint16_t *h1b, uint16_t *h2b, uint16_t *h3b, float *t) {
  __shared__ __attribute__((aligned(16))) uint16_t act[2][kMlpRows * kMlpLd];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row0 = blockIdx.x * kMlpRows, col = 32 * wave + (lane & 31);
  uint4 b1[1], b2[16];
  mlp_load<kMlpIn>(w1t + 32 * wave * kMlpIn, lane, b1);
  mlp_load<kMlpH>(w2t + 32 * wave * kMlpH, lane, b2);
  {
    // the inputs: beta / 30, ignition scaled to [-1, 1], zero padding
    const int r = tid >> 4, k = tid & 15, b = row0 + r;
    float v = 0.0f;
    if (b < B) {
      if (k < 5) v = x[b * 7 + k] * (1.0f / 30.0f);
      else if (k == 5) v = 2.0f * x[b * 7 + 5] * inv_w - 1.0f;
      else if (k == 6) v = 2.0f * x[b * 7 + 6] * inv_h - 1.0f;
    }
    const uint16_t q = f2bf(v);
    act[0][r * kMlpLd + k] = q;
    if (xb && b < B) xb[(int64_t)b * kMlpIn + k] = q;
  }
  __syncthreads();
  // a layer's outputs: bias, ReLU, bf16, into the next layer's buffer
  auto finish = [&](const f32x16_t &acc, const float *bias, uint16_t *to) {
    const float bc = bias[col];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int i = 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
      to[i * kMlpLd + col] = f2bf(fmaxf(acc[v] + bc, 0.0f));
    }
  };
  // the workgroup's rows of a layer to global memory
  auto keep = [&](const uint16_t *from, uint16_t *h) {
    if (!h) return;
    for (int i = tid; i < kMlpRows * (kMlpH / 8); i += kMlpThreads) {
      const int r = i / (kMlpH / 8), k = (i % (kMlpH / 8)) * 8;
      if (row0 + r < B)
        *reinterpret_cast<uint4 *>(h + (int64_t)(row0 + r) * kMlpH + k) =
            *reinterpret_cast<const uint4 *>(&from[r * kMlpLd + k]);
    }
  };
  finish(mlp_tile<kMlpIn>(act[0], lane, b1), c1, act[1]);
  __syncthreads();
  keep(act[1], h1b);
  const f32x16_t a2 = mlp_tile<kMlpH>(act[1], lane, b2);
  mlp_load<kMlpH>(w3t + 32 * wave * kMlpH, lane, b2);
  finish(a2, c2, act[0]);
  __syncthreads();
  keep(act[0], h2b);
  const f32x16_t a3 = mlp_tile<kMlpH>(act[0], lane, b2);
  finish(a3, c3, act[1]);
  __syncthreads();
  keep(act[1], h3b);
  if (wave == 0) {
    // the fitness head: one column
    uint4 bf[16];
#pragma unroll
    for (int s = 0; s < 16; ++s) {
      bf[s] = make_uint4(0u, 0u, 0u, 0u);
      if ((lane & 31) == 0) bf[s] = *reinterpret_cast<const uint4 *>(wf + 16 * s + 8 * (lane >> 5));
    }
    const f32x16_t q = mlp_tile<kMlpH>(act[1], lane, bf);
    if ((lane & 31) == 0) {
      const float c = cf[0];
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int i = row0 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
        if (i < B) t[i] = q[v] + c;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Elementwise and reduction kernels

// Where the second bf16 copy `wt` holds parameter i: W1, W2, W3 as [out][in],
// then Wf and Wd as they are, but on 16-byte boundaries (Wd's first element is
// an odd one in the flat order); -1 for the others. off: the first elements of
// W1, W2, W3, Wf and Wd in the flat order.
struct MlpOffsets {
  int64_t w1, w2, w3, wf, wd, wd_n;
};
__device__ __forceinline__ int64_t wt_index(const MlpOffsets &o, int64_t i) {
  constexpr int64_t kIn = kMlpIn * kMlpH, kSq = kMlpH * kMlpH;
  if (i < o.w1 + kIn) return i < o.w1 ? -1 : (i - o.w1) % kMlpH * kMlpIn + (i - o.w1) / kMlpH;
  if (i < o.w2 + kSq) return i < o.w2 ? -1 : kIn + (i - o.w2) % kMlpH * kMlpH + (i - o.w2) / kMlpH;
  if (i < o.w3 + kSq) return i < o.w3 ? -1 : kIn + kSq + (i - o.w3) % kMlpH * kMlpH + (i - o.w3) / kMlpH;
  if (i < o.wf + kMlpH) return i < o.wf ? -1 : kIn + 2 * kSq + (i - o.wf);
  return i >= o.wd && i < o.wd + o.wd_n ? kIn + 2 * kSq + kMlpH + (i - o.wd) : -1;
}

// the bf16 copies of the master weights
__global__ void refresh_weights_kernel(const float *w, uint16_t *wb, uint16_t *wt, MlpOffsets off,
                                       int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const uint16_t q = f2bf(w[i]);
    wb[i] = q;
    const int64_t t = wt_index(off, i);
    if (t >= 0) wt[t] = q;
  }
}

// The MLP's error chain in one launch, 32 rows a workgroup as in the forward
// pass: e3 = dt Wf^T + the kDhParts parts of dd0 Wd^T (dh, NULL without maps),
// e2 = e3' W3^T, e1 = e2' W2^T, each masked by its layer's ReLU (h the bf16
// activations), to g (fp32, for the bias gradients) and gb (bf16, what the next
// product and the weight gradients read). W3 and W2 are read along their rows,
// which is along k here. Bound, as the forward pass, by the chain itself (16
// workgroups at 512 rows): 15.5 us at 512 rows with every mask and error loaded
// ahead (41 us with a branch per row), after 86 us for three ReLU passes, two
// products, the rank-one product and an accumulating one over 2048.
__global__ __launch_bounds__(kMlpThreads) void mlp_backward_kernel(
    const uint16_t *dtb, const float *dh, int64_t part_stride, int B, const uint16_t *wf,
    const uint16_t *w3, const uint16_t *w2, const uint16_t *h3b, const uint16_t *h2b,
    const uint16_t *h1b, float *g3, float *g2, float *g1, uint16_t *gb3, uint16_t *gb2, uint16_t *gb1) {
  __shared__ __attribute__((aligned(16))) uint16_t act[2][kMlpRows * kMlpLd];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row0 = blockIdx.x * kMlpRows, col = 32 * wave + (lane & 31);
  uint4 w[16];
  mlp_load<kMlpH>(w3 + 32 * wave * kMlpH, lane, w);
  // this lane's outputs of a layer: rows row(v), column col. Loads take the
  // last row in place of the rows past it, so that none waits for a branch.
  auto row = [&](int v) { return row0 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3); };
  auto mask_load = [&](const uint16_t *h, uint16_t (&m)[16]) {
#pragma unroll
    for (int v = 0; v < 16; ++v) m[v] = h[(int64_t)min(row(v), B - 1) * kMlpH + col];
  };
  uint16_t m2[16], m1[16];
  mask_load(h2b, m2);
  constexpr int kQuads = kMlpRows * kMlpH / 4 / kMlpThreads;
  const int n = tid % (kMlpH / 4) * 4, r0 = tid / (kMlpH / 4);
  float4 d[kQuads];
  uint2 m3[kQuads];
  float dt[kQuads];
#pragma unroll
  for (int i = 0; i < kQuads; ++i) {
    const int b = min(row0 + r0 + i * (kMlpRows / kQuads), B - 1);
    const int64_t o = (int64_t)b * kMlpH + n;
    dt[i] = bf16_f32(dtb[b]);
    m3[i] = *reinterpret_cast<const uint2 *>(h3b + o);
    d[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (dh) {
      d[i] = *reinterpret_cast<const float4 *>(dh + o);
#pragma unroll
      for (int k = 1; k < kDhParts; ++k) {
        const float4 q = *reinterpret_cast<const float4 *>(dh + k * part_stride + o);
        d[i].x += q.x;
        d[i].y += q.y;
        d[i].z += q.z;
        d[i].w += q.w;
      }
    }
  }
  const uint2 wq = *reinterpret_cast<const uint2 *>(wf + n);
  const float wn[4] = {bf16_lo(wq.x), bf16_hi(wq.x), bf16_lo(wq.y), bf16_hi(wq.y)};
#pragma unroll
  for (int i = 0; i < kQuads; ++i) {
    const int r = r0 + i * (kMlpRows / kQuads), b = row0 + r;
    const float h[4] = {bf16_lo(m3[i].x), bf16_hi(m3[i].x), bf16_lo(m3[i].y), bf16_hi(m3[i].y)};
    const float dd[4] = {d[i].x, d[i].y, d[i].z, d[i].w};
    float v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = b < B && h[j] > 0.0f ? dd[j] + dt[i] * wn[j] : 0.0f;
    const uint2 q = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
    *reinterpret_cast<uint2 *>(&act[0][r * kMlpLd + n]) = q;
    if (b < B) {
      *reinterpret_cast<float4 *>(g3 + (int64_t)b * kMlpH + n) = make_float4(v[0], v[1], v[2], v[3]);
      *reinterpret_cast<uint2 *>(gb3 + (int64_t)b * kMlpH + n) = q;
    }
  }
  __syncthreads();
  auto finish = [&](const f32x16_t &acc, const uint16_t (&m)[16], float *g, uint16_t *gb, uint16_t *to) {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const float val = row(v) < B && bf16_f32(m[v]) > 0.0f ? acc[v] : 0.0f;
      const uint16_t q = f2bf(val);
      if (to) to[(row(v) - row0) * kMlpLd + col] = q;
      if (row(v) < B) {
        const int64_t o = (int64_t)row(v) * kMlpH + col;
        g[o] = val;
        gb[o] = q;
      }
    }
  };
  const f32x16_t a2 = mlp_tile<kMlpH>(act[0], lane, w);
  mlp_load<kMlpH>(w2 + 32 * wave * kMlpH, lane, w);
  mask_load(h1b, m1);
  finish(a2, m2, g2, gb2, act[1]);
  __syncthreads();
  finish(mlp_tile<kMlpH>(act[1], lane, w), m1, g1, gb1, nullptr);
}

// column sums of d [M][N] (bias gradients) in a fixed order: a workgroup of
// 256 threads takes 16 columns; row group r (0..15) sums rows r, r+16, ...
// in order (eight loads in flight), then the 16 partial sums are added
// pairwise: p0+p1, p2+p3, ..., then those pairwise, down to one. Several
// matrices of M rows in one launch: matrix i has blocks first[i] .. The five
// bias gradients over 512 rows: 4.9 us, after 51 us for five launches.
constexpr int kColsumCols = 16, kColsumGroups = 16, kMaxColsums = 5;
struct Colsums {
  const float *d[kMaxColsums];
  float *out[kMaxColsums];
  int N[kMaxColsums], first[kMaxColsums];
};
__global__ __launch_bounds__(256) void colsum_kernel(Colsums q, int M) {
  __shared__ float part[kColsumGroups][kColsumCols];
  int k = 0;
#pragma unroll
  for (int i = 1; i < kMaxColsums; ++i) k += (int)blockIdx.x >= q.first[i] ? 1 : 0;
  const float *d = q.d[k];
  const int N = q.N[k];
  const int c = threadIdx.x % kColsumCols, rg = threadIdx.x / kColsumCols;
  const int n = ((int)blockIdx.x - q.first[k]) * kColsumCols + c;
  float s = 0.0f;
  if (n < N) {
    int m = rg;
    for (; m + 7 * kColsumGroups < M; m += 8 * kColsumGroups) {
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = d[(int64_t)(m + j * kColsumGroups) * N + n];
#pragma unroll
      for (int j = 0; j < 8; ++j) s += v[j];
    }
    for (; m < M; m += kColsumGroups) s += d[(int64_t)m * N + n];
  }
  part[rg][c] = s;
  __syncthreads();
  if (rg == 0 && n < N) {
    float p[kColsumGroups];
#pragma unroll
    for (int i = 0; i < kColsumGroups; ++i) p[i] = part[i][c];
#pragma unroll
    for (int w = kColsumGroups; w > 1; w >>= 1)
#pragma unroll
      for (int i = 0; i < w / 2; ++i) p[i] = p[2 * i] + p[2 * i + 1];
    q.out[k][n] = p[0];
  }
}

// the column sums of n matrices d[i] [M][N[i]] into out[i]
hipError_t colsums(const float *const *d, const int *N, float *const *out, int n, int M, hipStream_t s) {
  Colsums q{};
  int at = 0;
  for (int i = 0; i < kMaxColsums; ++i) {
    q.first[i] = i < n ? at : 0x7FFFFFFF;
    if (i >= n) continue;
    q.d[i] = d[i];
    q.out[i] = out[i];
    q.N[i] = N[i];
    at += (N[i] + kColsumCols - 1) / kColsumCols;
  }
  hipLaunchKernelGGL(colsum_kernel, dim3(at), dim3(256), 0, s, q, M);
  return hipGetLastError();
}

__device__ float block_reduce(float v, float *red) {
  const int t = threadIdx.x;
  red[t] = v;
  __syncthreads();
  for (int o = blockDim.x / 2; o > 0; o >>= 1) {
    if (t < o) red[t] += red[t + o];
    __syncthreads();
  }
  const float r = red[0];
  __syncthreads();
  return r;
}

// fitness head: loss = mean((t - y)^2), dt = 2 (t - y) / B
__global__ __launch_bounds__(256) void loss_fit_kernel(const float *t, const float *y, int B,
                                                       float *dt, uint16_t *dtb, float *loss) {
  __shared__ float red[256];
  float acc = 0.0f;
  for (int b = threadIdx.x; b < B; b += 256) {
    const float e = t[b] - y[b];
    acc += e * e;
    const float g = 2.0f * e / (float)B;
    dt[b] = g;
    dtb[b] = f2bf(g);
  }
  const float s = block_reduce(acc, red);
  if (threadIdx.x == 0) loss[0] = s / (float)B;
}

__global__ __launch_bounds__(256) void sum_partials_kernel(const float *p, int n, float scale,
                                                           float *out) {
  __shared__ float red[256];
  float acc = 0.0f;
  for (int i = threadIdx.x; i < n; i += 256) acc += p[i];
  const float s = block_reduce(acc, red);
  if (threadIdx.x == 0) out[0] = s * scale;
}

// ---------------------------------------------------------------------------
// Decoder convolutions. A layer is out = conv3x3(up2(in)) with zero padding, in
// [8][S][S] and out [Co][2S][2S]; activations, kernels and back-propagated
// errors are bf16, sums fp32. Between the layers, activations and errors are
// bf16 only (the ReLU masks come from them) and channel-interleaved,
// [row][col][8]: a cell is one 16-byte load, store and MFMA fragment. (The dense
// layer's d0 and its gradient are planar, [8][16][16].) Workgroups take bands
// of rows, staged in LDS with a border of zeros so that no tap is tested
// against the edge, and every LDS offset of a lane is fixed before the loop.
//
// Products on v_mfma_f32_16x16x32_bf16: A 16x32 with lane l holding row l%16
// and k 8*(l/16)..+8; B 32x16 with lane l holding column l%16 and the same k;
// D 16x16 with lane l holding column l%16 and rows 4*(l/16)..+4. Rows are the
// channels and columns 16 pixels, so that a lane holds four channels of one
// pixel and stores 8 bytes; k = tap * 8 + channel in ascending order.
//
// With fp32 copies of every plane, bounds tests per tap and two-byte staging,
// a training batch of 512 spent 740 of its 890 us in these layers and the map
// loss: last forward layer 146, its loss and bf16 copy 57, its gradients 94,
// the other gradients 226, the other forward layers 78 us (rocprofv3). Now the
// last layer takes 40 with the loss (its 32 products and one exponential a pixel
// on VALU), its gradients 41 (73 sums a thread on VALU; 84 MB of traffic would
// take 18 at the 4.8 TB/s of a copy), the others 20 + 20 + 10 + 7 and 18 + 8 us,
// and the whole batch 260 us.
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;
typedef uint16_t u16x8_t __attribute__((ext_vector_type(8)));
constexpr int kConvCi = 8, kConvTaps = 9, kConvK = kConvCi * kConvTaps;  // 72
constexpr int kWgradCols = 80;  // 72 kernel taps, the bias column, padding
constexpr int kWgradRows = 16;  // output channels, padded
// workgroups of the gradient kernels that keep sums across samples: each adds
// its sums once, so a few samples a workgroup pay for it
constexpr int kConvGrid = 512, kCo1Grid = 1024;
constexpr int kWgradParts = kConvGrid > kCo1Grid ? kConvGrid : kCo1Grid;

__device__ __forceinline__ bf16x8_t as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8_t, v); }

// Cell (y, x) of a sample's [8][R][R] planes (PLANAR) or [R][R][8] cells.
template <bool PLANAR>
__device__ __forceinline__ uint4 load_cell(const uint16_t *src, int R, int y, int x) {
  if constexpr (PLANAR) {
    uint16_t v[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) v[c] = src[(c * R + y) * R + x];
    return make_uint4((uint32_t)v[0] | ((uint32_t)v[1] << 16), (uint32_t)v[2] | ((uint32_t)v[3] << 16),
                      (uint32_t)v[4] | ((uint32_t)v[5] << 16), (uint32_t)v[6] | ((uint32_t)v[7] << 16));
  } else {
    return reinterpret_cast<const uint4 *>(src)[y * R + x];
  }
}

// Rows row0 - 1 .. row0 + rows of a sample's R x R cells with a column to each
// side, zero outside, into cells [rows + 2][R + 2].
template <bool PLANAR>
__device__ __forceinline__ void stage_cells(uint4 *cells, const uint16_t *src, int R, int row0, int rows) {
  for (int i = threadIdx.x; i < (rows + 2) * (R + 2); i += blockDim.x) {
    const int y = row0 - 1 + i / (R + 2), x = i % (R + 2) - 1;
    cells[i] = (unsigned)y < (unsigned)R && (unsigned)x < (unsigned)R ? load_cell<PLANAR>(src, R, y, x)
                                                                      : make_uint4(0u, 0u, 0u, 0u);
  }
}

// Kernel fragments of the three k-steps for row `row` of the result: FWD the
// output channel (k over tap, input channel), else the input channel.
template <bool FWD>
__device__ __forceinline__ void kernel_fragments(const uint16_t *Kb, int row, int kq, bf16x8_t (&w)[3]) {
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    const int t = 4 * s + kq;
    u16x8_t v;
#pragma unroll
    for (int i = 0; i < 8; ++i)
      v[i] = t < kConvTaps && row < kConvCi
                 ? Kb[FWD ? (row * kConvCi + i) * kConvTaps + t : (i * kConvCi + row) * kConvTaps + t]
                 : (uint16_t)0;
    w[s] = __builtin_bit_cast(bf16x8_t, v);
  }
}

// Forward, 8 output channels: out[y][x][co] = relu(bias[co] + sum over taps and
// channels of K[co][ci][dy][dx] in[(y+dy-1)/2][(x+dx-1)/2][ci]). A
// workgroup: kBand output rows of a sample; a wave's rows have one parity, so the
// source cells of its taps lie at fixed offsets from the pixel's cell.
template <int S, bool PLANAR_IN>
__global__ __launch_bounds__(256) void upconv_kernel(const uint16_t *src, const uint16_t *Kb,
                                                     const float *bias, uint16_t *out) {
  constexpr int O = 2 * S, kBand = 32, kBands = O / kBand, kLd = S + 2;
  __shared__ __attribute__((aligned(16))) uint4 cells[(kBand / 2 + 2) * kLd];
  const int b = blockIdx.x / kBands, y0 = (blockIdx.x % kBands) * kBand;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, px = lane & 15, kq = lane >> 4;
  stage_cells<PLANAR_IN>(cells, src + (int64_t)b * kConvCi * S * S, S, y0 / 2, kBand / 2);
  bf16x8_t w[3];
  kernel_fragments<true>(Kb, px, kq, w);
  float bc[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) bc[v] = kq < 2 ? bias[4 * kq + v] : 0.0f;
  int off[3];
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    const int t = min(4 * s + kq, kConvTaps - 1);
    off[s] = ((((wave & 1) + t / 3 - 1) >> 1) + 1) * kLd + (((px & 1) + t % 3 - 1) >> 1) + 1 + (px >> 1);
  }
  __syncthreads();
  for (int r = wave; r < kBand; r += 4)
#pragma unroll
    for (int x0 = 0; x0 < O; x0 += 16) {
      const int base = (r >> 1) * kLd + x0 / 2;
      f32x4_t acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int s = 0; s < 3; ++s) {
        // (the third step has one tap: the other lanes read a border cell, zero)
        const int at = s < 2 || kq == 0 ? base + off[s] : 0;
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[s], as_bf16x8(cells[at]), acc, 0, 0, 0);
      }
      if (kq < 2) {
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = fmaxf(acc[i] + bc[i], 0.0f);
        *reinterpret_cast<uint2 *>(out + (((int64_t)b * O + y0 + r) * O + x0 + px) * kConvCi + 4 * kq) =
            make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
      }
    }
}

// 1 / x for x in [1, 3], one Newton step on the hardware's reciprocal
__device__ __forceinline__ float recip(float x) {
  const float r = __builtin_amdgcn_rcpf(x);
  return fmaf(r, fmaf(-x, r, 1.0f), r);
}

// log(1 + e) for e in [0, 1] (NaN to NaN): 2 atanh(s), s = e / (2 + e) <= 1/3,
// by its series in s^2 up to s^17 (the next term is below 2^-32 of the sum).
__device__ __forceinline__ float log1p_unit(float e) {
  const float s = e * recip(2.0f + e), q = s * s;
  float p = 1.0f / 17.0f;
#pragma unroll
  for (int k = 15; k >= 3; k -= 2) p = fmaf(p, q, 1.0f / (float)k);
  return 2.0f * fmaf(p * q, s, s);
}

// Last layer, one output channel, S = 64: an MFMA would fill one row of 16, so
// a thread takes two adjacent input cells and computes their eight output
// pixels on VALU. With nearest upsampling the nine taps of a pixel read four
// cells, and the taps on one cell are added first (fp32): 32 products a pixel.
// The epilogue is fused: TRAIN the map loss and its gradient, dz = w (sigmoid(z)
// - y) / n in bf16, the workgroup's partial loss to partial[block]; else
// sigmoid(z). What bounds it is the epilogue's VALU work on 8.4 M pixels (512
// maps): 40 us with one exponential, two Newton reciprocals and a series a
// pixel, 53 us with two exponentials, a division and the library's log1p. One
// cell a thread (twice the LDS reads of weights) is 1 us slower.
constexpr int kLastS = 64, kLastBand = 16, kLastBands = kLastS / kLastBand;  // cell rows a workgroup
template <bool TRAIN>
__global__ __launch_bounds__(256) void last_layer_kernel(const uint16_t *src, const uint16_t *Kb,
                                                         const float *bias, const uint8_t *y_map,
                                                         float w_map, float inv_n, uint16_t *gz,
                                                         float *partial, float *map) {
  constexpr int S = kLastS, O = 2 * S, kLd = S + 2;
  __shared__ __attribute__((aligned(16))) uint4 cells[(kLastBand + 2) * kLd];
  __shared__ __attribute__((aligned(16))) float4 wk[4][kConvCi];  // [parity][channel], its four cells
  __shared__ float red[256];
  const int b = blockIdx.x / kLastBands, Y0 = (blockIdx.x % kLastBands) * kLastBand, t = threadIdx.x;
  stage_cells<false>(cells, src + (int64_t)b * kConvCi * S * S, S, Y0, kLastBand);
  if (t < 4 * kConvCi * 4) {
    // cell (i, j) of parity (py, px): rows py - 1 + i, taps dy that read it
    const int j = t & 1, i = (t >> 1) & 1, c = (t >> 2) & 7, px = (t >> 5) & 1, py = t >> 6;
    float sum = 0.0f;
    for (int dy = 0; dy < 3; ++dy)
      for (int dx = 0; dx < 3; ++dx)
        if (((py + dy - 1) >> 1) == py - 1 + i && ((px + dx - 1) >> 1) == px - 1 + j)
          sum += bf16_f32(Kb[c * kConvTaps + 3 * dy + dx]);
    reinterpret_cast<float *>(&wk[2 * py + px][c])[2 * i + j] = sum;
  }
  const float bc = bias[0];
  __syncthreads();
  float acc_loss = 0.0f;
  const bool words = (reinterpret_cast<uintptr_t>(y_map) & 3) == 0;
  for (int q = t; q < kLastBand * S / 2; q += 256) {
    const int r = q / (S / 2), X = q % (S / 2) * 2;
    float z[2][4];  // [cell][parity]
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int p = 0; p < 4; ++p) z[h][p] = 0.0f;
    const uint32_t *cw = reinterpret_cast<const uint32_t *>(&cells[r * kLd + X]);
    // two channels at a time (all eight unrolled, the compiler keeps the 128
    // weights in registers and two waves a SIMD)
#pragma unroll 1
    for (int c = 0; c < kConvCi; c += 2) {
      uint32_t d[12];
#pragma unroll
      for (int k = 0; k < 12; ++k) d[k] = cw[((k / 4) * kLd + k % 4) * 4 + c / 2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        float v[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) v[k] = h ? bf16_hi(d[k]) : bf16_lo(d[k]);
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const float4 k4 = wk[p][c + h];
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const int o = 4 * (p >> 1) + (p & 1) + e;
            z[e][p] = fmaf(k4.x, v[o], z[e][p]);
            z[e][p] = fmaf(k4.y, v[o + 1], z[e][p]);
            z[e][p] = fmaf(k4.z, v[o + 4], z[e][p]);
            z[e][p] = fmaf(k4.w, v[o + 5], z[e][p]);
          }
        }
      }
    }
#pragma unroll
    for (int py = 0; py < 2; ++py) {
      const int64_t o = ((int64_t)b * O + 2 * (Y0 + r) + py) * O + 2 * X;  // a multiple of 4
      uint32_t y = 0;
      if constexpr (TRAIN) {
        if (words) y = *reinterpret_cast<const uint32_t *>(y_map + o);
        else
#pragma unroll
          for (int i = 0; i < 4; ++i) y |= (uint32_t)y_map[o + i] << (8 * i);
      }
      float out[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        // one exponential for the sigmoid and the loss
        const float zi = z[i >> 1][2 * py + (i & 1)] + bc, ex = expf(-fabsf(zi));
        const float rc = recip(1.0f + ex), sg = zi >= 0.0f ? rc : ex * rc;
        out[i] = sg;
        if constexpr (TRAIN) {
          const float yi = (y >> (8 * i)) & 0xFFu ? 1.0f : 0.0f;
          acc_loss += fmaxf(zi, 0.0f) - zi * yi + log1p_unit(ex);
          out[i] = w_map * (sg - yi) * inv_n;
        }
      }
      if constexpr (TRAIN)
        *reinterpret_cast<uint2 *>(gz + o) = make_uint2(pack_bf16(out[0], out[1]), pack_bf16(out[2], out[3]));
      else
#pragma unroll
        for (int i = 0; i < 4; ++i) map[o + i] = out[i];
    }
  }
  if constexpr (TRAIN) {
    const float sum = block_reduce(acc_loss, red);
    if (t == 0) partial[blockIdx.x] = sum;
  }
}

// Data gradient of a layer with 8 output channels: dU[u][v][ci] = sum over taps
// and channels of K[co][ci][dy][dx] g[u-dy+1][v-dx+1][co]; the 2x2 blocks of dU
// are summed (columns across two lanes, rows in the lane) and zeroed where the
// layer's input act is 0 (it is a ReLU's output). PLANAR: act and out are the
// dense layer's planes (out may be act: an element is read by the lane that
// then writes it) and the fp32 gradient goes to out_f too. A workgroup:
// kBand rows of a sample's 2S x 2S grid.
template <int S, bool PLANAR>
__global__ __launch_bounds__(256) void upconv_dgrad_kernel(const uint16_t *g, const uint16_t *Kb,
                                                           const uint16_t *act, uint16_t *out, float *out_f) {
  constexpr int O = 2 * S, kBand = 16, kBands = O / kBand, kLd = O + 2;
  __shared__ __attribute__((aligned(16))) uint4 cells[(kBand + 2) * kLd];
  const int b = blockIdx.x / kBands, u0 = (blockIdx.x % kBands) * kBand;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, px = lane & 15, kq = lane >> 4;
  stage_cells<false>(cells, g + (int64_t)b * kConvCi * O * O, O, u0, kBand);
  bf16x8_t w[3];
  kernel_fragments<false>(Kb, px, kq, w);
  int off[3];
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    const int t = min(4 * s + kq, kConvTaps - 1);
    off[s] = (2 - t / 3) * kLd + 2 - t % 3 + px;
  }
  __syncthreads();
  for (int r = 2 * wave; r < kBand; r += 8)
#pragma unroll
    for (int x0 = 0; x0 < O; x0 += 16) {
      f32x4_t acc[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        acc[h] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
        const int base = (r + h) * kLd + x0;
#pragma unroll
        for (int s = 0; s < 3; ++s) {
          const int at = s < 2 || kq == 0 ? base + off[s] : 0;
          acc[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[s], as_bf16x8(cells[at]), acc[h], 0, 0, 0);
        }
      }
      float sum[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float a[2];
#pragma unroll
        for (int h = 0; h < 2; ++h)  // plus the neighbouring column's (lanes 1 0 3 2 of a quad)
          a[h] = acc[h][v] + __int_as_float(__builtin_amdgcn_update_dpp(
                                 0, __float_as_int(acc[h][v]), 0xB1, 0xF, 0xF, true));
        sum[v] = a[0] + a[1];
      }
      if (kq < 2 && (px & 1) == 0) {
        const int sy = (u0 + r) >> 1, sx = (x0 + px) >> 1;
        if constexpr (PLANAR) {
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int64_t o = (((int64_t)b * kConvCi + 4 * kq + v) * S + sy) * S + sx;
            const float val = (act[o] & 0x7FFFu) ? sum[v] : 0.0f;
            out_f[o] = val;
            out[o] = f2bf(val);
          }
        } else {
          const int64_t o = (((int64_t)b * S + sy) * S + sx) * kConvCi + 4 * kq;
          const uint2 m = *reinterpret_cast<const uint2 *>(act + o);
          *reinterpret_cast<uint2 *>(out + o) =
              make_uint2(pack_bf16((m.x & 0x7FFFu) ? sum[0] : 0.0f, (m.x & 0x7FFF0000u) ? sum[1] : 0.0f),
                         pack_bf16((m.y & 0x7FFFu) ? sum[2] : 0.0f, (m.y & 0x7FFF0000u) ? sum[3] : 0.0f));
        }
      }
    }
}

// Kernel and bias gradients of a layer with 8 output channels: the contraction
// over the (2S)^2 pixels of every (sample, band) this workgroup takes, 32 per
// MFMA step:
//   P[co][k] += sum_p A[co][p] B[p][k],  A[co][p] = g[co][p] (bf16 error),
//   B[p][k] = in[ci][(y+dy-1)/2][(x+dx-1)/2] for k = ci*9 + dy*3 + dx < 72,
//   1 for k = 72 (the bias gradient; columns beyond it are not used);
// the four waves' sums are added in wave order and the workgroup writes its
// partial [16][80] to part; wgrad_finish_kernel adds the partials. Both
// operands run along pixels, so they are staged planar: the errors with a
// 16-byte skew per plane, the inputs with zero borders and a plane of ones.
// A lane's eight pixels of B read five cells of a row, each twice but for the
// ends: three LDS reads and four byte permutations, whose selectors depend on
// the lane's dx only.
template <int S, bool PLANAR_IN>
__global__ __launch_bounds__(256) void upconv_wgrad_kernel(const uint16_t *g_b, const uint16_t *in_b, int B,
                                                           float *part) {
  constexpr int O = 2 * S, kBand = 32, kBands = O / kBand, kRows = kBand / 2 + 2;
  constexpr int kGLd = kBand * O + 8, kRs = S + 8, kPl = kRows * kRs;
  // the waves' sums take the planes' place at the end
  __shared__ __attribute__((aligned(16))) uint16_t planes[kConvCi * kGLd + (kConvCi + 1) * kPl];
  static_assert(sizeof(planes) >= sizeof(float) * 4 * kWgradRows * kWgradCols, "");
  uint16_t *const gpl = planes, *const ipl = planes + kConvCi * kGLd;
  float(*const red)[kWgradRows * kWgradCols] =
      reinterpret_cast<float(*)[kWgradRows * kWgradCols]>(planes);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row = lane & 15, kq = lane >> 4;
  // each lane's B column per n-tile: k = 16 n + row
  int pl[5], dyv[5];
  uint32_t sa[5], sb[5];
#pragma unroll
  for (int n = 0; n < 5; ++n) {
    const int k = 16 * n + row, dx = (k % kConvTaps) % 3;
    pl[n] = (k < kConvK ? k / kConvTaps : kConvCi) * kPl + 4;
    dyv[n] = k < kConvK ? (k % kConvTaps) / 3 : 1;
    sa[n] = dx == 0 ? 0x05040302u : dx == 1 ? 0x05040504u : 0x07060504u;
    sb[n] = dx == 0 ? 0x03020100u : dx == 1 ? 0x03020302u : 0x05040302u;
  }
  f32x4_t acc[5];
#pragma unroll
  for (int n = 0; n < 5; ++n) acc[n] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
  // borders and the plane of ones: written once, the staging leaves them
  for (int i = tid; i < (kConvCi + 1) * kPl; i += 256) ipl[i] = i < kConvCi * kPl ? 0u : 0x3F80u;
  for (int item = blockIdx.x; item < B * kBands; item += gridDim.x) {
    const int b = item / kBands, y0 = (item % kBands) * kBand;
    __syncthreads();
    const uint4 *g = reinterpret_cast<const uint4 *>(g_b + ((int64_t)b * O + y0) * O * kConvCi);
    for (int i = tid; i < kBand * O / 2; i += 256) {
      const uint4 p = g[2 * i], q = g[2 * i + 1];
      const uint32_t pw[4] = {p.x, p.y, p.z, p.w}, qw[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
      for (int c = 0; c < kConvCi; ++c)
        *reinterpret_cast<uint32_t *>(&gpl[c * kGLd + 2 * i]) =
            __builtin_amdgcn_perm(qw[c / 2], pw[c / 2], c & 1 ? 0x07060302u : 0x05040100u);
    }
    const uint16_t *in = in_b + (int64_t)b * kConvCi * S * S;
    for (int i = tid; i < kRows * S; i += 256) {
      const int r = i / S, x = i % S, y = y0 / 2 - 1 + r;
      const uint4 p = (unsigned)y < (unsigned)S ? load_cell<PLANAR_IN>(in, S, y, x) : make_uint4(0u, 0u, 0u, 0u);
      const uint32_t pw[4] = {p.x, p.y, p.z, p.w};
#pragma unroll
      for (int c = 0; c < kConvCi; ++c)
        ipl[c * kPl + r * kRs + 4 + x] = (uint16_t)(c & 1 ? pw[c / 2] >> 16 : pw[c / 2]);
    }
    __syncthreads();
    for (int ch = wave; ch < kBand * O / 32; ch += 4) {
      const int p0 = ch * 32 + 8 * kq;  // this lane's 8 pixels (one row)
      const int y = p0 / O, c0 = (p0 % O) / 2;
      const uint4 a = row < kConvCi ? *reinterpret_cast<const uint4 *>(&gpl[row * kGLd + p0])
                                    : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
      for (int n = 0; n < 5; ++n) {
        // cells c0 - 2 .. c0 + 5 of the row that the lane's dy reads
        const uint16_t *q = &ipl[pl[n] + (((y + dyv[n] - 1) >> 1) + 1) * kRs + c0];
        const uint32_t wm = *reinterpret_cast<const uint32_t *>(q - 2);
        const uint2 wc = *reinterpret_cast<const uint2 *>(q);
        const uint32_t wp = *reinterpret_cast<const uint32_t *>(q + 4);
        const uint4 bv = make_uint4(__builtin_amdgcn_perm(wc.x, wm, sa[n]), __builtin_amdgcn_perm(wc.y, wc.x, sb[n]),
                                    __builtin_amdgcn_perm(wc.y, wc.x, sa[n]), __builtin_amdgcn_perm(wp, wc.y, sb[n]));
        acc[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a), as_bf16x8(bv), acc[n], 0, 0, 0);
      }
    }
  }
  __syncthreads();
  // D layout: lane holds column (16 n + row) and rows (co) 4 kq + v
#pragma unroll
  for (int n = 0; n < 5; ++n)
#pragma unroll
    for (int v = 0; v < 4; ++v) red[wave][(4 * kq + v) * kWgradCols + 16 * n + row] = acc[n][v];
  __syncthreads();
  for (int i = tid; i < kWgradRows * kWgradCols; i += 256)
    part[(int64_t)blockIdx.x * kWgradRows * kWgradCols + i] =
        ((red[0][i] + red[1][i]) + red[2][i]) + red[3][i];
}

// Kernel, bias and data gradients of a layer with one output channel (the
// last decoder layer), on the input's own grid. With nearest 2x upsampling,
// tap (dy, dx) of output pixel (y, x) reads input cell
// ((y + dy - 1) >> 1, (x + dx - 1) >> 1), so
//   dK[c][dy][dx] = sum over input cells (Y, X) of in[c][Y][X] times the
//                   sum of g over output rows {2Y+1-dy, 2Y+2-dy} and
//                   columns {2X+1-dx, 2X+2-dx} (pixels outside the output
//                   contribute nothing),
// a quarter of the multiply-adds of the per-pixel form and no im2col; the
// bias gradient is the sum of g over the 2x2 blocks {2Y, 2Y+1} x
// {2X, 2X+1}. With one output channel an MFMA tile would use one of its 16
// rows, so this runs on VALU. Thread item: one sample's input cells
// (Y, 2j) and (Y, 2j + 1); their error windows, rows 2Y-1 .. 2Y+2 and
// columns 4j-1 .. 4j+4, are three 8-byte loads per row, their inputs two
// 16-byte loads. Items are spread over the grid; each thread keeps 73 sums, reduced over the wave (a fixed shuffle tree) and then over
// the four waves in order, so the result does not depend on timing.
// Partials [gridDim.x][16][80] (row 0) as the MFMA form. S even, S <= 64.
// The same box sums also give the layer's data gradient: the
// error of input cell (Y, X), summed over its 2x2 upsampling block, is
// sum over taps of K[c][dy][dx] times box (dy, dx); it is zeroed where the
// layer's input (a ReLU's output) is 0 and written to din_b.
__global__ __launch_bounds__(256) void upconv_grads_co1_kernel(const uint16_t *__restrict__ g_b,
                                                               const uint16_t *__restrict__ in_b,
                                                               int B, int S, float *__restrict__ part,
                                                               const uint16_t *__restrict__ Kb,
                                                               uint16_t *__restrict__ din_b) {
  __shared__ float red[4][kConvK + 1];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int O = 2 * S, half = S / 2;
  float acc[kConvK + 1];
#pragma unroll
  for (int k = 0; k <= kConvK; ++k) acc[k] = 0.0f;
  float kw[kConvK];
#pragma unroll
  for (int k = 0; k < kConvK; ++k)  // (uniform: scalar registers)
    kw[k] = __uint_as_float(__builtin_amdgcn_readfirstlane((uint32_t)Kb[k] << 16));
  const int64_t items = (int64_t)B * S * half;
  for (int64_t it = (int64_t)blockIdx.x * blockDim.x + t; it < items;
       it += (int64_t)gridDim.x * blockDim.x) {
    const int b = (int)(it / (S * half)), pr = (int)(it % (S * half));
    const int Y = pr / half, j = pr % half;
    const uint16_t *gp = g_b + (int64_t)b * O * O;
    // w[i][m]: error at row 2Y - 1 + i, column 4j - 1 + m (0 outside)
    float w[4][6];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int y = 2 * Y - 1 + i;
      uint2 q0 = make_uint2(0u, 0u), q1 = make_uint2(0u, 0u), q2 = make_uint2(0u, 0u);
      if ((unsigned)y < (unsigned)O) {
        const uint2 *row = reinterpret_cast<const uint2 *>(gp + (int64_t)y * O);
        if (j > 0) q0 = row[j - 1];
        q1 = row[j];
        if (j + 1 < half) q2 = row[j + 1];
      }
      w[i][0] = __uint_as_float(q0.y & 0xFFFF0000u);
      w[i][1] = __uint_as_float(q1.x << 16);
      w[i][2] = __uint_as_float(q1.x & 0xFFFF0000u);
      w[i][3] = __uint_as_float(q1.y << 16);
      w[i][4] = __uint_as_float(q1.y & 0xFFFF0000u);
      w[i][5] = __uint_as_float(q2.x << 16);
    }
    const uint4 *ip = reinterpret_cast<const uint4 *>(in_b) + ((int64_t)b * S + Y) * S + 2 * j;
    const uint4 p0 = ip[0], p1 = ip[1];
    const uint32_t w0[4] = {p0.x, p0.y, p0.z, p0.w}, w1[4] = {p1.x, p1.y, p1.z, p1.w};
    float v0[kConvCi], v1[kConvCi];
#pragma unroll
    for (int c = 0; c < kConvCi; ++c) {
      v0[c] = c & 1 ? bf16_hi(w0[c / 2]) : bf16_lo(w0[c / 2]);
      v1[c] = c & 1 ? bf16_hi(w1[c / 2]) : bf16_lo(w1[c / 2]);
    }
    float dsum[2][kConvCi];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      // cell (Y, 2j + h): window columns 2h .. 2h + 3 of w
      float cp[4][3];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) cp[i][dx] = w[i][2 * h + 2 - dx] + w[i][2 * h + 3 - dx];
      float box[kConvTaps];
#pragma unroll
      for (int dy = 0; dy < 3; ++dy)
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) box[3 * dy + dx] = cp[2 - dy][dx] + cp[3 - dy][dx];
#pragma unroll
      for (int c = 0; c < kConvCi; ++c) {
        const float v = h ? v1[c] : v0[c];
        float d = 0.0f;
#pragma unroll
        for (int tap = 0; tap < kConvTaps; ++tap) {
          acc[c * kConvTaps + tap] = fmaf(box[tap], v, acc[c * kConvTaps + tap]);
          d = fmaf(kw[c * kConvTaps + tap], box[tap], d);
        }
        dsum[h][c] = d;
      }
      acc[kConvK] += (w[1][2 * h + 1] + w[1][2 * h + 2]) + (w[2][2 * h + 1] + w[2][2 * h + 2]);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float d[kConvCi];
#pragma unroll
      for (int c = 0; c < kConvCi; ++c) d[c] = (h ? v1[c] : v0[c]) > 0.0f ? dsum[h][c] : 0.0f;
      reinterpret_cast<uint4 *>(din_b)[((int64_t)b * S + Y) * S + 2 * j + h] = make_uint4(
          pack_bf16(d[0], d[1]), pack_bf16(d[2], d[3]), pack_bf16(d[4], d[5]), pack_bf16(d[6], d[7]));
    }
  }
#pragma unroll
  for (int k = 0; k <= kConvK; ++k) {
    float v = acc[k];
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) v += __shfl_xor(v, off);
    acc[k] = v;
  }
  if (lane == 0)
#pragma unroll
    for (int k = 0; k <= kConvK; ++k) red[wave][k] = acc[k];
  __syncthreads();
  float *out = part + (int64_t)blockIdx.x * kWgradRows * kWgradCols;
  for (int i = t; i < kWgradRows * kWgradCols; i += blockDim.x) {
    const int r = i / kWgradCols, k = i % kWgradCols;
    out[i] = (r == 0 && k <= kConvK) ? ((red[0][k] + red[1][k]) + red[2][k]) + red[3][k] : 0.0f;
  }
}

// dK[co][ci][dy][dx] and dkb[co] from the partials of `parts` workgroups:
// one workgroup per output; thread t adds partials t, t + 256, ... in
// order, then a pairwise tree over the 256 threads.
__global__ __launch_bounds__(256) void wgrad_finish_kernel(const float *part, int parts, int Co,
                                                           float *dK, float *dkb) {
  __shared__ float red[256];
  const int o = blockIdx.x;  // co * 73 + k
  const int co = o / (kConvK + 1), k = o % (kConvK + 1);
  float s = 0.0f;
  for (int p = threadIdx.x; p < parts; p += 256)
    s += part[(int64_t)p * kWgradRows * kWgradCols + co * kWgradCols + k];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    if (k < kConvK) dK[co * kConvK + k] = red[0];
    else dkb[co] = red[0];
  }
}

// ---------------------------------------------------------------------------
// Adam (bias-corrected), fp32 master weights; wb receives the bf16 copy of
// the updated weights the matrix products read, wt the MLP's transposed one
__global__ void adam_kernel(float *w, uint16_t *wb, uint16_t *wt, MlpOffsets off, float *m, float *v,
                            const float *g, int64_t n, float lr, float b1, float b2, float eps, float c1, float c2) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float wi = w[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    w[i] = wi;
    const uint16_t q = f2bf(wi);
    wb[i] = q;
    const int64_t t = wt_index(off, i);
    if (t >= 0) wt[t] = q;
  }
}

// Philox4x32-10 word 0 as the uniform source of the initial weights
__device__ uint32_t philox_word0(uint32_t c0, uint32_t c1, uint32_t k0, uint32_t k1) {
  uint32_t c2 = 0, c3 = 0;
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p2 = (uint64_t)0xCD9E8D57u * c2;
    const uint32_t n0 = (uint32_t)(p2 >> 32) ^ c1 ^ k0, n2 = (uint32_t)(p0 >> 32) ^ c3 ^ k1;
    c1 = (uint32_t)p2;
    c3 = (uint32_t)p0;
    c0 = n0;
    c2 = n2;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return c0;
}

__global__ void init_uniform_kernel(float *w, int64_t n, float limit, uint32_t tensor,
                                    uint32_t k0, uint32_t k1, int rows_used, int cols) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const uint32_t u = philox_word0((uint32_t)i, tensor, k0, k1);
    const float v = (2.0f * ((float)(u >> 8) * (1.0f / 16777216.0f)) - 1.0f) * limit;
    w[i] = (rows_used > 0 && (int)(i / cols) >= rows_used) ? 0.0f : v;
  }
}

__global__ void fill_f32_kernel(float *p, float v, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// maps: packed burn maps -> coarse uint8 occupancy grid
__global__ void pool_maps_kernel(const uint32_t *maps, int n, int W, int H, int64_t map_words,
                                 int ow, int oh, uint8_t *out) {
  const int64_t total = (int64_t)n * ow * oh;
  const int stride = (W + 31) / 32;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int X = (int)(i % ow), Y = (int)((i / ow) % oh), k = (int)(i / ((int64_t)ow * oh));
    const int x0 = (int)((int64_t)X * W / ow), x1 = (int)((int64_t)(X + 1) * W / ow);
    const int y0 = (int)((int64_t)Y * H / oh), y1 = (int)((int64_t)(Y + 1) * H / oh);
    const uint32_t *m = maps + (int64_t)k * map_words;
    uint8_t any = 0;
    for (int y = y0; y < y1 && !any; ++y)
      for (int x = x0; x < x1; ++x)
        if ((m[(int64_t)y * stride + (x >> 5)] >> (x & 31)) & 1u) { any = 1; break; }
    out[i] = any;
  }
}

// rank of each non-elite candidate by (score, index); one workgroup
__global__ __launch_bounds__(1024) void select_kernel(const double *cand, const float *score,
                                                      int n, int G, int keep, int k, double *out,
                                                      int32_t *out_idx) {
  // the scores are staged in LDS (n <= 4096): every thread reads all of
  // them, the same one at a time (a broadcast)
  __shared__ float sc[4096];
  for (int i = threadIdx.x; i < n; i += 1024) sc[i] = score[i];
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += 1024) {
    int slot;
    if (i < keep) {
      slot = i;
    } else {
      const float si = sc[i];
      const bool fi = isfinite(si);
      int rank = 0;
      for (int j = keep; j < n; ++j) {
        const float sj = sc[j];
        const bool fj = isfinite(sj);
        const bool before = (fj && !fi) || (fj == fi && ((fi && sj < si) || ((!fi || sj == si) && j < i)));
        rank += before ? 1 : 0;
      }
      slot = keep + rank;
    }
    if (slot < k) {
      for (int c = 0; c < G; ++c) out[(int64_t)slot * G + c] = cand[(int64_t)i * G + c];
      if (out_idx) out_idx[slot] = i;
    }
  }
}

// ---------------------------------------------------------------------------
// Training rows from simulation results: row i takes parameter row
// i / reps (binary64 -> fp32, round to nearest), the ignition (a row of
// `ign` or the constant pair) and the target log(1 + delta) of result i's
// Eq. 2 fitness (binary64 log1p, then rounded to fp32); delta itself is
// copied to out_fit. Any output may be NULL.
__global__ void rows_from_results_kernel(const double *params, int reps, const float *ign,
                                         float ign_x, float ign_y, const fire_result *res, int n,
                                         float *out_x, float *out_y, double *out_fit) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const double delta = res[i].fitness;
    if (out_fit) out_fit[i] = delta;
    if (out_y) out_y[i] = (float)log1p(delta);
    if (out_x) {
      const double *b = params + 5 * (int64_t)(i / reps);
      float *x = out_x + 7 * (int64_t)i;
      for (int k = 0; k < 5; ++k) x[k] = (float)b[k];
      x[5] = ign ? ign[2 * (int64_t)i] : ign_x;
      x[6] = ign ? ign[2 * (int64_t)i + 1] : ign_y;
    }
  }
}

// dst row k = src row rows[k]; rows of `words` 32-bit words, copied with
// 16-byte moves when `vec` (rows and both bases 16-byte aligned).
__global__ void gather_rows_kernel(const uint32_t *src, int64_t words, const int64_t *rows, int n,
                                   uint32_t *dst, int vec) {
  const int64_t per = vec ? words / 4 : words;
  const int64_t total = (int64_t)n * per;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t k = t / per, w = t % per;
    const int64_t r = rows[k];
    if (vec) {
      reinterpret_cast<uint4 *>(dst + k * words)[w] =
          reinterpret_cast<const uint4 *>(src + r * words)[w];
    } else {
      dst[k * words + w] = src[r * words + w];
    }
  }
}

// Screening candidates from `n_sets` offspring sets [n_sets][P][5]: all of
// set 0, then rows E..P-1 of every later set (its first E rows are the
// elites again); binary64 rows to cand, fp32 network inputs (parameters,
// then the constant ignition) to x.
__global__ void candidates_kernel(const double *sets, int n_sets, int P, int E, float ign_x,
                                  float ign_y, double *cand, float *x) {
  const int n = P + (n_sets - 1) * (P - E);
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    int src = i;
    if (i >= P) {
      const int o = 1 + (i - P) / (P - E), j = E + (i - P) % (P - E);
      src = o * P + j;
    }
    for (int k = 0; k < 5; ++k) {
      const double v = sets[5 * (int64_t)src + k];
      cand[5 * (int64_t)i + k] = v;
      x[7 * (int64_t)i + k] = (float)v;
    }
    x[7 * (int64_t)i + 5] = ign_x;
    x[7 * (int64_t)i + 6] = ign_y;
  }
}

}  // namespace
}  // namespace firenn

using namespace firenn;

// ---------------------------------------------------------------------------
// Handle

namespace {
constexpr int kH = 256, kIn = 16, kD0C = 8, kD0S = 16, kDec = kD0C * kD0S * kD0S;
constexpr int kP = FIRE_NN_MAP * FIRE_NN_MAP;
constexpr int64_t kWtWd = kIn * kH + 2 * kH * kH + kH;  // Wd in fire_nn::wt

struct Seg {
  int64_t off, n;
  int rows, cols;
};

struct Layout {
  Seg W1, c1, W2, c2, W3, c3, Wf, cf, Wd, cd, K1, k1, K2, k2, K3, k3;
  int64_t total;
  Layout() {
    int64_t o = 0;
    auto add = [&](int rows, int cols) { Seg s{o, (int64_t)rows * cols, rows, cols}; o += s.n; return s; };
    W1 = add(kIn, kH); c1 = add(1, kH);
    W2 = add(kH, kH); c2 = add(1, kH);
    W3 = add(kH, kH); c3 = add(1, kH);
    Wf = add(kH, 1); cf = add(1, 1);
    Wd = add(kH, kDec); cd = add(1, kDec);
    K1 = add(kD0C * kD0C, 9); k1 = add(1, kD0C);
    K2 = add(kD0C * kD0C, 9); k2 = add(1, kD0C);
    K3 = add(1 * kD0C, 9); k3 = add(1, 1);
    total = o;
  }
};
}  // namespace

struct fire_nn {
  int device = 0;
  fire_nn_cfg cfg{};
  std::string err;
  Layout L;
  float *w = nullptr, *m = nullptr, *v = nullptr, *g = nullptr;  // [total]
  uint16_t *wb = nullptr;  // bf16 copy [total], of which W2, W3 and the kernels are read
  uint16_t *wt = nullptr;  // bf16 W1, W2, W3 transposed ([out][in]), Wf, Wd
  // activations (max_batch rows)
  uint16_t *xb = nullptr, *h1b = nullptr, *h2b = nullptr, *h3b = nullptr, *d0b = nullptr, *dtb = nullptr;
  float *t = nullptr;
  // errors of h3, h2, h1 (gh fp32, ghb bf16) and the parts of dd0 Wd^T (dh)
  float *gt = nullptr, *gd0 = nullptr, *gh = nullptr, *dh = nullptr;
  uint16_t *ghb = nullptr;
  // bf16 copies the decoder's MFMA convolutions read
  uint16_t *d1b = nullptr, *d2b = nullptr, *gzb = nullptr, *gd1b = nullptr, *gd2b = nullptr;
  float *partial = nullptr, *loss = nullptr;
  float *wpart = nullptr;  // kernel-gradient partials [kWgradParts][16][80]
  std::vector<void *> allocs;
};

namespace {
fire_status nn_fail(fire_nn *nn, fire_status s, const char *fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  if (nn) nn->err = buf;
  return s;
}
#define NN_HIP(nn, expr)                                                            \
  do {                                                                              \
    hipError_t e_ = (expr);                                                         \
    if (e_ != hipSuccess)                                                           \
      return nn_fail((nn), e_ == hipErrorOutOfMemory ? FIRE_E_OOM : FIRE_E_DEVICE, \
                     "%s: %s", #expr, hipGetErrorString(e_));                       \
  } while (0)

template <class T>
hipError_t nn_alloc(fire_nn *nn, T **p, int64_t count) {
  hipError_t e = hipMalloc((void **)p, sizeof(T) * (size_t)(count > 0 ? count : 1));
  if (e == hipSuccess) nn->allocs.push_back(*p);
  return e;
}

MlpOffsets mlp_offsets(const Layout &L) {
  return {L.W1.off, L.W2.off, L.W3.off, L.Wf.off, L.Wd.off, L.Wd.n};
}

hipError_t refresh_bf16(fire_nn *nn, hipStream_t s) {
  hipLaunchKernelGGL(refresh_weights_kernel, dim3(blocks_for(nn->L.total)), dim3(256), 0, s, nn->w,
                     nn->wb, nn->wt, mlp_offsets(nn->L), nn->L.total);
  return hipGetLastError();
}

// Forward pass into t [B]; the decoder (dense layer and upsampling
// convolutions) runs only when `want_map` (the fitness head does not depend on
// it), and the activations are kept for it or for the backward pass (`train`).
hipError_t forward(fire_nn *nn, const float *x, int B, hipStream_t s, bool want_map, bool train,
                   float *t) {
  const Layout &L = nn->L;
  hipError_t e;
  const uint16_t *wb = nn->wb, *wt = nn->wt;
  const float *w = nn->w;
  hipLaunchKernelGGL(mlp_forward_kernel, dim3((B + kMlpRows - 1) / kMlpRows), dim3(kMlpThreads), 0, s,
                     x, B, 1.0f / (float)nn->cfg.lattice_w, 1.0f / (float)nn->cfg.lattice_h, wt,
                     wt + kIn * kH, wt + kIn * kH + kH * kH, wt + kIn * kH + 2 * kH * kH,
                     w + L.c1.off, w + L.c2.off, w + L.c3.off, w + L.cf.off,
                     train ? nn->xb : nullptr, train ? nn->h1b : nullptr,
                     train ? nn->h2b : nullptr, train || want_map ? nn->h3b : nullptr, t);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (!want_map) return hipSuccess;
  if ((e = gemm(B, kDec, kH, nn->h3b, kH, 1, wt + kWtWd, kDec, 1, nullptr, kDec, w + L.cd.off,
                1, 0, nn->d0b, s)) != hipSuccess) return e;
  // decoder: d0b (the dense layer's output) -> d1b -> d2b
  hipLaunchKernelGGL((upconv_kernel<16, true>), dim3(B), dim3(256), 0, s, nn->d0b, wb + L.K1.off,
                     w + L.k1.off, nn->d1b);
  hipLaunchKernelGGL((upconv_kernel<32, false>), dim3(2 * B), dim3(256), 0, s, nn->d1b, wb + L.K2.off,
                     w + L.k2.off, nn->d2b);
  return hipGetLastError();
}

// Kernel and bias gradients of one decoder layer: error g_b [B][2S][2S][8] and
// layer input in_b (both bf16).
template <int S, bool PLANAR_IN>
hipError_t conv_weight_grad(fire_nn *nn, const uint16_t *g_b, const uint16_t *in_b, int B, float *dK,
                            float *dkb, hipStream_t s) {
  const int64_t items = (int64_t)B * (2 * S / 32);
  const int parts = (int)(items < kConvGrid ? items : kConvGrid);
  hipLaunchKernelGGL((upconv_wgrad_kernel<S, PLANAR_IN>), dim3(parts), dim3(256), 0, s, g_b, in_b, B,
                     nn->wpart);
  hipLaunchKernelGGL(wgrad_finish_kernel, dim3(kConvCi * (kConvK + 1)), dim3(256), 0, s, nn->wpart,
                     parts, kConvCi, dK, dkb);
  return hipGetLastError();
}

// loss and gradients into nn->g (forward must have run on the same x)
hipError_t backward(fire_nn *nn, const float *y_t, const uint8_t *y_map, int B, hipStream_t s) {
  const Layout &L = nn->L;
  hipError_t e;
  float *g = nn->g;
  const uint16_t *wb = nn->wb;
  hipLaunchKernelGGL(loss_fit_kernel, dim3(1), dim3(256), 0, s, nn->t, y_t, B, nn->gt, nn->dtb,
                     nn->loss);
  const int64_t nz = (int64_t)B * kP;
  const bool use_map = y_map != nullptr && nn->cfg.w_map > 0.0f;
  if (use_map) {
    hipLaunchKernelGGL((last_layer_kernel<true>), dim3(kLastBands * B), dim3(256), 0, s, nn->d2b, wb + L.K3.off,
                       nn->w + L.k3.off, y_map, nn->cfg.w_map, 1.0f / (float)nz, nn->gzb, nn->partial,
                       nullptr);
    hipLaunchKernelGGL(sum_partials_kernel, dim3(1), dim3(256), 0, s, nn->partial,
                       B * kLastBands, 1.0f / (float)nz, nn->loss + 1);
    // decoder backward: each layer's error enters its two MFMA products as
    // bf16; the data gradient comes back summed over the 2x2 upsampling
    // blocks and masked by the layer input's ReLU.
    // Last layer (one output channel): kernel, bias and data gradients from
    // the same 2x2 box sums of the error
    {
      const int64_t blocks = ((int64_t)B * 64 * 32 + 255) / 256;
      const int parts = (int)(blocks < kCo1Grid ? blocks : kCo1Grid);
      hipLaunchKernelGGL(upconv_grads_co1_kernel, dim3(parts), dim3(256), 0, s, nn->gzb, nn->d2b, B, 64,
                         nn->wpart, wb + L.K3.off, nn->gd2b);
      hipLaunchKernelGGL(wgrad_finish_kernel, dim3(kConvK + 1), dim3(256), 0, s, nn->wpart, parts,
                         1, g + L.K3.off, g + L.k3.off);
    }
    if ((e = conv_weight_grad<32, false>(nn, nn->gd2b, nn->d1b, B, g + L.K2.off, g + L.k2.off, s)) != hipSuccess) return e;
    hipLaunchKernelGGL((upconv_dgrad_kernel<32, false>), dim3(4 * B), dim3(256), 0, s, nn->gd2b,
                       wb + L.K2.off, nn->d1b, nn->gd1b, nullptr);
    if ((e = conv_weight_grad<16, true>(nn, nn->gd1b, nn->d0b, B, g + L.K1.off, g + L.k1.off, s)) != hipSuccess) return e;
    // the last data gradient's bf16 copy replaces d0b, which the dense
    // layer's gradient products read next
    hipLaunchKernelGGL((upconv_dgrad_kernel<16, true>), dim3(2 * B), dim3(256), 0, s, nn->gd1b,
                       wb + L.K1.off, nn->d0b, nn->d0b, nn->gd0);
    // the decoder's part of the error of h3: dd0 Wd^T, in kDhParts parts
    GemmArgs q[kDhParts];
    constexpr int kPart = kDec / kDhParts;
    for (int i = 0; i < kDhParts; ++i)
      q[i] = GemmArgs{B, kH, kPart, nn->d0b + i * kPart, kDec, 1, nn->wt + kWtWd + i * kPart, 1, kDec,
                      nn->dh + i * ((int64_t)B * kH), kH, nullptr, 0, 0, nullptr};
    if ((e = gemm_batch<kAlongK, kAlongK>(q, kDhParts, s)) != hipSuccess) return e;
  } else {
    hipLaunchKernelGGL(fill_f32_kernel, dim3(1), dim3(64), 0, s, nn->loss + 1, 0.0f, (int64_t)1);
    const int64_t o = L.Wd.off, n = L.k3.off + L.k3.n - L.Wd.off;
    hipLaunchKernelGGL(fill_f32_kernel, dim3(blocks_for(n)), dim3(256), 0, s, g + o, 0.0f, n);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // the error chain through the hidden layers
  const int64_t bh = (int64_t)B * kH;
  float *g3 = nn->gh, *g2 = g3 + bh, *g1 = g2 + bh;
  uint16_t *gb3 = nn->ghb, *gb2 = gb3 + bh, *gb1 = gb2 + bh;
  hipLaunchKernelGGL(mlp_backward_kernel, dim3((B + kMlpRows - 1) / kMlpRows), dim3(kMlpThreads), 0, s,
                     nn->dtb, use_map ? nn->dh : nullptr, bh, B, nn->wt + kIn * kH + 2 * kH * kH,
                     wb + L.W3.off, wb + L.W2.off, nn->h3b, nn->h2b, nn->h1b, g3, g2, g1, gb3, gb2, gb1);
  // weight gradients (activations^T errors, over the batch) and bias gradients
  // (column sums), each kind in one launch: alone, none of them fills the chip
  const GemmArgs q[kMaxGemms] = {
      {kH, kDec, B, nn->h3b, 1, kH, nn->d0b, kDec, 1, g + L.Wd.off, kDec, nullptr, 0, 0, nullptr},
      {kH, kH, B, nn->h2b, 1, kH, gb3, kH, 1, g + L.W3.off, kH, nullptr, 0, 0, nullptr},
      {kH, kH, B, nn->h1b, 1, kH, gb2, kH, 1, g + L.W2.off, kH, nullptr, 0, 0, nullptr},
      {kIn, kH, B, nn->xb, 1, kIn, gb1, kH, 1, g + L.W1.off, kH, nullptr, 0, 0, nullptr},
      // (one column: read element by element, as the ends of rows are)
      {kH, 1, B, nn->h3b, 1, kH, nn->dtb, 1, 1, g + L.Wf.off, 1, nullptr, 0, 0, nullptr}};
  const int skip = use_map ? 0 : 1;  // without maps the decoder's gradients are zero
  if ((e = gemm_batch<kAlongRows, kAlongRows>(q + skip, kMaxGemms - skip, s)) != hipSuccess) return e;
  const float *const sums[kMaxColsums] = {nn->gd0, g3, g2, g1, nn->gt};
  const int cols[kMaxColsums] = {kDec, kH, kH, kH, 1};
  float *const outs[kMaxColsums] = {g + L.cd.off, g + L.c3.off, g + L.c2.off, g + L.c1.off, g + L.cf.off};
  if ((e = colsums(sums + skip, cols + skip, outs + skip, kMaxColsums - skip, B, s)) != hipSuccess) return e;
  return hipGetLastError();
}
}  // namespace

extern "C" {

fire_status fire_nn_create(int device, const fire_nn_cfg *cfg, uint64_t seed, fire_nn **out) {
  if (!out || !cfg) return FIRE_E_INVALID;
  *out = nullptr;
  if (cfg->max_batch < 1 || cfg->max_batch > (1 << 16) || cfg->lattice_w < 1 || cfg->lattice_h < 1 ||
      !(cfg->w_map >= 0.0f) || !(cfg->adam_b1 >= 0.0f && cfg->adam_b1 < 1.0f) ||
      !(cfg->adam_b2 >= 0.0f && cfg->adam_b2 < 1.0f) || !(cfg->adam_eps > 0.0f))
    return FIRE_E_INVALID;
  fire_nn *nn = new (std::nothrow) fire_nn();
  if (!nn) return FIRE_E_OOM;
  nn->device = device;
  nn->cfg = *cfg;
  const int64_t Bm = cfg->max_batch, T = nn->L.total;
  auto fail_out = [&](hipError_t e) {
    fire_nn_destroy(nn);
    return e == hipErrorOutOfMemory ? FIRE_E_OOM : FIRE_E_DEVICE;
  };
  hipError_t e = hipSetDevice(device);
  if (e == hipSuccess) e = nn_alloc(nn, &nn->w, T);
  if (e == hipSuccess) e = nn_alloc(nn, &nn->m, T);
  if (e == hipSuccess) e = nn_alloc(nn, &nn->v, T);
  if (e == hipSuccess) e = nn_alloc(nn, &nn->g, T);
  if (e == hipSuccess) e = nn_alloc(nn, &nn->wb, T);
  if (e == hipSuccess) e = nn_alloc(nn, &nn->wt, kWtWd + (int64_t)kH * kDec);
  if (e == hipSuccess) e = nn_alloc(nn, &nn->xb, Bm * kIn);
  if (e == hipSuccess) e = nn_alloc(nn, &nn->h1b, Bm * kH);
  if (e == hipSuccess) e = nn_alloc(nn, &nn->h2b, Bm * kH);
  if (e == hipSuccess) e = nn_alloc(nn, &nn->h3b, Bm * kH);
  if (e == hipSuccess) e = nn_alloc(nn, &nn->d0b, Bm * kDec);
  if (e == hipSuccess) e = nn_alloc(nn, &nn->dtb, Bm);
  if (e == hipSuccess) e = nn_alloc(nn, &nn->ghb, 3 * Bm * kH);
  if (e == hipSuccess) e = nn_alloc(nn, &nn->t, Bm);
  if (e == hipSuccess) e = nn_alloc(nn, &nn->gt, Bm);
  if (e == hipSuccess) e = nn_alloc(nn, &nn->gd0, Bm * kDec);
  if (e == hipSuccess) e = nn_alloc(nn, &nn->gh, 3 * Bm * kH);
  if (e == hipSuccess) e = nn_alloc(nn, &nn->dh, kDhParts * Bm * kH);
  if (e == hipSuccess) e = nn_alloc(nn, &nn->partial, Bm * kLastBands);
  if (e == hipSuccess) e = nn_alloc(nn, &nn->wpart, (int64_t)kWgradParts * kWgradRows * kWgradCols);
  if (e == hipSuccess) e = nn_alloc(nn, &nn->d1b, Bm * kD0C * 32 * 32);
  if (e == hipSuccess) e = nn_alloc(nn, &nn->d2b, Bm * kD0C * 64 * 64);
  if (e == hipSuccess) e = nn_alloc(nn, &nn->gzb, Bm * kP);
  if (e == hipSuccess) e = nn_alloc(nn, &nn->gd1b, Bm * kD0C * 32 * 32);
  if (e == hipSuccess) e = nn_alloc(nn, &nn->gd2b, Bm * kD0C * 64 * 64);
  if (e == hipSuccess) e = nn_alloc(nn, &nn->loss, 2);
  if (e != hipSuccess) return fail_out(e);
  // initial parameters
  const Layout &L = nn->L;
  const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
  hipLaunchKernelGGL(fill_f32_kernel, dim3(blocks_for(T)), dim3(256), 0, nullptr, nn->w, 0.0f, T);
  hipLaunchKernelGGL(fill_f32_kernel, dim3(blocks_for(T)), dim3(256), 0, nullptr, nn->m, 0.0f, T);
  hipLaunchKernelGGL(fill_f32_kernel, dim3(blocks_for(T)), dim3(256), 0, nullptr, nn->v, 0.0f, T);
  struct Init { const Seg *s; float fan_in, fan_out; int rows_used; };
  const Init inits[] = {{&L.W1, (float)FIRE_NN_IN, (float)kH, FIRE_NN_IN}, {&L.W2, kH, kH, 0},
                        {&L.W3, kH, kH, 0}, {&L.Wf, kH, 1, 0}, {&L.Wd, kH, kDec, 0},
                        {&L.K1, kD0C * 9.0f, kD0C * 9.0f, 0}, {&L.K2, kD0C * 9.0f, kD0C * 9.0f, 0},
                        {&L.K3, kD0C * 9.0f, 9.0f, 0}};
  uint32_t tensor = 1;
  for (const Init &in : inits) {
    const float limit = sqrtf(6.0f / (in.fan_in + in.fan_out));
    hipLaunchKernelGGL(init_uniform_kernel, dim3(blocks_for(in.s->n)), dim3(256), 0, nullptr,
                       nn->w + in.s->off, in.s->n, limit, tensor++, k0, k1, in.rows_used, in.s->cols);
  }
  e = refresh_bf16(nn, nullptr);
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (e != hipSuccess) return fail_out(e);
  *out = nn;
  return FIRE_OK;
}

void fire_nn_destroy(fire_nn *nn) {
  if (!nn) return;
  (void)hipSetDevice(nn->device);
  (void)hipDeviceSynchronize();
  for (void *p : nn->allocs) (void)hipFree(p);
  delete nn;
}

const char *fire_nn_last_error(const fire_nn *nn) { return nn ? nn->err.c_str() : "null handle"; }

int64_t fire_nn_num_params(const fire_nn *nn) { return nn ? nn->L.total : 0; }

fire_status fire_nn_get_params(fire_nn *nn, float *out, void *stream) {
  if (!nn) return FIRE_E_INVALID;
  if (!out) return nn_fail(nn, FIRE_E_INVALID, "null output");
  NN_HIP(nn, hipSetDevice(nn->device));
  NN_HIP(nn, hipMemcpyAsync(out, nn->w, sizeof(float) * nn->L.total, hipMemcpyDeviceToDevice,
                            (hipStream_t)stream));
  return FIRE_OK;
}

fire_status fire_nn_set_params(fire_nn *nn, const float *in, void *stream) {
  if (!nn) return FIRE_E_INVALID;
  if (!in) return nn_fail(nn, FIRE_E_INVALID, "null input");
  NN_HIP(nn, hipSetDevice(nn->device));
  NN_HIP(nn, hipMemcpyAsync(nn->w, in, sizeof(float) * nn->L.total, hipMemcpyDeviceToDevice,
                            (hipStream_t)stream));
  NN_HIP(nn, refresh_bf16(nn, (hipStream_t)stream));
  return FIRE_OK;
}

fire_status fire_nn_forward(fire_nn *nn, const float *x, int32_t B, float *out_t, float *out_map,
                            void *stream) {
  if (!nn) return FIRE_E_INVALID;
  if (!x || !out_t || B < 1 || B > nn->cfg.max_batch)
    return nn_fail(nn, FIRE_E_INVALID, "bad batch (1..%d) or null pointer", nn->cfg.max_batch);
  NN_HIP(nn, hipSetDevice(nn->device));
  hipStream_t s = (hipStream_t)stream;
  // The launch reads some rows of x after it has written other rows' scores:
  // scores that share memory with x go through the handle's own buffer.
  const uintptr_t xa = (uintptr_t)x, ta = (uintptr_t)out_t;
  const bool shared = ta < xa + sizeof(float) * FIRE_NN_IN * (size_t)B && xa < ta + sizeof(float) * (size_t)B;
  NN_HIP(nn, forward(nn, x, B, s, out_map != nullptr, false, shared ? nn->t : out_t));
  if (shared)
    NN_HIP(nn, hipMemcpyAsync(out_t, nn->t, sizeof(float) * (size_t)B, hipMemcpyDeviceToDevice, s));
  if (out_map) {
    hipLaunchKernelGGL((last_layer_kernel<false>), dim3(kLastBands * B), dim3(256), 0, s,
                       nn->d2b, nn->wb + nn->L.K3.off, nn->w + nn->L.k3.off, nullptr, 0.0f, 0.0f,
                       nullptr, nullptr, out_map);
    NN_HIP(nn, hipGetLastError());
  }
  return FIRE_OK;
}

fire_status fire_nn_gradients(fire_nn *nn, const float *x, const float *y_t, const uint8_t *y_map,
                              int32_t B, float *out_loss, float *out_grads, void *stream) {
  if (!nn) return FIRE_E_INVALID;
  if (!x || !y_t || !out_loss || B < 1 || B > nn->cfg.max_batch)
    return nn_fail(nn, FIRE_E_INVALID, "bad batch (1..%d) or null pointer", nn->cfg.max_batch);
  NN_HIP(nn, hipSetDevice(nn->device));
  hipStream_t s = (hipStream_t)stream;
  NN_HIP(nn, forward(nn, x, B, s, y_map != nullptr && nn->cfg.w_map > 0.0f, true, nn->t));
  NN_HIP(nn, backward(nn, y_t, y_map, B, s));
  NN_HIP(nn, hipMemcpyAsync(out_loss, nn->loss, 2 * sizeof(float), hipMemcpyDeviceToDevice, s));
  if (out_grads)
    NN_HIP(nn, hipMemcpyAsync(out_grads, nn->g, sizeof(float) * nn->L.total,
                              hipMemcpyDeviceToDevice, s));
  return FIRE_OK;
}

fire_status fire_nn_train_step(fire_nn *nn, const float *x, const float *y_t, const uint8_t *y_map,
                               int32_t B, float lr, int32_t step, float *out_loss, void *stream) {
  if (!nn) return FIRE_E_INVALID;
  if (!x || !y_t || B < 1 || B > nn->cfg.max_batch || step < 1 || !(lr > 0.0f))
    return nn_fail(nn, FIRE_E_INVALID, "bad batch, step or learning rate");
  NN_HIP(nn, hipSetDevice(nn->device));
  hipStream_t s = (hipStream_t)stream;
  NN_HIP(nn, forward(nn, x, B, s, y_map != nullptr && nn->cfg.w_map > 0.0f, true, nn->t));
  NN_HIP(nn, backward(nn, y_t, y_map, B, s));
  const float c1 = 1.0f - powf(nn->cfg.adam_b1, (float)step);
  const float c2 = 1.0f - powf(nn->cfg.adam_b2, (float)step);
  hipLaunchKernelGGL(adam_kernel, dim3(blocks_for(nn->L.total)), dim3(256), 0, s, nn->w, nn->wb,
                     nn->wt, mlp_offsets(nn->L), nn->m, nn->v, nn->g, nn->L.total, lr, nn->cfg.adam_b1, nn->cfg.adam_b2,
                     nn->cfg.adam_eps, c1, c2);
  NN_HIP(nn, hipGetLastError());
  if (out_loss)
    NN_HIP(nn, hipMemcpyAsync(out_loss, nn->loss, 2 * sizeof(float), hipMemcpyDeviceToDevice, s));
  return FIRE_OK;
}

fire_status fire_gemm_bf16(int M, int N, int K, const uint16_t *A, int64_t sam, int64_t sak,
                           const uint16_t *Bm, int64_t sbk, int64_t sbn, float *C, int64_t ldc,
                           const float *bias, int relu, int accumulate, uint16_t *Cb,
                           void *stream) {
  if (M < 1 || N < 1 || K < 1 || !A || !Bm || !C || ldc < N) return FIRE_E_INVALID;
  if (gemm(M, N, K, A, sam, sak, Bm, sbk, sbn, C, ldc, bias, relu, accumulate, Cb,
           (hipStream_t)stream) != hipSuccess)
    return FIRE_E_DEVICE;
  return FIRE_OK;
}

fire_status fire_pool_maps(const uint32_t *maps, int32_t n, int32_t W, int32_t H,
                           int64_t map_words, int32_t out_w, int32_t out_h, uint8_t *out,
                           void *stream) {
  if (!maps || !out || n < 0 || W < 1 || H < 1 || out_w < 1 || out_h < 1 || out_w > W ||
      out_h > H || map_words < (int64_t)H * ((W + 31) / 32))
    return FIRE_E_INVALID;
  if (n == 0) return FIRE_OK;
  const int64_t total = (int64_t)n * out_w * out_h;
  hipLaunchKernelGGL(pool_maps_kernel, dim3(blocks_for(total)), dim3(256), 0, (hipStream_t)stream,
                     maps, n, W, H, map_words, out_w, out_h, out);
  return hipGetLastError() == hipSuccess ? FIRE_OK : FIRE_E_DEVICE;
}

fire_status fire_colsum_f32(const float *d, int32_t M, int32_t N, float *out, void *stream) {
  if (!d || !out || M < 1 || N < 1) return FIRE_E_INVALID;
  return colsums(&d, &N, &out, 1, M, (hipStream_t)stream) == hipSuccess ? FIRE_OK : FIRE_E_DEVICE;
}

fire_status fire_nn_select(const double *cand, const float *score, int32_t n, int32_t G,
                           int32_t keep, int32_t k, double *out, int32_t *out_idx, void *stream) {
  if (!cand || !score || !out || n < 1 || n > 4096 || G < 1 || k < 1 || k > n || keep < 0 ||
      keep > k)
    return FIRE_E_INVALID;
  hipLaunchKernelGGL(select_kernel, dim3(1), dim3(1024), 0, (hipStream_t)stream, cand, score, n,
                     G, keep, k, out, out_idx);
  return hipGetLastError() == hipSuccess ? FIRE_OK : FIRE_E_DEVICE;
}

fire_status fire_nn_rows_from_results(const double *params, int32_t reps, const float *ign,
                                      float ign_x, float ign_y, const fire_result *results,
                                      int32_t n, float *out_x, float *out_y, double *out_fit,
                                      void *stream) {
  if (n < 0 || !results || reps < 1 || (out_x && !params)) return FIRE_E_INVALID;
  if (n == 0) return FIRE_OK;
  hipLaunchKernelGGL(rows_from_results_kernel, dim3(blocks_for(n)), dim3(256), 0,
                     (hipStream_t)stream, params, reps, ign, ign_x, ign_y, results, n, out_x,
                     out_y, out_fit);
  return hipGetLastError() == hipSuccess ? FIRE_OK : FIRE_E_DEVICE;
}

fire_status fire_gather_rows(const void *src, int64_t row_bytes, const int64_t *rows, int32_t n,
                             void *dst, void *stream) {
  if (n < 0 || row_bytes < 4 || row_bytes % 4 != 0 || (n > 0 && (!src || !rows || !dst)))
    return FIRE_E_INVALID;
  if (n == 0) return FIRE_OK;
  const int vec = row_bytes % 16 == 0 && (uintptr_t)src % 16 == 0 && (uintptr_t)dst % 16 == 0;
  const int64_t words = row_bytes / 4;
  hipLaunchKernelGGL(gather_rows_kernel,
                     dim3(blocks_for((int64_t)n * (vec ? words / 4 : words))), dim3(256), 0,
                     (hipStream_t)stream, (const uint32_t *)src, words, rows, n, (uint32_t *)dst,
                     vec);
  return hipGetLastError() == hipSuccess ? FIRE_OK : FIRE_E_DEVICE;
}

fire_status fire_nn_candidates(const double *sets, int32_t n_sets, int32_t P, int32_t E,
                               float ign_x, float ign_y, double *cand, float *x, void *stream) {
  if (!sets || !cand || !x || n_sets < 1 || P < 1 || E < 0 || E >= P) return FIRE_E_INVALID;
  const int n = P + (n_sets - 1) * (P - E);
  hipLaunchKernelGGL(candidates_kernel, dim3(blocks_for(n)), dim3(256), 0,
                     (hipStream_t)stream, sets, n_sets, P, E, ign_x, ign_y, cand, x);
  return hipGetLastError() == hipSuccess ? FIRE_OK : FIRE_E_DEVICE;
}

}  // extern "C"
