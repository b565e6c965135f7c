// Kernels of the learned variance surrogate: a 4 -> 256 -> 256 -> 256 -> 1 MLP with SiLU hidden
// units, trained in FP32 (forward, backward, Adam) and evaluated in FP32 or BF16 (MFMA).
//
// Parameter vector (row-major, 133,121 floats): W1 [256][4], b1, W2 [256][256], b2, W3 [256][256],
// b3, w4 [1][256], b4; followed in the state buffer by the normalisation mu_x[4], s_x[4], mu_t, s_t.
// Layer l: z = h W^T + b, h' = silu(z) = z / (1 + e^-z).  Loss: mean (y' - t')^2 over the batch.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "bs_mlp_k.h"

namespace {

__device__ __forceinline__ float silu(float z) { return z / (1.0f + expf(-z)); }
__device__ __forceinline__ float dsilu(float z) {
  const float s = 1.0f / (1.0f + expf(-z));
  return s * (1.0f + z * (1.0f - s));
}

// ---------------------------------------------------------------- FP32 network on FP32 MFMA
// Everything of a row but the weight gradients stays inside the row: forward, loss and the chain of
// dZ are row-local, so one kernel takes 16 rows through all of it in LDS, and only what the weight
// gradients contract over rows (H1, H2, dZ2, dZ3) is written out.  Bound: the weights' trip from L2
// (0.5 MB forward, 1 MB with the backward pass, per 16 rows) and the latency of the layer chain.
// 8 waves of 32 columns (two 16 x 16 tiles of mfma_f32_16x16x4_f32, K = 256): a layer's 128 weight
// registers per lane are loaded before the previous layer's barrier.  Loss and gradient
// of 3122 rows and 483 predictions: 2.96 ms in about 30 launches (2.3 ms of it column sums by one
// block) before, 0.14 ms in four now (rows 46 us, weight gradients 15, reduction 6, prediction 25).
typedef float f32x4m __attribute__((ext_vector_type(4)));
constexpr int MR_LD = MLP_HID + 4;   // LDS row stride: 16 rows of one 16-byte chunk hit distinct banks

// acc[t] += A (16 rows in LDS, K = 256) x the two column tiles held in wb; lane (c = lane & 15, g =
// lane >> 4) supplies row c and column c at k = 16 s + 4 g + e in MFMA step (s, e).
__device__ __forceinline__ void mr_mm(const float* __restrict__ A, const float4 (&wb)[2][16], int c, int g, f32x4m (&acc)[2]) {
#pragma unroll
  for (int s = 0; s < 16; ++s) {
    const float4 av = *(const float4*)&A[c * MR_LD + 16 * s + 4 * g];
#pragma unroll
    for (int t = 0; t < 2; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.x, wb[t][s].x, acc[t], 0, 0, 0);
#pragma unroll
    for (int t = 0; t < 2; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.y, wb[t][s].y, acc[t], 0, 0, 0);
#pragma unroll
    for (int t = 0; t < 2; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.z, wb[t][s].z, acc[t], 0, 0, 0);
#pragma unroll
    for (int t = 0; t < 2; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.w, wb[t][s].w, acc[t], 0, 0, 0);
  }
}
// The weights are read with buffer loads: one lane offset and scalar offsets for all 128 registers
// (as 64-bit addresses they are loop-invariant, and keeping them spilled 280 registers a lane).
// B of h W^T: columns col0 + 16 t + c, four consecutive k per load; W at float offset `off` of p.
typedef unsigned u32x4m __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void mr_load_fwd(__amdgpu_buffer_rsrc_t p, int off, int col0, int c, int g, float4 (&wb)[2][16]) {
  const int v = 4 * ((col0 + c) * MLP_HID + 4 * g);
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int s = 0; s < 16; ++s) {
      const u32x4m x = __builtin_amdgcn_raw_buffer_load_b128(p, v, 4 * (off + 16 * t * MLP_HID) + 64 * s, 0);
      wb[t][s] = __builtin_bit_cast(float4, x);
    }
}
// B of dZ W: columns col0 + 2 c + t (one 8-byte load serves both tiles at one k)
__device__ __forceinline__ void mr_load_bwd(__amdgpu_buffer_rsrc_t p, int off, int col0, int c, int g, float4 (&wb)[2][16]) {
  const int v = 4 * (4 * g * MLP_HID + col0 + 2 * c);
#pragma unroll
  for (int s = 0; s < 16; ++s) {
    float2 x[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      x[e] = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(p, v, 4 * (off + (16 * s + e) * MLP_HID), 0));
    wb[0][s] = make_float4(x[0].x, x[1].x, x[2].x, x[3].x);
    wb[1][s] = make_float4(x[0].y, x[1].y, x[2].y, x[3].y);
  }
}

// TRAIN: loss, row-local gradients and their column sums over the block's rows.  Otherwise the
// de-normalised prediction from raw inputs.
template <bool TRAIN>
__global__ __launch_bounds__(512) void k_mlp_rows(MlpRowArgs a) {
  extern __shared__ __attribute__((aligned(16))) float mr_sh[];
  float* HA = mr_sh;
  float* HB = HA + MR_ROWS * MR_LD;
  float* D1 = HB + MR_ROWS * MR_LD;      // TRAIN only: silu'(z) of the three layers
  float* D2 = D1 + MR_ROWS * MR_LD;
  float* D3 = D2 + MR_ROWS * MR_LD;
  __shared__ float Xs[MR_ROWS][4], ys[MR_ROWS], dys[MR_ROWS];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, c = lane & 15, g = lane >> 4;
  const int col0 = 32 * w, tc = tid & 255, half = tid >> 8;   // MFMA columns; column and row parity of the elementwise steps
  const float* __restrict__ p = a.p;
  const __amdgpu_buffer_rsrc_t pr = __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, MLP_NPARAM * 4, 0x00020000);
  const float4 w1 = *(const float4*)&p[MLP_OFF_W1 + 4 * tc];
  const float b1 = p[MLP_OFF_B1 + tc], w4 = p[MLP_OFF_W4 + tc];
  float s_b1 = 0.f, s_b2 = 0.f, s_b3 = 0.f, s_w4 = 0.f, s_w1[4] = {0.f, 0.f, 0.f, 0.f}, s_dy = 0.f;
  double s_loss = 0.0;
  const int ngroups = (a.n + MR_ROWS - 1) / MR_ROWS;
  for (int grp = blockIdx.x; grp < ngroups; grp += gridDim.x) {
    const int r0 = grp * MR_ROWS;
    float4 wb[2][16];
    mr_load_fwd(pr, MLP_OFF_W2, col0, c, g, wb);
    if (tid < 4 * MR_ROWS) {
      const int r = r0 + (tid >> 2), k = tid & 3;
      float x = r < a.n ? a.X[(size_t)r * 4 + k] : 0.f;
      if (!TRAIN) x = (x - a.norm[k]) / a.norm[4 + k];
      Xs[tid >> 2][k] = x;
    }
    __syncthreads();
    // layer 1
#pragma unroll
    for (int i = 0; i < MR_ROWS / 2; ++i) {
      const int r = half + 2 * i;
      const float z = fmaf(Xs[r][3], w1.w, fmaf(Xs[r][2], w1.z, fmaf(Xs[r][1], w1.y, Xs[r][0] * w1.x))) + b1;
      const float h = silu(z);
      HA[r * MR_LD + tc] = h;
      if (TRAIN) {
        D1[r * MR_LD + tc] = dsilu(z);
        if (r0 + r < a.n) a.H1[(size_t)(r0 + r) * MLP_HID + tc] = h;
      }
    }
    __syncthreads();
    // layers 2 (HA -> HB) and 3 (HB -> HA)
#pragma unroll
    for (int l = 0; l < 2; ++l) {
      f32x4m acc[2] = {};
      mr_mm(l ? HB : HA, wb, c, g, acc);
      __builtin_amdgcn_sched_barrier(0);   // the next layer's weights reuse these registers
      if (l == 0) mr_load_fwd(pr, MLP_OFF_W3, col0, c, g, wb);
      else if (TRAIN) mr_load_bwd(pr, MLP_OFF_W3, col0, c, g, wb);
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int col = col0 + 16 * t + c;
        const float b = p[(l ? MLP_OFF_B3 : MLP_OFF_B2) + col];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int r = 4 * g + i;
          const float z = acc[t][i] + b;
          const float h = silu(z);
          (l ? HA : HB)[r * MR_LD + col] = h;
          if (TRAIN) {
            (l ? D3 : D2)[r * MR_LD + col] = dsilu(z);
            if (l == 0 && r0 + r < a.n) a.H2[(size_t)(r0 + r) * MLP_HID + col] = h;
          }
        }
      }
      __syncthreads();
    }
    // output: wave w sums rows 2 w and 2 w + 1
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = 2 * w + i;
      const float4 h = *(const float4*)&HA[r * MR_LD + 4 * lane], v = *(const float4*)&p[MLP_OFF_W4 + 4 * lane];
      float s = fmaf(h.w, v.w, fmaf(h.z, v.z, fmaf(h.y, v.y, h.x * v.x)));
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
      const float y = s + p[MLP_OFF_B4];
      if (lane == 0) {
        if (TRAIN) {
          const float d = r0 + r < a.n ? y - a.t[r0 + r] : 0.f;
          ys[r] = d;
          dys[r] = 2.0f * d / (float)a.n;
        } else if (r0 + r < a.n) {
          a.y[r0 + r] = a.norm[8] + a.norm[9] * y;
        }
      }
    }
    __syncthreads();
    if constexpr (!TRAIN) continue;
    // dZ3 = dy w4 silu'(z3) into HB; sums of dy H3, dy and the squared residuals
#pragma unroll
    for (int i = 0; i < MR_ROWS / 2; ++i) {
      const int r = half + 2 * i;
      const float dy = dys[r], dz = dy * w4 * D3[r * MR_LD + tc];
      s_w4 = fmaf(dy, HA[r * MR_LD + tc], s_w4);
      s_b3 += dz;
      HB[r * MR_LD + tc] = dz;
      if (r0 + r < a.n) a.dZ3[(size_t)(r0 + r) * MLP_HID + tc] = dz;
    }
    if (tid == 0)
      for (int r = 0; r < MR_ROWS; ++r) {
        s_loss += (double)ys[r] * ys[r];
        s_dy += dys[r];
      }
    __syncthreads();
    // dZ2 = (dZ3 W3) silu'(z2) into HA, dZ1 = (dZ2 W2) silu'(z1) into HB
#pragma unroll
    for (int l = 0; l < 2; ++l) {
      f32x4m acc[2] = {};
      mr_mm(l ? HA : HB, wb, c, g, acc);
      __builtin_amdgcn_sched_barrier(0);
      if (l == 0) mr_load_bwd(pr, MLP_OFF_W2, col0, c, g, wb);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = 4 * g + i, col = col0 + 2 * c;
        const float2 d = *(const float2*)&(l ? D1 : D2)[r * MR_LD + col];
        const float2 dz = make_float2(acc[0][i] * d.x, acc[1][i] * d.y);
        *(float2*)&(l ? HB : HA)[r * MR_LD + col] = dz;
        if (l == 0 && r0 + r < a.n) *(float2*)&a.dZ2[(size_t)(r0 + r) * MLP_HID + col] = dz;
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < MR_ROWS / 2; ++i) {
        const int r = half + 2 * i;
        const float dz = (l ? HB : HA)[r * MR_LD + tc];
        if (l == 0) {
          s_b2 += dz;
        } else {
          s_b1 += dz;
#pragma unroll
          for (int k = 0; k < 4; ++k) s_w1[k] = fmaf(dz, Xs[r][k], s_w1[k]);
        }
      }
    }
    __syncthreads();   // Xs and the LDS rows are free for the next group
  }
  if constexpr (TRAIN) {
    float* q = a.vpart + (size_t)(2 * blockIdx.x + half) * MR_PART;
    *(float4*)&q[4 * tc] = make_float4(s_w1[0], s_w1[1], s_w1[2], s_w1[3]);
    q[1024 + tc] = s_b1;
    q[1280 + tc] = s_b2;
    q[1536 + tc] = s_b3;
    q[1792 + tc] = s_w4;
    if (tid == 0) {
      a.lpart[2 * blockIdx.x] = s_loss;
      a.lpart[2 * blockIdx.x + 1] = (double)s_dy;
    }
  }
}

// Weight gradients dW3 = dZ3^T H2 (blockIdx.y = 1) and dW2 = dZ2^T H1 (0): 64 x 64 block tiles
// (blockIdx.x), rows split over blockIdx.z and, four at a time, over the block's waves, each of
// which forms the whole tile (one 16-byte load of either operand serves four 16-wide tiles, 16 MFMAs
// per load pair); the waves' tiles are added through LDS.
__global__ __launch_bounds__(256) void k_mlp_wgrad(MlpRowArgs a, int chunk) {
  __shared__ __attribute__((aligned(16))) float red[4][64 * 64];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, c = lane & 15, g = lane >> 4;
  const int i0 = (blockIdx.x & 3) * 64, j0 = (blockIdx.x >> 2) * 64;
  const float* __restrict__ Z = (blockIdx.y ? a.dZ3 : a.dZ2) + i0 + 4 * c;
  const float* __restrict__ H = (blockIdx.y ? a.H2 : a.H1) + j0 + 4 * c;
  const int kb = blockIdx.z * chunk, ke = min(a.n, kb + chunk);
  f32x4m acc[4][4] = {};
  constexpr int U = 4;   // steps of 16 rows in flight
  for (int k0 = kb + 4 * w + g; k0 - g < ke; k0 += 16 * U) {
    float4 x[U], y[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = k0 + 16 * u;
      x[u] = y[u] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (r < ke) {
        x[u] = *(const float4*)&Z[(size_t)r * MLP_HID];
        y[u] = *(const float4*)&H[(size_t)r * MLP_HID];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float av[4] = {x[u].x, x[u].y, x[u].z, x[u].w}, bv[4] = {y[u].x, y[u].y, y[u].z, y[u].w};
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i], bv[j], acc[i][j], 0, 0, 0);
    }
  }
  // tile (i, j) element q of the lane: row 4 (4 g + q) + i, column 4 c + j
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      *(float4*)&red[w][(4 * (4 * g + q) + i) * 64 + 4 * c] = make_float4(acc[i][0][q], acc[i][1][q], acc[i][2][q], acc[i][3][q]);
  __syncthreads();
  float* out = a.wpart + ((size_t)blockIdx.z * 2 + blockIdx.y) * MLP_HID * MLP_HID;
  for (int e = tid; e < 64 * 16; e += 256) {
    const int r = e >> 4, q = (e & 15) * 4;
    float4 s = *(const float4*)&red[0][r * 64 + q];
#pragma unroll
    for (int k = 1; k < 4; ++k) {
      const float4 v = *(const float4*)&red[k][r * 64 + q];
      s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
    *(float4*)&out[(size_t)(i0 + r) * MLP_HID + j0 + q] = s;
  }
}

// The gradient from the partials, each in a fixed order: W2 and W3 over the row splits (blocks 0 ..
// 511, an element a thread), W1, b1, b2, b3 and w4 over the row blocks' halves (64 blocks of 32
// elements, eight interleaved runs each), b4 and the loss in the last block.
__global__ __launch_bounds__(256) void k_mlp_reduce(MlpRowArgs a, int splits, int nblk, float* __restrict__ grad,
                                                    double* __restrict__ loss) {
  const int b = blockIdx.x, tid = threadIdx.x;
  if (b < 512) {
    const int e = b * 256 + tid;   // W2 then W3
    float v[MLP_MAX_SPLITS], s = 0.f;   // every split's load in flight
#pragma unroll
    for (int z = 0; z < MLP_MAX_SPLITS; ++z) v[z] = z < splits ? a.wpart[(size_t)z * 2 * MLP_HID * MLP_HID + e] : 0.f;
#pragma unroll
    for (int z = 0; z < MLP_MAX_SPLITS; ++z) s += v[z];
    grad[e < MLP_HID * MLP_HID ? MLP_OFF_W2 + e : MLP_OFF_W3 + e - MLP_HID * MLP_HID] = s;
  } else if (b < 576) {
    __shared__ float red[8][32];
    const int e = (b - 512) * 32 + (tid & 31), q = tid >> 5;
    float s = 0.f;
    for (int k = q; k < 2 * nblk; k += 64) {   // eight loads in flight
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = k + 8 * u < 2 * nblk ? a.vpart[(size_t)(k + 8 * u) * MR_PART + e] : 0.f;
#pragma unroll
      for (int u = 0; u < 8; ++u) s += v[u];
    }
    red[q][tid & 31] = s;
    __syncthreads();
    if (q == 0) {
      for (int k = 1; k < 8; ++k) s += red[k][tid];
      const int o = e < 1280 ? e : e < 1536 ? MLP_OFF_B2 + e - 1280 : e < 1792 ? MLP_OFF_B3 + e - 1536 : MLP_OFF_W4 + e - 1792;
      grad[o] = s;   // W1 and b1 lie first in both layouts
    }
  } else {
    __shared__ double rl[256], rd[256];
    double l = 0.0, d = 0.0;
    for (int k = tid; k < nblk; k += 256) { l += a.lpart[2 * k]; d += a.lpart[2 * k + 1]; }
    rl[tid] = l;
    rd[tid] = d;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
      if (tid < w) { rl[tid] += rl[tid + w]; rd[tid] += rd[tid + w]; }
      __syncthreads();
    }
    if (tid == 0) {
      *loss = rl[0] / (double)a.n;
      grad[MLP_OFF_B4] = (float)rd[0];
    }
  }
}

// Adam with bias correction at step k = ts->step + 1 and learning rate
// lr_k = lr (1 + cos(pi local / K)) / 2 (cosine) or lr.
__global__ __launch_bounds__(256) void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                                              float* __restrict__ v, int n, const TrainState* __restrict__ ts) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int k = ts->step + 1;
  float lr = ts->lr;
  if (ts->cosine) lr *= 0.5f * (1.0f + cosf(3.14159265358979f * (float)ts->local / (float)ts->K));
  const float b1 = ts->b1, b2 = ts->b2;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.0f - b1) * gi;
  const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float mh = mi / (1.0f - powf(b1, (float)k));
  const float vh = vi / (1.0f - powf(b2, (float)k));
  p[i] -= lr * mh / (sqrtf(vh) + ts->eps);
}

__global__ void k_train_advance(TrainState* ts) {
  if (threadIdx.x == 0 && blockIdx.x == 0) { ts->step += 1; ts->local += 1; }
}

__global__ void k_train_set(TrainState* ts, float lr, int K, int cosine, int reset_step) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    ts->lr = lr; ts->K = K; ts->cosine = cosine; ts->local = 0;
    if (reset_step) ts->step = 0;
    ts->b1 = 0.9f; ts->b2 = 0.999f; ts->eps = 1e-8f;
  }
}

// ---------------------------------------------------------------- data and initialisation
// Normalisation of (X, t): per-column mean and population standard deviation (1 if zero),
// written to norm[0..9] = mu_x[4], s_x[4], mu_t, s_t.  One block, FP64 sums.
__global__ __launch_bounds__(256) void k_fit_norm(const float* __restrict__ X, const float* __restrict__ t, int n,
                                                  float* __restrict__ norm) {
  __shared__ double red[256];
  for (int c = 0; c < 5; ++c) {
    double s = 0.0, s2 = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) {
      const double x = c < 4 ? (double)X[(size_t)i * 4 + c] : (double)t[i];
      s += x;
      s2 += x * x;
    }
    double mean, var;
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
      if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
      __syncthreads();
    }
    mean = red[0] / n;
    __syncthreads();
    // second pass for the variance (sum of squared deviations)
    s2 = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) {
      const double x = c < 4 ? (double)X[(size_t)i * 4 + c] : (double)t[i];
      s2 += (x - mean) * (x - mean);
    }
    red[threadIdx.x] = s2;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
      if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
      __syncthreads();
    }
    var = red[0] / n;
    __syncthreads();
    if (threadIdx.x == 0) {
      const double sd = sqrt(var);
      if (c < 4) { norm[c] = (float)mean; norm[4 + c] = sd > 0 ? (float)sd : 1.0f; }
      else { norm[8] = (float)mean; norm[9] = sd > 0 ? (float)sd : 1.0f; }
    }
  }
}

// Xn = (X - mu_x) / s_x; tn = (t - mu_t) / s_t (t may be NULL).
__global__ __launch_bounds__(256) void k_normalise(const float* __restrict__ X, const float* __restrict__ t, int n,
                                                   const float* __restrict__ norm, float* __restrict__ Xn,
                                                   float* __restrict__ tn) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
#pragma unroll
  for (int c = 0; c < 4; ++c) Xn[(size_t)i * 4 + c] = (X[(size_t)i * 4 + c] - norm[c]) / norm[4 + c];
  if (t && tn) tn[i] = (t[i] - norm[8]) / norm[9];
}

// theta_j = a_j (2 u_j - 1), u_j the 24-bit uniform of word j % 4 of Philox4x64-10 block j / 4 under
// key (seed, 0x4D4C50), a_j = 1 / sqrt(fan_in) of the layer of parameter j.
__device__ __forceinline__ void philox4x64_10(unsigned long long* x, unsigned long long k0, unsigned long long k1) {
  const unsigned long long M0 = 0xD2E7470EE14C6C93ULL, M1 = 0xCA5A826395121157ULL;
  const unsigned long long W0 = 0x9E3779B97F4A7C15ULL, W1 = 0xBB67AE8584CAA73BULL;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) { k0 += W0; k1 += W1; }
    const unsigned long long h0 = __umul64hi(x[0], M0), l0 = x[0] * M0;
    const unsigned long long h1 = __umul64hi(x[2], M1), l1 = x[2] * M1;
    const unsigned long long y0 = h1 ^ x[1] ^ k0, y2 = h0 ^ x[3] ^ k1;
    x[0] = y0; x[1] = l1; x[2] = y2; x[3] = l0;
  }
}

__global__ __launch_bounds__(256) void k_mlp_init(float* __restrict__ p, unsigned long long seed) {
  const int blk = blockIdx.x * 256 + threadIdx.x;
  if (4 * blk >= MLP_NPARAM) return;
  unsigned long long x[4] = {(unsigned long long)blk, 0, 0, 0};
  philox4x64_10(x, seed, 0x4D4C50ULL);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int j = 4 * blk + q;
    if (j >= MLP_NPARAM) break;
    const double u = ((double)(x[q] >> 40) + 0.5) * 5.9604644775390625e-8;
    const double a = j < MLP_OFF_B1 ? 0.5 : (j < MLP_OFF_W2 ? 0.5 : 0.0625);  // 1/sqrt(4), 1/sqrt(256)
    p[j] = (float)(a * (2.0 * u - 1.0));
  }
}

// ---------------------------------------------------------------- BF16 inference
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__global__ __launch_bounds__(256) void k_to_bf16(const float* __restrict__ x, __bf16* __restrict__ y, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) y[i] = (__bf16)x[i];
}

// First layer in FP32 from normalised inputs: H1 = bf16(silu(Xn W1^T + b1)).
__global__ __launch_bounds__(256) void k_bf16_layer1(const float* __restrict__ Xn, int n, const float* __restrict__ p,
                                                     __bf16* __restrict__ H) {
  const long long e = (long long)blockIdx.x * 256 + threadIdx.x;
  if (e >= (long long)n * MLP_HID) return;
  const int r = (int)(e / MLP_HID), u = (int)(e - (long long)r * MLP_HID);
  float z = p[MLP_OFF_B1 + u];
#pragma unroll
  for (int k = 0; k < 4; ++k) z = fmaf(p[MLP_OFF_W1 + u * 4 + k], Xn[(size_t)r * 4 + k], z);
  H[e] = (__bf16)silu(z);
}

// Hidden layer on MFMA: Hout = bf16(silu(Hin Wb^T + b)), Hin [n][256] bf16, Wb [256][256] bf16.
// One wave per 32 x 32 output tile, K = 256 in 16 steps of mfma_f32_32x32x16_bf16.
__global__ __launch_bounds__(64) void k_bf16_hidden(const __bf16* __restrict__ Hin, int n, const __bf16* __restrict__ Wb,
                                                    const float* __restrict__ bias, __bf16* __restrict__ Hout) {
  const int lane = threadIdx.x;
  const int r0 = blockIdx.x * 32, c0 = blockIdx.y * 32;
  const int ra = r0 + (lane & 31), cb = c0 + (lane & 31), ks = (lane >> 5) * 8;
  f32x16 acc = {};
  const bf16x8 zero = {};
#pragma unroll 4
  for (int kk = 0; kk < MLP_HID; kk += 16) {
    const bf16x8 a = ra < n ? *(const bf16x8*)&Hin[(size_t)ra * MLP_HID + kk + ks] : zero;
    const bf16x8 b = *(const bf16x8*)&Wb[(size_t)cb * MLP_HID + kk + ks];
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int r = r0 + 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3);
    const int c = c0 + (lane & 31);
    if (r < n) Hout[(size_t)r * MLP_HID + c] = (__bf16)silu(acc[i] + bias[c]);
  }
}

// Output layer: y = mu_t + s_t (sum_u H3[u] w4[u] + b4), bf16 operands, FP32 sum.
__global__ __launch_bounds__(256) void k_bf16_out(const __bf16* __restrict__ H, int n, const __bf16* __restrict__ w4,
                                                  const float* __restrict__ p, const float* __restrict__ norm,
                                                  float* __restrict__ y) {
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= n) return;
  float s = 0.f;
  for (int u = 0; u < MLP_HID; ++u) s = fmaf((float)H[(size_t)r * MLP_HID + u], (float)w4[u], s);
  y[r] = norm[8] + norm[9] * (s + p[MLP_OFF_B4]);
}


// ---------------------------------------------------------------------------
// Gaussian flag proxy of the variance surrogate: the channel-domain cube whose delay transform is
// the window-convolved power P_w(k_perp, eta) = sum_q |w~(q)|^2 / nc^2 P(k_perp, eta - q).  By the
// convolution theorem its inverse DFT along eta is a(nu) xi_s(nu), with xi_s = IDFT_eta P (real:
// P is even in eta) and a(nu) = (1/nc) sum_mu w(mu) w(mu + nu) the window's autocorrelation.
// xi depends on the cell only through s = q_u^2 + q_v^2, so it is tabulated once per s.
// ---------------------------------------------------------------------------
// xi[s][nu] = (1/nc) sum_i P(s, i) cos(2 pi i nu / nc), P(s, i) = (cperp2 s + cpar2 eta_i^2)^(pk/2),
// eta_i the signed index of i; one block per s, threads over nu, P(s, .) and cos(2 pi m / nc) in LDS.
__global__ __launch_bounds__(256) void k_var_xi(int nc, double cperp2, double cpar2, double half_pk, double* xi) {
  extern __shared__ double sh[];   // [nc] P then [nc] cos table
  double* Ps = sh;
  double* ct = sh + nc;
  const int sidx = blockIdx.x;
  for (int i = threadIdx.x; i < nc; i += blockDim.x) {
    const int e = i < (nc + 1) / 2 ? i : i - nc;
    const double k2 = cperp2 * sidx + cpar2 * (double)e * e;
    Ps[i] = k2 > 0.0 ? pow(k2, half_pk) : 0.0;
    ct[i] = cos(2.0 * M_PI * (double)i / nc);
  }
  __syncthreads();
  for (int nu = threadIdx.x; nu < nc; nu += blockDim.x) {
    double acc = 0.0;
    int m = 0;   // i * nu mod nc
    for (int i = 0; i < nc; ++i) {
      acc = fma(Ps[i], ct[m], acc);
      m += nu;
      if (m >= nc) m -= nc;
    }
    xi[(size_t)sidx * nc + nu] = acc / nc;
  }
}

// V[nu][u][v] = a(nu) xi[s][nu] (complex128, imaginary part 0) on support cells 1 <= s <= smax.
__global__ __launch_bounds__(256) void k_var_cube(int n, int nh, int nc, int smax, const double* a, const double* xi,
                                                  double2* V) {
  const size_t total = (size_t)nc * n * nh;
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
    const int v = (int)(e % nh);
    const size_t r = e / nh;
    const int u = (int)(r % n);
    const int nu = (int)(r / n);
    const int qu = u < (n + 1) / 2 ? u : u - n;
    const int s = qu * qu + v * v;
    double x = 0.0;
    if (s >= 1 && s <= smax) x = a[nu] * xi[(size_t)s * nc + nu];
    V[e] = make_double2(x, 0.0);
  }
}
}  // namespace

// ---------------------------------------------------------------- launchers
// LDS of k_mlp_rows: two activation buffers, and the three of silu' when training
static size_t mr_lds(bool train) { return (train ? 5 : 2) * (size_t)MR_ROWS * MR_LD * sizeof(float); }
int mlp_row_blocks(int n) { return std::min((n + MR_ROWS - 1) / MR_ROWS, MR_MAX_BLOCKS); }
void launch_mlp_predict(const MlpRowArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_rows<false>, dim3(mlp_row_blocks(a.n)), dim3(512), mr_lds(false), s, a);
}
void launch_mlp_loss_grad(const MlpRowArgs& a, float* grad, double* loss, hipStream_t s) {
  const int nblk = mlp_row_blocks(a.n);
  (void)hipFuncSetAttribute((const void*)k_mlp_rows<true>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)mr_lds(true));
  hipLaunchKernelGGL(k_mlp_rows<true>, dim3(nblk), dim3(512), mr_lds(true), s, a);
  // 32 tiles: enough row splits for one block a CU, at least 64 rows each
  const int want = std::max(1, std::min(MLP_MAX_SPLITS, (a.n + 63) / 64));
  const int chunk = ((a.n + want - 1) / want + 15) / 16 * 16, splits = (a.n + chunk - 1) / chunk;
  hipLaunchKernelGGL(k_mlp_wgrad, dim3(16, 2, splits), dim3(256), 0, s, a, chunk);
  hipLaunchKernelGGL(k_mlp_reduce, dim3(577), dim3(256), 0, s, a, splits, nblk, grad, loss);
}
void launch_adam(float* p, const float* g, float* m, float* v, int n, const TrainState* ts, hipStream_t s) {
  hipLaunchKernelGGL(k_adam, dim3((n + 255) / 256), dim3(256), 0, s, p, g, m, v, n, ts);
  hipLaunchKernelGGL(k_train_advance, dim3(1), dim3(64), 0, s, (TrainState*)ts);
}
void launch_train_set(TrainState* ts, float lr, int K, int cosine, int reset_step, hipStream_t s) {
  hipLaunchKernelGGL(k_train_set, dim3(1), dim3(64), 0, s, ts, lr, K, cosine, reset_step);
}
void launch_fit_norm(const float* X, const float* t, int n, float* norm, hipStream_t s) {
  hipLaunchKernelGGL(k_fit_norm, dim3(1), dim3(256), 0, s, X, t, n, norm);
}
void launch_normalise(const float* X, const float* t, int n, const float* norm, float* Xn, float* tn, hipStream_t s) {
  hipLaunchKernelGGL(k_normalise, dim3((n + 255) / 256), dim3(256), 0, s, X, t, n, norm, Xn, tn);
}
void launch_mlp_init(float* p, unsigned long long seed, hipStream_t s) {
  const int nblk = (MLP_NPARAM + 3) / 4;
  hipLaunchKernelGGL(k_mlp_init, dim3((nblk + 255) / 256), dim3(256), 0, s, p, seed);
}
void launch_to_bf16(const float* x, void* y, int n, hipStream_t s) {
  hipLaunchKernelGGL(k_to_bf16, dim3((n + 255) / 256), dim3(256), 0, s, x, (__bf16*)y, n);
}
void launch_bf16_forward(const float* Xn, int n, const float* p, const float* norm, const void* W2b, const void* W3b,
                         const void* w4b, void* H1, void* H2, float* y, hipStream_t s) {
  const long long e = (long long)n * MLP_HID;
  hipLaunchKernelGGL(k_bf16_layer1, dim3((unsigned)((e + 255) / 256)), dim3(256), 0, s, Xn, n, p, (__bf16*)H1);
  dim3 grid((n + 31) / 32, MLP_HID / 32);
  hipLaunchKernelGGL(k_bf16_hidden, grid, dim3(64), 0, s, (const __bf16*)H1, n, (const __bf16*)W2b, p + MLP_OFF_B2,
                     (__bf16*)H2);
  hipLaunchKernelGGL(k_bf16_hidden, grid, dim3(64), 0, s, (const __bf16*)H2, n, (const __bf16*)W3b, p + MLP_OFF_B3,
                     (__bf16*)H1);
  hipLaunchKernelGGL(k_bf16_out, dim3((n + 255) / 256), dim3(256), 0, s, (const __bf16*)H1, n, (const __bf16*)w4b, p,
                     norm, y);
}

void launch_var_xi(int nc, int nsmax, double cperp2, double cpar2, double pk_index, double* xi, hipStream_t s) {
  const size_t lds = 2 * (size_t)nc * sizeof(double);
  hipLaunchKernelGGL(k_var_xi, dim3(nsmax + 1), dim3(256), lds, s, nc, cperp2, cpar2, 0.5 * pk_index, xi);
}
void launch_var_cube(int n, int nh, int nc, int smax, const double* a, const double* xi, void* V, hipStream_t s) {
  const size_t total = (size_t)nc * n * nh;
  size_t blocks = (total + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_var_cube, dim3((unsigned)blocks), dim3(256), 0, s, n, nh, nc, smax, a, xi, (double2*)V);
}
