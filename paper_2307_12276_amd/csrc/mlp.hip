// Learned spectral-interval predictor: field statistics and a 9-64-64-64-3
// tanh MLP in FP32 with hand-written forward, backward and Adam kernels.
//
// Packed parameters: for each layer l, W_l [in][out] row-major then b_l[out].
// Activation cache per row: X (9) | H1 (64) | H2 (64) | H3 (64).
//
// These networks are tiny (9155 parameters) and latency-bound: the forward
// kernel gives each sample one wave64 (one lane per hidden unit, activations
// in LDS); the backward kernel gives each block 16 columns of one layer's
// gradient, a fixed-order sum over samples (bitwise reproducible, no atomics).
#include "bounds.h"

namespace adl {

constexpr int kIn = 9, kH = 64, kOut = 3;
constexpr int oW1 = 0, oB1 = oW1 + kIn * kH;
constexpr int oW2 = oB1 + kH, oB2 = oW2 + kH * kH;
constexpr int oW3 = oB2 + kH, oB3 = oW3 + kH * kH;
constexpr int oW4 = oB3 + kH, oB4 = oW4 + kH * kOut;
constexpr int kParams = oB4 + kOut;
static_assert(kParams == 9155, "parameter count");
constexpr int kCache = kIn + 3 * kH;  // 201

// ---------------------------------------------------------------------------
// forward: one wave per sample
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void mlp_forward_kernel(const float* __restrict__ W, const float* __restrict__ X,
                                                          float* __restrict__ Y, float* __restrict__ cache, int B) {
  __shared__ float act[4][kH];
  __shared__ float xin[4][kIn];
  const int w = threadIdx.x >> 6, t = threadIdx.x & 63;
  const int b = blockIdx.x * 4 + w;
  const bool valid = b < B;
  if (valid && t < kIn) {
    const float v = X[(long)b * kIn + t];
    xin[w][t] = v;
    if (cache) cache[(long)b * kCache + t] = v;
  }
  __syncthreads();
  // layer 1
  float z = W[oB1 + t];
  for (int i = 0; i < kIn; ++i) z += xin[w][i] * W[oW1 + i * kH + t];
  float h = tanhf(z);
  if (valid && cache) cache[(long)b * kCache + kIn + t] = h;
  act[w][t] = h;
  __syncthreads();
  // layers 2 and 3
  for (int layer = 0; layer < 2; ++layer) {
    const int oW = layer == 0 ? oW2 : oW3, oB = layer == 0 ? oB2 : oB3;
    z = W[oB + t];
    for (int k = 0; k < kH; ++k) z += act[w][k] * W[oW + k * kH + t];
    h = tanhf(z);
    __syncthreads();
    act[w][t] = h;
    if (valid && cache) cache[(long)b * kCache + kIn + (layer + 1) * kH + t] = h;
    __syncthreads();
  }
  // output layer (linear)
  if (valid && t < kOut) {
    float y = W[oB4 + t];
    for (int k = 0; k < kH; ++k) y += act[w][k] * W[oW4 + k * kOut + t];
    Y[(long)b * kOut + t] = y;
  }
}

// ---------------------------------------------------------------------------
// backward:
//   G4 = dY;  G3 = (G4 W4^T) (1 - H3^2);  G2 = (G3 W3^T)(1 - H2^2);  G1 = ...
//   dW_l[i][o] = sum_b Hin_l[b][i] G_l[b][o],   db_l[o] = sum_b G_l[b][o]
//
// A block owns 16 columns of one layer's gradient (block 12: layer 4's three)
// and forms the G it needs itself, so that no sum crosses blocks: layer 3 needs
// 16 columns of G3, layer 2 of G2, layer 1 all of G2 and 16 columns of G1.  A
// wave owns every 16th tile of 16 samples; all products are 16 x 16 x 4 FP32
// matrix instructions (FP32 inputs and sums), the samples being the rows of
// G = (G W^T)(1 - H^2) and the contraction of dW = H^T G.  The contraction's
// order is free as long as both operands agree: lane (i, q) = (l mod 16, l / 16)
// takes columns 16 q + t in step t of G W^T (16 floats in a row of memory), and
// samples 4 q + r in step r of H^T G, where a result of the first product
// already lies.  Only G2 of the layer 1 blocks passes through LDS, and only
// within a wave.  The waves' sums meet in LDS, added in wave order: every
// gradient is a fixed-order sum (bitwise reproducible, no atomics).
//
// Bound by the layer 1 blocks' matrix instructions (84 per 16 samples, four
// waves a SIMD) and the latency of their loads.  256 samples: one block
// walking the batch in chunks of 32 with a thread per parameter took 310 us,
// this takes 18 us (1024 samples 1199 / 55, 16 samples 21.7 / 9.9), its error
// against 64-bit sums 1.9e-7 where that had 3.4e-7 (1024: 2.0e-7 / 6.2e-7).
// ---------------------------------------------------------------------------
constexpr int kBwdWaves = 16;
constexpr int kBwdTile = 16;              // samples of a tile, columns of a block
constexpr int kBwdRow = kH + 1;           // LDS row of a wave's G2 (odd: no bank conflicts)
constexpr int kBwdBlocks = 3 * (kH / kBwdTile) + 1;
typedef float mfrag __attribute__((ext_vector_type(4)));
struct __attribute__((packed, aligned(4))) MlpRow16 {
  float v[16];
};

__device__ __forceinline__ mfrag mlp_mfma(float a, float b, mfrag c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__global__ __launch_bounds__(64 * kBwdWaves) void mlp_backward_kernel(const float* __restrict__ W,
                                                                      const float* __restrict__ cache,
                                                                      const float* __restrict__ dY,
                                                                      float* __restrict__ dW, int B) {
  // a wave's G2 while the batch is walked, its sums afterwards
  __shared__ float sh[kBwdWaves][kBwdTile * kBwdRow];
  __shared__ float shb[kBwdWaves][kBwdTile];
  static_assert(kBwdTile * kBwdRow >= 16 * 64, "a wave's four tiles of sums");
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63, i = l & 15, q = l >> 4;
  const int layer = blockIdx.x == kBwdBlocks - 1 ? 4 : 1 + blockIdx.x / (kH / kBwdTile);
  const int col = layer == 4 ? 0 : blockIdx.x % (kH / kBwdTile) * kBwdTile + i;  // the lane's column of G
  const mfrag zero = {0.0f, 0.0f, 0.0f, 0.0f};
  mfrag acc[4] = {zero, zero, zero, zero};  // dW rows 16 a + 4 q + r, the lane's column
  float accb = 0.0f;

  // (G4 W4^T)[s][k]
  auto g3 = [&](const float (&g4)[kOut], int k) {
    float g = 0.0f;
#pragma unroll
    for (int o = 0; o < kOut; ++o) g += g4[o] * W[oW4 + k * kOut + o];
    return g;
  };
  for (int b0 = wave * kBwdTile; b0 < B; b0 += kBwdWaves * kBwdTile) {
    float G[4];  // G_layer of samples 4 q + r at the lane's column
    bool in[4];
    const float* hs[4];  // their rows of the cache (the last sample's past the end)
    float f[4] = {1.0f, 1.0f, 1.0f, 1.0f};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int s = b0 + 4 * q + r;
      in[r] = s < B;
      hs[r] = cache + (long)min(s, B - 1) * kCache;
      if (layer < 4) {
        const float h = hs[r][kIn + (layer - 1) * kH + col];
        f[r] = 1.0f - h * h;
      }
    }
    if (layer >= 3) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float* d = dY + (long)min(b0 + 4 * q + r, B - 1) * kOut;
        const float g4[kOut] = {d[0], d[1], d[2]};
        G[r] = layer == 4 ? (i < kOut ? d[min(i, kOut - 1)] : 0.0f) : g3(g4, col) * f[r];
      }
    } else {
      // G3 of sample b0 + i at columns 16 q .. 16 q + 15
      const int s = min(b0 + i, B - 1);
      const float* d = dY + (long)s * kOut;
      const float g4[kOut] = {d[0], d[1], d[2]};
      const MlpRow16 h3 = *reinterpret_cast<const MlpRow16*>(cache + (long)s * kCache + kIn + 2 * kH + 16 * q);
      float a[16];
#pragma unroll
      for (int t = 0; t < 16; ++t) a[t] = g3(g4, 16 * q + t) * (1.0f - h3.v[t] * h3.v[t]);
      if (layer == 2) {
        const MlpRow16 w3 = *reinterpret_cast<const MlpRow16*>(W + oW3 + col * kH + 16 * q);
        mfrag c = zero;
#pragma unroll
        for (int t = 0; t < 16; ++t) c = mlp_mfma(a[t], w3.v[t], c);
#pragma unroll
        for (int r = 0; r < 4; ++r) G[r] = c[r] * f[r];
      } else {
        const MlpRow16 h2 = *reinterpret_cast<const MlpRow16*>(cache + (long)s * kCache + kIn + kH + 16 * q);
        const MlpRow16 w2 = *reinterpret_cast<const MlpRow16*>(W + oW2 + col * kH + 16 * q);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const MlpRow16 w3 = *reinterpret_cast<const MlpRow16*>(W + oW3 + (16 * k + i) * kH + 16 * q);
          mfrag c = zero;
#pragma unroll
          for (int t = 0; t < 16; ++t) c = mlp_mfma(a[t], w3.v[t], c);
#pragma unroll
          for (int r = 0; r < 4; ++r) sh[wave][(4 * q + r) * kBwdRow + 16 * k + i] = c[r];
        }
        // (a wave's own LDS: its writes come before its reads)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        mfrag c = zero;
#pragma unroll
        for (int t = 0; t < 16; ++t)
          c = mlp_mfma(sh[wave][i * kBwdRow + 16 * q + t] * (1.0f - h2.v[t] * h2.v[t]), w2.v[t], c);
#pragma unroll
        for (int r = 0; r < 4; ++r) G[r] = c[r] * f[r];
      }
    }
    // dW += Hin^T G (samples past the end count zero)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      G[r] = in[r] ? G[r] : 0.0f;
      accb += G[r];
      if (layer == 1) {
        acc[0] = mlp_mfma(in[r] && i < kIn ? hs[r][min(i, kIn - 1)] : 0.0f, G[r], acc[0]);
      } else {
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          const float h = hs[r][kIn + (layer - 2) * kH + 16 * a + i];
          acc[a] = mlp_mfma(in[r] ? h : 0.0f, G[r], acc[a]);
        }
      }
    }
  }
  accb += __shfl_xor(accb, 16);
  accb += __shfl_xor(accb, 32);
  __syncthreads();
#pragma unroll
  for (int a = 0; a < 4; ++a) {
#pragma unroll
    for (int r = 0; r < 4; ++r) sh[wave][(4 * a + r) * 64 + l] = acc[a][r];
  }
  if (q == 0) shb[wave][i] = accb;
  __syncthreads();
  // entry e of the 64 x 16 sums: row 16 a + 4 q + r, column i
  const int oW = layer == 1 ? oW1 : layer == 2 ? oW2 : layer == 3 ? oW3 : oW4;
  const int oB = layer == 1 ? oB1 : layer == 2 ? oB2 : layer == 3 ? oB3 : oB4;
  const int nout = layer == 4 ? kOut : kH, nin = layer == 1 ? kIn : kH;
  const int c0 = layer == 4 ? 0 : col - i;
  {
    const int e = threadIdx.x, ei = e & 15, eq = (e >> 4) & 3, er = (e >> 6) & 3, ea = e >> 8;
    const int row = 16 * ea + 4 * eq + er, o = c0 + ei;
    if (row < nin && o < nout) {
      float v = 0.0f;
#pragma unroll
      for (int w = 0; w < kBwdWaves; ++w) v += sh[w][e];
      dW[oW + row * nout + o] = v;
    }
    if (e < kBwdTile && o < nout) {
      float v = 0.0f;
#pragma unroll
      for (int w = 0; w < kBwdWaves; ++w) v += shb[w][e];
      dW[oB + o] = v;
    }
  }
}

// Mean squared error L = mean((Y - T)^2) over B x 3 and dL/dY = 2 (Y - T) / (3 B);
// one block, fixed-order sum.
__global__ __launch_bounds__(256) void mlp_mse_grad_kernel(const float* __restrict__ Y, const float* __restrict__ T,
                                                           float* __restrict__ dY, float* __restrict__ loss, int B) {
  __shared__ float sh[256];
  const int n = B * kOut;
  const float sc = 2.0f / (float)n;
  float acc = 0.0f;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const float d = Y[i] - T[i];
    dY[i] = sc * d;
    acc += d * d;
  }
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0 && loss) loss[0] = sh[0] / (float)n;
}

// Adam (Kingma & Ba 2015): bias corrections bc1 = 1 - b1^t, bc2 = 1 - b2^t.
__global__ __launch_bounds__(256) void mlp_adam_kernel(float* __restrict__ W, const float* __restrict__ dW,
                                                       float* __restrict__ m1, float* __restrict__ m2, float lr,
                                                       float b1, float b2, float eps, float bc1, float bc2) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= kParams) return;
  const float g = dW[i];
  const float m = b1 * m1[i] + (1.0f - b1) * g;
  const float v = b2 * m2[i] + (1.0f - b2) * g * g;
  m1[i] = m;
  m2[i] = v;
  const float mh = m / bc1, vh = v / bc2;
  W[i] = W[i] - lr * mh / (sqrtf(vh) + eps);
}

// ---------------------------------------------------------------------------
// field statistics: per-node eigenvalues of [[Dxx, Dxy], [Dxy, Dyy]] and |a|
// ---------------------------------------------------------------------------
template <typename TF, bool ADVF>
__global__ __launch_bounds__(kBlock) void field_stats_kernel(FieldView F, double hx, double hy, double dt,
                                                             float* __restrict__ feats, double* partials,
                                                             Ctl* ctl) {
  field_stats_blocks<TF, ADVF>(F, hx, hy, dt, feats, partials, ctl, (int)gridDim.x, (int)blockIdx.x);
}

hipError_t launch_field_stats(const FieldView& f, double hx, double hy, double dt, float* feats, double* partials,
                              Ctl* ctl, hipStream_t st) {
  const int nb = stats_blocks((long)f.nx * f.ny);
  const bool advf = f.ax != nullptr;
  if (f.f32) {
    if (advf)
      hipLaunchKernelGGL((field_stats_kernel<float, true>), dim3(nb), dim3(kBlock), 0, st, f, hx, hy, dt, feats, partials, ctl);
    else
      hipLaunchKernelGGL((field_stats_kernel<float, false>), dim3(nb), dim3(kBlock), 0, st, f, hx, hy, dt, feats, partials, ctl);
  } else {
    if (advf)
      hipLaunchKernelGGL((field_stats_kernel<double, true>), dim3(nb), dim3(kBlock), 0, st, f, hx, hy, dt, feats, partials, ctl);
    else
      hipLaunchKernelGGL((field_stats_kernel<double, false>), dim3(nb), dim3(kBlock), 0, st, f, hx, hy, dt, feats, partials, ctl);
  }
  return hipGetLastError();
}

// Batched statistics: every job's ctl[0] and ctl[1] cleared, one thread per job.
__global__ __launch_bounds__(kBlock) void bound_jobs_reset_kernel(const BoundJob* __restrict__ jobs, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    Ctl* c = jobs[i].ctl;
    const Ctl z{};
    c[0] = z;
    c[1] = z;
  }
}

// Block b finds its job (the one i with blk0[i] <= b < blk0[i + 1]; blk0 is
// strictly increasing from 0 and the grid has blk0[n] blocks, so exactly one
// thread finds it) and runs that job's statistics or Gershgorin block.
__global__ __launch_bounds__(kBlock) void bound_stats_many_kernel(const BoundJob* __restrict__ jobs,
                                                                  const int* __restrict__ blk0, int n, double dt,
                                                                  float* __restrict__ feats, double* gmin) {
  __shared__ int s_job;
  const int b = blockIdx.x;
  for (int i = threadIdx.x; i < n; i += blockDim.x)
    if (blk0[i] <= b && b < blk0[i + 1]) s_job = i;
  __syncthreads();
  const int i = s_job;
  const BoundJob J = jobs[i];
  const int lb = b - J.blk0;
  const bool advf = J.f.ax != nullptr;
  if (lb < J.nb_s) {
    float* fo = feats + 9L * i;
    if (J.f.f32) {
      if (advf) field_stats_blocks<float, true>(J.f, J.hx, J.hy, dt, fo, J.partials, J.ctl, J.nb_s, lb);
      else field_stats_blocks<float, false>(J.f, J.hx, J.hy, dt, fo, J.partials, J.ctl, J.nb_s, lb);
    } else {
      if (advf) field_stats_blocks<double, true>(J.f, J.hx, J.hy, dt, fo, J.partials, J.ctl, J.nb_s, lb);
      else field_stats_blocks<double, false>(J.f, J.hx, J.hy, dt, fo, J.partials, J.ctl, J.nb_s, lb);
    }
  } else {
    double* pg = J.partials + kGershPartials;
    const int gb = lb - J.nb_s;
    if (J.f.f32) {
      if (advf) gershgorin_blocks<float, true>(J.f, pg, J.ctl + 1, J.nb_g, gb, gmin + i);
      else gershgorin_blocks<float, false>(J.f, pg, J.ctl + 1, J.nb_g, gb, gmin + i);
    } else {
      if (advf) gershgorin_blocks<double, true>(J.f, pg, J.ctl + 1, J.nb_g, gb, gmin + i);
      else gershgorin_blocks<double, false>(J.f, pg, J.ctl + 1, J.nb_g, gb, gmin + i);
    }
  }
}

hipError_t launch_bound_stats_many(const BoundJob* jobs, const int* blk0, int n, int nblocks, double dt,
                                   float* feats, double* gmin, hipStream_t st) {
  if (n < 1 || nblocks < n) return hipErrorInvalidValue;
  hipLaunchKernelGGL(bound_jobs_reset_kernel, dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0, st, jobs, n);
  hipLaunchKernelGGL(bound_stats_many_kernel, dim3(nblocks), dim3(kBlock), 0, st, jobs, blk0, n, dt, feats, gmin);
  return hipGetLastError();
}

hipError_t launch_mlp_forward(const float* W, const float* X, float* Y, float* cache, int B, hipStream_t st) {
  hipLaunchKernelGGL(mlp_forward_kernel, dim3((B + 3) / 4), dim3(256), 0, st, W, X, Y, cache, B);
  return hipGetLastError();
}

hipError_t launch_mlp_backward(const float* W, const float* cache, const float* dY, float* dW, int B, hipStream_t st) {
  hipLaunchKernelGGL(mlp_backward_kernel, dim3(kBwdBlocks), dim3(64 * kBwdWaves), 0, st, W, cache, dY, dW, B);
  return hipGetLastError();
}

hipError_t launch_mlp_mse_grad(const float* Y, const float* T, float* dY, float* loss, int B, hipStream_t st) {
  hipLaunchKernelGGL(mlp_mse_grad_kernel, dim3(1), dim3(256), 0, st, Y, T, dY, loss, B);
  return hipGetLastError();
}

hipError_t launch_mlp_adam(float* W, const float* dW, float* m1, float* m2, int t, float lr, float b1, float b2,
                           float eps, hipStream_t st) {
  const double bc1 = 1.0 - pow((double)b1, (double)t), bc2 = 1.0 - pow((double)b2, (double)t);
  hipLaunchKernelGGL(mlp_adam_kernel, dim3((kParams + 255) / 256), dim3(256), 0, st, W, dW, m1, m2, lr, b1, b2, eps,
                     (float)bc1, (float)bc2);
  return hipGetLastError();
}

}  // namespace adl
