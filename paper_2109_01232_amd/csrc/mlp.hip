// The parameter chooser's network 16-64-64-3 on the GPU: forward pass,
// mean-squared-error gradient and a fused Adam step.
//
// The network is tiny (5443 parameters, ~32 kFLOP per sample and step).  The
// forward kernel keeps the parameters in LDS, one thread per sample.  The
// gradient runs as one block: the parameters are updated in place and the
// entry points take no scratch memory, so there is nowhere to sum the partial
// gradients of several blocks.  Its products are fp32 matrix instructions
// (see mlp_grad_block); every sum has a fixed order.
#include <hip/hip_runtime.h>
#include <math.h>

#include "gmresir.h"
#include "internal.hpp"

namespace {

constexpr int NIN = 16, NH = 64, NOUT = 3;
constexpr int O_W1 = 0, O_B1 = O_W1 + NIN * NH, O_W2 = O_B1 + NH, O_B2 = O_W2 + NH * NH, O_W3 = O_B2 + NH,
              O_B3 = O_W3 + NH * NOUT, NPARAM = O_B3 + NOUT;
static_assert(NPARAM == 5443, "parameter count");

constexpr int TPB = 256;

// gradient kernel: 16 waves, chunks of 128 samples
constexpr int GT = 1024;
constexpr int GW = GT / 64;
constexpr int CH = 128;
constexpr int SPW = CH / GW;  // samples of a chunk per wave in the plain sums
// LDS row pitches = 2 mod 32: the 16 rows x 2 columns a half wave reads as a
// matrix operand fall into 32 different banks
constexpr int HP = NH + 2, XP = NIN + 2;
constexpr int NSUM = 5;  // per hidden unit summed without matrix instructions: b1, b2, three of W3

typedef float f32x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(TPB) void k_mlp_forward(const float* __restrict__ P, const float* __restrict__ shift,
                                                     const float* __restrict__ scale, const float* __restrict__ X,
                                                     float* __restrict__ Y, int batch) {
  __shared__ float sp[NPARAM];
  __shared__ float s_shift[NIN], s_scale[NIN];
  for (int i = threadIdx.x; i < NPARAM; i += TPB) sp[i] = P[i];
  if (threadIdx.x < NIN) {
    s_shift[threadIdx.x] = shift[threadIdx.x];
    s_scale[threadIdx.x] = scale[threadIdx.x];
  }
  __syncthreads();
  const int s = blockIdx.x * TPB + threadIdx.x;
  if (s >= batch) return;
  float x[NIN];
#pragma unroll
  for (int i = 0; i < NIN; ++i) x[i] = (X[(size_t)s * NIN + i] - s_shift[i]) * s_scale[i];
  float h1[NH];
#pragma unroll
  for (int o = 0; o < NH; ++o) {
    float a = sp[O_B1 + o];
#pragma unroll
    for (int i = 0; i < NIN; ++i) a += x[i] * sp[O_W1 + i * NH + o];
    h1[o] = tanhf(a);
  }
  float y[NOUT];
#pragma unroll
  for (int o = 0; o < NOUT; ++o) y[o] = sp[O_B3 + o];
  for (int o2 = 0; o2 < NH; ++o2) {
    float a = sp[O_B2 + o2];
#pragma unroll
    for (int i = 0; i < NH; ++i) a += h1[i] * sp[O_W2 + i * NH + o2];
    const float h2 = tanhf(a);
#pragma unroll
    for (int o = 0; o < NOUT; ++o) y[o] += h2 * sp[O_W3 + o2 * NOUT + o];
  }
#pragma unroll
  for (int o = 0; o < NOUT; ++o) Y[(size_t)s * NOUT + o] = y[o];
}

// Weights held by the block's waves for the whole call, as matrix operands:
// wave w works on the hidden units 16 (w % 4) .. + 15 of every product.
struct MlpWeights {
  float w1[NIN / 4];   // W1[4 q + l / 16][n]
  float w2[NH / 4];    // W2[4 q + l / 16][n]
  float w2t[NH / 4];   // W2[n][4 q + l / 16]
  float b1, b2;        // of unit n
};

// Gradient sums of the block (registers): the wave's 16 x 16 tile of W2 (and,
// waves 0..3, of W1), rows 4 (l / 16) + r, columns l % 16; sum: this wave's
// samples for unit `lane`.
struct MlpGrad {
  f32x4 w2, w1;
  float sum[NSUM];
  float b3;    // lanes 0..2
  float loss;  // threads 8 s
};

struct MlpShared {
  float x[CH * XP];
  float h1[CH * HP];
  float h2[CH * HP];  // h2, then the deltas of layer 1
  float d2[CH * HP];
  float dy[CH * 4];
  float w3[NH * NOUT], b3[NOUT];
  float shift[NIN], scale[NIN];
};

// rows m0 .. m0 + 15 of a (row pitch `pitch`, first column 0) times the wave's
// weight operand, K = 4 Q, added to acc
template <int Q>
__device__ __forceinline__ f32x4 rows_times(const float* a, int pitch, int m0, const float (&w)[Q], f32x4 acc,
                                            int lane) {
  const float* p = a + (m0 + (lane & 15)) * pitch + (lane >> 4);
#pragma unroll
  for (int q = 0; q < Q; ++q) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(p[4 * q], w[q], acc, 0, 0, 0);
  return acc;
}

// acc += a[0 .. 4 nq)^T b over the samples: units i0 + .. of a, o0 + .. of b
__device__ __forceinline__ f32x4 transposed_times(const float* a, int ap, int i0, const float* b, int bp, int o0,
                                                  int nq, f32x4 acc, int lane) {
  const float* pa = a + (lane >> 4) * ap + i0 + (lane & 15);
  const float* pb = b + (lane >> 4) * bp + o0 + (lane & 15);
#pragma unroll 4
  for (int q = 0; q < nq; ++q) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(pa[4 * q * ap], pb[4 * q * bp], acc, 0, 0, 0);
  return acc;
}

// Gradient of L = sum (y - t)^2 / (3 batch): 128 samples at a time through
// LDS.  The contractions (both hidden layers forward, layer 1's deltas, the
// gradients of W1 and W2) are v_mfma_f32_16x16x4 tiles, fp32 in and out:
// 8.4 MFLOP at batch 256, 14 us at one CU's matrix rate.  Four waves share a
// column of tiles and keep its weights in registers, so LDS holds activations
// only; the gradient tiles stay in registers over all chunks (16 tiles of W2,
// one a wave).  The few remaining sums (biases, W3) are split over the waves
// by sample and joined once at the end.  Rows past the batch have zero deltas.
// A training step at batch 256 takes 43 us; one thread per sample with the
// weights in LDS took 746 us.
__device__ __forceinline__ void mlp_grad_block(const float* __restrict__ P, const float* __restrict__ shift,
                                               const float* __restrict__ scale, const float* __restrict__ X,
                                               const float* __restrict__ T, int batch, MlpShared& S, MlpGrad& g) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid / 64);
  const int n0 = 16 * (wid % 4), n = n0 + (lane & 15), kq = lane >> 4;
  MlpWeights w;
#pragma unroll
  for (int q = 0; q < NIN / 4; ++q) w.w1[q] = P[O_W1 + (4 * q + kq) * NH + n];
#pragma unroll
  for (int q = 0; q < NH / 4; ++q) {
    w.w2[q] = P[O_W2 + (4 * q + kq) * NH + n];
    w.w2t[q] = P[O_W2 + n * NH + 4 * q + kq];
  }
  w.b1 = P[O_B1 + n];
  w.b2 = P[O_B2 + n];
  if (tid < NH * NOUT) S.w3[tid] = P[O_W3 + tid];
  if (tid < NOUT) S.b3[tid] = P[O_B3 + tid];
  if (tid < NIN) {
    S.shift[tid] = shift[tid];
    S.scale[tid] = scale[tid];
  }
  g.w2 = g.w1 = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < NSUM; ++q) g.sum[q] = 0.f;
  g.b3 = g.loss = 0.f;
  const float inv_n = 2.f / (3.f * (float)batch);
  __syncthreads();
  for (int c0 = 0; c0 < batch; c0 += CH) {
    const int cn = min(CH, batch - c0);
    const int mt = (cn + 15) / 16;  // tiles of 16 samples
    for (int i = tid; i < mt * 16 * NIN; i += GT) {
      const int s = i / NIN, k = i % NIN;
      S.x[s * XP + k] = s < cn ? (X[(size_t)c0 * NIN + i] - S.shift[k]) * S.scale[k] : 0.f;
    }
    __syncthreads();
    for (int m = wid / 4; m < mt; m += GW / 4) {
      const f32x4 a = rows_times(S.x, XP, 16 * m, w.w1, f32x4{w.b1, w.b1, w.b1, w.b1}, lane);
#pragma unroll
      for (int r = 0; r < 4; ++r) S.h1[(16 * m + 4 * kq + r) * HP + n] = tanhf(a[r]);
    }
    __syncthreads();
    for (int m = wid / 4; m < mt; m += GW / 4) {
      const f32x4 a = rows_times(S.h1, HP, 16 * m, w.w2, f32x4{w.b2, w.b2, w.b2, w.b2}, lane);
#pragma unroll
      for (int r = 0; r < 4; ++r) S.h2[(16 * m + 4 * kq + r) * HP + n] = tanhf(a[r]);
    }
    __syncthreads();
    {
      // output layer: eight threads per sample, eight hidden units each
      const int s = tid / 8, part = tid % 8;
      float y[NOUT] = {0.f, 0.f, 0.f};
      if (s < mt * 16) {
#pragma unroll
        for (int q = 0; q < NH / 8; ++q) {
          const int i = part + 8 * q;
          const float h = S.h2[s * HP + i];
#pragma unroll
          for (int o = 0; o < NOUT; ++o) y[o] += h * S.w3[i * NOUT + o];
        }
      }
#pragma unroll
      for (int o = 0; o < NOUT; ++o)
#pragma unroll
        for (int d = 1; d < 8; d *= 2) y[o] += __shfl_xor(y[o], d, 64);
      if (part == 0 && s < mt * 16) {
#pragma unroll
        for (int o = 0; o < NOUT; ++o) {
          const float d = s < cn ? y[o] + S.b3[o] - T[(size_t)(c0 + s) * NOUT + o] : 0.f;
          g.loss += d * d;
          S.dy[s * 4 + o] = inv_n * d;
        }
      }
    }
    __syncthreads();
    {
      // layer 2's deltas of unit `lane`, and this wave's samples of the plain sums
      float w3[NOUT];
#pragma unroll
      for (int o = 0; o < NOUT; ++o) w3[o] = S.w3[lane * NOUT + o];
#pragma unroll
      for (int q = 0; q < SPW; ++q) {
        const int s = wid + GW * q;
        if (s < mt * 16) {
          const float h = S.h2[s * HP + lane];
          float a = 0.f;
#pragma unroll
          for (int o = 0; o < NOUT; ++o) {
            const float dy = S.dy[s * 4 + o];
            a += dy * w3[o];
            g.sum[2 + o] += h * dy;
          }
          const float d = a * (1.f - h * h);
          S.d2[s * HP + lane] = d;
          g.sum[1] += d;
          if (lane < NOUT) g.b3 += S.dy[s * 4 + lane];
        }
      }
    }
    __syncthreads();
    for (int m = wid / 4; m < mt; m += GW / 4) {
      const f32x4 a = rows_times(S.d2, HP, 16 * m, w.w2t, f32x4{0.f, 0.f, 0.f, 0.f}, lane);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int s = 16 * m + 4 * kq + r;
        const float h = S.h1[s * HP + n];
        S.h2[s * HP + n] = a[r] * (1.f - h * h);
      }
    }
    g.w2 = transposed_times(S.h1, HP, 16 * (wid / 4), S.d2, HP, n0, mt * 4, g.w2, lane);
    __syncthreads();
    if (wid < 4) g.w1 = transposed_times(S.x, XP, 0, S.h2, HP, n0, mt * 4, g.w1, lane);
#pragma unroll
    for (int q = 0; q < SPW; ++q) {
      const int s = wid + GW * q;
      if (s < mt * 16) g.sum[0] += S.h2[s * HP + lane];
    }
    __syncthreads();
  }
}

// Hands every gradient entry to put(parameter, value) once, by the thread that
// holds it; returns the loss (thread 0).
template <typename F>
__device__ __forceinline__ float mlp_grad_store(MlpShared& S, const MlpGrad& g, int batch, F put) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid / 64);
  float* red = S.h1;              // [NSUM][GW][NH]
  float* red3 = S.d2;             // [GW][NOUT]
  float* redl = S.d2 + GW * NOUT; // [CH]
#pragma unroll
  for (int q = 0; q < NSUM; ++q) red[(q * GW + wid) * NH + lane] = g.sum[q];
  if (lane < NOUT) red3[wid * NOUT + lane] = g.b3;
  if (tid % 8 == 0) redl[tid / 8] = g.loss;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = 16 * (wid / 4) + 4 * (lane >> 4) + r, o = 16 * (wid % 4) + (lane & 15);
    put(O_W2 + i * NH + o, g.w2[r]);
    if (wid < 4) put(O_W1 + (4 * (lane >> 4) + r) * NH + o, g.w1[r]);
  }
  if (tid < NSUM * NH) {
    const int q = tid / NH, i = tid % NH;
    float a = 0.f;
    for (int v = 0; v < GW; ++v) a += red[(q * GW + v) * NH + i];
    put(q == 0 ? O_B1 + i : q == 1 ? O_B2 + i : O_W3 + i * NOUT + q - 2, a);
  } else if (tid >= GT - NOUT) {
    const int o = tid - (GT - NOUT);
    float a = 0.f;
    for (int v = 0; v < GW; ++v) a += red3[v * NOUT + o];
    put(O_B3 + o, a);
  }
  float loss = 0.f;
  if (tid == 0)
    for (int s = 0; s < CH; ++s) loss += redl[s];
  return loss / (3.f * (float)batch);
}

__global__ __launch_bounds__(GT) void k_mlp_loss_grad(const float* __restrict__ P, const float* __restrict__ shift,
                                                      const float* __restrict__ scale, const float* __restrict__ X,
                                                      const float* __restrict__ T, int batch, float* __restrict__ G,
                                                      float* __restrict__ loss) {
  __shared__ MlpShared S;
  MlpGrad g;
  mlp_grad_block(P, shift, scale, X, T, batch, S, g);
  const float l = mlp_grad_store(S, g, batch, [&](int p, float v) { G[p] = v; });
  if (threadIdx.x == 0) *loss = l;
}

__global__ __launch_bounds__(GT) void k_mlp_train_step(float* __restrict__ P, float* __restrict__ M,
                                                       float* __restrict__ Vv, const float* __restrict__ shift,
                                                       const float* __restrict__ scale, const float* __restrict__ X,
                                                       const float* __restrict__ T, int batch, float lr, int step,
                                                       float* __restrict__ loss) {
  __shared__ MlpShared S;
  MlpGrad g;
  mlp_grad_block(P, shift, scale, X, T, batch, S, g);
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  const float c1 = 1.f - powf(b1, (float)step);
  const float c2 = 1.f - powf(b2, (float)step);
  // P is read by every wave above and each entry written once here, by its one owner
  const float l = mlp_grad_store(S, g, batch, [&](int p, float gr) {
    const float m = b1 * M[p] + (1.f - b1) * gr;
    const float v = b2 * Vv[p] + (1.f - b2) * gr * gr;
    M[p] = m;
    Vv[p] = v;
    P[p] = P[p] - lr * (m / c1) / (sqrtf(v / c2) + eps);
  });
  if (threadIdx.x == 0) *loss = l;
}

}  // namespace

extern "C" {

int gmresir_mlp_forward(const float* params, const float* shift, const float* scale, const float* X, float* Y,
                        int32_t batch, void* stream) {
  if (!params || !shift || !scale || !X || !Y || batch < 1 || batch > (1 << 24)) {
    gir::set_error("gmresir_mlp_forward: bad arguments");
    return GMRESIR_ERR_INVALID_ARG;
  }
  const int g = (batch + TPB - 1) / TPB;
  hipLaunchKernelGGL(k_mlp_forward, dim3(g), dim3(TPB), 0, (hipStream_t)stream, params, shift, scale, X, Y, batch);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    gir::set_error("gmresir_mlp_forward: %s", hipGetErrorString(e));
    return GMRESIR_ERR_HIP;
  }
  return GMRESIR_OK;
}

int gmresir_mlp_loss_grad(const float* params, const float* shift, const float* scale, const float* X, const float* T,
                          int32_t batch, float* grad, float* loss, void* stream) {
  if (!params || !shift || !scale || !X || !T || !grad || !loss || batch < 1 || batch > 65536) {
    gir::set_error("gmresir_mlp_loss_grad: bad arguments");
    return GMRESIR_ERR_INVALID_ARG;
  }
  hipLaunchKernelGGL(k_mlp_loss_grad, dim3(1), dim3(GT), 0, (hipStream_t)stream, params, shift, scale, X, T, batch,
                     grad, loss);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    gir::set_error("gmresir_mlp_loss_grad: %s", hipGetErrorString(e));
    return GMRESIR_ERR_HIP;
  }
  return GMRESIR_OK;
}

int gmresir_mlp_train_step(float* params, float* adam_m, float* adam_v, const float* shift, const float* scale,
                           const float* X, const float* T, int32_t batch, float lr, int32_t step, float* loss,
                           void* stream) {
  if (!params || !adam_m || !adam_v || !shift || !scale || !X || !T || !loss || batch < 1 || batch > 65536 ||
      step < 1 || !(lr > 0.f)) {
    gir::set_error("gmresir_mlp_train_step: bad arguments");
    return GMRESIR_ERR_INVALID_ARG;
  }
  hipLaunchKernelGGL(k_mlp_train_step, dim3(1), dim3(GT), 0, (hipStream_t)stream, params, adam_m, adam_v, shift,
                     scale, X, T, batch, lr, step, loss);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    gir::set_error("gmresir_mlp_train_step: %s", hipGetErrorString(e));
    return GMRESIR_ERR_HIP;
  }
  return GMRESIR_OK;
}

}  // extern "C"
