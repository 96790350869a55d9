// sigma-surrogate network kernels (3-64-64-2 GELU MLP) for gfx950.
//
// A work-group of eight waves owns a 32-row tile at a time.  Layer 1 (K = 3) and layer
// 3 (N = 2) are plain FP32 fused multiply-adds on bfloat16-rounded operands; the 64x64
// products (forward layer 2, the W2 gradient and the back-propagated hidden-layer error)
// use v_mfma_f32_32x32x8_bf16, each 32x32 block in a wave of its own.  Intermediate
// activations live in LDS, the matrix operands in bfloat16 with the contraction index
// contiguous (a transposed copy where two products contract over different indexes), so
// that a lane reads its four values in one 8-byte access.  Gradients are accumulated per
// work-group (the W2 one in MFMA accumulators across tiles), written out per work-group
// and summed in a second pass in a fixed order, so results are deterministic.
//
// A batch of 1024 rows is 32 tiles: latency bounds the kernel, not work.  One wave per
// tile (every activation and gradient element in turn) took 45 us; eight waves with the
// elements dealt four to a thread, the gather of the minibatch in the same kernel and the
// sum over the work-groups fused with Adam, a training step went from 69 to 18.6 us, the
// forward pass of 4001 host rows from 61 to 23 us (one launch on pinned host memory
// instead of three copies and a launch).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <vector>

#include "lbm.h"
#include "lbm_mlp.h"

namespace mlp {

constexpr int NH = 64, TR = 32;
constexpr int OFF_W1 = 0, OFF_B1 = 192, OFF_W2 = 256, OFF_B2 = 4352, OFF_W3 = 4416, OFF_B3 = 4544;
constexpr int NP = MLP_NPARAMS;
constexpr int GMAX = 256;  // work-groups of the gradient pass

typedef short s4 __attribute__((ext_vector_type(4)));
typedef float f16v __attribute__((ext_vector_type(16)));

struct Norm {
  float in_mean[3], in_std[3], out_mean[2], out_std[2];
};

// float -> bfloat16 bits, round to nearest even (finite values)
__device__ __forceinline__ unsigned short f2bf(float f) {
  unsigned u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float bf2f(unsigned short b) { return __uint_as_float((unsigned)b << 16); }
__device__ __forceinline__ float qbf(float f) { return bf2f(f2bf(f)); }

__device__ __forceinline__ float gelu(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_d(float z) {
  return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

// MFMA 32x32x8 (bf16 in, FP32 accumulate), one wave:
//   C[m][n] += sum_k A(m, k) B(n, k),  m, n in [0, 32), k in [0, K), K % 8 == 0,
//   A(m, k) = a[m * sa + k], B(n, k) = b[n * sb + k]  (bfloat16 in LDS, strides a multiple of 4).
// Operand layout: lane l supplies row (l & 31) and k = k0 + 4 (l >> 5) + v, v < 4.
// Result layout: lane l, element i holds C[8 (i / 4) + 4 (l >> 5) + i % 4][l & 31].
template <int K>
__device__ __forceinline__ void mm32(const unsigned short* a, int sa, const unsigned short* b, int sb,
                                     f16v& c) {
  const int l = threadIdx.x & 63, r = l & 31, h = l >> 5;
#pragma unroll
  for (int k0 = 0; k0 < K; k0 += 8) {
    const s4 av = *reinterpret_cast<const s4*>(a + r * sa + k0 + 4 * h);
    const s4 bv = *reinterpret_cast<const s4*>(b + r * sb + k0 + 4 * h);
    c = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(av, bv, c, 0, 0, 0);
  }
}
__device__ __forceinline__ int crow(int i) { return 8 * (i >> 2) + 4 * ((threadIdx.x & 63) >> 5) + (i & 3); }

constexpr int NT = 512;                  // threads of a work-group
constexpr int SN = NH + 4, SM = TR + 4;  // row strides of the bfloat16 operands (contiguous in units, in rows)

struct alignas(16) MlpLds {
  unsigned short W2[NH * SN], W2t[NH * SN];         // [n][k] and [k][n]
  unsigned short h1[TR * SN], h1t[NH * SM];         // [m][k] and [k][m]
  unsigned short h2[TR * SN], dz[TR * SN], dzt[NH * SM];
  float W1[NH * 3], b1[NH], b2[NH], W3[2 * NH], b3[2];  // W1, W3 rounded to bfloat16
  float xs[TR][4];                                  // standardised inputs rounded to bfloat16
  float dy[TR][2];
  float za[TR][NH + 1], zb[TR][NH + 1];             // z2, then dZ2; dH1, then dZ1
  float red[NT];
};

// Forward pass of rows [0, B) of X (through idx where given), or the loss and its
// gradient.  Thread (wave w, lane l) of a tile owns unit l of rows w, w + 8, w + 16, w +
// 24 in both hidden layers.
template <bool TRAIN>
__global__ __launch_bounds__(NT) void k_mlp(const float* __restrict__ P, Norm nm,
                                            const float* __restrict__ X, const float* __restrict__ T,
                                            const int64_t* __restrict__ idx, float* __restrict__ Y, int B,
                                            float* __restrict__ gpart, float* __restrict__ lpart) {
  __shared__ MlpLds s;
  const int t = threadIdx.x, l = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  // the row's index (an epoch's permutation) and then the row itself are dependent loads:
  // the first tile's go out before the weights are staged, behind whose loads they hide
  const int ntiles = (B + TR - 1) / TR;
  float xin[3] = {0.f, 0.f, 0.f}, tgt = 0.f;  // input row l & 31 and its target of output l >> 5 (wave 0)
  auto load_row = [&](int tile) {
    const int r = tile * TR + (l & 31);
    if (w != 0 || r >= B) return;
    const int64_t rr = idx ? idx[r] : (int64_t)r;
    if (TRAIN) tgt = T[2 * rr + (l >> 5)];
#pragma unroll
    for (int i = 0; i < 3; ++i) xin[i] = X[3 * rr + i];
  };
  load_row(blockIdx.x);
#pragma unroll
  for (int i = t; i < NH * NH; i += NT) {
    const int n = i >> 6, k = i & 63;
    const unsigned short v = f2bf(P[OFF_W2 + i]);
    s.W2[n * SN + k] = v;
    if (TRAIN) s.W2t[k * SN + n] = v;
  }
  if (t < NH * 3) s.W1[t] = qbf(P[OFF_W1 + t]);
  if (t < NH) {
    s.b1[t] = P[OFF_B1 + t];
    s.b2[t] = P[OFF_B2 + t];
  }
  if (t < 2 * NH) s.W3[t] = qbf(P[OFF_W3 + t]);
  if (t < 2) s.b3[t] = P[OFF_B3 + t];

  // accumulators over the tiles of this work-group: waves 0..3 a 32x32 block of the W2
  // gradient; every thread one chain of b1 or W1 (see below); waves 6, 7 W3; wave 5 b2;
  // lanes 0, 1 of wave 4 b3; wave 0 the loss
  f16v gW2;
#pragma unroll
  for (int i = 0; i < 16; ++i) gW2[i] = 0.f;
  float g1 = 0.f, gW3 = 0.f, gb = 0.f, lsum = 0.f;

  for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int row0 = tile * TR;
    if (tile != (int)blockIdx.x) load_row(tile);
    if (w == 0 && l < TR) {  // standardised inputs; rows past B are zero and carry no gradient
#pragma unroll
      for (int i = 0; i < 3; ++i)
        s.xs[l][i] = qbf(row0 + l < B ? (xin[i] - nm.in_mean[i]) / nm.in_std[i] : 0.f);
    }
    __syncthreads();
    float d1[4];  // GELU'(z1)
    {             // layer 1
      const float w0 = s.W1[3 * l], w1 = s.W1[3 * l + 1], w2 = s.W1[3 * l + 2], b = s.b1[l];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int m = w + 8 * i;
        float acc = s.xs[m][0] * w0;
        acc = fmaf(s.xs[m][1], w1, acc);
        acc = fmaf(s.xs[m][2], w2, acc);
        const float z = acc + b;
        const unsigned short h = f2bf(gelu(z));
        s.h1[m * SN + l] = h;
        if (TRAIN) {
          s.h1t[l * SM + m] = h;
          d1[i] = gelu_d(z);
        }
      }
    }
    __syncthreads();
    if (w < 2) {  // layer 2: z2[m][n] = sum_k h1[m][k] W2[n][k] + b2[n], 32 columns a wave
      f16v c;
#pragma unroll
      for (int i = 0; i < 16; ++i) c[i] = 0.f;
      mm32<NH>(s.h1, SN, s.W2 + w * 32 * SN, SN, c);
      const int n = w * 32 + (l & 31);
#pragma unroll
      for (int i = 0; i < 16; ++i) s.za[crow(i)][n] = c[i] + s.b2[n];
    }
    __syncthreads();
    float d2[4];  // GELU'(z2)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int m = w + 8 * i;
      const float z = s.za[m][l];
      s.h2[m * SN + l] = f2bf(gelu(z));
      if (TRAIN) d2[i] = gelu_d(z);
    }
    __syncthreads();
    if (w == 0) {  // layer 3: lane -> row m, output o
      const int m = l & 31, o = l >> 5;
      float acc = 0.f;
#pragma unroll
      for (int n = 0; n < NH; n += 4) {
        const s4 h = *reinterpret_cast<const s4*>(s.h2 + m * SN + n);
#pragma unroll
        for (int v = 0; v < 4; ++v) acc = fmaf(bf2f((unsigned short)h[v]), s.W3[o * NH + n + v], acc);
      }
      const float y = acc + s.b3[o];
      const int r = row0 + m;
      if (!TRAIN) {
        if (r < B) Y[2 * r + o] = y * nm.out_std[o] + nm.out_mean[o];
      } else {
        float d = 0.f;
        if (r < B) {
          d = y - (tgt - nm.out_mean[o]) / nm.out_std[o];
          lsum = fmaf(d, d, lsum);
        }
        s.dy[m][o] = d / (float)B;
      }
    }
    if (TRAIN) {
      __syncthreads();
      {  // dZ2 = (dY W3) * GELU'(Z2)
        const float w0 = s.W3[l], w1 = s.W3[NH + l];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int m = w + 8 * i;
          const float g = fmaf(qbf(s.dy[m][1]), w1, qbf(s.dy[m][0]) * w0) * d2[i];
          const unsigned short q = f2bf(g);
          s.za[m][l] = g;
          s.dz[m * SN + l] = q;
          s.dzt[l * SM + m] = q;
        }
      }
      if (w >= 6) {  // W3: output w - 6, column l
#pragma unroll
        for (int m = 0; m < TR; ++m) gW3 = fmaf(qbf(s.dy[m][w - 6]), bf2f(s.h2[m * SN + l]), gW3);
      }
      __syncthreads();
      if (w < 4) {  // dW2[n][k] += sum_m dZ2[m][n] H1[m][k]
        mm32<TR>(s.dzt + (w >> 1) * 32 * SM, SM, s.h1t + (w & 1) * 32 * SM, SM, gW2);
      } else if (w == 4) {  // b3
        if (l < 2)
#pragma unroll
          for (int m = 0; m < TR; ++m) gb += s.dy[m][l];
      } else if (w == 5) {  // b2
#pragma unroll
        for (int m = 0; m < TR; ++m) gb += s.za[m][l];
      } else {  // dH1[m][k] = sum_n dZ2[m][n] W2[n][k], 32 columns a wave
        f16v c;
#pragma unroll
        for (int i = 0; i < 16; ++i) c[i] = 0.f;
        mm32<NH>(s.dz, SN, s.W2t + (w - 6) * 32 * SN, SN, c);
        const int k = (w - 6) * 32 + (l & 31);
#pragma unroll
        for (int i = 0; i < 16; ++i) s.zb[crow(i)][k] = c[i];
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 4; ++i) s.zb[w + 8 * i][l] *= d1[i];  // dZ1 = dH1 * GELU'(Z1)
      __syncthreads();
      // chains of unit l: wave w sums rows 8 j + 4 (w & 1) + (0..3) of b1 (w < 2) or of
      // column (w >> 1) - 1 of W1
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int m = 8 * (i >> 2) + 4 * (w & 1) + (i & 3);
        const float g = s.zb[m][l];
        g1 = w < 2 ? g1 + g : fmaf(qbf(g), s.xs[m][(w >> 1) - 1], g1);
      }
    }
    __syncthreads();  // the next tile overwrites LDS
  }
  if (!TRAIN) return;

  float* G = gpart + (size_t)blockIdx.x * NP;
  s.red[t] = g1;
  if (w == 0) s.dy[l >> 1][l & 1] = lsum;
  if (w < 4) {
#pragma unroll
    for (int i = 0; i < 16; ++i)
      G[OFF_W2 + ((w >> 1) * 32 + crow(i)) * NH + (w & 1) * 32 + (l & 31)] = gW2[i];
  }
  if (w == 5) G[OFF_B2 + l] = gb;
  if (w == 4 && l < 2) G[OFF_B3 + l] = gb;
  if (w >= 6) G[OFF_W3 + (w - 6) * NH + l] = gW3;
  __syncthreads();
  if ((w & 1) == 0) {  // the two row halves of a chain
    const float v = s.red[t] + s.red[t + 64];
    if (w == 0) G[OFF_B1 + l] = v;
    else G[OFF_W1 + 3 * l + (w >> 1) - 1] = v;
  }
  if (t == 64) {
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 64; ++i) sum += s.dy[i >> 1][i & 1];
    lpart[blockIdx.x] = sum;
  }
}

// Sum over the G work-groups in index order, 32 loads in flight.
__device__ __forceinline__ float group_sum(const float* __restrict__ g, int stride, int G) {
  float s = 0.f;
  int b = 0;
  for (; b + 32 <= G; b += 32) {
    float v[32];
#pragma unroll
    for (int i = 0; i < 32; ++i) v[i] = g[(size_t)(b + i) * stride];
#pragma unroll
    for (int i = 0; i < 32; ++i) s += v[i];
  }
  for (; b + 8 <= G; b += 8) {
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = g[(size_t)(b + i) * stride];
#pragma unroll
    for (int i = 0; i < 8; ++i) s += v[i];
  }
  for (; b < G; ++b) s += g[(size_t)b * stride];
  return s;
}

// One parameter's Adam step; c1 = 1 / (1 - beta1^t), c2 = 1 / (1 - beta2^t)
__device__ __forceinline__ void adam_one(float* __restrict__ P, float* __restrict__ m,
                                         float* __restrict__ v, int p, float gi, float lr, float b1,
                                         float b2, float eps, float c1, float c2) {
  const float mi = b1 * m[p] + (1.f - b1) * gi;
  const float vi = b2 * v[p] + (1.f - b2) * gi * gi;
  m[p] = mi;
  v[p] = vi;
  P[p] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
}

// grad[p] = sum over work-groups in index order; loss = sum / (2 B)
__global__ void k_reduce(const float* __restrict__ gpart, int G, float* __restrict__ grad,
                         const float* __restrict__ lpart, float* __restrict__ loss, int B) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p < NP) grad[p] = group_sum(gpart + p, NP, G);
  if (p == NP && loss) loss[0] = group_sum(lpart, 1, G) / (2.0f * (float)B);
}

// k_reduce and k_adam in one pass (a training step: two launches instead of three).
__global__ void k_reduce_adam(const float* __restrict__ gpart, int G, const float* __restrict__ lpart,
                              float* __restrict__ loss, int B, float* __restrict__ P, float* __restrict__ m,
                              float* __restrict__ v, float lr, float b1, float b2, float eps, float c1,
                              float c2) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p < NP) adam_one(P, m, v, p, group_sum(gpart + p, NP, G), lr, b1, b2, eps, c1, c2);
  if (p == NP && loss) loss[0] = group_sum(lpart, 1, G) / (2.0f * (float)B);
}

__global__ void k_adam(float* __restrict__ P, float* __restrict__ m, float* __restrict__ v,
                       const float* __restrict__ g, float lr, float b1, float b2, float eps, float c1,
                       float c2) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p < NP) adam_one(P, m, v, p, g[p], lr, b1, b2, eps, c1, c2);
}

}  // namespace mlp

using namespace mlp;

struct mlp_ctx {
  Norm nm;
  int max_batch;
  float *P, *m, *v, *grad, *gpart, *lpart, *loss;
  hipStream_t st;
  int64_t t;  // Adam steps taken
  float* host;  // pinned staging of mlp_forward_host: kHostRows rows of inputs, then outputs
  std::mutex host_lock;  // held while the staging is in use (callers on several threads)
};

namespace {
constexpr size_t kAl = 256;
size_t al(size_t x) { return (x + kAl - 1) / kAl * kAl; }
size_t layout(size_t* off) {
  size_t o = 0;
  const size_t sizes[7] = {NP * 4, NP * 4, NP * 4, NP * 4, (size_t)GMAX * NP * 4, GMAX * 4, 4};
  for (int i = 0; i < 7; ++i) {
    off[i] = o;
    o += al(sizes[i]);
  }
  return o;
}
Norm to_norm(const mlp_norm& n) {
  Norm r;
  std::memcpy(&r, &n, sizeof r);
  return r;
}
int grad_blocks(int B) { return std::min(GMAX, (B + TR - 1) / TR); }
int forward_blocks(int B) { return std::min(4096, (B + TR - 1) / TR); }
constexpr int kHostRows = 4096;
constexpr int kSumBlock = 64;  // threads of the summing kernels: 72 blocks for 4546 parameters and the loss
constexpr int kSumGrid = (NP + 1 + kSumBlock - 1) / kSumBlock;

// Bias corrections of Adam step t.
float bias_corr(float beta, int64_t t) { return (float)(1.0 / (1.0 - std::pow((double)beta, (double)t))); }

// Gradient and Adam (0.9, 0.999, 1e-8) of B rows (through idx where given): two launches.
int train_one(mlp_ctx* c, const float* X, const float* T, const int64_t* idx, int B, float lr, float* loss) {
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  const int G = grad_blocks(B);
  hipLaunchKernelGGL(k_mlp<true>, dim3(G), dim3(NT), 0, c->st, (const float*)c->P, c->nm, X, T, idx,
                     (float*)nullptr, B, c->gpart, c->lpart);
  if (hipGetLastError() != hipSuccess) return LBM_EHIP;
  c->t += 1;
  hipLaunchKernelGGL(k_reduce_adam, dim3(kSumGrid), dim3(kSumBlock), 0, c->st, (const float*)c->gpart, G,
                     (const float*)c->lpart, loss, B, c->P, c->m, c->v, lr, b1, b2, eps,
                     bias_corr(b1, c->t), bias_corr(b2, c->t));
  return hipGetLastError() == hipSuccess ? LBM_OK : LBM_EHIP;
}
}  // namespace

extern "C" {

int mlp_workspace_bytes(int32_t max_batch, size_t* bytes) {
  if (max_batch < 1 || !bytes) return LBM_EINVAL;
  size_t off[7];
  *bytes = layout(off);
  return LBM_OK;
}

int mlp_init(const float* host_params, const mlp_norm* norm, int32_t max_batch, void* ws,
             size_t ws_bytes, void* stream, mlp_ctx** out) {
  if (!host_params || !norm || max_batch < 1 || !ws || !out) return LBM_EINVAL;
  *out = nullptr;
  size_t off[7];
  if (ws_bytes < layout(off)) return LBM_ENOSPACE;
  if (reinterpret_cast<uintptr_t>(ws) % kAl) return LBM_EINVAL;
  for (int i = 0; i < 3; ++i)
    if (!(norm->in_std[i] > 0)) return LBM_EINVAL;
  for (int i = 0; i < 2; ++i)
    if (!(norm->out_std[i] > 0)) return LBM_EINVAL;
  mlp_ctx* c = new mlp_ctx{};
  char* w = static_cast<char*>(ws);
  c->P = reinterpret_cast<float*>(w + off[0]);
  c->m = reinterpret_cast<float*>(w + off[1]);
  c->v = reinterpret_cast<float*>(w + off[2]);
  c->grad = reinterpret_cast<float*>(w + off[3]);
  c->gpart = reinterpret_cast<float*>(w + off[4]);
  c->lpart = reinterpret_cast<float*>(w + off[5]);
  c->loss = reinterpret_cast<float*>(w + off[6]);
  c->nm = to_norm(*norm);
  c->max_batch = max_batch;
  c->st = static_cast<hipStream_t>(stream);
  int st = mlp_set_params(c, host_params);
  if (st != LBM_OK) {
    delete c;
    return st;
  }
  *out = c;
  return LBM_OK;
}

int mlp_set_params(mlp_ctx* c, const float* host_params) {
  if (!c || !host_params) return LBM_EINVAL;
  std::vector<float> zero(NP, 0.f);
  if (hipMemcpyAsync(c->P, host_params, NP * 4, hipMemcpyHostToDevice, c->st) != hipSuccess ||
      hipMemcpyAsync(c->m, zero.data(), NP * 4, hipMemcpyHostToDevice, c->st) != hipSuccess ||
      hipMemcpyAsync(c->v, zero.data(), NP * 4, hipMemcpyHostToDevice, c->st) != hipSuccess ||
      hipStreamSynchronize(c->st) != hipSuccess)
    return LBM_EHIP;
  c->t = 0;
  return LBM_OK;
}

int mlp_get_params(mlp_ctx* c, float* host_params) {
  if (!c || !host_params) return LBM_EINVAL;
  if (hipMemcpyAsync(host_params, c->P, NP * 4, hipMemcpyDeviceToHost, c->st) != hipSuccess ||
      hipStreamSynchronize(c->st) != hipSuccess)
    return LBM_EHIP;
  return LBM_OK;
}

int mlp_set_norm(mlp_ctx* c, const mlp_norm* norm) {
  if (!c || !norm) return LBM_EINVAL;
  c->nm = to_norm(*norm);
  return LBM_OK;
}

int mlp_forward(mlp_ctx* c, const float* X, float* Y, int32_t B) {
  if (!c || !X || !Y || B < 1 || B > c->max_batch) return LBM_EINVAL;
  hipLaunchKernelGGL(k_mlp<false>, dim3(forward_blocks(B)), dim3(NT), 0, c->st, (const float*)c->P, c->nm,
                     X, (const float*)nullptr, (const int64_t*)nullptr, Y, B, (float*)nullptr,
                     (float*)nullptr);
  return hipGetLastError() == hipSuccess ? LBM_OK : LBM_EHIP;
}

int mlp_forward_host(mlp_ctx* c, const float* X, float* Y, int32_t B) {
  if (!c || !X || !Y || B < 1 || B > c->max_batch) return LBM_EINVAL;
  const std::lock_guard<std::mutex> hold(c->host_lock);
  if (!c->host) {
    void* h = nullptr;
    if (hipHostMalloc(&h, kHostRows * 5 * sizeof(float), hipHostMallocDefault) != hipSuccess) return LBM_EHIP;
    c->host = static_cast<float*>(h);
  }
  float *hx = c->host, *hy = c->host + 3 * kHostRows;
  for (int32_t r = 0; r < B; r += kHostRows) {
    const int n = std::min<int32_t>(kHostRows, B - r);
    std::memcpy(hx, X + 3 * (size_t)r, 3 * (size_t)n * sizeof(float));
    const int st = mlp_forward(c, hx, hy, n);
    if (st != LBM_OK) return st;
    if (hipStreamSynchronize(c->st) != hipSuccess) return LBM_EHIP;
    std::memcpy(Y + 2 * (size_t)r, hy, 2 * (size_t)n * sizeof(float));
  }
  return LBM_OK;
}

int mlp_gradient(mlp_ctx* c, const float* X, const float* T, int32_t B, float* grad, float* loss) {
  if (!c || !X || !T || !grad || B < 1 || B > c->max_batch) return LBM_EINVAL;
  const int G = grad_blocks(B);
  hipLaunchKernelGGL(k_mlp<true>, dim3(G), dim3(NT), 0, c->st, (const float*)c->P, c->nm, X, T,
                     (const int64_t*)nullptr, (float*)nullptr, B, c->gpart, c->lpart);
  hipLaunchKernelGGL(k_reduce, dim3(kSumGrid), dim3(kSumBlock), 0, c->st, (const float*)c->gpart, G,
                     grad, (const float*)c->lpart, loss, B);
  return hipGetLastError() == hipSuccess ? LBM_OK : LBM_EHIP;
}

int mlp_adam(mlp_ctx* c, const float* grad, float lr, float b1, float b2, float eps) {
  if (!c || !grad || !(lr > 0) || !(b1 >= 0 && b1 < 1) || !(b2 >= 0 && b2 < 1) || !(eps > 0))
    return LBM_EINVAL;
  c->t += 1;
  hipLaunchKernelGGL(k_adam, dim3((NP + 255) / 256), dim3(256), 0, c->st, c->P, c->m, c->v, grad, lr, b1,
                     b2, eps, bias_corr(b1, c->t), bias_corr(b2, c->t));
  return hipGetLastError() == hipSuccess ? LBM_OK : LBM_EHIP;
}

int mlp_train_step(mlp_ctx* c, const float* X, const float* T, int32_t B, float lr, float* loss) {
  if (!c || !X || !T || B < 1 || B > c->max_batch) return LBM_EINVAL;
  if (!(lr > 0)) return LBM_EINVAL;
  return train_one(c, X, T, nullptr, B, lr, loss);
}

int mlp_train_steps(mlp_ctx* c, const float* X, const float* T, const int64_t* idx, int32_t B, int32_t n,
                    const float* lr, float* loss) {
  if (!c || !X || !T || !idx || !lr || B < 1 || B > c->max_batch || n < 1) return LBM_EINVAL;
  for (int32_t i = 0; i < n; ++i)
    if (!(lr[i] > 0)) return LBM_EINVAL;
  for (int32_t i = 0; i < n; ++i) {
    const int st = train_one(c, X, T, idx + (size_t)i * B, B, lr[i], loss);
    if (st != LBM_OK) return st;
  }
  return LBM_OK;
}

int mlp_destroy(mlp_ctx* c) {
  if (!c) return LBM_EINVAL;
  (void)hipStreamSynchronize(c->st);
  if (c->host) (void)hipHostFree(c->host);
  delete c;
  return LBM_OK;
}

}  // extern "C"
