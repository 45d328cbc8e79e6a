// mlp.hip -- the schedule-predicting network on gfx950: 32 -> 64 -> 64 -> 12,
// ReLU, softmax cross-entropy, Adam (Kingma & Ba 2015), all fp32.
//
// The network is tiny (7,052 parameters, ~14 kFLOP per sample and direction),
// so a step is bound by its launches and by the latency of each dependent
// pass over memory, not by arithmetic: twelve launches (three layers, loss,
// three weight gradients, two input gradients, mean loss, Adam, an event)
// took 52 us a step at batch 256.  Now it is two: sample_kernel takes every
// sample through the forward pass, the loss and the input gradients in one
// wave with the weights in LDS, and weight_kernel sums each weight's gradient
// over the batch and applies Adam to it: 16.5 us a step (5.8 and 5.5 us of
// kernels).  Every sum runs in a fixed order, so the results are
// deterministic run to run.  Parameter layout (flat, row-major): W1[64,32]
// b1[64] W2[64,64] b2[64] W3[12,64] b3[12].
//
#include "internal.h"
#include "mlp.h"

namespace hicr {

constexpr int kB1 = kMlpHidden * kMlpIn, kW2 = kB1 + kMlpHidden,
              kB2 = kW2 + kMlpHidden * kMlpHidden, kW3 = kB2 + kMlpHidden,
              kB3 = kW3 + kMlpOut * kMlpHidden;
static_assert(kB3 + kMlpOut == kMlpParams, "parameter layout");
static_assert(kMlpHidden == 64 && kMlpIn <= 64 && kMlpOut <= 16, "one lane per unit of a layer");

__device__ __forceinline__ float lane_of(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// Stage W[O][I] transposed, row i of O + 1 floats: lanes that read one row
// (the forward pass: lane = output) and lanes that read one column (the
// backward pass: lane = input) then both hit every bank once.
template <int I, int O>
__device__ __forceinline__ void stage(float *t, const float *W) {
  static_assert(I * O % 256 == 0, "whole rounds of the workgroup");
#pragma unroll
  for (int r = 0; r < I * O / 256; r++) {
    const int k = r * 256 + threadIdx.x;
    t[(k % I) * (O + 1) + k / I] = W[k];
  }
}

// Output `lane` of a layer: bias + sum_i W[o,i] x_i, from the bias in
// ascending i with fused multiply-adds (the host inference uses the same
// order); x_i is lane i's x.
template <int I, int O>
__device__ __forceinline__ float dense(const float *t, float bias, float x, int o) {
  float acc = bias;
#pragma unroll
  for (int i = 0; i < I; i++) acc = fmaf(t[i * (O + 1) + o], lane_of(x, i), acc);
  return acc;
}

// Input gradient `lane`: sum_o dy_o W[o,i], ascending o.
template <int O>
__device__ __forceinline__ float dense_back(const float *t, float dy, int i) {
  float acc = 0.f;
#pragma unroll
  for (int o = 0; o < O; o++) acc = fmaf(lane_of(dy, o), t[i * (O + 1) + o], acc);
  return acc;
}

// One wave per sample, four samples to a workgroup, persistent over the
// batch.  A workgroup stages the 28 KB of weights first (from the L2 after
// the first few), which costs about as much as one sample's chain of
// multiply-adds.  z gets the logits (forward only); with kTrain the
// activations and gradients that weight_kernel needs, dZ = (p - onehot(y)) / B,
// and the sample's cross-entropy log-sum-exp(z) - z_y.
constexpr uint32_t kSampleGroups = 1024;
template <bool kTrain>
__global__ __launch_bounds__(256) void sample_kernel(const float *params, const float *X,
                                                     const int32_t *y, uint32_t B, float *z_out,
                                                     MlpBufs m) {
  __shared__ float w1[kMlpIn * (kMlpHidden + 1)], w2[kMlpHidden * (kMlpHidden + 1)],
      w3[kMlpHidden * (kMlpOut + 1)];
  const int lane = threadIdx.x & 63;
  const int lo = lane < kMlpOut ? lane : 0;  // the last layer has fewer units than lanes
  const float b1 = params[kB1 + lane], b2 = params[kB2 + lane], b3 = params[kB3 + lo];
  stage<kMlpIn, kMlpHidden>(w1, params);
  stage<kMlpHidden, kMlpHidden>(w2, params + kW2);
  stage<kMlpHidden, kMlpOut>(w3, params + kW3);
  __syncthreads();
  for (size_t b = blockIdx.x * 4u + (threadIdx.x >> 6); b < B; b += gridDim.x * 4u) {
    const float x = lane < kMlpIn ? X[b * kMlpIn + lane] : 0.f;
    const float a1 = dense<kMlpIn, kMlpHidden>(w1, b1, x, lane);
    const float h1 = a1 > 0.f ? a1 : 0.f;
    const float a2 = dense<kMlpHidden, kMlpHidden>(w2, b2, h1, lane);
    const float h2 = a2 > 0.f ? a2 : 0.f;
    const float z = dense<kMlpHidden, kMlpOut>(w3, b3, h2, lo);
    if (!kTrain) {
      if (lane < kMlpOut) z_out[b * kMlpOut + lane] = z;
      continue;
    }
    float mx = lane_of(z, 0), sum = 0.f;
#pragma unroll
    for (int c = 1; c < kMlpOut; c++) mx = fmaxf(mx, lane_of(z, c));
    const float e = expf(z - mx);
#pragma unroll
    for (int c = 0; c < kMlpOut; c++) sum += lane_of(e, c);
    // A label outside [0, kMlpOut) is never used as an index: the sample's loss
    // is NaN (so a mean over the batch shows it) and it adds no gradient.
    const int yb = y[b];
    const bool valid = yb >= 0 && yb < kMlpOut;
    const float dz = valid ? (e / sum - (lane == yb ? 1.f : 0.f)) / (float)(int)B : 0.f;
    const float zy = __shfl(z, valid ? yb : 0);
    const float d2 = a2 > 0.f ? dense_back<kMlpOut>(w3, dz, lane) : 0.f;
    const float d1 = a1 > 0.f ? dense_back<kMlpHidden>(w2, d2, lane) : 0.f;
    m.h1[b * kMlpHidden + lane] = h1;
    m.h2[b * kMlpHidden + lane] = h2;
    m.d1[b * kMlpHidden + lane] = d1;
    m.d2[b * kMlpHidden + lane] = d2;
    if (lane < kMlpOut) m.dz[b * kMlpOut + lane] = dz;
    if (lane == 0) m.loss[b] = valid ? (mx + logf(sum)) - zy : __builtin_nanf("");
  }
}

struct WeightArgs {
  const float *X;
  MlpBufs m;
  uint32_t B;
  float *loss_mean;  // nullable
  float *grad;       // gradients out, or (null) the Adam step below
  float *p, *mo, *ve;
  float lr, bc1, bc2;
};

__device__ __forceinline__ void apply(const WeightArgs &a, int i, float g, float p, float mo,
                                      float ve) {
  if (a.grad) {
    a.grad[i] = g;
    return;
  }
  constexpr float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  const float mi = b1 * mo + (1.f - b1) * g;
  const float vi = b2 * ve + (1.f - b2) * g * g;
  a.mo[i] = mi;
  a.ve[i] = vi;
  a.p[i] = p - a.lr * (mi / a.bc1) / (sqrtf(vi / a.bc2) + eps);
}

// Sum of v over the workgroup's 1,024 threads, in every thread; fixed order.
__device__ __forceinline__ float group_sum(float v, float *wsum) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = v;
  __syncthreads();
  float s = 0.f;
#pragma unroll
  for (int w = 0; w < 16; w++) s += wsum[w];
  return s;
}

// dW[o,i] = sum_b dY[b,o] X[b,i] and db[o] = sum_b dY[b,o] for one output o:
// 1,024 / I threads share column i, each summing every (1,024 / I)-th sample,
// so a wave reads consecutive columns and a thread's loads (16 at batch 256)
// are all in flight at once; partial sums meet in LDS in a fixed order.
template <int I, int O>
__device__ __forceinline__ void weight_row(const WeightArgs &a, const float *dY, const float *X,
                                           int w_base, int b_base, int o) {
  __shared__ float part[1024];
  __shared__ float wsum[16];
  constexpr uint32_t kParts = 1024 / I;
  const uint32_t t = threadIdx.x, i = t % I, q = t / I;
  // threads 0..I-1 finish a weight each, thread I the bias
  const int mine = t < I ? w_base + o * I + (int)t : b_base + o;
  float p = 0.f, mo = 0.f, ve = 0.f;
  if (!a.grad && t <= I) {
    p = a.p[mine];
    mo = a.mo[mine];
    ve = a.ve[mine];
  }
  float acc = 0.f, bs = 0.f;
#pragma unroll 16
  for (size_t b = q; b < a.B; b += kParts) acc = fmaf(dY[b * O + o], X[b * I + i], acc);
  for (size_t b = t; b < a.B; b += 1024) bs += dY[b * O + o];
  part[t] = acc;
  const float db = group_sum(bs, wsum);  // (its barrier also covers part[])
  if (t < I) {
    float sum = 0.f;
#pragma unroll
    for (uint32_t k = 0; k < kParts; k++) sum += part[k * I + t];
    apply(a, mine, sum, p, mo, ve);
  } else if (t == I) {
    apply(a, mine, db, p, mo, ve);
  }
}

// One workgroup per output unit of the three layers, and one for the mean loss.
__global__ __launch_bounds__(1024) void weight_kernel(WeightArgs a) {
  const int o = blockIdx.x;
  if (o < kMlpHidden) {
    weight_row<kMlpHidden, kMlpHidden>(a, a.m.d2, a.m.h1, kW2, kB2, o);
  } else if (o < 2 * kMlpHidden) {
    weight_row<kMlpIn, kMlpHidden>(a, a.m.d1, a.X, 0, kB1, o - kMlpHidden);
  } else if (o < 2 * kMlpHidden + kMlpOut) {
    weight_row<kMlpHidden, kMlpOut>(a, a.m.dz, a.m.h2, kW3, kB3, o - 2 * kMlpHidden);
  } else {
    __shared__ float wsum[16];
    float acc = 0.f;
    for (size_t b = threadIdx.x; b < a.B; b += 1024) acc += a.m.loss[b];
    const float sum = group_sum(acc, wsum);
    if (threadIdx.x == 0) *a.loss_mean = sum / (float)(int)a.B;
  }
}

static inline uint32_t sample_groups(uint32_t B) {
  return B / 4 >= kSampleGroups ? kSampleGroups : (B + 3) / 4;
}

hipError_t mlp_forward(const float *params, const float *X, uint32_t B, float *z, hipStream_t s) {
  hipLaunchKernelGGL(sample_kernel<false>, dim3(sample_groups(B)), dim3(256), 0, s, params, X,
                     (const int32_t *)nullptr, B, z, MlpBufs{});
  return hipGetLastError();
}

static hipError_t train(WeightArgs a, const float *params, const int32_t *y, hipStream_t s) {
  hipLaunchKernelGGL(sample_kernel<true>, dim3(sample_groups(a.B)), dim3(256), 0, s, params, a.X,
                     y, a.B, (float *)nullptr, a.m);
  hipLaunchKernelGGL(weight_kernel, dim3(2 * kMlpHidden + kMlpOut + (a.loss_mean ? 1 : 0)),
                     dim3(1024), 0, s, a);
  return hipGetLastError();
}

hipError_t mlp_grad(const MlpBufs &m, const float *params, const float *X, const int32_t *y,
                    uint32_t B, float *grad, float *loss_mean, hipStream_t s) {
  WeightArgs a{};
  a.X = X;
  a.m = m;
  a.B = B;
  a.loss_mean = loss_mean;
  a.grad = grad;
  return train(a, params, y, s);
}

hipError_t mlp_step(const MlpBufs &m, float *params, float *mo, float *ve, const float *X,
                    const int32_t *y, uint32_t B, float lr, int t, float *loss_mean,
                    hipStream_t s) {
  WeightArgs a{};
  a.X = X;
  a.m = m;
  a.B = B;
  a.loss_mean = loss_mean;
  a.p = params;
  a.mo = mo;
  a.ve = ve;
  a.lr = lr;
  a.bc1 = 1.f - powf(0.9f, (float)t);
  a.bc2 = 1.f - powf(0.999f, (float)t);
  return train(a, params, y, s);
}

}  // namespace hicr
