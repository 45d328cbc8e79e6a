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
// over the batch and applies Adam to it: 9.4 us a step (4.2 and 4.4 us of
// kernels, of which about 2 each are their start and end).  Every sum runs in a fixed order, so the results are
// deterministic run to run.  Parameter layout (flat, row-major): W1[64,32]
// b1[64] W2[64,64] b2[64] W3[12,64] b3[12].
//
#include <algorithm>

#include "internal.h"
#include "mlp.h"
#include "span.h"

namespace hicr {

constexpr int kB1 = kMlpHidden * kMlpIn, kW2 = kB1 + kMlpHidden,
              kB2 = kW2 + kMlpHidden * kMlpHidden, kW3 = kB2 + kMlpHidden,
              kB3 = kW3 + kMlpOut * kMlpHidden;
static_assert(kB3 + kMlpOut == kMlpParams, "parameter layout");
static_assert(kMlpHidden == 64 && kMlpIn <= 64 && kMlpOut <= 16, "one lane per unit of a layer");
static_assert(kMlpIn % 4 == 0 && kMlpOut % 4 == 0 && kW2 % 4 == 0 && kW3 % 4 == 0, "16-byte reads");

__device__ __forceinline__ float lane_of(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// A layer's weights W[O][I] in LDS, rows of I + 4 floats: 16-byte reads of one
// row per lane (the forward pass: lane = output) and reads of one row by all
// lanes (the backward pass: lane = input) then both use every bank evenly.
template <int I, int O, int T>
__device__ __forceinline__ void stage(float *t, const float *W) {
#pragma unroll
  for (int r = 0; r < (I * O / 4 + T - 1) / T; r++) {
    const int k = 4 * (r * T + (int)threadIdx.x);
    if (I * O % (4 * T) == 0 || k < I * O)
      *(float4 *)&t[k / I * (I + 4) + k % I] = *(const float4 *)&W[k];
  }
}

// N floats of LDS in registers, read 16 bytes at a time.
template <int N>
struct Vec {
  float4 v[N / 4];
  __device__ __forceinline__ void load(const float *t) {
#pragma unroll
    for (int k = 0; k < N / 4; k++) v[k] = *(const float4 *)&t[4 * k];
  }
};

// Lane values of a wave, through its 64 floats of LDS into registers of every
// lane (passing them on by v_readlane cost 28 cycles a multiply-add, 4,500 for
// the forward pass and 1,650 for the backward pass; now 2,700 and 700).
template <int N>
__device__ __forceinline__ Vec<N> spread(float *s, float v, int lane) {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  s[lane] = v;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  Vec<N> r;
  r.load(s);
  return r;
}

// init + sum_i w_i x_i, ascending i with fused multiply-adds (the host
// inference uses the same order).
template <int N>
__device__ __forceinline__ float dot(float init, const Vec<N> &w, const Vec<N> &x) {
  float acc = init;
#pragma unroll
  for (int k = 0; k < N / 4; k++) {
    acc = fmaf(w.v[k].x, x.v[k].x, acc);
    acc = fmaf(w.v[k].y, x.v[k].y, acc);
    acc = fmaf(w.v[k].z, x.v[k].z, acc);
    acc = fmaf(w.v[k].w, x.v[k].w, acc);
  }
  return acc;
}

// Column i of the first N rows (of I + 4 floats) of a layer's weights.
template <int I, int N>
__device__ __forceinline__ Vec<N> column(const float *t, int i) {
  Vec<N> c;
#pragma unroll
  for (int k = 0; k < N / 4; k++)
    c.v[k] = make_float4(t[4 * k * (I + 4) + i], t[(4 * k + 1) * (I + 4) + i],
                         t[(4 * k + 2) * (I + 4) + i], t[(4 * k + 3) * (I + 4) + i]);
  return c;
}

// One wave per sample, kWaves samples to a workgroup, persistent over the
// batch.  A workgroup stages the 28 KB of weights first (from the L2 after
// the first few), which costs about as much as one sample's chain of
// multiply-adds.  z gets the logits (forward only); with kTrain the
// activations and gradients that weight_kernel needs, dZ = (p - onehot(y)) / B,
// and the sample's cross-entropy log-sum-exp(z) - z_y.
//
// Reading a sample's weights takes the LDS 500 cycles, so waves of one
// workgroup wait for each other; up to two samples per compute unit each has
// a workgroup of its own (a step of 256 samples 9.4 us, with four to a
// workgroup 10.0; of 512 11.4 and 11.8; of 768 the same; of 2,048 24.2 and 23.1).
constexpr uint32_t kSampleGroups = 1024, kFewSamples = 512;
template <bool kTrain, int kWaves>
__global__ __launch_bounds__(64 * kWaves) void sample_kernel(const float *params, const float *X,
                                                     const int32_t *y, uint32_t B, float *z_out,
                                                     MlpBufs m) {
  __shared__ __attribute__((aligned(16))) float w1[kMlpHidden * (kMlpIn + 4)],
      w2[kMlpHidden * (kMlpHidden + 4)], w3[kMlpOut * (kMlpHidden + 4)], vec[kWaves][64];
  const int lane = threadIdx.x & 63;
  float *v = vec[threadIdx.x >> 6];
  const int lo = lane < kMlpOut ? lane : 0;  // the last layer has fewer units than lanes
  // the first sample's inputs are on their way while the weights are staged
  // (and each next one's during the one before)
  size_t b = blockIdx.x * (unsigned)kWaves + (threadIdx.x >> 6);
  float x = 0.f;
  int yb = 0;
  auto fetch = [&](size_t k) {
    if (k >= B) return;
    if (lane < kMlpIn) x = X[k * kMlpIn + lane];
    if (kTrain) yb = y[k];
  };
  fetch(b);
  const float b1 = params[kB1 + lane], b2 = params[kB2 + lane], b3 = params[kB3 + lo];
  stage<kMlpIn, kMlpHidden, 64 * kWaves>(w1, params);
  stage<kMlpHidden, kMlpHidden, 64 * kWaves>(w2, params + kW2);
  stage<kMlpHidden, kMlpOut, 64 * kWaves>(w3, params + kW3);
  __syncthreads();
  for (; b < B; b += gridDim.x * (unsigned)kWaves) {
    const int label = yb;
    // each layer's weights are read before the layer above it is summed (in
    // the order of the code: left alone the compiler reads four at a time)
    Vec<kMlpIn> r1;
    r1.load(&w1[lane * (kMlpIn + 4)]);
    const Vec<kMlpIn> v0 = spread<kMlpIn>(v, x, lane);
    fetch(b + gridDim.x * (unsigned)kWaves);
    Vec<kMlpHidden> r2, r3;
    r2.load(&w2[lane * (kMlpHidden + 4)]);
    order();
    const float a1 = dot(b1, r1, v0);
    const float h1 = a1 > 0.f ? a1 : 0.f;
    const Vec<kMlpHidden> v1 = spread<kMlpHidden>(v, h1, lane);
    r3.load(&w3[lo * (kMlpHidden + 4)]);
    order();
    const float a2 = dot(b2, r2, v1);
    const float h2 = a2 > 0.f ? a2 : 0.f;
    const Vec<kMlpHidden> v2 = spread<kMlpHidden>(v, h2, lane);
    order();
    const float z = dot(b3, r3, v2);
    if (!kTrain) {
      if (lane < kMlpOut) z_out[b * kMlpOut + lane] = z;
      continue;
    }
    const Vec<kMlpOut> c3 = column<kMlpHidden, kMlpOut>(w3, lane);
    const Vec<kMlpHidden> c2 = column<kMlpHidden, kMlpHidden>(w2, lane);
    order();
    float mx = lane_of(z, 0), sum = 0.f;
#pragma unroll
    for (int c = 1; c < kMlpOut; c++) mx = fmaxf(mx, lane_of(z, c));
    const float e = expf(z - mx);
#pragma unroll
    for (int c = 0; c < kMlpOut; c++) sum += lane_of(e, c);
    // A label outside [0, kMlpOut) is never used as an index: the sample's loss
    // is NaN (so a mean over the batch shows it) and it adds no gradient.
    const bool valid = label >= 0 && label < kMlpOut;
    const float dz = valid ? (e / sum - (lane == label ? 1.f : 0.f)) / (float)(int)B : 0.f;
    const float zy = __shfl(z, valid ? label : 0);
    const float g2 = dot(0.f, c3, spread<kMlpOut>(v, dz, lane)), d2 = a2 > 0.f ? g2 : 0.f;
    const Vec<kMlpHidden> v3 = spread<kMlpHidden>(v, d2, lane);
    order();
    const float g1 = dot(0.f, c2, v3), d1 = a1 > 0.f ? g1 : 0.f;
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

template <bool kGrad>
__device__ __forceinline__ void apply(const WeightArgs &a, int i, float g, float p, float mo,
                                      float ve) {
  if (kGrad) {
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
// so a wave reads consecutive columns and a thread's loads (of 16 samples at
// batch 256) are all in flight at once; partial sums meet in LDS in a fixed order.  The
// parameters and the bias's first sample are read before, without a branch
// (threads that have none repeat another's): at the end of a branch the
// compiler waits for what was loaded in it.
template <bool kGrad, int I, int O>
__device__ __forceinline__ void weight_row(const WeightArgs &a, const float *dY, const float *X,
                                           int w_base, int b_base, int o) {
  __shared__ float part[1024];
  __shared__ float wsum[16];
  constexpr uint32_t kParts = 1024 / I;
  const uint32_t t = threadIdx.x, i = t % I, q = t / I;
  // threads 0..I-1 finish a weight each, thread I the bias
  const int mine = t < I ? w_base + o * I + (int)t : b_base + o;
  float p = 0.f, mo = 0.f, ve = 0.f;
  if (!kGrad) {
    p = a.p[mine];
    mo = a.mo[mine];
    ve = a.ve[mine];
  }
  const float first = dY[(size_t)(t < a.B ? t : a.B - 1) * O + o];
  float acc = 0.f, bs = t < a.B ? first : 0.f;
  constexpr uint32_t kRound = 256 / kParts;  // samples of a thread in one round of 256
  for (size_t b0 = q; b0 < a.B; b0 += 256) {
    float y[kRound], x[kRound];
#pragma unroll
    for (uint32_t k = 0; k < kRound; k++) {
      const size_t b = b0 + k * kParts < a.B ? b0 + k * kParts : a.B - 1;
      y[k] = dY[b * O + o];
      x[k] = X[b * I + i];
    }
    order();  // all of them first: left alone the compiler waits in between
#pragma unroll
    for (uint32_t k = 0; k < kRound; k++)
      acc = b0 + k * kParts < a.B ? fmaf(y[k], x[k], acc) : acc;
  }
  for (size_t b = t + 1024; b < a.B; b += 1024) bs += dY[b * O + o];
  part[t] = acc;
  const float db = group_sum(bs, wsum);  // (its barrier also covers part[])
  if (t < I) {
    float sum = 0.f;
#pragma unroll
    for (uint32_t k = 0; k < kParts; k++) sum += part[k * I + t];
    apply<kGrad>(a, mine, sum, p, mo, ve);
  } else if (t == I) {
    apply<kGrad>(a, mine, db, p, mo, ve);
  }
}

// One workgroup per output unit of the three layers, and one for the mean loss.
template <bool kGrad>
__global__ __launch_bounds__(1024) void weight_kernel(WeightArgs a) {
  const int o = blockIdx.x;
  if (o < kMlpHidden) {
    weight_row<kGrad, kMlpHidden, kMlpHidden>(a, a.m.d2, a.m.h1, kW2, kB2, o);
  } else if (o < 2 * kMlpHidden) {
    weight_row<kGrad, kMlpIn, kMlpHidden>(a, a.m.d1, a.X, 0, kB1, o - kMlpHidden);
  } else if (o < 2 * kMlpHidden + kMlpOut) {
    weight_row<kGrad, kMlpHidden, kMlpOut>(a, a.m.dz, a.m.h2, kW3, kB3, o - 2 * kMlpHidden);
  } else {
    __shared__ float wsum[16];
    float acc = 0.f;
    for (size_t b = threadIdx.x; b < a.B; b += 1024) acc += a.m.loss[b];
    const float sum = group_sum(acc, wsum);
    if (threadIdx.x == 0) *a.loss_mean = sum / (float)(int)a.B;
  }
}

template <bool kTrain>
static void launch_samples(const float *params, const float *X, const int32_t *y, uint32_t B,
                           float *z, const MlpBufs &m, hipStream_t s) {
  const uint32_t waves = B <= kFewSamples ? 1 : 4;
  const uint32_t groups = std::min((B + waves - 1) / waves, kSampleGroups);
  const auto kernel = waves == 1 ? sample_kernel<kTrain, 1> : sample_kernel<kTrain, 4>;
  hipLaunchKernelGGL(kernel, dim3(groups), dim3(64 * waves), 0, s, params, X, y, B, z, m);
}

hipError_t mlp_forward(const float *params, const float *X, uint32_t B, float *z, hipStream_t s) {
  launch_samples<false>(params, X, nullptr, B, z, MlpBufs{}, s);
  return hipGetLastError();
}

static hipError_t train(WeightArgs a, const float *params, const int32_t *y, hipStream_t s) {
  launch_samples<true>(params, a.X, y, a.B, nullptr, a.m, s);
  hipLaunchKernelGGL(a.grad ? weight_kernel<true> : weight_kernel<false>,
                     dim3(2 * kMlpHidden + kMlpOut + (a.loss_mean ? 1 : 0)), dim3(1024), 0, s, a);
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
