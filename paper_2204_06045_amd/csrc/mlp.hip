// Learned cost model: a 16-64-64-4 multilayer perceptron predicting the log
// launch time of a group under each kernel variant, trained on timings the
// autotuner measures.  Forward, backward and Adam are hand-written FP32
// kernels; every reduction runs in a fixed order, so results are
// deterministic.
//
// Parameter layout (floats): W1[16][64], b1[64], W2[64][64], b2[64],
// W3[64][4], b3[4], row-major with the input index first.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "mlp.hpp"

namespace qtn {
namespace {

// One pass over the batch.  A block holds the weights in LDS (W2 a second
// time, transposed, for the backward product) and walks chunks of kChunk
// samples: forward, and with STEP the loss, the backward pass and the weight
// gradient, which it accumulates in registers over its chunks and writes as
// one partial sum per block (k_mlp_reduce adds the partial sums in block
// order).  Without STEP it writes the outputs y.
//
// Bound: latency.  A batch of 4,000 samples is 0.13 GFLOP and 0.4 MB per
// epoch, under 2 us of either rate; what counts is how few dependent steps an
// epoch has.  Activations never leave LDS, and 16 samples per block give 250
// blocks for those 4,000.  Thread (i, j0) = (t / 16, 4 (t % 16)) forms four
// neighbouring units of sample i, so a weight row is read as float4 by 16
// lanes and an activation is broadcast; in the gradient the same thread owns
// the 4 x 4 tile of W2 at (4 i, j0).  Measured at 4,000 samples: 16.8 us, and
// 7.5 us for the reduction with the Adam step, an epoch; one launch per layer
// and direction, with a thread summing each weight's gradient over all
// samples (0.98 ms a launch), took 3.06 ms an epoch.
constexpr int kChunk = 16;
constexpr int kW2T = kMlpHidden + 4;  // padded row of the transposed copy
constexpr int kPartStride = (kMlpParams + 2 + 63) / 64 * 64;  // gradient, loss, mask count

__device__ __forceinline__ void fma4(float4 &a, float s, const float4 &w) {
  a.x = fmaf(s, w.x, a.x);
  a.y = fmaf(s, w.y, a.y);
  a.z = fmaf(s, w.z, a.z);
  a.w = fmaf(s, w.w, a.w);
}
__device__ __forceinline__ float4 ld4(const float *p) { return *(const float4 *)p; }
__device__ __forceinline__ void st4(float *p, const float4 &v) { *(float4 *)p = v; }

// a += in[0..K) . W[0..K)[j0..j0+3], W with rows of `ld` floats (LDS)
template <int K>
__device__ __forceinline__ float4 row4(float4 a, const float *in, const float *W, int ld, int j0) {
#pragma unroll 4
  for (int k = 0; k < K; k += 4) {
    const float4 h = ld4(in + k);
    fma4(a, h.x, ld4(W + k * ld + j0));
    fma4(a, h.y, ld4(W + (k + 1) * ld + j0));
    fma4(a, h.z, ld4(W + (k + 2) * ld + j0));
    fma4(a, h.w, ld4(W + (k + 3) * ld + j0));
  }
  return a;
}

template <bool STEP>
__global__ __launch_bounds__(256) void k_mlp_pass(const float *__restrict__ params,
                                                  const float *__restrict__ x,
                                                  const float *__restrict__ t,
                                                  const float *__restrict__ m, int n,
                                                  float *__restrict__ y, float *__restrict__ part) {
  constexpr int H = kMlpHidden, I = kMlpIn, O = kMlpOut;
  __shared__ __align__(16) float sW1[I * H], sW2[H * H], sW3[H * O], sb1[H], sb2[H], sb3[O];
  __shared__ __align__(16) float sW2t[STEP ? H * kW2T : 4];
  __shared__ __align__(16) float sx[kChunk * I], sh1[kChunk * H], sh2[kChunk * H], sdy[kChunk * O];
  __shared__ __align__(16) float sd1[STEP ? kChunk * H : 4], sd2[STEP ? kChunk * H : 4];
  const int tid = threadIdx.x, i = tid >> 4, j0 = (tid & 15) * 4;
  const float *W1 = params, *b1 = W1 + I * H, *W2 = b1 + H, *b2 = W2 + H * H, *W3 = b2 + H,
              *b3 = W3 + H * O;
  for (int e = tid; e < I * H; e += 256) sW1[e] = W1[e];
  for (int e = tid; e < H * H; e += 256) {
    const float w = W2[e];
    sW2[e] = w;
    if (STEP) sW2t[(e % H) * kW2T + e / H] = w;
  }
  for (int e = tid; e < H * O; e += 256) sW3[e] = W3[e];
  if (tid < H) {
    sb1[tid] = b1[tid];
    sb2[tid] = b2[tid];
  }
  if (tid < O) sb3[tid] = b3[tid];
  float4 g2[4], g1 = make_float4(0, 0, 0, 0);
  for (int r = 0; r < 4; r++) g2[r] = make_float4(0, 0, 0, 0);
  float g3 = 0, gb = 0, gl = 0, gm = 0;
  for (int c0 = blockIdx.x * kChunk; c0 < n; c0 += gridDim.x * kChunk) {
    const bool live = c0 + i < n;  // rows past the batch hold zeros throughout
    // kChunk * kMlpIn = 256: one input per thread
    sx[tid] = c0 + tid / I < n ? x[(size_t)c0 * I + tid] : 0.0f;
    __syncthreads();
    const float4 zero = make_float4(0, 0, 0, 0);
    float4 h = row4<I>(ld4(sb1 + j0), sx + i * I, sW1, H, j0);
    h = make_float4(fmaxf(h.x, 0.0f), fmaxf(h.y, 0.0f), fmaxf(h.z, 0.0f), fmaxf(h.w, 0.0f));
    st4(sh1 + i * H + j0, live ? h : zero);
    __syncthreads();
    h = row4<H>(ld4(sb2 + j0), sh1 + i * H, sW2, H, j0);
    h = make_float4(fmaxf(h.x, 0.0f), fmaxf(h.y, 0.0f), fmaxf(h.z, 0.0f), fmaxf(h.w, 0.0f));
    st4(sh2 + i * H + j0, live ? h : zero);
    __syncthreads();
    // output o of sample i: four lanes take a quarter of the hidden units each
    {
      const int o = (tid >> 2) & 3, q = tid & 3;
      float a = 0.0f;
      for (int k = q; k < H; k += 4) a = fmaf(sh2[i * H + k], sW3[k * O + o], a);
      a += __shfl_xor(a, 1);
      a += __shfl_xor(a, 2);
      if (q == 0) {
        a += sb3[o];
        float dy = 0.0f;
        if (live) {
          const size_t at = (size_t)(c0 + i) * O + o;
          if (STEP) {
            const float e = a - t[at], w = m[at];
            gl += w * e * e;
            gm += w;
            dy = 2.0f * w * e;  // divided by the mask sum in k_mlp_reduce
          } else {
            y[at] = a;
          }
        }
        if (STEP) sdy[i * O + o] = dy;
      }
    }
    __syncthreads();
    if (!STEP) continue;
    const float4 dy = ld4(sdy + i * O);
    float4 d;
    float *dp = &d.x;
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const float4 w = ld4(sW3 + (j0 + r) * O);
      const float a = fmaf(dy.w, w.w, fmaf(dy.z, w.z, fmaf(dy.y, w.y, dy.x * w.x)));
      dp[r] = sh2[i * H + j0 + r] > 0.0f ? a : 0.0f;
    }
    st4(sd2 + i * H + j0, d);
    __syncthreads();
    d = row4<H>(zero, sd2 + i * H, sW2t, kW2T, j0);
#pragma unroll
    for (int r = 0; r < 4; r++)
      if (!(sh1[i * H + j0 + r] > 0.0f)) dp[r] = 0.0f;
    st4(sd1 + i * H + j0, d);
    __syncthreads();
    const int k0 = 4 * i;  // the thread's rows of W2
#pragma unroll 4
    for (int s = 0; s < kChunk; s++) {
      const float4 a = ld4(sh1 + s * H + k0), e2 = ld4(sd2 + s * H + j0);
      fma4(g2[0], a.x, e2);
      fma4(g2[1], a.y, e2);
      fma4(g2[2], a.z, e2);
      fma4(g2[3], a.w, e2);
      fma4(g1, sx[s * I + i], ld4(sd1 + s * H + j0));
      g3 = fmaf(sh2[s * H + (tid >> 2)], sdy[s * O + (tid & 3)], g3);
    }
    if (tid < H)
      for (int s = 0; s < kChunk; s++) gb += sd1[s * H + tid];
    else if (tid < 2 * H)
      for (int s = 0; s < kChunk; s++) gb += sd2[s * H + tid - H];
    else if (tid < 2 * H + O)
      for (int s = 0; s < kChunk; s++) gb += sdy[s * O + tid - 2 * H];
    __syncthreads();
  }
  if (!STEP) return;
  float *P = part + (size_t)blockIdx.x * kPartStride;
  // single stores: the caller's workspace may be aligned to 4 bytes only
  auto put4 = [](float *p, const float4 &v) {
    p[0] = v.x;
    p[1] = v.y;
    p[2] = v.z;
    p[3] = v.w;
  };
  float *Pb1 = P + I * H, *P2 = Pb1 + H, *Pb2 = P2 + H * H, *P3 = Pb2 + H, *Pb3 = P3 + H * O;
  put4(P + i * H + j0, g1);
#pragma unroll
  for (int r = 0; r < 4; r++) put4(P2 + (4 * i + r) * H + j0, g2[r]);
  P3[tid] = g3;
  if (tid < H) Pb1[tid] = gb;
  else if (tid < 2 * H) Pb2[tid - H] = gb;
  else if (tid < 2 * H + O) Pb3[tid - 2 * H] = gb;
  // loss and mask count over the block, in a fixed order
  for (int d = 1; d < 64; d <<= 1) {
    gl += __shfl_xor(gl, d);
    gm += __shfl_xor(gm, d);
  }
  __syncthreads();
  if ((tid & 63) == 0) {
    sx[tid >> 6] = gl;
    sx[4 + (tid >> 6)] = gm;
  }
  __syncthreads();
  if (tid == 0) {
    P[kMlpParams] = (sx[0] + sx[1]) + (sx[2] + sx[3]);
    P[kMlpParams + 1] = (sx[4] + sx[5]) + (sx[6] + sx[7]);
  }
}

// Adds the blocks' partial gradients in a fixed order and divides by the mask
// sum; ADAM takes the parameter step with the result, otherwise it is written
// to g.  64 parameters x 16 slices of the partial sums per block: 16 loads
// in a row per thread for 250 partial sums (5.6 MB, out of L2).
struct AdamStep {
  float *p, *m1, *m2;
  float lr, b1, b2, eps, c1, c2;
  __device__ void operator()(int q, float gq) const {
    const float a = b1 * m1[q] + (1.0f - b1) * gq;
    const float b = b2 * m2[q] + (1.0f - b2) * gq * gq;
    m1[q] = a;
    m2[q] = b;
    p[q] -= lr * (a / c1) / (sqrtf(b / c2) + eps);
  }
};

template <bool ADAM>
__global__ __launch_bounds__(1024) void k_mlp_reduce(const float *part, int n_part, float *g,
                                                     float *loss, AdamStep adam) {
  constexpr int kSlices = 16;
  __shared__ float s[kSlices][64], sm[kSlices];
  const int q = threadIdx.x & 63, sl = threadIdx.x >> 6, at = blockIdx.x * 64 + q;
  float a = 0.0f, w = 0.0f;
  for (int b = sl; b < n_part; b += kSlices) a += part[(size_t)b * kPartStride + at];
  // the mask sum, by every block: lane q of slice sl takes block sl + 16 q'
  for (int b = sl + kSlices * q; b < n_part; b += kSlices * 64)
    w += part[(size_t)b * kPartStride + kMlpParams + 1];
  for (int d = 1; d < 64; d <<= 1) w += __shfl_xor(w, d);
  s[sl][q] = a;
  if (q == 0) sm[sl] = w;
  __syncthreads();
  if (sl != 0) return;
  float msum = 0.0f;
  a = 0.0f;
#pragma unroll
  for (int k = 0; k < kSlices; k++) {
    a += s[k][q];
    msum += sm[k];
  }
  const float v = a / fmaxf(msum, 1.0f);
  if (at < kMlpParams) {
    if (ADAM) adam(at, v);
    else g[at] = v;
  } else if (at == kMlpParams) {
    *loss = v;
  }
}

__global__ void k_mlp_adam(const float *__restrict__ g, AdamStep adam) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q < kMlpParams) adam(q, g[q]);
}

inline int blocks_for(int n) { return (n + 255) / 256; }

}  // namespace

MlpBuffers mlp_buffers(void *ws, int64_t n) {
  MlpBuffers b;
  float *f = (float *)ws;
  auto take = [&](int64_t count) {
    float *p = f;
    f += (count + 63) / 64 * 64;
    return p;
  };
  b.params = take(kMlpParams);
  b.grad = take(kMlpParams);
  b.m1 = take(kMlpParams);
  b.m2 = take(kMlpParams);
  b.x = take(n * kMlpIn);
  b.t = take(n * kMlpOut);
  b.m = take(n * kMlpOut);
  b.y = take(n * kMlpOut);
  // 388 floats a sample: a partial gradient for every 16 samples and more
  b.part = take(n * (6 * kMlpHidden + kMlpOut));
  b.loss = take(kMlpLosses);
  b.bytes = (size_t)((char *)f - (char *)ws);
  return b;
}

namespace {

// Partial sums of a step: one per block, as many as the activation part of
// the workspace holds (at least one per 16 samples for 15 samples and up); a
// single one sits in the gradient buffer, which k_mlp_reduce turns into the
// gradient element by element.
int step_blocks(const MlpBuffers &b, int n) {
  const int64_t room = (b.loss - b.part) / kPartStride;
  return (int)std::max<int64_t>(1, std::min<int64_t>({(n + kChunk - 1) / kChunk, room, 512}));
}
static_assert(kPartStride <= (kMlpParams + 63) / 64 * 64, "one partial sum fits the gradient buffer");

AdamStep adam_step(const MlpBuffers &b, int step, float lr) {
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  return {b.params, b.m1, b.m2, lr, b1, b2, eps, 1.0f - powf(b1, (float)step),
          1.0f - powf(b2, (float)step)};
}

constexpr int kReduceBlocks = kPartStride / 64;

}  // namespace

hipError_t mlp_forward(const MlpBuffers &b, int n, hipStream_t s) {
  const int nb = std::min((n + kChunk - 1) / kChunk, 1024);
  hipLaunchKernelGGL(k_mlp_pass<false>, dim3(nb), dim3(256), 0, s, b.params, b.x, b.t, b.m, n, b.y,
                     (float *)nullptr);
  return hipGetLastError();
}

hipError_t mlp_loss_grad(const MlpBuffers &b, int n, hipStream_t s) {
  const int nb = step_blocks(b, n);
  float *part = nb > 1 ? b.part : b.grad;
  hipLaunchKernelGGL(k_mlp_pass<true>, dim3(nb), dim3(256), 0, s, b.params, b.x, b.t, b.m, n, b.y,
                     part);
  hipLaunchKernelGGL(k_mlp_reduce<false>, dim3(kReduceBlocks), dim3(1024), 0, s, part, nb, b.grad,
                     b.loss, AdamStep());
  return hipGetLastError();
}

hipError_t mlp_train_step(const MlpBuffers &b, int n, int step, float lr, float *loss,
                          hipStream_t s) {
  const int nb = step_blocks(b, n);
  float *part = nb > 1 ? b.part : b.grad;
  hipLaunchKernelGGL(k_mlp_pass<true>, dim3(nb), dim3(256), 0, s, b.params, b.x, b.t, b.m, n, b.y,
                     part);
  hipLaunchKernelGGL(k_mlp_reduce<true>, dim3(kReduceBlocks), dim3(1024), 0, s, part, nb, b.grad,
                     loss, adam_step(b, step, lr));
  return hipGetLastError();
}

hipError_t mlp_adam(const MlpBuffers &b, int step, float lr, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_adam, dim3(blocks_for(kMlpParams)), dim3(256), 0, s, b.grad,
                     adam_step(b, step, lr));
  return hipGetLastError();
}

}  // namespace qtn
