// Backward-pass and optimiser kernels for training the fp32 U-Net on the GPU
// (Section 4.4 pixel loss in sRGB space, Section 5 Adam).  Every reduction
// has a fixed assignment of terms to lanes and blocks and a fixed combination
// order, so a gradient does not depend on scheduling.
#include "internal.h"

namespace lnm {
namespace {

// Block-wide sum in a fixed tree order (256 lanes).
__device__ __forceinline__ float block_sum(float v, float* sh) {
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
    __syncthreads();
  }
  const float r = sh[0];
  __syncthreads();
  return r;
}

// e = y - t; dz = 2 e y (1 - y) / n (mean-squared error through the sigmoid);
// partial[block] = sum of e^2 over the block's fixed element range.
__global__ __launch_bounds__(256) void loss_kernel(const float* __restrict__ y, const float* __restrict__ t,
                                                    float* __restrict__ dz, float* __restrict__ partial, long n) {
  __shared__ float sh[256];
  const float scale = 2.0f / (float)n;
  const long per = (n + gridDim.x - 1) / gridDim.x;
  const long lo = (long)blockIdx.x * per, hi = min(n, lo + per);
  float acc = 0.0f;
  for (long i = lo + threadIdx.x; i < hi; i += 256) {
    const float yy = y[i], e = yy - t[i];
    acc += e * e;
    dz[i] = scale * e * yy * (1.0f - yy);
  }
  acc = block_sum(acc, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = acc;
}

__global__ __launch_bounds__(256) void finish_sum(const float* __restrict__ partial, int n, float scale,
                                                   float* __restrict__ out) {
  __shared__ float sh[256];
  float acc = 0.0f;
  for (int i = threadIdx.x; i < n; i += 256) acc += partial[i];
  acc = block_sum(acc, sh);
  if (threadIdx.x == 0) *out = acc * scale;
}

// Head (1x1, C -> 6) backward in one pass over its input X: the data gradient
// with X's ReLU mask, E[p][c] = (sum_o W[o][c] dz[p][o]) * (X[p][c] > 0), and
// the weight and bias sums dz^T X of the block's pixels.  A block takes one
// contiguous run of pixels, 256 / C of them at a time with one lane per
// channel; partial[block][6 C + 6] is added up by head_bwd_finish.
// Bound by memory (X read, E written once): 8 x 256^2, C = 32 takes 40
// us against 769 us with a pass of its own over X per weight.
__global__ __launch_bounds__(256) void head_bwd(const float* __restrict__ dz, const float* __restrict__ w,
                                                const float* __restrict__ x, long P, int C, float* __restrict__ e,
                                                float* __restrict__ partial) {
  extern __shared__ float sh[];  // [256 / C][6 C + 6]
  const int subs = 256 / C, sub = threadIdx.x / C, c = threadIdx.x - sub * C, n = 6 * C + 6;
  const long per = (P + gridDim.x - 1) / gridDim.x;
  const long lo = (long)blockIdx.x * per, hi = min(P, lo + per);
  if (sub < subs) {
    float wc[6], gw[6], gb[6];
#pragma unroll
    for (int o = 0; o < 6; ++o) {
      wc[o] = w[o * C + c];
      gw[o] = gb[o] = 0.0f;
    }
#pragma unroll 2
    for (long p = lo + sub; p < hi; p += subs) {
      const float2* q = reinterpret_cast<const float2*>(dz + p * 6);
      const float2 d0 = q[0], d1 = q[1], d2 = q[2];
      const float d[6] = {d0.x, d0.y, d1.x, d1.y, d2.x, d2.y};
      const float xv = x[p * C + c];
      float s = 0.0f;
#pragma unroll
      for (int o = 0; o < 6; ++o) {
        s += wc[o] * d[o];
        gw[o] += d[o] * xv;
        gb[o] += d[o];
      }
      e[p * C + c] = xv > 0.0f ? s : 0.0f;
    }
#pragma unroll
    for (int o = 0; o < 6; ++o) {
      sh[sub * n + o * C + c] = gw[o];
      if (c == 0) sh[sub * n + 6 * C + o] = gb[o];
    }
  }
  __syncthreads();
  for (int q = threadIdx.x; q < n; q += 256) {
    float v = 0.0f;
    for (int k = 0; k < subs; ++k) v += sh[k * n + q];
    partial[(size_t)blockIdx.x * n + q] = v;
  }
}

// Sums over the blocks of head_bwd: eight lanes per sum, then in order.
__global__ __launch_bounds__(256) void head_bwd_finish(const float* __restrict__ partial, int blocks, int C,
                                                       float* __restrict__ gw, float* __restrict__ gb) {
  __shared__ float sh[8][32];
  const int el = threadIdx.x & 31, rl = threadIdx.x >> 5, n = 6 * C + 6, q = blockIdx.x * 32 + el;
  float v = 0.0f;
  if (q < n) {
#pragma unroll 8
    for (int k = rl; k < blocks; k += 8) v += partial[(size_t)k * n + q];
  }
  sh[rl][el] = v;
  __syncthreads();
  if (rl || q >= n) return;
#pragma unroll
  for (int k = 1; k < 8; ++k) v += sh[k][el];
  if (q < 6 * C)
    gw[q] = v;
  else
    gb[q - 6 * C] = v;
}

__global__ __launch_bounds__(256) void adam_kernel(float* __restrict__ p, const float* __restrict__ g,
                                                    float* __restrict__ m, float* __restrict__ v, long n, float lr,
                                                    float b1, float b2, float eps, float c1, float c2) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.0f - b1) * gi;
  const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// Packed fp32 layout [n_tile][chunk][tap][n (32)][c (ck)] from flat
// W[co][ci][3][3].  dgrad = 1: the layout of the convolution that propagates
// gradients, whose input channels are the layer's outputs and whose output
// channels are the layer's inputs, taps mirrored (8 - tap).
__global__ __launch_bounds__(256) void pack_f32(const float* __restrict__ w, const float* __restrict__ bsrc,
                                                 LayerDesc d, int dgrad, float* __restrict__ dst,
                                                 float* __restrict__ bdst, int src_ci, int src_co) {
  const long total = (long)d.co_pad * d.ci_pad * 9;
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i < total) {
    const int cc = i % d.ck;
    long r = i / d.ck;
    const int n = r % kBN;
    r /= kBN;
    const int tap = r % 9;
    r /= 9;
    const int nch = d.ci_pad / d.ck;
    const int ch = r % nch, t = r / nch;
    const int oc = t * kBN + n, ic = ch * d.ck + cc;  // output / input channel of this convolution
    float v = 0.0f;
    if (oc < d.co && ic < d.ci) {
      if (dgrad)
        v = w[((size_t)ic * src_ci + oc) * 9 + (8 - tap)];
      else
        v = w[((size_t)oc * src_ci + ic) * 9 + tap];
    }
    dst[i] = v;
  }
  if (bdst && i < d.co_pad) bdst[i] = (!dgrad && i < d.co) ? bsrc[i] : 0.0f;
  (void)src_co;
}

}  // namespace

hipError_t launch_loss(const float* y, const float* t, float* dz, float* partial, long n, float* loss, hipStream_t s) {
  hipLaunchKernelGGL(loss_kernel, dim3(kLossBlocks), dim3(256), 0, s, y, t, dz, partial, n);
  hipLaunchKernelGGL(finish_sum, dim3(1), dim3(256), 0, s, partial, kLossBlocks, 1.0f / (float)n, loss);
  return hipGetLastError();
}

hipError_t launch_head_bwd(const float* dz, const float* w, const float* x, long P, int C, float* e_out,
                           float* grad_w, float* grad_b, float* partial, hipStream_t s) {
  if (C < 1 || C > 256) return hipErrorInvalidValue;
  const int blocks = (int)std::min<long>(kHeadBwdBlocks, (P + 63) / 64), n = 6 * C + 6;
  hipLaunchKernelGGL(head_bwd, dim3(blocks), dim3(256), sizeof(float) * (256 / C) * n, s, dz, w, x, P, C, e_out,
                     partial);
  hipLaunchKernelGGL(head_bwd_finish, dim3((n + 31) / 32), dim3(256), 0, s, partial, blocks, C, grad_w, grad_b);
  return hipGetLastError();
}

hipError_t launch_adam(float* p, const float* g, float* m, float* v, long n, float lr, float b1, float b2, float eps,
                       int t, hipStream_t s) {
  const float c1 = (float)(1.0 - std::pow((double)b1, t)), c2 = (float)(1.0 - std::pow((double)b2, t));
  hipLaunchKernelGGL(adam_kernel, dim3((n + 255) / 256), dim3(256), 0, s, p, g, m, v, n, lr, b1, b2, eps, c1, c2);
  return hipGetLastError();
}

hipError_t launch_pack_f32(const float* flat_w, const float* flat_b, const LayerDesc& d, int dgrad, char* dst,
                           size_t w_off, size_t b_off, hipStream_t s) {
  // src_ci: input channels of the original layer (row length of flat W)
  const int src_ci = dgrad ? d.co : d.ci;
  const long total = (long)d.co_pad * d.ci_pad * 9;
  const long n = std::max<long>(total, d.co_pad);
  hipLaunchKernelGGL(pack_f32, dim3((n + 255) / 256), dim3(256), 0, s, flat_w, flat_b, d, dgrad,
                     reinterpret_cast<float*>(dst + w_off), dgrad ? nullptr : reinterpret_cast<float*>(dst + b_off),
                     src_ci, 0);
  return hipGetLastError();
}

}  // namespace lnm
