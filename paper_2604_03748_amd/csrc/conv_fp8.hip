// U-Net 3x3 convolutions (Section 4.3) in FP8 e4m3 (OCP) on the gfx950
// matrix cores (v_mfma_f32_16x16x32_fp8_fp8, fp32 accumulation).
//
// Quantisation: weights per output channel, q_w = rne(W / s_w[o]) with
// s_w[o] = max|W[o]| / 448; activations per stored tensor, q = rne(y / s_t)
// saturated to 448.  A layer computes y = s_in s_w[o] sum q_in q_w + b,
// applies ReLU and stores rne(y / s_out) for its consumers.  The two inputs
// of a decoder concatenation share one scale, so the K-sum factors.  The
// 3-channel input layer runs in bf16 within the second layer's launch.
#include "conv_low.h"
#include "internal.h"

namespace lnm {
namespace {

// Per-block maximum of |x| over a fixed range, then the maximum of those.
__global__ __launch_bounds__(256) void amax_partial(const float* __restrict__ x, long n, float* __restrict__ part) {
  __shared__ float sh[256];
  const long per = (n + gridDim.x - 1) / gridDim.x;
  const long lo = (long)blockIdx.x * per, hi = min(n, lo + per);
  float m = 0.0f;
  for (long i = lo + threadIdx.x; i < hi; i += 256) m = fmaxf(m, fabsf(x[i]));
  sh[threadIdx.x] = m;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) sh[threadIdx.x] = fmaxf(sh[threadIdx.x], sh[threadIdx.x + s]);
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

__global__ __launch_bounds__(256) void amax_finish(const float* __restrict__ part, int n, float* __restrict__ out) {
  __shared__ float sh[256];
  float m = 0.0f;
  for (int i = threadIdx.x; i < n; i += 256) m = fmaxf(m, part[i]);
  sh[threadIdx.x] = m;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) sh[threadIdx.x] = fmaxf(sh[threadIdx.x], sh[threadIdx.x + s]);
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = sh[0];
}

}  // namespace

hipError_t launch_conv3x3_fp8(int mode, const ConvArgs& a, hipStream_t s, const HeadFuse* head) {
  if (!a.w_scale) return hipErrorInvalidValue;
  return low::launch<low::Fp8>(mode, a, s, head);
}

hipError_t launch_amax(const float* x, long n, float* partial, float* out, hipStream_t s) {
  hipLaunchKernelGGL(amax_partial, dim3(kAmaxBlocks), dim3(256), 0, s, x, n, partial);
  hipLaunchKernelGGL(amax_finish, dim3(1), dim3(256), 0, s, partial, kAmaxBlocks, out);
  return hipGetLastError();
}

}  // namespace lnm
