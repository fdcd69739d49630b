// U-Net layers (Section 4.3) for gfx950, fp32.
//
// 3x3 convolution as an implicit GEMM on the fp32 matrix cores
// (v_mfma_f32_16x16x4_f32): M = output pixels, N = output channels,
// K = 9 taps x input channels.  Activations are NHWC.
//
// Workgroup = 4 wavefronts computing a TH x 16 pixel tile x 32 output
// channels.  Per 16-channel input chunk the (TH+2) x 18 input halo and the
// 9 x 32 x 16 weight slab are staged in LDS once and every tap reads them
// from there.  The gather that fills the halo fuses the zero padding, the
// 2x2 max-pool of the encoder (pooled input mode) and the decoder's nearest
// 2x upsample + skip concatenation (two-source mode), so none of those
// tensors is materialised.  The epilogue adds the bias and applies ReLU.
// Layers with few tiles are split over K and finished by splitk_reduce.  The
// trainer's forward pass and the fp8 calibration run these kernels (their
// ReLU masks and ranges are fp32's own); inference runs conv_split.hip's.
//
// K-slot permutation: MFMA step jj pairs lane group g (= lane / 16) with input
// channel 4g + jj for both operands, so each lane fetches its four channels of
// A and of B with one 16-byte LDS read.
#include "internal.h"
#include "halo_f32.h"
#include "head.h"

namespace lnm {
namespace {

// LDS float of channels 4c .. 4c + 3 of a row (a halo pixel or a weight row)
// with column `col` (the pixel's in the tile, the weight's output channel):
// rows without padding, the quads of every other run of four columns changed
// over in pairs, so that the 16 lanes that one cycle of a 16-byte read serves
// (columns 0-3 and 12-15 of one lane group, 4-11 of the next) lie on distinct
// banks, whichever column they start at.
template <int CK>
__device__ __forceinline__ int lds_at(int row, int col, int c) {
  return row * CK + 4 * (CK == 16 ? c ^ (((col >> 2) & 1) << 1) : c);
}

template <int CK, int MODE, int TH>
__global__ __launch_bounds__(256, 2) void conv3x3_f32(ConvArgs a) {
  constexpr int NF = kBN / 16;
  constexpr int MF = TH / 4;
  // two LDS buffers: the next chunk is fetched into registers while the
  // matrix cores work on the current one
  __shared__ __attribute__((aligned(16))) float s_in[2][(TH + 2) * kHW * CK];
  __shared__ __attribute__((aligned(16))) float s_w[2][9 * kBN * CK];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int tiles_y = (a.H + TH - 1) / TH;
  const int b = blockIdx.y / tiles_y;
  const int y0 = (blockIdx.y - b * tiles_y) * TH, x0 = blockIdx.x * kTW;
  const int nt = blockIdx.z % a.n_tiles, ks = blockIdx.z / a.n_tiles;
  const int nchunks = a.ci_pad / CK;
  const int ch_lo = ks * nchunks / a.splits, ch_hi = (ks + 1) * nchunks / a.splits;
  const float* wblk = static_cast<const float*>(a.w) + (size_t)nt * nchunks * 9 * kBN * CK;
  const int g = lane >> 4, li = lane & 15;
  const int wrow = wave * MF;

  f4 acc[MF][NF];
#pragma unroll
  for (int mf = 0; mf < MF; ++mf)
#pragma unroll
    for (int nf = 0; nf < NF; ++nf) acc[mf][nf] = f4{0.f, 0.f, 0.f, 0.f};

  // per chunk: the (TH+2) x 18 input halo and the weight slab [tap][n][c];
  // every load is unconditional (clamped index), masks apply at commit
  constexpr int NQ = (TH + 2) * kHW * (CK / 4), NW = 9 * kBN * CK / 4;
  constexpr int RQ = (NQ + 255) / 256, RW = (NW + 255) / 256;
  Halo<MODE> rq[RQ];
  f4 rw[RW];
  unsigned ok = 0;
  auto fetch = [&](int ch) {
    ok = 0;
#pragma unroll
    for (int r = 0; r < RQ; ++r) {
      const int q = min(tid + 256 * r, NQ - 1);
      const int c4 = q % (CK / 4), p = q / (CK / 4);
      const int y = y0 + p / kHW - 1, x = x0 + p % kHW - 1;
      const bool in = tid + 256 * r < NQ && y >= 0 && y < a.H && x >= 0 && x < a.W;
      ok |= (unsigned)in << r;
      rq[r] = halo_load<MODE>(a, b, min(max(y, 0), a.H - 1), min(max(x, 0), a.W - 1), ch * CK + 4 * c4);
    }
    const float* wsrc = wblk + (size_t)ch * 9 * kBN * CK;
#pragma unroll
    for (int r = 0; r < RW; ++r) rw[r] = *reinterpret_cast<const f4*>(wsrc + 4 * min(tid + 256 * r, NW - 1));
  };
  auto commit = [&](int buf) {
#pragma unroll
    for (int r = 0; r < RQ; ++r) {
      const int q = tid + 256 * r;
      if (q < NQ)
        *reinterpret_cast<f4*>(&s_in[buf][lds_at<CK>(q / (CK / 4), q / (CK / 4) % kHW, q % (CK / 4))]) =
            halo_value<MODE>(rq[r], (ok >> r) & 1u);
    }
#pragma unroll
    for (int r = 0; r < RW; ++r) {
      const int q = tid + 256 * r;
      if (q < NW) *reinterpret_cast<f4*>(&s_w[buf][lds_at<CK>(q / (CK / 4), q / (CK / 4), q % (CK / 4))]) = rw[r];
    }
  };

  if (ch_lo < ch_hi) {
    fetch(ch_lo);
    commit(0);
  }
  int at_x[3];  // the lane's halo reads, by the tap's column
#pragma unroll
  for (int dx = 0; dx < 3; ++dx)
    at_x[dx] = CK == 16 ? lds_at<CK>(wrow * kHW + li + dx, li + dx, g) : (wrow * kHW + li + dx) * CK + g;
  const int at_w = CK == 16 ? lds_at<CK>(li, li, g) : li * CK + g;
  __syncthreads();
  for (int ch = ch_lo; ch < ch_hi; ++ch) {
    const int cur = (ch - ch_lo) & 1;
    const bool more = ch + 1 < ch_hi;
    if (more) fetch(ch + 1);
    const float* si = s_in[cur];
    const float* sw = s_w[cur];
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      const int dy = tap / 3, dx = tap - 3 * (tap / 3);
      if constexpr (CK == 16) {
        f4 av[MF], bv[NF];
#pragma unroll
        for (int mf = 0; mf < MF; ++mf)
          av[mf] = *reinterpret_cast<const f4*>(&si[at_x[dx] + (mf + dy) * kHW * CK]);
#pragma unroll
        for (int nf = 0; nf < NF; ++nf)
          bv[nf] = *reinterpret_cast<const f4*>(&sw[at_w + (tap * kBN + nf * 16) * CK]);
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
#pragma unroll
          for (int mf = 0; mf < MF; ++mf)
#pragma unroll
            for (int nf = 0; nf < NF; ++nf)
              acc[mf][nf] = __builtin_amdgcn_mfma_f32_16x16x4f32(bv[nf][jj], av[mf][jj], acc[mf][nf], 0, 0, 0);
      } else {
        float av[MF], bv[NF];
#pragma unroll
        for (int mf = 0; mf < MF; ++mf) av[mf] = si[at_x[dx] + (mf + dy) * kHW * CK];
#pragma unroll
        for (int nf = 0; nf < NF; ++nf) bv[nf] = sw[at_w + (tap * kBN + nf * 16) * CK];
#pragma unroll
        for (int mf = 0; mf < MF; ++mf)
#pragma unroll
          for (int nf = 0; nf < NF; ++nf)
            acc[mf][nf] = __builtin_amdgcn_mfma_f32_16x16x4f32(bv[nf], av[mf], acc[mf][nf], 0, 0, 0);
      }
    }
    if (more) commit(cur ^ 1);
    __syncthreads();
  }

  // epilogue: the product is taken transposed, so the lane holds channels
  // 4g .. 4g + 3 of each 16-channel block at pixel li; the biases are loaded
  // ahead of the stores (a load after a store waits for it).  The stores are
  // non-temporal (the next layer reads the tensor from another XCD, so keeping
  // it in this XCD's L2 only adds to the write-back at the end of the kernel)
  f4 bias[NF];
  if (a.splits == 1) {
#pragma unroll
    for (int nf = 0; nf < NF; ++nf) bias[nf] = *reinterpret_cast<const f4*>(a.bias + nt * kBN + nf * 16 + 4 * g);
  }
  const int x = x0 + li;
  if (x >= a.W) return;
  const size_t row = (size_t)a.W * a.co;
  float* to = (a.splits > 1 ? a.partial + (size_t)ks * a.B * a.H * row : static_cast<float*>(a.out)) +
              ((size_t)(b * a.H + y0 + wrow) * a.W + x) * a.co + nt * kBN + 4 * g;
#pragma unroll
  for (int mf = 0; mf < MF; ++mf) {
    if (y0 + wrow + mf >= a.H) break;
#pragma unroll
    for (int nf = 0; nf < NF; ++nf) {
      if (nt * kBN + nf * 16 >= a.co) continue;  // the channel count is a multiple of 16
      f4 v = acc[mf][nf];
      if (a.splits == 1) {
        v += bias[nf];
        if (a.relu) {
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = fmaxf(v[r], 0.0f);
        }
      }
      __builtin_nontemporal_store(v, reinterpret_cast<f4*>(to + mf * row + nf * 16));
    }
  }
}

__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// Finish a split-K layer: sum the splits in order, then the layer epilogue.
// One lane per four consecutive output elements (channels of one pixel: the
// channel count is a multiple of 16); the S partial loads are issued before
// the in-order sum.
template <int S>
__global__ __launch_bounds__(256) void splitk_reduce(ConvArgs a, int out_type, long total4) {
  const long i4 = (long)blockIdx.x * 256 + threadIdx.x;
  if (i4 >= total4) return;
  const size_t total = (size_t)total4 * 4;
  f4 v[S];
#pragma unroll
  for (int k = 0; k < S; ++k) v[k] = *reinterpret_cast<const f4*>(a.partial + k * total + 4 * i4);
  const int n0 = (int)((4 * i4) % a.co);
  float y[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float acc = 0.0f;
#pragma unroll
    for (int k = 0; k < S; ++k) acc += v[k][e];
    const int n = n0 + e;
    if (out_type == 2) {
      float t = a.in_scale * a.w_scale[n] * acc + a.bias[n];
      t = t > 0.0f ? t * a.out_inv_scale : 0.0f;
      y[e] = fminf(t, 448.0f);
    } else if (out_type == 3) {
      y[e] = fmaxf(a.in_scale * a.w_scale[n] * acc + a.bias[n], 0.0f);
    } else {
      float t = acc + a.bias[n];
      if (a.relu) t = fmaxf(t, 0.0f);
      y[e] = t;
    }
  }
  if (out_type == 2) {
    uint32_t packed = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      packed |= ((uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(y[e], 0.0f, 0, false) & 0xffu) << (8 * e);
    static_cast<uint32_t*>(a.out)[i4] = packed;
  } else if (out_type == 1 || out_type == 3) {
    static_cast<uint2*>(a.out)[i4] = make_uint2((uint32_t)f32_to_bf16(y[0]) | ((uint32_t)f32_to_bf16(y[1]) << 16),
                                                (uint32_t)f32_to_bf16(y[2]) | ((uint32_t)f32_to_bf16(y[3]) << 16));
  } else {
    static_cast<f4*>(a.out)[i4] = f4{y[0], y[1], y[2], y[3]};
  }
}

// 1x1 head C -> 6 and sigmoid, one lane per pixel; fp32 arithmetic on fp32
// (IN = 0), bf16 (IN = 1) or e4m3 (IN = 2) activations.  With COMP the
// pixel is also shaded from the lightmap values it just stored (the frame's
// head and composite in one launch; same values as the separate kernels).
template <int IN, bool COMP>
__global__ __launch_bounds__(256) void head_kernel(HeadArgs a, CompositeArgs comp) {
  __shared__ float sw[6 * 256];
  __shared__ float sb[6];
  for (int q = threadIdx.x; q < 6 * a.C; q += 256) sw[q] = a.w[q];
  if (threadIdx.x < 6) sb[threadIdx.x] = a.b[threadIdx.x];
  __syncthreads();
  const int p = blockIdx.x * 256 + threadIdx.x;
  if (p >= a.P) return;
  float z[6];
#pragma unroll
  for (int o = 0; o < 6; ++o) z[o] = sb[o];
  for (int c = 0; c < a.C; c += 4) {
    f4 v;
    if constexpr (IN == 0) {
      v = *reinterpret_cast<const f4*>(static_cast<const float*>(a.in) + (size_t)p * a.C + c);
    } else if constexpr (IN == 2) {
      const int q = *reinterpret_cast<const int*>(static_cast<const uint8_t*>(a.in) + (size_t)p * a.C + c);
      v = f4{__builtin_amdgcn_cvt_f32_fp8(q, 0), __builtin_amdgcn_cvt_f32_fp8(q, 1),
             __builtin_amdgcn_cvt_f32_fp8(q, 2), __builtin_amdgcn_cvt_f32_fp8(q, 3)} *
          a.in_scale;
    } else {
      const uint2 q = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(a.in) + (size_t)p * a.C + c);
      v = f4{bf16_to_f32(q.x & 0xffff), bf16_to_f32(q.x >> 16), bf16_to_f32(q.y & 0xffff), bf16_to_f32(q.y >> 16)};
    }
#pragma unroll
    for (int o = 0; o < 6; ++o) {
      const float* w = sw + o * a.C + c;
      z[o] += w[0] * v.x + w[1] * v.y + w[2] * v.z + w[3] * v.w;
    }
  }
  float L[6];
#pragma unroll
  for (int o = 0; o < 6; ++o) {
    if (a.logits) a.logits[(size_t)p * 6 + o] = z[o];
    L[o] = 1.0f / (1.0f + expf(-z[o]));
    a.lm[(size_t)p * 6 + o] = L[o];
  }
  if constexpr (COMP) shade_pixel(comp, p, L);
}

// Six-way shading of stored lightmaps.
__global__ __launch_bounds__(256) void composite_kernel(CompositeArgs a) {
  const int p = blockIdx.x * 256 + threadIdx.x;
  if (p >= a.P) return;
  float L[6];
#pragma unroll
  for (int q = 0; q < 6; ++q) L[q] = a.lm[(size_t)p * 6 + q];
  shade_pixel(a, p, L);
}

// Six-way shading of a batch of images with per-image lights.
__global__ __launch_bounds__(256) void composite_batch_kernel(CompositeBatchArgs a) {
  const long p = (long)blockIdx.x * 256 + threadIdx.x;
  if (p >= (long)a.P * a.B) return;
  const int b = (int)(p / a.P);
  float L[6];
#pragma unroll
  for (int q = 0; q < 6; ++q) L[q] = a.lm[(size_t)p * 6 + q];
  shade_lights(a.l, a.rgb, a.light_lo[b], a.light_lo[b + 1], a.guide, a.rgba, (size_t)p, L);
}

template <int CK, int MODE, int TH>
hipError_t launch_th(const ConvArgs& a, hipStream_t s) {
  const dim3 grid((a.W + kTW - 1) / kTW, ((a.H + TH - 1) / TH) * a.B, a.n_tiles * a.splits);
  hipLaunchKernelGGL((conv3x3_f32<CK, MODE, TH>), grid, dim3(256), 0, s, a);
  return hipGetLastError();
}
// The tile height changes no sum: the tallest whose workgroups still number two
// per CU (all that 16-row tiles' LDS allows), over the whole batch; else the
// layer's own.  A training step of 8 x 256^2 (4 levels, base 32) took 3741 us
// with at most 8 rows, 3683 with 16; 3999 before with padded LDS rows (two
// cycles per read for conflicts) and epilogues whose bias loads waited for
// the stores of four bytes per lane before them.  The large layers now run at
// 114 TFLOP/s, 73% of the instruction's rate.
template <int MODE>
hipError_t launch_rows(const ConvArgs& a, hipStream_t s) {
  auto wgs = [&](int th) {
    return (long)((a.W + kTW - 1) / kTW) * ((a.H + th - 1) / th) * a.B * a.n_tiles * a.splits;
  };
  if (wgs(16) >= 512 && rows_fit(a.H, 16)) return launch_th<16, MODE, 16>(a, s);
  return a.th == 4 && (wgs(8) < 512 || !rows_fit(a.H, 8)) ? launch_th<16, MODE, 4>(a, s) : launch_th<16, MODE, 8>(a, s);
}

}  // namespace

hipError_t launch_conv3x3_f32(int mode, int ck, const ConvArgs& a, hipStream_t s, const HeadFuse* head) {
  if (a.co % 16) return hipErrorInvalidValue;
  if (mode == G_GUIDE && ck == 4 && !head) return launch_th<4, G_GUIDE, 8>(a, s);
  if (ck != 16) return hipErrorInvalidValue;
  if (a.split) return launch_conv3x3_split(mode, a, s, head);
  if (head) return hipErrorInvalidValue;
  switch (mode) {
    case G_PLAIN: return launch_rows<G_PLAIN>(a, s);
    case G_POOL: return launch_rows<G_POOL>(a, s);
    case G_CONCAT_UP: return launch_rows<G_CONCAT_UP>(a, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_splitk_reduce(const ConvArgs& a, int out_type, hipStream_t s) {
  if (a.co % 4) return hipErrorInvalidValue;
  const long total4 = (long)a.B * a.H * a.W * a.co / 4;
  const dim3 grid((unsigned)((total4 + 255) / 256));
  switch (a.splits) {
    case 2: hipLaunchKernelGGL(splitk_reduce<2>, grid, dim3(256), 0, s, a, out_type, total4); break;
    case 4: hipLaunchKernelGGL(splitk_reduce<4>, grid, dim3(256), 0, s, a, out_type, total4); break;
    case 8: hipLaunchKernelGGL(splitk_reduce<8>, grid, dim3(256), 0, s, a, out_type, total4); break;
    case 16: hipLaunchKernelGGL(splitk_reduce<16>, grid, dim3(256), 0, s, a, out_type, total4); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_head(const HeadArgs& a, hipStream_t s, const CompositeArgs* comp) {
  if (a.C > 256 || (a.C & 3) || a.in_type < 0 || a.in_type > 2) return hipErrorInvalidValue;
  const dim3 grid((a.P + 255) / 256);
  const CompositeArgs c = comp ? *comp : CompositeArgs{};
  if (comp) {
    if (a.in_type == 0) hipLaunchKernelGGL((head_kernel<0, true>), grid, dim3(256), 0, s, a, c);
    if (a.in_type == 1) hipLaunchKernelGGL((head_kernel<1, true>), grid, dim3(256), 0, s, a, c);
    if (a.in_type == 2) hipLaunchKernelGGL((head_kernel<2, true>), grid, dim3(256), 0, s, a, c);
  } else {
    if (a.in_type == 0) hipLaunchKernelGGL((head_kernel<0, false>), grid, dim3(256), 0, s, a, c);
    if (a.in_type == 1) hipLaunchKernelGGL((head_kernel<1, false>), grid, dim3(256), 0, s, a, c);
    if (a.in_type == 2) hipLaunchKernelGGL((head_kernel<2, false>), grid, dim3(256), 0, s, a, c);
  }
  return hipGetLastError();
}

hipError_t launch_composite(const CompositeArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(composite_kernel, dim3((a.P + 255) / 256), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_composite_batch(const CompositeBatchArgs& a, hipStream_t s) {
  const long n = (long)a.P * a.B;
  hipLaunchKernelGGL(composite_batch_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace lnm
