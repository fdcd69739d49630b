// The 3x3 convolution kernel of the bf16 and fp8 networks (device code only):
// an implicit GEMM on the 16 x 16 x 32 matrix instructions, fp32 accumulation.
//
// A workgroup of four wavefronts computes a 4 MF x 16 pixel tile x 16 NF
// output channels.  Per 32-channel input chunk the (4 MF + 2) x 18 halo and
// the 9 x 16 NF x 32 weight slab are staged in LDS and read by all nine taps,
// the next chunk's values being in registers meanwhile; the halo gather fuses
// zero padding, 2x2 max-pooling and the decoder's upsample + concatenation.
// The product is taken transposed (output channels as MFMA rows): a lane ends
// with four consecutive channels of one pixel, stored as one vector.
//
// Lane group g (= lane / 16) supplies input channels 8g .. 8g + 7 of the chunk
// to both operands.  Every output is summed over the chunks, taps and MFMA
// steps in that order whatever the tile, so all tiles give the same values
// bit for bit.  A layer whose sums are split over K (conv_layer_tiling) may
// run its `seq` splits one after the other in one workgroup, which adds them
// up as splitk_reduce does.
//
// Measured against tiles of at most 8 rows x 64 channels that recomputed
// their addresses per chunk (9 lane operations per MFMA): 16 x 256^2 on the
// 4-level base-32 bf16 network 1243 -> 519 us (655 TFLOP/s), the convolutions
// of a 1024^2 frame on the base-48 network 1680 -> 940 us, of a 512^2 fp8
// frame 250 -> 180 us.  The matrix cores are busy for about 40% of the large
// layers' time, LDS for 20%, vector instructions for 25%.
//
// The element type T gives: bytes per element ES, LDS bytes per row of 32
// channels kRow, the 8-channel group type Group, the MFMA, the maximum of
// non-negative groups, and the stored form of four outputs.
#pragma once
#include <type_traits>

#include "first_layer.h"
#include "head.h"
#include "internal.h"

namespace lnm {
namespace low {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
// native vectors: arrays of these stay in registers (arrays of HIP's structs
// are copied member-wise through memory and were kept in scratch)
typedef unsigned int u2 __attribute__((ext_vector_type(2)));
typedef unsigned int u4 __attribute__((ext_vector_type(4)));
typedef short s2 __attribute__((ext_vector_type(2)));

constexpr int kTW = 16, kHW = kTW + 2, kCK = 32;

__device__ __forceinline__ uint32_t pk_bf16(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{a, b}, bf16x2));
}
__device__ __forceinline__ uint32_t max_i16x2(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s2, a), __builtin_bit_cast(s2, b)));
}

// Lane rows (16 lanes) 0 .. 3 hold a word of quads 0 .. 3 of one 16-channel
// block in p and of the next block in q.  Afterwards row 0 holds p's quads 0
// and 1, row 2 its quads 2 and 3, row 1 q's quads 0 and 1, row 3 its quads 2
// and 3: eight consecutive channels in every lane.
__device__ __forceinline__ u2 join_quads(uint32_t p, uint32_t q) {
  const auto r = __builtin_amdgcn_permlane16_swap(p, q, false, false);
  return u2{r[0], r[1]};
}
__device__ __forceinline__ u4 join_quads(u2 p, u2 q) {
  const u2 x = join_quads(p.x, q.x), y = join_quads(p.y, q.y);
  return u4{x.x, y.x, x.y, y.y};
}

// The element type T: T::store(a, each) calls each(a.out, f) with f turning
// four channels' values into what is stored.
struct Bf16 {
  static constexpr int ES = 2, kRow = 64;
  typedef u4 Group;
  typedef bf16x8 Frag;
  static __device__ __forceinline__ f4 mfma(Frag w, Frag x, f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, x, c, 0, 0, 0);
  }
  // ReLU outputs are not negative (a -0 counts as less than everything), so
  // their bf16 bits order like signed 16-bit numbers
  static __device__ __forceinline__ Group max4(const Group (&v)[4]) {
    Group r;
#pragma unroll
    for (int k = 0; k < 4; ++k) r[k] = max_i16x2(max_i16x2(v[0][k], v[1][k]), max_i16x2(v[2][k], v[3][k]));
    return r;
  }
  // first layer's outputs as stored: ReLU, one rounding
  typedef u2 Quad;
  static __device__ __forceinline__ Quad first(const ConvArgs&, f4 v) {
    return u2{pk_bf16(fmaxf(v.x, 0.0f), fmaxf(v.y, 0.0f)), pk_bf16(fmaxf(v.z, 0.0f), fmaxf(v.w, 0.0f))};
  }
  // epilogue: what four channels' sums need, loaded before any store (a load
  // after a store would wait for it), and the value
  struct Scale {
    f4 bias;
  };
  static __device__ __forceinline__ Scale scale(const ConvArgs& a, int n) {
    return {*reinterpret_cast<const f4*>(a.bias + n)};
  }
  static __device__ __forceinline__ f4 scaled(const ConvArgs&, f4 acc, const Scale& s) { return acc + s.bias; }
  template <class F>
  static __device__ __forceinline__ void store(const ConvArgs& a, const F& each) {
    each(static_cast<uint16_t*>(a.out), [&](f4 v) {
      if (a.relu) {
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = fmaxf(v[r], 0.0f);
      }
      return u2{pk_bf16(v.x, v.y), pk_bf16(v.z, v.w)};
    });
  }
};

struct Fp8 {
  static constexpr int ES = 1, kRow = 40;
  typedef u2 Group;
  typedef long Frag;
  static __device__ __forceinline__ f4 mfma(Frag w, Frag x, f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(w, x, c, 0, 0, 0);
  }
  // stored activations are ReLU outputs (+0 encoded as 0): their e4m3 bytes
  // order like unsigned numbers; even and odd bytes as 16-bit pairs
  static __device__ __forceinline__ Group max4(const Group (&v)[4]) {
    Group r;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      uint32_t lo = v[0][k] & 0x00ff00ffu, hi = (v[0][k] >> 8) & 0x00ff00ffu;
#pragma unroll
      for (int q = 1; q < 4; ++q) {
        lo = max_i16x2(lo, v[q][k] & 0x00ff00ffu);
        hi = max_i16x2(hi, (v[q][k] >> 8) & 0x00ff00ffu);
      }
      r[k] = lo | (hi << 8);
    }
    return r;
  }
  // e4m3 of four values, round to nearest even, saturating at +-448
  static __device__ __forceinline__ uint32_t e4m3(f4 v) {
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = fminf(fmaxf(v[r], -448.0f), 448.0f);
    int p = __builtin_amdgcn_cvt_pk_fp8_f32(v.x, v.y, 0, false);
    p = __builtin_amdgcn_cvt_pk_fp8_f32(v.z, v.w, p, true);
    return (uint32_t)p;
  }
  static __device__ __forceinline__ uint32_t relu_e4m3(f4 v, float inv_scale) {
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = v[r] > 0.0f ? v[r] * inv_scale : 0.0f;
    return e4m3(v);
  }
  typedef uint32_t Quad;
  static __device__ __forceinline__ Quad first(const ConvArgs& a, f4 v) { return relu_e4m3(v, a.w0_out_inv); }
  struct Scale {
    f4 w, bias;
  };
  static __device__ __forceinline__ Scale scale(const ConvArgs& a, int n) {
    return {*reinterpret_cast<const f4*>(a.w_scale + n), *reinterpret_cast<const f4*>(a.bias + n)};
  }
  static __device__ __forceinline__ f4 scaled(const ConvArgs& a, f4 acc, const Scale& s) {
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[r] = a.in_scale * s.w[r] * acc[r] + s.bias[r];
    return acc;
  }
  template <class F>
  static __device__ __forceinline__ void store(const ConvArgs& a, const F& each) {
    if (a.out_bf16)  // for a bf16 consumer: unscaled
      each(static_cast<uint16_t*>(a.out), [&](f4 v) {
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = fmaxf(v[r], 0.0f);
        return u2{pk_bf16(v.x, v.y), pk_bf16(v.z, v.w)};
      });
    else
      each(static_cast<uint8_t*>(a.out), [&](f4 v) { return relu_e4m3(v, a.out_inv_scale); });
  }
};

// First layer (bf16 in both networks: K slot k = 9 dy + 3 dx + channel of the
// 3x3 window, k < 27; packed weights [n-tile][n (32)][k (32)]): the guide over
// the tile and a two-pixel border, rounded to bf16 once per value, in rows of
// 20 pixels x 3 channels, zero outside the image.
constexpr int kGuideRow = 64;  // bf16 per staged guide row (60 used)
template <int TH>
__device__ __forceinline__ void stage_guide_bf16(const ConvArgs& a, int b, int y0, int x0, uint16_t* s_g) {
  const float* gs = static_cast<const float*>(a.src0);
  for (int q = threadIdx.x; q < (TH + 4) * 60; q += 256) {
    const int r = q / 60, e = q - 60 * r, y = y0 + r - 2, x = x0 + e / 3 - 2;
    const bool in = y >= 0 && y < a.H && x >= 0 && x < a.W;
    const float v = gs[in ? ((size_t)(b * a.H + y) * a.W + x) * 3 + e % 3 : 0];
    s_g[r * kGuideRow + e] = (uint16_t)pk_bf16(in ? v : 0.0f, 0.0f);
  }
}

// LDS byte of 8-channel group c of a row (a halo pixel or a weight row) with
// column `col` (the pixel's in the tile, the weight's output channel).  bf16:
// rows without padding, the groups of every other run of four columns changed
// over in pairs, so that the 16 lanes which one cycle of a 16-byte read serves
// (columns 0-3 and 12-15 of one lane group, 4-11 of the next) lie on distinct
// banks, whichever column they start at; rows padded to 80 bytes, as it was,
// took two cycles (8.0 instead of 4.8 cycles per LDS instruction in all).  fp8:
// rows padded to 40 bytes (its 8-byte reads gain nothing from the change-over).
template <class T>
__device__ __forceinline__ int lds_at(int row, int col, int c) {
  return row * T::kRow + 8 * T::ES * (T::ES == 2 ? c ^ (((col >> 2) & 1) << 1) : c);
}

template <class T, int MODE, int MF, int NF, bool HEAD, bool SEQ>
__global__ __launch_bounds__(256, 2) void conv3x3_low(ConvArgs a, HeadFuse hf) {
  typedef typename T::Group Group;
  typedef typename T::Frag Frag;
  constexpr int TH = 4 * MF, BN = 16 * NF;
  constexpr int NQ = (TH + 2) * kHW * 4, RQ = (NQ + 255) / 256;        // 8-channel groups of the halo
  constexpr int WV = kCK * T::ES / 16;                                 // 16-byte vectors per weight row
  constexpr int NW = 9 * BN * WV, RW = (NW + 255) / 256;
  constexpr int kRow = T::kRow;
  constexpr int kHeadBytes = HEAD ? (TH * kTW * (BN + 1) + 6 * BN) * 4 : 0;
  constexpr int kWBytes = 9 * BN * kRow > kHeadBytes ? 9 * BN * kRow : kHeadBytes;
  __shared__ __attribute__((aligned(16))) uint8_t s_in[(TH + 2) * kHW * kRow];
  __shared__ __attribute__((aligned(16))) uint8_t s_w[kWBytes];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int tiles_y = (a.H + TH - 1) / TH;
  const int b = blockIdx.y / tiles_y;
  const int y0 = (blockIdx.y - b * tiles_y) * TH, x0 = blockIdx.x * kTW;
  const int g = lane >> 4, li = lane & 15, wrow = wave * MF;
  const int groups = (a.co + BN - 1) / BN;
  const int n0 = (blockIdx.z % groups) * BN, ks = blockIdx.z / groups;
  const int nchunks = a.ci_pad / kCK, ci = a.c0 + a.c1;  // the rest of ci_pad is zero padding
  const int splits = SEQ ? a.seq : a.splits;

  f4 acc[MF][NF], tot[SEQ ? MF : 1][SEQ ? NF : 1];
#pragma unroll
  for (int mf = 0; mf < MF; ++mf)
#pragma unroll
    for (int nf = 0; nf < NF; ++nf) {
      acc[mf][nf] = f4{0.f, 0.f, 0.f, 0.f};
      if constexpr (SEQ) tot[mf][nf] = f4{0.f, 0.f, 0.f, 0.f};
    }

  // G_FIRST: the first layer's outputs on the halo, one product per 16 halo
  // pixels and 16 channels with the first layer's own operands and rounding
  using FT = first::Tile<TH>;
  __shared__ uint16_t s_g[MODE == G_FIRST ? (TH + 4) * kGuideRow : 1];
  typename T::Quad fr[MODE == G_FIRST ? FT::BPW : 1][2];
  int at_k[MODE == G_FIRST ? 8 : 1];
  if constexpr (MODE == G_FIRST) {
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int k = min(8 * g + s, 26);
      at_k[s] = (k / 9) * kGuideRow + k % 9;
    }
  }
  auto first_layer = [&](int ch) {
    const uint16_t* w0 = static_cast<const uint16_t*>(a.w0) + (size_t)ch * kBN * 32;
    bf16x8 wv[2];
    f4 bias[2];
#pragma unroll
    for (int nf = 0; nf < 2; ++nf) {
      wv[nf] = *reinterpret_cast<const bf16x8*>(w0 + (nf * 16 + li) * 32 + 8 * g);
      bias[nf] = *reinterpret_cast<const f4*>(a.b0 + ch * kBN + nf * 16 + 4 * g);
    }
#pragma unroll
    for (int bb = 0; bb < FT::BPW; ++bb) {
      const int p = min((wave * FT::BPW + bb) * 16 + li, FT::HP - 1), py = p / kHW;
      const uint16_t* s = s_g + py * kGuideRow + 3 * (p - py * kHW);
      u4 x;
#pragma unroll
      for (int q = 0; q < 4; ++q) x[q] = (uint32_t)s[at_k[2 * q]] | ((uint32_t)s[at_k[2 * q + 1]] << 16);
      if (g == 3) x = u4{x.x, x.y & 0xffffu, 0u, 0u};  // slots 27 .. 31
#pragma unroll
      for (int nf = 0; nf < 2; ++nf) {
        const f4 d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv[nf], __builtin_bit_cast(bf16x8, x),
                                                             f4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        f4 v;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = 1.0f * d[r] + bias[nf][r];
        fr[bb][nf] = T::first(a, v);
      }
    }
  };

  // The lane's halo groups as byte offsets from the tile's first pixel
  // (clamped into the image) and its weight vectors as offsets from the
  // slab: the same for every chunk.  Every load is unconditional.
  Group rq[MODE == G_FIRST ? 1 : RQ][MODE == G_POOL ? 4 : 1];
  u4 rw[RW];
  const int yb = max(y0 - 1, 0), xb = max(x0 - 1, 0);
  const uint8_t *src0 = nullptr, *src1 = nullptr;
  uint32_t e0[MODE == G_FIRST ? 1 : RQ], e1[MODE == G_CONCAT_UP ? RQ : 1];  // in units of 16 channels
  unsigned ok = 0;
  if constexpr (MODE != G_FIRST) {
    constexpr int S = MODE == G_POOL ? 2 : 1;
    src0 = static_cast<const uint8_t*>(a.src0) +
           ((size_t)(b * S * a.H + S * yb) * (S * a.W) + S * xb) * a.c0 * T::ES;
    if constexpr (MODE == G_CONCAT_UP)
      src1 = static_cast<const uint8_t*>(a.src1) +
             ((size_t)(b * (a.H >> 1) + (yb >> 1)) * (a.W >> 1) + (xb >> 1)) * a.c1 * T::ES;
#pragma unroll
    for (int r = 0; r < RQ; ++r) {
      const int p = min(tid + 256 * r, NQ - 1) >> 2;
      const int y = y0 + p / kHW - 1, x = x0 + p % kHW - 1;
      ok |= (unsigned)(y >= 0 && y < a.H && x >= 0 && x < a.W) << r;
      const int yc = min(max(y, 0), a.H - 1), xc = min(max(x, 0), a.W - 1);
      e0[r] = (uint32_t)(((size_t)(S * (yc - yb)) * (S * a.W) + S * (xc - xb)) * (a.c0 / 16));
      if constexpr (MODE == G_CONCAT_UP)
        e1[r] = (uint32_t)(((size_t)((yc >> 1) - (yb >> 1)) * (a.W >> 1) + (xc >> 1) - (xb >> 1)) * (a.c1 / 16));
    }
  }
  // LDS row (tap, n of BN) <- packed [n / 32][chunk][tap][n % 32][32 channels]
  // (past the last tile: the last tile's rows, whose outputs are not stored)
  uint32_t ew[RW];
#pragma unroll
  for (int r = 0; r < RW; ++r) {
    const int q = min(tid + 256 * r, NW - 1), row = q / WV, tap = row / BN, n = n0 + row - tap * BN;
    const int t = min(n / kBN, a.n_tiles - 1);
    ew[r] = (uint32_t)(t * nchunks * 9 + tap) * kBN * kCK * T::ES + (n % kBN) * kCK * T::ES + 16 * (q % WV);
  }
  bool live = true;  // the lane's channels of the fetched chunk exist
  auto fetch = [&](int ch) {
    if constexpr (MODE != G_FIRST) {
      int c = ch * kCK + 8 * (tid & 3);
      live = c < ci;
      c = live ? c : 8 * (tid & 3) % a.c0;  // any valid channel
      const bool up = MODE == G_CONCAT_UP && c >= a.c0;
      const uint8_t* src = up ? src1 + (size_t)(c - a.c0) * T::ES : src0 + (size_t)c * T::ES;
#pragma unroll
      for (int r = 0; r < RQ; ++r) {
        uint32_t at = e0[r];
        if constexpr (MODE == G_CONCAT_UP) at = up ? uint32_t(e1[r]) : at;
        const uint8_t* q = src + (size_t)at * (16 * T::ES);
        rq[r][0] = *reinterpret_cast<const Group*>(q);
        if constexpr (MODE == G_POOL) {
          const size_t px = (size_t)a.c0 * T::ES, row = 2 * (size_t)a.W * px;
          rq[r][1] = *reinterpret_cast<const Group*>(q + px);
          rq[r][2] = *reinterpret_cast<const Group*>(q + row);
          rq[r][3] = *reinterpret_cast<const Group*>(q + row + px);
        }
      }
    }
    const uint8_t* w = static_cast<const uint8_t*>(a.w) + (size_t)ch * 9 * kBN * kCK * T::ES;
#pragma unroll
    for (int r = 0; r < RW; ++r) rw[r] = *reinterpret_cast<const u4*>(w + ew[r]);
    if constexpr (MODE == G_FIRST) first_layer(ch);
  };
  auto commit = [&]() {
    if constexpr (MODE == G_FIRST) {
#pragma unroll
      for (int bb = 0; bb < FT::BPW; ++bb) {
        const int q = (wave * FT::BPW + bb) * 16 + li;
        if (q < FT::HP) {
          const bool in = first::halo_inside(a, y0, x0, q);  // zero padding outside the image
#pragma unroll
          for (int nf = 0; nf < 2; ++nf)
            *reinterpret_cast<typename T::Quad*>(s_in + lds_at<T>(q, q % kHW, 2 * nf + (g >> 1)) + 4 * T::ES * (g & 1)) =
                in ? fr[bb][nf] : typename T::Quad{};
        }
      }
    } else {
#pragma unroll
      for (int r = 0; r < RQ; ++r) {
        const int q = tid + 256 * r;
        Group v;
        if constexpr (MODE == G_POOL)
          v = T::max4(rq[r]);
        else
          v = rq[r][0];
        if (q < NQ)
          *reinterpret_cast<Group*>(s_in + lds_at<T>(q >> 2, (q >> 2) % kHW, q & 3)) =
              live && ((ok >> r) & 1u) ? v : Group{};
      }
    }
#pragma unroll
    for (int r = 0; r < RW; ++r) {
      const int q = tid + 256 * r;
      if (q < NW) {
        uint8_t* d = s_w + lds_at<T>(q / WV, q / WV, q % WV * (4 / WV));
        if constexpr (kRow % 16 == 0) {
          *reinterpret_cast<u4*>(d) = rw[r];
        } else {
          *reinterpret_cast<u2*>(d) = u2{rw[r].x, rw[r].y};
          *reinterpret_cast<u2*>(d + 8) = u2{rw[r].z, rw[r].w};
        }
      }
    }
  };

  if constexpr (MODE == G_FIRST) {
    stage_guide_bf16<TH>(a, b, y0, x0, s_g);
    __syncthreads();
  }
  const uint8_t* px[3];  // by the tap's column
#pragma unroll
  for (int dx = 0; dx < 3; ++dx) px[dx] = s_in + lds_at<T>(wrow * kHW + li + dx, li + dx, g);
  const uint8_t* pw = s_w + lds_at<T>(li, li, g);
  const int sp_lo = SEQ ? 0 : ks, sp_hi = SEQ ? splits : ks + 1;
  const int ch_lo = sp_lo * nchunks / splits, ch_end = sp_hi * nchunks / splits;
  if (ch_lo < ch_end) fetch(ch_lo);
  int sp = sp_lo, sp_end = (sp_lo + 1) * nchunks / splits;  // the current split's last chunk + 1
  for (int ch = ch_lo; ch < ch_end; ++ch) {
    commit();
    __syncthreads();
    if (ch + 1 < ch_end) fetch(ch + 1);
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      Frag wv[NF], xv[MF];
#pragma unroll
      for (int nf = 0; nf < NF; ++nf) wv[nf] = *reinterpret_cast<const Frag*>(pw + (tap * BN + nf * 16) * kRow);
#pragma unroll
      for (int mf = 0; mf < MF; ++mf)
        xv[mf] = *reinterpret_cast<const Frag*>(px[tap % 3] + (mf + tap / 3) * kHW * kRow);
#pragma unroll
      for (int mf = 0; mf < MF; ++mf)
#pragma unroll
        for (int nf = 0; nf < NF; ++nf) acc[mf][nf] = T::mfma(wv[nf], xv[mf], acc[mf][nf]);
    }
    if constexpr (SEQ) {
      if (ch + 1 == sp_end) {
#pragma unroll
        for (int mf = 0; mf < MF; ++mf)
#pragma unroll
          for (int nf = 0; nf < NF; ++nf) {
            tot[mf][nf] += acc[mf][nf];
            acc[mf][nf] = f4{0.f, 0.f, 0.f, 0.f};
          }
        ++sp;
        sp_end = (sp + 1) * nchunks / splits;
      }
    }
    __syncthreads();
  }
  auto sum = [&](int mf, int nf) {
    if constexpr (SEQ)
      return tot[mf][nf];
    else
      return acc[mf][nf];
  };

  // channels past the last tile (not stored) take any valid ones' scales
  typename T::Scale sc[NF];
  if (SEQ || a.splits == 1) {
#pragma unroll
    for (int nf = 0; nf < NF; ++nf) sc[nf] = T::scale(a, n0 + nf * 16 < a.co ? n0 + nf * 16 + 4 * g : 0);
  }
  if constexpr (HEAD) {
    // head epilogue: the activations as they would be stored (bf16) and the
    // head weights in LDS (the weight buffer is free after the last chunk's
    // barrier), then two lanes per pixel
    float* sh = reinterpret_cast<float*>(s_w);
    float* shw = sh + TH * kTW * (BN + 1);
    head_weights<BN>(hf, a.co, shw);
#pragma unroll
    for (int mf = 0; mf < MF; ++mf)
#pragma unroll
      for (int nf = 0; nf < NF; ++nf) {
        const int n = nf * 16 + 4 * g;
        const f4 v = T::scaled(a, sum(mf, nf), sc[nf]);
        float* d = sh + ((wrow + mf) * kTW + li) * (BN + 1) + n;
#pragma unroll
        for (int r = 0; r < 4; r += 2) {
          const uint32_t p = pk_bf16(fmaxf(v[r], 0.0f), fmaxf(v[r + 1], 0.0f));
          d[r] = __uint_as_float(p << 16);
          d[r + 1] = __uint_as_float(p & 0xffff0000u);
        }
      }
    __syncthreads();
    head_finish<TH, BN>(hf, sh, shw, b, a.H, a.W, y0, x0);
    return;
  }
  const int x = x0 + li;
  if (x >= a.W) return;
  const size_t at0 = ((size_t)(b * a.H + y0 + wrow) * a.W + x) * a.co + n0 + 4 * g, row = (size_t)a.W * a.co;
  if (!SEQ && a.splits > 1) {
    float* to = a.partial + (size_t)ks * a.B * a.H * a.W * a.co + at0;
#pragma unroll
    for (int mf = 0; mf < MF; ++mf)
#pragma unroll
      for (int nf = 0; nf < NF; ++nf)
        if (y0 + wrow + mf < a.H && n0 + nf * 16 < a.co)
          *reinterpret_cast<f4*>(to + mf * row + nf * 16) = acc[mf][nf];
    return;
  }
  // two 16-channel blocks' quads joined (see join_quads): half as many stores,
  // of 64 bytes per pixel instead of 32 (bf16)
  const size_t at2 = at0 - 4 * g + 16 * (g & 1) + 8 * (g >> 1);
  T::store(a, [&](auto* out, const auto& quad) __attribute__((always_inline)) {
#pragma unroll
    for (int mf = 0; mf < MF; ++mf) {
      if (y0 + wrow + mf >= a.H) break;
#pragma unroll
      for (int nf = 0; nf < NF; nf += 2) {  // the channel count is a multiple of 16
        const auto p = quad(T::scaled(a, sum(mf, nf), sc[nf]));
        if (nf + 1 < NF && n0 + (nf + 1) * 16 < a.co) {
          constexpr int last = NF - 1;
          const auto v = join_quads(p, quad(T::scaled(a, sum(mf, min(nf + 1, last)), sc[min(nf + 1, last)])));
          *reinterpret_cast<std::remove_const_t<decltype(v)>*>(out + at2 + mf * row + nf * 16) = v;
        } else if (n0 + nf * 16 < a.co) {
          *reinterpret_cast<std::remove_const_t<decltype(p)>*>(out + at0 + mf * row + nf * 16) = p;
        }
      }
    }
  });
}

template <class T, int MODE, int MF, int NF, bool SEQ>
hipError_t launch_tile(const ConvArgs& a, hipStream_t s, const HeadFuse* head) {
  constexpr int TH = 4 * MF;
  const dim3 grid((a.W + kTW - 1) / kTW, ((a.H + TH - 1) / TH) * a.B,
                  ((a.co + 16 * NF - 1) / (16 * NF)) * (SEQ ? 1 : a.splits));
  if constexpr (T::ES == 2 && MODE == G_PLAIN && MF <= 2 && NF <= 3 && !SEQ) {
    if (head) {
      hipLaunchKernelGGL((conv3x3_low<T, MODE, MF, NF, true, SEQ>), grid, dim3(256), 0, s, a, *head);
      return hipGetLastError();
    }
  }
  if (head) return hipErrorInvalidValue;
  hipLaunchKernelGGL((conv3x3_low<T, MODE, MF, NF, false, SEQ>), grid, dim3(256), 0, s, a, HeadFuse{});
  return hipGetLastError();
}

// Tiles do not change any sum, so they follow the whole batch's workgroups:
// the largest ones that still give the 256 CUs two workgroups each, else
// the layer's own tile height with 32 channels.  Widths of 48 per workgroup
// serve layers of a multiple of 48 that is no multiple of 64.  Pooled input
// and the fused first layer keep 8 rows (their prefetched values would not
// fit in the registers).
template <class T, int MODE>
hipError_t launch_layer(const ConvArgs& a, hipStream_t s, const HeadFuse* head) {
  auto wgs = [&](int rows, int nf) {
    return (long)((a.W + kTW - 1) / kTW) * ((a.H + rows - 1) / rows) * a.B * ((a.co + 16 * nf - 1) / (16 * nf));
  };
  if (a.seq > 1) {
    if constexpr (MODE == G_PLAIN || MODE == G_CONCAT_UP) {
      if (wgs(16, 2) >= 512 && rows_fit(a.H, 16)) return launch_tile<T, MODE, 4, 2, true>(a, s, head);
    }
    return launch_tile<T, MODE, 2, 2, true>(a, s, head);
  }
  const int nf = a.co % 64 == 0 ? 4 : a.co % 48 == 0 ? 3 : a.co > 32 ? 4 : 2;
  if (a.splits == 1) {
    if constexpr (MODE == G_PLAIN || MODE == G_CONCAT_UP) {
      if (!head && wgs(16, nf) >= 512 && rows_fit(a.H, 16)) {
        if (nf == 4) return launch_tile<T, MODE, 4, 4, false>(a, s, head);
        if (nf == 3) return launch_tile<T, MODE, 4, 3, false>(a, s, head);
        return launch_tile<T, MODE, 4, 2, false>(a, s, head);
      }
    }
    const bool fit = rows_fit(a.H, 8);
    if (nf == 3 && (head || (fit && wgs(8, nf) >= 512))) return launch_tile<T, MODE, 2, 3, false>(a, s, head);
    if (nf == 4 && fit && wgs(8, nf) >= 512) return launch_tile<T, MODE, 2, 4, false>(a, s, head);
    if (fit && wgs(8, 2) >= 512) return launch_tile<T, MODE, 2, 2, false>(a, s, head);
  }
  return a.th == 4 ? launch_tile<T, MODE, 1, 2, false>(a, s, head) : launch_tile<T, MODE, 2, 2, false>(a, s, head);
}

template <class T>
hipError_t launch(int mode, const ConvArgs& a, hipStream_t s, const HeadFuse* head) {
  if (a.co % 16 || a.c0 % 16 || a.c1 % 16) return hipErrorInvalidValue;
  if (head && (a.splits != 1 || a.seq > 1 || a.co > 48 || !a.relu)) return hipErrorInvalidValue;
  switch (mode) {
    case G_FIRST:
      if (!a.w0 || !a.b0) return hipErrorInvalidValue;
      return launch_layer<T, G_FIRST>(a, s, head);
    case G_PLAIN: return launch_layer<T, G_PLAIN>(a, s, head);
    case G_POOL: return launch_layer<T, G_POOL>(a, s, head);
    case G_CONCAT_UP: return launch_layer<T, G_CONCAT_UP>(a, s, head);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace low
}  // namespace lnm
