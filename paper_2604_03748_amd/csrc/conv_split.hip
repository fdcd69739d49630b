// U-Net 3x3 convolutions (Section 4.3) in fp32 on the bf16 matrix cores.
//
// Every fp32 operand is the sum of three bf16 numbers (hi, mid, lo: each the
// remainder of the ones before it, rounded to nearest even; 8 + 8 + 8 bits,
// so the sum is the operand to its last bit or so), and a product is the six
// partial products whose size reaches fp32's own rounding:
//   a b = ah bh + (ah bm + am bh + am bm + ah bl + al bh),
// each exact in the fp32 accumulator of v_mfma_f32_16x16x32_bf16.  The first
// term and the five small ones have accumulators of their own, added once at
// the end, so the sum of the large terms takes one rounding per 32 products
// (the fp32 instruction: one per 4) and the error against fp64 is no larger
// than the fp32 instruction's (lightmaps of 8 x 256^2, 4 levels, base 32:
// 2.5e-7 against 6.8e-7).  Six bf16 products take 96 cycles per 16 x 16 x 32
// block against 256 for fp32's.  Measured on that network: inference 1805 ->
// 971 us (175 TFLOP/s of fp32 products), one 256^2 frame 355 -> 290 us; the
// data gradients of a training batch, with the masking, pooling and
// concatenation passes that they now carry, 2140 -> 1065 us.
//
// Same tiles as the fp32-instruction kernel: a workgroup of four wavefronts
// computes a 4 MF x 16 pixel tile x 32 output channels; per 16-channel input
// chunk the halo and the 9 x 32 x 16 weight slab are split and staged in LDS
// (the next chunk's fp32 values in registers meanwhile), and the K = 32
// steps take two taps x 16 channels.  LDS rows hold a pixel's (or weight
// row's) three 16-channel pieces in 96 bytes without padding: the 16 lanes
// that one LDS cycle serves (rows 0-3 and 12-15 of one lane group, 4-11 of
// the next) then lie on distinct banks.  (Rows padded to 112 bytes looked
// safer and took two cycles: 1023 -> 971 us for the inference above.)  The
// product is taken transposed (channels as MFMA rows), so a lane ends with
// four consecutive channels of one pixel: 16-byte stores, and the gradient's
// routing (see Route) on whole vectors.
#include <type_traits>

#include "first_layer.h"
#include "halo_f32.h"
#include "head.h"
#include "internal.h"
#include "split_bf16.h"

namespace lnm {
namespace {

constexpr int kCh = 16;     // input channels per chunk
constexpr int kRow = 48;    // bf16 per LDS row: 3 pieces x 16 channels
constexpr int kSteps = 5;   // K = 32 steps per chunk: taps (0, 1), (2, 3), (4, 5), (6, 7), (8, none)

// channels [c, c + 4) of an LDS row
template <bool SAFE>
__device__ __forceinline__ void store_row(uint16_t* row, int c, f4 v, float& over) {
  const Pieces p = split<SAFE>(v, over);
  *reinterpret_cast<u2*>(row + c) = p.hi;
  *reinterpret_cast<u2*>(row + kCh + c) = p.mid;
  *reinterpret_cast<u2*>(row + 2 * kCh + c) = p.lo;
}

// What becomes of the outputs: stored (with bias and ReLU, or as split-K
// partials), or, for a data gradient, passed on to the layers' gradients:
//   R_MASK    through the ReLU of the layer below (its output in y0);
//   R_POOL    each 2x2 window's gradient g0 (the skip connection's part so
//             far) takes the value at its first maximum in raster order and
//             passes the ReLU (outputs y0);
//   R_CONCAT  channels [0, c_skip) to g0; the others summed over each 2x2
//             block, through the ReLU of the low-resolution layer (y1), to g1.
template <int MODE, int MF, bool HEAD, int ROUTE>
__global__ __launch_bounds__(256, 2) void conv3x3_split(ConvArgs a, HeadFuse hf) {
  constexpr int TH = 4 * MF, NF = kBN / 16;
  // the halo rows, and zeros that the lanes without a tap read in the last step
  constexpr int kHaloElems = (TH + 2) * kHW * kRow;
  constexpr int kZero = ((MF - 1) * kHW > (NF - 1) * 16 ? (MF - 1) * kHW : (NF - 1) * 16) * kRow + kRow;
  __shared__ __attribute__((aligned(16))) uint16_t s_in[kHaloElems + kZero];
  __shared__ __attribute__((aligned(16))) uint16_t s_w[9 * kBN * kRow];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int tiles_y = (a.H + TH - 1) / TH;
  const int b = blockIdx.y / tiles_y;
  const int y0 = (blockIdx.y - b * tiles_y) * TH, x0 = blockIdx.x * kTW;
  const int nt = blockIdx.z % a.n_tiles, ks = blockIdx.z / a.n_tiles;
  const int nchunks = a.ci_pad / kCh;
  const int ch_lo = ks * nchunks / a.splits, ch_hi = (ks + 1) * nchunks / a.splits;
  const float* wblk = static_cast<const float*>(a.w) + (size_t)nt * nchunks * 9 * kBN * kCh;
  const int g = lane >> 4, li = lane & 15;
  const int wrow = wave * MF;

  f4 acc[MF][NF], cor[MF][NF];
#pragma unroll
  for (int mf = 0; mf < MF; ++mf)
#pragma unroll
    for (int nf = 0; nf < NF; ++nf) acc[mf][nf] = cor[mf][nf] = f4{0.f, 0.f, 0.f, 0.f};

  // G_FIRST: per chunk, the first layer's outputs at the halo pixels (fp32
  // products in the first layer's own K order, taken transposed: lane (li, g)
  // gets channels 4g .. 4g + 3 of halo pixel 16 blk + li), bias and ReLU
  using FT = first::Tile<TH>;
  __shared__ f4 s_g[MODE == G_FIRST ? FT::NG : 1];
  f4 fr[MODE == G_FIRST ? FT::BPW : 1];
  auto first_layer = [&](int ch) {
    const int n = ch * kCh + li;
    const float* w = static_cast<const float*>(a.w0) + (size_t)(n / kBN) * 9 * kBN * 4 + (n % kBN) * 4;
    float wk[7];
#pragma unroll
    for (int st = 0; st < 7; ++st) {
      const int k = 4 * st + g;
      wk[st] = k < 27 ? w[(k / 3) * kBN * 4 + k % 3] : 0.0f;
    }
    const f4 bias = *reinterpret_cast<const f4*>(a.b0 + ch * kCh + 4 * g);
#pragma unroll
    for (int bb = 0; bb < FT::BPW; ++bb) {
      const int blk = wave * FT::BPW + bb;
      if (blk >= FT::HB) break;
      const int p = min(blk * 16 + li, FT::HP - 1);
      f4 d = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int st = 0; st < 7; ++st)
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(wk[st], first::guide_slot(s_g, p, 4 * st + g), d, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) fr[bb][r] = fmaxf(d[r] + bias[r], 0.0f);
    }
  };

  constexpr int NQ = (TH + 2) * kHW * (kCh / 4), NW = 9 * kBN * kCh / 4;
  constexpr int RQ = (NQ + 255) / 256, RW = (NW + 255) / 256;
  Halo<MODE> rq[MODE == G_FIRST ? 1 : RQ];
  f4 rw[RW];
  // The lane's halo entries as element offsets from the tile's first pixel
  // (clamped into the image; the same for every chunk), so that a chunk's
  // loads need one addition each.
  const int yb = max(y0 - 1, 0), xb = max(x0 - 1, 0);
  const float *src0 = nullptr, *src1 = nullptr;
  size_t e0[RQ], e1[MODE == G_CONCAT_UP ? RQ : 1];
  unsigned ok = 0;
  if constexpr (MODE != G_FIRST) {
    constexpr int S = MODE == G_POOL ? 2 : 1;
    src0 = static_cast<const float*>(a.src0) + ((size_t)(b * S * a.H + S * yb) * (S * a.W) + S * xb) * a.c0;
    if constexpr (MODE == G_CONCAT_UP)
      src1 = static_cast<const float*>(a.src1) +
             ((size_t)(b * (a.H >> 1) + (yb >> 1)) * (a.W >> 1) + (xb >> 1)) * a.c1;
#pragma unroll
    for (int r = 0; r < RQ; ++r) {
      const int q = min(tid + 256 * r, NQ - 1);
      const int c4 = q % (kCh / 4), p = q / (kCh / 4);
      const int y = y0 + p / kHW - 1, x = x0 + p % kHW - 1;
      ok |= (unsigned)(y >= 0 && y < a.H && x >= 0 && x < a.W) << r;
      const int yc = min(max(y, 0), a.H - 1), xc = min(max(x, 0), a.W - 1);
      e0[r] = ((size_t)(S * (yc - yb)) * (S * a.W) + S * (xc - xb)) * a.c0 + 4 * c4;
      if constexpr (MODE == G_CONCAT_UP)
        e1[r] = ((size_t)((yc >> 1) - (yb >> 1)) * (a.W >> 1) + (xc >> 1) - (xb >> 1)) * a.c1 + 4 * c4;
    }
  }
  auto fetch = [&](int ch) {
    if constexpr (MODE != G_FIRST) {
      const int c = ch * kCh;  // a chunk lies in one of the concatenation's sources
      const bool up = MODE == G_CONCAT_UP && c >= a.c0;
      const float* src = up ? src1 + (c - a.c0) : src0 + c;
#pragma unroll
      for (int r = 0; r < RQ; ++r) {
        const float* q = src + (MODE == G_CONCAT_UP && up ? e1[MODE == G_CONCAT_UP ? r : 0] : e0[r]);
        rq[r].v[0] = *reinterpret_cast<const f4*>(q);
        if constexpr (MODE == G_POOL) {
          const size_t row = 2 * (size_t)a.W * a.c0;
          rq[r].v[1] = *reinterpret_cast<const f4*>(q + a.c0);
          rq[r].v[2] = *reinterpret_cast<const f4*>(q + row);
          rq[r].v[3] = *reinterpret_cast<const f4*>(q + row + a.c0);
        }
      }
    }
    const float* wsrc = wblk + (size_t)ch * 9 * kBN * kCh;
#pragma unroll
    for (int r = 0; r < RW; ++r) rw[r] = *reinterpret_cast<const f4*>(wsrc + 4 * min(tid + 256 * r, NW - 1));
    if constexpr (MODE == G_FIRST) first_layer(ch);
  };
  // (Lanes past the end hold the last entry again.  Storing it once more is
  // cheaper than a branch per entry where the registers let all entries' splits
  // overlap, up to 8-row tiles.)
  auto commit = [&]() {
    float over = 0.0f;
    auto put = [&](auto safe, int q, uint16_t* rows, f4 v) {
      store_row<decltype(safe)::value>(rows + (q / (kCh / 4)) * kRow, 4 * (q % (kCh / 4)), v, over);
    };
    constexpr int NV = MODE == G_FIRST ? FT::BPW : RQ;
    f4 v[NV];
#pragma unroll
    for (int r = 0; r < NV; ++r) {
      if constexpr (MODE == G_FIRST) {
        const int q = (wave * FT::BPW + r) * 16 + li;  // zero padding outside the image
        v[r] = q < FT::HP && first::halo_inside(a, y0, x0, q) ? fr[r] : f4{0.f, 0.f, 0.f, 0.f};
      } else {
        v[r] = halo_value<MODE>(rq[r], (ok >> r) & 1u);
      }
    }
    auto all = [&](auto safe) {
#pragma unroll
      for (int r = 0; r < NV; ++r) {
        if constexpr (MODE == G_FIRST) {
          const int q = (wave * FT::BPW + r) * 16 + li;
          if (q < FT::HP) store_row<decltype(safe)::value>(s_in + q * kRow, 4 * g, v[r], over);
        } else {
          if (MF <= 2 || tid + 256 * r < NQ) put(safe, min(tid + 256 * r, NQ - 1), s_in, v[r]);
        }
      }
#pragma unroll
      for (int r = 0; r < RW; ++r)
        if (MF <= 2 || tid + 256 * r < NW) put(safe, min(tid + 256 * r, NW - 1), s_w, rw[r]);
    };
    all(std::false_type{});
    if (__builtin_expect(!(over == over), 0)) all(std::true_type{});
  };

  // the lane's LDS offsets per step: tap 2 st + g / 2 (none in the last step's
  // upper half: zeros), channels 8 (g % 2) .. + 7
  int at_in[kSteps], at_w[kSteps];
  const uint16_t* last_w = s_w;
#pragma unroll
  for (int st = 0; st < kSteps; ++st) {
    const int tap = min(2 * st + (g >> 1), 8);
    at_in[st] = ((wrow + tap / 3) * kHW + li + tap % 3) * kRow + 8 * (g & 1);
    at_w[st] = (tap * kBN + li) * kRow + 8 * (g & 1);
  }
  if (g >= 2) {
    at_in[kSteps - 1] = kHaloElems;
    last_w = s_in;
    at_w[kSteps - 1] = kHaloElems;
  }
  for (int q = tid; q < kZero / 8; q += 256) *reinterpret_cast<f4*>(s_in + kHaloElems + 8 * q) = f4{0.f, 0.f, 0.f, 0.f};

  if constexpr (MODE == G_FIRST) {
    first::stage_guide<TH>(a, b, y0, x0, s_g);
    __syncthreads();
  }
  constexpr int MG = MF < 2 ? MF : 2;  // pixel rows whose products alternate
  // The staged chunk's products, and the next one's loads.  Each step's
  // operands are read among the step before's products and the loads issued
  // among the first steps' in 4-row tiles, whose few wavefronts hide neither
  // (2040 -> 1290 cycles for 60 products by the reads alone; the
  // base-16 network's small images 65 -> 62 us, a 256^2 frame 300 -> 294).
  // Taller tiles gain nothing.
  auto products = [&](int ch, auto more) __attribute__((always_inline)) {
    if constexpr (decltype(more)::value) fetch(ch + 1);
#pragma unroll
    for (int st = 0; st < kSteps; ++st) {
      const uint16_t* pw = (st == kSteps - 1 ? last_w : s_w) + at_w[st];
      const uint16_t* px = s_in + at_in[st];
      bf16x8 wv[NF][3];
#pragma unroll
      for (int nf = 0; nf < NF; ++nf)
#pragma unroll
        for (int q = 0; q < 3; ++q) wv[nf][q] = *reinterpret_cast<const bf16x8*>(pw + nf * 16 * kRow + q * kCh);
#pragma unroll
      for (int m0 = 0; m0 < MF; m0 += MG) {
        bf16x8 xv[MG][3];
#pragma unroll
        for (int mf = 0; mf < MG; ++mf)
#pragma unroll
          for (int q = 0; q < 3; ++q)
            xv[mf][q] = *reinterpret_cast<const bf16x8*>(px + (m0 + mf) * kHW * kRow + q * kCh);
#pragma unroll
        for (int t = 0; t < 6; ++t)
#pragma unroll
          for (int mf = 0; mf < MG; ++mf)
#pragma unroll
            for (int nf = 0; nf < NF; ++nf) {
              f4& c = t < 5 ? cor[m0 + mf][nf] : acc[m0 + mf][nf];
              c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv[nf][kSplitTerm[t][0]], xv[mf][kSplitTerm[t][1]], c, 0, 0, 0);
            }
      }
    }
    if constexpr (MF == 1) {
      constexpr int kReads = 3 * (NF + MF), kMul = 6 * NF * MF;
      constexpr int kLoads = decltype(more)::value ? RW + (MODE == G_FIRST ? 0 : RQ * (MODE == G_POOL ? 4 : 1)) : 0;
      __builtin_amdgcn_sched_group_barrier(0x100, kReads, 0);
#pragma unroll
      for (int st = 0; st < kSteps; ++st) {
#pragma unroll
        for (int k = 0; k < kReads; ++k) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          if (st + 1 < kSteps) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          if (k % 3 == 0 && st * (kReads / 3) + k / 3 < kLoads) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, kMul - kReads, 0);
      }
    }
  };
  if (ch_lo < ch_hi) fetch(ch_lo);
  for (int ch = ch_lo; ch < ch_hi; ++ch) {
    commit();
    __syncthreads();
    if constexpr (MF == 1) {
      if (ch + 1 < ch_hi)
        products(ch, std::true_type{});
      else
        products(ch, std::false_type{});
    } else {
      if (ch + 1 < ch_hi) fetch(ch + 1);
      products(ch, std::false_type{});
    }
    __syncthreads();
  }
  // (a sum past fp32's range is infinite by its large terms alone; the small
  // ones, of either sign, are then infinite too and would make it NaN)
  float top = 0.0f;
#pragma unroll
  for (int mf = 0; mf < MF; ++mf)
#pragma unroll
    for (int nf = 0; nf < NF; ++nf) {
      const f4 v = acc[mf][nf];
      top = fmaxf(top, fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
    }
  if (__builtin_expect(top == INFINITY, 0)) {
#pragma unroll
    for (int mf = 0; mf < MF; ++mf)
#pragma unroll
      for (int nf = 0; nf < NF; ++nf)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (fabsf(acc[mf][nf][r]) == INFINITY) cor[mf][nf][r] = 0.0f;
  }
#pragma unroll
  for (int mf = 0; mf < MF; ++mf)
#pragma unroll
    for (int nf = 0; nf < NF; ++nf) acc[mf][nf] += cor[mf][nf];

  if constexpr (HEAD) {
    // head epilogue (one 32-channel tile, unsplit, ReLU layer): activations
    // and head weights to LDS, then two threads per pixel finish the head
    static_assert((TH * kTW * 33 + 6 * kBN) * 4 <= (int)sizeof(s_w), "head tile must fit the weight buffer");
    float* sh = reinterpret_cast<float*>(s_w);
    float* shw = sh + TH * kTW * 33;
    head_weights(hf, a.co, shw);
#pragma unroll
    for (int nf = 0; nf < NF; ++nf) {
      const int n = nf * 16 + 4 * g;
      const f4 bias = *reinterpret_cast<const f4*>(a.bias + n);  // padded to whole tiles
#pragma unroll
      for (int mf = 0; mf < MF; ++mf)
#pragma unroll
        for (int r = 0; r < 4; ++r) sh[((wrow + mf) * kTW + li) * 33 + n + r] = fmaxf(acc[mf][nf][r] + bias[r], 0.0f);
    }
    __syncthreads();
    head_finish<TH>(hf, sh, shw, b, a.H, a.W, y0, x0);
    return;
  }

  const int x = x0 + li;
  // everything the outputs need is loaded ahead of the stores: a load issued
  // after a store waits for it
  f4 bias[ROUTE == R_NONE ? NF : 1];
  if constexpr (ROUTE == R_NONE) {
    if (a.splits == 1) {
#pragma unroll
      for (int nf = 0; nf < NF; ++nf) bias[nf] = *reinterpret_cast<const f4*>(a.bias + nt * kBN + nf * 16 + 4 * g);
    }
  }
  f4 mask[ROUTE == R_MASK ? MF : 1][ROUTE == R_MASK ? NF : 1];
  if constexpr (ROUTE == R_MASK) {
#pragma unroll
    for (int mf = 0; mf < MF; ++mf)
#pragma unroll
      for (int nf = 0; nf < NF; ++nf)
        mask[mf][nf] = *reinterpret_cast<const f4*>(
            a.y0 + ((size_t)(b * a.H + min(y0 + wrow + mf, a.H - 1)) * a.W + min(x, a.W - 1)) * a.co +
            min(nt * kBN + nf * 16, a.co - 16) + 4 * g);
  }
#pragma unroll
  for (int mf = 0; mf < MF; ++mf) {
    const int y = y0 + wrow + mf;
    const bool in = y < a.H && x < a.W;
    const size_t pix = (size_t)(b * a.H + min(y, a.H - 1)) * a.W + min(x, a.W - 1);
#pragma unroll
    for (int nf = 0; nf < NF; ++nf) {
      const int n = nt * kBN + nf * 16 + 4 * g;
      if (nt * kBN + nf * 16 >= a.co) continue;  // the channel count is a multiple of 16
      f4 v = acc[mf][nf];
      if constexpr (ROUTE == R_NONE) {
        if (!in) continue;
        if (a.splits > 1) {
          __builtin_nontemporal_store(
              v, reinterpret_cast<f4*>(a.partial + ((size_t)ks * a.B * a.H * a.W + pix) * a.co + n));
          continue;
        }
        v += bias[nf];
        if (a.relu) {
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = fmaxf(v[r], 0.0f);
        }
        __builtin_nontemporal_store(v, reinterpret_cast<f4*>(static_cast<float*>(a.out) + pix * a.co + n));
      } else if constexpr (ROUTE == R_MASK) {
        if (!in) continue;
        const f4 ym = mask[mf][nf];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = ym[r] > 0.0f ? v[r] : 0.0f;
        *reinterpret_cast<f4*>(a.g0 + pix * a.co + n) = v;
      } else if constexpr (ROUTE == R_POOL) {
        if (!in) continue;
        const size_t W2 = 2 * (size_t)a.W, at = (((size_t)b * 2 * a.H + 2 * y) * W2 + 2 * x) * a.co + n;
        const size_t o[4] = {at, at + a.co, at + W2 * a.co, at + W2 * a.co + a.co};
        f4 yy[4], gg[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          yy[k] = *reinterpret_cast<const f4*>(a.y0 + o[k]);
          gg[k] = *reinterpret_cast<const f4*>(a.g0 + o[k]);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float m = yy[0][r];
          int best = 0;
#pragma unroll
          for (int k = 1; k < 4; ++k)
            if (yy[k][r] > m) {
              m = yy[k][r];
              best = k;
            }
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const float s = k == best ? gg[k][r] + v[r] : gg[k][r];
            gg[k][r] = yy[k][r] > 0.0f ? s : 0.0f;
          }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) *reinterpret_cast<f4*>(a.g0 + o[k]) = gg[k];
      } else {
        if (nt * kBN + nf * 16 < a.c_skip) {  // a multiple of 16: the block lies on one side
          if (in) *reinterpret_cast<f4*>(a.g0 + pix * a.c_skip + n) = v;
        } else if (mf % 2 == 0) {
          // this row and the next, this column and its neighbour's, in raster order
          const f4 w = acc[mf + (MF > 1)][nf];
          f4 s;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float v1 = __shfl_xor(v[r], 1), w1 = __shfl_xor(w[r], 1);
            s[r] = ((v[r] + v1) + w[r]) + w1;
          }
          if (in && (li & 1) == 0) {
            const int c1 = a.co - a.c_skip;
            const size_t o = (((size_t)b * (a.H >> 1) + (y >> 1)) * (a.W >> 1) + (x >> 1)) * c1 + n - a.c_skip;
            const f4 ym = *reinterpret_cast<const f4*>(a.y1 + o);
#pragma unroll
            for (int r = 0; r < 4; ++r) s[r] = ym[r] > 0.0f ? s[r] : 0.0f;
            *reinterpret_cast<f4*>(a.g1 + o) = s;
          }
        }
      }
    }
  }
}

template <int MODE, int MF, int ROUTE>
hipError_t launch_mf(const ConvArgs& a, hipStream_t s, const HeadFuse* head) {
  constexpr int TH = 4 * MF;
  const dim3 grid((a.W + kTW - 1) / kTW, ((a.H + TH - 1) / TH) * a.B, a.n_tiles * a.splits);
  if constexpr (MODE == G_PLAIN && MF <= 2 && ROUTE == R_NONE) {
    if (head) {
      hipLaunchKernelGGL((conv3x3_split<MODE, MF, true, ROUTE>), grid, dim3(256), 0, s, a, *head);
      return hipGetLastError();
    }
  }
  if (head) return hipErrorInvalidValue;
  hipLaunchKernelGGL((conv3x3_split<MODE, MF, false, ROUTE>), grid, dim3(256), 0, s, a, HeadFuse{});
  return hipGetLastError();
}

// The tile height does not change any sum, so it follows the whole batch's
// workgroups: the tallest tiles that still give the 256 CUs two workgroups
// each (all that 16-row tiles' LDS allows).  Taller tiles read less LDS per
// product (a 4-row tile's reads take longer than its products) and split
// the weights for more pixels: 8 x 256^2 on the 4-level base-32 network took
// 1.27 times as long with the 4-row tiles that one image takes in the deep
// levels.  For one image 512 is the best as well: a 256^2 frame takes 294
// us, 300 with 8-row tiles from 256 workgroups on and 304 from 1024 on.
int tile_rows(const ConvArgs& a, int tallest) {
  auto wgs = [&](int th) {
    return (long)((a.W + kTW - 1) / kTW) * ((a.H + th - 1) / th) * a.B * a.n_tiles * a.splits;
  };
  if (tallest >= 4 && wgs(16) >= 512 && rows_fit(a.H, 16)) return 4;
  return wgs(8) >= 512 && rows_fit(a.H, 8) ? 2 : 1;
}

template <int MODE>
hipError_t launch_layer(const ConvArgs& a, hipStream_t s, const HeadFuse* head) {
  const int mf = tile_rows(a, MODE == G_POOL || MODE == G_FIRST || head ? 2 : 4);
  if constexpr (MODE == G_PLAIN || MODE == G_CONCAT_UP) {
    if (mf == 4) return launch_mf<MODE, 4, R_NONE>(a, s, head);
  }
  return mf == 2 ? launch_mf<MODE, 2, R_NONE>(a, s, head) : launch_mf<MODE, 1, R_NONE>(a, s, head);
}
template <int ROUTE>
hipError_t launch_route(const ConvArgs& a, hipStream_t s) {
  const int mf = tile_rows(a, 4);
  if (mf == 4) return launch_mf<G_PLAIN, 4, ROUTE>(a, s, nullptr);
  if constexpr (ROUTE != R_CONCAT) {  // whose 2x2 sums need two rows per wavefront
    if (mf == 1) return launch_mf<G_PLAIN, 1, ROUTE>(a, s, nullptr);
  }
  return launch_mf<G_PLAIN, 2, ROUTE>(a, s, nullptr);
}

}  // namespace

hipError_t launch_conv3x3_split(int mode, const ConvArgs& a, hipStream_t s, const HeadFuse* head) {
  if (head && (a.n_tiles != 1 || a.splits != 1 || a.co > kBN || !a.relu)) return hipErrorInvalidValue;
  if (a.co % 16) return hipErrorInvalidValue;
  if (a.route != R_NONE) {
    if (mode != G_PLAIN || a.splits != 1 || head) return hipErrorInvalidValue;
    switch (a.route) {
      case R_MASK: return launch_route<R_MASK>(a, s);
      case R_POOL: return launch_route<R_POOL>(a, s);
      case R_CONCAT:
        if (a.c_skip % 16 || a.H % 2 || a.W % 2) return hipErrorInvalidValue;
        return launch_route<R_CONCAT>(a, s);
      default: return hipErrorInvalidValue;
    }
  }
  switch (mode) {
    case G_FIRST:
      if (!a.w0 || !a.b0) return hipErrorInvalidValue;
      return launch_layer<G_FIRST>(a, s, head);
    case G_PLAIN: return launch_layer<G_PLAIN>(a, s, head);
    case G_POOL: return launch_layer<G_POOL>(a, s, head);
    case G_CONCAT_UP: return launch_layer<G_CONCAT_UP>(a, s, head);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace lnm
