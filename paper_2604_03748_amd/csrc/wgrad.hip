// Weight gradient of a 3x3 layer: dW[o][c][tap] = sum_p E[p][o] X[p + tap][c]
// as a matrix product with M = output channels, N = input channels, K =
// pixels.  A workgroup sums 16 WM output x 16 WN input channels x 9 taps over a
// group of 8 x 16 pixel tiles: its four wavefronts take the WM x WN channel
// blocks and, where that leaves wavefronts over, WK shares of each tile's rows
// (added in order through LDS at the end), so a group writes one partial sum
// per weight.  X is gathered exactly as the forward pass reads it (pooled /
// upsampled-concatenated inputs stay virtual).  The next tile's loads are in
// registers while the matrix cores work on the current one.  The workgroups
// of the first input-channel block also sum E itself, the bias gradient.
//
// The products run on the bf16 matrix cores as three-piece splits
// (split_bf16.h), the first layer's (3 input channels) on the fp32 ones.
// At 8 x 256^2 on the 4-level base-32 network all layers' sums and reductions
// take 1120 us, half the rate of the six bf16 products; 1804 with the fp32
// instruction everywhere (74% of its rate in the large layers).  What bounds
// it now is the work between the products (gather, split, LDS) and the
// barriers around it: two workgroups per CU are what registers and LDS allow.
#include <type_traits>

#include "halo_f32.h"
#include "internal.h"
#include "split_bf16.h"

namespace lnm {
namespace {

constexpr int kWTH = 8, kWTilePix = kWTH * kTW, kWHaloPix = (kWTH + 2) * kHW;

// LDS floats per pixel of a 16- or 32-channel tile: rows 16-byte aligned, the
// four pixels that a wavefront reads together on distinct bank halves
constexpr int wgrad_pitch(int channels) { return channels == 32 ? 40 : 24; }

// End of a workgroup: the row shares of each channel block added in order
// through LDS (`smem`, free by now), the partial sums stored, and, in the
// workgroups of the first input-channel block, the bias sums (lanes tid % QE
// hold one channel quad each: added in lane order).
template <int WM, int WN>
__device__ __forceinline__ void end_sums(const WgradArgs& a, void* smem, f4 (&acc)[9], f4 bsum) {
  constexpr int WK = 4 / (WM * WN), BM = 16 * WM, QE = BM / 4;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, li = lane & 15;
  const int wm = wave % WM, wn = (wave / WM) % WN, wk = wave / (WM * WN);
  const int o0 = blockIdx.y * BM, c0 = blockIdx.z * 16 * WN;
  if constexpr (WK > 1) {
    f4* sh = static_cast<f4*>(smem);
    if (wk > 0) {
#pragma unroll
      for (int tap = 0; tap < 9; ++tap) sh[((wave - WM * WN) * 9 + tap) * 64 + lane] = acc[tap];
    }
    __syncthreads();
    if (wk == 0) {
#pragma unroll
      for (int k = 1; k < WK; ++k)
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) acc[tap] += sh[((wave + (k - 1) * WM * WN) * 9 + tap) * 64 + lane];
    }
  }
  if (wk == 0) {
#pragma unroll
    for (int tap = 0; tap < 9; ++tap)
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        const int o = o0 + 16 * wm + 4 * g + rr, c = c0 + 16 * wn + li;
        a.partial[(((size_t)blockIdx.x * a.co_pad + o) * 9 + tap) * a.ci_pad + c] = acc[tap][rr];
      }
  }
  if (blockIdx.z == 0) {
    __syncthreads();
    f4* sh = static_cast<f4*>(smem);
    sh[tid] = bsum;
    __syncthreads();
    if (tid < BM) {
      float v = 0.0f;
      for (int k = 0; k < 256 / QE; ++k) v += sh[k * QE + tid / 4][tid % 4];
      a.bias_partial[(size_t)blockIdx.x * a.co_pad + o0 + tid] = v;
    }
  }
}

// The first layer on the fp32 matrix instruction; a lane walks a tile column,
// so each row of X is read from LDS once for its three taps.
template <int WM>
__global__ __launch_bounds__(256, 2) void wgrad_first_f32(WgradArgs a) {
  constexpr int MODE = G_GUIDE, WN = 1, WK = 4 / (WM * WN), BM = 16 * WM, BC = 16 * WN;
  constexpr int PE = wgrad_pitch(BM), PX = wgrad_pitch(BC);
  constexpr int QE = BM / 4, QX = BC / 4;  // 16-byte groups per pixel
  constexpr int RE = kWTilePix * QE / 256, RX = (kWHaloPix * QX + 255) / 256;
  __shared__ __attribute__((aligned(16))) float smem[kWTilePix * PE + kWHaloPix * PX];
  static_assert((WK - 1) * WM * WN * 9 * 256 <= kWTilePix * PE + kWHaloPix * PX, "row shares must fit in LDS");
  float* s_e = smem;
  float* s_x = smem + kWTilePix * PE;
  const ConvArgs& x = a.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, li = lane & 15;
  const int wm = wave % WM, wn = (wave / WM) % WN, wk = wave / (WM * WN);
  const int tiles_x = (x.W + kTW - 1) / kTW, tiles_y = (x.H + kWTH - 1) / kWTH;
  const int n_tiles = x.B * tiles_x * tiles_y;
  const int o0 = blockIdx.y * BM, c0 = blockIdx.z * BC;

  Halo<MODE> rx[RX];
  f4 re[RE];
  unsigned ok_e = 0, ok_x = 0;
  auto fetch = [&](int t) {
    const int b = t / (tiles_x * tiles_y), r = t - b * tiles_x * tiles_y;
    const int y0 = (r / tiles_x) * kWTH, x0 = (r - (r / tiles_x) * tiles_x) * kTW;
    ok_e = ok_x = 0;
#pragma unroll
    for (int q = 0; q < RE; ++q) {
      const int p = (tid + 256 * q) / QE, o = o0 + 4 * (tid % QE);
      const int y = y0 + p / kTW, xx = x0 + p % kTW;
      ok_e |= (unsigned)(y < x.H && xx < x.W && o < a.co) << q;
      re[q] = *reinterpret_cast<const f4*>(
          a.e + ((size_t)(b * x.H + min(y, x.H - 1)) * x.W + min(xx, x.W - 1)) * a.co + min(o, a.co - 4));
    }
#pragma unroll
    for (int q = 0; q < RX; ++q) {
      const int e = min(tid + 256 * q, kWHaloPix * QX - 1), p = e / QX, c = c0 + 4 * (e % QX);
      const int y = y0 + p / kHW - 1, xx = x0 + p % kHW - 1;
      ok_x |= (unsigned)(y >= 0 && y < x.H && xx >= 0 && xx < x.W && c < a.ci) << q;
      rx[q] = halo_load<MODE>(x, b, min(max(y, 0), x.H - 1), min(max(xx, 0), x.W - 1), c < a.ci ? c : 0);
    }
  };
  f4 bsum = f4{0.f, 0.f, 0.f, 0.f};
  auto commit = [&]() {
#pragma unroll
    for (int q = 0; q < RE; ++q) {
      const f4 v = (ok_e >> q) & 1u ? re[q] : f4{0.f, 0.f, 0.f, 0.f};
      bsum += v;
      *reinterpret_cast<f4*>(&s_e[((tid + 256 * q) / QE) * PE + 4 * (tid % QE)]) = v;
    }
#pragma unroll
    for (int q = 0; q < RX; ++q) {
      const int e = tid + 256 * q;
      if (e < kWHaloPix * QX)
        *reinterpret_cast<f4*>(&s_x[(e / QX) * PX + 4 * (e % QX)]) = halo_value<MODE>(rx[q], (ok_x >> q) & 1u);
    }
  };

  f4 acc[9];
#pragma unroll
  for (int t = 0; t < 9; ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};
  const int t_end = min(n_tiles, (int)(blockIdx.x + 1) * a.tiles_per_group);
  int t = blockIdx.x * a.tiles_per_group;
  if (t < t_end) fetch(t);
  for (; t < t_end; ++t) {
    commit();
    __syncthreads();
    if (t + 1 < t_end) fetch(t + 1);
    constexpr int NR = kWTH / WK;
    const int r0 = wk * NR;
#pragma unroll 1
    for (int cg = 0; cg < kTW / 4; ++cg) {
      const float* pe = s_e + (r0 * kTW + 4 * cg + g) * PE + 16 * wm + li;
      const float* px = s_x + (r0 * kHW + 4 * cg + g) * PX + 16 * wn + li;
      float xr[3][3];
#pragma unroll
      for (int dy = 0; dy < 2; ++dy)
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) xr[dy][dx] = px[(dy * kHW + dx) * PX];
#pragma unroll
      for (int r = 0; r < NR; ++r) {
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) xr[(r + 2) % 3][dx] = px[((r + 2) * kHW + dx) * PX];
        const float av = pe[r * kTW * PE];
#pragma unroll
        for (int tap = 0; tap < 9; ++tap)
          acc[tap] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, xr[(r + tap / 3) % 3][tap % 3], acc[tap], 0, 0, 0);
      }
    }
    __syncthreads();
  }
  end_sums<WM, WN>(a, smem, acc, bsum);
}

__device__ __attribute__((aligned(16))) const float kZeros[4] = {0.f, 0.f, 0.f, 0.f};

// The other layers.  LDS holds, per pixel, the three pieces of each channel
// block in the order they were loaded (channels innermost); the operands,
// which want eight consecutive pixels of one channel per lane, come through
// the transposing LDS read (16 lanes fetch four pixels x 16 channels, lane li
// receives channel li of the four pixels).  A K = 32 step covers two tile
// rows.  X is read once for the three horizontal taps: the order of the
// pixels along K is free as long as E's is the same, so the next tap's
// operand is the last one with its oldest pixel replaced by the newest (half
// a register per tap, where shifting all eight takes four operations), and E
// turns round with it.  The rows of a step's third vertical tap stay in
// registers as the next step's first.
typedef short s4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s4 LdsS4;
typedef unsigned int u4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ u2 read_tr(const uint16_t* p) {
  return __builtin_bit_cast(
      u2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsS4*)(const __attribute__((address_space(3))) uint16_t*)p));
}
// bf16 per pixel: 3 pieces x channels, in 32-channel tiles padded so that the
// four pixels of a transposing read lie on distinct banks (24 words apart mod 32)
constexpr int split_row(int channels) { return channels == 32 ? 112 : 48; }

template <int MODE, int WM, int WN>
__global__ __launch_bounds__(256, 2) void wgrad3x3_split(WgradArgs a) {
  constexpr int WK = 4 / (WM * WN), BM = 16 * WM, BC = 16 * WN;
  constexpr int PE = split_row(BM), PX = split_row(BC);
  constexpr int QE = BM / 4, QX = BC / 4;  // 16-byte groups per pixel
  constexpr int RE = kWTilePix * QE / 256, RX = (kWHaloPix * QX + 255) / 256;
  // the last row's twelve-pixel reads end two pixels past the halo (not used)
  constexpr int kElems = kWTilePix * PE + (kWHaloPix + 2) * PX;
  __shared__ __attribute__((aligned(16))) uint16_t smem[kElems];
  static_assert((WK - 1) * WM * WN * 9 * 64 * 16 <= 2 * kElems && 256 * 16 <= 2 * kElems, "end sums must fit in LDS");
  uint16_t* s_e = smem;
  uint16_t* s_x = smem + kWTilePix * PE;
  const ConvArgs& x = a.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, li = lane & 15;
  const int wm = wave % WM, wn = (wave / WM) % WN, wk = wave / (WM * WN);
  const int tiles_x = (x.W + kTW - 1) / kTW, tiles_y = (x.H + kWTH - 1) / kWTH;
  const int n_tiles = x.B * tiles_x * tiles_y;
  const int o0 = blockIdx.y * BM, c0 = blockIdx.z * BC;

  // The lane's loads as element offsets from the tile's first halo pixel, the
  // same for every tile, and that pixel's place in the halo as (row, column)
  // in the two halves of a word whose top bits guard the differences taken in
  // fetch(); a lane past the halo or the channels never lies in range.
  constexpr unsigned kGuard = 0x80008000u;
  constexpr int S = MODE == G_POOL ? 2 : 1;
  const int cx = c0 + 4 * (tid % QX), oe = o0 + 4 * (tid % QE);
  const bool up = MODE == G_CONCAT_UP && cx >= x.c0;
  const uint32_t row = up ? (uint32_t)(x.W >> 1) * x.c1 : (uint32_t)(S * x.W) * x.c0, col = up ? x.c1 : x.c0;
  uint32_t off[RX], at[RX];
#pragma unroll
  for (int q = 0; q < RX; ++q) {
    const int p = (tid + 256 * q) / QX, py = p / kHW, pxl = p % kHW;
    at[q] = p < kWHaloPix && cx < a.ci ? kGuard | (uint32_t)py << 16 | pxl : kGuard | 0x7fff0000u;
    // the upsampled source: rows and columns (y0 + py - 1) / 2, y0 and x0 even
    off[q] = up ? (uint32_t)((py + 1) >> 1) * row + ((pxl + 1) >> 1) * col + (cx - x.c0)
                : (uint32_t)(S * py) * row + S * pxl * col + cx;
  }
  const int ey = tid / QE / kTW, ex = tid / QE % kTW;
  const uint32_t offe = ((uint32_t)ey * x.W + ex) * a.co + oe;

  // POOL over 32 channels takes its four source pixels per entry in two
  // halves, one per half of the row pairs (all at once they do not fit the
  // registers beside the operands)
  constexpr int kHalf = MODE == G_POOL && WN == 2 ? RX / 2 : RX;
  Halo<MODE> rx[kHalf];
  f4 first_half[RX - kHalf + 1], re[RE];
  unsigned ok = 0;  // POOL: halo pixels inside the image (elsewhere zeros are loaded)
  auto fetch = [&](int t, int half) {
    const int b = t / (tiles_x * tiles_y), r = t - b * tiles_x * tiles_y;
    const int y0 = (r / tiles_x) * kWTH, x0 = (r - (r / tiles_x) * tiles_x) * kTW;
    const float* e0 = a.e + ((size_t)(b * x.H + y0) * x.W + x0) * a.co;
    const bool oke = x0 + ex < x.W && oe < a.co;
    if (half == 0) {
      ok = 0;
#pragma unroll
      for (int q = 0; q < RE; ++q) {
        const float* p = e0 + (size_t)q * (256 / QE / kTW) * x.W * a.co + offe;
        re[q] = *reinterpret_cast<const f4*>(oke && y0 + ey + q * (256 / QE / kTW) < x.H ? p : kZeros);
      }
    }
    const float* s0 = static_cast<const float*>(x.src0) +
                      ((ptrdiff_t)(b * S * x.H + S * (y0 - 1)) * (S * x.W) + S * (x0 - 1)) * x.c0;
    if constexpr (MODE == G_CONCAT_UP) {
      const float* s1 = static_cast<const float*>(x.src1) +
                        ((ptrdiff_t)(b * (x.H >> 1) + (y0 >> 1) - 1) * (x.W >> 1) + (x0 >> 1) - 1) * x.c1;
      s0 = up ? s1 : s0;
    }
    const uint32_t lo = (uint32_t)(y0 == 0) << 16 | (uint32_t)(x0 == 0);
    const uint32_t hi = (uint32_t)min(kWTH + 1, x.H - y0) << 16 | (uint32_t)min(kTW + 1, x.W - x0);
#pragma unroll
    for (int k = 0; k < kHalf; ++k) {
      const int q = half * kHalf + k;
      const bool in = ((at[q] - lo) & ((hi | kGuard) + kGuard - at[q]) & kGuard) == kGuard;
      if constexpr (MODE == G_POOL) {
        // outside: the tile's first pixel, always in the image
        const float* p = s0 + (in ? off[q] : 2 * row + 2 * col + (uint32_t)min(cx, x.c0 - 4));
        ok |= (unsigned)in << q;
        rx[k].v[0] = *reinterpret_cast<const f4*>(p);
        rx[k].v[1] = *reinterpret_cast<const f4*>(p + col);
        rx[k].v[2] = *reinterpret_cast<const f4*>(p + row);
        rx[k].v[3] = *reinterpret_cast<const f4*>(p + row + col);
      } else {
        const float* p = s0 + off[q];
        rx[k].v[0] = *reinterpret_cast<const f4*>(in ? p : kZeros);
      }
    }
  };
  f4 bsum = f4{0.f, 0.f, 0.f, 0.f};
  auto commit = [&]() {
    float over = 0.0f;  // becomes NaN where a value rounds to infinity in bf16 or is none
    auto put = [&](auto safe, uint16_t* row, int channels, f4 v) {
      const Pieces p = split<decltype(safe)::value>(v, over);
      *reinterpret_cast<u2*>(row) = p.hi;
      *reinterpret_cast<u2*>(row + channels) = p.mid;
      *reinterpret_cast<u2*>(row + 2 * channels) = p.lo;
    };
    auto all = [&](auto safe) {
#pragma unroll
      for (int q = 0; q < RE; ++q) put(safe, s_e + ((tid + 256 * q) / QE) * PE + 4 * (tid % QE), BM, re[q]);
#pragma unroll
      for (int q = 0; q < RX; ++q) {
        const int e = tid + 256 * q;
        const bool in = MODE != G_POOL || ((ok >> q) & 1u);
        const f4 v = kHalf < RX && q < kHalf ? first_half[q < kHalf && kHalf < RX ? q : 0]
                                             : halo_value<MODE>(rx[q % kHalf], in);
        if (e < kWHaloPix * QX) put(safe, s_x + (e / QX) * PX + 4 * (e % QX), BC, v);
      }
    };
#pragma unroll
    for (int q = 0; q < RE; ++q) bsum += re[q];
    all(std::false_type{});
    if (__builtin_expect(!(over == over), 0)) all(std::true_type{});
  };

  f4 acc[9];
#pragma unroll
  for (int t = 0; t < 9; ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};
  // a transposing read's address: pixel li / 4 of the four, channels 4 (li % 4)
  // .. + 3; lane group g takes row g / 2 of the step's two, columns 8 (g % 2) .. + 7
  const uint16_t* pe = s_e + ((g >> 1) * kTW + 8 * (g & 1) + (li >> 2)) * PE + 16 * wm + 4 * (li & 3);
  const uint16_t* px = s_x + ((g >> 1) * kHW + 8 * (g & 1) + (li >> 2)) * PX + 16 * wn + 4 * (li & 3);
  // the same for E pixels 6 7 0 1
  const uint16_t* pr = pe + ((li >> 2) < 2 ? 6 : -2) * PE;
  const int t_end = min(n_tiles, (int)(blockIdx.x + 1) * a.tiles_per_group);
  int t = blockIdx.x * a.tiles_per_group;
  auto pool_half = [&]() {
    if constexpr (kHalf < RX) {
#pragma unroll
      for (int q = 0; q < kHalf; ++q) first_half[q] = halo_value<MODE>(rx[q], (ok >> q) & 1u);
    }
  };
  if (t < t_end) {
    fetch(t, 0);
    if constexpr (kHalf < RX) {
      pool_half();
      fetch(t, 1);
    }
  }
  for (; t < t_end; ++t) {
    commit();
    __syncthreads();
    if (t + 1 < t_end) fetch(t + 1, 0);
    constexpr int NR = kWTH / 2 / WK;  // row pairs per wavefront
    u4 xv[3][3], ev[3], er[3];  // [dy][piece]
    uint32_t x0[3], x8[3][3];
    auto read_e = [&](const uint16_t* p0, const uint16_t* p1, int rp, int q) {
      const u2 e0 = read_tr(p0 + 2 * rp * kTW * PE + q * BM), e1 = read_tr(p1 + 2 * rp * kTW * PE + q * BM);
      return u4{e0.x, e0.y, e1.x, e1.y};
    };
#pragma unroll
    for (int rk = 0; rk < NR; ++rk) {
      if constexpr (kHalf < RX) {
        if (rk == NR / 2 && t + 1 < t_end) {
          pool_half();
          fetch(t + 1, 1);
        }
      }
      const int rp = wk * NR + rk;
#pragma unroll
      for (int q = 0; q < 3; ++q) ev[q] = read_e(pe, pe + 4 * PE, rp, q);
      if (rk > 0) {  // the rows of the last step's third tap
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          xv[0][q] = u4{x0[q], xv[2][q].y, xv[2][q].z, xv[2][q].w};
          x8[0][q] = x8[2][q];
        }
      }
#pragma unroll
      for (int dy = rk > 0; dy < 3; ++dy)
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          const uint16_t* p = px + (2 * rp + dy) * kHW * PX + q * BC;
          const u2 b0 = read_tr(p), b1 = read_tr(p + 4 * PX), b2 = read_tr(p + 8 * PX);
          xv[dy][q] = u4{b0.x, b0.y, b1.x, b1.y};
          x8[dy][q] = b2.x;
        }
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        er[q] = read_e(pr, pe + 2 * PE, rp, q);
        x0[q] = xv[2][q].x;
      }
      auto products = [&](int dx) {
#pragma unroll
        for (int dy = 0; dy < 3; ++dy)
#pragma unroll
          for (int k = 0; k < 6; ++k)
            acc[3 * dy + dx] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(bf16x8, ev[kSplitTerm[k][0]]),
                __builtin_bit_cast(bf16x8, xv[dy][kSplitTerm[k][1]]), acc[3 * dy + dx], 0, 0, 0);
      };
      products(0);
#pragma unroll
      for (int q = 0; q < 3; ++q) {  // E pixels 7 0 1 .. 6, X pixels 8 1 2 .. 7
        const u4 e = ev[q];
        ev[q] = u4{__builtin_amdgcn_alignbit(e.x, e.w, 16), __builtin_amdgcn_alignbit(e.y, e.x, 16),
                   __builtin_amdgcn_alignbit(e.z, e.y, 16), __builtin_amdgcn_alignbit(e.w, e.z, 16)};
#pragma unroll
        for (int dy = 0; dy < 3; ++dy) xv[dy][q].x = (xv[dy][q].x & 0xffff0000u) | (x8[dy][q] & 0xffffu);
      }
      products(1);
#pragma unroll
      for (int q = 0; q < 3; ++q) {  // E pixels 6 7 0 .. 5, X pixels 8 9 2 .. 7
        ev[q] = er[q];
#pragma unroll
        for (int dy = 0; dy < 3; ++dy) xv[dy][q].x = x8[dy][q];
      }
      products(2);
    }
    __syncthreads();
  }
  end_sums<WM, WN>(a, smem, acc, bsum);
}

// Finish a layer's weight and bias gradients: each sum over the groups'
// partials by eight lanes (every eighth group each, then added in order), 32
// neighbouring sums per block, so that layers with few weights and many
// groups still fill the chip.
__global__ __launch_bounds__(256) void wgrad_reduce(WgradArgs a, int groups, int w_blocks) {
  __shared__ float sh[8][32];
  const int el = threadIdx.x & 31, rl = threadIdx.x >> 5;
  const bool bias = (int)blockIdx.x >= w_blocks;
  const size_t n = bias ? (size_t)a.co_pad : (size_t)a.co_pad * 9 * a.ci_pad;
  const size_t e = (size_t)(bias ? blockIdx.x - w_blocks : blockIdx.x) * 32 + el;
  const float* src = (bias ? a.bias_partial : a.partial) + e;
  float s = 0.0f;
  if (e < n) {
    int k = rl;
    for (; k + 24 < groups; k += 32) {
      float v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = src[(size_t)(k + 8 * u) * n];
#pragma unroll
      for (int u = 0; u < 4; ++u) s += v[u];
    }
    for (; k < groups; k += 8) s += src[(size_t)k * n];
  }
  sh[rl][el] = s;
  __syncthreads();
  if (rl || e >= n) return;
#pragma unroll
  for (int k = 1; k < 8; ++k) s += sh[k][el];
  if (bias) {
    if ((int)e < a.co) a.grad_b[e] = s;
    return;
  }
  const int c = (int)(e % a.ci_pad), tap = (int)((e / a.ci_pad) % 9), o = (int)(e / ((size_t)9 * a.ci_pad));
  if (o < a.co && c < a.ci) a.grad_w[((size_t)o * a.ci + c) * 9 + tap] = s;
}

template <int MODE>
hipError_t launch_wgrad_mode(const WgradArgs& a, const WgradTiling& t, hipStream_t s) {
  const dim3 grid(t.groups, t.co_pad / (16 * t.wm), t.ci_pad / (16 * t.wn));
  if constexpr (MODE == G_GUIDE) {
    if (t.wn != 1) return hipErrorInvalidValue;
    if (t.wm == 2)
      hipLaunchKernelGGL(wgrad_first_f32<2>, grid, dim3(256), 0, s, a);
    else
      hipLaunchKernelGGL(wgrad_first_f32<1>, grid, dim3(256), 0, s, a);
  } else {
    if (t.wm == 2 && t.wn == 2)
      hipLaunchKernelGGL((wgrad3x3_split<MODE, 2, 2>), grid, dim3(256), 0, s, a);
    else if (t.wm == 2)
      hipLaunchKernelGGL((wgrad3x3_split<MODE, 2, 1>), grid, dim3(256), 0, s, a);
    else if (t.wn == 2)
      hipLaunchKernelGGL((wgrad3x3_split<MODE, 1, 2>), grid, dim3(256), 0, s, a);
    else
      hipLaunchKernelGGL((wgrad3x3_split<MODE, 1, 1>), grid, dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_wgrad3x3(int mode, const WgradArgs& a0, hipStream_t s) {
  WgradArgs a = a0;
  const WgradTiling t = wgrad_tiling(a.co, a.ci, a.x.B, a.x.H, a.x.W);
  a.co_pad = t.co_pad;
  a.ci_pad = t.ci_pad;
  a.tiles_per_group = t.tiles_per_group;
  hipError_t e;
  switch (mode) {
    case G_GUIDE: e = launch_wgrad_mode<G_GUIDE>(a, t, s); break;
    case G_PLAIN: e = launch_wgrad_mode<G_PLAIN>(a, t, s); break;
    case G_POOL: e = launch_wgrad_mode<G_POOL>(a, t, s); break;
    case G_CONCAT_UP: e = launch_wgrad_mode<G_CONCAT_UP>(a, t, s); break;
    default: return hipErrorInvalidValue;
  }
  if (e != hipSuccess) return e;
  const unsigned w_blocks = (unsigned)(((size_t)t.co_pad * 9 * t.ci_pad + 31) / 32), b_blocks = (t.co_pad + 31) / 32;
  hipLaunchKernelGGL(wgrad_reduce, dim3(w_blocks + b_blocks), dim3(256), 0, s, a, t.groups, (int)w_blocks);
  return hipGetLastError();
}

}  // namespace lnm
