// The fp32 3x3 convolutions' gather of their (virtual) input: zero padding, the
// encoder's 2x2 max-pool, the decoder's upsample + concatenation (device code
// only).
#pragma once
#include "internal.h"

namespace lnm {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kTW = 16;        // tile width in pixels (= the MFMA's 16)
constexpr int kHW = kTW + 2;   // halo width

// Raw loads of one halo entry (four channels at pixel (y, x), both clamped
// into the image): the pooled mode keeps its four source pixels, the others
// one value.  They are combined and masked only when written to LDS, so the
// loads of a chunk are all in flight together and nothing waits on them
// before the matrix work of the current chunk.
template <int MODE>
struct Halo {
  f4 v[MODE == G_POOL ? 4 : 1];
};

template <int MODE>
__device__ __forceinline__ Halo<MODE> halo_load(const ConvArgs& a, int b, int y, int x, int c) {
  const float* s0 = static_cast<const float*>(a.src0);
  Halo<MODE> h;
  if constexpr (MODE == G_GUIDE) {
    const float* g = s0 + ((size_t)(b * a.H + y) * a.W + x) * 3;
    h.v[0] = f4{g[0], g[1], g[2], 0.0f};
  } else if constexpr (MODE == G_PLAIN) {
    h.v[0] = *reinterpret_cast<const f4*>(s0 + ((size_t)(b * a.H + y) * a.W + x) * a.c0 + c);
  } else if constexpr (MODE == G_POOL) {
    const size_t W2 = 2 * (size_t)a.W, c0 = (size_t)a.c0;
    const float* p = s0 + ((size_t)(b * 2 * a.H + 2 * y) * W2 + 2 * x) * c0 + c;
    h.v[0] = *reinterpret_cast<const f4*>(p);
    h.v[1] = *reinterpret_cast<const f4*>(p + c0);
    h.v[2] = *reinterpret_cast<const f4*>(p + W2 * c0);
    h.v[3] = *reinterpret_cast<const f4*>(p + W2 * c0 + c0);
  } else {  // G_CONCAT_UP: channels [0, c0) from the skip, then the upsampled low-res tensor
    const int Hl = a.H >> 1, Wl = a.W >> 1;
    const float* skip = s0 + ((size_t)(b * a.H + y) * a.W + x) * a.c0 + c;
    const float* up = static_cast<const float*>(a.src1) + ((size_t)(b * Hl + (y >> 1)) * Wl + (x >> 1)) * a.c1 +
                      max(c - a.c0, 0);
    h.v[0] = *reinterpret_cast<const f4*>(c < a.c0 ? skip : up);
  }
  return h;
}

template <int MODE>
__device__ __forceinline__ f4 halo_value(const Halo<MODE>& h, bool ok) {
  f4 v = h.v[0];
  if constexpr (MODE == G_POOL) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = fmaxf(fmaxf(h.v[0][e], h.v[1][e]), fmaxf(h.v[2][e], h.v[3][e]));
  }
  return ok ? v : f4{0.f, 0.f, 0.f, 0.f};
}

}  // namespace lnm
