// U-Net 3x3 convolutions (Section 4.3) in bf16 on the gfx950 matrix cores
// (v_mfma_f32_16x16x32_bf16, fp32 accumulation).  Activations and weights
// are bf16 (round to nearest even), bias and ReLU are applied to the fp32
// accumulator, and the result is rounded to bf16 once.  The 3-channel input
// layer packs all 27 (tap, channel) pairs of its 3x3 window into one 32-wide
// K step and runs within the second layer's launch.
#include "conv_low.h"
#include "internal.h"

namespace lnm {

hipError_t launch_conv3x3_bf16(int mode, const ConvArgs& a, hipStream_t s, const HeadFuse* head) {
  return low::launch<low::Bf16>(mode, a, s, head);
}

}  // namespace lnm
