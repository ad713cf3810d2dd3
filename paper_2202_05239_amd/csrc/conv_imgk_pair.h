// Two 3x3 layers of 64 or 128 channels, one behind the other, with the first one's input as the second one's shortcut (a
// basic residual block) in one launch.  See conv_imgk_pair.hip.
#pragma once

#include "f8_device.h"

namespace f8 {

struct ConvPairParams {
  const uint8_t *x;                // [B][H][W][C]
  const int8_t *wa, *wb;           // weights in fragment order (launch_conv_img_weights)
  const int32_t *acc_a, *acc_b;    // [C] folded start values
  uint8_t *y;                      // [B][H][W][C]
  int B, H, W, C;
  uint32_t x_xor, e_xor;           // 0x80808080 where x / the first result is unsigned
  int shift_a, lo_a, hi_a;         // requantisation (shifts >= 0)
  int shift_b, lo_b, hi_b;
  int has_res, res_d;              // x is the second layer's residual, res_d >= 0
};

bool conv_pair_applicable(int C, int H, int W, int shift_a, int shift_b, bool has_res, int res_d, const void *x, const void *y);
// A hipError_t as int.
int launch_conv_pair(const ConvPairParams &p, hipStream_t stream);

}  // namespace f8
