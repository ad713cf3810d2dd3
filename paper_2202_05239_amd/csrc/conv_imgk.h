// Image-stationary 3x3 convolution, stride 1, pad 1, C -> C channels (C = 64, 128, 256, 512), for batches that
// give the chip one or two workgroups per CU: K shared among the waves.  See conv_imgk.hip.
#pragma once

#include "f8_device.h"

namespace f8 {

struct ConvImgkParams {
  const uint8_t *x;      // [B][H][W][C]
  const int8_t *w;       // weights in fragment order (launch_conv_img_weights); fold: [C][3][3][C]
  const int32_t *acc0;   // [C] folded accumulator start values; fold: the bias, or null
  uint8_t *y;            // [B][H][W][C], unsigned or signed bytes
  const uint8_t *res;    // residual of y's shape, 8 bits, or null
  int B, H, W, C;
  int shift, lo, hi;     // requantisation (shift >= 0)
  uint32_t x_xor;        // 0x80808080 when x is unsigned
  int res_signed, res_d;
  int wk;                // waves that share K: 1, 2 or 4, up to conv_imgk_most_waves(C)
  int fold;              // 1 (64 channels only): form the start values here
};

// Geometry and operand checks.
bool conv_imgk_applicable(int Cin, int Cout, int R, int S, int sh, int sw, int ph, int pw, int H, int W, int shift,
                          const void *x, const void *y, const void *res);
int conv_imgk_most_waves(int C);
// Whether images of this size fill the accumulators of a workgroup to two thirds at least.
bool conv_imgk_fills(int C, int H, int W);
// Workgroups of a launch with wk waves sharing K.
long long conv_imgk_workgroups(int C, int B, int H, int W, int wk);
// A hipError_t as int.
int launch_conv_imgk(const ConvImgkParams &p, hipStream_t stream);

}  // namespace f8
