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
// Whether images of this size fill the accumulators of a workgroup to two thirds at least.  Below that the best number of
// waves against the best other kernel measures, in us, at 64, 128, 256 images: 256 channels on 12 x 12 (64 % full) 11.1 / 15.9,
// 15.4 / 20.7, 25.7 / 25.9; 10 x 10 (45 %) 10.5 / 12.8, 14.6 / 15.5, 24.0 / 21.5; 8 x 8 8.5 / 7.5, 11.1 / 13.2, 15.0 / 16.2; 512 on 5 x 5 11.0 /
// 9.9, 15.9 / 22.0, 27.2 / 26.3; 128 on 16 x 16 8.3 / 8.5, 9.9 / 10.1, 15.4 / 16.8: ahead at some batches and behind at others; the
// line lies above all of them.
bool conv_imgk_fills(int C, int H, int W);
// Workgroups of a launch with wk waves sharing K.
long long conv_imgk_workgroups(int C, int B, int H, int W, int wk);
// A hipError_t as int.
int launch_conv_imgk(const ConvImgkParams &p, hipStream_t stream);

}  // namespace f8
