// Image-stationary 3x3 convolution, stride 2, pad 1, C -> N channels (C = 64, 128, 256), and the 1x1 stride-2 layer on the same
// input beside it (the shortcut projection of a basic residual block), in one launch.  See conv_s2.hip.
#pragma once

#include "f8_device.h"

namespace f8 {

struct ConvS2Params {
  const uint8_t *x;      // [B][H][W][C]
  const int8_t *w;       // launch_conv_s2_weights, 9 taps
  const int32_t *acc0;   // [N] folded accumulator start values
  uint8_t *y;            // [B][P][Q][N], unsigned or signed bytes
  const int32_t *acc0p;  // the 1x1 layer's, or null: none
  const int8_t *wp;      // its weights: launch_conv_s2_weights, one tap
  uint8_t *yp;           // its output, of y's shape
  int B, H, W, C, N;
  int shift, lo, hi;     // requantisation (shift >= 0)
  int shiftp, lop, hip;
  uint32_t x_xor;        // 0x80808080 when x is unsigned
  int wk;                // waves that share K: 1, 2 or 4, up to conv_s2_most_waves(C)
};

// Geometry and operand checks.
bool conv_s2_applicable(int Cin, int Cout, int R, int S, int sh, int sw, int ph, int pw, int H, int W, int shift, const void *x, const void *y);
int conv_s2_most_waves(int C);
// Whether images of this size fill the accumulators of a workgroup to two thirds at least.
bool conv_s2_fills(int C, int H, int W);
// Workgroups of a launch with wk waves sharing K.
long long conv_s2_workgroups(int C, int N, int B, int H, int W, int wk);
// [N][taps][C] weights into the order the kernel streams them in.  A hipError_t as int.
int launch_conv_s2_weights(const int8_t *w, int8_t *wf, int taps, int C, int N, hipStream_t stream);
// A hipError_t as int.
int launch_conv_s2(const ConvS2Params &p, hipStream_t stream);

}  // namespace f8
