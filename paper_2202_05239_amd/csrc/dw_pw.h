// Depthwise 3x3 layer (pad 1, stride 1 or 2) and the 1x1 layer that reads it, in one kernel.  See dw_pw.hip.
#pragma once

#include "f8_device.h"

namespace f8 {

struct DwPwParams {
  const uint8_t *x;        // [B][H][W][C]
  const int8_t *wd;        // [3][3][C]
  const int32_t *bias;     // [C] or null: the depthwise layer's
  const int8_t *wf;        // the 1x1 layer's weights in fragment order (launch_dw_pw_weights)
  const int32_t *acc0;     // [N] its folded start values
  uint8_t *y;              // [B][P][Q][N]
  const uint8_t *res;      // residual of y's shape, 8 bits, or null
  int B, H, W, C, N, P, Q, stride;
  uint32_t x_xor, d_xor;   // 0x80808080 when x / the depthwise result is unsigned
  int d_shift, d_lo, d_hi; // depthwise requantisation (shift >= 0)
  int shift, lo, hi;       // the 1x1 layer's (shift >= 0)
  int res_signed, res_d;
};

// Geometry, types and alignment of the pair.
bool dw_pw_applicable(int C, int N, int Q, int d_shift, int shift, const void *x, const void *wd, const void *y, const void *res);
// Slices of 32 input channels that a wave of the 1x1 part works through one after the other.
int dw_pw_slices(int C, int N);
size_t dw_pw_weight_bytes(int C, int N);
int launch_dw_pw_weights(const int8_t *w, int8_t *wf, int C, int N, hipStream_t stream);
// A hipError_t as int.
int launch_dw_pw(const DwPwParams &p, hipStream_t stream);

}  // namespace f8
