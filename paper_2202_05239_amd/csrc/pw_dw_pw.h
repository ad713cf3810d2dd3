// 1x1 layer, the depthwise 3x3 layer that is its only reader and the 1x1 layer that is that one's only reader (an
// inverted-residual block) in one kernel.  See pw_dw_pw.hip.
#pragma once

#include "f8_device.h"

namespace f8 {

struct PwDwPwParams {
  const uint8_t *x;        // [B][H][W][Cin]
  const int8_t *w1;        // first layer's weights in fragment order (launch_dw_pw_weights of Ce x Cin)
  const int8_t *consts;    // depthwise weights and all start values (launch_pw_dw_pw_consts)
  const int8_t *w2;        // last layer's weights in fragment order (launch_dw_pw_weights of Cout x Ce)
  uint8_t *y;              // [B][P][Q][Cout]
  int B, H, W, P, Q, stride, Cin, Ce, Cout;
  uint32_t x_xor, e_xor, d_xor;   // 0x80808080 where x / the first / the depthwise result is unsigned
  int shift1, lo1, hi1;           // requantisation (shifts >= 0)
  int shiftd, lod, hid;
  int shift2, lo2, hi2;
  int H0;                         // launch_image_dw_pw: rows of x, [B][H0][2 W][3]; else not read
  int has_res, res_d;             // the block's input is the last layer's residual (stride 1, Cin = Cout), res_d >= 0
};

// Channel counts, image size, shifts and the alignment of y that the kernel takes.
bool pw_dw_pw_applicable(int Cin, int Ce, int Cout, int H, int W, int stride, int shift1, int shiftd, int shift2, bool has_res, int res_d,
                         const void *x, const void *y);
// Whether it is ahead, for a batch of B, of three launches or (pair) of two, the first layer and the pair behind it.
bool pw_dw_pw_pays(int Cin, int Ce, int Cout, int H, int W, int stride, int B, bool pair);
size_t pw_dw_pw_const_bytes(int Ce, int Cout);
// wd: [3][3][Ce]; acc1, accd, acc2: folded start values of the three layers, [channels to 32]; res_bias: 128 << res_d where the
// shortcut is unsigned, else 0.
int launch_pw_dw_pw_consts(const int8_t *wd, const int32_t *acc1, const int32_t *accd, const int32_t *acc2, int8_t *to, int Ce, int Cout, int res_bias,
                           hipStream_t stream);
// A hipError_t as int.
int launch_pw_dw_pw(const PwDwPwParams &p, hipStream_t stream);

// The same where the first layer is a 3x3 layer of stride 2 and padding 1 on an H x W image of three channels (its weights: launch_dw_pw_weights of
// Ce x [3][4][4], the fourth pixel and channel zeros).
bool image_dw_pw_applicable(int Ce, int Cout, int H, int W, int stride, int shift1, int shiftd, int shift2, const void *x, const void *y);
int launch_image_dw_pw(const PwDwPwParams &p, hipStream_t stream);

}  // namespace f8
