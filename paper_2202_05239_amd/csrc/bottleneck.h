// The 3x3 layer of a bottleneck block, the 1x1 layer that closes the block (with its residual) and, where it follows, the
// 1x1 layer that opens the next block, in one kernel.  See bottleneck.hip.
#pragma once

#include "f8_device.h"

namespace f8 {

struct BottleneckParams {
  const uint8_t *x;        // [B][H][W][C]: input of the 3x3 layer (pad 1)
  const int8_t *wf;        // weights of all layers in the order the waves take them, and the start values (launch_bottleneck_weights)
  const uint8_t *res;      // [B][P][Q][4 C] residual of the closing layer, 8 bits, or null
  const uint8_t *xp;       // [B][Hp][Wp][PC] input of a projection whose result is the residual instead (res: null), or null
  uint8_t *y, *y2;         // [B][P][Q][4 C] the closing layer's output, and in a second format (or null)
  uint8_t *ya;             // [B][P][Q][NA] output of the layer behind it
  int B, H, W, C, P, Q, stride;
  int NA;                  // channels of the layer behind: 0 (none), C or 2 C
  uint32_t x_xor, b_xor, y_xor;   // 0x80808080 where x / the 3x3 layer's result / y is unsigned
  int shift_b, lo_b, hi_b;        // requantisation (shifts >= 0)
  int shift_c, lo_c, hi_c;
  int shift_2, lo_2, hi_2, add_2; // second format: add_2 swaps the rounding addend
  int shift_a, lo_a, hi_a;
  int res_signed, res_d;          // res_d >= 0; also of the projection's result
  int Hp, Wp, PC, sp;             // the projection: 1x1, stride sp
  uint32_t xp_xor;
  int shift_p, lo_p, hi_p;
  int force;                      // tuning aid: see bottleneck_wide
};

// Channel counts, geometry and shifts the kernel takes (NA: 0, C or 2 C).
bool bottleneck_applicable(int C, int H, int W, int stride, int NA, int shift_b, int shift_c, int shift_a, int shift_2, int res_d);
// Whether it takes a projection of PC channels and stride ps along (as bottleneck_applicable says yes to the rest).
bool bottleneck_projects(int C, int H, int W, int stride, int NA, int PC, int ps);
// Whether a launch takes the wider of the two tiles (force: 3 never, 4 wherever it fits).
bool bottleneck_wide(int C, int H, int W, int stride, int B, int force, bool projection);
size_t bottleneck_weight_bytes(int C, int NA, int PC);
// wb: [C][3][3][C], wc: [4 C][C], wa: [NA][4 C] (or null), wp: [4 C][PC] (or null); acc_*: the layers' folded start values; res_bias: 128 << res_d
// where the residual is unsigned, else 0.  A hipError_t as int.
int launch_bottleneck_weights(const int8_t *wb, const int8_t *wc, const int8_t *wa, const int8_t *wp, const int32_t *acc_b, const int32_t *acc_c,
                              const int32_t *acc_a, const int32_t *acc_p, int8_t *wf, int C, int NA, int PC, int res_bias, hipStream_t stream);
int launch_bottleneck(const BottleneckParams &p, hipStream_t stream);

}  // namespace f8
