// Fused ImageNet stem: 7x7 stride-2 convolution of a 3-channel image to 64 channels, unsigned requantisation and the
// 3x3 stride-2 pad-1 max pool behind it.
#pragma once

#include "f8_device.h"

namespace f8 {

struct StemPoolParams {
  const uint8_t *x;      // [B][H][W][3], any alignment (whole dwords that hold bytes of an image are read)
  const int8_t *wp;      // [64][7][8][4], zeros in the first tap and the fourth channel
  const int32_t *acc0;   // [64] folded accumulator start values (bias, rounding addend, sign correction)
  uint8_t *y;            // [B][PP][QP][64] pooled output
  int B, H, W;
  uint32_t x_xor;        // 0x80808080 for unsigned images
  int P, Q;              // convolution output size
  int PP, QP;            // pooled size: (P - 1) / 2 + 1, (Q - 1) / 2 + 1
  int shift, lo, hi;     // requantisation of the convolution (shift >= 0, 0 <= lo <= hi <= 255)
  int ntiles;            // filled in by launch_stem_pool
  FastDiv fd_tiles, fd_tj;
};

// The layer geometry the kernel is built for (Sp = taps per re-laid-out window row).
bool stem_pool_applicable(int Cout, int R, int S, int sh, int sw, int ph, int pw, int Sp);
// Checks the remaining assumptions (sizes, alignment) and launches; a hipError_t as int.
int launch_stem_pool(StemPoolParams p, hipStream_t stream);

}  // namespace f8
