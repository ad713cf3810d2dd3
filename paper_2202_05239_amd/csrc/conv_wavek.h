// Dense layers whose output is too small to fill the chip with GEMM tiles: small tiles, the K range of a
// tile shared out among the waves of its workgroup.  Also any channel count and alignment.  See
// conv_wavek.hip.
#pragma once

#include "conv_params.h"

namespace f8 {

// Tile shapes (output pixels x channels, waves that share K).
enum { WK_32x32_W8 = 0, WK_32x32_W4 = 1, WK_64x32_W8 = 2, WK_64x64_W8 = 3, WK_VARIANTS = 4 };

// x and w can be fetched in 16-byte units (whole channels of one tap, 16-byte aligned); otherwise the kernel
// gathers them.  It can take every layer the entry points accept.
bool conv_wavek_direct(const ConvParams &p);
// The tile shape for this layer; -1 where another kernel is the faster one: conv_fast or, for layers that it does
// not take (general), conv_igemm.
int conv_wavek_variant(const ConvParams &p, bool general);
const char *conv_wavek_name(int variant, bool direct);
// fold == false: p.acc0 holds the folded start values.  fold == true: the kernel forms them itself from the
// weights and the bias (null for none); p.acc0 is not read.  A hipError_t as int.
int launch_conv_wavek(const ConvParams &p, int variant, bool fold, const int32_t *bias, hipStream_t stream);

}  // namespace f8
