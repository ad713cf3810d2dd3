// Dense layers that conv_fast does not take, with many tiles: four waves share a tile's area.  See conv_igemm.hip.
#pragma once

#include "conv_params.h"

namespace f8 {

// The widest of 16, 4, 1 bytes that divides the channel count and the alignment of x and w: a gather unit.
int conv_igemm_vec(const ConvParams &p);
// Name of the kernel for N output channels.
const char *conv_igemm_name(int N);
// Any shape, type and alignment.  fold: form the accumulator start values here, from `bias` (may be null); p.acc0 and
// p.zero are not read then.  A hipError_t as int.
int launch_conv_igemm(const ConvParams &p, bool fold, const int32_t *bias, hipStream_t stream);

}  // namespace f8
