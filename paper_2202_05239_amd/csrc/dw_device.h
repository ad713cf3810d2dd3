// Device-side pieces of the depthwise kernels: byte transposes, packed dot products, clip and shift-into-byte.
#pragma once

#include "f8_device.h"

namespace f8 {

__device__ __forceinline__ uint32_t perm(uint32_t hi, uint32_t lo, uint32_t sel) {
  return __builtin_amdgcn_perm(hi, lo, sel);
}

// (a, b, c, d) = 4 pixels x 4 channels  ->  t[ch] = bytes (a.ch, b.ch, c.ch, d.ch)
__device__ __forceinline__ void transpose4(uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint32_t t[4]) {
  const uint32_t ab_lo = perm(b, a, 0x05010400u), ab_hi = perm(b, a, 0x07030602u);
  const uint32_t cd_lo = perm(d, c, 0x05010400u), cd_hi = perm(d, c, 0x07030602u);
  t[0] = perm(cd_lo, ab_lo, 0x05040100u);
  t[1] = perm(cd_lo, ab_lo, 0x07060302u);
  t[2] = perm(cd_hi, ab_hi, 0x05040100u);
  t[3] = perm(cd_hi, ab_hi, 0x07060302u);
}

// clamp with lo <= hi as one instruction
__device__ __forceinline__ int med3(int v, int lo, int hi) {
  int r;
  asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(v), "v"(lo), "v"(hi));
  return r;
}

// The same clamp for a value that a packed dot product has just written: a different kind of vector
// instruction may read such a result only three wait states later, and the compiler, which inserts
// those waits for its own instructions, cannot see into an asm statement.
__device__ __forceinline__ int med3_after_dot(int v, int lo, int hi) {
  int r;
  asm("s_nop 2\n\tv_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(v), "v"(lo), "v"(hi));
  return r;
}

// d = dot4(a, b) + c with a destination of its own (the builtin's accumulate-in-place form
// needs a copy of the start value first)
__device__ __forceinline__ int dot4_from(uint32_t a, uint32_t b, int c) {
  int r;
  asm("v_dot4_i32_i8 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// acc >> shift written into byte BYTE of dst, the other bytes kept: the arithmetic shift and the
// packing of four results into one dword are one instruction (sub-dword addressing of the
// destination).  acc has been clamped to [lo << shift, ((hi + 1) << shift) - 1] before, so the
// shifted value is the clipped output and its low byte is all of it.  A vector instruction that
// reads a register right after a sub-dword write to it needs one wait state on this chip; the
// compiler cannot see into the asm statement, so the wait is part of it.  Byte 0 goes first and
// clears the rest of dst; the shift count is uniform (a scalar register).
template <int BYTE>
__device__ __forceinline__ void shift_into_byte(uint32_t &dst, int acc, int shift) {
  if (BYTE == 0) asm("v_ashrrev_i32_sdwa %0, %1, %2 dst_sel:BYTE_0 dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:DWORD\n\ts_nop 0" : "=v"(dst) : "s"(shift), "v"(acc));
  if (BYTE == 1) asm("v_ashrrev_i32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD\n\ts_nop 0" : "+v"(dst) : "s"(shift), "v"(acc));
  if (BYTE == 2) asm("v_ashrrev_i32_sdwa %0, %1, %2 dst_sel:BYTE_2 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD\n\ts_nop 0" : "+v"(dst) : "s"(shift), "v"(acc));
  if (BYTE == 3) asm("v_ashrrev_i32_sdwa %0, %1, %2 dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD\n\ts_nop 0" : "+v"(dst) : "s"(shift), "v"(acc));
}

}  // namespace f8
