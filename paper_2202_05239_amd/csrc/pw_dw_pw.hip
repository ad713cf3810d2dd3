// An inverted-residual block (1x1 layer to Ce channels, depthwise 3x3 layer with stride 1 or 2, 1x1 layer back, identity
// shortcut), F8Net Eq. 6 three times, in one launch.
//
// At small and medium batch the block's launches are bound by what a launch costs beyond its work (1.6 to 2.4 us behind
// another one, cold operands, one wave's serial chain).  A workgroup of eight waves takes a few output rows of an image with
// all channels: it computes the expanded rows under them (the rows above and below are computed by the neighbours
// too: that is the price), keeps them in LDS with a border of zeros, runs the depthwise layer on them and the last layer on
// that; only the block's input is read and its output written.
//
// The depthwise layer runs on the matrix cores: for 32 channels and one tap the left operand is the diagonal matrix of the
// tap's weights (each lane masks its row's byte out of a replicated one), the right operand the pixels the tap meets, so a
// block of 32 pixels x 32 channels takes nine matrix instructions on fragments that lie in LDS as they are.  The packed dot products
// of dw_pw.hip need the bytes of neighbouring pixels side by side first: nine vector instructions per result where
// this has six, of which none waits for a transposition.
//
// The front of a network (3x3 stride-2 layer on an image of three channels, depthwise layer, 1x1 layer) has a kernel of its own
// below, with at most 32 channels in the middle.
#include "pw_dw_pw.h"

#include <atomic>

namespace f8 {
namespace {

typedef int v16i __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) uint8_t lds_u8;
typedef __attribute__((address_space(3))) v4i lds_v4i;
typedef __attribute__((address_space(3))) v2i lds_v2i;
typedef __attribute__((address_space(3))) uint32_t lds_u32;

constexpr int NT = 512, NWAVE = NT / 64;
constexpr int PART_PITCH = 32 * 4 + 16;

// Division by a divisor that is known anyway.
struct Div {
  uint32_t mul, shr;
  Div() = default;
  __host__ explicit Div(int d) { const FastDiv f((uint32_t)d); mul = f.mul; shr = f.shr; }
  __device__ __forceinline__ int of(int n) const { return (int)(__umulhi((uint32_t)n << 1, mul) >> shr); }
};

// What a launch needs, all of it loaded at once: a wave alone on its SIMD waits for every load of an argument.
struct Args {
  const uint8_t *x;
  const int8_t *w1, *consts, *w2;
  uint8_t *y;
  int x_bytes, w1_bytes, const_bytes;
  int H, W, P, Q, stride, c8, cout;    // c8: 8-byte pieces per input pixel
  int rows, bands;           // output rows per workgroup, workgroups per image
  int nb1, nb3;              // 32-channel blocks of Ce, Cout
  int mb1, mb2;              // most blocks of 32 pixels: of expanded rows, of output rows
  int m1, g1, m2, g2;        // in the first two layers: pixel blocks side by side, waves per pixel block
  int xp, ep;                // bytes of a pixel in LDS: input; expanded and depthwise result
  int at_const, at_e, at_d;  // LDS offsets (the input rows lie at 0)
  int kg;                    // waves that share the last layer's K
  int has_res, res_d;
  uint32_t x_xor, e_xor, d_xor;
  ScaledClip clip1, clipd;
  int shift1, shiftd, shift2, lo2, hi2;
  Div by_bands, by_m1, by_m2, by_w, by_q, by_c8, by_pe, by_np, by_u3, by_nb3;
};

// Behind the depthwise taps of a launch's constants: start values of the three layers.
__host__ __device__ constexpr int tap_bytes(int nb1) { return nb1 * 32 * 9 * 4; }

__device__ __forceinline__ v4i lds_read(uint32_t at) { return *(lds_v4i *)(uintptr_t)at; }
__device__ __forceinline__ void lds_write(uint32_t at, v4i v) { *(lds_v4i *)(uintptr_t)at = v; }

// 16 accumulators of a lane, already holding the rounding addend, to 16 bytes, in signed form.
__device__ __forceinline__ v4i requant16(v16i &a, ScaledClip c, int shift, int x) {
  settle_matrix_result(a);
  int v[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = clamp_med3(a[i], c.lo, c.hi);
  const v4i r = shift_pack16(v, shift);
  return v4i{r.x ^ x, r.y ^ x, r.z ^ x, r.w ^ x};
}

template <int KS1>
__global__ __launch_bounds__(NT, 2) void pw_dw_pw_kernel(const Args a) {
  pin_args(a.x, a.w1, a.consts, a.w2, a.y, a.x_bytes, a.w1_bytes, a.const_bytes, a.H, a.W, a.P, a.Q, a.stride, a.c8, a.cout, a.rows, a.bands,
           a.nb1, a.nb3, a.mb1, a.mb2, a.m1, a.g1, a.m2, a.g2, a.xp, a.ep, a.at_const, a.at_e, a.at_d, a.kg, a.has_res, a.res_d, a.x_xor, a.e_xor, a.d_xor, a.clip1.lo,
           a.clip1.hi, a.clipd.lo, a.clipd.hi, a.shift1, a.shiftd, a.shift2, a.lo2, a.hi2, a.by_bands.mul, a.by_bands.shr, a.by_m1.mul,
           a.by_m1.shr, a.by_m2.mul, a.by_m2.shr, a.by_w.mul, a.by_w.shr, a.by_q.mul, a.by_q.shr, a.by_c8.mul, a.by_c8.shr, a.by_pe.mul,
           a.by_pe.shr, a.by_np.mul, a.by_np.shr, a.by_u3.mul, a.by_u3.shr, a.by_nb3.mul, a.by_nb3.shr);
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const uint32_t base = (uint32_t)(uintptr_t)((lds_u8 *)lds);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  const int wg = (int)xcd_remap(blockIdx.x, gridDim.x);
  const int img = a.by_bands.of(wg), p0 = (wg - img * a.bands) * a.rows;
  const int out_rows = min(a.rows, a.P - p0);
  const int ih0 = p0 * a.stride - 1, e_rows = (out_rows - 1) * a.stride + 3;
  const int r_lo = max(ih0, 0), r_hi = min(ih0 + e_rows, a.H);        // input rows inside the image
  const int npx = (r_hi - r_lo) * a.W, opx = out_rows * a.Q;

  // ---- input rows: contiguous in memory, 8 bytes at a time (pixels of 24 bytes), into rows of whole fragments
  const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(a.x), 0, a.x_bytes, 0x00027000);
  const int n8 = npx * a.c8, x_first = (img * a.H + r_lo) * a.W * a.c8 * 8;
  constexpr int XU = 2;
  v2i xv[XU];
  auto fetch = [&](int i0) {
#pragma unroll
    for (int k = 0; k < XU; ++k) {
      const int i = i0 + k * NT + tid;
      xv[k] = __builtin_bit_cast(v2i, __builtin_amdgcn_raw_buffer_load_b64(xres, i < n8 ? (uint32_t)(x_first + i * 8) : 0x80000000u, 0, 0));
    }
  };
  auto put = [&](int i0) {
#pragma unroll
    for (int k = 0; k < XU; ++k) {
      const int i = i0 + k * NT + tid, px = a.by_c8.of(i);
      if (i < n8) *(lds_v2i *)(uintptr_t)(base + px * a.xp + (i - px * a.c8) * 8) = v2i{xv[k].x ^ (int)a.x_xor, xv[k].y ^ (int)a.x_xor};
    }
  };
  fetch(0);
  // first weights of this wave
  const __amdgpu_buffer_rsrc_t w1res = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t *>(a.w1), 0, a.w1_bytes, 0x00027000);
  const int slot1 = a.by_m1.of(wave), m1 = wave - slot1 * a.m1;
  v4i wn[KS1];
  auto load_w1 = [&](int nb) {
#pragma unroll
    for (int k = 0; k < KS1; ++k)
      wn[k] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(w1res, lane * 16, (nb * KS1 + k) * 1024, 0));
  };
  load_w1(min(slot1, a.nb1 - 1));      // (of the waves without a block too: the descriptor does not bound the scalar offset)
  // ---- depthwise weights and start values, straight into LDS
  {
    const __amdgpu_buffer_rsrc_t cres = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t *>(a.consts), 0, a.const_bytes, 0x00027000);
    for (int at = wave * 1024; at < a.const_bytes; at += NWAVE * 1024)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(cres, (lds_void *)(lds + a.at_const + at), 16, lane * 16, at, 0, 0);
  }
  // ---- zeros around the expanded rows: the columns beside the image, and whole rows above or below it
  {
    const int ez = (int)a.e_xor, pe = a.ep >> 4, ew = a.W + 2;
    for (int i = tid; i < e_rows * 2 * pe; i += NT) {
      const int cell = a.by_pe.of(i);
      lds_write(base + a.at_e + ((cell >> 1) * ew + (cell & 1) * (ew - 1)) * a.ep + (i - cell * pe) * 16, v4i{ez, ez, ez, ez});
    }
    if (r_hi - r_lo < e_rows)
      for (int i = tid; i < a.W * pe; i += NT) {
        const int cell = a.by_pe.of(i);
        const uint32_t to = base + a.at_e + (1 + cell) * a.ep + (i - cell * pe) * 16;
        if (ih0 < 0) lds_write(to, v4i{ez, ez, ez, ez});
        if (r_hi == a.H) for (int r = a.H - ih0; r < e_rows; ++r) lds_write(to + r * ew * a.ep, v4i{ez, ez, ez, ez});
      }
  }
  put(0);
  for (int i0 = XU * NT; i0 < n8; i0 += XU * NT) { fetch(i0); put(i0); }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // the constants have arrived
  __syncthreads();

  auto start16 = [&](int block) {
    v16i v;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const v4i s = lds_read(base + a.at_const + tap_bytes(a.nb1) + block * 128 + half * 64 + g * 16);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[4 * g + i] = s[i];
    }
    return v;
  };

  // ---- first layer: a wave keeps its block of pixels and takes every g1-th block of channels
  if (slot1 < a.g1) {
    for (int mb = m1; mb < a.mb1; mb += a.m1) {
      const int i = mb * 32 + l32, r = a.by_w.of(i), c = i - r * a.W;
      const uint32_t from = base + min(i, npx - 1) * a.xp + half * 16;
      const uint32_t to = base + a.at_e + ((r + r_lo - ih0) * (a.W + 2) + c + 1) * a.ep + half * 16;
      v4i xf[KS1];
#pragma unroll
      for (int k = 0; k < KS1; ++k) xf[k] = lds_read(from + k * 32);
      for (int nb = slot1; nb < a.nb1; nb += a.g1) {
        v16i acc = start16(nb);
#pragma unroll
        for (int k = 0; k < KS1; ++k) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(wn[k], xf[k], acc, 0, 0, 0);
        const int next = nb + a.g1 < a.nb1 ? nb + a.g1 : slot1;
        load_w1(next);
        const v4i v = requant16(acc, a.clip1, a.shift1, (int)a.e_xor);
        if (i < npx) lds_write(to + nb * 32, v);
      }
    }
  }
  __syncthreads();

  // ---- last layer's first weights, requested ahead of the depthwise layer
  const int u3 = a.nb3 * a.mb2, part = a.by_u3.of(wave), first_unit = wave - part * u3;
  const bool active = part < a.kg;
  constexpr int PF = 4;
  v4i wq[PF];
  auto weights_of = [&](int unit, int &mbi, int &nbi) {
    mbi = a.by_nb3.of(unit);
    nbi = unit - mbi * a.nb3;
    return a.w2 + ((size_t)nbi * a.nb1 * 64 + lane) * 16;
  };
  auto load_first = [&](const int8_t *wf) {
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      const int s = part + i * a.kg;
      wq[i] = *reinterpret_cast<const v4i *>(wf + (size_t)(s < a.nb1 ? s : part) * 1024);
    }
  };
  int mbi, nbi;
  const int8_t *wf = weights_of(first_unit, mbi, nbi);
  if (active) load_first(wf);
  // ---- depthwise layer: the same over output pixels.  (The nine products are one chain, each waiting 64 cycles for the last,
  // half of them idle: the other wave of the SIMD has them.)
  const int slot2 = a.by_m2.of(wave);
  if (slot2 < a.g2) {
    // the lane's row of the diagonal matrix: channel weight_row(l32) of the block, its byte among the lane's 16
    const int ch = weight_row(l32);
    uint32_t mask[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) mask[d] = (ch >> 4) == half && ((ch >> 2) & 3) == d ? 0xffu << (8 * (ch & 3)) : 0u;
    for (int mb = wave - slot2 * a.m2; mb < a.mb2; mb += a.m2) {
      const int j = mb * 32 + l32, jc = min(j, opx - 1), pr = a.by_q.of(jc), q = jc - pr * a.Q;
      const uint32_t first = base + a.at_e + (pr * a.stride * (a.W + 2) + q * a.stride) * a.ep + half * 16;
      const uint32_t to = base + a.at_d + j * a.ep + half * 16;
      for (int cb = slot2; cb < a.nb1; cb += a.g2) {
        const uint32_t taps = base + a.at_const + cb * (9 * 128) + ch * 4;
        uint32_t t9[9], at = first + cb * 32;
        v4i f[9];
#pragma unroll
        for (int t = 0; t < 9; ++t) {
          t9[t] = *(lds_u32 *)(uintptr_t)(taps + t * 128);
          f[t] = lds_read(at);
          at += t % 3 == 2 ? a.W * a.ep : a.ep;
        }
        v16i acc = start16(a.nb1 + cb);
#pragma unroll
        for (int t = 0; t < 9; ++t) {
          const v4i d = {(int)(t9[t] & mask[0]), (int)(t9[t] & mask[1]), (int)(t9[t] & mask[2]), (int)(t9[t] & mask[3])};
          acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(d, f[t], acc, 0, 0, 0);
        }
        lds_write(to + cb * 32, requant16(acc, a.clipd, a.shiftd, (int)a.d_xor));
      }
    }
  }
  __syncthreads();

  // ---- last layer: waves share the output blocks and, where there are fewer than waves, K
  if (active) {
    for (int unit = first_unit;;) {
      v16i acc;
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[i] = 0;
      const uint32_t from = base + a.at_d + (mbi * 32 + l32) * a.ep + half * 16;
      for (int s0 = part; s0 < a.nb1; s0 += PF * a.kg) {
        v4i xf[PF];
#pragma unroll
        for (int i = 0; i < PF; ++i) {
          const int s = s0 + i * a.kg;
          xf[i] = lds_read(from + (s < a.nb1 ? s : part) * 32);
        }
#pragma unroll
        for (int i = 0; i < PF; ++i) {
          const int s = s0 + i * a.kg;
          if (s < a.nb1) {                           // uniform
            acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(wq[i], xf[i], acc, 0, 0, 0);
            const int ahead = s + PF * a.kg;
            if (ahead < a.nb1) wq[i] = *reinterpret_cast<const v4i *>(wf + (size_t)ahead * 1024);
          }
        }
      }
      // (the expanded rows are no longer read: their place takes the sums)
      const uint32_t to = base + a.at_e + ((part * a.mb2 + mbi) * a.nb3 + nbi) * (32 * PART_PITCH) + l32 * PART_PITCH + half * 64;
#pragma unroll
      for (int g = 0; g < 4; ++g) lds_write(to + g * 16, v4i{acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]});
      unit += NWAVE;
      if (a.kg > 1 || unit >= u3) break;             // (more blocks than waves: nobody shares K)
      wf = weights_of(unit, mbi, nbi);
      load_first(wf);
    }
  }
  __syncthreads();
  const size_t y_first = ((size_t)img * a.P + p0) * a.Q;
  const int shortcut = (p0 - r_lo) * a.W, np = a.cout >> 2;
  for (int it = tid; it < opx * np; it += NT) {
    const int m = a.by_np.of(it), n = (it - m * np) * 4;
    v4i v = lds_read(base + a.at_const + tap_bytes(a.nb1) + 2 * a.nb1 * 128 + n * 4);
    for (int k = 0; k < a.kg; ++k)
      v += lds_read(base + a.at_e + ((k * a.mb2 + (m >> 5)) * a.nb3 + (n >> 5)) * (32 * PART_PITCH) + (m & 31) * PART_PITCH + (n & 31) * 4);
    if (a.has_res) {
      const uint32_t r = *(lds_u32 *)(uintptr_t)(base + (m + shortcut) * a.xp + n);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] += (int)(int8_t)(r >> (8 * i)) << a.res_d;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = requant<false>(v[i], a.shift2, a.lo2, a.hi2);
    *reinterpret_cast<uint32_t *>(a.y + (y_first + m) * a.cout + n) = pack4(v.x, v.y, v.z, v.w);
  }
}

// The constants: dword [block of 32 channels][tap][c] = the tap's weight of channel c in all four bytes (zeros past Ce), then the start values of
// the three layers, the last with what makes an unsigned shortcut signed.
__global__ __launch_bounds__(256) void pw_dw_pw_consts_kernel(const int8_t *__restrict__ wd, const int32_t *__restrict__ acc1,
                                                              const int32_t *__restrict__ accd, const int32_t *__restrict__ acc2,
                                                              int32_t *__restrict__ to, int Ce, int padded, int n3, int res_bias) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < 9 * padded) {
    const int c = i / 288 * 32 + i % 32, tap = i / 32 % 9;
    to[i] = c < Ce ? (int)((uint32_t)(uint8_t)wd[(size_t)tap * Ce + c] * 0x01010101u) : 0;
  } else if (i < 10 * padded) {
    to[i] = acc1[i - 9 * padded];
  } else if (i < 11 * padded) {
    to[i] = accd[i - 10 * padded];
  } else if (i < 11 * padded + n3) {
    to[i] = acc2[i - 11 * padded] + res_bias;
  }
}

// ---- the front of a network
//
// The image's rows are spread to four bytes per pixel in LDS, so that four pixels of a window row are half a fragment: two slices
// of K for the three rows, where the weights of the fourth channel, pixel and row are zeros.  With one block of 32
// channels in the middle a lane's 16 depthwise results are the fragment that the last layer takes: they stay in registers, as do the nine
// diagonal matrices.
//
// MobileNetV2's front, 27 images of 224 x 224: 26.0 -> 10.3 us (three launches of 14.8, 7.4 and 3.7), 128: 75.2 -> 37.2, of which image and
// result are some 9 us of memory traffic: bound by vector instructions (about 300 per 32 pixels, two thirds of them requantisation and
// packing).  With the general kernel above (depthwise result through LDS, diagonals rebuilt for every block) it was 14.5 and 56.7.
struct ImageArgs {
  const uint8_t *x;
  const int8_t *w1, *consts, *w2;
  uint8_t *y;
  int x_bytes, const_bytes, w2_bytes;
  int H0, H, W, P, Q, stride, cout, groups;    // image rows; first layer's result; groups of four pixels per image row
  int rows, bands, nb3, mb1, mb2;              // as in Args
  int xp, at_const, at_w2, at_e;               // bytes of an image row in LDS; LDS offsets
  uint32_t x_xor, e_xor, d_xor;
  ScaledClip clip1, clipd, clip2;
  int shift1, shiftd, shift2;
  Div by_bands, by_w, by_q, by_groups;
};

constexpr int EP = 48;       // bytes of a pixel of the first layer's result in LDS: 16 pixels of a row start on different banks

__global__ __launch_bounds__(NT, 2) void image_dw_pw_kernel(const ImageArgs a) {
  typedef int v3i __attribute__((ext_vector_type(3)));
  pin_args(a.x, a.w1, a.consts, a.w2, a.y, a.x_bytes, a.const_bytes, a.w2_bytes, a.H0, a.H, a.W, a.P, a.Q, a.stride, a.cout, a.groups, a.rows,
           a.bands, a.nb3, a.mb1, a.mb2, a.xp, a.at_const, a.at_w2, a.at_e, a.x_xor, a.e_xor, a.d_xor, a.clip1.lo, a.clip1.hi, a.clipd.lo,
           a.clipd.hi, a.clip2.lo, a.clip2.hi, a.shift1, a.shiftd, a.shift2, a.by_bands.mul, a.by_bands.shr, a.by_w.mul, a.by_w.shr, a.by_q.mul,
           a.by_q.shr, a.by_groups.mul, a.by_groups.shr);
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const uint32_t base = (uint32_t)(uintptr_t)((lds_u8 *)lds);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  const int wg = (int)xcd_remap(blockIdx.x, gridDim.x);
  const int img = a.by_bands.of(wg), p0 = (wg - img * a.bands) * a.rows;
  const int out_rows = min(a.rows, a.P - p0);
  const int ih0 = p0 * a.stride - 1, e_rows = (out_rows - 1) * a.stride + 3;
  const int r_lo = max(ih0, 0), r_hi = min(ih0 + e_rows, a.H);        // rows of the first layer's result inside it
  const int npx = (r_hi - r_lo) * a.W, opx = out_rows * a.Q;

  // ---- image rows under them, four pixels at a time, pixel c at 4 (c + 1) of its row
  const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(a.x), 0, a.x_bytes, 0x00027000);
  const int ir0 = 2 * r_lo - 1, n = (2 * (r_hi - r_lo) + 1) * a.groups, first = (img * a.H0 + ir0) * a.groups * 12;
  constexpr int XU = 3;
  v3i xv[XU];
  auto fetch = [&](int i0) {
#pragma unroll
    for (int k = 0; k < XU; ++k) {
      const int i = i0 + k * NT + tid, row = a.by_groups.of(i);
      const bool in = i < n && (uint32_t)(ir0 + row) < (uint32_t)a.H0;
      xv[k] = __builtin_bit_cast(v3i, __builtin_amdgcn_raw_buffer_load_b96(xres, in ? (uint32_t)(first + i * 12) : 0x80000000u, 0, 0));
    }
  };
  auto put = [&](int i0) {
#pragma unroll
    for (int k = 0; k < XU; ++k) {
      const int i = i0 + k * NT + tid, row = a.by_groups.of(i), g = i - row * a.groups;
      if (i >= n) continue;
      // (the fourth byte of a pixel meets zero weights)
      const uint32_t to = base + row * a.xp + g * 16 + 4, d0 = xv[k].x, d1 = xv[k].y, d2 = xv[k].z;
      *(lds_u32 *)(uintptr_t)to = d0 ^ a.x_xor;
      *(lds_v2i *)(uintptr_t)(to + 4) = v2i{(int)(__builtin_amdgcn_alignbyte(d1, d0, 3) ^ a.x_xor), (int)(__builtin_amdgcn_alignbyte(d2, d1, 2) ^ a.x_xor)};
      *(lds_u32 *)(uintptr_t)(to + 12) = (d2 >> 8) ^ a.x_xor;
      if (g == 0) *(lds_u32 *)(uintptr_t)(to - 4) = a.x_xor;           // the column left of the image
    }
  };
  fetch(0);
  v4i w1[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) w1[k] = *reinterpret_cast<const v4i *>(a.w1 + k * 1024 + lane * 16);
  // ---- depthwise weights and start values, and the last layer's weights, straight into LDS
  {
    const __amdgpu_buffer_rsrc_t cres = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t *>(a.consts), 0, a.const_bytes, 0x00027000);
    for (int at = wave * 1024; at < a.const_bytes; at += NWAVE * 1024)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(cres, (lds_void *)(lds + a.at_const + at), 16, lane * 16, at, 0, 0);
    const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t *>(a.w2), 0, a.w2_bytes, 0x00027000);
    if (wave < a.nb3) __builtin_amdgcn_raw_ptr_buffer_load_lds(wres, (lds_void *)(lds + a.at_w2 + wave * 1024), 16, lane * 16, wave * 1024, 0, 0);
  }
  // ---- zeros around the first layer's result
  {
    const int ez = (int)a.e_xor, ew = a.W + 2;
    for (int i = tid; i < e_rows * 4; i += NT)
      lds_write(base + a.at_e + ((i >> 2) * ew + ((i >> 1) & 1) * (ew - 1)) * EP + (i & 1) * 16, v4i{ez, ez, ez, ez});
    if (r_hi - r_lo < e_rows)
      for (int i = tid; i < a.W * 2; i += NT) {
        const uint32_t to = base + a.at_e + (1 + (i >> 1)) * EP + (i & 1) * 16;
        if (ih0 < 0) lds_write(to, v4i{ez, ez, ez, ez});
        if (r_hi == a.H) for (int r = a.H - ih0; r < e_rows; ++r) lds_write(to + r * ew * EP, v4i{ez, ez, ez, ez});
      }
  }
  put(0);
  for (int i0 = XU * NT; i0 < n; i0 += XU * NT) { fetch(i0); put(i0); }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // the constants have arrived
  __syncthreads();

  auto start16 = [&](int block) {
    v16i v;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const v4i s = lds_read(base + a.at_const + tap_bytes(1) + block * 128 + half * 64 + g * 16);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[4 * g + i] = s[i];
    }
    return v;
  };

  // ---- first layer
  {
    const v16i start = start16(0);
    for (int mb = wave; mb < a.mb1; mb += NWAVE) {
      const int i = mb * 32 + l32, ic = min(i, npx - 1), r = a.by_w.of(ic), c = ic - r * a.W;
      // slice 0: rows 0 and 1 of the window, slice 1: row 2 (whose other half meets zero weights)
      const uint32_t from = base + (2 * r + half) * a.xp + c * 8, last = from + (2 - half) * a.xp;
      const v2i x0 = *(lds_v2i *)(uintptr_t)from, x1 = *(lds_v2i *)(uintptr_t)(from + 8);
      const v2i x2 = *(lds_v2i *)(uintptr_t)last, x3 = *(lds_v2i *)(uintptr_t)(last + 8);
      v16i acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(w1[0], v4i{x0.x, x0.y, x1.x, x1.y}, start, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(w1[1], v4i{x2.x, x2.y, x3.x, x3.y}, acc, 0, 0, 0);
      const v4i v = requant16(acc, a.clip1, a.shift1, (int)a.e_xor);
      if (i < npx) lds_write(base + a.at_e + ((r + r_lo - ih0) * (a.W + 2) + c + 1) * EP + half * 16, v);
    }
  }
  // the lane's rows of the nine diagonal matrices: channel weight_row(l32), its byte among the lane's 16
  const int ch = weight_row(l32);
  v4i diag[9];
#pragma unroll
  for (int t = 0; t < 9; ++t) {
    const uint32_t w = *(lds_u32 *)(uintptr_t)(base + a.at_const + t * 128 + ch * 4);
#pragma unroll
    for (int d = 0; d < 4; ++d) diag[t][d] = (ch >> 4) == half && ((ch >> 2) & 3) == d ? (int)(w & (0xffu << (8 * (ch & 3)))) : 0;
  }
  const v16i startd = start16(1);
  __syncthreads();

  // ---- depthwise layer and last layer of 32 pixels at a time
  uint8_t *const y = a.y + ((size_t)img * a.P + p0) * a.Q * a.cout;
  for (int mb = wave; mb < a.mb2; mb += NWAVE) {
    const int j = mb * 32 + l32, jc = min(j, opx - 1), pr = a.by_q.of(jc), q = jc - pr * a.Q;
    uint32_t at = base + a.at_e + (pr * (a.W + 2) + q) * (a.stride * EP) + half * 16;
    v16i acc = startd;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(diag[t], lds_read(at + t % 3 * EP), acc, 0, 0, 0);
      if (t % 3 == 2) at += (a.W + 2) * EP;
    }
    const v4i d = requant16(acc, a.clipd, a.shiftd, (int)a.d_xor);
    for (int nb = 0; nb < a.nb3; ++nb) {
      v16i out = __builtin_amdgcn_mfma_i32_32x32x32_i8(lds_read(base + a.at_w2 + nb * 1024 + lane * 16), d, start16(2 + nb), 0, 0, 0);
      const v4i v = requant16(out, a.clip2, a.shift2, 0);
      const int c = nb * 32 + half * 16;
      uint8_t *to = y + j * a.cout + c;
      if (j < opx && c < a.cout) *reinterpret_cast<v2i *>(to) = v2i{v.x, v.y};
      if (j < opx && c + 8 < a.cout) *reinterpret_cast<v2i *>(to + 8) = v2i{v.z, v.w};
    }
  }
}

constexpr int LDS_MOST = 160 * 1024;
constexpr int KS1_MOST = 6;

struct Shape {
  int rows, bands, mb1, mb2, xp, ep, at_const, at_e, at_d, bytes;
};

// LDS and blocks of a launch with `rows` output rows per workgroup.
Shape shape_of(int Cin, int Ce, int Cout, int H, int W, int P, int Q, int stride, int rows) {
  Shape s;
  s.rows = rows;
  s.bands = (P + rows - 1) / rows;
  const int e_rows = (rows - 1) * stride + 3, in_rows = e_rows < H ? e_rows : H, nb1 = (Ce + 31) / 32, nb3 = (Cout + 31) / 32;
  s.mb1 = (in_rows * W + 31) / 32;
  s.mb2 = (rows * Q + 31) / 32;
  s.xp = (Cin + 31) / 32 * 32 + 16;
  s.ep = nb1 * 32 + 16;
  s.at_const = (in_rows * W * s.xp + 15) / 16 * 16;
  s.at_e = s.at_const + (int)pw_dw_pw_const_bytes(Ce, Cout);
  const int kg = nb3 * s.mb2 <= NWAVE ? NWAVE / (nb3 * s.mb2) : 1;
  const int e = e_rows * (W + 2) * s.ep, sums = kg * nb3 * s.mb2 * 32 * PART_PITCH;
  s.at_d = s.at_e + (e > sums ? e : sums);
  s.bytes = s.at_d + s.mb2 * 32 * s.ep;
  return s;
}

// Cycles of one workgroup: set-up and the units of the three layers that a wave works through one after the other.
long long workgroup_cycles(const Shape &s, int Cin, int Ce, int Cout) {
  const int nb1 = (Ce + 31) / 32, nb3 = (Cout + 31) / 32, ks1 = (Cin + 31) / 32;
  auto units = [&](int mb) {
    const int m = mb < NWAVE ? mb : NWAVE, g = NWAVE / m;
    return (long long)((mb + m - 1) / m) * ((nb1 + g - 1) / g);
  };
  const int u3 = nb3 * s.mb2, kg = u3 < NWAVE ? NWAVE / u3 : 1;
  return 3500 + units(s.mb1) * (450 + 60 * ks1) + units(s.mb2) * 900 + (u3 + NWAVE - 1) / NWAVE * (long long)((nb1 + kg - 1) / kg) * 120;
}

// Tenths of a workgroup's time that a launch takes: rounds of 256 workgroups, of which two share a CU at 0.8 of the time each where
// they fit.
long long launch_tenths(const Shape &s, int B) {
  const long long rounds = ((long long)B * s.bands + 255) / 256;
  return 2 * s.bytes <= LDS_MOST ? rounds / 2 * 16 + rounds % 2 * 10 : rounds * 10;
}

// Rows per workgroup, by what a launch of them would take.  0: no number of rows fits.
int rows_for(int Cin, int Ce, int Cout, int H, int W, int P, int Q, int stride, int B) {
  int best = 0;
  long long least = 0;
  for (int rows = 1; rows <= P; ++rows) {
    const Shape s = shape_of(Cin, Ce, Cout, H, W, P, Q, stride, rows);
    if (s.bytes > LDS_MOST) break;
    const long long cost = workgroup_cycles(s, Cin, Ce, Cout) * launch_tenths(s, B);
    if (best == 0 || cost < least) { best = rows; least = cost; }
  }
  return best;
}

template <typename A, void (*k)(const A)>
int launch_one(const A &a, int lds, long long grid, hipStream_t stream) {
  static std::atomic<unsigned long long> done_mask{0};         // devices whose LDS limit has been raised
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return (int)hipErrorInvalidDevice;
  if (dev < 0 || dev > 63 || !((done_mask.load(std::memory_order_relaxed) >> dev) & 1ull)) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, LDS_MOST);
    if (e != hipSuccess) return (int)e;
    if (dev >= 0 && dev <= 63) done_mask.fetch_or(1ull << dev, std::memory_order_relaxed);
  }
  hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(NT), lds, stream, a);
  return (int)hipGetLastError();
}

// LDS and blocks of the front's launch with `rows` output rows per workgroup.
struct ImageShape {
  int rows, bands, mb1, mb2, xp, at_const, at_w2, at_e, bytes;
};

ImageShape image_shape_of(int Ce, int Cout, int H, int W, int P, int Q, int stride, int rows) {
  ImageShape s;
  s.rows = rows;
  s.bands = (P + rows - 1) / rows;
  const int e_rows = (rows - 1) * stride + 3, in_rows = e_rows < H ? e_rows : H;
  s.mb1 = (in_rows * W + 31) / 32;
  s.mb2 = (rows * Q + 31) / 32;
  s.xp = (2 * W + 4) * 4;
  s.at_const = (2 * in_rows + 1) * s.xp;
  s.at_w2 = s.at_const + (int)pw_dw_pw_const_bytes(Ce, Cout);
  s.at_e = s.at_w2 + (Cout + 31) / 32 * 1024;
  s.bytes = s.at_e + e_rows * (W + 2) * EP;
  return s;
}

// As rows_for.
int image_rows_for(int Ce, int Cout, int H, int W, int P, int Q, int stride, int B) {
  int best = 0;
  long long least = 0;
  for (int rows = 1; rows <= P; ++rows) {
    const ImageShape s = image_shape_of(Ce, Cout, H, W, P, Q, stride, rows);
    if (s.bytes > LDS_MOST) break;
    const long long one = 3500 + (s.mb1 + NWAVE - 1) / NWAVE * 400 + (s.mb2 + NWAVE - 1) / NWAVE * (900 + 200 * ((Cout + 31) / 32));
    const long long rounds = ((long long)B * s.bands + 255) / 256;
    const long long cost = 2 * s.bytes <= LDS_MOST ? one * (rounds / 2 * 16 + rounds % 2 * 10) : one * rounds * 10;
    if (best == 0 || cost < least) { best = rows; least = cost; }
  }
  return best;
}

}  // namespace

bool pw_dw_pw_applicable(int Cin, int Ce, int Cout, int H, int W, int stride, int shift1, int shiftd, int shift2, bool has_res, int res_d,
                         const void *x, const void *y) {
  if (Cin < 8 || (Cin & 7) || Cin > 32 * KS1_MOST || Ce < 16 || Ce > 1024 || Cout < 8 || (Cout & 7) || Cout > 256) return false;
  if ((stride != 1 && stride != 2) || H < 1 || W < 1 || W > 1024 || shift1 < 0 || shiftd < 0 || shift2 < 0) return false;
  if (has_res && (stride != 1 || Cin != Cout || res_d < 0 || res_d > 16)) return false;
  if ((reinterpret_cast<uintptr_t>(x) & 7) || (reinterpret_cast<uintptr_t>(y) & 3)) return false;
  return rows_for(Cin, Ce, Cout, H, W, (H - 1) / stride + 1, (W - 1) / stride + 1, stride, 1) > 0;
}

// What the launch takes against what the layers take apart: 29200 cycles (12.2 us: 9.5 as measured alone, and 2 - 4 that launches cost more
// in a forward) and the bytes they move at 6.25 TB/s (384 cycles a MB; a pair keeps the depthwise result to itself).  Beside the cycles by
// which rows_for chooses, a workgroup waits for its input (1500 cycles for each 8 KiB of it) and adds, requantises and writes its result
// (600 for each 2 KiB).
// Random blocks (Cin to 192, Ce to 1024, Cout to 256, 4 x 4 to 112 x 112, batch 1 to 128) alone, one launch against three: of 1924 this was
// fitted to 402 lost more than 3 %, up to half their speed (192 -> 576 -> 96 on 33 x 33, batch 120, 98 -> 201 us: one row per
// workgroup, so the first layer is computed three times); with it 50.  Of 3913 fresh ones, against three launches or two, it lets 56 lose, the worst
// 18 % (64 -> 256 -> 24 from 83 x 83, stride 2, batch 48, 62 -> 76).  In MobileNetV2's forwards the two sides at the line: 960 channels on
// 7 x 7, batch 192, 764 us with one launch, 780 with three.
bool pw_dw_pw_pays(int Cin, int Ce, int Cout, int H, int W, int stride, int B, bool pair) {
  const int P = (H - 1) / stride + 1, Q = (W - 1) / stride + 1;
  const int rows = rows_for(Cin, Ce, Cout, H, W, P, Q, stride, B);
  if (rows == 0) return false;
  const Shape s = shape_of(Cin, Ce, Cout, H, W, P, Q, stride, rows);
  const int in_rows = (rows - 1) * stride + 3 < H ? (rows - 1) * stride + 3 : H;
  const long long loads = ((long long)in_rows * W * Cin / 8 + 1023) / 1024, stores = ((long long)rows * Q * Cout / 4 + 511) / 512;
  const long long cycles = (workgroup_cycles(s, Cin, Ce, Cout) + 1500 * loads + 600 * stores) * launch_tenths(s, B) / 10;
  const long long apart = (long long)B * ((long long)H * W * (Cin + 2 * Ce) + (long long)P * Q * (pair ? Cout : 2 * Ce + Cout));
  return cycles < 29200 + apart / 2604;
}

size_t pw_dw_pw_const_bytes(int Ce, int Cout) {
  const size_t nb1 = (Ce + 31) / 32, nb3 = (Cout + 31) / 32;
  return (tap_bytes((int)nb1) + (2 * nb1 + nb3) * 128 + 1023) / 1024 * 1024;
}

int launch_pw_dw_pw_consts(const int8_t *wd, const int32_t *acc1, const int32_t *accd, const int32_t *acc2, int8_t *to, int Ce, int Cout, int res_bias,
                           hipStream_t stream) {
  const int padded = (Ce + 31) / 32 * 32, n3 = (Cout + 31) / 32 * 32;
  hipLaunchKernelGGL(pw_dw_pw_consts_kernel, dim3((11 * padded + n3 + 255) / 256), dim3(256), 0, stream, wd, acc1, accd, acc2,
                     reinterpret_cast<int32_t *>(to), Ce, padded, n3, res_bias);
  return (int)hipGetLastError();
}

int launch_pw_dw_pw(const PwDwPwParams &p, hipStream_t stream) {
  if (p.B <= 0) return 0;
  if (!pw_dw_pw_applicable(p.Cin, p.Ce, p.Cout, p.H, p.W, p.stride, p.shift1, p.shiftd, p.shift2, p.has_res != 0, p.res_d, p.x, p.y) ||
      ((reinterpret_cast<uintptr_t>(p.w1) | reinterpret_cast<uintptr_t>(p.consts) | reinterpret_cast<uintptr_t>(p.w2)) & 15) ||
      (long long)p.B * p.H * p.W * p.Cin > 0x7fffffffLL)
    return (int)hipErrorInvalidValue;
  const int rows = rows_for(p.Cin, p.Ce, p.Cout, p.H, p.W, p.P, p.Q, p.stride, p.B);
  const Shape s = shape_of(p.Cin, p.Ce, p.Cout, p.H, p.W, p.P, p.Q, p.stride, rows);
  const int ks1 = (p.Cin + 31) / 32;
  Args a;
  a.x = p.x; a.w1 = p.w1; a.consts = p.consts; a.w2 = p.w2; a.y = p.y;
  a.H = p.H; a.W = p.W; a.P = p.P; a.Q = p.Q; a.stride = p.stride; a.c8 = p.Cin / 8; a.cout = p.Cout;
  a.rows = rows; a.bands = s.bands;
  a.nb1 = (p.Ce + 31) / 32; a.nb3 = (p.Cout + 31) / 32;
  a.mb1 = s.mb1; a.mb2 = s.mb2;
  a.m1 = a.mb1 < NWAVE ? a.mb1 : NWAVE; a.g1 = NWAVE / a.m1;
  a.m2 = a.mb2 < NWAVE ? a.mb2 : NWAVE; a.g2 = NWAVE / a.m2;
  a.xp = s.xp; a.ep = s.ep;
  a.at_const = s.at_const; a.at_e = s.at_e; a.at_d = s.at_d;
  const int u3 = a.nb3 * a.mb2, kg = u3 < NWAVE ? NWAVE / u3 : 1;
  a.kg = kg < a.nb1 ? kg : a.nb1;
  a.x_bytes = p.B * p.H * p.W * p.Cin;
  a.w1_bytes = a.nb1 * ks1 * 1024;
  a.const_bytes = (int)pw_dw_pw_const_bytes(p.Ce, p.Cout);
  a.has_res = p.has_res; a.res_d = p.res_d;
  a.x_xor = p.x_xor; a.e_xor = p.e_xor; a.d_xor = p.d_xor;
  a.clip1 = scaled_clip(p.lo1, p.hi1, p.shift1);
  a.clipd = scaled_clip(p.lod, p.hid, p.shiftd);
  a.shift1 = p.shift1; a.shiftd = p.shiftd; a.shift2 = p.shift2; a.lo2 = p.lo2; a.hi2 = p.hi2;
  a.by_bands = Div(s.bands); a.by_m1 = Div(a.m1); a.by_m2 = Div(a.m2); a.by_w = Div(p.W); a.by_q = Div(p.Q); a.by_c8 = Div(a.c8);
  a.by_pe = Div(s.ep / 16); a.by_np = Div(p.Cout / 4); a.by_u3 = Div(u3); a.by_nb3 = Div(a.nb3);
  const long long grid = (long long)p.B * s.bands;
  if (grid > 0x7fffffffLL) return (int)hipErrorInvalidValue;
  switch (ks1) {
    case 1: return launch_one<Args, pw_dw_pw_kernel<1>>(a, s.bytes, grid, stream);
    case 2: return launch_one<Args, pw_dw_pw_kernel<2>>(a, s.bytes, grid, stream);
    case 3: return launch_one<Args, pw_dw_pw_kernel<3>>(a, s.bytes, grid, stream);
    case 4: return launch_one<Args, pw_dw_pw_kernel<4>>(a, s.bytes, grid, stream);
    case 5: return launch_one<Args, pw_dw_pw_kernel<5>>(a, s.bytes, grid, stream);
    default: return launch_one<Args, pw_dw_pw_kernel<6>>(a, s.bytes, grid, stream);
  }
}

bool image_dw_pw_applicable(int Ce, int Cout, int H, int W, int stride, int shift1, int shiftd, int shift2, const void *x, const void *y) {
  if (Ce < 4 || Ce > 32 || (Ce & 3) || Cout < 8 || (Cout & 7) || Cout > 256 || (stride != 1 && stride != 2)) return false;
  if (H < 1 || W < 4 || (W & 3) || W > 1024 || shift1 < 0 || shiftd < 0 || shift2 < 0) return false;
  if ((reinterpret_cast<uintptr_t>(x) & 3) || (reinterpret_cast<uintptr_t>(y) & 7)) return false;
  const int H1 = (H - 1) / 2 + 1, W1 = W / 2;
  return image_rows_for(Ce, Cout, H1, W1, (H1 - 1) / stride + 1, (W1 - 1) / stride + 1, stride, 1) > 0;
}

int launch_image_dw_pw(const PwDwPwParams &p, hipStream_t stream) {
  if (p.B <= 0) return 0;
  const int W0 = 2 * p.W;
  if (!image_dw_pw_applicable(p.Ce, p.Cout, p.H0, W0, p.stride, p.shift1, p.shiftd, p.shift2, p.x, p.y) || (p.H0 - 1) / 2 + 1 != p.H || p.has_res ||
      ((reinterpret_cast<uintptr_t>(p.w1) | reinterpret_cast<uintptr_t>(p.consts) | reinterpret_cast<uintptr_t>(p.w2)) & 15) ||
      (long long)p.B * p.H0 * W0 * 3 > 0x7fffffffLL)
    return (int)hipErrorInvalidValue;
  const int rows = image_rows_for(p.Ce, p.Cout, p.H, p.W, p.P, p.Q, p.stride, p.B);
  const ImageShape s = image_shape_of(p.Ce, p.Cout, p.H, p.W, p.P, p.Q, p.stride, rows);
  ImageArgs a;
  a.x = p.x; a.w1 = p.w1; a.consts = p.consts; a.w2 = p.w2; a.y = p.y;
  a.H0 = p.H0; a.H = p.H; a.W = p.W; a.P = p.P; a.Q = p.Q; a.stride = p.stride; a.cout = p.Cout; a.groups = W0 / 4;
  a.rows = rows; a.bands = s.bands; a.nb3 = (p.Cout + 31) / 32; a.mb1 = s.mb1; a.mb2 = s.mb2;
  a.xp = s.xp; a.at_const = s.at_const; a.at_w2 = s.at_w2; a.at_e = s.at_e;
  a.x_bytes = p.B * p.H0 * W0 * 3;
  a.const_bytes = (int)pw_dw_pw_const_bytes(p.Ce, p.Cout);
  a.w2_bytes = a.nb3 * 1024;
  a.x_xor = p.x_xor; a.e_xor = p.e_xor; a.d_xor = p.d_xor;
  a.clip1 = scaled_clip(p.lo1, p.hi1, p.shift1);
  a.clipd = scaled_clip(p.lod, p.hid, p.shiftd);
  a.clip2 = scaled_clip(p.lo2, p.hi2, p.shift2);
  a.shift1 = p.shift1; a.shiftd = p.shiftd; a.shift2 = p.shift2;
  a.by_bands = Div(s.bands); a.by_w = Div(p.W); a.by_q = Div(p.Q); a.by_groups = Div(a.groups);
  const long long grid = (long long)p.B * s.bands;
  if (grid > 0x7fffffffLL) return (int)hipErrorInvalidValue;
  return launch_one<ImageArgs, image_dw_pw_kernel>(a, s.bytes, grid, stream);
}

}  // namespace f8
