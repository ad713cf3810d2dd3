// Depthwise 3x3 (pad 1, stride 1 or 2) followed by the 1x1 layer that is its only reader (the second and third
// layer of a MobileNetV2 block, both layers of a MobileNetV1 block), F8Net Eq. 6 twice, in one launch.
//
// At small and medium batch these layers are a few microseconds each, of which most is the launch and the
// first touch of data that another XCD wrote.  A workgroup takes a few rows of an image: its eight waves
// first compute the depthwise result of those pixels, all channels, into LDS (packed dot products as in
// dwconv_pool.hip; a lane keeps four channels, so their weights are unpacked once, and takes strips of four
// output columns), already in the signed form the matrix instructions take; that is the activation operand of the 1x1
// layer, whose weights stream from L2 in fragment order.  Waves share the output channels, 32 each, and where
// there are fewer blocks of 32 than waves, K; the sums meet in LDS and leave with the residual added,
// requantised, as 8-byte pieces.  The tensor between the layers is neither written nor read.
//
// Microseconds of the pair, two launches -> this one, batch 27: 28x28 C192 -> 32 9.5 -> 8.4, 28x28 (stride 2) C144 -> 32
// 10.4 -> 7.8, 14x14 (stride 2) C192 -> 64 8.6 -> 5.9, 14x14 C384 -> 64 8.1 -> 7.1; batch 1: 112x112 C32 -> 16 7.7 -> 4.5.  What
// bounds it there is the chain load, dot products, barrier, MFMA, barrier, store of one workgroup per CU.  On large
// maps the depthwise part loses to dwconv_pool.hip's, which reads each input row once for many output rows:
// 112x112 C32, batch 27, 11.2 -> 22.8.  (Requesting the next strip, or the residual, ahead: 8.4 -> 8.6, 94 VGPRs for 80.)
#include "dw_pw.h"

#include <atomic>

#include "dw_device.h"

namespace f8 {
namespace {

typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int NT = 512, NWAVE = NT / 64;
constexpr int PART_PITCH = 32 * 4 + 16;

struct DwPwTiling {
  int rows, tiles;           // output rows per workgroup, workgroups per image
  int dw, groups, strips;    // channel dwords; lane groups of that many lanes; strips of 4 columns
  int pitch;                 // bytes of a pixel in LDS
  int ks, nb, kg;            // K slices, 32-channel blocks, waves that share K
  int np;                    // 8-byte pieces per output pixel
  int x_image, lo_scaled, hi_scaled;
  FastDiv fd_tiles, fd_dw, fd_strips, fd_np;
};

// A different kind of vector instruction may read a packed dot product's result only three wait states later, and
// the compiler, which inserts those for its own instructions, cannot see into the statements that follow.
__device__ __forceinline__ void settle_dots(int (&a)[16]) {
  asm volatile("s_nop 2" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7]), "+v"(a[8]),
               "+v"(a[9]), "+v"(a[10]), "+v"(a[11]), "+v"(a[12]), "+v"(a[13]), "+v"(a[14]), "+v"(a[15]));
}

template <int STRIDE, int MB>
__global__ __launch_bounds__(NT, 4) void dw_pw_kernel(const DwPwParams p, const DwPwTiling tl) {
  constexpr int NCOL = 3 * STRIDE + 3;               // input columns under four output columns
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  // tiles of an image share input rows: neighbours on one XCD
  const uint32_t wg = xcd_remap(blockIdx.x, gridDim.x);
  const int img = (int)tl.fd_tiles.div(wg), p0 = (int)(wg - (uint32_t)img * tl.fd_tiles.d) * tl.rows;
  const int rows = min(tl.rows, p.P - p0), npx = rows * p.Q;
  const size_t px0 = ((size_t)img * p.P + p0) * p.Q;

  // ---- depthwise: lane -> channels 4 d .. 4 d + 3, items (row, strip) g, g + groups, ... ------------------
  const int g = (int)tl.fd_dw.div((uint32_t)tid), c = (tid - g * tl.dw) * 4;
  if (g < tl.groups) {
    const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t *>(p.x) + (size_t)img * tl.x_image, 0, tl.x_image, 0x00027000);
    const int row_bytes = p.W * p.C;
    const int items = rows * tl.strips;
    // wt[r][ch][0] = bytes (w[r][0][ch], w[r][1][ch], w[r][2][ch], 0), [1] = the same one byte up
    uint32_t wt[3][4][STRIDE == 1 ? 2 : 1];
    int acc0[4];
    const int rnd = p.d_shift > 0 ? 1 << (p.d_shift - 1) : 0;
#pragma unroll
    for (int ch = 0; ch < 4; ++ch) acc0[ch] = rnd + (p.bias ? p.bias[c + ch] : 0);
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      const uint32_t w0 = *reinterpret_cast<const uint32_t *>(p.wd + (size_t)(3 * r + 0) * p.C + c);
      const uint32_t w1 = *reinterpret_cast<const uint32_t *>(p.wd + (size_t)(3 * r + 1) * p.C + c);
      const uint32_t w2 = *reinterpret_cast<const uint32_t *>(p.wd + (size_t)(3 * r + 2) * p.C + c);
      const uint32_t lo = perm(w1, w0, 0x05010400u), hi = perm(w1, w0, 0x07030602u);
      wt[r][0][0] = perm(w2, lo, 0x0c040100u);
      wt[r][1][0] = perm(w2, lo, 0x0c050302u);
      wt[r][2][0] = perm(w2, hi, 0x0c060100u);
      wt[r][3][0] = perm(w2, hi, 0x0c070302u);
#pragma unroll
      for (int ch = 0; ch < 4; ++ch) {
        if (p.x_xor) acc0[ch] += 128 * __builtin_amdgcn_sdot4((int)wt[r][ch][0], 0x01010101, 0, false);
        if (STRIDE == 1) wt[r][ch][1] = wt[r][ch][0] << 8;
      }
    }
    for (int it = g; it < items; it += tl.groups) {
      const int pl = (int)tl.fd_strips.div((uint32_t)it), q0 = (it - pl * tl.strips) * 4;
      const int iy = (p0 + pl) * STRIDE - 1, ix = q0 * STRIDE - 1;
      // offsets: bit 31 set for a row or a column outside the image (the descriptor rejects them: zeros)
      uint32_t raw[3][NCOL], col[NCOL];
#pragma unroll
      for (int j = 0; j < NCOL; ++j) col[j] = (unsigned)(ix + j) < (unsigned)p.W ? 0u : 0x80000000u;
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        const uint32_t out = (unsigned)(iy + r) < (unsigned)p.H ? 0u : 0x80000000u;
        const int at = (iy + r) * row_bytes + ix * p.C + c;
#pragma unroll
        for (int j = 0; j < NCOL; ++j) raw[r][j] = __builtin_amdgcn_raw_buffer_load_b32(xres, (uint32_t)(at + j * p.C) | out | col[j], 0, 0);
      }
      int a[16];                                     // [column][channel]
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int ch = 0; ch < 4; ++ch) a[4 * q + ch] = acc0[ch];
#pragma unroll
      for (int r = 0; r < 3; ++r) {
#pragma unroll
        for (int j = 0; j < NCOL; ++j) raw[r][j] ^= p.x_xor;
        uint32_t t[4], u[4], win[4][4];
        transpose4(raw[r][0], raw[r][1], raw[r][2], raw[r][3], t);
        if (STRIDE == 1) {
          const uint32_t ef_lo = perm(raw[r][5], raw[r][4], 0x05010400u), ef_hi = perm(raw[r][5], raw[r][4], 0x07030602u);
          u[0] = ef_lo; u[1] = ef_lo >> 16; u[2] = ef_hi; u[3] = ef_hi >> 16;
#pragma unroll
          for (int ch = 0; ch < 4; ++ch) {
            win[ch][0] = t[ch];
            win[ch][1] = __builtin_amdgcn_alignbyte(u[ch], t[ch], 2);
          }
        } else {
          transpose4(raw[r][4], raw[r][5], raw[r][NCOL - 3], raw[r][NCOL - 2], u);
#pragma unroll
          for (int ch = 0; ch < 4; ++ch) {
            win[ch][0] = t[ch];
            win[ch][1] = __builtin_amdgcn_alignbyte(u[ch], t[ch], 2);
            win[ch][2] = u[ch];
            win[ch][3] = __builtin_amdgcn_alignbyte(raw[r][NCOL - 1] >> (8 * ch), u[ch], 2);
          }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int ch = 0; ch < 4; ++ch)
            a[4 * q + ch] = __builtin_amdgcn_sdot4((int)win[ch][STRIDE == 1 ? q >> 1 : q], (int)wt[r][ch][STRIDE == 1 ? q & 1 : 0], a[4 * q + ch], false);
      }
      // the last dot products' wait states once for all sixteen, then clip and shift-and-pack
      settle_dots(a);
#pragma unroll
      for (int i = 0; i < 16; ++i) a[i] = clamp_med3(a[i], tl.lo_scaled, tl.hi_scaled);
      const v4i out = shift_pack16(a, p.d_shift);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (q0 + q < p.Q) *reinterpret_cast<uint32_t *>(lds + (pl * p.Q + q0 + q) * tl.pitch + c) = (uint32_t)out[q] ^ p.d_xor;
    }
  }

  // ---- 1x1: wave -> channel block wave % nb, K slices wave / nb, + kg, ... ---------------------------------
  const int nbi = wave % tl.nb, kgi = wave / tl.nb;
  const bool active = kgi < tl.kg;
  const int8_t *wf = p.wf + ((size_t)nbi * tl.ks * 64 + lane) * 16;
  constexpr int PF = 4;                              // slices of weights on their way
  v4i wq[PF];
  if (active) {
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      const int s = kgi + i * tl.kg;
      wq[i] = *reinterpret_cast<const v4i *>(wf + (size_t)(s < tl.ks ? s : kgi) * 1024);
    }
  }
  v16i acc[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[mb][i] = 0;
  __syncthreads();                                   // the depthwise result is complete
  if (active) {
    for (int s0 = kgi; s0 < tl.ks; s0 += PF * tl.kg) {
#pragma unroll
      for (int i = 0; i < PF; ++i) {
        const int s = s0 + i * tl.kg;
        if (s < tl.ks) {                             // uniform
          const v4i w = wq[i];
          const int ahead = s + PF * tl.kg;
          if (ahead < tl.ks) wq[i] = *reinterpret_cast<const v4i *>(wf + (size_t)ahead * 1024);
#pragma unroll
          for (int mb = 0; mb < MB; ++mb) {
            const v4i x = *reinterpret_cast<const v4i *>(lds + (mb * 32 + l32) * tl.pitch + s * 32 + half * 16);
            acc[mb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w, x, acc[mb], 0, 0, 0);
          }
        }
      }
    }
  }
  __syncthreads();                                   // nobody reads the depthwise result any more
  if (active) {
    uint8_t *part = lds + (kgi * tl.nb + nbi) * (MB * 32 * PART_PITCH) + l32 * PART_PITCH + half * 64;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<v4i *>(part + mb * (32 * PART_PITCH) + q * 16) =
            v4i{acc[mb][4 * q], acc[mb][4 * q + 1], acc[mb][4 * q + 2], acc[mb][4 * q + 3]};
  }
  __syncthreads();
  for (int it = tid; it < npx * tl.np; it += NT) {
    const int m = (int)tl.fd_np.div((uint32_t)it), n = (it - m * tl.np) * 8;
    const size_t o = (px0 + m) * p.N + n;
    const v2i res = p.res ? *reinterpret_cast<const v2i *>(p.res + o) : v2i{0, 0};
    int v[8];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      v4i a = *reinterpret_cast<const v4i *>(p.acc0 + n + 4 * q);
      for (int k = 0; k < tl.kg; ++k)
        a += *reinterpret_cast<const v4i *>(lds + (k * tl.nb + (n >> 5)) * (MB * 32 * PART_PITCH) + m * PART_PITCH + ((n & 31) + 4 * q) * 4);
      v[4 * q] = a.x; v[4 * q + 1] = a.y; v[4 * q + 2] = a.z; v[4 * q + 3] = a.w;
    }
    if (p.res) {
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] += align_res(byte_of((uint32_t)res[i >> 2], i & 3, p.res_signed != 0), p.res_d);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = requant<false>(v[i], p.shift, p.lo, p.hi);
    *reinterpret_cast<v2i *>(p.y + o) = v2i{(int)pack4(v[0], v[1], v[2], v[3]), (int)pack4(v[4], v[5], v[6], v[7])};
  }
}

// Fragment (32-channel block nb, K slice s) is 64 pieces of 16 bytes; piece `lane` is channel 32 nb + frag(l32), bytes
// 32 s + 16 half .. + 16 of its C; zeros past N or C.
__global__ __launch_bounds__(256) void dw_pw_weights_kernel(const int8_t *__restrict__ w, int8_t *__restrict__ wf, int C, int N, int total) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  const int ks = (C + 31) / 32;
  const int lane = i & 63, s = (i >> 6) % ks, nb = (i >> 6) / ks;
  const int n = 32 * nb + weight_row(lane & 31), k = 32 * s + 16 * (lane >> 5);
  union { int8_t b[16]; v4i v; } u;
#pragma unroll
  for (int j = 0; j < 16; ++j) u.b[j] = n < N && k + j < C ? w[(size_t)n * C + k + j] : 0;
  *reinterpret_cast<v4i *>(wf + (size_t)i * 16) = u.v;
}

template <int STRIDE, int MB>
int launch_shape(const DwPwParams &p, const DwPwTiling &tl, int lds, long long grid, hipStream_t stream) {
  const void *fn = reinterpret_cast<const void *>(dw_pw_kernel<STRIDE, MB>);
  static std::atomic<unsigned long long> done_mask{0};         // devices whose LDS limit has been raised
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return (int)hipErrorInvalidDevice;
  if (dev < 0 || dev > 63 || !((done_mask.load(std::memory_order_relaxed) >> dev) & 1ull)) {
    const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return (int)e;
    if (dev >= 0 && dev <= 63) done_mask.fetch_or(1ull << dev, std::memory_order_relaxed);
  }
  hipLaunchKernelGGL((dw_pw_kernel<STRIDE, MB>), dim3((unsigned)grid), dim3(NT), lds, stream, p, tl);
  return (int)hipGetLastError();
}

}  // namespace

int dw_pw_slices(int C, int N) {
  const int ks = (C + 31) / 32, share = NWAVE / ((N + 31) / 32);     // waves that share K (N is at most 256)
  return (ks + share - 1) / share;
}

size_t dw_pw_weight_bytes(int C, int N) { return (size_t)((N + 31) / 32) * ((C + 31) / 32) * 1024; }

int launch_dw_pw_weights(const int8_t *w, int8_t *wf, int C, int N, hipStream_t stream) {
  const int total = (int)(dw_pw_weight_bytes(C, N) / 16);
  hipLaunchKernelGGL(dw_pw_weights_kernel, dim3((total + 255) / 256), dim3(256), 0, stream, w, wf, C, N, total);
  return (int)hipGetLastError();
}

bool dw_pw_applicable(int C, int N, int Q, int d_shift, int shift, const void *x, const void *wd, const void *y, const void *res) {
  if (C < 16 || (C & 15) || C > 1024 || N < 8 || (N & 7) || N > 256 || Q < 1 || Q > 128 || d_shift < 0 || shift < 0) return false;
  return ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(wd)) & 3) == 0 &&
         ((reinterpret_cast<uintptr_t>(y) | reinterpret_cast<uintptr_t>(res)) & 7) == 0;
}

int launch_dw_pw(const DwPwParams &p, hipStream_t stream) {
  if (p.B <= 0) return 0;
  if (!dw_pw_applicable(p.C, p.N, p.Q, p.d_shift, p.shift, p.x, p.wd, p.y, p.res) || (p.stride != 1 && p.stride != 2) ||
      (long long)p.H * p.W * p.C > 0x7fffffffLL || (reinterpret_cast<uintptr_t>(p.acc0) & 15) || (reinterpret_cast<uintptr_t>(p.wf) & 15))
    return (int)hipErrorInvalidValue;
  DwPwTiling tl;
  // rows per workgroup: as few as give 192 workgroups (a row at least), as many as fit 64 pixels (128 where a row is longer)
  const int cap = p.Q > 64 ? 128 : 64;
  int rows = cap / p.Q;
  while (rows > 1 && (long long)p.B * ((p.P + rows - 1) / rows) < 192) --rows;
  tl.rows = rows > p.P ? p.P : rows;
  tl.tiles = (p.P + tl.rows - 1) / tl.rows;
  const int px = tl.rows * p.Q, mb = px > 64 ? 4 : px > 32 ? 2 : 1;
  tl.dw = p.C / 4;
  tl.groups = NT / tl.dw;
  tl.strips = (p.Q + 3) / 4;
  tl.pitch = (p.C / 16) & 1 ? p.C : p.C + 16;          // an odd number of 16-byte pieces: 16 pixels' reads spread over all banks
  tl.ks = (p.C + 31) / 32;
  tl.nb = (p.N + 31) / 32;
  tl.kg = NWAVE / tl.nb < tl.ks ? NWAVE / tl.nb : tl.ks;
  tl.np = p.N / 8;
  tl.x_image = p.H * p.W * p.C;
  const ScaledClip sc = scaled_clip(p.d_lo, p.d_hi, p.d_shift);
  tl.lo_scaled = sc.lo; tl.hi_scaled = sc.hi;
  tl.fd_tiles = FastDiv((uint32_t)tl.tiles);
  tl.fd_dw = FastDiv((uint32_t)tl.dw);
  tl.fd_strips = FastDiv((uint32_t)tl.strips);
  tl.fd_np = FastDiv((uint32_t)tl.np);
  // the depthwise result of mb * 32 pixels (and what the last K slice of the last pixel reads past it), then the sums
  const int result = mb * 32 * tl.pitch + 32, sums = tl.kg * tl.nb * mb * 32 * PART_PITCH;
  const int lds = result > sums ? result : sums;
  const long long grid = (long long)p.B * tl.tiles;
  if (lds > 160 * 1024 || grid > 0x7fffffffLL) return (int)hipErrorInvalidValue;
  switch (p.stride * 8 + mb) {
    case 8 + 1: return launch_shape<1, 1>(p, tl, lds, grid, stream);
    case 8 + 2: return launch_shape<1, 2>(p, tl, lds, grid, stream);
    case 8 + 4: return launch_shape<1, 4>(p, tl, lds, grid, stream);
    case 16 + 1: return launch_shape<2, 1>(p, tl, lds, grid, stream);
    case 16 + 2: return launch_shape<2, 2>(p, tl, lds, grid, stream);
    case 16 + 4: return launch_shape<2, 4>(p, tl, lds, grid, stream);
    default: return (int)hipErrorInvalidValue;
  }
}

}  // namespace f8
