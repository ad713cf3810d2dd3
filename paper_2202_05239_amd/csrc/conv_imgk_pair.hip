// A basic residual block of 64 or 128 channels (3x3, 3x3, shortcut; F8Net Eq. 6 twice) in one launch, image-stationary as
// conv_imgk.hip.
//
// Apart, each of the two layers reads and writes the whole tensor (12.8 MB each way for 64 images of 56 x 56) and pays for
// a launch, its own prologue and its last stores.  A workgroup of eight waves takes a band of output rows: the input rows
// under it (two more on either side) lie in LDS, the first layer's result (one more row on either side: computed by the neighbours
// too, that is the price) beside them, and only the second layer's result leaves.  The shortcut is read from the input rows.
//
// 64 channels: a wave holds one layer's weights, all 36 fragments, in registers and takes every eighth block of 32 pixels with all
// channels, so a pixel fragment is read from LDS once for two matrix instructions: with one block of channels
// per wave the reads alone would take as long as the products.  128 channels: a wave holds the 36 fragments of one block of 32 channels
// and takes 64 pixels at a time.  The second layer's weights come in as the last block of the
// first is done with the first's.
//
// 64 images of 56 x 56 (256 workgroups, one per CU): 25.2 us in two launches, 19.6 in one; the products alone are 7.7 at the full rate, the
// input rows and the weights in front of them 3 - 4, the stores behind them 2.
#include "conv_imgk_pair.h"

#include <atomic>
#include <type_traits>

namespace f8 {
namespace {

typedef int v16i __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) uint8_t lds_u8;
typedef __attribute__((address_space(3))) v4i lds_v4i;

constexpr int NT = 512, NWAVE = NT / 64;
constexpr int LDS_MOST = 160 * 1024;
constexpr int px_bytes(int C) { return C + 16; }        // of a pixel in LDS: 16 pixels of a row start on different banks
// A wave's share: blocks of channels, blocks of pixels at a time, waves side by side over the channels.
constexpr int channel_blocks(int C) { return C == 64 ? 2 : 1; }
constexpr int pixel_blocks(int C) { return 3 - channel_blocks(C); }
constexpr int waves_across(int C) { return C / 32 / channel_blocks(C); }

struct Args {
  const uint8_t *x;
  const int8_t *wa, *wb;
  const int32_t *acc_a, *acc_b;
  uint8_t *y;
  int x_bytes, H, W, rows, bands, at_e, at_start;
  uint32_t x_xor, e_xor;
  ScaledClip clip_a, clip_b;
  int shift_a, shift_b, has_res, res_d, res_bias;
  FastDiv by_bands, by_w;
};

__device__ __forceinline__ v4i lds_read(uint32_t at) { return *(lds_v4i *)(uintptr_t)at; }
__device__ __forceinline__ void lds_write(uint32_t at, v4i v) { *(lds_v4i *)(uintptr_t)at = v; }

__device__ __forceinline__ v4i requant16(v16i &a, ScaledClip c, int shift, int x) {
  settle_matrix_result(a);
  int v[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = clamp_med3(a[i], c.lo, c.hi);
  const v4i r = shift_pack16(v, shift);
  return v4i{r.x ^ x, r.y ^ x, r.z ^ x, r.w ^ x};
}

template <int C>
__global__ __launch_bounds__(NT, 1) void conv_pair_kernel(const Args a) {
  constexpr int PX = px_bytes(C), KS = C / 32, SLICES = 9 * KS, PIECES = C / 16;
  constexpr int CB = channel_blocks(C), PB = pixel_blocks(C), WN = waves_across(C), MW = NWAVE / WN;
  pin_args(a.x, a.wa, a.wb, a.acc_a, a.acc_b, a.y, a.x_bytes, a.H, a.W, a.rows, a.bands, a.at_e, a.at_start, a.x_xor, a.e_xor, a.clip_a.lo,
           a.clip_a.hi, a.clip_b.lo, a.clip_b.hi, a.shift_a, a.shift_b, a.has_res, a.res_d, a.res_bias, a.by_bands.mul, a.by_bands.shr,
           a.by_bands.d, a.by_w.mul, a.by_w.shr, a.by_w.d);
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const uint32_t base = (uint32_t)(uintptr_t)((lds_u8 *)lds);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5, nb0 = wave % WN * CB, mw = wave / WN;
  const int wg = (int)xcd_remap(blockIdx.x, gridDim.x);
  const int img = (int)a.by_bands.div((uint32_t)wg), p0 = (wg - img * a.bands) * a.rows;
  const int out_rows = min(a.rows, a.H - p0), lw = a.W + 2;            // LDS rows have a column of zeros at either end
  const int x_lo = max(p0 - 2, 0), x_hi = min(p0 + out_rows + 2, a.H); // input rows; LDS row 0 is row p0 - 2
  const int e_lo = max(p0 - 1, 0), e_hi = min(p0 + out_rows + 1, a.H); // rows of the first result; LDS row 0 is row p0 - 1
  const int npx = (e_hi - e_lo) * a.W, opx = out_rows * a.W;

  // ---- input rows: contiguous in memory
  const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(a.x), 0, a.x_bytes, 0x00027000);
  const int n16 = (x_hi - x_lo) * a.W * (C / 16), first = (img * a.H + x_lo) * a.W * C, xm = (int)a.x_xor, em = (int)a.e_xor;
  constexpr int XU = 8;
  v4i piece[XU];
  auto fetch = [&](int i0) {
#pragma unroll
    for (int k = 0; k < XU; ++k) {
      const int i = i0 + k * NT + tid;
      piece[k] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(xres, i < n16 ? (uint32_t)(first + i * 16) : 0x80000000u, 0, 0));
    }
  };
  auto put = [&](int i0) {
#pragma unroll
    for (int k = 0; k < XU; ++k) {
      const int i = i0 + k * NT + tid, px = i / PIECES, r = (int)a.by_w.div((uint32_t)px), c = px - r * a.W;
      if (i < n16)
        lds_write(base + ((r + x_lo - (p0 - 2)) * lw + c + 1) * PX + i % PIECES * 16,
                  v4i{piece[k].x ^ xm, piece[k].y ^ xm, piece[k].z ^ xm, piece[k].w ^ xm});
    }
  };
  fetch(0);
  // ---- this layer's weights
  v4i w[CB * SLICES];
  const __amdgpu_buffer_rsrc_t ares = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t *>(a.wa), 0, KS * SLICES * 1024, 0x00027000);
  const __amdgpu_buffer_rsrc_t bres = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t *>(a.wb), 0, KS * SLICES * 1024, 0x00027000);
  auto weight = [&](__amdgpu_buffer_rsrc_t from, int t) {
    return __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(from, lane * 16, (nb0 * SLICES + t) * 1024, 0));
  };
#pragma unroll
  for (int t = 0; t < CB * SLICES; ++t) w[t] = weight(ares, t);
  if (tid < 2 * C) {
    const int v = tid < C ? a.acc_a[tid] : a.acc_b[tid - C] + a.res_bias;
    *(__attribute__((address_space(3))) int *)(uintptr_t)(base + a.at_start + tid * 4) = v;
  }
  // ---- zeros around the rows of both tensors: the columns beside the image, and whole rows above or below it
  {
    auto zero_row = [&](uint32_t row, int z) {
      for (int i = tid; i < lw * PIECES; i += NT) lds_write(row + i / PIECES * PX + i % PIECES * 16, v4i{z, z, z, z});
    };
    for (int i = tid; i < (2 * out_rows + 6) * 2 * PIECES; i += NT) {
      const int row = i / (2 * PIECES), side = i / PIECES & 1;
      const bool e = row >= out_rows + 4;
      const uint32_t at = base + (e ? a.at_e + (row - out_rows - 4) * lw * PX : row * lw * PX) + side * (lw - 1) * PX + i % PIECES * 16;
      const int z = e ? em : xm;
      lds_write(at, v4i{z, z, z, z});
    }
    for (int r = 0; r < out_rows + 4; ++r)
      if (p0 - 2 + r < 0 || p0 - 2 + r >= a.H) zero_row(base + r * lw * PX, xm);
    if (p0 == 0) zero_row(base + a.at_e, em);
    if (p0 + out_rows == a.H) zero_row(base + a.at_e + (out_rows + 1) * lw * PX, em);
  }
  put(0);
  for (int i0 = XU * NT; i0 < n16; i0 += XU * NT) { fetch(i0); put(i0); }
  __syncthreads();

  auto start16 = [&](int block) {
    v16i v;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const v4i s = lds_read(base + a.at_start + block * 128 + half * 64 + g * 16);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[4 * g + i] = s[i];
    }
    return v;
  };
  // Two blocks of 32 pixels x 32 channels, their windows from `from` on (this lane's pixels), fragments read ahead; REPLACE: each
  // fragment of the weights gives way to the second layer's when it has been used.  (The barriers keep the compiler from
  // reading all fragments first: with 36 of the weights there are no registers for them.)
  auto products = [&](const uint32_t (&from)[PB], v16i (&acc)[2], auto replace) {
    constexpr int AHEAD = 4;
    v4i f[AHEAD][PB];
    auto pixel = [&](int t, int p) { return lds_read(from[p] + (t / KS / 3) * lw * PX + (t / KS % 3) * PX + t % KS * 32); };
#pragma unroll
    for (int t = 0; t < AHEAD; ++t)
#pragma unroll
      for (int p = 0; p < PB; ++p) f[t][p] = pixel(t, p);
#pragma unroll
    for (int t = 0; t < SLICES; ++t) {
#pragma unroll
      for (int b = 0; b < 2; ++b)
        acc[b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w[b % CB * SLICES + t], f[t % AHEAD][b % PB], acc[b], 0, 0, 0);
      if constexpr (decltype(replace)::value)
#pragma unroll
        for (int b = 0; b < CB; ++b) w[b * SLICES + t] = weight(bres, b * SLICES + t);
      if (t + AHEAD < SLICES)
#pragma unroll
        for (int p = 0; p < PB; ++p) f[t % AHEAD][p] = pixel(t + AHEAD, p);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // ---- first layer
  const int mb1 = (npx + 32 * PB - 1) / (32 * PB), mb2 = (opx + 32 * PB - 1) / (32 * PB);
  auto first_unit = [&](int mb, auto replace) {
    uint32_t from[PB], to[PB];
#pragma unroll
    for (int p = 0; p < PB; ++p) {
      const int ic = min((mb * PB + p) * 32 + l32, npx - 1), r = (int)a.by_w.div((uint32_t)ic), c = ic - r * a.W;
      from[p] = base + ((r + e_lo - p0 + 1) * lw + c) * PX + half * 16;
      to[p] = base + a.at_e + ((r + e_lo - (p0 - 1)) * lw + c + 1) * PX + half * 16 + nb0 * 32;
    }
    v16i acc[2] = {start16(nb0), start16(nb0 + CB - 1)};
    products(from, acc, replace);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const v4i v = requant16(acc[b], a.clip_a, a.shift_a, em);
      if ((mb * PB + b % PB) * 32 + l32 < npx) lds_write(to[b % PB] + b % CB * 32, v);
    }
  };
  int mb = mw;
  for (; mb + MW < mb1; mb += MW) first_unit(mb, std::false_type{});
  first_unit(mb, std::true_type{});       // (past the last block: nothing is stored, the weights change all the same)
  __syncthreads();

  // ---- second layer
  uint8_t *const y = a.y + ((size_t)img * a.H + p0) * a.W * C + half * 16 + nb0 * 32;
  for (mb = mw; mb < mb2; mb += MW) {
    uint32_t from[PB], shortcut[PB];
#pragma unroll
    for (int p = 0; p < PB; ++p) {
      const int jc = min((mb * PB + p) * 32 + l32, opx - 1), r = (int)a.by_w.div((uint32_t)jc), c = jc - r * a.W;
      from[p] = base + a.at_e + (r * lw + c) * PX + half * 16;
      shortcut[p] = base + ((r + 2) * lw + c + 1) * PX + half * 16 + nb0 * 32;
    }
    v16i acc[2] = {start16(KS + nb0), start16(KS + nb0 + CB - 1)};
    products(from, acc, std::false_type{});
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      settle_matrix_result(acc[b]);
      if (a.has_res) {
        const v4i s = lds_read(shortcut[b % PB] + b % CB * 32);
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[b][i] += (int)(int8_t)((uint32_t)s[i >> 2] >> (8 * (i & 3))) << a.res_d;
      }
      const v4i v = requant16(acc[b], a.clip_b, a.shift_b, 0);
      const int j = (mb * PB + b % PB) * 32 + l32;
      if (j < opx) *reinterpret_cast<v4i *>(y + (size_t)j * C + b % CB * 32) = v;
    }
  }
}

int at_e_of(int C, int W, int rows) { return (rows + 4) * (W + 2) * px_bytes(C); }
int at_start_of(int C, int W, int rows) { return at_e_of(C, W, rows) + (rows + 2) * (W + 2) * px_bytes(C); }
int lds_bytes(int C, int W, int rows) { return at_start_of(C, W, rows) + 2 * C * 4; }

// Output rows per workgroup, by what a launch of them would take: set-up and the blocks a wave works through one after the
// other, in rounds of one workgroup per CU.  0: no number of rows fits.
int rows_for(int C, int H, int W, int B) {
  const int px = 32 * pixel_blocks(C), mw = NWAVE / waves_across(C);
  int best = 0;
  long long least = 0;
  for (int rows = 1; rows <= H && lds_bytes(C, W, rows) <= LDS_MOST; ++rows) {
    const int e_rows = rows + 2 < H ? rows + 2 : H, bands = (H + rows - 1) / rows;
    const int units = ((e_rows * W + px - 1) / px + mw - 1) / mw + ((rows * W + px - 1) / px + mw - 1) / mw;
    const long long cost = (9000 + (C == 64 ? 2600ll : 5200ll) * units) * (((long long)B * bands + 255) / 256);
    if (best == 0 || cost < least) { best = rows; least = cost; }
  }
  return best;
}

template <int C>
int launch_one(const Args &a, int lds, long long grid, hipStream_t stream) {
  static std::atomic<unsigned long long> done_mask{0};         // devices whose LDS limit has been raised
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return (int)hipErrorInvalidDevice;
  if (dev < 0 || dev > 63 || !((done_mask.load(std::memory_order_relaxed) >> dev) & 1ull)) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(conv_pair_kernel<C>), hipFuncAttributeMaxDynamicSharedMemorySize, LDS_MOST);
    if (e != hipSuccess) return (int)e;
    if (dev >= 0 && dev <= 63) done_mask.fetch_or(1ull << dev, std::memory_order_relaxed);
  }
  hipLaunchKernelGGL((conv_pair_kernel<C>), dim3((unsigned)grid), dim3(NT), lds, stream, a);
  return (int)hipGetLastError();
}

}  // namespace

bool conv_pair_applicable(int C, int H, int W, int shift_a, int shift_b, bool has_res, int res_d, const void *x, const void *y) {
  if ((C != 64 && C != 128) || H < 1 || W < 1 || W > 512 || shift_a < 0 || shift_b < 0 || (has_res && (res_d < 0 || res_d > 16))) return false;
  if ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(y)) & 15) return false;
  return rows_for(C, H, W, 1) > 0;
}

int launch_conv_pair(const ConvPairParams &p, hipStream_t stream) {
  if (p.B <= 0) return 0;
  if (!conv_pair_applicable(p.C, p.H, p.W, p.shift_a, p.shift_b, p.has_res != 0, p.res_d, p.x, p.y) ||
      ((reinterpret_cast<uintptr_t>(p.wa) | reinterpret_cast<uintptr_t>(p.wb)) & 15) || (long long)p.B * p.H * p.W * p.C > 0x7fffffffLL)
    return (int)hipErrorInvalidValue;
  Args a;
  a.x = p.x; a.wa = p.wa; a.wb = p.wb; a.acc_a = p.acc_a; a.acc_b = p.acc_b; a.y = p.y;
  a.x_bytes = p.B * p.H * p.W * p.C;
  a.H = p.H; a.W = p.W;
  a.rows = rows_for(p.C, p.H, p.W, p.B);
  a.bands = (p.H + a.rows - 1) / a.rows;
  a.at_e = at_e_of(p.C, p.W, a.rows);
  a.at_start = at_start_of(p.C, p.W, a.rows);
  a.x_xor = p.x_xor; a.e_xor = p.e_xor;
  a.clip_a = scaled_clip(p.lo_a, p.hi_a, p.shift_a);
  a.clip_b = scaled_clip(p.lo_b, p.hi_b, p.shift_b);
  a.shift_a = p.shift_a; a.shift_b = p.shift_b;
  a.has_res = p.has_res; a.res_d = p.has_res ? p.res_d : 0;
  a.res_bias = p.has_res && p.x_xor ? 128 << a.res_d : 0;
  a.by_bands = FastDiv((uint32_t)a.bands);
  a.by_w = FastDiv((uint32_t)p.W);
  const long long grid = (long long)p.B * a.bands;
  if (grid > 0x7fffffffLL) return (int)hipErrorInvalidValue;
  const int lds = lds_bytes(p.C, p.W, a.rows);
  return p.C == 64 ? launch_one<64>(a, lds, grid, stream) : launch_one<128>(a, lds, grid, stream);
}

}  // namespace f8
