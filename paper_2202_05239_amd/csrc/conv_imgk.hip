// Image-stationary 3x3 convolution, stride 1, pad 1, with K shared among the waves of a workgroup (the 3x3
// layers of ResNet stages 2-4 at small and medium batch), with the residual / shift / clip epilogue of
// F8Net Eq. 2 / Eq. 9.
//
// With one GEMM tile per CU a step of 128 bytes of K costs the wave's own chain of barrier, LDS reads and
// address work (0.5 - 0.7 us whatever the tile or the depth of the ring; the matrix instructions in it take
// 0.12 - 0.25 us): 17 us for 256 -> 256 channels on 64 images of 14 x 14, 25 us for 512 -> 512 on 64 of
// 7 x 7, of which 4 us are matrix work.  Here, as in conv_img.hip, the input pixels of a workgroup sit in
// LDS once with a border of zeros (an activation is read from memory once, not nine times), every tap's
// fragment is read from that patch at a constant offset, weights stream from L2 straight into registers in
// fragment order (RING slices ahead: 1300 - 1800 cycles), and the loop has no barrier.  Unlike there, a workgroup
// computes only a part of the output channels, which makes workgroups out of few images: wave wn has 32
// channels of its own, and where that still leaves CUs idle, WK waves share K instead (wave kg takes the input
// channels kg * C / WK onwards of every tap) and their sums meet in LDS at the end.
//   C = 256: a whole image of up to 224 pixels (7 blocks of 32); C = 512: two 7 x 7 images (4 blocks);
//   C = 128: a band of up to 224 pixels.
// Now 12.2 us for 256 channels on 64 images and 12.2 us for 512 (two waves share K), 17.7 / 19.2 us on 128 images
// (22.4 / 28.6 before); 9.5 k cycles of a workgroup's 19.5 k are the loop (8.1 k of matrix instructions),
// 5.3 k the patch (82 - 92 KiB at the 60 bytes per clock a CU gets from L2, then memory latency), 4 k the sums in
// LDS and the stores.  With 64 channels per wave and four waves sharing K the loop reads half as much from LDS
// but the sums take twice as long: 12.8 us.
#include "conv_imgk.h"

#include <atomic>

namespace f8 {
namespace {

typedef int v16i __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) const v4i lds_v4i;
typedef __attribute__((address_space(3))) const uint8_t lds_u8;

constexpr int NT = 256;
constexpr int PART_PITCH = 32 * 4 + 16;              // a pixel's 32 partial sums

// MB: 32-pixel blocks of a workgroup; a wave's part of the patch is RPW rows of up to NI KiB.
template <int C> struct Shape;
template <> struct Shape<128> { static constexpr int MB = 7, RPW = 3, NI = 4; };
template <> struct Shape<256> { static constexpr int MB = 7, RPW = 5, NI = 4; };
template <> struct Shape<512> { static constexpr int MB = 4, RPW = 5, NI = 5; };

// How the batch is cut into units of one workgroup: whole images, or bands of rows of one image.
struct Units {
  int images;             // images per unit
  int rows;               // output rows of an image per unit (H for whole images)
  int bands;              // units per image (1 for whole images)
  int prows, pcols;       // patch rows per image and patch columns
  int all_rows;           // patch rows
  int group;              // bytes of one K group's part of the patch
  int lds;
  long long units;
};

template <int C> Units cut(int B, int H, int W, int WK) {
  using S = Shape<C>;
  constexpr int cap = S::MB * 32, max_rows = 4 * S::RPW;
  const int gpitch = C / WK + 16;
  Units u{};
  if (H < 1 || W < 1 || W > cap || (W + 2) * C > S::NI * 1024) return u;
  u.images = H + 2 > max_rows ? 0 : cap / (H * W);
  if (u.images > max_rows / (H + 2)) u.images = max_rows / (H + 2);
  if (u.images >= 1) {
    u.rows = H; u.bands = 1;
  } else {
    const int most = cap / W < max_rows - 2 ? cap / W : max_rows - 2;
    u.images = 1;
    u.bands = (H + most - 1) / most;
    u.rows = (H + u.bands - 1) / u.bands;            // bands of equal height
    u.bands = (H + u.rows - 1) / u.rows;
  }
  u.prows = u.rows + 2; u.pcols = W + 2;
  u.all_rows = u.images * u.prows;
  // (behind the patch: what the fragment reads issued after the last slice touch)
  u.group = ((u.all_rows + 1) * u.pcols + 2) * gpitch;
  const int part = WK == 1 ? 0 : 4 * S::MB * 32 * PART_PITCH, patch = WK * u.group;
  u.lds = patch > part ? patch : part;
  u.units = u.bands > 1 ? (long long)B * u.bands : (B + u.images - 1) / u.images;
  if (u.lds > 160 * 1024) u.images = 0;              // does not fit
  return u;
}

// Channel fed as row r of a 32-channel block: see conv_img.hip (the fragment order has it built in).

template <int C, int WK>
__global__ __launch_bounds__(NT, WK == 1 ? 2 : 1) void conv_imgk_kernel(const ConvImgkParams p, const Units u, const FastDiv fd_w, const FastDiv fd_px,
                                                          const FastDiv fd_prows, const FastDiv fd_units) {
  using S = Shape<C>;
  constexpr int MB = S::MB, WN = 4 / WK;
  constexpr int KPT = C / 32;                        // K slices per tap
  constexpr int KSW = KPT / WK;                      // of which a wave takes this many
  constexpr int KS = 9 * KPT;
  constexpr int CG = C / WK, GP = CG + 16;           // bytes of a patch pixel in one K group
  constexpr int PIECES = C / 16;                     // 16-byte pieces per pixel
  constexpr int ROW_SLICES = 3 * KSW;                // K slices per window row
  constexpr int RING = MB == 7 ? (ROW_SLICES % 8 == 0 ? 8 : 6) : 12;
  static_assert(ROW_SLICES % RING == 0 && ROW_SLICES % 2 == 0, "slots and fragment sets repeat from row to row");
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  const int kg = wave % WK, wn = wave / WK;
  // workgroups of one channel slice are neighbours on an XCD: they stream the same weights
  const uint32_t bid = xcd_remap(blockIdx.x, gridDim.x);
  const int slice = (int)fd_units.div(bid), unit = (int)bid - slice * (int)fd_units.d;
  const int n0 = slice * (32 * WN);
  int img0, y0, nimg, rows;
  if (u.bands > 1) {
    img0 = unit / u.bands;
    y0 = (unit - img0 * u.bands) * u.rows;
    nimg = 1; rows = min(u.rows, p.H - y0);
  } else {
    img0 = unit * u.images;
    y0 = 0;
    nimg = min(u.images, p.B - img0); rows = p.H;
  }
  const int npx = nimg * rows * p.W;                 // output pixels of this unit, consecutive in memory
  const size_t px0 = ((size_t)img0 * p.H + y0) * p.W;

  // ---- this wave's weights: channel block n0 / 32 + wn, K slices kg * KSW .. + KSW of every tap.  Slice sc of window
  // row r is requested RING slices ahead.
  const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<int8_t *>(p.wf) + (size_t)(n0 / 32 + wn) * (KS * 1024), 0, KS * 1024, 0x00027000);
  const int lane16 = lane * 16, wbase = kg * (KSW * 1024);
  auto slice_at = [](int sc) { return ((sc / KSW) * KPT + sc % KSW) * 1024; };
  v4i bq[RING];
#pragma unroll
  for (int sc = 0; sc < RING; ++sc) bq[sc] = __builtin_amdgcn_raw_buffer_load_b128(wres, lane16, wbase + slice_at(sc), 0);

  // ---- the input pixels and a border of zeros into LDS, xor 0x80 when unsigned.  A wave takes the patch rows
  // wave, wave + 4, ...; a row's pixels are consecutive in memory, so a lane's 16-byte pieces of a row lie at
  // fixed offsets from its first pixel (the scalar part of the address) and at fixed places in a patch row.
  // Border columns: an offset the descriptor rejects, which reads as zero; border rows: an empty descriptor.
  const size_t image_bytes = (size_t)p.H * p.W * C;
  uint8_t *xbase = const_cast<uint8_t *>(p.x) + (size_t)img0 * image_bytes;
  uint32_t x_at[S::NI];
  v4i px[S::RPW][S::NI];
#pragma unroll
  for (int i = 0; i < S::NI; ++i) {
    const int col = (i * 64 + lane) / PIECES;
    x_at[i] = (unsigned)(col - 1) < (unsigned)p.W ? (uint32_t)((i * 64 + lane) * 16 - C) : 0x80000000u;
  }
#pragma unroll
  for (int k = 0; k < S::RPW; ++k) {
    const int row = wave + 4 * k;                    // uniform
    const int img = (int)fd_prows.div((uint32_t)row), y = y0 + row - img * u.prows - 1;
    const bool in = img < nimg && (unsigned)y < (unsigned)p.H;
    const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(xbase, 0, in ? nimg * (int)image_bytes : 0, 0x00027000);
    const int at = in ? (img * p.H + y) * p.W * C : 0;
#pragma unroll
    for (int i = 0; i < S::NI; ++i) px[k][i] = __builtin_amdgcn_raw_buffer_load_b128(xres, x_at[i], at, 0);
  }
  __builtin_amdgcn_sched_barrier(0);

  // (while they are on their way)
  // Fragment row 32 j + l32 is output pixel m of the unit; its window starts at patch pixel (image, y, x).
  // Rows past the last pixel read the patch's first window; their sums are dropped.
  lds_u8 *ar[MB];
#pragma unroll
  for (int j = 0; j < MB; ++j) {
    const int m = 32 * j + l32;
    int at = 0;
    if (m < npx) {
      const int img = (int)fd_px.div((uint32_t)m), rem = m - img * (int)fd_px.d;
      const int y = (int)fd_w.div((uint32_t)rem), x = rem - y * p.W;
      at = (img * u.prows + y) * u.pcols + x;
    }
    ar[j] = (lds_u8 *)lds + kg * u.group + at * GP + 16 * half;
  }
  v16i acc[MB];
#pragma unroll
  for (int j = 0; j < MB; ++j)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[j][i] = 0;
  int to[S::NI];
#pragma unroll
  for (int i = 0; i < S::NI; ++i) {
    const int col = (i * 64 + lane) / PIECES, piece = lane % PIECES;
    // (pieces past the last column are fetched as zeros and not kept)
    to[i] = col < u.pcols ? (piece / (CG / 16)) * u.group + col * GP + (piece % (CG / 16)) * 16 : -1;
  }
  static_assert(64 % PIECES == 0, "a lane keeps its piece of a pixel");
  __builtin_amdgcn_sched_barrier(0);
  const int zx = (int)p.x_xor;
#pragma unroll
  for (int k = 0; k < S::RPW; ++k) {
    const int row = wave + 4 * k;
    if (row < u.all_rows) {
#pragma unroll
      for (int i = 0; i < S::NI; ++i)
        if (to[i] >= 0)
          *reinterpret_cast<v4i *>(lds + row * u.pcols * GP + to[i]) = v4i{px[k][i].x ^ zx, px[k][i].y ^ zx, px[k][i].z ^ zx, px[k][i].w ^ zx};
    }
  }
  __syncthreads();                                   // the patch is complete

  // ---- K loop: a pass is a row of the window, 3 taps x KSW slices; activation fragments one slice ahead,
  // one request at a time behind the matrix instructions
  v4i xf[2][MB];
#pragma unroll
  for (int j = 0; j < MB; ++j) xf[0][j] = *(lds_v4i *)(ar[j]);
  const int row_step = u.pcols * GP;
#pragma unroll 1
  for (int r = 0; r < 3; ++r) {
    const int wrow = wbase + r * (3 * KPT * 1024);
#pragma unroll
    for (int sc = 0; sc < ROW_SLICES; ++sc) {
      const int cur = sc & 1, nxt = cur ^ 1;
      const bool last = sc + 1 == ROW_SLICES;
      const int off = last ? 0 : ((sc + 1) / KSW) * GP + 32 * ((sc + 1) % KSW);
      if (last) {
#pragma unroll
        for (int j = 0; j < MB; ++j) ar[j] += row_step;
      }
#pragma unroll
      for (int j = 0; j < MB; ++j) {
        acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(bq[sc % RING], xf[cur][j], acc[j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        xf[nxt][j] = *(lds_v4i *)(ar[j] + off);
        __builtin_amdgcn_sched_barrier(0);
      }
      const int ahead = sc + RING;
      if (ahead < ROW_SLICES)
        bq[sc % RING] = __builtin_amdgcn_raw_buffer_load_b128(wres, lane16, wrow + slice_at(ahead), 0);
      else if (r < 2)
        bq[sc % RING] = __builtin_amdgcn_raw_buffer_load_b128(wres, lane16, wrow + 3 * KPT * 1024 + slice_at(ahead - ROW_SLICES), 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  const ScaledClip c1 = scaled_clip(p.lo, p.hi, p.shift);
  const int sh = p.shift;
  auto finish = [&](int (&v)[16], const v4i &rv) {
    if (p.res) {
#pragma unroll
      for (int i = 0; i < 16; ++i) v[i] += align_res(byte_of((uint32_t)rv[i >> 2], i & 3, p.res_signed != 0), p.res_d);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = clamp_med3(v[i], c1.lo, c1.hi);
    return shift_pack16(v, sh);
  };
  if constexpr (WK == 1) {
    // every wave has its sums complete: a lane's 16 channels of a pixel are a 16-byte piece of an output row
    const int n = n0 + 32 * wn + 16 * half;
    v4i a0[4], rv[MB];
#pragma unroll
    for (int g = 0; g < 4; ++g) a0[g] = *reinterpret_cast<const v4i *>(p.acc0 + n + 4 * g);
#pragma unroll
    for (int j = 0; j < MB; ++j) {
      rv[j] = v4i{0, 0, 0, 0};
      if (p.res && 32 * j + l32 < npx) rv[j] = *reinterpret_cast<const v4i *>(p.res + (px0 + 32 * j + l32) * C + n);
    }
#pragma unroll
    for (int j = 0; j < MB; ++j) {
      settle_matrix_result(acc[j]);
      int v[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) v[i] = acc[j][i] + a0[i >> 2][i & 3];
      const v4i out = finish(v, rv[j]);
      if (32 * j + l32 < npx) *reinterpret_cast<v4i *>(p.y + (px0 + 32 * j + l32) * C + n) = out;
    }
  } else {
    // the waves' sums meet; thread -> piece of 16 channels of the pixels tid / (2 WN) + k * IPP
    constexpr int IPP = NT / (2 * WN), ITEMS = (MB * 32 + IPP - 1) / IPP;
    const int piece = tid % (2 * WN), pixel0 = tid / (2 * WN);
    const int n = n0 + piece * 16;
    v4i rv[ITEMS], a0[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) a0[g] = *reinterpret_cast<const v4i *>(p.acc0 + n + 4 * g);
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
      rv[k] = v4i{0, 0, 0, 0};
      if (p.res && pixel0 + k * IPP < npx) rv[k] = *reinterpret_cast<const v4i *>(p.res + (px0 + pixel0 + k * IPP) * C + n);
    }
    __syncthreads();                                 // the patch is no longer read
    uint8_t *part = lds + wave * (MB * 32 * PART_PITCH) + l32 * PART_PITCH + half * 64;
#pragma unroll
    for (int j = 0; j < MB; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<v4i *>(part + j * (32 * PART_PITCH) + g * 16) =
            v4i{acc[j][4 * g], acc[j][4 * g + 1], acc[j][4 * g + 2], acc[j][4 * g + 3]};
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
      const int m = pixel0 + k * IPP;
      if (m >= npx) continue;
      const uint8_t *from = lds + (piece >> 1) * (WK * MB * 32 * PART_PITCH) + m * PART_PITCH + (piece & 1) * 64;
      int v[16];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        v4i a = a0[g];
#pragma unroll
        for (int w = 0; w < WK; ++w) a += *reinterpret_cast<const v4i *>(from + w * (MB * 32 * PART_PITCH) + g * 16);
        v[4 * g] = a.x; v[4 * g + 1] = a.y; v[4 * g + 2] = a.z; v[4 * g + 3] = a.w;
      }
      *reinterpret_cast<v4i *>(p.y + (px0 + m) * C + n) = finish(v, rv[k]);
    }
  }
}

template <int C, int WK> int launch_c(const ConvImgkParams &p, hipStream_t stream) {
  const Units u = cut<C>(p.B, p.H, p.W, WK);
  if (u.images < 1) return (int)hipErrorInvalidValue;
  const long long grid = u.units * (C / (32 * (4 / WK)));
  if (grid > 0x7fffffffLL) return (int)hipErrorInvalidValue;
  // up to one workgroup per CU: ask for more than half of the LDS, or two of them may share a CU while
  // another stays idle (256 workgroups for 128 channels on 64 images: 13.3 us, with this 10.6 us)
  const int lds = grid <= 256 && u.lds < 84 * 1024 ? 84 * 1024 : u.lds;
  const void *fn = reinterpret_cast<const void *>(conv_imgk_kernel<C, WK>);
  static std::atomic<unsigned long long> done_mask{0};         // devices whose LDS limit has been raised
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return (int)hipErrorInvalidDevice;
  if (dev < 0 || dev > 63 || !((done_mask.load(std::memory_order_relaxed) >> dev) & 1ull)) {
    const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return (int)e;
    if (dev >= 0 && dev <= 63) done_mask.fetch_or(1ull << dev, std::memory_order_relaxed);
  }
  hipLaunchKernelGGL((conv_imgk_kernel<C, WK>), dim3((unsigned)grid), dim3(NT), lds, stream, p, u, FastDiv((uint32_t)p.W),
                     FastDiv((uint32_t)(u.rows * p.W)), FastDiv((uint32_t)u.prows), FastDiv((uint32_t)u.units));
  return (int)hipGetLastError();
}

Units cut_any(int C, int B, int H, int W, int WK) { return C == 128 ? cut<128>(B, H, W, WK) : C == 256 ? cut<256>(B, H, W, WK) : cut<512>(B, H, W, WK); }

}  // namespace

bool conv_imgk_applicable(int Cin, int Cout, int R, int S, int sh, int sw, int ph, int pw, int H, int W, int shift,
                          const void *x, const void *y, const void *res) {
  if (Cin != Cout || (Cin != 128 && Cin != 256 && Cin != 512) || R != 3 || S != 3 || sh != 1 || sw != 1 || ph != 1 || pw != 1) return false;
  if (shift < 0 || H < 1 || W < 1 || (long long)H * W * Cin * 8 > 0x7fffffffLL) return false;
  for (int wk = 1; wk <= 4; wk *= 2)
    if (cut_any(Cin, 1, H, W, wk).images < 1) return false;
  return ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(y) | reinterpret_cast<uintptr_t>(res)) & 15) == 0;
}

long long conv_imgk_workgroups(int C, int B, int H, int W, int wk) { return cut_any(C, B, H, W, wk).units * (C / (32 * (4 / wk))); }

int launch_conv_imgk(const ConvImgkParams &p, hipStream_t stream) {
  if (p.B <= 0) return 0;
  if (!conv_imgk_applicable(p.C, p.C, 3, 3, 1, 1, 1, 1, p.H, p.W, p.shift, p.x, p.y, p.res) || p.lo > p.hi ||
      ((reinterpret_cast<uintptr_t>(p.wf) | reinterpret_cast<uintptr_t>(p.acc0)) & 15))
    return (int)hipErrorInvalidValue;
  switch (p.C * 8 + p.wk) {
    case 128 * 8 + 1: return launch_c<128, 1>(p, stream);
    case 128 * 8 + 2: return launch_c<128, 2>(p, stream);
    case 256 * 8 + 1: return launch_c<256, 1>(p, stream);
    case 256 * 8 + 2: return launch_c<256, 2>(p, stream);
    case 256 * 8 + 4: return launch_c<256, 4>(p, stream);
    case 512 * 8 + 1: return launch_c<512, 1>(p, stream);
    case 512 * 8 + 2: return launch_c<512, 2>(p, stream);
    case 512 * 8 + 4: return launch_c<512, 4>(p, stream);
    default: return (int)hipErrorInvalidValue;
  }
}

}  // namespace f8
