// Image-stationary 3x3 convolution, stride 2, pad 1, with K shared among the waves of a workgroup, and the 1x1 stride-2 layer
// that reads the same input in the same launch: the first 3x3 layer of a ResNet stage and its block's shortcut projection, with
// the shift / clip epilogue of F8Net Eq. 2 / Eq. 9.
//
// The input pixels under a workgroup's output lie in LDS once, with a border of zeros, and every tap's fragment is read
// from that patch at a constant offset, windows two pixels apart; weights stream from L2 into registers in fragment order, no barrier
// in the loop (conv_imgk.hip has the reasons).  The 1x1 layer's operand is the middle tap's, which is on chip already: it costs
// C / 32 slices of K of 9 C / 32 more, one more requantisation and no launch.  Its blocks of pixels are dealt to the waves that share
// the 3x3 layer's K, each with the whole of the 1x1 layer's, so that only one of the two needs its sums exchanged.
//
// Bound by the chain of a workgroup (one per CU up to medium batch): operands in, loop, sums, stores.  Eight waves, two to a
// SIMD: the second has the same channels and share of K (its weights are in L1) and the other half of the pixels.  Microseconds
// of the launch at 64 images (two launches of conv_fast / four waves / eight): 64 -> 128 channels from 56 x 56 14.9 / 11.1 / 9.9, 128 -> 256
// from 28 x 28 13.8 / 11.9 / 10.0, 256 -> 512 from 14 x 14 17.3 / 11.0 / 9.6.
#include "conv_s2.h"

#include <atomic>
#include <type_traits>

namespace f8 {
namespace {

typedef int v16i __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) const v4i lds_v4i;
typedef __attribute__((address_space(3))) const uint8_t lds_u8;

constexpr int NW = 8, NT = 64 * NW;                  // waves w and w + 4 share a SIMD, channels and K, and have the pixels of half the blocks each
constexpr int NG = 4;                                // (groups of channels) x (shares of K)
constexpr int PART_PITCH = 32 * 4 + 16;              // a pixel's 32 partial sums
constexpr int LDS_MOST = 160 * 1024;

// MB 32-pixel blocks; a wave's part of the patch is RPW rows of up to NI KiB.
template <int C> struct Shape;
template <> struct Shape<64> { static constexpr int MB = 7, RPW = 4, NI = 4; };
template <> struct Shape<128> { static constexpr int MB = 7, RPW = 4, NI = 4; };
template <> struct Shape<256> { static constexpr int MB = 4, RPW = 4, NI = 4; };

// How the batch is cut into units of one workgroup: whole images, or bands of output rows of one image.
struct Units {
  int images;             // images per unit
  int rows;               // output rows of an image per unit (P for whole images)
  int bands;              // units per image (1 for whole images)
  int P, Q;
  int prows, pcols;       // patch rows per image and patch columns
  int all_rows;           // patch rows
  int group;              // bytes of one K group's part of the patch
  int lds;
  long long units;
  int by_unit;            // neighbouring workgroups share a unit (else a slice of channels)
};

template <int C> Units cut(int B, int H, int W, int WK) {
  using S = Shape<C>;
  constexpr int cap = S::MB * 32, max_rows = NW * S::RPW;
  const int gpitch = C / WK + 16, part = WK == 1 ? 0 : NG * S::MB * 32 * PART_PITCH;
  Units u{};
  u.P = (H - 1) / 2 + 1; u.Q = (W - 1) / 2 + 1;
  u.pcols = W + 2;
  if (H < 1 || W < 1 || u.Q > cap || u.pcols * C > S::NI * 1024) return u;
  auto fits = [&](int images, int rows) {
    u.prows = 2 * rows + 1;
    u.all_rows = images * u.prows;
    // (behind the patch: what the fragment reads issued after the last slice touch)
    u.group = ((u.all_rows + 1) * u.pcols + 2) * gpitch;
    u.lds = WK * u.group > part ? WK * u.group : part;
    return u.all_rows <= max_rows && images * rows * u.Q <= cap && u.lds <= LDS_MOST;
  };
  u.bands = 1;
  u.images = 0;
  if ((long long)u.P * u.Q <= cap)
    for (int n = cap / (u.P * u.Q); n >= 1 && u.images == 0; --n)
      if (fits(n, u.P)) { u.images = n; u.rows = u.P; }
  for (int bands = 2; bands <= u.P && u.images == 0; ++bands) {
    const int rows = (u.P + bands - 1) / bands;          // bands of equal height
    if (fits(1, rows)) { u.images = 1; u.rows = rows; u.bands = (u.P + rows - 1) / rows; }
  }
  u.units = u.images == 0 ? 0 : u.bands > 1 ? (long long)B * u.bands : (B + u.images - 1) / u.images;
  return u;
}

__device__ __forceinline__ v4i requant16(const v16i &a, const ScaledClip &c, int shift) {
  int v[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = clamp_med3(a[i], c.lo, c.hi);
  return shift_pack16(v, shift);
}

template <int C, int WK>
__global__ __launch_bounds__(NT, 1) void conv_s2_kernel(const ConvS2Params p, const Units u, const FastDiv fd_q, const FastDiv fd_px,
                                                        const FastDiv fd_prows, const FastDiv fd_fast) {
  using S = Shape<C>;
  constexpr int MB = S::MB, MH = (MB + 1) / 2, WN = NG / WK;
  constexpr int KPT = C / 32;                        // K slices per tap
  constexpr int KSW = KPT / WK;                      // of which a wave takes this many
  constexpr int KS = 9 * KPT;
  constexpr int CG = C / WK, GP = CG + 16;           // bytes of a patch pixel in one K group
  constexpr int PIECES = C / 16;                     // 16-byte pieces per pixel
  constexpr int ROW_SLICES = 3 * KSW;                // K slices per window row
  constexpr int RING = ROW_SLICES % 8 == 0 ? 8 : 6;  // slices of weights in flight
  constexpr int PB = (MH + WK - 1) / WK;             // blocks of the 1x1 layer per wave
  static_assert(ROW_SLICES % RING == 0 && ROW_SLICES % 2 == 0, "slots and fragment sets repeat from row to row");
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  const int kg = wave % WK, wn = wave % NG / WK, b0 = wave < NG ? 0 : MH;      // (b0: this wave's first block)
  const bool proj = p.acc0p != nullptr;
  const uint32_t bid = xcd_remap(blockIdx.x, gridDim.x);
  const int slow = (int)fd_fast.div(bid), fast = (int)bid - slow * (int)fd_fast.d;
  const int slice = u.by_unit ? fast : slow, unit = u.by_unit ? slow : fast;
  const int n0 = slice * (32 * WN);
  int img0, y0, nimg, rows;
  if (u.bands > 1) {
    img0 = unit / u.bands;
    y0 = (unit - img0 * u.bands) * u.rows;
    nimg = 1; rows = min(u.rows, u.P - y0);
  } else {
    img0 = unit * u.images;
    y0 = 0;
    nimg = min(u.images, p.B - img0); rows = u.P;
  }
  const int npx = nimg * rows * u.Q;                 // output pixels of this unit, consecutive in memory
  const size_t px0 = ((size_t)img0 * u.P + y0) * u.Q;

  // ---- this wave's weights: channel block n0 / 32 + wn, K slices kg * KSW .. + KSW of every tap, requested RING slices ahead
  const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<int8_t *>(p.w) + (size_t)(n0 / 32 + wn) * (KS * 1024), 0, KS * 1024, 0x00027000);
  const int lane16 = lane * 16, wbase = kg * (KSW * 1024);
  auto slice_at = [](int sc) { return ((sc / KSW) * KPT + sc % KSW) * 1024; };
  const int n_lane = n0 + 32 * wn + 16 * half;       // this lane's 16 channels (registers 0..15 of a block)

  // ---- the input pixels and a border of zeros into LDS, xor 0x80 when unsigned.  A wave takes the patch rows
  // wave, wave + NW, ...; a row's pixels are consecutive in memory, so a lane's 16-byte pieces of a row lie at
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
    const int row = wave + NW * k;                       // uniform
    const int img = (int)fd_prows.div((uint32_t)row), y = 2 * y0 + row - img * u.prows - 1;
    const bool in = img < nimg && (unsigned)y < (unsigned)p.H;
    if (row >= u.all_rows) continue;
    const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(xbase, 0, in ? nimg * (int)image_bytes : 0, 0x00027000);
    const int at = in ? (img * p.H + y) * p.W * C : 0;
#pragma unroll
    for (int i = 0; i < S::NI; ++i) px[k][i] = __builtin_amdgcn_raw_buffer_load_b128(xres, x_at[i], at, 0);
  }
  v4i wp[KPT], bq[RING], a0[4], a0p[4];
  if (proj) {
    const int8_t *from = p.wp + (size_t)(n0 / 32 + wn) * (KPT * 1024) + lane16;
#pragma unroll
    for (int ks = 0; ks < KPT; ++ks) wp[ks] = *reinterpret_cast<const v4i *>(from + ks * 1024);
#pragma unroll
    for (int g = 0; g < 4; ++g) a0p[g] = *reinterpret_cast<const v4i *>(p.acc0p + n_lane + 4 * g);
  }
#pragma unroll
  for (int g = 0; g < 4; ++g) a0[g] = kg == 0 ? *reinterpret_cast<const v4i *>(p.acc0 + n_lane + 4 * g) : v4i{0, 0, 0, 0};
#pragma unroll
  for (int sc = 0; sc < RING; ++sc) bq[sc] = __builtin_amdgcn_raw_buffer_load_b128(wres, lane16, wbase + slice_at(sc), 0);
  __builtin_amdgcn_sched_barrier(0);

  // (while they are on their way)
  // Fragment row 32 j + l32 is output pixel m of the unit; its window starts at patch pixel (image, 2 y, 2 x).
  // Rows past the last pixel read the patch's first window; their sums are dropped.
  int at_px[MH];
#pragma unroll
  for (int j = 0; j < MH; ++j) {
    const int m = 32 * (b0 + j) + l32;
    at_px[j] = 0;
    if (m < npx) {
      const int img = (int)fd_px.div((uint32_t)m), rem = m - img * (int)fd_px.d;
      const int y = (int)fd_q.div((uint32_t)rem), x = rem - y * u.Q;
      at_px[j] = (img * u.prows + 2 * y) * u.pcols + 2 * x;
    }
  }
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
    const int row = wave + NW * k;
    if (row < u.all_rows) {
#pragma unroll
      for (int i = 0; i < S::NI; ++i)
        if (to[i] >= 0)
          *reinterpret_cast<v4i *>(lds + row * u.pcols * GP + to[i]) = v4i{px[k][i].x ^ zx, px[k][i].y ^ zx, px[k][i].z ^ zx, px[k][i].w ^ zx};
    }
  }
  __syncthreads();                                   // the patch is complete

  const int out_bytes = npx * p.N;
  // (pixels past the unit: an offset the descriptors reject; stores are dropped)
  auto out_at = [&](int m, int n) { return m < npx ? (uint32_t)(m * p.N + n) : 0x80000000u; };
  // ---- the 1x1 layer: blocks kg, kg + WK, ... of pixels, all of K
  if (proj) {
    const ScaledClip cp = scaled_clip(p.lop, p.hip, p.shiftp);
    const __amdgpu_buffer_rsrc_t pres = __builtin_amdgcn_make_buffer_rsrc(p.yp + px0 * p.N, 0, out_bytes, 0x00027000);
    v16i acc[PB];
    lds_u8 *xr[PB];
#pragma unroll
    for (int i = 0; i < PB; ++i) {
      // (uniform selects: the block's number depends on the wave)
      int at = at_px[0];
#pragma unroll
      for (int j = 1; j < MH; ++j) at = kg + WK * i == j ? at_px[j] : at;
      xr[i] = (lds_u8 *)lds + (at + u.pcols + 1) * GP + 16 * half;
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][e] = a0p[e >> 2][e & 3];
    }
#pragma unroll
    for (int ks = 0; ks < KPT; ++ks)
#pragma unroll
      for (int i = 0; i < PB; ++i)
        acc[i] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wp[ks], *(lds_v4i *)(xr[i] + (ks / KSW) * u.group + 32 * (ks % KSW)), acc[i], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < PB; ++i) {
      settle_matrix_result(acc[i]);
      const int j = kg + WK * i;
      __builtin_amdgcn_raw_buffer_store_b128(requant16(acc[i], cp, p.shiftp), pres, out_at(j < MH ? 32 * (b0 + j) + l32 : npx, n_lane), 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  }

  const ScaledClip c1 = scaled_clip(p.lo, p.hi, p.shift);
  const __amdgpu_buffer_rsrc_t yres = __builtin_amdgcn_make_buffer_rsrc(p.y + px0 * p.N, 0, out_bytes, 0x00027000);
  // ---- K loop over the wave's MBW blocks: a pass is a row of the window, 3 taps x KSW slices; activation fragments one slice ahead,
  // one request at a time behind the matrix instructions
  v16i acc[MH];
#pragma unroll
  for (int j = 0; j < MH; ++j)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[j][i] = a0[i >> 2][i & 3];
  auto contract = [&](auto blocks) {
  constexpr int MBW = decltype(blocks)::value;
  lds_u8 *ar[MBW];
  v4i xf[2][MBW];
#pragma unroll
  for (int j = 0; j < MBW; ++j) {
    ar[j] = (lds_u8 *)lds + kg * u.group + at_px[j] * GP + 16 * half;
    xf[0][j] = *(lds_v4i *)(ar[j]);
  }
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
        for (int j = 0; j < MBW; ++j) ar[j] += row_step;
      }
#pragma unroll
      for (int j = 0; j < MBW; ++j) {
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
  };
  if (b0 == 0 || MB % 2 == 0) contract(std::integral_constant<int, MH>{});
  else contract(std::integral_constant<int, MB - MH>{});      // (the block past the last: start values, which go nowhere)

  if constexpr (WK == 1) {
    // every wave has its sums complete: a lane's 16 channels of a pixel are a 16-byte piece of an output row
#pragma unroll
    for (int j = 0; j < MH; ++j) {
      if (MH * 2 > MB && b0 + j >= MB) continue;
      settle_matrix_result(acc[j]);
      __builtin_amdgcn_raw_buffer_store_b128(requant16(acc[j], c1, p.shift), yres, out_at(32 * (b0 + j) + l32, n_lane), 0, 0);
    }
  } else {
    __syncthreads();                                 // the patch is no longer read (behind the lambda: both halves of the waves at one barrier)
    uint8_t *part = lds + ((wave % NG) * MB + b0) * (32 * PART_PITCH) + l32 * PART_PITCH + half * 64;
#pragma unroll
    for (int j = 0; j < MH; ++j) {
      if (MH * 2 > MB && b0 + j >= MB) continue;
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<v4i *>(part + j * (32 * PART_PITCH) + g * 16) =
            v4i{acc[j][4 * g], acc[j][4 * g + 1], acc[j][4 * g + 2], acc[j][4 * g + 3]};
    }
    // the waves' sums meet; then piece tid % (2 WN) of the pixels tid / (2 WN) + k * IPP
    constexpr int IPP = NT / (2 * WN), ITEMS = (MB * 32 + IPP - 1) / IPP;
    const int piece = tid % (2 * WN), pixel0 = tid / (2 * WN);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
      const int m = pixel0 + k * IPP;                // (past the last block: reads sums of other pixels, drops the store)
      const uint8_t *from = lds + (piece >> 1) * (WK * MB * 32 * PART_PITCH) + (m < MB * 32 ? m : 0) * PART_PITCH + (piece & 1) * 64;
      v16i v;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        v4i a = *reinterpret_cast<const v4i *>(from + g * 16);
#pragma unroll
        for (int w = 1; w < WK; ++w) a += *reinterpret_cast<const v4i *>(from + w * (MB * 32 * PART_PITCH) + g * 16);
        v[4 * g] = a.x; v[4 * g + 1] = a.y; v[4 * g + 2] = a.z; v[4 * g + 3] = a.w;
      }
      __builtin_amdgcn_raw_buffer_store_b128(requant16(v, c1, p.shift), yres, out_at(m, n0 + piece * 16), 0, 0);
    }
  }
}

// Piece i (16 bytes) of the weights: block of 32 channels by block, the taps C / 32 slices tap by tap; a slice is 64 pieces, piece `lane`
// the bytes that lane feeds to the matrix instruction.
__global__ __launch_bounds__(256) void conv_s2_weights_kernel(const int8_t *__restrict__ w, int8_t *__restrict__ wf, int taps, int C, int pieces) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= pieces) return;
  const int kpt = C / 32, ks = taps * kpt;
  const int lane = i & 63, t = (i >> 6) % ks, nb = (i >> 6) / ks;
  const int n = 32 * nb + weight_row(lane & 31), half = lane >> 5;
  const int8_t *src = w + ((size_t)n * taps + t / kpt) * C + 32 * (t % kpt);
  *reinterpret_cast<v4i *>(wf + (size_t)i * 16) = *reinterpret_cast<const v4i *>(src + 16 * half);
}

Units cut_any(int C, int B, int H, int W, int WK) {
  return C == 64 ? cut<64>(B, H, W, WK) : C == 128 ? cut<128>(B, H, W, WK) : cut<256>(B, H, W, WK);
}

template <int C, int WK> int launch_c(const ConvS2Params &p, hipStream_t stream) {
  Units u = cut<C>(p.B, p.H, p.W, WK);
  if (u.images < 1) return (int)hipErrorInvalidValue;
  const int slices = p.N / (32 * (NG / WK));
  const long long grid = u.units * slices;
  if (grid > 0x7fffffffLL) return (int)hipErrorInvalidValue;
  // unit by unit where that fetches less from other XCDs (see conv_imgk.hip)
  const long long share = u.units * slices / 8 < u.units ? u.units * slices / 8 : u.units;
  u.by_unit = share * u.images * u.prows * p.W * C > (p.acc0p ? 10ll : 9ll) * C * p.N;
  // one workgroup per CU while there are no more (see conv_imgk.hip)
  const int lds = grid <= 256 && u.lds < 84 * 1024 ? 84 * 1024 : u.lds;
  const void *fn = reinterpret_cast<const void *>(conv_s2_kernel<C, WK>);
  static std::atomic<unsigned long long> done_mask{0};         // devices whose LDS limit has been raised
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return (int)hipErrorInvalidDevice;
  if (dev < 0 || dev > 63 || !((done_mask.load(std::memory_order_relaxed) >> dev) & 1ull)) {
    const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, LDS_MOST);
    if (e != hipSuccess) return (int)e;
    if (dev >= 0 && dev <= 63) done_mask.fetch_or(1ull << dev, std::memory_order_relaxed);
  }
  hipLaunchKernelGGL((conv_s2_kernel<C, WK>), dim3((unsigned)grid), dim3(NT), lds, stream, p, u, FastDiv((uint32_t)u.Q),
                     FastDiv((uint32_t)(u.rows * u.Q)), FastDiv((uint32_t)u.prows), FastDiv((uint32_t)(u.by_unit ? slices : u.units)));
  return (int)hipGetLastError();
}

}  // namespace

bool conv_s2_fills(int C, int H, int W) {
  const Units u = cut_any(C, 1, H, W, 1);
  return u.images * u.rows * u.Q * 3 >= (C == 256 ? 4 : 7) * 32 * 2;
}

int conv_s2_most_waves(int C) { return C == 64 ? 1 : C == 128 ? 2 : 4; }

bool conv_s2_applicable(int Cin, int Cout, int R, int S, int sh, int sw, int ph, int pw, int H, int W, int shift, const void *x, const void *y) {
  if ((Cin != 64 && Cin != 128 && Cin != 256) || Cout < 128 || (Cout & 127) || R != 3 || S != 3 || sh != 2 || sw != 2 || ph != 1 || pw != 1) return false;
  if (shift < 0 || H < 1 || W < 1 || (long long)H * W * Cin * 8 > 0x7fffffffLL || (long long)H * W * Cout * 2 > 0x7fffffffLL) return false;
  for (int wk = 1; wk <= conv_s2_most_waves(Cin); wk *= 2)
    if (cut_any(Cin, 1, H, W, wk).images < 1) return false;
  return ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(y)) & 15) == 0;
}

long long conv_s2_workgroups(int C, int N, int B, int H, int W, int wk) { return cut_any(C, B, H, W, wk).units * (N / (32 * (NG / wk))); }

int launch_conv_s2_weights(const int8_t *w, int8_t *wf, int taps, int C, int N, hipStream_t stream) {
  if (!w || !wf || (C & 31) || (N & 31) || ((reinterpret_cast<uintptr_t>(w) | reinterpret_cast<uintptr_t>(wf)) & 15)) return (int)hipErrorInvalidValue;
  const int pieces = (int)((size_t)N * taps * C / 16);
  hipLaunchKernelGGL(conv_s2_weights_kernel, dim3((pieces + 255) / 256), dim3(256), 0, stream, w, wf, taps, C, pieces);
  return (int)hipGetLastError();
}

int launch_conv_s2(const ConvS2Params &p, hipStream_t stream) {
  if (p.B <= 0) return 0;
  if (!conv_s2_applicable(p.C, p.N, 3, 3, 2, 2, 1, 1, p.H, p.W, p.shift, p.x, p.y) || p.lo > p.hi ||
      ((reinterpret_cast<uintptr_t>(p.w) | reinterpret_cast<uintptr_t>(p.acc0) | reinterpret_cast<uintptr_t>(p.acc0p) | reinterpret_cast<uintptr_t>(p.wp) | reinterpret_cast<uintptr_t>(p.yp)) & 15) ||
      (p.acc0p && (!p.yp || !p.wp || p.shiftp < 0 || p.lop > p.hip)))
    return (int)hipErrorInvalidValue;
  switch (p.C * 8 + p.wk) {
    case 64 * 8 + 1: return launch_c<64, 1>(p, stream);
    case 128 * 8 + 1: return launch_c<128, 1>(p, stream);
    case 128 * 8 + 2: return launch_c<128, 2>(p, stream);
    case 256 * 8 + 1: return launch_c<256, 1>(p, stream);
    case 256 * 8 + 2: return launch_c<256, 2>(p, stream);
    case 256 * 8 + 4: return launch_c<256, 4>(p, stream);
    default: return (int)hipErrorInvalidValue;
  }
}

}  // namespace f8
