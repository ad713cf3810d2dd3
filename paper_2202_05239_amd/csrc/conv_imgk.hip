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
//   C = 64: a band of up to 224 pixels, two waves (MG = 2: four) of 32 channels, every weight of a wave in its registers;
//   C = 256: a whole image of up to 224 pixels (7 blocks of 32); C = 512: two 7 x 7 images (4 blocks);
//   C = 128: a band of up to 224 pixels.
// With one wave per SIMD 12.0 us for 256 channels on 64 images (two waves share K), with two 11.1; 16.4 us on 128 images
// (22.4 before); with one wave per SIMD 9.3 k cycles of a workgroup's 19.7 k are the loop (8.1 k of matrix instructions),
// 6 k the patch (82 - 92 KiB at the 60 bytes per clock a CU gets from L2, then memory latency), 4 k the sums in
// LDS and the stores.  With 64 channels per wave and four waves sharing K the loop reads half as much from LDS
// but the sums take twice as long: 12.8 us.  64 channels on 64 images of 56 x 56 with a residual: 13.5 us (18.9 in
// conv_fast).
// MG = 2: twice the waves, w and w + NW on one SIMD with the same channels and share of K and half of the pixels' blocks each.
// NAT (64 channels, single-layer calls): the weights are read as they are and
// summed for the start values on the way, so that the call is one launch: 8.6 us a call on 32 images of
// 56 x 56 (10.7 with half the waves, 11.9 for fold and conv_ws).
#include "conv_imgk.h"

#include <atomic>
#include <type_traits>

namespace f8 {
namespace {

typedef int v16i __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) const v4i lds_v4i;
typedef __attribute__((address_space(3))) const uint8_t lds_u8;

constexpr int PART_PITCH = 32 * 4 + 16;              // a pixel's 32 partial sums

// NW waves, MB 32-pixel blocks; a wave's part of the patch is RPW rows of up to NI KiB.
template <int C> struct Shape;
template <> struct Shape<64> { static constexpr int NW = 2, MB = 7, RPW = 5, NI = 4; };
template <> struct Shape<128> { static constexpr int NW = 4, MB = 7, RPW = 3, NI = 4; };
template <> struct Shape<256> { static constexpr int NW = 4, MB = 7, RPW = 5, NI = 4; };
template <> struct Shape<512> { static constexpr int NW = 4, MB = 4, RPW = 5, NI = 5; };

// NAT: the weights of 64 channels as rows of 9 taps, 16 bytes more than their length apart: 8 rows' pieces share no bank
constexpr int NAT_PITCH = 9 * 64 + 16, NAT_BYTES = 64 * NAT_PITCH;

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
  int by_unit;            // neighbouring workgroups share a unit (else a slice of channels)
};

template <int C> Units cut(int B, int H, int W, int WK) {
  using S = Shape<C>;
  constexpr int cap = S::MB * 32, max_rows = S::NW * S::RPW;
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

// Channel fed as row r of a 32-channel block (the fragment order of launch_conv_img_weights has it built in).
__device__ __forceinline__ int frag_channel(int r) { return 16 * ((r >> 2) & 1) + 4 * (r >> 3) + (r & 3); }

template <int C, int WK, bool NAT, int MG>
__global__ __launch_bounds__(64 * Shape<C>::NW * MG, MG == 2 ? (C == 64 ? 2 : 1) : WK == 1 ? 2 : 1) void conv_imgk_kernel(const ConvImgkParams p, const Units u, const FastDiv fd_w, const FastDiv fd_px,
                                                          const FastDiv fd_prows, const FastDiv fd_fast) {
  using S = Shape<C>;
  constexpr int NW = S::NW, NWG = NW * MG, NT = 64 * NWG, MB = S::MB, WN = NW / WK;
  constexpr int MH = (MB + MG - 1) / MG;             // blocks per wave
  constexpr int RPW = (NW * S::RPW + NWG - 1) / NWG;
  constexpr int KPT = C / 32;                        // K slices per tap
  constexpr int KSW = KPT / WK;                      // of which a wave takes this many
  constexpr int KS = 9 * KPT;
  constexpr int CG = C / WK, GP = CG + 16;           // bytes of a patch pixel in one K group
  constexpr int PIECES = C / 16;                     // 16-byte pieces per pixel
  constexpr int ROW_SLICES = 3 * KSW;                // K slices per window row
  constexpr int RING = C == 64 ? KS : MB == 7 ? (ROW_SLICES % 8 == 0 ? 8 : 6) : 12;      // slices of weights in flight
  constexpr bool ALL = RING == KS;                   // every slice is requested before the loop
  static_assert((ALL || ROW_SLICES % RING == 0) && ROW_SLICES % 2 == 0, "slots and fragment sets repeat from row to row");
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  const int kg = wave % WK, wn = wave % NW / WK, b0 = wave < NW ? 0 : MH;      // (b0: this wave's first block)
  // neighbours on an XCD: the workgroups of one channel slice, which stream the same weights, or of one unit
  const uint32_t bid = xcd_remap(blockIdx.x, gridDim.x);
  const int slow = (int)fd_fast.div(bid), fast = (int)bid - slow * (int)fd_fast.d;
  const int slice = u.by_unit ? fast : slow, unit = u.by_unit ? slow : fast;
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
      const_cast<int8_t *>(p.w) + (size_t)(n0 / 32 + wn) * (KS * 1024), 0, NAT ? 0 : KS * 1024, 0x00027000);
  const int lane16 = lane * 16, wbase = kg * (KSW * 1024);
  auto slice_at = [](int sc) { return ((sc / KSW) * KPT + sc % KSW) * 1024; };
  // start values of this lane's 16 channels (registers 0..15 of a block): the wave that takes the first share of K
  // starts its accumulators there
  v4i a0[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int n = n0 + 32 * wn + 16 * half + 4 * g;
    if (!NAT) a0[g] = kg == 0 ? *reinterpret_cast<const v4i *>(p.acc0 + n) : v4i{0, 0, 0, 0};
    else a0[g] = p.acc0 ? v4i{p.acc0[n], p.acc0[n + 1], p.acc0[n + 2], p.acc0[n + 3]} : v4i{0, 0, 0, 0};
  }
  v4i bq[RING];
  constexpr bool STAGE = NAT && MG == 2;             // by way of LDS
  constexpr int NATP = STAGE ? C * 9 * C / 16 / NT : 1;
  v4i wraw[NATP];
  const int8_t *w_nat = p.w + (size_t)(n0 + 32 * wn + frag_channel(l32)) * (9 * C) + 16 * half;
  if (STAGE) {
    // as they lie in memory; they change places in LDS, behind the patch (32 bytes of each of 32 rows, as a wave needs them, the load
    // unit takes a row at a time: 16 bytes per clock)
#pragma unroll
    for (int i = 0; i < NATP; ++i) wraw[i] = *reinterpret_cast<const v4i *>(p.w + (size_t)(i * NT + tid) * 16);
  } else {
#pragma unroll
    for (int sc = 0; sc < RING; ++sc)
      bq[sc] = NAT ? *reinterpret_cast<const v4i *>(w_nat + 32 * sc) : __builtin_amdgcn_raw_buffer_load_b128(wres, lane16, wbase + slice_at(sc), 0);      // (ALL: slices of all rows; KSW == KPT then)
  }

  // ---- the input pixels and a border of zeros into LDS, xor 0x80 when unsigned.  A wave takes the patch rows
  // wave, wave + NWG, ...; a row's pixels are consecutive in memory, so a lane's 16-byte pieces of a row lie at
  // fixed offsets from its first pixel (the scalar part of the address) and at fixed places in a patch row.
  // Border columns: an offset the descriptor rejects, which reads as zero; border rows: an empty descriptor.
  const size_t image_bytes = (size_t)p.H * p.W * C;
  uint8_t *xbase = const_cast<uint8_t *>(p.x) + (size_t)img0 * image_bytes;
  uint32_t x_at[S::NI];
  v4i px[RPW][S::NI];
#pragma unroll
  for (int i = 0; i < S::NI; ++i) {
    const int col = (i * 64 + lane) / PIECES;
    x_at[i] = (unsigned)(col - 1) < (unsigned)p.W ? (uint32_t)((i * 64 + lane) * 16 - C) : 0x80000000u;
  }
#pragma unroll
  for (int k = 0; k < RPW; ++k) {
    const int row = wave + NWG * k;                      // uniform
    const int img = (int)fd_prows.div((uint32_t)row), y = y0 + row - img * u.prows - 1;
    const bool in = img < nimg && (unsigned)y < (unsigned)p.H;
    if (row >= u.all_rows) continue;
    const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(xbase, 0, in ? nimg * (int)image_bytes : 0, 0x00027000);
    const int at = in ? (img * p.H + y) * p.W * C : 0;
#pragma unroll
    for (int i = 0; i < S::NI; ++i) px[k][i] = __builtin_amdgcn_raw_buffer_load_b128(xres, x_at[i], at, 0);
  }
  // the residual pieces this thread will need at the end: WK == 1: its lane's 16 channels of every block; otherwise
  // piece tid % (2 WN) of the pixels tid / (2 WN) + k * IPP
  constexpr int IPP = NT / (2 * WN), ITEMS = WK == 1 ? MH : (MB * 32 + IPP - 1) / IPP;
  const int piece = tid % (2 * WN), pixel0 = WK == 1 ? 32 * b0 + l32 : tid / (2 * WN);
  const int n_out = WK == 1 ? n0 + 32 * wn + 16 * half : n0 + piece * 16;
  constexpr int ITEM_STEP = WK == 1 ? 32 : IPP;
  // (pixels past the unit: an offset the descriptors reject: loads return zeros, stores are dropped)
  const int out_bytes = npx * C;
  v4i rv[ITEMS];
  uint32_t out_at[ITEMS];
#pragma unroll
  for (int k = 0; k < ITEMS; ++k)
    out_at[k] = pixel0 + k * ITEM_STEP < npx ? (uint32_t)((pixel0 + k * ITEM_STEP) * C + n_out) : 0x80000000u;
  if (p.res) {
    const __amdgpu_buffer_rsrc_t rres = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(p.res) + px0 * C, 0, out_bytes, 0x00027000);
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) rv[k] = __builtin_amdgcn_raw_buffer_load_b128(rres, out_at[k], 0, 0);
  }
  __builtin_amdgcn_sched_barrier(0);

  // (while they are on their way)
  // Fragment row 32 j + l32 is output pixel m of the unit; its window starts at patch pixel (image, y, x).
  // Rows past the last pixel read the patch's first window; their sums are dropped.
  lds_u8 *ar[MH];
#pragma unroll
  for (int j = 0; j < MH; ++j) {
    const int m = 32 * (b0 + j) + l32;
    int at = 0;
    if (m < npx) {
      const int img = (int)fd_px.div((uint32_t)m), rem = m - img * (int)fd_px.d;
      const int y = (int)fd_w.div((uint32_t)rem), x = rem - y * p.W;
      at = (img * u.prows + y) * u.pcols + x;
    }
    ar[j] = (lds_u8 *)lds + kg * u.group + at * GP + 16 * half;
  }
  int to[S::NI];
#pragma unroll
  for (int i = 0; i < S::NI; ++i) {
    const int col = (i * 64 + lane) / PIECES, piece = lane % PIECES;
    // (pieces past the last column are fetched as zeros and not kept)
    to[i] = col < u.pcols ? (piece / (CG / 16)) * u.group + col * GP + (piece % (CG / 16)) * 16 : -1;
  }
  if (STAGE) {
#pragma unroll
    for (int i = 0; i < NATP; ++i) {
      const int at = i * NT + tid, row = at / (9 * PIECES);
      *reinterpret_cast<v4i *>(lds + u.lds - NAT_BYTES + row * NAT_PITCH + (at - row * (9 * PIECES)) * 16) = wraw[i];
    }
    __syncthreads();
    const uint8_t *w_row = lds + u.lds - NAT_BYTES + (32 * wn + frag_channel(l32)) * NAT_PITCH + 16 * half;
#pragma unroll
    for (int sc = 0; sc < RING; ++sc) bq[sc] = *reinterpret_cast<const v4i *>(w_row + 32 * sc);
  }
  if (NAT) {
    int wsum = 0;
    // the sum of this lane's weights: with the other half's, 128 times it belongs in the start value
#pragma unroll
    for (int sc = 0; sc < RING; ++sc)
#pragma unroll
      for (int d = 0; d < 4; ++d) wsum = __builtin_amdgcn_sdot4(bq[sc][d], 0x01010101, wsum, false);
    wsum += __shfl_xor(wsum, 32, 64);
    // lane r holds the sum of channel frag_channel(r): channels 16 half + 4 g .. + 3 are rows 8 g + 4 half ..
    const int rnd = p.shift > 0 ? 1 << (p.shift - 1) : 0;
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int i = 0; i < 4; ++i) a0[g][i] += rnd + (p.x_xor ? 128 * __shfl(wsum, 8 * g + 4 * half + i, 64) : 0);
  }
  static_assert(64 % PIECES == 0, "a lane keeps its piece of a pixel");
  __builtin_amdgcn_sched_barrier(0);
  const int zx = (int)p.x_xor;
#pragma unroll
  for (int k = 0; k < RPW; ++k) {
    const int row = wave + NWG * k;
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
  v16i acc[MH];
#pragma unroll
  for (int j = 0; j < MH; ++j)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[j][i] = a0[i >> 2][i & 3];
  auto contract = [&](auto blocks) {
  constexpr int MBW = decltype(blocks)::value;
  v4i xf[2][MBW];
#pragma unroll
  for (int j = 0; j < MBW; ++j) xf[0][j] = *(lds_v4i *)(ar[j]);
  const int row_step = u.pcols * GP;
#pragma unroll ALL ? 3 : 1
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
        acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(bq[ALL ? r * ROW_SLICES + sc : sc % RING], xf[cur][j], acc[j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        xf[nxt][j] = *(lds_v4i *)(ar[j] + off);
        __builtin_amdgcn_sched_barrier(0);
      }
      const int ahead = sc + RING;
      if (ALL) continue;
      if (ahead < ROW_SLICES)
        bq[sc % RING] = __builtin_amdgcn_raw_buffer_load_b128(wres, lane16, wrow + slice_at(ahead), 0);
      else if (r < 2)
        bq[sc % RING] = __builtin_amdgcn_raw_buffer_load_b128(wres, lane16, wrow + 3 * KPT * 1024 + slice_at(ahead - ROW_SLICES), 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  };
  if (MG == 1 || MB % 2 == 0 || b0 == 0) contract(std::integral_constant<int, MH>{});
  else contract(std::integral_constant<int, MB - MH>{});      // (the block past the last: start values, whose stores are dropped)

  const ScaledClip c1 = scaled_clip(p.lo, p.hi, p.shift);
  const int sh = p.shift, d = p.res_d;
  const __amdgpu_buffer_rsrc_t yres = __builtin_amdgcn_make_buffer_rsrc(p.y + px0 * C, 0, out_bytes, 0x00027000);
  // One instance for each residual kind (RK: 0 none, 1 unsigned, 2 signed) and direction (RLEFT: shifted left, else
  // rounded right); the choice is uniform.
  auto finish = [&](auto rk_tag, auto rleft_tag) {
    constexpr int RK = decltype(rk_tag)::value;
    constexpr bool RLEFT = decltype(rleft_tag)::value;
    const int rhalf = RLEFT ? 0 : 1 << (-d - 1);
    auto store = [&](int (&v)[16], int k) {
      if (RK != 0) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int b = RK == 2 ? (int)__builtin_amdgcn_sbfe(rv[k][i >> 2], 8 * (i & 3), 8)
                                : (int)__builtin_amdgcn_ubfe((uint32_t)rv[k][i >> 2], 8 * (i & 3), 8);
          v[i] += RLEFT ? (b << d) : ((b + rhalf) >> (-d));
        }
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) v[i] = clamp_med3(v[i], c1.lo, c1.hi);
      __builtin_amdgcn_raw_buffer_store_b128(shift_pack16(v, sh), yres, out_at[k], 0, 0);
    };
    if constexpr (WK == 1) {
      // every wave has its sums complete: a lane's 16 channels of a pixel are a 16-byte piece of an output row
#pragma unroll
      for (int j = 0; j < MH; ++j) {
        settle_matrix_result(acc[j]);
        int v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = acc[j][i];
        store(v, j);
      }
    } else {
#pragma unroll
      for (int k = 0; k < ITEMS; ++k) {
        const int m = pixel0 + k * IPP;              // (past the last block: reads sums of other pixels, drops the store)
        const uint8_t *from = lds + (piece >> 1) * (WK * MB * 32 * PART_PITCH) + (m < MB * 32 ? m : 0) * PART_PITCH + (piece & 1) * 64;
        int v[16];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          v4i a = *reinterpret_cast<const v4i *>(from + g * 16);
#pragma unroll
          for (int w = 1; w < WK; ++w) a += *reinterpret_cast<const v4i *>(from + w * (MB * 32 * PART_PITCH) + g * 16);
          v[4 * g] = a.x; v[4 * g + 1] = a.y; v[4 * g + 2] = a.z; v[4 * g + 3] = a.w;
        }
        store(v, k);
      }
    }
  };
  if constexpr (WK > 1) {
    // the waves' sums meet
    __syncthreads();                                 // the patch is no longer read
    uint8_t *part = lds + ((wave % NW) * MB + b0) * (32 * PART_PITCH) + l32 * PART_PITCH + half * 64;
#pragma unroll
    for (int j = 0; j < MH; ++j) {
      if (MH * MG > MB && b0 + j >= MB) continue;
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<v4i *>(part + j * (32 * PART_PITCH) + g * 16) =
            v4i{acc[j][4 * g], acc[j][4 * g + 1], acc[j][4 * g + 2], acc[j][4 * g + 3]};
    }
    __syncthreads();
  }
  using std::integral_constant;
  if (!p.res) finish(integral_constant<int, 0>{}, std::true_type{});
  else if (p.res_signed) { if (d >= 0) finish(integral_constant<int, 2>{}, std::true_type{}); else finish(integral_constant<int, 2>{}, std::false_type{}); }
  else { if (d >= 0) finish(integral_constant<int, 1>{}, std::true_type{}); else finish(integral_constant<int, 1>{}, std::false_type{}); }
}

template <int C, int WK, bool NAT, int MG> int launch_as(const ConvImgkParams &p, hipStream_t stream) {
  using S = Shape<C>;
  Units u = cut<C>(p.B, p.H, p.W, WK);
  if (u.images < 1) return (int)hipErrorInvalidValue;
  const int slices = C / (32 * (S::NW / WK));
  const long long grid = u.units * slices;
  if (grid > 0x7fffffffLL) return (int)hipErrorInvalidValue;
  // Unit by unit an XCD reads all weights, and of the images only the eighth of the batch that it computes and, the layers before being
  // ordered alike, mostly wrote itself: those lie in its L2.  Slice by slice it reads an eighth of the weights and images that
  // other XCDs wrote, from beyond its L2 at half the rate (64 KB per workgroup: 5.1 k cycles where this XCD wrote them, 10.3 k elsewhere).
  // Whichever fetches less from there; ResNet-18, us of a forward, slice by slice / unit by unit: 224 x 224, 24 images 174.7 / 169.2,
  // 32 187.6 / 178.1, 64 250.7 / 244.0, 128 386 / 380; 512 channels at 192 (2.4 MB of weights) the other way, 531 / 535, by this line 524.
  const long long share = u.units * slices / 8 < u.units ? u.units * slices / 8 : u.units;
  u.by_unit = share * u.images * u.rows * p.W * C > 9ll * C * C;
  if (NAT && MG == 2) u.lds += NAT_BYTES;
  // up to one workgroup per CU: ask for more than half of the LDS, or two of them may share a CU while
  // another stays idle (256 workgroups for 128 channels on 64 images: 13.3 us, with this 10.6 us)
  const int lds = grid <= 256 && u.lds < 84 * 1024 ? 84 * 1024 : u.lds;
  const void *fn = reinterpret_cast<const void *>(conv_imgk_kernel<C, WK, NAT, MG>);
  static std::atomic<unsigned long long> done_mask{0};         // devices whose LDS limit has been raised
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return (int)hipErrorInvalidDevice;
  if (dev < 0 || dev > 63 || !((done_mask.load(std::memory_order_relaxed) >> dev) & 1ull)) {
    const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return (int)e;
    if (dev >= 0 && dev <= 63) done_mask.fetch_or(1ull << dev, std::memory_order_relaxed);
  }
  hipLaunchKernelGGL((conv_imgk_kernel<C, WK, NAT, MG>), dim3((unsigned)grid), dim3(64 * S::NW * MG), lds, stream, p, u, FastDiv((uint32_t)p.W),
                     FastDiv((uint32_t)(u.rows * p.W)), FastDiv((uint32_t)u.prows), FastDiv((uint32_t)(u.by_unit ? slices : u.units)));
  return (int)hipGetLastError();
}

template <int C, int WK, bool NAT> int launch_c(const ConvImgkParams &p, hipStream_t stream) {
  // Twice the waves where a workgroup has a CU (64 channels: half a one) to itself; with more of them, workgroups of fewer waves side by
  // side cover one another's waits.  Microseconds of a layer, single / twice the waves, 3x3 layers of 64 channels on 56 x 56 at 16 images
  // 6.97 / 5.52, 32 9.73 / 7.55, 64 (896 workgroups) 13.42 / 13.34, with a residual (beyond 1024 workgroups they all have one) 50 x 50 at 128 (1664) 40.1 / 42.1, 35 x 35 at
  // 299 (1794) 43.5 / 45.6, 56 x 56 at 96 (1344) 37.7 / 38.5; 128 on 28 x 28 at 16 8.4 / 7.2, 64 11.5 / 10.8, 128 (512 workgroups)
  // 20.0 / 22.4; 256 on 14 x 14 at 32 8.8 / 7.9, 64 12.0 / 11.1, 128 17.6 / 17.5, 192 27.7 / 31.2; 512 on 7 x 7 at 32 9.5 / 9.0, 64 14.2 / 13.4, 256 39.7 / 40.6.
  const Units u = cut<C>(p.B, p.H, p.W, WK);
  // Weights as they are (a single call), 64 channels on 56 x 56, at 8 images 9.0 (conv_wavek) / 6.3, 16 7.9 / 6.7, 32 10.7 / 8.6, 64 14.5 / 16.0.
  return u.units * (C / (32 * (Shape<C>::NW / WK))) <= (NAT ? 512 : C == 64 ? 1024 : 256) ? launch_as<C, WK, NAT, 2>(p, stream) : launch_as<C, WK, NAT, 1>(p, stream);
}

Units cut_any(int C, int B, int H, int W, int WK) {
  return C == 64 ? cut<64>(B, H, W, WK) : C == 128 ? cut<128>(B, H, W, WK) : C == 256 ? cut<256>(B, H, W, WK) : cut<512>(B, H, W, WK);
}

}  // namespace

bool conv_imgk_fills(int C, int H, int W) {
  const Units u = cut_any(C, 1, H, W, 1);
  return u.images * u.rows * W * 3 >= (C == 512 ? 4 : 7) * 32 * 2;
}

int conv_imgk_most_waves(int C) { return C == 64 ? 1 : C == 128 ? 2 : 4; }

bool conv_imgk_applicable(int Cin, int Cout, int R, int S, int sh, int sw, int ph, int pw, int H, int W, int shift,
                          const void *x, const void *y, const void *res) {
  if (Cin != Cout || (Cin != 64 && Cin != 128 && Cin != 256 && Cin != 512) || R != 3 || S != 3 || sh != 1 || sw != 1 || ph != 1 || pw != 1) return false;
  if (shift < 0 || H < 1 || W < 1 || (long long)H * W * Cin * 8 > 0x7fffffffLL) return false;
  for (int wk = 1; wk <= conv_imgk_most_waves(Cin); wk *= 2)
    if (cut_any(Cin, 1, H, W, wk).images < 1) return false;
  return ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(y) | reinterpret_cast<uintptr_t>(res)) & 15) == 0;
}

long long conv_imgk_workgroups(int C, int B, int H, int W, int wk) {
  return cut_any(C, B, H, W, wk).units * (C / (32 * ((C == 64 ? 2 : 4) / wk)));
}

int launch_conv_imgk(const ConvImgkParams &p, hipStream_t stream) {
  if (p.B <= 0) return 0;
  if (!conv_imgk_applicable(p.C, p.C, 3, 3, 1, 1, 1, 1, p.H, p.W, p.shift, p.x, p.y, p.res) || p.lo > p.hi ||
      (reinterpret_cast<uintptr_t>(p.w) & 15) || (reinterpret_cast<uintptr_t>(p.acc0) & (p.fold ? 3 : 15)))
    return (int)hipErrorInvalidValue;
  if (p.fold) return p.C == 64 && p.wk == 1 ? launch_c<64, 1, true>(p, stream) : (int)hipErrorInvalidValue;
  switch (p.C * 8 + p.wk) {
    case 64 * 8 + 1: return launch_c<64, 1, false>(p, stream);
    case 128 * 8 + 1: return launch_c<128, 1, false>(p, stream);
    case 128 * 8 + 2: return launch_c<128, 2, false>(p, stream);
    case 256 * 8 + 1: return launch_c<256, 1, false>(p, stream);
    case 256 * 8 + 2: return launch_c<256, 2, false>(p, stream);
    case 256 * 8 + 4: return launch_c<256, 4, false>(p, stream);
    case 512 * 8 + 1: return launch_c<512, 1, false>(p, stream);
    case 512 * 8 + 2: return launch_c<512, 2, false>(p, stream);
    case 512 * 8 + 4: return launch_c<512, 4, false>(p, stream);
    default: return (int)hipErrorInvalidValue;
  }
}

}  // namespace f8
