// ImageNet stem in one kernel: 7x7 stride-2 convolution of a 3-channel image, requantisation to
// unsigned 8 bits (F8Net Eq. 2, which is also the ReLU) and the 3x3 stride-2 max pool behind it.
// The 112x112x64 tensor between the two never leaves the chip, and never exists as bytes at all: the
// maximum is taken over the 32-bit accumulators (shift and clip are monotonic, so they commute with
// it), and only the pooled pixel is requantised.
//
// Operands: the image as the caller has it, [B][H][W][3], and wp [64][7][8][4], the weights with zeros in the
// first of eight taps of a window row and in the fourth channel.  A window row of convolution pixel q is then the
// eight pixels 2 q - 4 .. 2 q + 3 of four bytes each = one K slice of a 32x32x32 int8 matrix instruction (K = 7 slices),
// and the pixels of a tile fall into groups of four that start at multiples of four, so that the left edge of the
// image never lies inside a group.  What the fourth byte of a pixel and the first tap hold does not matter.
//
// Rows of the implicit GEMM are ordered by pooled pixel, not by convolution pixel.  Pooled pixel
// (i, j) covers convolution rows 2 i - 1 .. 2 i + 1 and columns 2 j - 1 .. 2 j + 1.  The
// convolution pixels fall into four classes by the parity of their row and column; lane (i, j) of
// class (a, b) computes convolution pixel (2 i + a, 2 j + b).  The nine pixels of a pool window are
// then the lane's own four classes, two values of its left neighbour (odd columns), and the
// row maximum over the odd row of the lane above: the first two come through a lane shift inside the
// register file, the last through a small LDS buffer.  Nothing else of the convolution result is
// ever stored.
//
// Every wave works alone (no barrier after set-up) on tiles of 8 x 8 positions: 7 x 7 pooled pixels
// plus the row above and the column to the left, which only feed their neighbours.  The 37 x 40
// pixel patch under a tile is requested while the previous tile's results are requantised and stored, twelve bytes (four
// pixels) per lane and load, spread to four bytes per pixel in registers, put into signed form there (unsigned images
// xor 0x80; pixels outside the image are loads that the descriptor rejects, zeros) and written to the wave's own LDS.
// That costs 50 vector instructions per tile of 750 and replaces a launch that wrote a padded copy of the image to
// memory (batch 256: 17 us of 74).  Rows 8-15 and 24-31 of the patch are stored 8 bytes to the right, which
// makes the fragment reads of the four rows of positions a matrix operand touches fall on
// different banks.
//
// With up to 2048 tiles a wave takes 32 of the 64 channels (NF = 1): twice the waves, half the chain of each, and a third
// workgroup per CU (154 registers).  Microseconds of a launch on images of 224 x 224 (64 tiles each), pad pass + kernel before /
// 64 channels / 32: batch 1 10.7 / 8.3 / 6.0, 8 11.9 / 9.1 / 6.5, 16 13.9 / 9.8 / 8.4, 32 19.6 / 13.0 / 12.3, 48 25.3 / 16.8 /
// 17.3, 64 30.4 / 21.1 / 21.2, 128 47.3 / 37.4 / 38.6, 256 89.7 / 75.4 / 79.3; rows off the four-byte grid (199 x 199) 1 10.8 / 8.7 / 6.3,
// 64 29.5 / 21.6 / 22.3.
// Bound by the vector instructions of the maxima and the requantisation, then by the matrix instructions.  The addresses of
// pieces are worked out anew for every tile (the lane number passes through an empty asm statement): kept in registers over the loop they
// cost 20 of them, spills with 64 channels and the third workgroup with 32.
#include <atomic>

#include "stem_pool.h"

namespace f8 {
namespace {

typedef int v16i __attribute__((ext_vector_type(16)));
typedef int v3i __attribute__((ext_vector_type(3)));

constexpr int SP_NT = 256;
constexpr int TP = 7;                           // pooled rows / columns per tile
constexpr int PROWS = 4 * TP + 9;               // patch rows: 37
constexpr int PPITCH = 160;                     // 40 pixels of 4 bytes
constexpr int PATCH_BYTES = PROWS * PPITCH;     // 5920, contiguous
constexpr int PIECES = PATCH_BYTES / 16;        // 370 pieces of 16 bytes, 10 per row
constexpr int NPIECE = (PIECES + 63) / 64;      // pieces per lane
template <int NF>                               // blocks of 32 channels per wave
struct Lds {
  static constexpr int EPITCH = 128 * NF + 16;            // one position in the exchange buffer: 32 NF channels x 4 bytes + 16
  static constexpr int EROW = 8 * EPITCH;                 // one row of positions
  static constexpr int E_BYTES = 5 * EROW;                // five rows: the four of a block and the last of the block above
  static constexpr int WAVE = PATCH_BYTES + E_BYTES;      // 16800 with 64 channels
};

// Row r of a 32-channel weight fragment holds channel frag_channel(r) of its block: the matrix
// instruction then leaves a lane with 16 consecutive channels of its position (16 half .. 16 half + 15).
__device__ __forceinline__ int frag_channel(int r) { return 16 * ((r >> 2) & 1) + 4 * (r >> 3) + (r & 3); }

// The value of the lane to the left (lane - 1 inside each row of 16 lanes).
__device__ __forceinline__ int from_left(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true); }

// ROWS4: the rows of the image start on multiples of four bytes (x does and W is one of four pixels).
template <int NF, bool ROWS4>
__global__ __launch_bounds__(SP_NT, NF == 1 ? 3 : 2) void stem_pool_kernel(const StemPoolParams p) {
  constexpr int EPITCH = Lds<NF>::EPITCH, EROW = Lds<NF>::EROW;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  __shared__ __attribute__((aligned(16))) int32_t start[64];      // accumulator start values
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  const int ip = l32 >> 3, jp = l32 & 7;        // this lane's position inside a block of 4 x 8 positions
  const int patch_at = wave * Lds<NF>::WAVE, ebuf_at = patch_at + PATCH_BYTES;
  const int nf0 = NF == 2 ? 0 : wave & 1;       // this wave's first block of channels

  auto tile_coords = [&](int t, int &b, int &ti, int &tj) {
    const uint32_t bi = p.fd_tiles.div((uint32_t)t);
    const uint32_t rem = (uint32_t)t - bi * p.fd_tiles.d;
    const uint32_t i = p.fd_tj.div(rem);
    b = (int)bi; ti = (int)i; tj = (int)(rem - i * p.fd_tj.d);
  };
  // (offsets are unsigned: those of rows above and below the image may wrap and are not used)
  const uint32_t row_bytes = 3u * (uint32_t)p.W, image_bytes = (uint32_t)p.H * row_bytes;
  // Piece 64 k + lane of a patch: pixels 4 pc .. 4 pc + 3 of patch row `row`; patch pixel (0, 0) is image pixel
  // (28 ti - 7, 28 tj - 8).
  auto piece_row = [](int k, int lane) { return ((64 * k + lane) * 205) >> 11; };        // / 10 for pieces below 1024
  // The patch of tile t into registers: the 12 bytes of each piece, or the four aligned dwords that cover them.  Pieces
  // outside the image get an offset that the descriptor rejects: zeros.  (A load that starts inside the descriptor returns the
  // dwords that lie inside it.)
  v4i raw[NPIECE];
  auto fetch_patch = [&](int t) {
    int pl = lane;
    asm volatile("" : "+v"(pl));
    int b, ti, tj;
    tile_coords(t, b, ti, tj);
    const uint8_t *image = p.x + (size_t)b * (size_t)image_bytes;
    const uint32_t skew = ROWS4 ? 0u : (uint32_t)(reinterpret_cast<uintptr_t>(image) & 3);
    const __amdgpu_buffer_rsrc_t xres =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(image - skew), 0, (int)((image_bytes + skew + 3) & ~3u), 0x00027000);
    const int gy0 = 4 * TP * ti - 7, gx0 = 4 * TP * tj - 8;
    const uint32_t at0 = (uint32_t)gy0 * row_bytes + 3u * (uint32_t)gx0 + skew;
#pragma unroll
    for (int k = 0; k < NPIECE; ++k) {
      const int row = piece_row(k, pl), pc = 64 * k + pl - 10 * row;
      const bool in = (unsigned)(gy0 + row) < (unsigned)p.H && (unsigned)(gx0 + 4 * pc) < (unsigned)p.W;
      const uint32_t at = at0 + (uint32_t)row * row_bytes + 12u * (uint32_t)pc;
      const uint32_t off = in ? at & ~3u : 0x80000000u;
      if (ROWS4) {
        const v3i d = __builtin_amdgcn_raw_buffer_load_b96(xres, off, 0, 0);
        raw[k] = v4i{d.x, d.y, d.z, 0};
      } else {
        raw[k] = __builtin_amdgcn_raw_buffer_load_b128(xres, off, 0, 0);
      }
    }
  };
  // The same patch from the registers to LDS.
  auto place_patch = [&](int t) {
    int pl = lane;
    asm volatile("" : "+v"(pl));
    int b, ti, tj;
    tile_coords(t, b, ti, tj);
    const int gy0 = 4 * TP * ti - 7, gx0 = 4 * TP * tj - 8;
    const int xm = (int)p.x_xor;
    const uint32_t skew0 =
        ROWS4 ? 0u : (uint32_t)gy0 * row_bytes + 3u * (uint32_t)gx0 + (uint32_t)((reinterpret_cast<uintptr_t>(p.x) + (size_t)b * (size_t)image_bytes) & 3);
    lanes_meet();                                  // the last tile's fragments are read
#pragma unroll
    for (int k = 0; k < NPIECE; ++k) {
      const int row = piece_row(k, pl), pc = 64 * k + pl - 10 * row;
      int d0 = raw[k].x, d1 = raw[k].y, d2 = raw[k].z;
      int px[4];
      if (ROWS4) {
        d0 ^= xm; d1 ^= xm; d2 ^= xm;
        px[0] = d0;
        px[1] = (int)__builtin_amdgcn_alignbyte(d1, d0, 3);
        px[2] = (int)__builtin_amdgcn_alignbyte(d2, d1, 2);
        px[3] = (int)((uint32_t)d2 >> 8);
      } else {
        const uint32_t sh = (skew0 + (uint32_t)row * row_bytes + 12u * (uint32_t)pc) & 3u;
        const int u0 = (int)__builtin_amdgcn_alignbyte(d1, d0, sh), u1 = (int)__builtin_amdgcn_alignbyte(d2, d1, sh),
                  u2 = (int)__builtin_amdgcn_alignbyte(raw[k].w, d2, sh);
        px[0] = u0;
        px[1] = (int)__builtin_amdgcn_alignbyte(u1, u0, 3);
        px[2] = (int)__builtin_amdgcn_alignbyte(u2, u1, 2);
        px[3] = (int)((uint32_t)u2 >> 8);
        // pixels of the piece to the right of the image (a row's first piece starts at the image's left edge or before it)
#pragma unroll
        for (int i = 0; i < 4; ++i) px[i] = (gx0 + 4 * pc + i < p.W ? px[i] : 0) ^ xm;
      }
      // the last two pixels of a row belong to no window, and in a row stored to the right they would lie in the next
      // one: their place is the first two's, written after them
      const int at = patch_at + 1024 * k + 16 * pl + 8 * ((row >> 3) & 1);
      if (64 * k + 63 < PIECES || 64 * k + pl < PIECES) {
        *reinterpret_cast<v2i *>(lds + at + (pc == 9 ? 0 : 8)) = v2i{px[2], px[3]};
        asm volatile("" ::: "memory");
        *reinterpret_cast<v2i *>(lds + at) = v2i{px[0], px[1]};
      }
    }
    lanes_meet();
  };

  constexpr int TPG = 2 * NF;                    // tiles of a workgroup at a time
  const XcdRange tiles = xcd_range(p.ntiles, TPG);
  const int nw = tiles.step, t_end = tiles.end;
  int t = tiles.first + (NF == 2 ? wave : wave >> 1);
  if (t < t_end) fetch_patch(t);

  // weights: fa[nf][r] = channel 32 (nf0 + nf) + frag_channel(l32), bytes 32 r + 16 half .. + 16 of its 224
  v4i fa[NF][7];
#pragma unroll
  for (int nf = 0; nf < NF; ++nf)
#pragma unroll
    for (int r = 0; r < 7; ++r)
      fa[nf][r] = *reinterpret_cast<const v4i *>(p.wp + (size_t)(32 * (nf0 + nf) + frag_channel(l32)) * 224 + 32 * r + 16 * half);
  if (tid < 64) start[tid] = p.acc0[tid];
  __syncthreads();                               // the only barrier

  // Where the window rows of this lane's positions start in the patch.  Position row i' (of the first
  // block; the second lies 16 patch rows lower), class row a, window row r: patch row 4 i' + 2 a + r =
  // 4 i' + c with c = 0 .. 8; class column b adds 8 bytes.
  int fr[3];                                     // by c / 4
#pragma unroll
  for (int c = 0; c < 3; ++c) fr[c] = patch_at + 4 * ip * PPITCH + 8 * (((ip + c) >> 1) & 1) + 16 * jp + 16 * half;
  // exchange buffer: this lane's 16 channels of block nf of position (row slot, jp)
  const int e_lane = ebuf_at + jp * EPITCH + 64 * half;
  const ScaledClip sc = scaled_clip(p.lo, p.hi, p.shift);

  for (; t < t_end; t += nw) {
    int b, ti, tj;
    tile_coords(t, b, ti, tj);
    const int gi0 = TP * ti - 1, gj0 = TP * tj - 1;                   // pooled coordinates of position (0, 0)
    // any convolution pixel of the tile outside the image?  (uniform over the wave)
    const bool edge = ti == 0 || tj == 0 || 2 * (gi0 + 7) + 1 >= p.P || 2 * (gj0 + 7) + 1 >= p.Q;
    place_patch(t);

#pragma unroll
    for (int mf = 0; mf < 2; ++mf) {
      // acc[2 a + b][nf][e]: class (a, b), channel 32 nf + 16 half + e of position (4 mf + ip, jp).
      // The start values are the addend of the first matrix instructions (equal for all classes of a
      // channel, so they commute with the maximum too).
      v16i acc[4][NF], sv[NF];
#pragma unroll
      for (int nf = 0; nf < NF; ++nf)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const v4i s0 = *reinterpret_cast<const v4i *>(start + 32 * (nf0 + nf) + 16 * half + 4 * g);
          sv[nf][4 * g] = s0.x; sv[nf][4 * g + 1] = s0.y; sv[nf][4 * g + 2] = s0.z; sv[nf][4 * g + 3] = s0.w;
        }
      auto frag = [&](int r, int cls) {
        const int a = cls >> 1, bb = cls & 1;
        const uint8_t *src = lds + fr[(2 * a + r) / 4] + (2 * a + r) * PPITCH + 8 * bb + mf * (16 * PPITCH);
        const v2i lo = *reinterpret_cast<const v2i *>(src);
        const v2i hi = *reinterpret_cast<const v2i *>(src + 8);
        return v4i{lo.x, lo.y, hi.x, hi.y};
      };
      v4i fb[2][4];
#pragma unroll
      for (int cls = 0; cls < 4; ++cls) fb[0][cls] = frag(0, cls);
#pragma unroll
      for (int r = 0; r < 7; ++r) {
        if (r + 1 < 7) {
#pragma unroll
          for (int cls = 0; cls < 4; ++cls) fb[(r + 1) & 1][cls] = frag(r + 1, cls);
        }
#pragma unroll
        for (int cls = 0; cls < 4; ++cls)
#pragma unroll
          for (int nf = 0; nf < NF; ++nf)
            acc[cls][nf] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[nf][r], fb[r & 1][cls], r == 0 ? sv[nf] : acc[cls][nf], 0, 0, 0);
      }
      // the next tile's patch is requested before this block's results are worked on
      if (mf == 1 && t + nw < t_end) fetch_patch(t + nw);

      const int gi = gi0 + 4 * mf + ip, gj = gj0 + jp;                // this lane's pooled pixel
      if (edge) {
        // convolution pixels outside the image take part in no maximum
#pragma unroll
        for (int cls = 0; cls < 4; ++cls) {
          const bool ok = (unsigned)(2 * gi + (cls >> 1)) < (unsigned)p.P && (unsigned)(2 * gj + (cls & 1)) < (unsigned)p.Q;
#pragma unroll
          for (int nf = 0; nf < NF; ++nf)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[cls][nf][e] = ok ? acc[cls][nf][e] : (int)0x80000000;
        }
      }
      // Row maxima: he over the even convolution row of the window (columns 2 j - 1, 2 j, 2 j + 1), ho over
      // the odd row below it; ho goes to the exchange buffer for the lane below.  Row slots: position row
      // i goes to slot (i + 1) % 5, so the second block still finds row 3 of the first.
      const int slot_w = mf == 0 ? ip + 1 : ip;
      const int slot_r = mf == 0 ? ip : (ip == 0 ? 4 : ip - 1);
      int he[NF][16], ho[NF][16];
#pragma unroll
      for (int nf = 0; nf < NF; ++nf) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int ee = acc[0][nf][e], eo = acc[1][nf][e], oe = acc[2][nf][e], oo = acc[3][nf][e];
          he[nf][e] = max(max(ee, eo), from_left(eo));
          ho[nf][e] = max(max(oe, oo), from_left(oo));
        }
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *reinterpret_cast<v4i *>(lds + e_lane + slot_w * EROW + 128 * nf + 16 * g) =
              v4i{ho[nf][4 * g], ho[nf][4 * g + 1], ho[nf][4 * g + 2], ho[nf][4 * g + 3]};
      }
      const bool store = 4 * mf + ip >= 1 && jp >= 1 && gi < p.PP && gj < p.QP;
      uint8_t *dst = p.y + (((size_t)b * p.PP + gi) * p.QP + gj) * 64 + 32 * nf0 + 16 * half;
#pragma unroll
      for (int nf = 0; nf < NF; ++nf) {
        int v[16];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const v4i up = *reinterpret_cast<const v4i *>(lds + e_lane + slot_r * EROW + 128 * nf + 16 * g);
#pragma unroll
          for (int j = 0; j < 4; ++j) v[4 * g + j] = max(max(he[nf][4 * g + j], ho[nf][4 * g + j]), up[j]);
        }
        // clip at the accumulator's scale, then one shift-and-pack instruction per value
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = clamp_med3(v[e], sc.lo, sc.hi);
        const v4i pk = shift_pack16(v, p.shift);
        if (store) *reinterpret_cast<v4i *>(dst + 32 * nf) = pk;
      }
    }
  }
}

}  // namespace

bool stem_pool_applicable(int Cout, int R, int S, int sh, int sw, int ph, int pw, int Sp) {
  return Cout == 64 && R == 7 && S == 7 && sh == 2 && sw == 2 && ph == 3 && pw == 3 && Sp == 8;
}

template <int NF, bool ROWS4>
static int launch_as(const StemPoolParams &p, hipStream_t stream) {
  constexpr int bytes = 4 * Lds<NF>::WAVE, limit = NF == 1 ? 768 : 512;   // three or two workgroups per CU walk over the tiles
  static std::atomic<unsigned long long> done_mask{0};    // raising the dynamic LDS limit is per device and idempotent
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return (int)hipErrorInvalidDevice;
  if (dev < 0 || dev > 63 || !((done_mask >> dev) & 1ull)) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(stem_pool_kernel<NF, ROWS4>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e != hipSuccess) return (int)e;
    if (dev >= 0 && dev <= 63) done_mask |= 1ull << dev;
  }
  hipLaunchKernelGGL((stem_pool_kernel<NF, ROWS4>), dim3((unsigned)xcd_grid(p.ntiles, 2 * NF, limit)), dim3(SP_NT), bytes, stream, p);
  return (int)hipGetLastError();
}

int launch_stem_pool(StemPoolParams p, hipStream_t stream) {
  if (p.B <= 0) return 0;
  // what the kernel's indexing assumes, checked before anything is launched
  if (p.P < 1 || p.Q < 1 || p.P != (p.H - 1) / 2 + 1 || p.Q != (p.W - 1) / 2 + 1 || p.H < 1 || p.W < 1 ||
      (long long)p.H * p.W * 3 > 0x7ffffff8LL ||      // (and up to 6 bytes more: whole dwords at any address)
      p.PP != (p.P - 1) / 2 + 1 || p.QP != (p.Q - 1) / 2 + 1 || p.shift < 0 || p.lo < 0 || p.hi > 255 || p.lo > p.hi ||
      (reinterpret_cast<uintptr_t>(p.wp) & 15) || (reinterpret_cast<uintptr_t>(p.acc0) & 15) || (reinterpret_cast<uintptr_t>(p.y) & 15))
    return (int)hipErrorInvalidValue;
  const int tiles_i = (p.PP + TP - 1) / TP, tiles_j = (p.QP + TP - 1) / TP;
  const long long ntiles = (long long)p.B * tiles_i * tiles_j;
  if (ntiles > 0x7fffffffLL) return (int)hipErrorInvalidValue;
  p.ntiles = (int)ntiles;
  p.fd_tiles = FastDiv((uint32_t)(tiles_i * tiles_j));
  p.fd_tj = FastDiv((uint32_t)tiles_j);
  const bool rows4 = ((reinterpret_cast<uintptr_t>(p.x) | (uintptr_t)p.W) & 3) == 0;
  if (ntiles <= 2048) return rows4 ? launch_as<1, true>(p, stream) : launch_as<1, false>(p, stream);
  return rows4 ? launch_as<2, true>(p, stream) : launch_as<2, false>(p, stream);
}

}  // namespace f8
