// Dense fixed-point convolution / GEMM (F8Net Eq. 6 in integer form) for layers with few output tiles, and
// for channel counts and alignments that the LDS-direct kernel (conv_fast_kernel.h) does not take, where K is long or
// odd (conv_igemm.hip takes the others: what lies between the two is in conv_wavek_variant).
//
// What bounds such a layer is not bandwidth or the matrix pipes but one serial chain: a workgroup walks
// along K a step at a time, and a step costs the latency of its operand loads however few workgroups
// there are (0.53 us per 128 bytes of K with two steps in flight: 20.7 us for the 3x3 512 -> 512 layer on
// one 7 x 7 image, whose operands take 0.5 us at the copy rate).  So here
//  * the tile is small (32 x 32 to 64 x 64), which makes workgroups out of a small output, and
//  * the waves of a workgroup share the tile's K range instead of its area: wave w takes the 128-byte
//    K chunks w, w + NW, ..., copies them into LDS of its own (no barrier in the loop, D chunks in flight
//    per wave: 128 KiB in flight per workgroup, 96 for 64 x 32, 64 with four waves, of which two share a CU) and
//    accumulates the whole tile for them.  The partial sums meet in LDS once, at the end; integer sums do not
//    depend on the order.
//  A wave's fragments are then shared by all of its tile (64 x 64: 16 KiB read from LDS per 16 matrix
//  instructions, where four waves that share the area read twice that).
//
// Operands reach LDS in one of two ways.
//  Direct: 16-byte units (16 channels of one tap, or whole taps of a window row that is never clipped),
//  copied by the load unit; units outside the image, past K or past the last row get an offset that the
//  buffer descriptor rejects, which writes zeros.
//  Gather: any channel count and any alignment.  The 16 bytes of a unit are taken from at most two runs of
//  memory (a window row is one run of S * C bytes, of which the image border cuts off a part at either
//  end), each fetched as one unaligned 16-byte load and masked; only units at the very ends of a tensor, or
//  windows whose rows are shorter than 16 bytes, are put together byte by byte.
//
// FOLD: the single-layer calls get their accumulator start values (bias, rounding addend, 128 * sum of the
// weights for unsigned activations) from here too, so that a small call is one launch instead of two: the
// weights of a tile pass through its waves anyway, and four packed dot products per fragment sum them.
#include "conv_wavek.h"

#include "conv_igemm.h"
#include "f8_host.h"

namespace f8 {

namespace {

typedef int v16i __attribute__((ext_vector_type(16)));
typedef int v4i_any __attribute__((ext_vector_type(4), aligned(1)));
typedef __attribute__((address_space(3))) void lds_void;

constexpr int BK = 128;              // bytes of K per chunk

// How operands are fetched: GEMM (1x1, stride 1, no padding: an offset per row, nothing to decode), TAP (at
// most 32 taps of whole multiples of 64 channels: decoded on the scalar unit, a bit mask per row says which
// taps lie inside the image), ANY (16-byte units decoded per lane), GATHER (bytes).
enum { M_GEMM = 0, M_TAP = 1, M_ANY = 2, M_GATHER = 3 };

struct WkTiling {
  int ntiles;
  int m_fast;                        // neighbouring workgroups share the channel tile (else the pixel tile)
  FastDiv fd_fast;                   // by the tiles that neighbouring workgroups walk along
  int x_bytes;
  int run;                           // bytes of a window row: S * C
  int short_runs;                    // a unit can touch more than two window rows
  FastDiv fd_run;
  const int32_t *bias;
};

// Channel fed as row r of a 32-channel block, so that registers 0..15 of a lane are 16 consecutive channels.
__device__ __forceinline__ int frag_channel(int r) { return 16 * ((r >> 2) & 1) + 4 * (r >> 3) + (r & 3); }

// Fragments of two K slices (32 bytes each): MB blocks of pixels, NB blocks of channels, 4 KiB apart each,
// the channel rows WOFF bytes behind the pixel rows.  Reads and wait are one statement: nothing can use or
// reuse the registers before the data is there, and the compiler, which cannot tell these reads from the
// copies into LDS that are still in flight for other chunks, does not wait for those.
template <int MB, int NB, int WOFF>
__device__ __forceinline__ void read_slices(uint32_t s0, uint32_t s1, v4i (&x)[2][MB], v4i (&w)[2][NB]) {
  if constexpr (MB == 1 && NB == 1) {
    asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %4 offset:%6\n\tds_read_b128 %2, %5\n\tds_read_b128 %3, %5 offset:%6\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(x[0][0]), "=&v"(w[0][0]), "=&v"(x[1][0]), "=&v"(w[1][0])
                 : "v"(s0), "v"(s1), "n"(WOFF) : "memory");
  } else if constexpr (MB == 2 && NB == 1) {
    asm volatile("ds_read_b128 %0, %6\n\tds_read_b128 %1, %6 offset:4096\n\tds_read_b128 %2, %6 offset:%8\n\t"
                 "ds_read_b128 %3, %7\n\tds_read_b128 %4, %7 offset:4096\n\tds_read_b128 %5, %7 offset:%8\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(x[0][0]), "=&v"(x[0][1]), "=&v"(w[0][0]), "=&v"(x[1][0]), "=&v"(x[1][1]), "=&v"(w[1][0])
                 : "v"(s0), "v"(s1), "n"(WOFF) : "memory");
  } else {
    static_assert(MB == 2 && NB == 2, "tile shapes");
    asm volatile("ds_read_b128 %0, %8\n\tds_read_b128 %1, %8 offset:4096\n\tds_read_b128 %2, %8 offset:%10\n\tds_read_b128 %3, %8 offset:%11\n\t"
                 "ds_read_b128 %4, %9\n\tds_read_b128 %5, %9 offset:4096\n\tds_read_b128 %6, %9 offset:%10\n\tds_read_b128 %7, %9 offset:%11\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(x[0][0]), "=&v"(x[0][1]), "=&v"(w[0][0]), "=&v"(w[0][1]), "=&v"(x[1][0]), "=&v"(x[1][1]), "=&v"(w[1][0]), "=&v"(w[1][1])
                 : "v"(s0), "v"(s1), "n"(WOFF), "n"(WOFF + 4096) : "memory");
  }
}

// Wait until at most n chunks of LPC loads each are still on their way (n <= MAXN).
template <int MAXN, int LPC>
__device__ __forceinline__ void wait_chunks(int n) {
  if constexpr (MAXN <= 0) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  } else {
    static_assert(MAXN * LPC < 64, "the load counter holds 63");
    if (n >= MAXN) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(MAXN * LPC) : "memory");
    else wait_chunks<MAXN - 1, LPC>(n);
  }
}

// Bytes [a, b) of a dword that starts at byte 4 d of a unit.
__device__ __forceinline__ uint32_t byte_mask(int a, int b, int d) {
  const int lo = min(max(a - 4 * d, 0), 4), hi = min(max(b - 4 * d, 0), 4);
  const uint32_t below_hi = hi == 4 ? 0xffffffffu : (1u << (8 * hi)) - 1u;
  const uint32_t below_lo = lo == 4 ? 0xffffffffu : (1u << (8 * lo)) - 1u;
  return below_hi & ~below_lo;
}

// Bytes [a, b) of the 16 bytes at base + off, the others zero.  Only bytes [a, b) are known to lie inside the
// tensor of `size` bytes.
__device__ __forceinline__ v4i gather_run(const uint8_t *base, int off, int size, int a, int b) {
  v4i v = {0, 0, 0, 0};
  if (a >= b) return v;
  if (off >= 0 && off <= size - 16) {
    v = *reinterpret_cast<const v4i_any *>(base + off);
    if (a > 0 || b < 16) {
#pragma unroll
      for (int d = 0; d < 4; ++d) v[d] &= (int)byte_mask(a, b, d);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (i >= a && i < b) v[i >> 2] |= (int)((uint32_t)base[off + i] << (8 * (i & 3)));
  }
  return v;
}

template <int TM, int TN, int NW, int D, int MODE, bool FOLD>
__global__ __launch_bounds__(64 * NW, MODE == M_GATHER && NW == 4 ? 2 : 1) void conv_wavek_kernel(const ConvParams p, const WkTiling tl) {
  constexpr int NT = 64 * NW;
  constexpr bool GATHER = MODE == M_GATHER;
  constexpr int MB = TM / 32, NB = TN / 32;
  constexpr int XR = TM / 8, WR = TN / 8;         // 1 KiB copies (8 rows) per chunk
  constexpr int LPC = XR + WR;
  constexpr int STAGE = (TM + TN) * BK;           // bytes of one chunk in LDS
  constexpr int PITCH = TN * 4 + 16;              // row pitch of the partial sums
  constexpr int GROUPS = TM * TN / 4;             // results leave in groups of four channels
  constexpr int GPT = (GROUPS + NT - 1) / NT;
  constexpr int GROW = TN / 4;                    // groups per pixel
  static_assert(NT % GROW == 0, "a thread keeps its channels");

  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];

  pin_args(tl.ntiles, tl.fd_fast.mul, tl.fd_fast.shr, tl.fd_fast.d, tl.m_fast, tl.x_bytes, p.x, p.w, p.C, p.N, p.M, p.K, p.acc0, p.res);
  if (MODE != M_GEMM) pin_args(p.fd_pq.mul, p.fd_pq.shr, p.fd_pq.d, p.fd_q.mul, p.fd_q.shr, p.fd_q.d, p.H, p.W, p.sh, p.sw, p.ph, p.pw);
  if (MODE == M_TAP) pin_args(p.fd_c.mul, p.fd_c.shr, p.fd_c.d, p.fd_s.mul, p.fd_s.shr, p.fd_s.d, p.R, p.S, p.tap_rep);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  const uint32_t tile = xcd_remap(blockIdx.x, (uint32_t)tl.ntiles);
  const int slow = (int)tl.fd_fast.div(tile), fast = (int)tile - slow * (int)tl.fd_fast.d;
  const int m0 = (tl.m_fast ? fast : slow) * TM, n0 = (tl.m_fast ? slow : fast) * TN;

  // ---- loader: row 8 i + lane / 8 of the tile, physical 16-byte piece lane % 8 of its 128 bytes.  The pieces
  // of a row are permuted by the row number (conflict-free fragment reads); rows 8 i with even and odd i hold
  // logical pieces that differ in bit 2.
  const int lrow = lane >> 3;
  const int piece[2] = {(lane & 7) ^ (lane >> 4), (lane & 7) ^ (lane >> 4) ^ 4};
  // What the rows need: byte offset of the window's first tap, and (GEMM) nothing else, (TAP) the mask of taps
  // outside the image, (ANY, GATHER) the window's first row and column.  Lane l works it out for row l of the
  // tile and the lanes that fetch the row get it from there.
  int x_off[XR], x_ih[XR], x_iw[XR];
  if (MODE == M_GEMM) {
    // (rows past the last pixel lie past the end of the tensor)
    const int first = (m0 + lrow) * p.C;
#pragma unroll
    for (int i = 0; i < XR; ++i) {
      x_ih[i] = x_iw[i] = 0;
      x_off[i] = first + i * (8 * p.C) + piece[i & 1] * 16;
    }
  } else {
    // (a row past the last pixel: no tap inside)
    int off = 0, ih = MODE == M_TAP ? -1 : -(1 << 28), iw = 0;
    const int m = m0 + (lane & (TM - 1));
    if (m < p.M) {
      const uint32_t b = p.fd_pq.div((uint32_t)m);
      const uint32_t rem = (uint32_t)m - b * p.fd_pq.d;
      const uint32_t pp = p.fd_q.div(rem);
      const uint32_t qq = rem - pp * p.fd_q.d;
      ih = (int)pp * p.sh - p.ph;
      iw = (int)qq * p.sw - p.pw;
      off = (((int)b * p.H + ih) * p.W + iw) * p.C;
      if (MODE == M_TAP) {
        // taps inside the image form a rectangle of the window: its bit mask is (column bits) times (one
        // bit per valid row, S bits apart)
        const int r_lo = max(0, -ih), r_hi = min(p.R, p.H - ih), s_lo = max(0, -iw), s_hi = min(p.S, p.W - iw);
        uint32_t in = 0;
        if (r_hi > r_lo && s_hi > s_lo) {
          const uint32_t cols = (s_hi >= 32 ? 0u : (1u << s_hi)) - (1u << s_lo);
          const uint32_t top = r_hi * p.S >= 32 ? 0u : (1u << (r_hi * p.S));
          in = cols * ((top - (1u << (r_lo * p.S))) & p.tap_rep);
        }
        ih = (int)~in;
      }
    }
#pragma unroll
    for (int i = 0; i < XR; ++i) {
      x_off[i] = __shfl(off, 8 * i + lrow, 64);
      x_ih[i] = __shfl(ih, 8 * i + lrow, 64);
      x_iw[i] = MODE == M_TAP ? 0 : __shfl(iw, 8 * i + lrow, 64);
    }
  }
  int w_off[WR];
  // (from the tile's first channel on; row 8 i + lrow of a block of 32 is channel frag_channel(lrow) + 4 i, and rows past the
  // last channel lie past the end of the tile's weights)
  const int w_first = frag_channel(lrow) * p.K;
#pragma unroll
  for (int i = 0; i < WR; ++i) {
    const int n = n0 + 32 * (i >> 2) + 4 * (i & 3) + frag_channel(lrow);
    const int off = w_first + (32 * (i >> 2) + 4 * (i & 3)) * p.K;
    if (GATHER) w_off[i] = n < p.N ? off : -1;
    else w_off[i] = off + piece[i & 1] * 16;
  }
  uint8_t *own = lds + wave * (D * STAGE);
  const uint32_t own_at = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) uint8_t *)own);
  const int nchunks = (p.K + BK - 1) / BK;
  const int mine = wave < nchunks ? (nchunks - wave + NW - 1) / NW : 0;     // chunks wave, wave + NW, ...

  const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(p.x), 0, tl.x_bytes, 0x00027000);
  const uint8_t *w_tile = reinterpret_cast<const uint8_t *>(p.w) + (size_t)n0 * p.K;
  const int w_bytes = min(TN, p.N - n0) * p.K;                   // K <= 65536: at most 4 MiB
  const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(w_tile), 0, w_bytes, 0x00027000);

  const bool k_tail = (p.K & (BK - 1)) != 0;
  auto copy_chunk = [&](int chunk, int stage) {
    const int k0 = chunk * BK;
    const bool tail = k_tail && chunk == nchunks - 1;            // pieces past K: zeros (uniform)
    uint8_t *to = own + stage * STAGE;
    int toff[2] = {0, 0}, r[2] = {0, 0}, s[2] = {0, 0};
    const bool in_k[2] = {k0 + piece[0] * 16 < p.K, k0 + piece[1] * 16 < p.K};
    if (MODE == M_TAP) {
      // the two 64-channel halves of the chunk on the scalar unit, then each lane picks its own
      int off[2], sh[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const uint32_t k = (uint32_t)(k0 + 64 * q), tap = p.fd_c.div(k), rr = p.fd_s.div(tap);
        off[q] = ((int)rr * p.W + (int)(tap - rr * p.fd_s.d)) * p.C + (int)(k - tap * p.fd_c.d);
        sh[q] = 31 - (int)tap;                                   // (a half past K: any value, masked below)
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const bool hi = (piece[h] & 4) != 0;
        toff[h] = (hi ? off[1] : off[0]) + (piece[h] & 3) * 16;
        s[h] = hi ? sh[1] : sh[0];
      }
    } else if (MODE == M_ANY) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t k = (uint32_t)(k0 + piece[h] * 16);
        const uint32_t tap = p.fd_c.div(k);
        const uint32_t rr = p.fd_s.div(tap);
        r[h] = (int)rr;
        s[h] = (int)(tap - rr * p.fd_s.d);
        toff[h] = (r[h] * p.W + s[h]) * p.C + (int)(k - tap * p.fd_c.d);
      }
    }
#pragma unroll
    for (int i = 0; i < XR; ++i) {
      const int h = i & 1;
      uint32_t off;
      if (MODE == M_GEMM) {
        off = (uint32_t)x_off[i];
      } else if (MODE == M_TAP) {
        off = (uint32_t)(x_off[i] + toff[h]) | (((uint32_t)x_ih[i] << (s[h] & 31)) & 0x80000000u);
      } else {
        const bool ok = in_k[h] && (unsigned)(x_ih[i] + r[h]) < (unsigned)p.H && (unsigned)(x_iw[i] + s[h]) < (unsigned)p.W;
        off = ok ? (uint32_t)(x_off[i] + toff[h]) : 0x80000000u;
      }
      if (MODE != M_ANY && tail && !in_k[h]) off = 0x80000000u;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(xres, (lds_void *)(to + i * 1024), 16, off, MODE == M_GEMM ? k0 : 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < WR; ++i) {
      const uint32_t off = tail && !in_k[i & 1] ? 0x80000000u : (uint32_t)w_off[i];
      __builtin_amdgcn_raw_ptr_buffer_load_lds(wres, (lds_void *)(to + TM * BK + i * 1024), 16, off, k0, 0, 0);
    }
  };

  auto gather_chunk = [&](int chunk) {
    v4i xv[XR], wv[WR];
#pragma unroll
    for (int i = 0; i < WR; ++i) {
      const int k0 = chunk * BK + piece[i & 1] * 16;
      wv[i] = w_off[i] >= 0 ? gather_run(w_tile, w_off[i] + k0, w_bytes, 0, min(16, p.K - k0))
                            : v4i{0, 0, 0, 0};
    }
    if (tl.short_runs) {
#pragma unroll
      for (int i = 0; i < XR; ++i) {
        xv[i] = v4i{0, 0, 0, 0};
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const int k = chunk * BK + piece[i & 1] * 16 + j;
          const uint32_t tap = p.fd_c.div((uint32_t)k);
          const int c = k - (int)(tap * p.fd_c.d);
          const int r = (int)p.fd_s.div(tap), s = (int)tap - r * p.S;
          if (k < p.K && (unsigned)(x_ih[i] + r) < (unsigned)p.H && (unsigned)(x_iw[i] + s) < (unsigned)p.W)
            xv[i][j >> 2] |= (int)((uint32_t)p.x[x_off[i] + (r * p.W + s) * p.C + c] << (8 * (j & 3)));
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < XR; ++i) {
        // bytes j0 .. of window row r, then (from byte t of the unit on) the start of row r + 1
        const uint32_t k0 = (uint32_t)(chunk * BK + piece[i & 1] * 16);
        const int r = (int)tl.fd_run.div(k0), j0 = (int)(k0 - (uint32_t)r * tl.fd_run.d);
        const int t = tl.run - j0;
        // the part of a window row that lies inside the image
        const int lo = max(0, -x_iw[i]) * p.C, hi = min(p.S, p.W - x_iw[i]) * p.C;
        const bool in0 = r < p.R && (unsigned)(x_ih[i] + r) < (unsigned)p.H;
        const bool in1 = r + 1 < p.R && (unsigned)(x_ih[i] + r + 1) < (unsigned)p.H;
        const int off = x_off[i] + r * p.W * p.C + j0;
        xv[i] = gather_run(p.x, off, tl.x_bytes, max(lo - j0, 0), in0 ? min(hi - j0, 16) : 0);
        if (t < 16) {
          const v4i v = gather_run(p.x, x_off[i] + (r + 1) * p.W * p.C - t, tl.x_bytes, lo + t, in1 ? min(hi + t, 16) : 0);
#pragma unroll
          for (int d = 0; d < 4; ++d) xv[i][d] |= v[d];
        }
      }
    }
#pragma unroll
    for (int i = 0; i < XR; ++i) *reinterpret_cast<v4i *>(own + i * 1024 + lane * 16) = xv[i];
#pragma unroll
    for (int i = 0; i < WR; ++i) *reinterpret_cast<v4i *>(own + TM * BK + i * 1024 + lane * 16) = wv[i];
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // the wave's own writes, read back below
  };

  // ---- K loop ------------------------------------------------------------------------------
  v16i acc[NB][MB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[nb][mb][i] = 0;
  int wsum[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) wsum[nb] = 0;
  const int xm = (int)p.xor_mask;
  uint32_t foff[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) foff[ks] = (uint32_t)(l32 * BK + (((2 * ks + half) ^ ((l32 >> 1) & 7)) * 16));

  if (!GATHER) {
#pragma unroll
    for (int s = 0; s < D; ++s)
      if (s < mine) copy_chunk(wave + s * NW, s);
  }
  __builtin_amdgcn_sched_barrier(0);
  // ---- what the epilogue needs from memory, requested behind the first operands: four channels n .. n + 3 per
  // thread, pixels row0 + k * (NT / GROW)
  const int n = n0 + (tid % GROW) * 4, row0 = tid / GROW;
  const bool n_vec = (p.N & 3) == 0;
  v4i start = {0, 0, 0, 0};
  if (n < p.N) {
    if (FOLD) {
      const int rnd = p.shift > 0 ? 1 << (p.shift - 1) : 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) start[i] = rnd + (tl.bias && n + i < p.N ? tl.bias[n + i] : 0);
    } else {
      start = *reinterpret_cast<const v4i *>(p.acc0 + n);
    }
  }
  const bool r_vec = n_vec && (reinterpret_cast<uintptr_t>(p.res) & 3) == 0;
  uint32_t res8[GPT];
  if (p.res && p.res_type != T_S32) {
#pragma unroll
    for (int k = 0; k < GPT; ++k) {
      const int row = row0 + k * (NT / GROW), m = m0 + row;
      res8[k] = 0;
      if (row < TM && m < p.M && n < p.N) {
        const uint8_t *rp = static_cast<const uint8_t *>(p.res) + (size_t)m * p.N + n;
        if (r_vec) {
          res8[k] = *reinterpret_cast<const uint32_t *>(rp);
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (n + i < p.N) res8[k] |= (uint32_t)rp[i] << (8 * i);
        }
      }
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  int stage = 0;
  for (int j = 0; j < mine; ++j) {
    if (GATHER) gather_chunk(wave + j * NW);
    else wait_chunks<D - 1, LPC>(min(D - 1, mine - 1 - j));
    const uint32_t at = own_at + (uint32_t)(stage * STAGE);
    v4i fx[2][2][MB], fw[2][2][NB];
    read_slices<MB, NB, TM * BK>(at + foff[0], at + foff[1], fx[0], fw[0]);
    read_slices<MB, NB, TM * BK>(at + foff[2], at + foff[3], fx[1], fw[1]);
    if (!GATHER && j + D < mine) {
      __builtin_amdgcn_sched_barrier(0);
      copy_chunk(wave + (j + D) * NW, stage);                // every fragment of the chunk is in registers
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int h = t >> 1, ks = t & 1;
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        fx[h][ks][mb].x ^= xm; fx[h][ks][mb].y ^= xm; fx[h][ks][mb].z ^= xm; fx[h][ks][mb].w ^= xm;
      }
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        if (FOLD) {
#pragma unroll
          for (int d = 0; d < 4; ++d) wsum[nb] = __builtin_amdgcn_sdot4(fw[h][ks][nb][d], 0x01010101, wsum[nb], false);
        }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
          acc[nb][mb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fw[h][ks][nb], fx[h][ks][mb], acc[nb][mb], 0, 0, 0);
      }
    }
    if (++stage == D || GATHER) stage = 0;
  }
  __syncthreads();                    // no wave reads its chunks any more: LDS takes the partial sums

  // ---- partial sums: [wave][pixel][channel], then the sums of the weights [wave][channel] -----
  uint8_t *part = lds + wave * (TM * PITCH);
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<v4i *>(part + (mb * 32 + l32) * PITCH + nb * 128 + half * 64 + g * 16) =
            v4i{acc[nb][mb][4 * g], acc[nb][mb][4 * g + 1], acc[nb][mb][4 * g + 2], acc[nb][mb][4 * g + 3]};
  int *sums = reinterpret_cast<int *>(lds + NW * TM * PITCH);
  if (FOLD) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int s = wsum[nb] + __shfl_xor(wsum[nb], 32, 64);
      if (half == 0) sums[wave * TN + nb * 32 + frag_channel(l32)] = s;
    }
  }
  __syncthreads();

  if (n >= p.N) return;
  if (FOLD && xm != 0) {
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const v4i s = *reinterpret_cast<const v4i *>(sums + w * TN + (n - n0));
#pragma unroll
      for (int i = 0; i < 4; ++i) start[i] += 128 * s[i];
    }
  }
  // ---- epilogue: residual, rounding shift, clip, pack, store ---------------------------------
  const bool y_vec = n_vec && (reinterpret_cast<uintptr_t>(p.y) & (p.y_type == T_S32 ? 15 : 3)) == 0;
#pragma unroll
  for (int k = 0; k < GPT; ++k) {
    const int row = row0 + k * (NT / GROW), m = m0 + row;
    if (row >= TM || m >= p.M) continue;
    const size_t o = (size_t)m * p.N + n;
    int v[4] = {start.x, start.y, start.z, start.w};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const v4i a = *reinterpret_cast<const v4i *>(lds + w * (TM * PITCH) + row * PITCH + (n - n0) * 4);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] += a[i];
    }
    if (p.res) {
      if (p.res_type == T_S32) {
        const int32_t *rp = static_cast<const int32_t *>(p.res) + o;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (n + i < p.N) v[i] += align_res(rp[i], p.res_d);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] += align_res(byte_of(res8[k], i, p.res_type == T_S8), p.res_d);
      }
    }
    if (p.y_type == T_S32) {
      int32_t *yp = static_cast<int32_t *>(p.y) + o;
      if (y_vec) {
        *reinterpret_cast<v4i *>(yp) = v4i{v[0], v[1], v[2], v[3]};
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (n + i < p.N) yp[i] = v[i];
      }
      continue;
    }
    if (p.y2) {
      // second format of the same accumulator: swap the rounding addend, shift, clip
      int u[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        u[i] = p.shift2 >= 0 ? requant<false>(v[i] + p.add2, p.shift2, p.lo2, p.hi2)
                             : requant<true>(v[i] + p.add2, p.shift2, p.lo2, p.hi2);
      uint8_t *yp2 = static_cast<uint8_t *>(p.y2) + o;
      if (n_vec && (reinterpret_cast<uintptr_t>(p.y2) & 3) == 0) {
        *reinterpret_cast<uint32_t *>(yp2) = pack4(u[0], u[1], u[2], u[3]);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (n + i < p.N) yp2[i] = (uint8_t)u[i];
      }
    }
    if (p.shift >= 0) {
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = requant<false>(v[i], p.shift, p.lo, p.hi);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = requant<true>(v[i], p.shift, p.lo, p.hi);
    }
    uint8_t *yp = static_cast<uint8_t *>(p.y) + o;
    if (y_vec) {
      *reinterpret_cast<uint32_t *>(yp) = pack4(v[0], v[1], v[2], v[3]);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (n + i < p.N) yp[i] = (uint8_t)v[i];
    }
  }
}

template <int TM, int TN, int NW, int D, int MODE, bool FOLD>
int launch_one(const ConvParams &p, const int32_t *bias, hipStream_t stream) {
  WkTiling tl;
  const int tiles_m = (p.M + TM - 1) / TM, tiles_n = (p.N + TN - 1) / TN;
  const long long ntiles = (long long)tiles_m * tiles_n;
  if (ntiles > 0x7fffffffLL) return (int)hipErrorInvalidValue;
  tl.ntiles = (int)ntiles;
  tl.x_bytes = p.B * p.H * p.W * p.C;
  // neighbouring tiles run on one XCD: let them share the larger operand
  tl.m_fast = (long long)p.N * p.K > tl.x_bytes;
  tl.fd_fast = FastDiv((uint32_t)(tl.m_fast ? tiles_m : tiles_n));
  tl.run = p.S * p.C;
  tl.short_runs = p.R > 1 && tl.run < 16;
  tl.fd_run = FastDiv((uint32_t)tl.run);
  tl.bias = bias;
  // the chunks, later the partial sums of pixels and of weights
  constexpr int ring = NW * D * (TM + TN) * BK, partial = NW * (TM * (TN * 4 + 16) + TN * 4);
  constexpr int smem = ring > partial ? ring : partial;
  auto k = conv_wavek_kernel<TM, TN, NW, D, MODE, FOLD>;
  // per device and idempotent; remember which devices have it
  static std::atomic<unsigned long long> done_mask{0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return (int)hipErrorInvalidDevice;
  if (dev < 0 || dev > 63 || !((done_mask.load(std::memory_order_relaxed) >> dev) & 1ull)) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    if (e != hipSuccess) return (int)e;
    if (dev >= 0 && dev <= 63) done_mask.fetch_or(1ull << dev, std::memory_order_relaxed);
  }
  hipLaunchKernelGGL(k, dim3((unsigned)ntiles), dim3(64 * NW), smem, stream, p, tl);
  return (int)hipGetLastError();
}

template <int TM, int TN, int NW>
int launch_gather(const ConvParams &p, bool fold, const int32_t *bias, hipStream_t stream) {
  return fold ? launch_one<TM, TN, NW, 1, M_GATHER, true>(p, bias, stream) : launch_one<TM, TN, NW, 1, M_GATHER, false>(p, bias, stream);
}

template <int TM, int TN, int NW, int D, bool FOLD>
int launch_mode(const ConvParams &p, const int32_t *bias, hipStream_t stream) {
  if (p.gemm) return launch_one<TM, TN, NW, D, M_GEMM, FOLD>(p, bias, stream);
  if ((p.C & 63) == 0 && p.R * p.S <= 32) return launch_one<TM, TN, NW, D, M_TAP, FOLD>(p, bias, stream);
  return launch_one<TM, TN, NW, D, M_ANY, FOLD>(p, bias, stream);
}

template <int TM, int TN, int NW, int D>
int launch_direct(const ConvParams &p, bool fold, const int32_t *bias, hipStream_t stream) {
  return fold ? launch_mode<TM, TN, NW, D, true>(p, bias, stream) : launch_mode<TM, TN, NW, D, false>(p, bias, stream);
}

}  // namespace

bool conv_wavek_direct(const ConvParams &p) {
  if ((reinterpret_cast<uintptr_t>(p.x) | reinterpret_cast<uintptr_t>(p.w)) & 15) return false;
  // small C: whole taps of one window row, when no window is ever clipped by the image border
  const bool packed = p.C < 16 && 16 % p.C == 0 && ((p.S * p.C) & 15) == 0 && p.ph == 0 && p.pw == 0 &&
                      (p.P - 1) * p.sh + p.R <= p.H && (p.Q - 1) * p.sw + p.S <= p.W;
  return (p.C & 15) == 0 || packed;
}

// Up to how many 32 x 32 tiles this kernel is ahead of conv_igemm on layers that conv_fast does not take, by K and by the
// width of that kernel's gather.  A tile costs more here (the sums of the waves), a chunk of K less; measured on 1900
// layers of 1000 to 400000 pixels (us, here / there):
//   16 bytes: 64 -> 255 on 3136 pixels (784 tiles) 6.2 / 10.8, on 12544 (3136) 17.5 / 11.4; K = 512 18.7 / 16.1; K = 1024 21.0 / 21.3;
//     K = 2048 27 / 32, on 50176 pixels (12544) 86 / 79.  One tile wide (N <= 32): 256 -> 30 on 50176 pixels (1568) 10.5 / 9.0, K =
//     1024 16.1 / 22.7, 2048 on 200704 (6272) 89 / 105;
//   4 bytes: K = 108 -> 49 with a 32-bit residual on 9212 (576) 11.7 / 20.1, 60 -> 62 on 12544 (784) 14.5 / 10.7, 124 -> 130 there
//     (1960) 21.0 / 12.0, 1800 -> 130 there 37 / 48, 1980 -> 256 on 7800 (1952) 28.7 / 51.5;
//   single bytes, which keep that kernel's gather busy: 401 -> 255 on 200704 (50176) 293 / 576, 147 -> 62 there (12544) 82 / 85,
//     75 -> 62 on 50176 (3136) 26.5 / 26.0, 27 -> 62 there 26.1 / 18.5, on 12544 (784) 14.4 / 17.7.
static long long general_limit(const ConvParams &p) {
  const int K = p.K;
  const bool one = p.N <= 32;
  const long long any = 1LL << 62;
  const int vec = conv_igemm_vec(p);
  // windows whose rows are shorter than 16 bytes: each wave gathers them byte by byte, one row of pixels after another
  // (3x3 on three channels, 32 of them out of 12544 pixels, 16.7 / 14.5; 401408 pixels 331 / 51); ahead on few pixels of
  // odd channel counts only (1 -> 62, 3136 pixels: 13.0 / 15.6)
  if (p.R > 1 && p.S * p.C < 16) return vec == 1 && !one ? 768 : -1;
  long long limit;
  if (vec == 16) limit = one ? (K < 256 ? 512 : K < 1024 ? 1536 : K < 2048 ? 3072 : any) : (K < 64 ? 1024 : K < 256 ? 1536 : K < 1024 ? 2048 : 4096);
  else if (vec == 4) limit = one ? (K < 128 ? 512 : K < 256 ? 768 : K < 1024 ? 1536 : K < 1536 ? 2048 : any) : (K < 128 ? 768 : K < 256 ? 1536 : K < 1536 ? 2048 : 8192);
  else limit = K >= 256 ? any : K >= 128 ? (p.R == 1 && p.S == 1 ? 16384 : 6144) : one ? 1024 : K < 64 ? 1536 : 2048;
  // a residual or a second format of odd rows goes byte by byte in conv_igemm's epilogue (16 -> 102 with both on 8954 pixels,
  // 1120 tiles: 12.0 / 19.0; 400 -> 473 with both, 2265: 20.5 / 25.4)
  return (p.N & 3) != 0 && (p.res || p.y2) && limit < any ? limit + limit / 2 : limit;
}

int conv_wavek_variant(const ConvParams &p, bool general) {
  const int f = tuning().wavek_variant.load(std::memory_order_relaxed);      // tuning aid: force one tile shape
  if (f >= 0 && f < WK_VARIANTS) return f;
  if (tuning().wavek.load(std::memory_order_relaxed) == 0) return -1;
  if (!general && tuning().conv_variant.load(std::memory_order_relaxed) >= 0) return -1;
  // Measured against each other and against conv_fast on the layers of ResNet-50 and MobileNetV2 at batch 1
  // to 64, where every CU has at most one workgroup (two of the 64 KiB shape):
  //  * up to one 32 x 32 tile per CU: eight waves share K when it is long (7 x 7 3x3 512 -> 512, one image:
  //    6.0 us, four waves 7.0, conv_fast 20.7), four otherwise (28 x 28 1x1 512 -> 256: 2.8 / 2.9 / 5.1);
  //  * up to two per CU: 64 x 32 tiles for long K (batch 16 of the 3x3 layer above: 8.3 us, two 32 x 32
  //    tiles per CU 9.1, conv_fast 21.4), else two 32 x 32 (1x1 512 -> 128 at batch 4: 3.3 / 5.7);
  //  * up to one 64 x 64 tile per CU, K from 512 on (14 x 14 3x3 256 -> 256, batch 16: 8.0 / 13.7; 1x1 with
  //    K = 512: 4.6 / 5.7, with K = 256: 4.4 / 4.1).
  // Beyond that every further round of workgroups costs its whole latency chain again and conv_fast, which
  // keeps several tiles per CU in flight, is ahead (3x3 256 -> 256 at batch 32: 15.0 / 13.0).
  auto tiles = [&](int bm, int bn) { return (long long)((p.M + bm - 1) / bm) * ((p.N + bn - 1) / bn); };
  const long long t32 = tiles(32, 32);
  if (general) {
    if (t32 > general_limit(p)) return -1;
    // gathered: 64 x 64 tiles, which halve the gathering, from four to six 32 x 32 tiles per CU on (us, 32 x 32 / 64 x 64: K =
    // 900 -> 76 channels, 588 of them, 13.3 / 18.9; 612 -> 157, 980, 17.7 / 19.2; 459 -> 49, 1176, 16.8 / 16.3; 162 -> 50,
    // 1520, 16.3 / 16.1; 558 -> 48, 1914, 28.7 / 21.5), earlier where one 64 x 64 tile per CU is all there is (157 -> 1208,
    // 874 and 228 tiles: 14.0 / 12.4); where N is one tile wide 32 x 32 (900 -> 23, 1078: 20.9, 64 x 32 27.5), but for
    // the fourth per CU (729 -> 30, 816: 20.1, 64 x 32 16.9)
    if (!conv_wavek_direct(p)) {
      if (t32 <= 256 && p.K >= 1024) return WK_32x32_W8;
      if (p.N <= 32) return t32 > 768 && t32 <= 1024 ? WK_64x32_W8 : WK_32x32_W4;
      return t32 <= 768 || (t32 <= (p.K < 256 ? 1536 : 1024) && tiles(64, 64) > 256) ? WK_32x32_W4 : WK_64x64_W8;
    }
  }
  if (t32 <= 256) return p.K >= 1024 ? WK_32x32_W8 : WK_32x32_W4;
  if (t32 <= 512 && p.K < 2048) return WK_32x32_W4;
  if (tiles(64, 32) <= 256) return WK_64x32_W8;
  if (tiles(64, 64) <= 256 && (p.K >= 512 || (general && p.N > 32))) return WK_64x64_W8;
  if (!general) return -1;
  return p.N <= 32 || (t32 <= 1536 && p.K < 1024) ? WK_32x32_W4 : WK_64x64_W8;
}

const char *conv_wavek_name(int variant, bool direct) {
  static const char *const names[2][WK_VARIANTS] = {
      {"conv_wavek_gather<32x32,w8>", "conv_wavek_gather<32x32,w4>", "conv_wavek_gather<64x32,w4>", "conv_wavek_gather<64x64,w4>"},
      {"conv_wavek<32x32,w8>", "conv_wavek<32x32,w4>", "conv_wavek<64x32,w8>", "conv_wavek<64x64,w8>"}};
  return variant >= 0 && variant < WK_VARIANTS ? names[direct][variant] : "?";
}

int launch_conv_wavek(const ConvParams &p, int variant, bool fold, const int32_t *bias, hipStream_t stream) {
  if (!conv_wavek_direct(p)) {
    // a wave gathers the next chunk itself, into registers first: one chunk in LDS; four waves per workgroup
    // for the 64-pixel tiles, so that two or three workgroups share a CU
    switch (variant) {
      case WK_32x32_W8: return launch_gather<32, 32, 8>(p, fold, bias, stream);
      case WK_32x32_W4: return launch_gather<32, 32, 4>(p, fold, bias, stream);
      case WK_64x32_W8: return launch_gather<64, 32, 4>(p, fold, bias, stream);
      case WK_64x64_W8: return launch_gather<64, 64, 4>(p, fold, bias, stream);
      default: return -1;
    }
  }
  switch (variant) {
    case WK_32x32_W8: return launch_direct<32, 32, 8, 2>(p, fold, bias, stream);
    case WK_32x32_W4: return launch_direct<32, 32, 4, 2>(p, fold, bias, stream);
    case WK_64x32_W8: return launch_direct<64, 32, 8, 1>(p, fold, bias, stream);
    case WK_64x64_W8: return launch_direct<64, 64, 8, 1>(p, fold, bias, stream);
    default: return -1;
  }
}

}  // namespace f8
