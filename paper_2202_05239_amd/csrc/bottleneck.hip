// Three layers of a bottleneck network in one launch: the 3x3 layer C -> C (pad 1, stride 1 or 2), the 1x1 layer C -> 4 C
// behind it with residual and up to two output formats, and the 1x1 layer 4 C -> C (or 2 C) that opens the next block.
//
// At small and medium batch each of the three is bound by what one launch costs beyond its work: a launch behind another
// one takes 1.6 us in a graph and 2.4 us on a stream even if it does nothing, then weights and activations come cold from
// the other XCDs' writes, and one wave's serial chain follows.  The three act on the same output pixels, so a workgroup
// takes TM of them through all three layers: the input rows under its pixels lie in LDS (as in conv_imgk), the 3x3
// result and the block output stay there as operands of the next layer, and only tensors that others read are written.
// The price: every workgroup streams all 17 C^2 bytes of weights (about 60 bytes per clock and CU), so the kernel
// pays where that stream, TM pixels at a time, is cheaper than two launches and the round trips of the tensors between.
//
// In the first block of a stage the residual is a 1x1 layer's result, the projection of the block's input.  It has no other reader, so the launch
// computes it too, ahead of the 3x3 layer, into the place where the residual would be fetched to: 4 PJ C^2 more bytes of weights a
// workgroup for one launch and the round trip of its tensor.  ResNet-50, us of a forward, apart / together: one image 176.2 / 173.0, 16 288 / 273, 40
// 413 / 389, 64 592 / 569, 128 1027 / 1011; each of the three stages by itself ahead or level at 1 to 192 images of 224 and 128 pixels.
//
// A wave owns one block of 32 channels of the 3x3 layer, four of the closing one and NA / C of the last, over MBW blocks
// of 32 pixels.  Its weights lie in memory as one stream of 1 KiB fragments in the order of use and go straight into
// registers, R fragments ahead; the whole sequence is unrolled, so ring slots are registers.
#include "bottleneck.h"

#include "f8_host.h"

namespace f8 {

namespace {

typedef int v16i __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) uint8_t lds_u8;
typedef __attribute__((address_space(3))) v4i lds_v4i;

struct BnTiling {
  int M, tiles;
  int x_bytes;
  int patch_w;              // W + 2
  FastDiv fd_pq, fd_q;      // pixel -> image, row
  FastDiv fd_h2;            // by H + 2: padded row -> image
  FastDiv fd_kpr;           // by 1 KiB loads per image row
  uint32_t res_xor;         // makes the residual signed
  int res_bytes;            // 0: no residual
  ScaledClip clip_b, clip_c, clip_2, clip_a, clip_p;
  int xp_bytes;             // the projection's input
};

// Start values of the three layers, with a projection its own behind them, in whole KiB behind the weights.
constexpr int start_bytes(int C, bool projection) { return ((projection ? 11 : 7) * C * 4 + 1023) / 1024 * 1024; }

// LDS: [block output TM x 4 C][start values][projection's input TM x PJ C][3x3 result TM x (C + 16)][patch rows].  Where that leaves room for one
// workgroup per CU only, the 3x3 result takes the place of the patch, one barrier more.
template <int C, int TM, int PJ>
struct BnLds {
  static constexpr int Y = 0;
  static constexpr int ACC = TM * 4 * C;
  static constexpr int XP = ACC + start_bytes(C, PJ != 0);
  static constexpr int BT = XP + TM * PJ * C;
  static constexpr int PITCH = C + 16;
  static constexpr bool SHARED = C == 64 && TM == 128;
  static constexpr int PATCH = SHARED ? BT : BT + TM * PITCH;
};

__device__ __forceinline__ v4i lds_read(uint32_t at) { return *(lds_v4i *)(uintptr_t)at; }
__device__ __forceinline__ void lds_write(uint32_t at, v4i v) { *(lds_v4i *)(uintptr_t)at = v; }

// Blocks of channels of the closing layer that a wave works on side by side.
constexpr int BB = 2;

// 16 accumulators of a lane, already holding the rounding addend, to 16 bytes.
__device__ __forceinline__ v4i requant16(const v16i &a, int lo, int hi, int shift) {
  int v[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = clamp_med3(a[i], lo, hi);
  return shift_pack16(v, shift);
}

// PJ: channels of the projection's input / C (0: no projection, the residual is read).
template <int C, int TM, int MW, int R, int NAB, bool DUAL, int PJ>
__global__ __launch_bounds__(C / 32 * MW * 64, 2) void bottleneck_kernel(const BottleneckParams p, const BnTiling tl) {
  using L = BnLds<C, TM, PJ>;
  constexpr int START = start_bytes(C, PJ != 0);
  constexpr int NWN = C / 32, NT = NWN * MW * 64;
  constexpr int KS = C / 32, MBW = TM / 32 / MW;
  constexpr int PP = C / 16, YP = 4 * C / 16;           // 16-byte pieces per pixel of x, of y
  constexpr int F0 = 4 * PJ * KS, F1 = F0 + 9 * KS, F2 = 4 * KS, F3 = NAB * 4 * KS, FT = F1 + F2 + F3;
  constexpr int NWV = NT / 64, UNITS = 8;               // loads of the patch a wave has in flight
  pin_args(tl.tiles, tl.M, tl.x_bytes, tl.patch_w, tl.fd_pq.mul, tl.fd_pq.shr, tl.fd_pq.d, tl.fd_q.mul, tl.fd_q.shr, tl.fd_q.d, tl.fd_h2.mul,
           tl.fd_h2.shr, tl.fd_h2.d, tl.fd_kpr.mul, tl.fd_kpr.shr, tl.fd_kpr.d, p.x, p.wf, p.res, p.H, p.W, p.stride, p.x_xor);
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  const uint32_t base = (uint32_t)(uintptr_t)((lds_u8 *)lds);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nw = wave % NWN, mw = wave / NWN;
  const int l32 = lane & 31, half = lane >> 5;
  const int m0 = (int)xcd_remap(blockIdx.x, (uint32_t)tl.tiles) * TM;

  // ---- weights: this wave's stream of fragments
  const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<int8_t *>(p.wf) + (size_t)nw * (FT * 1024), 0, FT * 1024, 0x00027000);
  const __amdgpu_buffer_rsrc_t sres = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<int8_t *>(p.wf) + (size_t)NWN * (FT * 1024), 0, START, 0x00027000);
  v4i ring[R];
  auto load_w = [&](int i) {
    return __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(wres, lane * 16, i * 1024, 0));
  };

#pragma unroll
  for (int i = 0; i < R; ++i) ring[i] = load_w(i);
  __builtin_amdgcn_sched_barrier(0);

  // ---- patch: padded rows pr0 .. of the padded images (H + 2 rows each), one behind the other
  auto top_row = [&](int m, int &ow) {       // first padded row and column of pixel m's window
    const uint32_t b = tl.fd_pq.div((uint32_t)m), rem = (uint32_t)m - b * tl.fd_pq.d;
    const uint32_t oh = tl.fd_q.div(rem);
    ow = (int)(rem - oh * tl.fd_q.d) * p.stride;
    return (int)b * (p.H + 2) + (int)oh * p.stride;
  };
  int unused;
  const int pr0 = __builtin_amdgcn_readfirstlane(top_row(m0, unused));
  const int rows = __builtin_amdgcn_readfirstlane(top_row(min(m0 + TM, tl.M) - 1, unused)) + 3 - pr0;
  const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(p.x), 0, tl.x_bytes, 0x00027000);
  // A wave takes whole KiB of image rows, one a load; lane j works out where the wave's load j reads and writes.
  const int xm = (int)p.x_xor;
  const uint32_t lane_at = base + L::PATCH + L::PITCH + (lane / PP) * L::PITCH + (lane % PP) * 16;
  const int kpr = (int)tl.fd_kpr.d;
  uint32_t from, to;         // byte offset in x (beyond its end: zeros), in the patch
  int pieces;                // 16-byte pieces that lie in the row
  auto plan = [&](int j0) {
    const uint32_t u = (uint32_t)(wave + (j0 + lane) * NWV), row = tl.fd_kpr.div(u), k = u - row * kpr;
    const uint32_t pr = (uint32_t)pr0 + row, b = tl.fd_h2.div(pr);
    const int ih = (int)(pr - b * tl.fd_h2.d) - 1;
    from = (unsigned)ih < (unsigned)p.H ? ((b * p.H + ih) * p.W) * C + k * 1024u : 0x80000000u;
    to = (row * tl.patch_w + k * (64 / PP)) * L::PITCH;
    pieces = (int)row < rows ? p.W * PP - (int)k * 64 : 0;
  };
  v4i piece[UNITS];
  auto fetch = [&]() {
#pragma unroll
    for (int j = 0; j < UNITS; ++j)
      piece[j] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(xres, __builtin_amdgcn_readlane(from, j) + lane * 16, 0, 0));
  };
  auto put = [&]() {
#pragma unroll
    for (int j = 0; j < UNITS; ++j) {
      const uint32_t at = lane_at + __builtin_amdgcn_readlane(to, j);
      if (lane < __builtin_amdgcn_readlane(pieces, j)) lds_write(at, v4i{piece[j].x ^ xm, piece[j].y ^ xm, piece[j].z ^ xm, piece[j].w ^ xm});
    }
  };
  plan(0);
  fetch();
  __builtin_amdgcn_sched_barrier(0);
  // ---- start values; residual rows (or zeros) into the place of the block output, 16-byte pieces permuted by the row number
#pragma unroll
  for (int k = 0; k < (START / 1024 + NWV - 1) / NWV; ++k) {
    const int i = wave + k * NWV;
    if (i < START / 1024)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(sres, (lds_void *)(lds + L::ACC + i * 1024), 16, lane * 16, i * 1024, 0, 0);
  }
  constexpr int CI = PJ * C, CIP = PJ == 0 ? 1 : CI / 16;       // the projection's input: bytes and 16-byte pieces of a pixel
  // a row's pieces are permuted so that eight rows' pieces share no bank
  auto perm = [](int row) { return CI >= 256 ? row & 15 : (row / (CI == 0 ? 1 : 256 / CI)) & (CIP - 1); };
  if constexpr (PJ != 0) {
    const __amdgpu_buffer_rsrc_t pres = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(p.xp), 0, tl.xp_bytes, 0x00027000);
#pragma unroll
    for (int k = 0; k < TM * CIP / NT; ++k) {
      const int u = (wave + k * NWV) * 64 + lane, row = u / CIP, ph = u % CIP, m = m0 + row;
      const uint32_t b = tl.fd_pq.div((uint32_t)m), rem = (uint32_t)m - b * tl.fd_pq.d, oh = tl.fd_q.div(rem), ow = rem - oh * tl.fd_q.d;
      const uint32_t off = (((b * p.Hp + oh * p.sp) * p.Wp + ow * p.sp) * CI) + (uint32_t)((ph ^ perm(row)) * 16);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(pres, (lds_void *)(lds + L::XP + (wave + k * NWV) * 1024), 16, m < tl.M ? off : 0x80000000u, 0, 0, 0);
    }
  } else {
    const __amdgpu_buffer_rsrc_t rres = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(p.res), 0, tl.res_bytes, 0x00027000);
#pragma unroll
    for (int k = 0; k < TM * YP / NT; ++k) {
      const int u = (wave + k * NWV) * 64 + lane, row = u / YP, ph = u % YP;
      const uint32_t off = (uint32_t)(m0 + row) * (4 * C) + (uint32_t)((ph ^ (row & 15)) * 16);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rres, (lds_void *)(lds + L::Y + (wave + k * NWV) * 1024), 16, off, 0, 0, 0);
    }
  }
  // ---- the border columns of the patch
  for (int i = tid; i < rows * 2 * PP; i += NT) {
    const int row = i / (2 * PP), side = (i / PP) & 1;
    lds_write(base + L::PATCH + (row * tl.patch_w + (side ? tl.patch_w - 1 : 0)) * L::PITCH + (i % PP) * 16, v4i{xm, xm, xm, xm});
  }
  // ---- this lane's pixels
  uint32_t win[MBW];
#pragma unroll
  for (int mb = 0; mb < MBW; ++mb) {
    int ow;
    const int pr = top_row(min(m0 + (mw * MBW + mb) * 32 + l32, tl.M - 1), ow);
    win[mb] = base + L::PATCH + ((pr - pr0) * tl.patch_w + ow) * L::PITCH + half * 16;
  }
  put();
  for (int j0 = UNITS; wave + j0 * NWV < rows * kpr; j0 += UNITS) {
    plan(j0);
    fetch();
    put();
  }
  // the start values and the residual must have arrived too (the ring's first fragments were requested before them)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();

  // Accumulators of block nb of a layer start at its folded values.
  auto start16 = [&](int first) {
    v16i a;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const v4i s = lds_read(base + L::ACC + (first + half * 16 + g * 4) * 4);
#pragma unroll
      for (int i = 0; i < 4; ++i) a[4 * g + i] = s[i];
    }
    return a;
  };

  // where a lane's 16 channels of block b of the closing layer lie: the shortcut before it, the block output after it
  auto own = [&](int b, int mb) {
    const int row = (mw * MBW + mb) * 32 + l32;
    return base + L::Y + row * (4 * C) + (((nw * 8 + b * 2 + half) ^ (row & 15)) * 16);
  };
  // ---- the projection: its result takes the place of the residual
  if constexpr (PJ != 0) {
    constexpr int KP = PJ * KS, G = KP < 4 ? KP : 4;      // fragments are read a group of four slices ahead
    const int px = (int)p.xp_xor;
#pragma unroll
    for (int b0 = 0; b0 < 4; b0 += BB) {
      v16i acc[BB][MBW];
      v4i xf[2][G][MBW];
      auto read_group = [&](int g, v4i (&f)[G][MBW]) {
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
          for (int t = 0; t < G; ++t) {
            const int row = (mw * MBW + mb) * 32 + l32;
            f[t][mb] = lds_read(base + L::XP + row * CI + (((g * G + t) * 2 + half) ^ perm(row)) * 16);
          }
      };
#pragma unroll
      for (int b = 0; b < BB; ++b)
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb) acc[b][mb] = start16(7 * C + nw * 128 + (b0 + b) * 32);
      read_group(0, xf[0]);
#pragma unroll
      for (int g = 0; g < KP / G; ++g) {
        __builtin_amdgcn_sched_barrier(0);
        if (g + 1 < KP / G) read_group(g + 1, xf[(g + 1) & 1]);
#pragma unroll
        for (int t = 0; t < G; ++t) {
#pragma unroll
          for (int mb = 0; mb < MBW; ++mb) {
            v4i &x = xf[g & 1][t][mb];
            x.x ^= px; x.y ^= px; x.z ^= px; x.w ^= px;
          }
#pragma unroll
          for (int b = 0; b < BB; ++b) {
            const int i = b0 * KP + (g * G + t) * BB + b;
#pragma unroll
            for (int mb = 0; mb < MBW; ++mb)
              acc[b][mb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ring[i % R], xf[g & 1][t][mb], acc[b][mb], 0, 0, 0);
            if (i + R < FT) ring[i % R] = load_w(i + R);
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int b = 0; b < BB; ++b)
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb) {
          settle_matrix_result(acc[b][mb]);
          lds_write(own(b0 + b, mb), requant16(acc[b][mb], tl.clip_p.lo, tl.clip_p.hi, p.shift_p));
        }
    }
    __builtin_amdgcn_sched_barrier(0);
  }

  // ---- 3x3 layer: a tap's fragments are read while the previous tap's are multiplied
  {
    // (a matrix instruction waits 64 cycles for the result of the one before it, half of them idle: two sums where a
    // wave has one block of pixels)
    constexpr int CH = MBW == 1 ? 2 : 1;
    v16i acc[CH][MBW];
#pragma unroll
    for (int mb = 0; mb < MBW; ++mb) {
      acc[0][mb] = start16(nw * 32);
      if (CH == 2)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[CH - 1][mb][i] = 0;
    }
    v4i xf[2][KS][MBW];
    auto read_tap = [&](int tap, v4i (&f)[KS][MBW]) {
      const uint32_t off = (uint32_t)(((tap / 3) * tl.patch_w + tap % 3) * L::PITCH);
#pragma unroll
      for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
        for (int s = 0; s < KS; ++s) f[s][mb] = lds_read(win[mb] + off + s * 32);
    };
    read_tap(0, xf[0]);
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      __builtin_amdgcn_sched_barrier(0);
      if (tap < 8) read_tap(tap + 1, xf[(tap + 1) & 1]);
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const int i = F0 + tap * KS + s;
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb)
          acc[i % CH][mb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ring[i % R], xf[tap & 1][s][mb], acc[i % CH][mb], 0, 0, 0);
        if (i + R < FT) ring[i % R] = load_w(i + R);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    const ScaledClip cl = tl.clip_b;
    const int bx = (int)p.b_xor;
    if (L::SHARED) __syncthreads();
#pragma unroll
    for (int mb = 0; mb < MBW; ++mb) {
      if (CH == 2)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[0][mb][i] += acc[CH - 1][mb][i];
      settle_matrix_result(acc[0][mb]);
      v4i v = requant16(acc[0][mb], cl.lo, cl.hi, p.shift_b);
      v.x ^= bx; v.y ^= bx; v.z ^= bx; v.w ^= bx;
      lds_write(base + L::BT + ((mw * MBW + mb) * 32 + l32) * L::PITCH + nw * 32 + half * 16, v);
    }
  }
  __syncthreads();

  // ---- closing layer: four blocks of channels
  v4i second[DUAL ? 4 : 1][MBW];
  {
    v4i xf[KS][MBW];
#pragma unroll
    for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
      for (int s = 0; s < KS; ++s)
        xf[s][mb] = lds_read(base + L::BT + ((mw * MBW + mb) * 32 + l32) * L::PITCH + s * 32 + half * 16);
    const ScaledClip cl = tl.clip_c, cl2 = tl.clip_2;
    const int yx = (int)p.y_xor, rx = (int)tl.res_xor;
#pragma unroll
    for (int b0 = 0; b0 < 4; b0 += BB) {
      v16i acc[BB][MBW];
      v4i r[BB][MBW];
#pragma unroll
      for (int b = 0; b < BB; ++b)
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb) acc[b][mb] = start16(C + nw * 128 + (b0 + b) * 32);
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int b = 0; b < BB; ++b) {
          const int i = F1 + b0 * KS + s * BB + b;
#pragma unroll
          for (int mb = 0; mb < MBW; ++mb)
            acc[b][mb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ring[i % R], xf[s][mb], acc[b][mb], 0, 0, 0);
          if (i + R < FT) ring[i % R] = load_w(i + R);
        }
#pragma unroll
      for (int b = 0; b < BB; ++b)
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb) r[b][mb] = lds_read(own(b0 + b, mb));
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int b = 0; b < BB; ++b)
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb) {
          v16i &a = acc[b][mb];
          settle_matrix_result(a);
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int v = (int)((uint32_t)(r[b][mb][i >> 2] ^ rx) << (24 - 8 * (i & 3))) >> 24;
            a[i] += v << p.res_d;
          }
          if (DUAL) {
            v16i a2;
#pragma unroll
            for (int i = 0; i < 16; ++i) a2[i] = a[i] + p.add_2;
            second[b0 + b][mb] = requant16(a2, cl2.lo, cl2.hi, p.shift_2);
          }
          v4i v = requant16(a, cl.lo, cl.hi, p.shift_c);
          v.x ^= yx; v.y ^= yx; v.z ^= yx; v.w ^= yx;
          lds_write(own(b0 + b, mb), v);
        }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  __syncthreads();

  // ---- the layer behind: K = 4 C, operand the block output (in signed form)
  if constexpr (NAB > 0) {
    constexpr int CH = NAB * MBW == 1 ? 2 : 1;
    v16i acc[NAB * CH][MBW];
#pragma unroll
    for (int j = 0; j < NAB; ++j)
#pragma unroll
      for (int mb = 0; mb < MBW; ++mb) {
        acc[j][mb] = start16(5 * C + (nw * NAB + j) * 32);
        if (CH == 2)
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[NAB * CH - 1][mb][i] = 0;
      }
    constexpr int G = 4, NG = 4 * KS / G;               // fragments are read a group of four slices ahead
    v4i xf[2][G][MBW];
    uint32_t yrow[MBW];
#pragma unroll
    for (int mb = 0; mb < MBW; ++mb) {
      const int row = (mw * MBW + mb) * 32 + l32;
      yrow[mb] = base + L::Y + row * (4 * C) + ((half ^ (row & 15)) * 16);
    }
    auto read_group = [&](int g, v4i (&f)[G][MBW]) {
#pragma unroll
      for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
        for (int t = 0; t < G; ++t) f[t][mb] = lds_read(yrow[mb] ^ (uint32_t)((g * G + t) * 32));
    };
    read_group(0, xf[0]);
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      __builtin_amdgcn_sched_barrier(0);
      if (g + 1 < NG) read_group(g + 1, xf[(g + 1) & 1]);
#pragma unroll
      for (int t = 0; t < G; ++t)
#pragma unroll
        for (int j = 0; j < NAB; ++j) {
          const int i = F1 + F2 + (g * G + t) * NAB + j;
#pragma unroll
          for (int mb = 0; mb < MBW; ++mb)
            acc[CH == 2 ? t % 2 : j][mb] =
                __builtin_amdgcn_mfma_i32_32x32x32_i8(ring[i % R], xf[g & 1][t][mb], acc[CH == 2 ? t % 2 : j][mb], 0, 0, 0);
          if (i + R < FT) ring[i % R] = load_w(i + R);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    const ScaledClip cl = tl.clip_a;
    const __amdgpu_buffer_rsrc_t ares = __builtin_amdgcn_make_buffer_rsrc(p.ya, 0, tl.M * (NAB * C), 0x00027000);
#pragma unroll
    for (int j = 0; j < NAB; ++j)
#pragma unroll
      for (int mb = 0; mb < MBW; ++mb) {
        if (CH == 2)
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[0][mb][i] += acc[NAB * CH - 1][mb][i];
        settle_matrix_result(acc[j][mb]);
        const v4i v = requant16(acc[j][mb], cl.lo, cl.hi, p.shift_a);
        const uint32_t off = (uint32_t)(m0 + (mw * MBW + mb) * 32 + l32) * (NAB * C) + (uint32_t)((nw * NAB + j) * 32 + half * 16);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(__attribute__((ext_vector_type(4))) unsigned, v), ares, off, 0, 0);
      }
  }
  // ---- block output: whole rows out of LDS; the second format from the registers
  {
    const __amdgpu_buffer_rsrc_t yres = __builtin_amdgcn_make_buffer_rsrc(p.y, 0, tl.M * (4 * C), 0x00027000);
    const int yx = (int)p.y_xor;
#pragma unroll
    for (int k = 0; k < TM * YP / NT; ++k) {
      const int u = tid + k * NT, row = u / YP, ph = u % YP;
      v4i v = lds_read(base + L::Y + u * 16);
      v.x ^= yx; v.y ^= yx; v.z ^= yx; v.w ^= yx;
      const uint32_t off = (uint32_t)(m0 + row) * (4 * C) + (uint32_t)((ph ^ (row & 15)) * 16);
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(__attribute__((ext_vector_type(4))) unsigned, v), yres, off, 0, 0);
    }
    if constexpr (DUAL) {
      const __amdgpu_buffer_rsrc_t y2res = __builtin_amdgcn_make_buffer_rsrc(p.y2, 0, tl.M * (4 * C), 0x00027000);
#pragma unroll
      for (int blk = 0; blk < 4; ++blk)
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb) {
          const uint32_t off = (uint32_t)(m0 + (mw * MBW + mb) * 32 + l32) * (4 * C) + (uint32_t)(nw * 128 + blk * 32 + half * 16);
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(__attribute__((ext_vector_type(4))) unsigned, second[blk][mb]), y2res, off, 0, 0);
        }
    }
  }
}

// Piece i (16 bytes) of the stream: wave nw's fragments, four blocks of pj KS of the projection (BB blocks side by side), 9 KS of the 3x3 layer (tap by tap), four blocks of KS of the
// closing layer (BB blocks side by side), then slice by slice NAB blocks of the layer behind; behind all waves' fragments
// the start values.
__global__ __launch_bounds__(256) void bottleneck_weights_kernel(const int8_t *__restrict__ wb, const int8_t *__restrict__ wc,
                                                                 const int8_t *__restrict__ wa, const int8_t *__restrict__ wp, int8_t *__restrict__ wf, int C, int nab, int pj) {
  const int ks = C / 32, ft = (13 + 4 * nab + 4 * pj) * ks;
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= ks * ft * 64) return;
  const int lane = i & 63, f = (i >> 6) % ft - 4 * pj * ks, nw = (i >> 6) / ft;
  const int row = weight_row(lane & 31), half = lane >> 5;
  const int8_t *src;
  if (f < 0) {
    const int kp = pj * ks, g = f + 4 * kp, first = g / (BB * kp) * BB, h = g % (BB * kp);
    src = wp + (size_t)(nw * 128 + (first + h % BB) * 32 + row) * (pj * C) + h / BB * 32;
  } else if (f < 9 * ks) {
    src = wb + ((size_t)(nw * 32 + row) * 9 + f / ks) * C + f % ks * 32;
  } else if (f < 13 * ks) {
    const int g = f - 9 * ks;
    const int first = g / (BB * ks) * BB, h = g % (BB * ks);
    src = wc + (size_t)(nw * 128 + (first + h % BB) * 32 + row) * C + h / BB * 32;
  } else {
    const int g = f - 13 * ks;
    src = wa + (size_t)((nw * nab + g % nab) * 32 + row) * (4 * C) + g / nab * 32;
  }
  *reinterpret_cast<v4i *>(wf + (size_t)i * 16) = *reinterpret_cast<const v4i *>(src + half * 16);
}

// The start values: the closing layer's with what makes an unsigned residual signed, 128 at the residual's scale.
__global__ __launch_bounds__(256) void bottleneck_start_kernel(const int32_t *__restrict__ b, const int32_t *__restrict__ c,
                                                               const int32_t *__restrict__ a, const int32_t *__restrict__ pr, int32_t *__restrict__ to, int C, int NA, int res_bias) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < C) to[i] = b[i];
  else if (i < 5 * C) to[i] = c[i - C] + res_bias;
  else if (i < 7 * C) to[i] = i - 5 * C < NA ? a[i - 5 * C] : 0;
  else if (i < 11 * C && pr) to[i] = pr[i - 7 * C];
}

// Patch rows a tile of TM pixels can need: its output rows, and two border rows per image boundary inside it.
int most_rows(int P, int Q, int stride, int H, int TM) {
  const int out_rows = (TM - 2) / Q + 2, crossings = (TM - 2) / (P * Q) + 1;
  return (out_rows - 1) * stride + 3 + crossings * (H + 2 - stride * P > 0 ? H + 2 - stride * P : 0);
}

template <int C, int TM, int PJ = 0>
int lds_bytes(const BottleneckParams &p) {
  using L = BnLds<C, TM, PJ>;
  const int patch = most_rows(p.P, p.Q, p.stride, p.H, TM) * (p.W + 2) * L::PITCH;
  return L::PATCH + (L::SHARED && patch < TM * L::PITCH ? TM * L::PITCH : patch);
}

constexpr int LDS_MOST = 160 * 1024;

template <int C, int TM, int MW, int R, int NAB, bool DUAL, int PJ = 0>
int launch_one(const BottleneckParams &p, hipStream_t stream) {
  const int smem = lds_bytes<C, TM, PJ>(p);
  if (smem > LDS_MOST) return (int)hipErrorInvalidValue;
  BnTiling tl;
  tl.M = p.B * p.P * p.Q;
  tl.tiles = (tl.M + TM - 1) / TM;
  tl.x_bytes = p.B * p.H * p.W * C;
  tl.patch_w = p.W + 2;
  tl.fd_pq = FastDiv((uint32_t)(p.P * p.Q));
  tl.fd_q = FastDiv((uint32_t)p.Q);
  tl.fd_h2 = FastDiv((uint32_t)(p.H + 2));
  tl.fd_kpr = FastDiv((uint32_t)((p.W * C + 1023) / 1024));
  tl.res_xor = (p.res || PJ != 0) && !p.res_signed ? 0x80808080u : 0u;
  tl.res_bytes = p.res ? tl.M * 4 * C : 0;
  tl.clip_b = scaled_clip(p.lo_b, p.hi_b, p.shift_b);
  tl.clip_c = scaled_clip(p.lo_c, p.hi_c, p.shift_c);
  tl.clip_2 = scaled_clip(p.lo_2, p.hi_2, p.shift_2);
  tl.clip_a = scaled_clip(p.lo_a, p.hi_a, p.shift_a);
  tl.clip_p = scaled_clip(p.lo_p, p.hi_p, p.shift_p);
  tl.xp_bytes = p.B * p.Hp * p.Wp * PJ * C;
  auto k = bottleneck_kernel<C, TM, MW, R, NAB, DUAL, PJ>;
  static std::atomic<unsigned long long> done_mask{0};          // devices whose LDS limit has been raised
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return (int)hipErrorInvalidDevice;
  if (dev < 0 || dev > 63 || !((done_mask.load(std::memory_order_relaxed) >> dev) & 1ull)) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, LDS_MOST);
    if (e != hipSuccess) return (int)e;
    if (dev >= 0 && dev <= 63) done_mask.fetch_or(1ull << dev, std::memory_order_relaxed);
  }
  hipLaunchKernelGGL(k, dim3((unsigned)tl.tiles), dim3(C / 32 * MW * 64), smem, stream, p, tl);
  return (int)hipGetLastError();
}

template <int C, int TM, int MW, int R>
int launch_shape(const BottleneckParams &p, hipStream_t stream) {
  const bool dual = p.y2 != nullptr;
  // (a projection's input has C channels in the first stage, 2 C behind it)
  constexpr int PJ = C == 64 ? 1 : 2;
  if (p.xp) return dual ? launch_one<C, TM, MW, R, 1, true, PJ>(p, stream) : launch_one<C, TM, MW, R, 1, false, PJ>(p, stream);
  if (p.NA == 0) return dual ? launch_one<C, TM, MW, R, 0, true>(p, stream) : launch_one<C, TM, MW, R, 0, false>(p, stream);
  if (p.NA == C) return dual ? launch_one<C, TM, MW, R, 1, true>(p, stream) : launch_one<C, TM, MW, R, 1, false>(p, stream);
  return dual ? launch_one<C, TM, MW, R, 2, true>(p, stream) : launch_one<C, TM, MW, R, 2, false>(p, stream);
}

}  // namespace

static BottleneckParams geometry(int H, int W, int stride) {
  BottleneckParams p;
  p.H = H; p.W = W; p.stride = stride;
  p.P = (H + 2 - 3) / stride + 1; p.Q = (W + 2 - 3) / stride + 1;
  return p;
}

bool bottleneck_applicable(int C, int H, int W, int stride, int NA, int shift_b, int shift_c, int shift_a, int shift_2, int res_d) {
  if ((C != 64 && C != 128 && C != 256) || (NA != 0 && NA != C && NA != 2 * C) || (stride != 1 && stride != 2)) return false;
  if (H < 1 || W < 1 || H > 4096 || W > 4096 || shift_b < 0 || shift_c < 0 || shift_a < 0 || shift_2 < 0 || res_d < 0 || res_d > 16) return false;
  const BottleneckParams p = geometry(H, W, stride);
  return (C == 64 ? lds_bytes<64, 64>(p) : C == 128 ? lds_bytes<128, 32>(p) : lds_bytes<256, 32>(p)) <= LDS_MOST;
}

bool bottleneck_projects(int C, int H, int W, int stride, int NA, int PC, int ps) {
  if (C != 64 && C != 128 && C != 256) return false;
  if (NA != C || PC != (C == 64 ? C : 2 * C) || (ps != 1 && ps != 2) || H < 1 || W < 1 || H > 4096 || W > 4096) return false;
  const BottleneckParams p = geometry(H, W, stride);
  return (C == 64 ? lds_bytes<64, 64, 1>(p) : C == 128 ? lds_bytes<128, 32, 2>(p) : lds_bytes<256, 32, 2>(p)) <= LDS_MOST;
}

// Twice the pixels per workgroup halve the weight stream and spread a tile's set-up over more pixels, but leave
// CUs idle where there are few.  us, narrow / wide tiles, first and second stride-1 block of a stage, ResNet-50:
//   64 channels, 56 x 56: batch 8 10.0 / 10.4, 12 12.2 / 11.3, 16 14.8 / 13.4, 32 22.9 / 22.9, 64 38.8 / 36.0, 128 69 / 59
//   128 channels, 28 x 28: batch 4 7.3 / 8.2, 8 7.5 / 9.4, 12 11.1 / 10.0, 16 11.6 / 9.5, 32 19.5 / 14.8, 128 53 / 44;
//     stride 2: batch 8 8.2 / 10.1, 12 14.1 / 10.1, 32 25.3 / 20.0
//   256 channels, 14 x 14, where the stream is everything: one narrow tile per CU as long as there are no more (batch 16 14.3 / 17.0,
//     32, 196 tiles, 15.0 / 17.8), wide ones beyond (48, 294 tiles, 24.6 / 19.5, 64 27.2 / 22.1, 128 52.6 / 40.8)
bool bottleneck_wide(int C, int H, int W, int stride, int B, int force, bool projection) {
  const BottleneckParams p = geometry(H, W, stride);
  const int lds = projection ? (C == 64 ? lds_bytes<64, 128, 1>(p) : C == 128 ? lds_bytes<128, 64, 2>(p) : lds_bytes<256, 64, 2>(p))
                             : C == 64 ? lds_bytes<64, 128>(p) : C == 128 ? lds_bytes<128, 64>(p) : lds_bytes<256, 64>(p);
  if (lds > LDS_MOST || force == 3) return false;
  const long long M = (long long)B * p.P * p.Q;
  return force == 4 || M > (C == 64 ? 32768 : 8192);
}

static size_t fragment_bytes(int C, int NA, int PC) { return (size_t)C * (13 * C + 4 * NA + 4 * PC); }
size_t bottleneck_weight_bytes(int C, int NA, int PC) { return fragment_bytes(C, NA, PC) + start_bytes(C, PC != 0); }

int launch_bottleneck_weights(const int8_t *wb, const int8_t *wc, const int8_t *wa, const int8_t *wp, const int32_t *acc_b, const int32_t *acc_c,
                              const int32_t *acc_a, const int32_t *acc_p, int8_t *wf, int C, int NA, int PC, int res_bias, hipStream_t stream) {
  if (!wb || !wc || !acc_b || !acc_c || (NA && (!wa || !acc_a)) || (PC && (!wp || !acc_p)) || !wf ||
      ((reinterpret_cast<uintptr_t>(wb) | reinterpret_cast<uintptr_t>(wc) | reinterpret_cast<uintptr_t>(wa) | reinterpret_cast<uintptr_t>(wp) |
        reinterpret_cast<uintptr_t>(wf)) & 15))
    return (int)hipErrorInvalidValue;
  const int pieces = (int)(fragment_bytes(C, NA, PC) / 16);
  hipLaunchKernelGGL(bottleneck_weights_kernel, dim3((pieces + 255) / 256), dim3(256), 0, stream, wb, wc, wa, wp, wf, C, NA / C, PC / C);
  hipLaunchKernelGGL(bottleneck_start_kernel, dim3((11 * C + 255) / 256), dim3(256), 0, stream, acc_b, acc_c, acc_a, PC ? acc_p : nullptr,
                     reinterpret_cast<int32_t *>(wf + fragment_bytes(C, NA, PC)), C, NA, res_bias);
  return (int)hipGetLastError();
}

int launch_bottleneck(const BottleneckParams &p, hipStream_t stream) {
  if (p.B <= 0) return 0;
  if (!bottleneck_applicable(p.C, p.H, p.W, p.stride, p.NA, p.shift_b, p.shift_c, p.NA ? p.shift_a : 0, p.y2 ? p.shift_2 : 0, p.res ? p.res_d : 0) ||
      ((reinterpret_cast<uintptr_t>(p.x) | reinterpret_cast<uintptr_t>(p.wf) | reinterpret_cast<uintptr_t>(p.res) |
        reinterpret_cast<uintptr_t>(p.y) | reinterpret_cast<uintptr_t>(p.y2) | reinterpret_cast<uintptr_t>(p.ya)) & 15) ||
      (long long)p.B * p.P * p.Q * 4 * p.C > 0x7fffffffLL || (long long)p.B * p.H * p.W * p.C > 0x7fffffffLL)
    return (int)hipErrorInvalidValue;
  if (p.xp && (!bottleneck_projects(p.C, p.H, p.W, p.stride, p.NA, p.PC, p.sp) || p.res || p.shift_p < 0 || p.res_d < 0 || p.res_d > 16 ||
               (reinterpret_cast<uintptr_t>(p.xp) & 15) || (p.Hp - 1) / p.sp + 1 != p.P || (p.Wp - 1) / p.sp + 1 != p.Q ||
               (long long)p.B * p.Hp * p.Wp * p.PC > 0x7fffffffLL))
    return (int)hipErrorInvalidValue;
  const bool wide = bottleneck_wide(p.C, p.H, p.W, p.stride, p.B, p.force, p.xp != nullptr);
  if (p.C == 64) return wide ? launch_shape<64, 128, 2, 18>(p, stream) : launch_shape<64, 64, 2, 18>(p, stream);
  if (p.C == 128) return wide ? launch_shape<128, 64, 1, 16>(p, stream) : launch_shape<128, 32, 1, 16>(p, stream);
  return wide ? launch_shape<256, 64, 1, 16>(p, stream) : launch_shape<256, 32, 1, 16>(p, stream);
}

}  // namespace f8
