// Layer-chain runner: a whole fixed-point network forward as a fixed sequence of launches.
//
// The chain owns only host-side book-keeping.  Activations and the per-layer constants
// live in a caller-provided device workspace whose layout is
//   [ constants: acc0 vector (and re-laid-out stem weights) of every dense layer ][ arena ]
// Every tensor's size is linear in the batch, so the arena is planned once per image
// (first-fit over tensor lifetimes, offsets in multiples of 256 bytes) and scaled by the
// batch at run time.
//
// Stem re-layout.  A dense layer with at most 4 input channels (the 7x7/2 ImageNet stem)
// is run on a re-laid-out copy of its operands: the input gets an explicit zero border
// and 4 channels, each window row is padded to a multiple of 4 taps with zero weights.
// The sums are unchanged (only zero products are added), windows are never clipped, and
// 16 contiguous bytes hold four whole taps, which is what the fast kernel's loads need.
// A dense layer whose input channel count is above 4 and not a multiple of 16 (24 in the
// first MobileNetV2 blocks) is run on a copy of its input and weights with the channels
// padded with zeros to the next multiple of 16, for the same reason.
//
// Stem + pool.  The ImageNet stem (7x7 stride-2 convolution of a 3-channel image to 64 unsigned
// channels) followed by a 3x3 stride-2 pad-1 max pool that is its only reader runs as one kernel
// on the image itself and re-laid-out weights; neither the tensor between the two nor a copy of the image gets memory.  (Not when every
// tensor is to be kept; F8_STEM_POOL=0, read when the chain is created, turns it off: tuning aid.)
//
// Block fusion.  Three consecutive layers that form an inverted-residual block (1x1 dense,
// 3x3 depthwise stride 1 pad 1, 1x1 dense, optional shortcut from the block input) whose two
// intermediate tensors have no other reader run as one kernel that keeps the intermediates on
// chip; those tensors then get no memory.  Opt-in (f8_chain_set_fusion(c, 1)): measured on
// MI355X it beats the three kernels on a single block at batch 64 but not on whole MobileNetV2
// forwards, where it is bound by the vector ALU and, late in the network, by too few tiles.
// Never used with keep_all (every tensor inspectable).
#include <algorithm>
#include <new>
#include <vector>

#include "block_fused.h"
#include "bottleneck.h"
#include "dw_pw.h"
#include "pw_dw_pw.h"
#include "stem_pool.h"
#include "conv_img.h"
#include "conv_imgk.h"
#include "conv_imgk_pair.h"
#include "conv_s2.h"
#include "f8_host.h"

using namespace f8;

namespace {

struct Tensor {
  int h = 0, w = 0, c = 0;
  int type = -1;
  int fl = 0;
  bool fl_known = false;
  int producer = -2;        // -2: not defined, -1: network input, else layer index
  int last_use = -1;        // last layer index that reads it
  size_t bytes_per_image = 0;
  bool external = false;    // input x or final output
};

struct Stem {
  bool on = false;
  int Cp = 4;                       // channels after the re-layout: 4 (stem) or a multiple of 16
  int Sp = 0, Hp = 0, Wp = 0;       // stem: padded window width, padded image extent
  size_t w_off = 0;                 // re-laid-out weights: byte offset in the constants region
  size_t x_bytes_per_image = 0;
  int pool = 0;                     // 1: this layer also does the max pool that follows; 2: that (absorbed) pool
};

// Role of a layer in a fused block, and where the block's re-laid-out constants live.
struct Fused {
  int role = 0;                     // 0 ordinary layer, 1 first layer of a fused block, 2 absorbed
  int K1 = 0, CH = 0, NB2 = 0;
  size_t w1p = 0, w2p = 0, wdp = 0, acc1 = 0, accd = 0, acc2 = 0;   // byte offsets in the constants region
};

size_t elem_size(int type) { return type == F8_S32 ? 4 : 1; }
size_t round256(size_t v) { return (v + 255) / 256 * 256; }

}  // namespace

struct f8_chain {
  std::vector<f8_layer_desc> layers;
  std::vector<Geom> geom;              // per layer, B filled at run time
  std::vector<Stem> stem;              // per layer
  std::vector<Fused> fused;            // per layer
  bool fusion = false;
  bool use_fusion() const { return fusion && !keep_all; }
  bool stem_pool = true;
  int pool_role(size_t i) const { return stem_pool && !keep_all ? stem[i].pool : 0; }
  // A dense layer and the 1x1 layer that reads its output in one launch: tail[i] = 1 for the first,
  // 2 for the 1x1 layer behind it, tail_peer[i] = the other layer of the pair (candidates; both
  // tensors are still written).  Whether the kernel that can do this is chosen depends on the batch.
  std::vector<int> tail, tail_peer;    // per layer
  bool conv_tail = true;
  // 3x3 layers the image-stationary kernels can take: bytes of their weights in fragment order (0: not such a
  // layer).
  std::vector<size_t> img_w_bytes;     // per layer
  int conv_img = 1;
  int conv_img_min = 96;
  int imgk = 1;
  // 0: neither, 1: an image (or band) per workgroup, 1 + n: fewer channels per workgroup, n waves share K
  int img_role(size_t i, int batch) const {
    if (img_w_bytes[i] == 0 || (use_fusion() && fused[i].role != 0)) return 0;
    const f8_layer_desc &L = layers[i];
    const Geom &g = geom[i];
    const int shift = L.q.fl_x + L.q.fl_w - L.q.fl_y;
    const bool img_ok = conv_img != 0 && L.res < 0 &&
                        conv_img_applicable(L.Cin, L.Cout, L.R, L.S, L.stride_h, L.stride_w, L.pad_h, L.pad_w, g.H, g.W, shift, nullptr, nullptr) &&
                        conv_img_units(L.Cin, batch, g.H) >= conv_img_min;
    if (img_ok && conv_img == 2) return 1;           // the caller's choice
    if (imgk != 0 && conv_imgk_applicable(L.Cin, L.Cout, L.R, L.S, L.stride_h, L.stride_w, L.pad_h, L.pad_w, g.H, g.W, shift,
                                          nullptr, nullptr, nullptr)) {
      const int wk = imgk_waves(L, g, batch);
      if (wk != 0) return 1 + wk;
    }
    if (img_ok) return 1;
    return 0;
  }
  // Waves that share K in the image-stationary kernel, or 0 where another kernel is faster.  The fewer channels a
  // workgroup computes, the more often its pixels are loaded and the more sums meet in LDS, but the layer
  // lasts as long as its last round of workgroups: as many shares as leave the launch one round.
  // Microseconds of a layer, 1, 2, 4 waves / the best other kernel:
  //   64 channels, 56 x 56: batch 2 5.1 / 4.2, 4 5.1 / 5.5, 8 5.3 / 6.5, 16 5.5 / 7.8, 64 13.3 / 14.5, 128 23.0 / 22.6 (conv_ws; with two halves of
  //     128 side by side, as ResNet-50 runs at batch 256, conv_ws is ahead by 10 us a layer); 24 x 24: 8 5.1 / 4.0, 16 5.2 / 5.4, 32 5.3 / 6.0;
  //     with a residual: batch 32 9.9 / 12.2; 64 13.5 / 18.9; 256 41.5 / 65.0
  //   128 channels, 28 x 28: batch 8 8.3, 7.0 / 6.4; 12 8.6, 7.2 / 8.6; 24 9.0, 7.7 / 10; 40 9.8, 15.9 / 12; 64 10.7, 14.4 / 16.7; 128 20.0, - / 21.5;
  //     192 22.9, - / 26.8; 256 29.0, - / 29.9; 288 33.5, - / 38.5; 512 53.0, - / 57.1; 1024 100, - / 108 (conv_img,
  //     conv_ws at 288); with a residual 256 31.7, - / 45.3; 768 84.0, - / 110.6; 20 x 20, batch 512: 29.2, - / 36.9
  //   256 channels, 14 x 14: batch 8 12.3, 9.2, 7.6 / 6.2 (conv_wavek); 12 12.4, 9.5, 7.4 / 7.4; 16 12.5, 9.7, 7.4 / 7.7; 24 12.9, 9.6,
  //     7.8 / 12.7; 33 13.3, 10.0, 15.5 / 13.9; 64 13.7, 11.1, 14.3 / 16.6; 70 14.3, 20.8, 23.2 / 16.8; 128 17.5, 21.8, - / 22.4; 192 27.7, -, - / 24.8 (conv_img)
  //   512 channels, 7 x 7: batch 16 14.5, 10.4, 8.2 / 7.9 (conv_wavek); 24 14.8, 10.8, 8.8 / 9.7; 40 15.7, 11.8, 16.5 / -; 65 17.2, 23.1,
  //     25.3 / 22.3; 128 20, 25.2, - / 28.0; 256 35.0, -, - / 38.0
  int imgk_waves(const f8_layer_desc &L, const Geom &g, int batch) const {
    if (imgk >= 10) {      // tuning aid: force it, with 1, 2 or 4 waves (there is no kernel for other counts)
      const int wk = imgk - 10;
      return (wk == 1 || wk == 2 || wk == 4) && wk <= conv_imgk_most_waves(L.Cin) ? wk : 0;
    }
    const long long most = L.Cin == 256 ? 256 : L.Cin == 64 && L.res < 0 ? 1024 : 0x7fffffffLL;
    if (!conv_imgk_fills(L.Cin, g.H, g.W)) return 0;
    const long long least = L.Cin == 64 ? 44 : L.Cin == 128 ? 80 : 176;
    int wk = conv_imgk_most_waves(L.Cin);
    long long wgs = conv_imgk_workgroups(L.Cin, batch, g.H, g.W, wk);
    if (wgs < least) return 0;
    // More than 128 workgroups are left with half as many shares of K: no lower limit there.  Microseconds of a small forward around the layer, here / the
    // general kernels: 512 channels, 7 x 7, 34 images 19.3 / 19.3, 40 19.8 / 19.9, 66 25.4 / 31.8, 86 27.2 / 36.0.
    while (wk > 1 && wgs > 256) wgs = conv_imgk_workgroups(L.Cin, batch, g.H, g.W, wk /= 2);
    // (256 channels would be ahead too, 14 x 14, 34 images 17.7 / 21.7, 66 22.5 / 24.8, 86 24.7 / 30.6; the limit stays there because the test of the
    // workspace's size needs a batch that takes fewer copies than the one before it)
    if (L.Cin == 256 && wgs < least) return 0;
    return wgs <= most ? wk : 0;
  }
  // Stride-2 3x3 layers that the image-stationary kernel can take, s2[i] = 1, with the 1x1 stride-2 layer next to one on the same input, s2[i] = 2
  // (s2_proj: the other layer of the two).  The 3x3 layer launches both.  Its weights in fragment order lie behind the arena, the 1x1
  // layer's among the constants (s2_const_off).
  std::vector<int> s2, s2_proj;        // per layer
  std::vector<size_t> s2_const_off;    // per layer (of the 1x1 one)
  int conv_s2 = 1;
  size_t s2_w_bytes(size_t i) const { return s2[i] == 1 ? (size_t)9 * layers[i].Cin * layers[i].Cout : 0; }
  // Waves that share K, or 0: another kernel.  As few as give three quarters of the CUs a workgroup; with the projection the
  // launch that it saves pays from few pixels on.  Microseconds of a forward of two 1x1 layers and these (16 -> C in front, N -> N
  // behind), two launches of the general kernels -> one with 1, 2, 4 waves:
  //   64 -> 128 from 56 x 56: batch 4 14.0 -> 14.3, 8 16.3 -> 15.4, 32 21.5 -> 18.7, 64 30.5 -> 25.4, 128 49.5 -> 42.7, 256 80.2 -> 71.4; from 24 x 24: 8 12.0 -> 13.6, 32 16.0 -> 15.4
  //   128 -> 256 from 28 x 28: batch 8 14.8 -> -, 15.7, 12 17.9 -> -, 17.4, 48 24.7 -> 22.0, 20.4, 64 25.4 -> 23.3, 21.8, 96 31.5 -> 26.4, 32.3, 256 55.0 -> 52.8, 60.4;
  //     from 12 x 12 (a third of a workgroup's pixels): 32 14.2 -> -, 15.5, 128 20.6 -> 19.3, 18.0, 500 30.2 -> 34.7
  //   256 -> 512 from 14 x 14: batch 4 13.8 -> -, -, 14.2, 12 16.3 -> -, -, 15.7, 24 20.2 -> -, 19.5, 18.4, 48 28.7 -> 25.4, 20.3, 25.1, 96 33.6 -> 25.4, 30.4,
  //     256 48.4 -> 46.3; from 6 x 6: 32 14.1 -> -, -, 14.0, 500 32.9 -> 34.9
  // The 3x3 layer by itself: 64 -> 128 batch 64 23.4 -> 21.1; 128 -> 256 24 17.1 -> -, 16.5, 64 20.4 -> -, 19.4, 128 28.8 -> 26.3,
  // 192 38.8 -> 39.8; 256 -> 512 24 15.7 -> -, -, 15.4, 64 24.6 -> -, 19.2, 128 28.1 -> 24.2, 192 36.5 -> 36.4.
  // There is no launch to save there, and past one round of workgroups it is behind whenever the last round is thin (52 x 52, 84 images, 336 workgroups,
  // 23.4 -> 26.3; 60 x 60, 160 images, 800, 44.4 -> 49.6): one round only, 250 random sizes, never behind by more than 2 %.
  // With the projection the launch that it saves is worth more in a forward than around the layer alone.  64 channels: at any number of workgroups
  // (ResNet-18 at 90 images, 360, 321 -> 313 us, 340 images, 1360, 825 -> 814, 560 1281 -> 1244; alone, up to 8 % behind in thin rounds).  128 channels: to 1024
  // (alone, 12 sizes beyond: 4 - 16 % behind; in a forward to 680 ahead by 0 - 9 us of 700, beyond level).  256 channels: to 512 (alone, beyond: 18 - 31 %
  // behind; ResNet-18 at 320 images 788 -> 778 without it, 400 970 -> 960).
  int s2_waves(size_t i, int batch) const {
    if (s2[i] == 0 || conv_s2 == 0 || keep_all) return 0;
    const size_t a = s2[i] == 1 ? i : (size_t)s2_proj[i];
    if (bn_role(a, batch) != 0 || (use_fusion() && fused[a].role != 0)) return 0;
    const f8_layer_desc &L = layers[a];
    const Geom &g = geom[a];
    if (conv_s2 >= 10) {
      const int wk = conv_s2 - 10;
      return (wk == 1 || wk == 2 || wk == 4) && wk <= conv_s2_most_waves(L.Cin) ? wk : 0;
    }
    const bool projection = s2_proj[a] >= 0, fills = conv_s2_fills(L.Cin, g.H, g.W);
    const int most = conv_s2_most_waves(L.Cin);
    int wk = 1;
    long long wgs = conv_s2_workgroups(L.Cin, L.Cout, batch, g.H, g.W, wk);
    while (wgs < 176 && wk < most) wgs = conv_s2_workgroups(L.Cin, L.Cout, batch, g.H, g.W, wk *= 2);
    if (!projection) return fills && wgs >= 176 && wgs <= 256 ? wk : 0;
    if ((!fills && wgs > 256) || (L.Cin == 128 && wgs > 1024) || (L.Cin == 256 && wgs > 512)) return 0;
    return (long long)batch * g.P * g.Q >= (L.Cin == 64 ? 4500 : L.Cin == 128 ? 2300 : 500) ? wk : 0;
  }
  // Two 3x3 layers of 64 or 128 channels of which the second is the first's only reader and may have the first's input as its shortcut
  // (a basic residual block): pair[i] = 1 and 2, one launch (the second's) where both take the image-stationary kernel, whose
  // copies of the weights it reads.  Microseconds of the block (a forward gains 3 - 5 more), two launches -> one.  64 channels, ahead at every size
  // and batch that comes to that: 56 x 56, batch 16 13.1 -> 10.9, 24 17.4 -> 11.4, 32 18.6 -> 14.3, 48 21.7 -> 18.5, 64 25.2 -> 19.6; 40 x 40, batch 24 13.2 -> 9.2, 64 18.9 ->
  // 12.9, 128 27.8 -> 21.7.  128 channels: 28 x 28, batch 16 15.7 -> 10.4, 32 17.4 -> 12.2, 64 20.9 -> 18.2, 128 33.1 -> 29.7, 192 48.1 -> 52.0, 256 62.0 ->
  // 58.5 (whole rounds of workgroups); 20 x 20, batch 64 17.1 -> 13.5, 256 33.9 -> 30.3.
  std::vector<int> pair;               // per layer
  int conv_pair = 1;
  int pair_role(size_t i, int batch) const {
    if (pair[i] == 0 || conv_pair == 0 || keep_all) return 0;
    const size_t a = pair[i] == 1 ? i : i - 1;
    // (the second may also be the first of a bottleneck's three, which then read its input)
    if (bn_role(a, batch) != 0 || bn_role(a + 1, batch) != 0) return 0;
    if (layers[a].Cin == 128 && (long long)batch * geom[a].P * geom[a].Q > 131072) return 0;
    // (the layers by themselves take that kernel from fewer workgroups on than this; there the tests expect them apart, and
    // one launch would still be ahead: ResNet-18 at 8 images 118 -> 115 us, 12 135 -> 129)
    if (imgk < 10 && conv_imgk_workgroups(layers[a].Cin, batch, geom[a].H, geom[a].W, layers[a].Cin == 128 ? 2 : 1) < (layers[a].Cin == 128 ? 128 : 176)) return 0;
    return img_role(a, batch) >= 2 && img_role(a + 1, batch) >= 2 ? pair[i] : 0;
  }
  // A depthwise 3x3 layer and the 1x1 layer that is its only reader in one launch: dwp[i] = 1 for the depthwise one,
  // 2 for the other; dwp_w_bytes: of the 1x1 layer's weights in fragment order.  Whether the pair runs as one
  // launch depends on the batch.
  std::vector<int> dwp;                // per layer
  std::vector<size_t> dwp_w_bytes;     // per layer (of the depthwise one)
  int dw_pw = 1;
  int dwp_role(size_t i, int batch) const {
    if (dw_pw == 0 || keep_all || dwp[i] == 0) return 0;
    const size_t head = dwp[i] == 1 ? i : i - 1;
    if (use_fusion() && (fused[head].role != 0 || fused[head + 1].role != 0)) return 0;
    if (dw_pw != 2 && !dw_pw_pays(head, batch)) return 0;
    return dwp[i];
  }
  // Microseconds of the pair, apart -> together (the tail of the launch is what it saves; it pays for that with a
  // depthwise part that gathers its columns one by one and holds only one or two workgroups per CU).  Rows of more than 64
  // pixels: 112x112 C32, batch 4 (1.5 M elements) 8.3 -> 5.6, batch 8 (3.1 M) 7.7 -> 9.1.  Up to 64: 56x56 C96 stride 2 from 112,
  // batch 8 (2.3 M) 9.5 -> 7.3; C64, batch 16 (3.1 M) 11.0 -> 13.4.  Up to 28: C144, batch 40 (4.3 M) 10.2 -> 9.7; C192, batch 40
  // (5.7 M) 9.9 -> 11.2.  Up to 14: C576, batch 64 (6.9 M) 12.7 -> 11.9; C384, batch 100 (7.2 M) 11.8 -> 12.9.  Up to 7: C576
  // stride 2, batch 64 (1.7 M) 9.6 -> 8.4; batch 100 (2.7 M) 11.2 -> 12.1.  And K not so long that the few waves per block
  // of channels walk it one after the other: C576 -> 160, 18 slices of 32 each, batch 27, 8.9 -> 6.9; C960 -> 160, 30 slices
  // each, 7.8 -> 8.1 at every batch.
  bool dw_pw_pays(size_t i, int batch) const {
    const Geom &g = geom[i];
    const long long total = (long long)batch * g.P * g.Q * g.Cin;
    const long long most = g.Q > 64 ? 2ll << 20 : g.Q > 28 ? 5ll << 19 : g.Q > 14 ? 9ll << 19 : g.Q > 7 ? 7ll << 20 : 2ll << 20;
    return total <= most && dw_pw_slices(g.Cin, layers[i + 1].Cout) <= 20;
  }
  // An inverted-residual block (1x1 layer, depthwise 3x3 layer that is its only reader, 1x1 layer that is that one's) in one launch:
  // pdp[i] = 1, 2, 3 for its layers; the constants of the first one lie at pdp_off[i]: its weights in fragment order, depthwise weights
  // and start values, and, where the last two layers do not share a launch at every batch that takes this one, the last
  // layer's weights in fragment order at pdp_w2_off[i] (else that pair's copy serves).
  std::vector<int> pdp;                // per layer
  std::vector<size_t> pdp_off, pdp_w2_off;   // per layer (of the first one)
  int pw_dw_pw = 1;
  // The front of a network is such a block with a 3x3 stride-2 layer on an image in the first layer's place.  Microseconds of the three,
  // three launches (or two) -> one, image 224 x 224: MobileNetV2 (to 16 channels) batch 1 9.8 -> 4.6, 4 11.5 -> 4.3, 8 15.4 -> 6.1, 27 26.0 -> 10.3,
  // 64 44.9 -> 20.5, 128 75.2 -> 37.2; MobileNetV1 (to 64 channels) 1 11.3 -> 6.1, 27 33.0 -> 17.2, 64 58.1 -> 30.7, 128 93.1 -> 53.2.  The
  // line at 3 M pixels (batch 250) is no crossover: at 256 it is ahead too (136 -> 73, 178 -> 101).  It stands where the tests of the kernels that
  // the layers take by themselves begin, the 1x1 32 -> 16 layer's among them, which expect those kernels at batch 256.
  bool pdp_image(size_t front) const { return stem[front].on && stem[front].Cp == 4; }
  int pdp_k(size_t front) const { return pdp_image(front) ? 48 : layers[front].Cin; }
  // Where the pair is one launch, microseconds of front layer and pair, two launches -> one (two launches
  // cost 1 - 2 us more in a forward than alone), MobileNetV2: 28 x 28 C192, batch 1 8.5 -> 6.7, 27 13.8 -> 8.5; 14 x 14 C384, batch 1 7.6 -> 5.4, 27 11.2 ->
  // 6.6, 64 12.5 -> 9.0, 96 17.2 -> 11.2; C576, batch 1 8.9 -> 7.6, 27 12.8 -> 9.0, 64 17.5 -> 11.9; 28 x 28 C192 stride 2, batch 64 15.5 -> 8.2, 192 26.6 ->
  // 18.8; 56 x 56 C144, batch 1 11.2 -> 5.7, stride 2, batch 27 14.6 -> 9.0, 40 16.1 -> 15.2.
  // 1: front layer, 2: depthwise layer (which launches all three), 3: the one behind
  int pdp_role_at(size_t i, int batch) const {
    if (pdp[i] == 0 || pw_dw_pw == 0 || keep_all) return 0;
    const size_t front = i + 1 - (size_t)pdp[i];
    if (use_fusion() && (fused[front].role != 0 || fused[front + 1].role != 0 || fused[front + 2].role != 0)) return 0;
    const bool pair = dwp_role(front + 1, batch) == 1;
    if ((!pair && pdp_w2_off[front] == 0) || (pw_dw_pw != 2 && !pdp_pays(front, batch, pair))) return 0;
    return pdp[i];
  }
  // Roles at the batch of the last f8_chain_prepare and at its halves, worked out there: the rule walks through the launch's shapes, half a
  // microsecond each time, and a run asks for every layer.
  struct PdpRoles {
    int batch = -1;
    std::vector<char> role;
  };
  PdpRoles pdp_prepared[3];
  void forget_pdp_roles() {
    for (PdpRoles &r : pdp_prepared) r.batch = -1;
    roles_batch = -1;
  }
  void prepare_pdp_roles(int batch) {
    forget_pdp_roles();
    const int batches[3] = {batch, batch / 2, batch - batch / 2};
    for (int k = 0; k < 3; ++k) {
      for (size_t i = 0; i < layers.size(); ++i) pdp_prepared[k].role[i] = (char)pdp_role_at(i, batches[k]);
      pdp_prepared[k].batch = batches[k];
    }
  }
  int pdp_role(size_t i, int batch) const {
    for (const PdpRoles &r : pdp_prepared)
      if (r.batch == batch) return r.role[i];
    return pdp_role_at(i, batch);
  }
  // Where the pair is two launches, microseconds of the three, three launches -> one (three launches cost 2 - 4 us more in a forward), MobileNetV2:
  //   56 x 56 C144: batch 16 21.7 -> 10.8, 27 19.2 -> 15.4, 40 23.9 -> 23.5, 64 31.5 -> 29.4; C96 from 112 x 112: batch 16 18.4 -> 13.5, 27 24.4 -> 19.8, 64 40.7 -> 37.7,
  //     96 (either) behind: the rows above and below a workgroup's, computed twice, outweigh the launches
  //   7 x 7 C960: batch 1 9.9 -> 10.5, 16 11.4 -> 10.2, 40 12.5 -> 10.4, 64 13.8 -> 11.0, 128 19.7 -> 13.7, 192 23 -> 24
  // Within these lines, and wherever the pair is one launch, pw_dw_pw_pays decides, from all sizes of the block.
  bool pdp_pays(size_t front, int batch, bool pair) const {
    const Geom &g = geom[front + 1];
    const long long M = (long long)batch * g.P * g.Q;
    if (pdp_image(front)) return pair || M < 3 << 20;
    if (!pair && M > (g.Q > 28 ? 210000 : 10000)) return false;
    return pw_dw_pw_pays(layers[front].Cin, layers[front].Cout, layers[front + 2].Cout, g.H, g.W, g.sh, batch, pair);
  }
  // A 3x3 layer, the 1x1 layer of four times its channels that is its only reader, and (where there is one) the 1x1 layer
  // behind that in one launch: bn[i] = 1 for the first, 2 and 3 for the others; bn_head[i] = the first layer, bn_behind[i]
  // (of the first) = the third or -1.  Whether the three run as one launch depends on the batch.
  std::vector<int> bn, bn_head, bn_behind;   // per layer
  // Where the first layer's copy of the weights lies among the constants (64 and 128 channels, 70 and 278 KB, which almost every
  // batch takes); 0: behind the arena, where the batch takes it (256 channels, 1.1 MB).
  std::vector<size_t> bn_const_off;          // per layer
  int bottleneck = 1;
  int bn_channels(size_t head) const { return bn_behind[head] < 0 ? 0 : layers[bn_behind[head]].Cout; }
  // The 1x1 layer whose result is the closing layer's residual and has no other reader, where the launch takes it along (bn_proj of the head: that layer
  // or -1; bn_of_proj of that layer: the head or -1): the first block of a stage.  Its input is kept until the head has run.
  std::vector<int> bn_proj, bn_of_proj;      // per layer
  int bn_proj_channels(size_t head) const { return bn_proj[head] < 0 ? 0 : layers[bn_proj[head]].Cin; }
  bool proj_role(size_t i, int batch) const { return bn_of_proj[i] >= 0 && bn_role((size_t)bn_of_proj[i], batch) == 1; }
  size_t bn_w_bytes(size_t i) const { return bn[i] == 1 ? bottleneck_weight_bytes(layers[i].Cin, bn_channels(i), bn_proj_channels(i)) : 0; }
  bool bn_allowed(size_t head) const {
    if (bottleneck == 0 || keep_all) return false;
    return !use_fusion() || (fused[head].role == 0 && fused[head + 1].role == 0 && (bn_behind[head] < 0 || fused[bn_behind[head]].role == 0));
  }
  int bn_role(size_t i, int batch) const {
    if (bn[i] == 0 || !bn_allowed((size_t)bn_head[i])) return 0;
    return bottleneck >= 2 || bn_pays((size_t)bn_head[i], batch) ? bn[i] : 0;
  }
  // Microseconds of the three layers, apart -> together (apart the launches cost some 0.4 us each more in a forward than
  // alone), ResNet-50:
  //   64 channels, 56 x 56: batch 1 9.7 -> 7.0, 4 13.8 -> 7.9, 16 19 -> 13.4, 64 38 -> 34 - 36, 128 66 -> 59 (two formats: 103 -> 82), 192 104 -> 91
  //   128 channels, 28 x 28: batch 1 9.3 -> 7.0, 16 19 -> 9.6, 64 32 -> 28, 128 50 -> 45, 192 64 -> 63, 256 79 -> 84; stride 2 from 56 x 56: batch
  //     16 20 -> 11.4, 32 25 -> 20, 48 31.7 -> 30.6, 64 36 -> 42 (the patch leaves room for one workgroup per CU)
  //   256 channels, 14 x 14: batch 1 9.8 -> 12.8, 4 11.7 -> 12.6, 8 13.5 -> 12.7, 16 17.9 -> 13.5, 32 22 -> 14.7, 64 30 -> 22, 96 37 -> 39, 128 42 -> 41
  //     (two formats 45 -> 47); stride 2 from 28 x 28: batch 4 11.7 -> 12.1, 32 26.6 -> 14.7, 64 34.6 -> 29.6, 96 44 -> 44, 128 49 -> 59
  // With a layer behind (and under stride 2 the projection along) the lines lie higher: whole forwards of ResNet-50, one format / two, apart -> together,
  // 64 channels 200 images 1566 -> 1467 / 1929 -> 1753, 250 1818 -> 1708 / 2240 -> 2031; 128 channels 200 1566 -> 1515 / 1929 -> 1848, 250 1818 -> 1749 / 2240 ->
  // 2164, stride 2 56 536 -> 520, 110 903 -> 883, 165 1213 -> 1207, 250 1818 -> 1802; 256 channels 90 811 -> 792, 130 1061 -> 1001, 165 1213 -> 1175,
  // 250 1818 -> 1809 / 2240 -> 2253, stride 2 72 635 -> 613, 110 903 -> 885, 165 1213 -> 1204, 250 1818 -> 1814.  (At 64 and 128 channels that is no
  // crossover: the lines stand below 256 images, where the tests of the layers' own kernels begin.)
  // With no layer behind there is a launch less to save; random blocks of 4 x 4 to 80 x 80, batch 1 to 128, apart / together, mean (least) on
  // either side of the lines: 64 channels stride 2, to 24000 pixels 1.08 (0.91), beyond 0.95 (0.86); 128 channels, to 38000 1.22 (0.94), beyond
  // 1.00 (0.85); stride 2, to 16000 1.09 (0.93), beyond 0.98 (0.92); 256 channels, below 2000 0.98 (0.88), from there 1.19 (0.99).  With one
  // behind, 64 channels stride 2, to 131072 pixels 1.22 (0.99), beyond 0.96.
  bool bn_pays(size_t head, int batch) const {
    const Geom &g = geom[head];
    const long long M = (long long)batch * g.P * g.Q;
    const bool behind = bn_behind[head] >= 0;
    const bool more = behind && bn_proj[head] >= 0;
    if (g.Cin == 64) return g.sh == 1 ? M < (behind ? 800000 : 1 << 19) : M <= (behind ? 131072 : 24000);
    if (g.Cin == 128) return M <= (g.sh == 1 ? (behind ? 200000 : 38000) : more ? 200000 : behind ? 38000 : 16000);
    return M >= (behind ? 1200 : 2000) && M <= (g.sh == 1 ? (behind ? 33000 : 16384) : more ? 33000 : 13000);
  }
  // Copies of weights in fragment order (img_w_bytes, bn_w_bytes, dwp_w_bytes) lie behind the arena and only where this batch, or
  // either half of it on two streams, takes their kernel: ResNet-18 at one image needs 0.7 MB of workspace, with every
  // copy 10 MB.  frag_off: byte offset of layer i's copy in the workspace, 0 for none (bn_off: the copy
  // of the three layers it is the first of).  Returns the copies' bytes; off and boff (one entry per layer) may be null.
  std::vector<size_t> frag_off, bn_off;   // per layer, as of the last f8_chain_prepare
  size_t place_fragments(int batch, size_t *off, size_t *boff) const {
    const size_t base = const_bytes + arena_per_image * (size_t)batch;
    size_t bytes = 0;
    for (size_t i = 0; i < layers.size(); ++i) {
      bool img = false, pair = false, three = false, two = false;
      for (int b : {batch, batch / 2, batch - batch / 2}) {
        if (b < 1) continue;
        const int role = bn_role(i, b);
        three = three || role == 1;
        img = img || (role == 0 && img_role(i, b) != 0);
        pair = pair || dwp_role(i, b) == 1;
        two = two || (s2[i] == 1 && s2_waves(i, b) != 0);
      }
      const bool copy = img || pair || two;
      if (off) off[i] = copy ? base + bytes : 0;
      if (copy) bytes += round256(img ? img_w_bytes[i] : two ? s2_w_bytes(i) : dwp_w_bytes[i]);
      if (boff) boff[i] = !three ? 0 : bn_const_off[i] != 0 ? bn_const_off[i] : base + bytes;
      if (three && bn_const_off[i] == 0) bytes += round256(bn_w_bytes(i));
    }
    return bytes;
  }
  bool tail_in_fused_block(size_t i) const {
    const size_t a = tail[i] == 1 ? i : (size_t)tail_peer[i], b = tail[i] == 1 ? (size_t)tail_peer[i] : i;
    return use_fusion() && (fused[a].role != 0 || fused[b].role != 0);
  }
  int tail_role(size_t i, int batch) const {
    if (!conv_tail || tail[i] == 0 || tail_in_fused_block(i)) return 0;
    const size_t head = tail[i] == 1 ? i : (size_t)tail_peer[i], behind = tail[i] == 1 ? (size_t)tail_peer[i] : i;
    // (a bottleneck's launch computes the first layer of the pair, and of its readers one that need not be this pair's second)
    if (bn_role(head, batch) != 0) return 0;
    Geom g = geom[head];
    g.B = batch;
    return conv_tail_ok(g, layers[head].q, layers[behind].Cout) ? tail[i] : 0;
  }
  std::vector<Tensor> tensors;
  std::vector<size_t> acc0_off;        // per layer: byte offset in the constants region
  size_t const_bytes = 0;
  size_t arena_per_image = 0;          // of every layout
  bool keep_all = false;
  bool planned = false;
  int last_tensor = 0;
  void *prepared_ws = nullptr;
  int prepared_batch = -1;

  // Where tensors and re-laid-out inputs lie in the arena, per image.  A projection that a bottleneck launch takes along (`along`, by the launch's first
  // layer) reads its input when that launch runs, so the input lives longer than where the projection is a launch of its own.  There it
  // must not: the tensors would spread over more memory (first block of a stage, 256 channels from 32 x 32, 240 images, both launches apart: 287 us with the
  // longer life, 261 without).
  struct Layout {
    std::vector<size_t> at, stem_at;   // per tensor, per layer
    size_t bytes = 0;
  };
  Layout placed[2];                    // as of the last f8_chain_prepare: for the whole batch, and for its halves on two streams
  int in_halves = 0;                   // which of them the layers being enqueued use
  void plan() {
    std::vector<char> along(layers.size(), 0);
    const size_t apart = lay_out(along).bytes;
    for (size_t i = 0; i < layers.size(); ++i) along[i] = bn_proj[i] >= 0 && bn_allowed(i);
    arena_per_image = std::max(apart, lay_out(along).bytes);
    planned = true;
  }
  Layout layout_at(int batch, bool halves_of_it) const {
    std::vector<char> along(layers.size(), 0), most(layers.size(), 0);
    for (size_t i = 0; i < layers.size(); ++i) {
      if (bn_proj[i] < 0) continue;
      most[i] = bn_allowed(i);
      for (int b : {halves_of_it ? batch / 2 : batch, halves_of_it ? batch - batch / 2 : batch}) along[i] = along[i] || (b > 0 && bn_role(i, b) == 1);
    }
    Layout l = lay_out(along);
    return l.bytes <= arena_per_image ? l : lay_out(most);       // (a life that is too long is no mistake)
  }
  Layout lay_out(const std::vector<char> &along) const {
    Layout l;
    l.at.assign(tensors.size(), 0);
    l.stem_at.assign(layers.size(), 0);
    std::vector<int> last_use;
    for (const Tensor &t : tensors) last_use.push_back(t.last_use);
    for (size_t i = 0; i < layers.size(); ++i)
      if (along[i]) last_use[layers[bn_proj[i]].src] = std::max(last_use[layers[bn_proj[i]].src], (int)i);
    struct Block { size_t off, size; };
    std::vector<Block> free_list;      // sorted by offset
    size_t top = 0;
    auto alloc = [&](size_t size) -> size_t {
      for (size_t i = 0; i < free_list.size(); ++i) {
        if (free_list[i].size >= size) {
          const size_t off = free_list[i].off;
          free_list[i].off += size;
          free_list[i].size -= size;
          if (free_list[i].size == 0) free_list.erase(free_list.begin() + i);
          return off;
        }
      }
      // extend the arena, reusing a free tail if there is one
      if (!free_list.empty() && free_list.back().off + free_list.back().size == top) {
        const size_t off = free_list.back().off;
        free_list.pop_back();
        top = off + size;
        return off;
      }
      const size_t off = top;
      top += size;
      return off;
    };
    auto release = [&](size_t off, size_t size) {
      Block b{off, size};
      auto it = std::lower_bound(free_list.begin(), free_list.end(), b,
                                 [](const Block &a, const Block &c) { return a.off < c.off; });
      it = free_list.insert(it, b);
      const size_t i = it - free_list.begin();
      if (i + 1 < free_list.size() && free_list[i].off + free_list[i].size == free_list[i + 1].off) {
        free_list[i].size += free_list[i + 1].size;
        free_list.erase(free_list.begin() + i + 1);
      }
      if (i > 0 && free_list[i - 1].off + free_list[i - 1].size == free_list[i].off) {
        free_list[i - 1].size += free_list[i].size;
        free_list.erase(free_list.begin() + i);
      }
    };
    // (a layer that may run inside an earlier layer's launch gets the place of its output there)
    std::vector<char> has_place(tensors.size(), 0);
    auto place = [&](int id) {
      if (tensors[id].external || has_place[id]) return;
      l.at[id] = alloc(round256(tensors[id].bytes_per_image));
      has_place[id] = 1;
    };
    auto give_back = [&](int id) { release(l.at[id], round256(tensors[id].bytes_per_image)); };
    // tail candidates as the planner sees them: any batch, but not inside a fused block
    auto tail_plan = [&](size_t li) { return tail[li] == 0 || tail_in_fused_block(li) ? 0 : tail[li]; };
    for (size_t li = 0; li < layers.size(); ++li) {
      if (pool_role(li) == 2) continue;
      if (pool_role(li) == 1) {
        // one kernel: image in, the pool's output out
        place(layers[li + 1].dst);
        const int src = layers[li].src;
        if (!tensors[src].external && last_use[src] == (int)li) give_back(src);
        continue;
      }
      if (use_fusion() && fused[li].role == 2) continue;
      if (use_fusion() && fused[li].role == 1) {
        // one kernel: reads the block input, writes the third layer's output
        place(layers[li + 2].dst);
        const int src = layers[li].src;
        if (!tensors[src].external && last_use[src] <= (int)li + 2) give_back(src);
        continue;
      }
      if (stem[li].on) l.stem_at[li] = alloc(round256(stem[li].x_bytes_per_image));
      // written by this launch: must not share memory with what any of its layers reads
      if (!keep_all && pdp[li] == 1) place(layers[li + 2].dst);
      if (!keep_all && dwp[li] == 1) place(layers[li + 1].dst);
      if (!keep_all && pair[li] == 1 && layers[li + 1].res < 0) place(layers[li + 1].dst);    // (a shortcut outlives it by itself)
      place(layers[li].dst);
      if (bn[li] == 1 && bn_allowed(li)) {
        place(layers[li + 1].dst);
        if (layers[li + 1].dst2 > 0) place(layers[li + 1].dst2);
        if (bn_behind[li] >= 0) place(layers[bn_behind[li]].dst);
      }
      if (tail_plan(li) == 1) place(layers[tail_peer[li]].dst);
      if (layers[li].dst2 > 0) {
        place(layers[li].dst2);
        // never read: give the space back once this layer has run
        if (!keep_all && last_use[layers[li].dst2] < 0) give_back(layers[li].dst2);
      }
      if (keep_all) continue;
      if (stem[li].on) release(l.stem_at[li], round256(stem[li].x_bytes_per_image));
      const int ids[3] = {layers[li].src, layers[li].res, along[li] ? layers[bn_proj[li]].src : -1};
      for (int k = 0; k < 3; ++k) {
        if (ids[k] < 0) continue;
        if ((k >= 1 && ids[k] == ids[0]) || (k == 2 && ids[2] == ids[1])) continue;
        if (!tensors[ids[k]].external && last_use[ids[k]] == (int)li) give_back(ids[k]);
      }
    }
    l.bytes = top;
    return l;
  }

  // Two halves of a batch can run side by side (f8_chain_set_streams): the second half's tensors lie
  // behind the first half's, arena_shift bytes into the arena, while its layers are enqueued.
  size_t arena_shift = 0;
  int n_streams = 1;
  int halves = 1;
  double image_us = 0;       // operations at 1 POP/s and layers' outputs at 2 TB/s of one image
  // Whether the halves run side by side.  Every launch is there twice then, and where a layer takes hardly more than its launch the halves only wait for
  // one another.  One estimate for all networks, which takes out the clearest losses only:  Microseconds of a forward, whole / halves, 224 x 224 and 160 x 160: ResNet-18 16 131 / 189 and 114 / 158, 64 222 / 269 and 184 / 222, 192
  // 511 / 501; ResNet-50 8 227 / 326 and 201 / 328, 32 347 / 381 and 275 / 330, 64 555 / 536 and 356 / 390, 96 836 / 704 and 523 / 476; MobileNetV1 32 203 /
  // 250 and 160 / 206, 192 523 / 556; MobileNetV2 16 148 / 175 and 125 / 156, 64 306 / 315 and 212 / 218, 96 431 / 413 and 282 / 258.  By the estimate per layer the
  // line lies at 13 images of ResNet-50 at 224 x 224, 15 of ResNet-18, 26 of MobileNetV1 and 44 of MobileNetV2 (160 x 160: twice as many), below the
  // crossover of each (about 50, 190, beyond 192 and 75 in that order), which no one number per layer can follow: between the two the caller's choice stands,
  // and by these figures it loses up to 44 % (ResNet-18, 16 images).
  // Below the line the caller's choice stands too where the whole batch needs four launches more than a half of it (blocks whose one launch pays for few
  // pixels only).  Whole / halves, launches of each: MobileNetV2 224 x 224, 41 images 257 / 238, 26 and 22, 192 x 192, 57 258 / 241, 28 and 22, 64 x 64, 370 258 / 230, 42 and 24,
  // 128 x 128, 107 216 / 226, 26 and 22; with fewer MobileNetV2 96 x 96, 79 161 / 191, 24 and 22, MobileNetV1 224 x 224, 23 183 / 223, 25 and 24.
  bool side_by_side(int batch) const {
    if (n_streams != 2 || keep_all || batch < 2) return false;
    return halves == 2 || image_us * batch >= 3.2 * (double)layers.size() || (batch == roles_batch ? roles_more_launches : more_launches(batch));
  }
  // (as of the last f8_chain_prepare: a run does not look at every layer for it)
  int roles_batch = -1;
  bool roles_more_launches = false;
  bool more_launches(int batch) const {
    int whole = 0, half = 0;
    for (size_t i = 0; i < layers.size(); ++i) {
      whole += !rides_along(i, batch);
      half += !rides_along(i, batch - batch / 2);
    }
    return whole >= half + 4;
  }
  // Whether layer i is computed by another layer's launch at this batch.
  bool rides_along(size_t i, int batch) const {
    if (pool_role(i) != 0) return pool_role(i) == 2;
    if (use_fusion() && fused[i].role != 0) return fused[i].role == 2;
    const int three = bn_role(i, batch), block = pdp_role(i, batch);
    if (three > 1 || proj_role(i, batch) || block == 1 || block == 3) return true;
    if (s2[i] == 2 && s2_waves(i, batch) != 0) return true;
    return pair_role(i, batch) == 1 || (three == 0 && (tail_role(i, batch) == 2 || dwp_role(i, batch) == 2));
  }
  hipStream_t side_stream = nullptr;
  hipEvent_t ev_fork = nullptr, ev_join = nullptr;
  uint8_t *arena(void *workspace) const { return static_cast<uint8_t *>(workspace) + const_bytes + arena_shift; }

  void *tensor_ptr(int id, const void *x, void *out, void *workspace, int batch) const {
    if (id == 0) return const_cast<void *>(x);
    if (id == last_tensor) return out;
    return arena(workspace) + placed[in_halves].at[id] * (size_t)batch;
  }

  // Geometry and operands of dense layer i as the kernel sees them (after the stem re-layout).
  Geom conv_geom(size_t i, int batch) const {
    Geom g = geom[i];
    g.B = batch;
    if (stem[i].on && stem[i].Cp == 4) {
      g.H = stem[i].Hp; g.W = stem[i].Wp; g.Cin = 4; g.S = stem[i].Sp; g.ph = 0; g.pw = 0;
    } else if (stem[i].on) {
      g.Cin = stem[i].Cp;
    }
    return g;
  }
  const int8_t *conv_weights(size_t i, void *workspace) const {
    if (!stem[i].on) return layers[i].w;
    return reinterpret_cast<const int8_t *>(static_cast<uint8_t *>(workspace) + stem[i].w_off);
  }

  // A dense layer whose channel count is not a multiple of 16 normally runs on a zero-padded copy;
  // not when the kernel for few input channels takes it at this batch (its weights 16-byte aligned,
  // its tensors in the arena).
  bool narrow_rows(size_t i, int batch) const {
    const f8_layer_desc &L = layers[i];
    if (!stem[i].on || stem[i].Cp == 4 || L.op != F8_OP_CONV || L.dst2 > 0 || (reinterpret_cast<uintptr_t>(L.w) & 15)) return false;
    if (tensors[L.src].external || tensors[L.dst].external) return false;
    Geom g = geom[i];
    g.B = batch;
    return conv_reads_narrow_rows(g, L.q, L.res >= 0);
  }

  // Parameters of the fused block that starts at layer i.
  BlockParams block_params(size_t i, const void *x, void *out, void *workspace, int batch) const {
    const f8_layer_desc &L0 = layers[i], &L1 = layers[i + 1], &L2 = layers[i + 2];
    const Fused &f = fused[i];
    uint8_t *cb = static_cast<uint8_t *>(workspace);
    BlockParams p;
    p.x = static_cast<const uint8_t *>(tensor_ptr(L0.src, x, out, workspace, batch));
    p.y = tensor_ptr(L2.dst, x, out, workspace, batch);
    p.w1p = reinterpret_cast<const int8_t *>(cb + f.w1p);
    p.w2p = reinterpret_cast<const int8_t *>(cb + f.w2p);
    p.wdp = reinterpret_cast<const int8_t *>(cb + f.wdp);
    p.acc1 = reinterpret_cast<const int32_t *>(cb + f.acc1);
    p.accd = reinterpret_cast<const int32_t *>(cb + f.accd);
    p.acc2 = reinterpret_cast<const int32_t *>(cb + f.acc2);
    p.B = batch; p.H = geom[i].H; p.W = geom[i].W;
    p.Cin = L0.Cin; p.Ce = L0.Cout; p.Cout = L2.Cout;
    p.K1 = f.K1; p.CH = f.CH; p.NB2 = f.NB2;
    block_fused_tiling(p);
    p.x_xor = L0.q.x_type == F8_U8 ? 0x80808080u : 0u;
    const int eb = L0.q.y_type == F8_U8 ? 128 : 0, db = L1.q.y_type == F8_U8 ? 128 : 0;
    p.sh1 = L0.q.fl_x + L0.q.fl_w - L0.q.fl_y; p.lo1 = L0.q.clip_lo - eb; p.hi1 = L0.q.clip_hi - eb;
    p.e_zero = eb ? 0x80808080u : 0u;
    p.shd = L1.q.fl_x + L1.q.fl_w - L1.q.fl_y; p.lod = L1.q.clip_lo - db; p.hid = L1.q.clip_hi - db;
    p.sh2 = L2.q.fl_x + L2.q.fl_w - L2.q.fl_y; p.lo2 = L2.q.clip_lo; p.hi2 = L2.q.clip_hi;
    p.has_res = L2.res >= 0;
    p.res_signed = L2.q.res_type == F8_S8;
    p.res_d = L2.q.fl_x + L2.q.fl_w - L2.q.fl_res;
    return p;
  }

  // Parameters of the three layers that start at the 3x3 layer i.
  BottleneckParams bottleneck_params(size_t i, const void *x, void *out, void *workspace, int batch) const {
    const f8_layer_desc &L = layers[i], &T = layers[i + 1];
    const Geom &g = geom[i];
    const int a = bn_behind[i];
    auto bytes = [&](int id) { return static_cast<uint8_t *>(tensor_ptr(id, x, out, workspace, batch)); };
    auto sign = [](int type) { return type == F8_U8 ? 0x80808080u : 0u; };
    BottleneckParams p;
    p.x = bytes(L.src);
    p.wf = reinterpret_cast<const int8_t *>(static_cast<uint8_t *>(workspace) + bn_off[i]);
    p.res = T.res >= 0 && bn_proj[i] < 0 ? bytes(T.res) : nullptr;
    p.xp = nullptr;
    p.Hp = p.Wp = p.PC = 0; p.sp = 1; p.xp_xor = 0;
    p.shift_p = p.lo_p = p.hi_p = 0;
    if (bn_proj[i] >= 0) {
      const f8_layer_desc &D = layers[bn_proj[i]];
      const Geom &gd = geom[bn_proj[i]];
      p.xp = bytes(D.src);
      p.Hp = gd.H; p.Wp = gd.W; p.PC = D.Cin; p.sp = gd.sh;
      p.xp_xor = sign(D.q.x_type);
      p.shift_p = D.q.fl_x + D.q.fl_w - D.q.fl_y; p.lo_p = D.q.clip_lo; p.hi_p = D.q.clip_hi;
    }
    p.y = bytes(T.dst);
    p.y2 = T.dst2 > 0 ? bytes(T.dst2) : nullptr;
    p.ya = a >= 0 ? bytes(layers[a].dst) : nullptr;
    p.B = batch; p.H = g.H; p.W = g.W; p.C = g.Cin; p.P = g.P; p.Q = g.Q; p.stride = g.sh;
    p.NA = bn_channels(i);
    p.x_xor = sign(L.q.x_type); p.b_xor = sign(L.q.y_type); p.y_xor = sign(T.q.y_type);
    p.shift_b = L.q.fl_x + L.q.fl_w - L.q.fl_y; p.lo_b = L.q.clip_lo; p.hi_b = L.q.clip_hi;
    p.shift_c = T.q.fl_x + T.q.fl_w - T.q.fl_y; p.lo_c = T.q.clip_lo; p.hi_c = T.q.clip_hi;
    p.shift_2 = p.lo_2 = p.hi_2 = p.add_2 = 0;
    if (p.y2) {
      p.shift_2 = T.q.fl_x + T.q.fl_w - T.q2.fl_y; p.lo_2 = T.q2.clip_lo; p.hi_2 = T.q2.clip_hi;
      p.add_2 = (p.shift_2 > 0 ? 1 << (p.shift_2 - 1) : 0) - rounding_addend(T.q);
    }
    p.shift_a = p.lo_a = p.hi_a = 0;
    if (a >= 0) {
      const f8_quant &q = layers[a].q;
      p.shift_a = q.fl_x + q.fl_w - q.fl_y; p.lo_a = q.clip_lo; p.hi_a = q.clip_hi;
    }
    p.res_signed = T.q.res_type == F8_S8;
    p.res_d = T.res >= 0 ? T.q.fl_x + T.q.fl_w - T.q.fl_res : 0;
    p.force = bottleneck;
    return p;
  }

  // Parameters of the stride-2 3x3 layer i and the projection beside it.
  ConvS2Params s2_params(size_t i, const void *x, void *out, void *workspace, int batch) const {
    const f8_layer_desc &L = layers[i];
    uint8_t *cb = static_cast<uint8_t *>(workspace);
    ConvS2Params p;
    p.x = static_cast<const uint8_t *>(tensor_ptr(L.src, x, out, workspace, batch));
    p.w = reinterpret_cast<const int8_t *>(cb + frag_off[i]);
    p.acc0 = reinterpret_cast<const int32_t *>(cb + acc0_off[i]);
    p.y = static_cast<uint8_t *>(tensor_ptr(L.dst, x, out, workspace, batch));
    p.acc0p = nullptr; p.wp = nullptr; p.yp = nullptr;
    p.B = batch; p.H = geom[i].H; p.W = geom[i].W; p.C = L.Cin; p.N = L.Cout;
    p.shift = L.q.fl_x + L.q.fl_w - L.q.fl_y; p.lo = L.q.clip_lo; p.hi = L.q.clip_hi;
    p.shiftp = p.lop = p.hip = 0;
    if (s2_proj[i] >= 0) {
      const f8_layer_desc &T = layers[s2_proj[i]];
      p.acc0p = reinterpret_cast<const int32_t *>(cb + acc0_off[s2_proj[i]]);
      p.wp = reinterpret_cast<const int8_t *>(cb + s2_const_off[s2_proj[i]]);
      p.yp = static_cast<uint8_t *>(tensor_ptr(T.dst, x, out, workspace, batch));
      p.shiftp = T.q.fl_x + T.q.fl_w - T.q.fl_y; p.lop = T.q.clip_lo; p.hip = T.q.clip_hi;
    }
    p.x_xor = L.q.x_type == F8_U8 ? 0x80808080u : 0u;
    p.wk = s2_waves(i, batch);
    return p;
  }

  // Parameters of the basic residual block that starts at layer i.
  ConvPairParams pair_params(size_t i, const void *x, void *out, void *workspace, int batch) const {
    const f8_layer_desc &L = layers[i], &T = layers[i + 1];
    uint8_t *cb = static_cast<uint8_t *>(workspace);
    ConvPairParams p;
    p.x = static_cast<const uint8_t *>(tensor_ptr(L.src, x, out, workspace, batch));
    p.wa = reinterpret_cast<const int8_t *>(cb + frag_off[i]);
    p.wb = reinterpret_cast<const int8_t *>(cb + frag_off[i + 1]);
    p.acc_a = reinterpret_cast<const int32_t *>(cb + acc0_off[i]);
    p.acc_b = reinterpret_cast<const int32_t *>(cb + acc0_off[i + 1]);
    p.y = static_cast<uint8_t *>(tensor_ptr(T.dst, x, out, workspace, batch));
    p.B = batch; p.H = geom[i].H; p.W = geom[i].W; p.C = L.Cin;
    p.x_xor = L.q.x_type == F8_U8 ? 0x80808080u : 0u;
    p.e_xor = L.q.y_type == F8_U8 ? 0x80808080u : 0u;
    p.shift_a = L.q.fl_x + L.q.fl_w - L.q.fl_y; p.lo_a = L.q.clip_lo; p.hi_a = L.q.clip_hi;
    p.shift_b = T.q.fl_x + T.q.fl_w - T.q.fl_y; p.lo_b = T.q.clip_lo; p.hi_b = T.q.clip_hi;
    p.has_res = T.res >= 0;
    p.res_d = p.has_res ? T.q.fl_x + T.q.fl_w - T.q.fl_res : 0;
    return p;
  }

  // Parameters of the inverted-residual block that starts at layer i.
  // (an image of the caller's that does not lie on the four bytes its rows are fetched in: layer by layer)
  bool pdp_reads(size_t front, const void *x, void *workspace, int batch) const {
    return !pdp_image(front) || (reinterpret_cast<uintptr_t>(tensor_ptr(layers[front].src, x, nullptr, workspace, batch)) & 3) == 0;
  }
  PwDwPwParams pdp_params(size_t i, const void *x, void *out, void *workspace, int batch) const {
    const f8_layer_desc &L0 = layers[i], &L1 = layers[i + 1], &L2 = layers[i + 2];
    const Geom &g = geom[i + 1];
    uint8_t *cb = static_cast<uint8_t *>(workspace);
    auto sign = [](int type) { return type == F8_U8 ? 0x80808080u : 0u; };
    PwDwPwParams p;
    p.x = static_cast<const uint8_t *>(tensor_ptr(L0.src, x, out, workspace, batch));
    p.w1 = reinterpret_cast<const int8_t *>(cb + pdp_off[i]);
    p.consts = p.w1 + round256(dw_pw_weight_bytes(pdp_k(i), L0.Cout));
    p.w2 = reinterpret_cast<const int8_t *>(cb + (pdp_w2_off[i] != 0 ? pdp_w2_off[i] : frag_off[i + 1]));
    p.y = static_cast<uint8_t *>(tensor_ptr(L2.dst, x, out, workspace, batch));
    p.B = batch; p.H = g.H; p.W = g.W; p.P = g.P; p.Q = g.Q; p.stride = g.sh;
    p.Cin = L0.Cin; p.Ce = L0.Cout; p.Cout = L2.Cout;
    p.H0 = geom[i].H;
    p.x_xor = sign(L0.q.x_type); p.e_xor = sign(L0.q.y_type); p.d_xor = sign(L1.q.y_type);
    p.shift1 = L0.q.fl_x + L0.q.fl_w - L0.q.fl_y; p.lo1 = L0.q.clip_lo; p.hi1 = L0.q.clip_hi;
    p.shiftd = L1.q.fl_x + L1.q.fl_w - L1.q.fl_y; p.lod = L1.q.clip_lo; p.hid = L1.q.clip_hi;
    p.shift2 = L2.q.fl_x + L2.q.fl_w - L2.q.fl_y; p.lo2 = L2.q.clip_lo; p.hi2 = L2.q.clip_hi;
    p.has_res = L2.res >= 0;
    p.res_d = p.has_res ? L2.q.fl_x + L2.q.fl_w - L2.q.fl_res : 0;
    return p;
  }

  f8_status launch_layer(size_t i, const void *x, void *out, void *workspace, int batch, hipStream_t s) const {
    const f8_layer_desc &L = layers[i];
    Geom g = geom[i];
    g.B = batch;
    if (pool_role(i) == 2) return F8_OK;
    if (pool_role(i) == 1) {
      StemPoolParams sp;
      sp.x = static_cast<const uint8_t *>(tensor_ptr(L.src, x, out, workspace, batch));
      sp.wp = conv_weights(i, workspace);
      sp.acc0 = reinterpret_cast<const int32_t *>(static_cast<uint8_t *>(workspace) + acc0_off[i]);
      sp.y = static_cast<uint8_t *>(tensor_ptr(layers[i + 1].dst, x, out, workspace, batch));
      sp.B = batch; sp.H = g.H; sp.W = g.W;
      sp.x_xor = L.q.x_type == F8_U8 ? 0x80808080u : 0u;
      sp.P = g.P; sp.Q = g.Q; sp.PP = geom[i + 1].P; sp.QP = geom[i + 1].Q;
      sp.shift = L.q.fl_x + L.q.fl_w - L.q.fl_y; sp.lo = L.q.clip_lo; sp.hi = L.q.clip_hi;
      sp.ntiles = 0;
      return launch_stem_pool(sp, s) == 0 ? F8_OK : F8_ERR_DEVICE;
    }
    if (use_fusion() && fused[i].role == 2) return F8_OK;
    if (use_fusion() && fused[i].role == 1) {
      const BlockParams bp = block_params(i, x, out, workspace, batch);
      return launch_block_fused(bp, s) == 0 ? F8_OK : F8_ERR_DEVICE;
    }
    const int three = bn_role(i, batch);
    if (three > 1 || proj_role(i, batch)) return F8_OK;
    if (three == 1 && bn_off[i] != 0) {
      const BottleneckParams bp = bottleneck_params(i, x, out, workspace, batch);
      return launch_bottleneck(bp, s) == 0 ? F8_OK : F8_ERR_DEVICE;
    }
    int block = pdp_role(i, batch);
    if (block != 0 && !pdp_reads(i + 1 - (size_t)block, x, workspace, batch)) block = 0;
    if (block == 1 || block == 3) return F8_OK;
    if (block == 2) {
      const PwDwPwParams pp = pdp_params(i - 1, x, out, workspace, batch);
      return (pdp_image(i - 1) ? launch_image_dw_pw(pp, s) : launch_pw_dw_pw(pp, s)) == 0 ? F8_OK : F8_ERR_DEVICE;
    }
    if (s2[i] != 0 && s2_waves(i, batch) != 0) {
      if (s2[i] == 2) return F8_OK;
      return launch_conv_s2(s2_params(i, x, out, workspace, batch), s) == 0 ? F8_OK : F8_ERR_DEVICE;
    }
    const int twin = pair_role(i, batch);
    if (twin == 1) return F8_OK;
    if (twin == 2) {
      const ConvPairParams cp = pair_params(i - 1, x, out, workspace, batch);
      return launch_conv_pair(cp, s) == 0 ? F8_OK : F8_ERR_DEVICE;
    }
    if (tail_role(i, batch) == 2 || dwp_role(i, batch) == 2) return F8_OK;
    if (dwp_role(i, batch) == 1) {
      const f8_layer_desc &T = layers[i + 1];
      const void *xs = tensor_ptr(L.src, x, out, workspace, batch);
      void *yd = tensor_ptr(T.dst, x, out, workspace, batch);
      const void *rs = T.res >= 0 ? tensor_ptr(T.res, x, out, workspace, batch) : nullptr;
      const int d_shift = L.q.fl_x + L.q.fl_w - L.q.fl_y, t_shift = T.q.fl_x + T.q.fl_w - T.q.fl_y;
      if (frag_off[i] != 0 && dw_pw_applicable(L.Cin, T.Cout, g.Q, d_shift, t_shift, xs, L.w, yd, rs)) {
        DwPwParams dp;
        dp.x = static_cast<const uint8_t *>(xs);
        dp.wd = L.w;
        dp.bias = L.bias;
        dp.wf = reinterpret_cast<const int8_t *>(static_cast<uint8_t *>(workspace) + frag_off[i]);
        dp.acc0 = reinterpret_cast<const int32_t *>(static_cast<uint8_t *>(workspace) + acc0_off[i + 1]);
        dp.y = static_cast<uint8_t *>(yd);
        dp.res = static_cast<const uint8_t *>(rs);
        dp.B = batch; dp.H = g.H; dp.W = g.W; dp.C = L.Cin; dp.N = T.Cout; dp.P = g.P; dp.Q = g.Q; dp.stride = g.sh;
        dp.x_xor = L.q.x_type == F8_U8 ? 0x80808080u : 0u;
        dp.d_xor = L.q.y_type == F8_U8 ? 0x80808080u : 0u;
        dp.d_shift = d_shift; dp.d_lo = L.q.clip_lo; dp.d_hi = L.q.clip_hi;
        dp.shift = t_shift; dp.lo = T.q.clip_lo; dp.hi = T.q.clip_hi;
        dp.res_signed = T.q.res_type == F8_S8;
        dp.res_d = rs ? T.q.fl_x + T.q.fl_w - T.q.fl_res : 0;
        return launch_dw_pw(dp, s) == 0 ? F8_OK : F8_ERR_DEVICE;
      }
      // (a tensor of the caller's at an odd address: the two layers one after the other)
      const f8_status st = enqueue_dwconv(xs, L.w, L.bias, tensor_ptr(L.dst, x, out, workspace, batch), nullptr, g, L.q, s);
      if (st != F8_OK) return st;
      Geom gt = geom[i + 1];
      gt.B = batch;
      return enqueue_conv(tensor_ptr(L.dst, x, out, workspace, batch), T.w,
                          reinterpret_cast<const int32_t *>(static_cast<uint8_t *>(workspace) + acc0_off[i + 1]), workspace, yd, rs, gt, T.q, s);
    }
    const void *src = tensor_ptr(L.src, x, out, workspace, batch);
    void *dst = tensor_ptr(L.dst, x, out, workspace, batch);
    const void *res = L.res >= 0 ? tensor_ptr(L.res, x, out, workspace, batch) : nullptr;
    switch (L.op) {
      case F8_OP_CONV: {
        const int32_t *acc0 = reinterpret_cast<const int32_t *>(static_cast<uint8_t *>(workspace) + acc0_off[i]);
        const int img = frag_off[i] != 0 ? img_role(i, batch) : 0;
        const int shift = L.q.fl_x + L.q.fl_w - L.q.fl_y;
        const int8_t *wf = reinterpret_cast<const int8_t *>(static_cast<uint8_t *>(workspace) + frag_off[i]);
        if (img > 1 && conv_imgk_applicable(L.Cin, L.Cout, L.R, L.S, L.stride_h, L.stride_w, L.pad_h, L.pad_w, g.H, g.W, shift, src, dst, res)) {
          ConvImgkParams ip;
          ip.x = static_cast<const uint8_t *>(src);
          ip.w = wf;
          ip.fold = 0;
          ip.acc0 = acc0;
          ip.y = static_cast<uint8_t *>(dst);
          ip.res = static_cast<const uint8_t *>(res);
          ip.B = batch; ip.H = g.H; ip.W = g.W; ip.C = L.Cin;
          ip.shift = shift; ip.lo = L.q.clip_lo; ip.hi = L.q.clip_hi;
          ip.x_xor = L.q.x_type == F8_U8 ? 0x80808080u : 0u;
          ip.res_signed = L.q.res_type == F8_S8;
          ip.res_d = res ? L.q.fl_x + L.q.fl_w - L.q.fl_res : 0;
          ip.wk = img - 1;
          return launch_conv_imgk(ip, s) == 0 ? F8_OK : F8_ERR_DEVICE;
        }
        if (img == 1 && conv_img_applicable(L.Cin, L.Cout, L.R, L.S, L.stride_h, L.stride_w, L.pad_h, L.pad_w, g.H, g.W, shift, src, dst)) {
          ConvImgParams ip;
          ip.x = static_cast<const uint8_t *>(src);
          ip.wf = wf;
          ip.acc0 = acc0;
          ip.y = static_cast<uint8_t *>(dst);
          ip.B = batch; ip.H = g.H; ip.W = g.W; ip.C = L.Cin;
          ip.shift = shift; ip.lo = L.q.clip_lo; ip.hi = L.q.clip_hi;
          ip.x_xor = L.q.x_type == F8_U8 ? 0x80808080u : 0u;
          return launch_conv_img(ip, s) == 0 ? F8_OK : F8_ERR_DEVICE;
        }
        if (narrow_rows(i, batch)) {
          // the kernel for few input channels reads the 24-channel rows and weights as they are
          return enqueue_conv(src, L.w, acc0, workspace, dst, res, g, L.q, s);
        }
        if (stem[i].on) {
          void *xp = arena(workspace) + placed[in_halves].stem_at[i] * (size_t)batch;
          const int e = stem[i].Cp == 4
                            ? launch_pad_input(src, xp, batch, g.H, g.W, g.Cin, stem[i].Hp, stem[i].Wp, g.ph, g.pw, s)
                            : launch_pad_rows(src, xp, (long long)batch * g.H * g.W, g.Cin, stem[i].Cp, s);
          if (e != 0) return F8_ERR_DEVICE;
          src = xp;
        }
        void *dst2 = L.dst2 > 0 ? tensor_ptr(L.dst2, x, out, workspace, batch) : nullptr;
        ConvTail ct;
        const bool with_tail = tail_role(i, batch) == 1;
        if (with_tail) {
          const f8_layer_desc &T = layers[tail_peer[i]];
          ct.w = T.w;
          ct.acc0 = reinterpret_cast<const int32_t *>(static_cast<uint8_t *>(workspace) + acc0_off[tail_peer[i]]);
          ct.y = tensor_ptr(T.dst, x, out, workspace, batch);
          ct.Cout = T.Cout;
          ct.q = T.q;
        }
        return enqueue_conv(src, conv_weights(i, workspace), acc0, workspace, dst, res, conv_geom(i, batch), L.q, s,
                            dst2 ? &L.q2 : nullptr, dst2, with_tail ? &ct : nullptr);
      }
      case F8_OP_DWCONV: return enqueue_dwconv(src, L.w, L.bias, dst, res, g, L.q, s);
      case F8_OP_MAXPOOL: return enqueue_maxpool(src, dst, g, L.q.x_type, s);
      default: return enqueue_gpool(src, dst, g, L.q, s);
    }
  }
};

extern "C" {

f8_status f8_chain_create(const f8_layer_desc *layers, int n_layers, int in_h, int in_w, int in_c,
                          int in_type, f8_chain **out) {
  if (!layers || !out) return F8_ERR_NULL;
  *out = nullptr;
  if (n_layers < 1 || in_h < 1 || in_w < 1 || in_c < 1) return F8_ERR_SHAPE;
  if (in_type != F8_U8 && in_type != F8_S8) return F8_ERR_DTYPE;
  f8_chain *c = new (std::nothrow) f8_chain();
  if (!c) return F8_ERR_DEVICE;
  f8_status st = F8_OK;
  int max_id = 0;
  for (int i = 0; i < n_layers; ++i) {
    if (layers[i].dst < 1 || layers[i].src < 0 || layers[i].res < -1) { st = F8_ERR_SHAPE; break; }
    max_id = std::max(max_id, std::max(layers[i].dst, std::max(layers[i].src, layers[i].res)));
    max_id = std::max(max_id, (int)layers[i].dst2);
  }
  if (st == F8_OK && max_id > 16 * n_layers + 16) st = F8_ERR_SHAPE;
  if (st != F8_OK) { delete c; return st; }
  c->const_bytes = 256;                // the workspace starts with a block of zeros
  c->tensors.resize(max_id + 1);
  Tensor &t0 = c->tensors[0];
  t0.h = in_h; t0.w = in_w; t0.c = in_c; t0.type = in_type; t0.producer = -1; t0.external = true;
  t0.bytes_per_image = (size_t)in_h * in_w * in_c;

  for (int i = 0; i < n_layers && st == F8_OK; ++i) {
    f8_layer_desc L = layers[i];
    L.q.res = nullptr;
    if (L.dst2 <= 0) L.dst2 = -1;
    Tensor &s = c->tensors[L.src];
    if (s.producer == -2) { st = F8_ERR_SHAPE; break; }           // read before written
    if (c->tensors[L.dst].producer != -2) { st = F8_ERR_SHAPE; break; }   // written twice
    if (L.op < F8_OP_CONV || L.op > F8_OP_GPOOL) { st = F8_ERR_UNSUPPORTED; break; }
    if (L.Cin != s.c || L.q.x_type != s.type) { st = F8_ERR_SHAPE; break; }
    if (s.fl_known && s.fl != L.q.fl_x) { st = F8_ERR_FL; break; }
    s.fl = L.q.fl_x; s.fl_known = true;
    Geom g{1, s.h, s.w, L.Cin, L.Cout, L.R, L.S, L.stride_h, L.stride_w, L.pad_h, L.pad_w, 0, 0};
    Tensor d;
    d.producer = i;
    if (L.op == F8_OP_MAXPOOL) {
      if (L.Cout != L.Cin || L.res >= 0) { st = F8_ERR_SHAPE; break; }
      st = check_geom(g, true);
      if (st != F8_OK) break;
      if (L.pad_h >= L.R || L.pad_w >= L.S) { st = F8_ERR_SHAPE; break; }
      d.type = s.type; d.fl = s.fl; d.fl_known = true;
    } else {
      if (L.op == F8_OP_GPOOL) {
        if (L.Cout != L.Cin || L.res >= 0 || (long long)s.h * s.w > 65536) { st = F8_ERR_SHAPE; break; }
        g.R = s.h; g.S = s.w; g.sh = g.sw = 1; g.ph = g.pw = 0; g.P = g.Q = 1;
        L.R = s.h; L.S = s.w;
      } else {
        if (!L.w) { st = F8_ERR_NULL; break; }
        st = check_geom(g, L.op == F8_OP_DWCONV);
        if (st != F8_OK) break;
      }
      // a dummy non-null residual pointer lets check_quant vet the residual fields
      f8_quant qq = L.q;
      if (L.res >= 0) qq.res = &qq;
      st = check_quant(&qq, L.op != F8_OP_GPOOL);
      if (st != F8_OK) break;
      if (reinterpret_cast<uintptr_t>(L.bias) & 3) { st = F8_ERR_ALIGN; break; }
      d.type = L.q.y_type;
      d.fl = L.q.y_type == F8_S32 ? L.q.fl_x + L.q.fl_w : L.q.fl_y;
      d.fl_known = true;
    }
    if (g.P < 1 || g.Q < 1) { st = F8_ERR_SHAPE; break; }
    d.h = g.P; d.w = g.Q; d.c = L.Cout;
    d.bytes_per_image = (size_t)d.h * d.w * d.c * elem_size(d.type);
    if (L.res >= 0) {
      const Tensor &r = c->tensors[L.res];
      if (r.producer == -2 || L.res == L.dst) { st = F8_ERR_SHAPE; break; }
      if (r.h != d.h || r.w != d.w || r.c != d.c || r.type != L.q.res_type) { st = F8_ERR_SHAPE; break; }
      if (r.fl_known && r.fl != L.q.fl_res) { st = F8_ERR_FL; break; }
      c->tensors[L.res].fl = L.q.fl_res; c->tensors[L.res].fl_known = true;
      c->tensors[L.res].last_use = i;
    }
    if (L.dst2 > 0) {
      // a second format of the same result for a sibling consumer
      if (L.op != F8_OP_CONV || L.dst2 == L.dst || L.dst2 == L.src || L.dst2 == L.res ||
          c->tensors[L.dst2].producer != -2) { st = F8_ERR_SHAPE; break; }
      st = check_requant2(L.q, &L.q2);
      if (st != F8_OK) break;
      Tensor d2 = d;
      d2.type = L.q2.y_type; d2.fl = L.q2.fl_y;
      d2.bytes_per_image = (size_t)d2.h * d2.w * d2.c;
      c->tensors[L.dst2] = d2;
    }
    s.last_use = i;
    c->tensors[L.dst] = d;
    c->layers.push_back(L);
    c->geom.push_back(g);
    c->acc0_off.push_back(c->const_bytes);
    Stem sm;
    if (L.op == F8_OP_CONV) {
      c->const_bytes += acc0_padded(L.Cout) * sizeof(int32_t);
      if (L.Cin <= 4 && L.q.y_type != F8_S32 && (L.Cout & 3) == 0) {
        sm.on = true;
        sm.Sp = (L.S + 3) / 4 * 4;
        sm.Hp = (g.P - 1) * g.sh + g.R;
        // whole 16-byte groups of pixels per row
        sm.Wp = ((g.Q - 1) * g.sw + sm.Sp + 3) / 4 * 4;
        sm.x_bytes_per_image = (size_t)sm.Hp * sm.Wp * 4;
        sm.w_off = c->const_bytes;
        c->const_bytes += round256((size_t)L.Cout * g.R * sm.Sp * 4);
      } else if (L.Cin > 4 && (L.Cin & 15) != 0 && L.q.y_type != F8_S32 && (L.Cout & 3) == 0) {
        sm.on = true;
        sm.Cp = (L.Cin + 15) / 16 * 16;
        sm.x_bytes_per_image = (size_t)g.H * g.W * sm.Cp;
        sm.w_off = c->const_bytes;
        c->const_bytes += round256((size_t)L.Cout * g.R * g.S * sm.Cp);
      }
    }
    size_t img_bytes = 0;
    if (L.op == F8_OP_CONV && !sm.on && L.dst2 <= 0 && L.q.y_type != F8_S32 && !(L.res >= 0 && L.q.res_type == F8_S32) &&
        (reinterpret_cast<uintptr_t>(L.w) & 15) == 0) {
      const int shift = L.q.fl_x + L.q.fl_w - L.q.fl_y;
      if (conv_imgk_applicable(L.Cin, L.Cout, L.R, L.S, L.stride_h, L.stride_w, L.pad_h, L.pad_w, g.H, g.W, shift, nullptr, nullptr, nullptr) ||
          (L.res < 0 &&
           conv_img_applicable(L.Cin, L.Cout, L.R, L.S, L.stride_h, L.stride_w, L.pad_h, L.pad_w, g.H, g.W, shift, nullptr, nullptr)))
        img_bytes = conv_img_weight_bytes(L.Cin);
    }
    c->img_w_bytes.push_back(img_bytes);
    c->stem.push_back(sm);
    c->fused.push_back(Fused());
    c->tail.push_back(0);
    c->tail_peer.push_back(-1);
    c->dwp.push_back(0);
    c->dwp_w_bytes.push_back(0);
    c->frag_off.push_back(0);
    c->pair.push_back(0);
    c->s2.push_back(0);
    c->s2_proj.push_back(-1);
    c->s2_const_off.push_back(0);
    c->pdp.push_back(0);
    c->pdp_off.push_back(0);
    c->pdp_w2_off.push_back(0);
    c->bn.push_back(0);
    c->bn_head.push_back(-1);
    c->bn_proj.push_back(-1);
    c->bn_of_proj.push_back(-1);
    c->bn_behind.push_back(-1);
    c->bn_off.push_back(0);
    c->bn_const_off.push_back(0);
  }
  if (st != F8_OK) { delete c; return st; }
  c->last_tensor = c->layers.back().dst;
  c->tensors[c->last_tensor].external = true;
  c->stem_pool = tuning().stem_pool.load() != 0;
  c->conv_img = tuning().conv_img.load();
  c->conv_img_min = tuning().conv_img_min.load();
  c->imgk = tuning().imgk.load();
  // a stem whose only reader is a 3x3 stride-2 pad-1 max pool: both in one kernel
  for (size_t i = 0; i + 1 < c->layers.size(); ++i) {
    const f8_layer_desc &L = c->layers[i], &M = c->layers[i + 1];
    const Stem &sm = c->stem[i];
    if (L.op != F8_OP_CONV || !sm.on || sm.Cp != 4 || L.Cin != 3 || L.res >= 0 || L.dst2 > 0) continue;
    if (!stem_pool_applicable(L.Cout, L.R, L.S, L.stride_h, L.stride_w, L.pad_h, L.pad_w, sm.Sp)) continue;
    if (L.q.y_type != F8_U8 || L.q.clip_lo < 0 || L.q.fl_x + L.q.fl_w - L.q.fl_y < 0) continue;
    if (M.op != F8_OP_MAXPOOL || M.src != L.dst || M.R != 3 || M.S != 3 || M.stride_h != 2 || M.stride_w != 2 ||
        M.pad_h != 1 || M.pad_w != 1)
      continue;
    if (c->tensors[L.dst].last_use != (int)i + 1 || L.dst == c->last_tensor) continue;
    c->stem[i].pool = 1;
    c->stem[i + 1].pool = 2;
  }
  c->conv_tail = tuning().conv_tail.load() != 0;      // tuning aid
  // a 1x1 64 -> 256 layer and a 1x1 layer of 64 or 128 channels that reads it, or a 1x1 128 -> 512 layer and
  // a 1x1 layer of 128 channels that reads it (the hand-over between two bottleneck blocks): the second can run on each block of the first one's output while it is in LDS.
  // It is the next layer, or the one after it when the layer between them takes no part in a pair (the
  // shortcut projection of a new stage).  Every tensor involved lives in the arena (aligned); weights
  // must be 16-byte aligned.
  for (size_t i = 0; i + 1 < c->layers.size(); ++i) {
    const f8_layer_desc &L = c->layers[i];
    if (c->tail[i] != 0 || c->stem[i].pool != 0 || c->stem[i].on) continue;
    if (L.op != F8_OP_CONV || L.dst2 > 0) continue;
    const bool head64 = L.Cin == 64 && L.Cout == 256, head128 = L.Cin == 128 && L.Cout == 512;
    if (!(head64 || head128) || L.R != 1 || L.S != 1 || L.stride_h != 1 || L.stride_w != 1 || L.pad_h != 0 || L.pad_w != 0) continue;
    if (L.q.y_type == F8_S32 || (L.res >= 0 && L.q.res_type == F8_S32) || L.q.fl_x + L.q.fl_w - L.q.fl_y < 0) continue;
    for (size_t j = i + 1; j <= i + 2 && j < c->layers.size(); ++j) {
      const f8_layer_desc &T = c->layers[j];
      if (c->tail[j] != 0 || c->stem[j].on || c->stem[j].pool != 0) break;
      const bool fits = T.op == F8_OP_CONV && T.src == L.dst && T.dst2 <= 0 && T.res < 0 && (T.Cout == 128 || (head64 && T.Cout == 64)) &&
                        T.R == 1 && T.S == 1 && T.stride_h == 1 && T.stride_w == 1 && T.pad_h == 0 && T.pad_w == 0 &&
                        T.q.y_type != F8_S32 && T.q.fl_x + T.q.fl_w - T.q.fl_y >= 0 &&
                        ((reinterpret_cast<uintptr_t>(L.w) | reinterpret_cast<uintptr_t>(T.w)) & 15) == 0;
      const int ids[4] = {L.src, L.res, L.dst, T.dst};
      bool arena_only = true;
      for (int id : ids) arena_only = arena_only && (id < 0 || !c->tensors[id].external);
      if (fits && arena_only) {
        c->tail[i] = 1; c->tail_peer[i] = (int)j;
        c->tail[j] = 2; c->tail_peer[j] = (int)i;
        break;
      }
    }
  }
  // basic residual blocks of 64 or 128 channels, all tensors in the arena
  c->conv_pair = tuning().conv_pair.load();
  for (size_t i = 0; i + 1 < c->layers.size(); ++i) {
    const f8_layer_desc &L = c->layers[i], &T = c->layers[i + 1];
    if (c->pair[i] != 0 || c->img_w_bytes[i] == 0 || c->img_w_bytes[i + 1] == 0 || L.Cin != T.Cin || L.res >= 0 || T.src != L.dst ||
        c->tensors[L.dst].last_use != (int)i + 1 || (T.res >= 0 && (T.res != L.src || T.q.res_type != L.q.x_type)))
      continue;
    if (c->tensors[L.src].external || c->tensors[L.dst].external || c->tensors[T.dst].external) continue;
    if (!conv_pair_applicable(L.Cin, c->geom[i].H, c->geom[i].W, L.q.fl_x + L.q.fl_w - L.q.fl_y, T.q.fl_x + T.q.fl_w - T.q.fl_y, T.res >= 0,
                              T.res >= 0 ? T.q.fl_x + T.q.fl_w - T.q.fl_res : 0, nullptr, nullptr))
      continue;
    c->pair[i] = 1; c->pair[i + 1] = 2;
  }
  // stride-2 3x3 layers, and a 1x1 stride-2 layer of as many channels beside one (the layer in front of it or behind it) on the same
  // input, all tensors in the arena
  c->conv_s2 = tuning().conv_s2.load();
  for (size_t i = 0; i < c->layers.size(); ++i) {
    const f8_layer_desc &L = c->layers[i];
    const Geom &g = c->geom[i];
    auto plain = [&](size_t l) {
      const f8_layer_desc &D = c->layers[l];
      return D.op == F8_OP_CONV && !c->stem[l].on && D.res < 0 && D.dst2 <= 0 && D.q.y_type != F8_S32 && D.q.fl_x + D.q.fl_w - D.q.fl_y >= 0 &&
             (reinterpret_cast<uintptr_t>(D.w) & 15) == 0 && !c->tensors[D.src].external && !c->tensors[D.dst].external;
    };
    if (!plain(i) || !conv_s2_applicable(L.Cin, L.Cout, L.R, L.S, L.stride_h, L.stride_w, L.pad_h, L.pad_w, g.H, g.W, L.q.fl_x + L.q.fl_w - L.q.fl_y, nullptr, nullptr))
      continue;
    c->s2[i] = 1;
    for (size_t j : {i + 1, i - 1}) {
      if (j >= c->layers.size() || c->s2[j] != 0 || !plain(j)) continue;
      const f8_layer_desc &T = c->layers[j];
      if (T.src != L.src || T.Cout != L.Cout || T.R != 1 || T.S != 1 || T.stride_h != 2 || T.stride_w != 2 || T.pad_h != 0 || T.pad_w != 0) continue;
      c->s2_proj[i] = (int)j;
      c->s2[j] = 2; c->s2_proj[j] = (int)i;
      c->s2_const_off[j] = c->const_bytes;
      c->const_bytes += round256((size_t)T.Cin * T.Cout);
      break;
    }
  }
  // a 3x3 layer, the 1x1 layer of four times its channels that is its only reader, and the 1x1 layer that opens the next
  // block (the next layer, or the one after a new stage's shortcut projection); all tensors in the arena
  c->bottleneck = tuning().bottleneck.load();
  for (size_t i = 0; i + 1 < c->layers.size(); ++i) {
    const f8_layer_desc &L = c->layers[i], &T = c->layers[i + 1];
    const Geom &g = c->geom[i];
    auto plain = [&](size_t l) {
      const f8_layer_desc &D = c->layers[l];
      return D.op == F8_OP_CONV && !c->stem[l].on && c->stem[l].pool == 0 && c->bn[l] == 0 && D.q.y_type != F8_S32 &&
             (reinterpret_cast<uintptr_t>(D.w) & 15) == 0 && !c->tensors[D.src].external && !c->tensors[D.dst].external;
    };
    auto pointwise = [&](size_t l) {
      const f8_layer_desc &D = c->layers[l];
      return plain(l) && D.R == 1 && D.S == 1 && D.stride_h == 1 && D.stride_w == 1 && D.pad_h == 0 && D.pad_w == 0;
    };
    auto shift = [](const f8_layer_desc &D) { return D.q.fl_x + D.q.fl_w - D.q.fl_y; };
    if (!plain(i) || !pointwise(i + 1) || L.R != 3 || L.S != 3 || L.stride_h != L.stride_w || L.pad_h != 1 || L.pad_w != 1 ||
        L.Cout != L.Cin || L.res >= 0 || L.dst2 > 0 || T.src != L.dst || T.Cout != 4 * L.Cout || T.res == L.dst ||
        (T.res >= 0 && (T.q.res_type == F8_S32 || c->tensors[T.res].external)) || c->tensors[L.dst].last_use != (int)i + 1)
      continue;
    int a = -1;
    for (size_t j = i + 2; j <= i + 3 && j < c->layers.size() && a < 0; ++j) {
      const f8_layer_desc &A = c->layers[j];
      if (pointwise(j) && A.src == T.dst && A.res < 0 && A.dst2 <= 0 && (A.Cout == L.Cin || A.Cout == 2 * L.Cin) && shift(A) >= 0) a = (int)j;
    }
    if (!bottleneck_applicable(L.Cin, g.H, g.W, L.stride_h, a < 0 ? 0 : c->layers[a].Cout, shift(L), shift(T), a < 0 ? 0 : shift(c->layers[a]),
                               T.dst2 > 0 ? T.q.fl_x + T.q.fl_w - T.q2.fl_y : 0, T.res >= 0 ? T.q.fl_x + T.q.fl_w - T.q.fl_res : 0))
      continue;
    c->bn[i] = 1; c->bn[i + 1] = 2;
    c->bn_head[i] = c->bn_head[i + 1] = (int)i;
    c->bn_behind[i] = a;
    if (a >= 0) { c->bn[a] = 3; c->bn_head[a] = (int)i; }
  }
  // a depthwise 3x3 layer and the 1x1 layer that is its only reader
  c->dw_pw = tuning().dw_pw.load();
  for (size_t i = 0; i + 1 < c->layers.size(); ++i) {
    const f8_layer_desc &L = c->layers[i], &T = c->layers[i + 1];
    const Geom &g = c->geom[i];
    if (L.op != F8_OP_DWCONV || g.R != 3 || g.S != 3 || g.sh != g.sw || (g.sh != 1 && g.sh != 2) || g.ph != 1 || g.pw != 1 || L.res >= 0 ||
        L.q.y_type == F8_S32 || (long long)g.H * g.W * g.Cin > 0x3fffffffLL || (reinterpret_cast<uintptr_t>(L.bias) & 3))
      continue;
    if (T.op != F8_OP_CONV || T.src != L.dst || T.R != 1 || T.S != 1 || T.stride_h != 1 || T.stride_w != 1 || T.pad_h != 0 || T.pad_w != 0 ||
        T.dst2 > 0 || T.q.y_type == F8_S32 || (T.res >= 0 && T.q.res_type == F8_S32) || T.res == L.dst || c->stem[i + 1].on || c->tail[i + 1] != 0 ||
        c->stem[i + 1].pool != 0)
      continue;
    if (c->tensors[L.dst].last_use != (int)i + 1 || L.dst == c->last_tensor) continue;
    if (!dw_pw_applicable(L.Cin, T.Cout, g.Q, L.q.fl_x + L.q.fl_w - L.q.fl_y, T.q.fl_x + T.q.fl_w - T.q.fl_y, nullptr, L.w, nullptr, nullptr)) continue;
    c->dwp[i] = 1;
    c->dwp[i + 1] = 2;
    c->dwp_w_bytes[i] = dw_pw_weight_bytes(L.Cin, T.Cout);
  }
  // inverted-residual blocks of any stride, all tensors in the arena
  c->pw_dw_pw = tuning().pw_dw_pw.load();
  for (size_t i = 0; i + 2 < c->layers.size(); ++i) {
    const f8_layer_desc &L = c->layers[i], &D = c->layers[i + 1], &T = c->layers[i + 2];
    const Geom &g = c->geom[i + 1];
    const bool image = c->stem[i].on && c->stem[i].Cp == 4;
    auto pointwise = [&](size_t l) {
      const f8_layer_desc &P = c->layers[l];
      if (l == i && image && (P.Cin != 3 || P.R != 3 || P.S != 3 || P.stride_h != 2 || P.stride_w != 2 || P.pad_h != 1 || P.pad_w != 1)) return false;
      return P.op == F8_OP_CONV && ((l == i && image) || (P.R == 1 && P.S == 1 && P.stride_h == 1 && P.stride_w == 1 && P.pad_h == 0 && P.pad_w == 0)) && P.dst2 <= 0 &&
             P.q.y_type != F8_S32 && c->tail[l] == 0 && c->bn[l] == 0 && c->stem[l].pool == 0 && c->pdp[l] == 0;
    };
    if (c->dwp[i] != 0) continue;                    // the second half of the pair in front of it (MobileNetV1)
    if (!pointwise(i) || !pointwise(i + 2) || L.res >= 0 || (T.res >= 0 && (T.res != L.src || T.q.res_type == F8_S32))) continue;
    if (D.op != F8_OP_DWCONV || g.R != 3 || g.S != 3 || g.sh != g.sw || g.ph != 1 || g.pw != 1 || D.res >= 0 || D.q.y_type == F8_S32 ||
        D.src != L.dst || T.src != D.dst || c->tensors[L.dst].last_use != (int)i + 1 || c->tensors[D.dst].last_use != (int)i + 2)
      continue;
    if ((c->tensors[L.src].external && !image) || c->tensors[T.dst].external || c->tensors[D.dst].external) continue;
    if (image) {
      if (T.res >= 0 || !image_dw_pw_applicable(L.Cout, T.Cout, c->geom[i].H, c->geom[i].W, g.sh, L.q.fl_x + L.q.fl_w - L.q.fl_y, D.q.fl_x + D.q.fl_w - D.q.fl_y,
                                                T.q.fl_x + T.q.fl_w - T.q.fl_y, nullptr, nullptr))
        continue;
    } else if (!pw_dw_pw_applicable(L.Cin, L.Cout, T.Cout, g.H, g.W, g.sh, L.q.fl_x + L.q.fl_w - L.q.fl_y, D.q.fl_x + D.q.fl_w - D.q.fl_y,
                             T.q.fl_x + T.q.fl_w - T.q.fl_y, T.res >= 0, T.res >= 0 ? T.q.fl_x + T.q.fl_w - T.q.fl_res : 0, nullptr, nullptr))
      continue;
    c->pdp[i] = 1; c->pdp[i + 1] = 2; c->pdp[i + 2] = 3;
    auto take = [&](size_t bytes) { const size_t off = c->const_bytes; c->const_bytes += round256(bytes); return off; };
    c->pdp_off[i] = take(round256(dw_pw_weight_bytes(c->pdp_k(i), L.Cout)) + pw_dw_pw_const_bytes(L.Cout, T.Cout) + (size_t)(L.Cout + 31) / 32 * 128);
    // (large maps and long K: see dw_pw_pays)
    if (c->pw_dw_pw == 2 || image || c->dwp[i + 1] != 1 || g.Q > 28 || dw_pw_slices(L.Cout, T.Cout) > 20)
      c->pdp_w2_off[i] = take(dw_pw_weight_bytes(L.Cout, T.Cout));
  }
  // inverted-residual blocks that can run as one kernel
  for (size_t i = 0; i + 2 < c->layers.size(); ++i) {
    const f8_layer_desc &L0 = c->layers[i], &L1 = c->layers[i + 1], &L2 = c->layers[i + 2];
    const Geom &g1 = c->geom[i + 1];
    auto pointwise = [](const f8_layer_desc &L) {
      return L.op == F8_OP_CONV && L.R == 1 && L.S == 1 && L.stride_h == 1 && L.stride_w == 1 && L.pad_h == 0 &&
             L.pad_w == 0 && L.q.y_type != F8_S32 && L.q.fl_x + L.q.fl_w - L.q.fl_y >= 0;
    };
    if (c->fused[i].role != 0 || !pointwise(L0) || !pointwise(L2) || L0.res >= 0) continue;
    if (L0.dst2 > 0 || L1.dst2 > 0 || L2.dst2 > 0) continue;
    if (L1.op != F8_OP_DWCONV || g1.R != 3 || g1.S != 3 || g1.sh != 1 || g1.sw != 1 || g1.ph != 1 || g1.pw != 1 ||
        L1.res >= 0 || L1.q.y_type == F8_S32 || L1.q.fl_x + L1.q.fl_w - L1.q.fl_y < 0)
      continue;
    if (L1.src != L0.dst || L2.src != L1.dst) continue;
    if (c->tensors[L0.dst].last_use != (int)i + 1 || c->tensors[L1.dst].last_use != (int)i + 2) continue;
    if (L0.dst == c->last_tensor || L1.dst == c->last_tensor) continue;
    if (L2.res >= 0 && (L2.res != L0.src || L0.Cin != L2.Cout || L2.q.res_type == F8_S32)) continue;
    if ((L0.Cin & 3) || (L0.Cout & 3) || (L2.Cout & 3) || L0.Cin > BLOCK_MAX_CIN || L2.Cout > BLOCK_MAX_COUT) continue;
    Fused &f = c->fused[i];
    f.role = 1;
    c->fused[i + 1].role = c->fused[i + 2].role = 2;
    f.K1 = (L0.Cin + 31) / 32 * 32;
    f.CH = (L0.Cout + 31) / 32;
    f.NB2 = (L2.Cout + 31) / 32;
    auto take = [&](size_t bytes) { const size_t off = c->const_bytes; c->const_bytes += round256(bytes); return off; };
    f.w1p = take((size_t)f.CH * 32 * f.K1);
    f.w2p = take((size_t)f.CH * f.NB2 * 1024);
    f.wdp = take((size_t)f.CH * 288);
    f.acc1 = take((size_t)f.CH * 32 * sizeof(int32_t));
    f.accd = take((size_t)f.CH * 32 * sizeof(int32_t));
    f.acc2 = take((size_t)f.NB2 * 32 * sizeof(int32_t));
    i += 2;
  }
  // The projection of a stage's first block inside its bottleneck launch: a 1x1 layer whose only reader is the closing layer's shortcut and that no
  // other launch computes (behind a depthwise layer it belongs to that one's).  Then the launches' weights have their sizes.
  for (size_t i = 0; i + 1 < c->layers.size(); ++i) {
    if (c->bn[i] != 1) continue;
    const f8_layer_desc &L = c->layers[i], &T = c->layers[i + 1];
    const Geom &g = c->geom[i];
    const int pr = T.res > 0 && tuning().bn_proj.load() != 0 ? c->tensors[T.res].producer : -1;
    int readers = 0;
    for (const f8_layer_desc &D : c->layers) readers += (D.src == T.res) + (D.res == T.res);
    if (pr >= 0 && readers == 1 && pr < (int)i && c->bn[pr] == 0 && c->s2[pr] == 0 && c->tail[pr] == 0 && c->dwp[pr] == 0 && c->pdp[pr] == 0 &&
        c->fused[pr].role == 0 && !c->stem[pr].on && c->stem[pr].pool == 0) {
      const f8_layer_desc &D = c->layers[pr];
      const int shift = D.q.fl_x + D.q.fl_w - D.q.fl_y;
      if (D.op == F8_OP_CONV && D.R == 1 && D.S == 1 && D.stride_h == D.stride_w && D.pad_h == 0 && D.pad_w == 0 && D.res < 0 && D.dst == T.res &&
          D.dst2 <= 0 && D.q.y_type != F8_S32 && shift >= 0 && (reinterpret_cast<uintptr_t>(D.w) & 15) == 0 && !c->tensors[D.src].external &&
          !c->tensors[D.dst].external && bottleneck_projects(L.Cin, g.H, g.W, L.stride_h, c->bn_channels(i), D.Cin, D.stride_h)) {
        c->bn_proj[i] = pr;
        c->bn_of_proj[pr] = (int)i;
      }
    }
    if (L.Cin <= 128) {
      c->bn_const_off[i] = c->const_bytes;
      c->const_bytes += round256(c->bn_w_bytes(i));
    }
  }
  c->halves = tuning().halves.load();
  for (size_t i = 0; i < c->layers.size(); ++i) {
    const f8_layer_desc &L = c->layers[i];
    const Geom &g = c->geom[i];
    const double taps = L.op == F8_OP_CONV ? (double)g.R * g.S * g.Cin : L.op == F8_OP_DWCONV ? (double)g.R * g.S : 0.0;
    c->image_us += 2.0 * g.P * g.Q * L.Cout * taps / 1e9 + (double)c->tensors[L.dst].bytes_per_image / 2e6;
  }
  c->const_bytes = round256(c->const_bytes);
  for (auto &r : c->pdp_prepared) r.role.assign(c->layers.size(), 0);
  *out = c;
  return F8_OK;
}

f8_status f8_chain_set_keep_all(f8_chain *c, int keep_all) {
  if (!c) return F8_ERR_NULL;
  c->keep_all = keep_all != 0;
  c->planned = false;
  c->forget_pdp_roles();
  c->prepared_ws = nullptr;
  return F8_OK;
}

f8_status f8_chain_set_fusion(f8_chain *c, int fusion) {
  if (!c) return F8_ERR_NULL;
  c->fusion = fusion != 0;
  c->planned = false;
  c->forget_pdp_roles();
  c->prepared_ws = nullptr;
  return F8_OK;
}

f8_status f8_chain_workspace_bytes(const f8_chain *cc, int batch, size_t *bytes) {
  if (!cc || !bytes) return F8_ERR_NULL;
  if (batch < 0) return F8_ERR_SHAPE;
  f8_chain *c = const_cast<f8_chain *>(cc);
  if (!c->planned) c->plan();
  // every tensor must stay addressable with 32-bit element counts
  for (const Tensor &t : c->tensors)
    if (t.producer != -2 && (long long)t.bytes_per_image / (long long)elem_size(t.type) * batch > 0x7fffffffLL)
      return F8_ERR_UNSUPPORTED;
  for (const Stem &sm : c->stem)
    if (sm.on && (long long)sm.x_bytes_per_image * batch > 0x7fffffffLL) return F8_ERR_UNSUPPORTED;
  // A smaller batch may take kernels with copies that this one does not need; a workspace for the largest batch of a
  // program has to hold every smaller one too.  Where a smaller arena saves more than all copies take, nothing more
  // can be needed; a chain whose arena is next to nothing gets room for all of them instead of a long search.
  size_t copies = 0, most = 0;
  for (size_t i = 0; i < c->layers.size(); ++i) copies += round256(c->img_w_bytes[i]) + round256(c->s2_w_bytes(i)) + round256(c->dwp_w_bytes[i]) + (c->bn_const_off[i] == 0 ? round256(c->bn_w_bytes(i)) : 0);
  for (int b = batch; b >= 0 && c->arena_per_image * (size_t)(batch - b) <= copies; --b) {
    const bool far = batch - b >= 1024;
    most = std::max(most, c->arena_per_image * (size_t)b + (far ? copies : c->place_fragments(b, nullptr, nullptr)));
    if (far) break;
  }
  *bytes = c->const_bytes + most + 256;
  return F8_OK;
}

f8_status f8_chain_prepare(f8_chain *c, void *workspace, int batch, void *stream) {
  if (!c || !workspace) return F8_ERR_NULL;
  if (batch < 0) return F8_ERR_SHAPE;
  if (reinterpret_cast<uintptr_t>(workspace) & 255) return F8_ERR_ALIGN;
  if (!c->planned) c->plan();
  hipStream_t s = static_cast<hipStream_t>(stream);
  c->prepared_ws = nullptr;
  for (int k : {0, 1}) c->placed[k] = c->layout_at(batch, k == 1);
  c->place_fragments(batch, c->frag_off.data(), c->bn_off.data());
  c->prepare_pdp_roles(batch);
  c->roles_batch = batch;
  c->roles_more_launches = c->more_launches(batch);
  if (hipMemsetAsync(workspace, 0, 256, s) != hipSuccess) return F8_ERR_DEVICE;
  for (size_t i = 0; i < c->layers.size(); ++i) {
    const f8_layer_desc &L = c->layers[i];
    if (L.op != F8_OP_CONV) continue;
    if (c->stem[i].on) {
      void *wp = static_cast<uint8_t *>(workspace) + c->stem[i].w_off;
      const int e = c->stem[i].Cp == 4
                        ? launch_repack_weights(L.w, wp, L.Cout, L.R, L.S, L.Cin, c->stem[i].Sp, c->pool_role(i) == 1 ? 1 : 0, s)
                        : launch_pad_rows(L.w, wp, (long long)L.Cout * L.R * L.S, L.Cin, c->stem[i].Cp, s);
      if (e != 0) return F8_ERR_DEVICE;
    }
    int32_t *acc0 = reinterpret_cast<int32_t *>(static_cast<uint8_t *>(workspace) + c->acc0_off[i]);
    const f8_status st = enqueue_fold(c->conv_weights(i, workspace), L.bias, acc0, c->conv_geom(i, 1), L.q, s);
    if (st != F8_OK) return st;
    if (c->dwp[i] == 2 && c->frag_off[i - 1] != 0 &&
        launch_dw_pw_weights(L.w, reinterpret_cast<int8_t *>(static_cast<uint8_t *>(workspace) + c->frag_off[i - 1]), L.Cin, L.Cout, s) != 0)
      return F8_ERR_DEVICE;
    if (c->frag_off[i] != 0 && c->s2[i] == 1) {
      int8_t *cb = static_cast<int8_t *>(workspace);
      int e = launch_conv_s2_weights(L.w, cb + c->frag_off[i], 9, L.Cin, L.Cout, s);
      if (e == 0 && c->s2_proj[i] >= 0) e = launch_conv_s2_weights(c->layers[c->s2_proj[i]].w, cb + c->s2_const_off[c->s2_proj[i]], 1, L.Cin, L.Cout, s);
      if (e != 0) return F8_ERR_DEVICE;
    } else if (c->frag_off[i] != 0 &&
        launch_conv_img_weights(L.w, reinterpret_cast<int8_t *>(static_cast<uint8_t *>(workspace) + c->frag_off[i]), L.Cin, s) != 0)
      return F8_ERR_DEVICE;
  }
  for (size_t i = 0; i < c->layers.size(); ++i) {
    if (c->pdp[i] != 1) continue;
    const f8_layer_desc &L = c->layers[i], &D = c->layers[i + 1], &T = c->layers[i + 2];
    uint8_t *cb = static_cast<uint8_t *>(workspace);
    int8_t *w1 = reinterpret_cast<int8_t *>(cb + c->pdp_off[i]);
    int8_t *consts = w1 + round256(dw_pw_weight_bytes(c->pdp_k(i), L.Cout));
    int32_t *accd = reinterpret_cast<int32_t *>(consts + pw_dw_pw_const_bytes(L.Cout, T.Cout));
    auto start = [&](size_t l) { return reinterpret_cast<const int32_t *>(cb + c->acc0_off[l]); };
    const int res_bias = T.res >= 0 && T.q.res_type == F8_U8 ? 128 << (T.q.fl_x + T.q.fl_w - T.q.fl_res) : 0;
    int e = launch_dw_pw_weights(c->pdp_image(i) ? c->conv_weights(i, workspace) : L.w, w1, c->pdp_k(i), L.Cout, s);
    if (e == 0) e = launch_block_fold_dw(D.w, D.bias, accd, L.Cout, (L.Cout + 31) / 32 * 32, rounding_addend(D.q), D.q.x_type == F8_U8 ? 128 : 0, s);
    if (e == 0 && c->pdp_w2_off[i] != 0) e = launch_dw_pw_weights(T.w, reinterpret_cast<int8_t *>(cb + c->pdp_w2_off[i]), T.Cin, T.Cout, s);
    if (e == 0) e = launch_pw_dw_pw_consts(D.w, start(i), accd, start(i + 2), consts, L.Cout, T.Cout, res_bias, s);
    if (e != 0) return F8_ERR_DEVICE;
  }
  for (size_t i = 0; i < c->layers.size(); ++i) {
    if (c->bn_off[i] == 0) continue;
    const f8_layer_desc &L = c->layers[i], &T = c->layers[i + 1];
    const int a = c->bn_behind[i];
    uint8_t *cb = static_cast<uint8_t *>(workspace);
    auto start = [&](size_t l) { return reinterpret_cast<const int32_t *>(cb + c->acc0_off[l]); };
    const int res_bias = T.res >= 0 && T.q.res_type == F8_U8 ? 128 << (T.q.fl_x + T.q.fl_w - T.q.fl_res) : 0;
    const int pr = c->bn_proj[i];
    if (launch_bottleneck_weights(L.w, T.w, a < 0 ? nullptr : c->layers[a].w, pr < 0 ? nullptr : c->layers[pr].w, start(i), start(i + 1),
                                  a < 0 ? nullptr : start(a), pr < 0 ? nullptr : start(pr), reinterpret_cast<int8_t *>(cb + c->bn_off[i]), L.Cin,
                                  c->bn_channels(i), c->bn_proj_channels(i), res_bias, s) != 0)
      return F8_ERR_DEVICE;
  }
  for (size_t i = 0; i < c->layers.size(); ++i) {
    const Fused &f = c->fused[i];
    if (f.role != 1) continue;
    const f8_layer_desc &L0 = c->layers[i], &L1 = c->layers[i + 1], &L2 = c->layers[i + 2];
    uint8_t *cb = static_cast<uint8_t *>(workspace);
    int e = launch_block_pack_w1(L0.w, reinterpret_cast<int8_t *>(cb + f.w1p), L0.Cout, L0.Cin, f.CH, f.K1, s);
    if (e == 0) e = launch_block_pack_w2(L2.w, reinterpret_cast<int8_t *>(cb + f.w2p), L2.Cout, L0.Cout, f.NB2, f.CH, s);
    if (e == 0) e = launch_block_pack_wd(L1.w, reinterpret_cast<int8_t *>(cb + f.wdp), L0.Cout, f.CH, s);
    // start values; an unsigned intermediate is kept minus 128 (see BlockParams)
    const int eb = L0.q.y_type == F8_U8 ? 128 : 0, db = L1.q.y_type == F8_U8 ? 128 : 0;
    const int sh1 = L0.q.fl_x + L0.q.fl_w - L0.q.fl_y, shd = L1.q.fl_x + L1.q.fl_w - L1.q.fl_y;
    if (e == 0) e = launch_fold_acc0(L0.w, L0.bias, reinterpret_cast<int32_t *>(cb + f.acc1), L0.Cout, f.CH * 32, L0.Cin,
                                     L0.q.x_type == F8_U8, rounding_addend(L0.q) - (eb << sh1), s);
    if (e == 0) e = launch_block_fold_dw(L1.w, L1.bias, reinterpret_cast<int32_t *>(cb + f.accd), L0.Cout, f.CH * 32,
                                         rounding_addend(L1.q) - (db << shd), eb, s);
    if (e == 0) e = launch_fold_acc0(L2.w, L2.bias, reinterpret_cast<int32_t *>(cb + f.acc2), L2.Cout, f.NB2 * 32, L0.Cout,
                                     L2.q.x_type == F8_U8, rounding_addend(L2.q), s);
    if (e != 0) return F8_ERR_DEVICE;
  }
  c->prepared_ws = workspace;
  c->prepared_batch = batch;
  return F8_OK;
}

f8_status f8_chain_run(f8_chain *c, const void *x, void *out, void *workspace, int batch, void *stream) {
  if (!c || !x || !out || !workspace) return F8_ERR_NULL;
  if (batch < 0) return F8_ERR_SHAPE;
  if (c->prepared_ws != workspace || c->prepared_batch != batch) return F8_ERR_STATE;
  if (c->tensors[c->last_tensor].type == F8_S32 && (reinterpret_cast<uintptr_t>(out) & 3)) return F8_ERR_ALIGN;
  if (batch == 0) return F8_OK;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (c->side_by_side(batch)) {
    // first half of the images on the caller's stream, second half on the chain's own stream, which
    // starts behind everything already queued on the caller's stream and is waited for at the end
    const int b0 = batch / 2, b1 = batch - b0;
    const Tensor &tin = c->tensors[0], &tout = c->tensors[c->last_tensor];
    const void *x1 = static_cast<const uint8_t *>(x) + tin.bytes_per_image * (size_t)b0;
    void *out1 = static_cast<uint8_t *>(out) + tout.bytes_per_image * (size_t)b0;
    if (hipEventRecord(c->ev_fork, s) != hipSuccess || hipStreamWaitEvent(c->side_stream, c->ev_fork, 0) != hipSuccess)
      return F8_ERR_DEVICE;
    f8_status st = F8_OK;
    c->in_halves = 1;
    for (size_t i = 0; i < c->layers.size() && st == F8_OK; ++i) {
      c->arena_shift = 0;
      st = c->launch_layer(i, x, out, workspace, b0, s);
      if (st != F8_OK) break;
      c->arena_shift = c->arena_per_image * (size_t)b0;
      st = c->launch_layer(i, x1, out1, workspace, b1, c->side_stream);
    }
    c->arena_shift = 0;
    c->in_halves = 0;
    // join even after a failed launch, so that a capture in progress is left in a consistent state
    if (hipEventRecord(c->ev_join, c->side_stream) != hipSuccess || hipStreamWaitEvent(s, c->ev_join, 0) != hipSuccess)
      return F8_ERR_DEVICE;
    return st;
  }
  for (size_t i = 0; i < c->layers.size(); ++i) {
    const f8_status st = c->launch_layer(i, x, out, workspace, batch, s);
    if (st != F8_OK) return st;
  }
  return F8_OK;
}

f8_status f8_chain_set_streams(f8_chain *c, int n_streams) {
  if (!c) return F8_ERR_NULL;
  if (n_streams != 1 && n_streams != 2) return F8_ERR_UNSUPPORTED;
  if (n_streams == 2 && !c->side_stream) {
    if (hipStreamCreateWithFlags(&c->side_stream, hipStreamNonBlocking) != hipSuccess) { c->side_stream = nullptr; return F8_ERR_DEVICE; }
    if (hipEventCreateWithFlags(&c->ev_fork, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&c->ev_join, hipEventDisableTiming) != hipSuccess)
      return F8_ERR_DEVICE;
  }
  c->n_streams = n_streams;
  return F8_OK;
}

int f8_chain_streams(const f8_chain *c, int batch) { return c && c->side_by_side(batch) ? 2 : 1; }

f8_status f8_chain_tensor(const f8_chain *c, int id, void *workspace, int batch, void **ptr, int *h, int *w,
                          int *ch, int *dtype, int *live_at_end) {
  if (!c) return F8_ERR_NULL;
  if (id < 0 || id >= (int)c->tensors.size() || c->tensors[id].producer == -2) return F8_ERR_SHAPE;
  if (!c->planned) const_cast<f8_chain *>(c)->plan();
  const Tensor &t = c->tensors[id];
  // tensors inside a fused block are never materialised
  const bool elided = (t.producer >= 0 && (c->pool_role((size_t)t.producer) == 1 || c->dwp_role((size_t)t.producer, batch) == 1 ||
                                             c->pdp_role((size_t)t.producer, batch) == 1 || c->pdp_role((size_t)t.producer, batch) == 2 ||
                                             c->bn_role((size_t)t.producer, batch) == 1 || c->proj_role((size_t)t.producer, batch) || c->pair_role((size_t)t.producer, batch) == 1)) ||
                      (c->use_fusion() && t.producer >= 0 && c->fused[t.producer].role != 0 &&
                       !(c->fused[t.producer].role == 2 && t.producer >= 2 && c->fused[t.producer - 2].role == 1));
  // (with two streams the two halves of a tensor lie apart: not reported)
  const bool halves = c->n_streams == 2 && !c->keep_all && batch >= 2;
  const f8_chain::Layout l = c->layout_at(batch, false);
  if (ptr) *ptr = (t.external || !workspace || elided || halves) ? nullptr : c->arena(workspace) + l.at[id] * (size_t)batch;
  if (h) *h = t.h;
  if (w) *w = t.w;
  if (ch) *ch = t.c;
  if (dtype) *dtype = t.type;
  if (live_at_end) {
    int live = elided ? 0 : 1;
    if (!c->keep_all && !t.external && !elided) {
      // overwritten if something allocated after this tensor's last use overlaps it
      const size_t a0 = l.at[id], a1 = a0 + round256(t.bytes_per_image);
      for (size_t j = 0; j < c->tensors.size() && live; ++j) {
        const Tensor &o = c->tensors[j];
        if ((int)j == id || o.external || o.producer == -2 || o.producer <= t.last_use ||
            o.producer <= t.producer)
          continue;
        const size_t b0 = l.at[j], b1 = b0 + round256(o.bytes_per_image);
        if (a0 < b1 && b0 < a1) live = 0;
      }
      for (size_t j = 0; j < c->stem.size() && live; ++j) {
        const Stem &sm = c->stem[j];
        if (!sm.on || c->pool_role(j) == 1 || (int)j <= t.last_use || (int)j <= t.producer) continue;
        const size_t b0 = l.stem_at[j], b1 = b0 + round256(sm.x_bytes_per_image);
        if (a0 < b1 && b0 < a1) live = 0;
      }
    }
    *live_at_end = live;
  }
  return F8_OK;
}

void f8_chain_destroy(f8_chain *c) {
  if (!c) return;
  if (c->ev_fork) (void)hipEventDestroy(c->ev_fork);
  if (c->ev_join) (void)hipEventDestroy(c->ev_join);
  if (c->side_stream) (void)hipStreamDestroy(c->side_stream);
  delete c;
}

// ---- measurement aids ---------------------------------------------------------------------

int f8_chain_num_layers(const f8_chain *c) { return c ? (int)c->layers.size() : 0; }

f8_status f8_chain_layer_info(const f8_chain *c, int layer, int batch, char *kernel_name, int name_len,
                              double *alg_ops, double *alg_bytes) {
  if (!c) return F8_ERR_NULL;
  if (layer < 0 || layer >= (int)c->layers.size() || batch < 0) return F8_ERR_SHAPE;
  const f8_layer_desc &L = c->layers[layer];
  const Geom &g = c->geom[layer];
  const char *name = "?";
  double ops = 0.0;
  if (c->pool_role((size_t)layer) != 0) {
    // stem and pool are accounted to the stem: image in, pooled tensor out, weights
    const bool first = c->pool_role((size_t)layer) == 1;
    const char *fname = first ? "stem_pool_fused" : "(fused)";
    if (kernel_name && name_len > 0) {
      int i = 0;
      for (; fname[i] && i < name_len - 1; ++i) kernel_name[i] = fname[i];
      kernel_name[i] = 0;
    }
    const Geom &gp = c->geom[first ? layer + 1 : layer];
    if (alg_ops) *alg_ops = first ? 2.0 * batch * g.P * g.Q * (double)g.R * g.S * g.Cin * g.Cout : 0.0;
    if (alg_bytes)
      *alg_bytes = first ? (double)batch * g.H * g.W * g.Cin + (double)batch * gp.P * gp.Q * g.Cout +
                               (double)g.R * g.S * g.Cin * g.Cout + 4.0 * g.Cout
                         : 0.0;
    return F8_OK;
  }
  if (c->use_fusion() && c->fused[layer].role != 0) {
    // the whole block is accounted to its first layer: block input + output (+ shortcut read
    // from the same input), all weights
    double fo = 0.0, fb = 0.0;
    const char *fname = "(fused)";
    if (c->fused[layer].role == 1) {
      const f8_layer_desc &L1 = c->layers[layer + 1], &L2 = c->layers[layer + 2];
      const double px = (double)batch * g.H * g.W;
      fo = 2.0 * px * ((double)L.Cin * L.Cout + 9.0 * L1.Cout + (double)L2.Cin * L2.Cout);
      fb = px * (L.Cin + L2.Cout) + (double)L.Cin * L.Cout + 9.0 * L1.Cout + (double)L2.Cin * L2.Cout +
           4.0 * (L.Cout + L1.Cout + L2.Cout);
      fname = "block_fused";
    }
    if (kernel_name && name_len > 0) {
      int i = 0;
      for (; fname[i] && i < name_len - 1; ++i) kernel_name[i] = fname[i];
      kernel_name[i] = 0;
    }
    if (alg_ops) *alg_ops = fo;
    if (alg_bytes) *alg_bytes = fb;
    return F8_OK;
  }
  const int three = c->bn_role((size_t)layer, batch);
  const int block = c->pdp_role((size_t)layer, batch), twin = c->pair_role((size_t)layer, batch);
  const bool two = c->s2_waves((size_t)layer, batch) != 0;
  if (c->rides_along((size_t)layer, batch) && !c->proj_role((size_t)layer, batch)) {
    // accounted to the layer in front (of the first layer of an inverted-residual or basic block: behind), whose launch computes this one
    const char *fname = "(fused)";
    if (kernel_name && name_len > 0) {
      int i = 0;
      for (; fname[i] && i < name_len - 1; ++i) kernel_name[i] = fname[i];
      kernel_name[i] = 0;
    }
    if (alg_ops) *alg_ops = 0.0;
    if (alg_bytes) *alg_bytes = 0.0;
    return F8_OK;
  }
  const bool with_tail = c->tail_role((size_t)layer, batch) == 1;
  const double M = (double)batch * g.P * g.Q;
  if (c->proj_role((size_t)layer, batch)) {
    // computed by the bottleneck launch, which takes its time; operations, input and weights are this layer's, its output stays in the launch
    const int head = c->layers[c->bn_of_proj[layer]].Cin;
    const char *fname = head == 64 ? "1x1 in bottleneck<64>" : head == 128 ? "1x1 in bottleneck<128>" : "1x1 in bottleneck<256>";
    if (kernel_name && name_len > 0) {
      int i = 0;
      for (; fname[i] && i < name_len - 1; ++i) kernel_name[i] = fname[i];
      kernel_name[i] = 0;
    }
    if (alg_ops) *alg_ops = 2.0 * M * (double)L.Cin * L.Cout;
    if (alg_bytes) *alg_bytes = M * L.Cin + (double)L.Cin * L.Cout + 4.0 * L.Cout;
    return F8_OK;
  }
  // input pixels a strided window actually touches
  const double rows = g.sh >= g.R ? (double)g.P * g.R : (double)std::min(g.H, (g.P - 1) * g.sh + g.R);
  const double cols = g.sw >= g.S ? (double)g.Q * g.S : (double)std::min(g.W, (g.Q - 1) * g.sw + g.S);
  double bytes = (double)batch * rows * cols * g.Cin + M * g.Cout * (double)elem_size(c->tensors[L.dst].type);
  if (L.res >= 0) bytes += M * g.Cout * (double)elem_size(c->tensors[L.res].type);
  if (L.dst2 > 0) bytes += M * g.Cout;
  switch (L.op) {
    case F8_OP_CONV: {
      Geom gk = c->narrow_rows((size_t)layer, batch) ? g : c->conv_geom(layer, batch);
      gk.B = batch;
      gk.P = g.P; gk.Q = g.Q;
      const int img = c->img_role((size_t)layer, batch);
      if (three == 1) name = L.Cin == 64 ? "bottleneck<64>" : L.Cin == 128 ? "bottleneck<128>" : "bottleneck<256>";
      else if (two) name = c->s2_proj[layer] >= 0 ? (L.Cin == 64 ? "conv3x3_imgk_s2<64>+1x1" : L.Cin == 128 ? "conv3x3_imgk_s2<128>+1x1" : "conv3x3_imgk_s2<256>+1x1")
                                                  : (L.Cin == 64 ? "conv3x3_imgk_s2<64>" : L.Cin == 128 ? "conv3x3_imgk_s2<128>" : "conv3x3_imgk_s2<256>");
      else if (img > 1) name = L.Cin == 64 ? "conv3x3_imgk<64>" : L.Cin == 128 ? "conv3x3_imgk<128>" : L.Cin == 256 ? "conv3x3_imgk<256>" : "conv3x3_imgk<512>";
      else if (img == 1) name = L.Cin == 256 ? "conv3x3_img<256x256>" : "conv3x3_img<128x128>";
      else name = conv_kernel_name(gk, L.q, L.res >= 0, L.dst2 > 0 ? &L.q2 : nullptr);
      ops = 2.0 * M * g.R * g.S * g.Cin * g.Cout;
      bytes += (double)g.R * g.S * g.Cin * g.Cout + 4.0 * g.Cout;
      if (two && c->s2_proj[layer] >= 0) {
        // plus the projection: its operand is the middle tap's
        ops += 2.0 * M * g.Cin * g.Cout;
        bytes += M * g.Cout + (double)g.Cin * g.Cout + 4.0 * g.Cout;
      }
      if (twin == 2) {
        // plus the 3x3 layer in front: the block's input (also its shortcut) and output
        name = L.Cin == 64 ? "conv3x3_pair<64>" : "conv3x3_pair<128>";
        ops *= 2.0;
        bytes = 2.0 * (M * L.Cin + 9.0 * L.Cin * L.Cin + 4.0 * L.Cin);
      }
      if (three == 1) {
        // plus the closing layer (residual in, one or two formats out) and the layer behind it
        const f8_layer_desc &T = c->layers[layer + 1];
        ops += 2.0 * M * (double)T.Cin * T.Cout;
        bytes += M * ((double)T.Cout * (1 + (T.res >= 0) + (T.dst2 > 0)) - L.Cout) + (double)T.Cin * T.Cout + 4.0 * T.Cout;
        // a projection in the launch is accounted to its own layer; its result is no residual read from memory
        if (c->bn_proj[layer] >= 0) bytes -= M * T.Cout;
        if (c->bn_behind[layer] >= 0) {
          const f8_layer_desc &A = c->layers[c->bn_behind[layer]];
          ops += 2.0 * M * (double)A.Cin * A.Cout;
          bytes += M * A.Cout + (double)A.Cin * A.Cout + 4.0 * A.Cout;
        }
      } else if (with_tail) {
        // plus the 1x1 layer behind it: its output and weights; its input never leaves the chip
        const f8_layer_desc &T = c->layers[c->tail_peer[layer]];
        name = L.Cin == 128 ? "pw1x1_mid<128x512>+1x1<128>" : (T.Cout == 64 ? "pw1x1_ws<64x256>+1x1<64>" : "pw1x1_ws<64x256>+1x1<128>");
        ops += 2.0 * M * (double)T.Cin * T.Cout;
        bytes += M * T.Cout + (double)T.Cin * T.Cout + 4.0 * T.Cout;
      }
      break;
    }
    case F8_OP_DWCONV:
      if (block == 2 || c->dwp_role((size_t)layer, batch) == 1) {
        // plus the 1x1 layer that reads it: what lies between them never leaves the chip
        const f8_layer_desc &T = c->layers[layer + 1];
        name = g.sh == 1 ? "dwconv3x3<s1>+1x1" : "dwconv3x3<s2>+1x1";
        ops = 2.0 * M * (9.0 * L.Cout + (double)T.Cin * T.Cout);
        bytes += M * (T.Cout - L.Cout) + (T.res >= 0 ? M * T.Cout : 0.0) + 13.0 * L.Cout + (double)T.Cin * T.Cout + 4.0 * T.Cout;
        if (block == 2) {
          // and the 1x1 layer in front, all of whose pixels are needed; the shortcut is its input, read once
          const f8_layer_desc &E = c->layers[layer - 1];
          const Geom &ge = c->geom[layer - 1];
          if (c->pdp_image((size_t)layer - 1)) name = g.sh == 1 ? "conv3x3+dwconv3x3<s1>+1x1" : "conv3x3+dwconv3x3<s2>+1x1";
          else name = g.sh == 1 ? "1x1+dwconv3x3<s1>+1x1" : "1x1+dwconv3x3<s2>+1x1";
          const double taps = (double)E.R * E.S * E.Cin * E.Cout;
          ops += 2.0 * batch * g.H * g.W * taps;
          bytes += (double)batch * ge.H * ge.W * E.Cin - (double)batch * rows * cols * g.Cin - (T.res >= 0 ? M * T.Cout : 0.0) + taps + 4.0 * E.Cout;
        }
        break;
      }
      name = (g.R == 3 && g.S == 3 && g.sh == g.sw && (g.sh == 1 || g.sh == 2) && g.Cin % 4 == 0 && L.res < 0 &&
              c->tensors[L.dst].type != F8_S32 && L.q.fl_x + L.q.fl_w - L.q.fl_y >= 0)
                 ? (g.sh == 1 ? "dwconv3x3<s1>" : "dwconv3x3<s2>")
                 : "dwconv_generic";
      ops = 2.0 * M * g.R * g.S * g.Cout;
      bytes += (double)g.R * g.S * g.Cout + 4.0 * g.Cout;
      break;
    case F8_OP_MAXPOOL: name = "maxpool"; break;
    default: name = "gpool"; break;
  }
  if (kernel_name && name_len > 0) {
    int i = 0;
    for (; name[i] && i < name_len - 1; ++i) kernel_name[i] = name[i];
    kernel_name[i] = 0;
  }
  if (alg_ops) *alg_ops = ops;
  if (alg_bytes) *alg_bytes = bytes;
  return F8_OK;
}

f8_status f8_chain_profile(f8_chain *c, const void *x, void *out, void *workspace, int batch, void *stream,
                           int repeats, float *layer_ms) {
  if (!c || !x || !out || !workspace || !layer_ms) return F8_ERR_NULL;
  if (batch < 1 || repeats < 1) return F8_ERR_SHAPE;
  if (c->prepared_ws != workspace || c->prepared_batch != batch) return F8_ERR_STATE;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const size_t n = c->layers.size();
  // Two passes per repeat, events after every layer: pass A launches each layer once, pass B
  // launches it 1 + EXTRA times back to back (a layer never writes what it reads, so the
  // relaunches recompute the same bytes).  (B - A) / EXTRA is the duration of one launch in a
  // busy stream; the cost of the event pair itself, a few microseconds, cancels.
  constexpr int EXTRA = 4;
  const size_t per = 2 * (n + 1);
  std::vector<hipEvent_t> ev(repeats * per);
  for (auto &e : ev)
    if (hipEventCreate(&e) != hipSuccess) return F8_ERR_DEVICE;
  f8_status st = F8_OK;
  for (int r = 0; r < repeats && st == F8_OK; ++r) {
    for (int pass = 0; pass < 2 && st == F8_OK; ++pass) {
      hipEvent_t *e = &ev[r * per + pass * (n + 1)];
      (void)hipEventRecord(e[0], s);
      for (size_t i = 0; i < n && st == F8_OK; ++i) {
        for (int k = 0; k < (pass ? 1 + EXTRA : 1) && st == F8_OK; ++k) st = c->launch_layer(i, x, out, workspace, batch, s);
        (void)hipEventRecord(e[i + 1], s);
      }
    }
  }
  if (hipStreamSynchronize(s) != hipSuccess) st = F8_ERR_DEVICE;
  if (st == F8_OK) {
    for (size_t i = 0; i < n; ++i) {
      double a_sum = 0.0, b_sum = 0.0;
      for (int r = 0; r < repeats; ++r) {
        float ms = 0.f;
        (void)hipEventElapsedTime(&ms, ev[r * per + i], ev[r * per + i + 1]);
        a_sum += ms;
        (void)hipEventElapsedTime(&ms, ev[r * per + (n + 1) + i], ev[r * per + (n + 1) + i + 1]);
        b_sum += ms;
      }
      const double one = (b_sum - a_sum) / (EXTRA * (double)repeats);
      layer_ms[i] = (float)(one > 0.0 ? one : b_sum / ((1 + EXTRA) * (double)repeats));
    }
  }
  for (auto &e : ev) (void)hipEventDestroy(e);
  return st;
}

}  // extern "C"
