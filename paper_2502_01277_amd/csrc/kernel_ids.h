// Kernel ids of the convolution launchers: which template instance a launch ran, as decimal digits, so that a profile by layer
// can be laid beside one by kernel name (bench.py's conv_name decodes them; tests/test_kernel_names.py walks every
// launcher's instances through both).  Host arithmetic only: no HIP header is needed to compile this file.
#pragma once

namespace octo {

// general kernel (conv.hip): 1 BBB PPP K M V - channel tile, pixel tile, 16-byte vectors per K step, workgroups per compute unit the
// registers are sized for, flags (1: vectorised gather, 2: straight to LDS, 4: pipelined loop)
constexpr int conv_kernel_id(int bc, int bp, int kv, int minb, bool vec, bool dma, bool pipe) {
  return 1000000000 + bc * 1000000 + bp * 1000 + kv * 100 + minb * 10 + (vec ? 1 : 0) + (dma ? 2 : 0) + (pipe ? 4 : 0);
}

// general form whose loads run across tiles (conv_flow.h), digits 12 M BBB PPP K: how addresses are made, channel tile, pixel tile, 16-byte
// vectors per K step
constexpr int flow_kernel_id(int bc, int bp, int kv, int mode) { return 1200000000 + mode * 10000000 + bc * 10000 + bp * 10 + kv; }

// launches of few tiles (conv_small.h), digits 13 M BBB PPP W: how addresses are made, channel tile, pixel tile, wavefronts along the channels
constexpr int small_kernel_id(int bc, int bp, int wc, int mode) { return 1300000000 + mode * 10000000 + bc * 10000 + bp * 10 + wc; }

// 3x3 layers with the input patch in LDS (conv3x3_mid.h), digits FF Q BBB CCC: family (17: more than 64 output channels, 18: up to
// 64, 14: input channels not in whole slices), pixel tile (0: 128, 1: 256, 2: 64, 3: 128 with a patch of five passes), channel
// tile, input channels whose patch the two buffers hold.  vn: values per 16-byte vector
constexpr int mid_kernel_id(int bc, int bp, int kv, int vn, int passes, int cin, int cout) {
  const int family = cin % (kv * vn) ? 1400000000 : (cout > 64 ? 1700000000 : 1800000000);
  const int q = bp == 128 ? (passes == 5 ? 3 : 0) : (bp == 256 ? 1 : 2);
  return family + q * 1000000 + bc * 1000 + 2 * kv * vn;
}

// their streaming form (conv3x3_stream.h): the same digits with Q = 5, wc blocks of 32 channels, kc groups of 16 input channels
constexpr int stream3_kernel_id(int wc, int kc, int kv, int cin) {
  return (cin % (kv * 8) ? 1400000000 : 1800000000) + 5000000 + wc * 32000 + kc * 16;
}

// streaming 1x1 kernel (conv1x1.hip), digits 15 BBB KKK: channel tile, input channels
constexpr int stream1_kernel_id(int tc, int cin) { return 1500000000 + 32 * tc * 1000 + cin; }

// split-K kernel (conv_ksplit.h), digits 16 S BBB PPP: K split, channel tile, pixel tile
constexpr int ksplit_kernel_id(int bc, int bp, int ks) { return 1600000000 + ks * 1000000 + bc * 1000 + bp; }

// 3x3 layers of few tiles (conv3x3_held.h), digits 20 S K BBB PPP: stride, wavefronts that share K, channel tile, pixel tile
constexpr int held_kernel_id(int bc, int bp, int ks, int s) { return 2000000000 + s * 10000000 + ks * 1000000 + bc * 1000 + bp; }

// first layers (stem.hip), digits 19 F BBB KK P: with the max-pool behind it, channel tile, kernel height, kernel width on the
// pixel-pair view.  With the max-pool, SiLU and channel counts that are no multiple of 8 run stem_pool_any_kernel under the same id
constexpr int stem_kernel_id(int bc, int kh, int pkw, bool pool) { return 1900000000 + (pool ? 1000000 : 0) + bc * 1000 + kh * 10 + pkw; }

// the first layers of a detector in one launch (entry.hip)
constexpr int KID_ENTRY = 2100000000;
// a cross-stage block of 32 channels in one launch (block.hip), last digit 1: without a shortcut
constexpr int block_kernel_id(bool shortcut) { return 2110000000 + (shortcut ? 0 : 1); }
constexpr bool is_block(int id) { return id / 10000000 == 211; }
// the entry of a cross-stage block in one launch (lead.hip), digits 212 P BBB KKK: pixel tile / 16, channels of a layer, input channels
constexpr int lead_kernel_id(int c, int cin, int np) { return 2120000000 + np * 1000000 + c * 1000 + cin; }
constexpr bool is_lead(int id) { return id / 10000000 == 212; }
// several layers of conv_small_kernel in one launch (conv_small.h), digits 213 G BBB PPP: G = twice the number of layers + how addresses are made, tile.  The layer that had its
// arguments collected first reports it, the others KID_NONE
constexpr int group_kernel_id(int bc, int bp, int count, int mode) { return 2130000000 + (2 * count + mode) * 1000000 + bc * 1000 + bp; }
constexpr int group_layers(int id) { return id / 10000000 == 213 ? id / 1000000 % 10 / 2 : 0; }

}  // namespace octo
