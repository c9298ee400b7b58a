// Which form of a kernel a launch takes, by the sizes of the launch.  Host code only, and apart from the kernels, so that a test
// without a GPU can hold every choice against what was measured on both sides of it.
#pragma once

#include "qoda_kernels.h"

namespace qoda {

// Blocks of an octet that a wave of the other decode passes takes, for G tiles: 2, 4 or 8.  While its waves do not fill the device a
// pass is a chain of loads and table reads, K nodes one after the other: the shorter a wave's part the better (G up to 256, 128 for
// the mean).  Then a wave's fixed work and its loads of part of a word weigh more, and whole octets are best, except: (1) with one
// or two nodes there is no chain to speak of, and many short waves hide the loads and stores of the iterates; (2) wide codes, and bucket
// norms, take more registers for whole octets (80 to 92 under bucket scope: five or six waves a SIMD), so that half octets win
// from two thirds of a fill on; (3) where whole octets just fill the device (1100 to 1500 tiles, with bucket norms 513 to 640) they win;
// (4) with decode tables above 8 KiB a part of two blocks serves half the octets that the others serve with one set of tables.
// us of a call with 8 / 4 / 2 blocks:
//   mean         5 bits, K = 4: 64 5.6 / 4.8 / 4.3, 128 5.8 / 5.9 / 5.8, 256 6.8 / 7.7 / 8.4; 9 bits, K = 2: 256
//                7.2 / 6.7 / 7.3, 600 13.4 / 14.9 / 15.8, 1000 23.5 / 20.9 / 23.4; bucket norms, 8 bits, K = 8:
//                600 26.2 / 29.0 / 30.1, 1000 46.0 / 42.8 / 47.0, 6400 279 / 250 / 275
//   extrapolate  5 bits, K = 8: 200 16.6 / 14.2 / 14.2, 320 18.9 / 16.9 / 18.8, 512 22.1 / 21.8 / 24.3, 600 25.4
//                / 27.9 / 28.9; K = 16: 384 26.3 / 25.8 / 30.2, 512 30.2 / 31.1 / 35.5; bucket norms, 8 bits, K
//                = 4: 600 23.6 / 26.3 / 25.4, 700 33.0 / 28.2 / 28.4, 3200 128 / 114 / 113; 5 bits, K = 8: 700
//                29.6 / 32.0 / 34.9, 800 38.6 / 34.5 / 40.6, 1300 51.1 / 51.6 / 60.5
//   update       5 bits, K = 1: 600 33.5 / 35.9 / 29.4, 2400 119 / 120 / 108; K = 2: 600 34.2 / 37.2 / 31.5, 3200
//                155 / 152 / 146; K = 8: 200 23.8 / 20.1 / 18.7, 320 27.4 / 26.0 / 26.9, 450 33.3 / 35.0 / 32.1,
//                600 40.8 / 45.0 / 41.3, 3200 188 / 188 / 183; 9 bits, K = 8: 256 28.1 / 24.8 / 24.5, 512 41.2 /
//                41.8 / 46.0, 1000 86.5 / 79.9 / 86.9; bucket norms, 8 bits, K = 4: 600 37.5 / 41.5 / 37.5, 800
//                56.2 / 51.3 / 49.7, 3200 198 / 186 / 172; 5 bits, K = 8: 600 41.6 / 45.8 / 44.0, 800 60.0 /
//                56.2 / 57.2, 1300 82.2 / 85.5 / 86.0
inline int decode_blocks(int G, int K, int mode, bool bucket, int bits) {
  const bool wide = bits >= 7, tables = (long long)K << bits > 2048;   // tables: 8 KiB
  const int full = bucket && bits >= 6 ? 640 : 750;                   // where whole octets need a second fill
  if (mode == kDecodeMean) {
    if (G <= 128) return tables && G > 64 ? 4 : 2;
    if (G <= 160) return bits >= 8 && K > 2 && !tables ? 2 : 4;
    if (K == 1) return (G > 512 && G <= (!bucket ? 850 : wide ? 640 : 750)) || (bucket && !wide && bits != 5 && G > 1000) ? 8 : 4;
    if (tables ? G <= (bits == 9 ? 320 : 200) : K == 2 && G <= (wide ? 512 : 256)) return 4;
    if (bucket) return (wide ? G > (K <= 8 ? full : 900) : K == 2 && G > 850 && G <= 1100) ? 4 : 8;
    return K == 2 && bits >= 8 && G > 900 ? 4 : 8;
  }
  const bool update = mode == kDecodeUpdate;
  if (update) {
    if (G <= 256 || K <= 2) return 2;
    if (tables) { if (G <= 400) return 4; }
    else if (wide && K <= (bits == 7 ? 4 : 8)) return K >= 4 && G > 512 && G <= (bucket ? full : 850) ? 8 : 2;
    else if (K <= 4 ? G <= 512 || (G > 2000 && G <= 5600) : K <= 8 && G > 330 && G <= 450) return 2;
    else if (K > 4 && G <= 384) return 4;
  } else {
    if (G <= (tables || K > 16 ? 160 : 256)) return 2;
    if (G <= (wide || K <= 8 ? 512 : 384)) return 4;
    if (K == 1) return G > (bucket ? full : 1100) ? 2 : 8;
  }
  // from about one fill on
  if (tables && G > 1024 && G <= 1150) return 8;
  if (bucket && bits >= 6) return G > full ? 4 : 8;
  if (bucket) return (G > full && G <= 900) || (K <= (update ? 16 : 8) && G > full && (G <= 1100 || G > 1500)) ? 4 : 8;
  if (tables) return (G > 900 && G <= 1024) || G > 1800 ? 4 : 8;
  return K <= 8 && G > 2400 && (update || bits >= 5) ? 4 : 8;
}

// Whether the mean in whole octets requests node 0's record before it sets up its tables.  Codes of up to 6 bits, time with that
// against without, mean over 200 to 6400 tiles: K = 1 and 2, 3 to 5 bits 0.96 to 0.98; K = 3 and 5, 4 to 6 bits 0.985 to 1.0 (from 1200
// tiles on 0.93 to 0.99); K = 8 to 16 1.00 to 1.015; bucket norms, K = 1 0.97, K = 2 0.97 to 1.005, K = 3 to 16 1.01 to 1.045.  Other
// passes: 1.005 to 1.03 for every K; wider codes: 1.0 to 1.01.  With 5 bits and bucket norms it costs the sixth wave of a SIMD (81
// registers).
constexpr bool mean_early(int G, int K, bool bucket, int bits) {
  return bits <= 6 && (K <= 2 ? !bucket || bits != 5 : !bucket && K <= 6 && G > 900);
}

// Blocks of a tile's 64 that a wave of the (Alt) decode pass takes, one workgroup a tile: 8 (eight waves) or 16 (four waves, two
// octets one after the other).  Two workgroups of eight waves fit a CU, four of four waves (three under bucket scope, and with codes
// of 6 bits and more a few spilled registers): just beyond 512 tiles, where the second half of a launch in eight waves is mostly
// empty, four waves are faster, for few nodes; with more of them the chain over the nodes, twice as long in four waves, weighs
// more.  us of a call in 8 / 16 blocks, 5-bit codes: K = 1 512 tiles 34.6 / 41.4, 576 46.6 / 45.1, 640 47.8 / 45.1, 768 50.9 / 48.0,
// 960 59.7 / 59.6, 1024 61.3 / 55.7, 1100 74.7 / 83.9; K = 4 576 53.8 / 51.2, 768 58.7 / 55.6, 1100 80.5 / 97.1; K = 8 576 59.4 / 59.9,
// 768 65.6 / 66.2; 8-bit codes, K = 1 704 52.1 / 49.4, 832 55.7 / 55.9, K = 4 640 55.8 / 55.6; bucket norms, K = 1 640 50.3 / 45.8, 768
// 53.5 / 49.3, 832 56.9 / 73.5; K = 4 704 59.0 / 55.2, 11 k 589.0 / 686.1.
inline int alt_blocks(int G, int K, bool bucket, int bits) {
  if (G <= 768) return G > 512 && K <= 4 ? 16 : 8;
  return !bucket && bits <= 5 && G <= 1024 && K <= 2 ? 16 : 8;
}

// Whether k_quantize looks levels up by grid bin (one read of 128 bits, 4 KiB of table to fetch per workgroup) rather than by byte and
// tau (two reads one after the other, 1 KiB), for n tiles of all nodes of the launch.  Without a previous message and with codes of up
// to 6 bits the bins take 82 to 84 registers, the bytes at most 80: five against six workgroups a CU, which shows where 1281 to 1536
// tiles are one wave of the chip with bytes and two with bins.  With the previous message and 9 bits it is 98 against 96 registers, four
// workgroups a CU against five.  us with bins / with bytes: no previous message, 3 bits, 400 tiles 12.2 / 12.0, 1280 19.5 / 20.1, 1500
// 26.4 / 23.4, 1700 28.7 / 29.1, 10 k 123.9 / 125.9, 74 k 886 / 907; 5 bits, 400 12.3 / 12.3, 1500 27.3 / 24.5, 10 k 130.5 / 133.0; 6 bits,
// 400 12.5 / 13.1, 1280 20.6 / 20.9, 1500 27.8 / 24.7, 10 k 134.6 / 137.4; previous message, 8 bits, 400 14.2 / 14.8, 1280 25.1 / 25.9,
// 3100 56.6 / 57.5, 10 k 165.8 / 166.3; 9 bits, 400 14.5 / 14.8, 1280 29.3 / 26.6, 2000 40.1 / 40.8, 3100 61.8 / 60.5, 74 k 1218 / 1300.
// Elsewhere both take the same time, within 1 %, or the bytes less.
constexpr bool quantize_bins_width(bool prev, int bits) { return prev ? bits >= 8 : bits <= 6; }   // widths that have the form
constexpr bool quantize_bytes_width(bool prev, int bits) { return !prev || bits != 8; }
inline bool quantize_bins(long long n, bool prev, int bits) {
  if (!quantize_bins_width(prev, bits)) return false;
  if (prev) return bits == 8 || n <= 1024 || n > 4096;
  return n > 1536 || (bits == 6 && n <= 1280);
}

// Which tiles of a call that computes norms and codes are held from the one to the other (k_quantize_held: one read of the vectors)
// and which go through the norm pass, its combination and the quantizer.  A group (a layer's tiles; under vector scope a
// node's) waits for its last tile, so what counts is how its tiles share the slots of the device with others that load or quantize
// meanwhile.  us with the separate kernels / held, of a whole pass of K nodes (quantize, decode, and what else is in it), but `call`: of
// quantize calls one after the other (most of these with a layer whose end is ragged):
//   * All tiles on the device at once: call, 5 bits 640 tiles 30 / 24, 1024 in one layer 36 / 29, in layers of 64 36 / 29; one norm per
//     vector 960 38 / 29.  (Launches of k_quantize_small and a little beyond stay as they are.)
//   * Layers of up to two fifths of the slots, vectors of up to half: there are always some that load and some that quantize.  Vectors
//     of 389 tiles, K = 3 60 / 55, 4 73 / 62, 7 111 / 94, 16 191 / 180, of 230 K = 3 57 / 48, 12 124 / 111, of 512 K = 8 call 108 / 101;
//     layers of up to 389, K = 4 97 / 86, 8 152 / 133, of up to 198 with 8 bits, K = 4 1459 / 1247; call, 12 k tiles in layers of 1
//     342 / 243, 64 326 / 259, 256 309 / 285.  Larger ones among them do no harm up to a quarter of the tiles (511 of 2815, 8 bits,
//     K = 4 455 / 407); beyond that they do: 511 of 640 tiles, K = 4 117 / 121, 8 186 / 199.
//   * Larger groups: up to two fills.  Vectors of 650, K = 2 97 / 92; layers of up to 700, K = 2 107 / 99, 8 242 / 246; up to 991, K = 1
//     106 / 103, 2 138 / 143.  Not three or more groups of over half of the slots, which come one after the other: vectors of 560, K = 3
//     67 / 74, with ragged ends 75 / 77; layers of 650, K = 3 72 / 79.  (Layers with ragged ends 600, K = 3 77 / 76, 650 77 / 79.)
//   * Layers that all end with a whole octet: the separate kernels, which take a ragged one block by block, are 5 to 8 us faster there.  Little
//     more than a fill is not held then.  One layer a node: 342 tiles, K = 3 43 / 46, with ragged ends 48 / 44; 513, K = 2 43 / 47; 409,
//     K = 3 48 / 50; 150, K = 7 44 / 46, 9 56 / 52; 300, K = 4 46 / 48, 5 58 / 54; 256, K = 5 47 / 47; layers of 16 and fewer 1030 tiles 57 / 57 and
//     55 / 51.  9 bits: layers of 16, 780 tiles 48 / 54, 1152 61 / 65, 1300 69 / 66; of 64, 1000 tiles 53 / 56, 1152 59 / 60.
//     Left as they are: whole vectors of a third of the slots (342, K = 5 67 / 69, 8 100 / 96, 12 132 / 133), 9 bits with layers of 16, 2.1
//     to 2.6 fills (1650 tiles 87 / 92, 2000 99 / 101).
//   * 9 bits (three workgroups a CU), previous message, calls: layers of 16 to 64 tiles 3 k 105 / 100, 12 k 354 / 348; 192 1.5 k 57 / 57,
//     3 k 104 / 102, 6 k 178 / 188; 384 3 k 104 / 107.
//   * Where not all are held: layers of up to held_small() are, beside larger ones (whether the device could hold those or not) that go
//     through the separate kernels.  Two sets of launches, two more tails: only where the small ones are many and a good part of all.  20
//     k tiles in layers of up to 53 beside 54 k, 4 bits 2223 / 2131; 11.7 k beside 5.9 k, 5 bits 587 / 534; 12 k in layers of 256 beside
//     148 k, 3 bits 7352 / 7408; one node, 2.5 k beside 6.8 k 250 / 254.
enum HeldTiles { kHoldNone = 0, kHoldAll = 1, kHoldSmall = 2 };
constexpr long long kHeldLeast = 640, kHeldLeastVector = 832;   // tiles of a launch
constexpr long long kHeldSmallLeast = 8192;
struct HeldModel {
  int scope, slots;
  long long tiles, small_tiles;   // of a node; in layers of up to held_small()
  int largest;                    // tiles of the largest layer
  int over_half;                  // layers of more than half of the slots
  bool whole;                     // every layer ends with a whole octet
};
inline int held_small(const HeldModel &h) { return h.slots != kHeldSlots ? h.slots / 12 : h.scope == kScopeVector ? h.slots / 2 : 2 * h.slots / 5; }
inline HeldTiles held_tiles(const HeldModel &h, int nodes) {
  const long long n = h.tiles * nodes, least = h.scope == kScopeVector ? kHeldLeastVector : kHeldLeast;
  const int group = h.scope == kScopeVector ? (int)(h.tiles < INT32_MAX ? h.tiles : INT32_MAX) : h.largest;
  if (h.scope == kScopeBucket || n < least) return kHoldNone;
  if (group <= h.slots) {
    const bool vec = h.scope == kScopeVector, wide = h.slots != kHeldSlots;
    if (n <= h.slots) return kHoldAll;
    if (h.whole && (wide ? 2 * n <= 3 * h.slots : group > 16 && 8 * n < (4 * group > h.slots ? 10 : 9) * h.slots)) return kHoldNone;
    if (vec ? group <= held_small(h) : 4 * h.small_tiles >= 3 * h.tiles) return kHoldAll;
    if (wide) return 4 * group <= h.slots && n <= 4 * h.slots ? kHoldAll : kHoldNone;
    const long long over_half = (vec ? 1ll : h.over_half) * nodes;   // (a vector that comes here is)
    if (n <= 2 * h.slots && (over_half <= 2 || !(vec || h.whole))) return kHoldAll;
  }
  return h.scope == kScopeLayer && h.small_tiles * nodes >= kHeldSmallLeast && 5 * h.small_tiles >= h.tiles ? kHoldSmall : kHoldNone;
}

}  // namespace qoda
