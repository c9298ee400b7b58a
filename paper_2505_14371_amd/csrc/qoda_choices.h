// Which form of a kernel a launch takes, by the sizes of the launch.  Host code only, and apart from the kernels, so that a test
// without a GPU can hold every choice against what was measured on both sides of it.
#pragma once

#include "qoda_kernels.h"

namespace qoda {

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

}  // namespace qoda
