// The integer rules of the split kernel: its variants, the order of its reduction, and which packed weights a wavefront
// asks for.  Plain C++, shared by the kernel, the host that packs and launches, and a host program that walks every load.
#pragma once

#ifdef __HIPCC__
#define CPRUNE_HD __host__ __device__ __forceinline__
#else
#define CPRUNE_HD inline
#endif

// Variants: id, wavefronts along filters / pixels / rounds, 16-filter and 16-pixel blocks per wavefront, staging
// items per thread (what patch the pixel block may have: at most 64 * nib pixels)
#define CPRUNE_SPLIT_LIST(X) \
  X(0, 2, 2, 1, 2, 4, 4)  \
  X(1, 2, 2, 1, 2, 2, 2)  \
  X(2, 4, 1, 1, 1, 4, 2)  \
  X(3, 2, 2, 1, 3, 4, 4)  \
  X(4, 1, 4, 1, 3, 2, 4)  \
  X(5, 1, 4, 1, 2, 2, 4)  \
  X(6, 2, 1, 2, 1, 4, 2)  \
  X(7, 1, 1, 4, 2, 4, 2)  \
  X(8, 1, 1, 4, 2, 2, 2)  \
  X(9, 1, 1, 4, 1, 2, 2) \
  X(10, 2, 2, 1, 1, 2, 5) \
  X(11, 2, 2, 1, 2, 2, 5) \
  X(12, 1, 4, 1, 2, 4, 6)

namespace cprune {

constexpr int kNumSplit = 13;

// Rounds of the whole reduction: full chunks of 32 channels take one per tap, the last chunk as many as its 8-channel
// groups need.
inline int split_rounds(int c, int taps, int* nfull, int* groups_last, int* rounds_last) {
  const int groups = (c + 7) / 8, nf = groups / 4, gl = groups % 4, rl = (taps * gl + 3) / 4;
  if (nfull) *nfull = nf;
  if (groups_last) *groups_last = gl;
  if (rounds_last) *rounds_last = rl;
  return nf * taps + rl;
}

// 16-filter blocks are dealt out evenly, first to the tiles (base each, one more in the first rem) and then to a tile's
// wavefronts: a layer costs what its blocks cost, not what its tiles would hold.
struct SplitShare { int first, count; };
CPRUNE_HD SplitShare split_share(int tile_m, int wm, int waves, int base, int rem) {
  const int tblk = base + (tile_m < rem ? 1 : 0);
  const int q = tblk / waves, r = tblk % waves;
  return SplitShare{tile_m * base + (tile_m < rem ? tile_m : rem) + wm * q + (wm < r ? wm : r), q + (wm < r ? 1 : 0)};
}

// The round whose weights are asked for during round q of a chunk of R rounds that begins at rg0: WK further on, or this
// wavefront's first of the next chunk.
CPRUNE_HD int split_next_round(int q, int wk, int waves_k, int R, int rg0, int taps) {
  return q + waves_k < R ? rg0 + q + waves_k : rg0 + taps + wk;
}

// What is really read: a wavefront without a block, and the request behind the last round, take weights that exist (and
// use none of them).  A weight's address is scalar, and whether the range check of a buffer load counts the scalar part
// is not something to rely on: no load may reach past the packed weights by itself.
CPRUNE_HD int split_weight_block(int blk, int blocks) { return blk < blocks ? blk : blocks - 1; }
CPRUNE_HD int split_weight_round(int rg, int rounds) { return rg < rounds ? rg : rounds - 1; }

}  // namespace cprune
