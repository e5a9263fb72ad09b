"""The split kernel's weight loads, walked on the host over its own index rules: none may leave the packed weights."""
import os
import subprocess

from paper_2207_01260_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# every tile, wavefront and chunk of every variant on layers at the edges of the 16-filter block, the 8-channel group and
# the 32-channel chunk; the loads of a chunk are those of the kernel's main loop: the next round's during each round
WALK = r"""
#include "split_index.hpp"
#include <cstdio>
using namespace cprune;
struct V { int wm, wn, ks, mb; };
#define ROW(ID, WM, WN, WK, MB, NB, NIB) {WM, WN, WK, MB},
static const V variants[] = {CPRUNE_SPLIT_LIST(ROW)};
int main() {
  const int filters[] = {1, 15, 16, 17, 32, 33, 47, 48, 83, 112, 130, 512};
  const int channels[] = {1, 3, 8, 9, 24, 31, 32, 33, 64, 70, 128};
  const int windows[] = {1, 9, 25, 49};
  long loads = 0, outside = 0, moved = 0, missing = 0;
  for (const V& v : variants) for (int O : filters) for (int C : channels) for (int taps : windows) {
    int nfull, groups_last, rounds_last;
    const int rtot = split_rounds(C, taps, &nfull, &groups_last, &rounds_last);
    const int blocks = (O + 15) / 16, tile = v.wm * v.mb, tiles = (blocks + tile - 1) / tile;
    const int base = blocks / tiles, rem = blocks % tiles;
    int given = 0;
    for (int tm = 0; tm < tiles; ++tm) for (int wm = 0; wm < v.wm; ++wm) {
      const SplitShare s = split_share(tm, wm, v.wm, base, rem);
      if (s.count > v.mb || (s.count && s.first != given)) ++missing;
      given += s.count;
      for (int wk = 0; wk < v.ks; ++wk) {
        auto load = [&](int round, bool used) {
          const int rg = split_weight_round(round, rtot);
          if (used && rg != round) ++moved;
          for (int i = 0; i < (s.count ? s.count : 1); ++i, ++loads) {
            const int blk = split_weight_block(s.first, blocks) + i;
            if (blk < 0 || rg < 0 || (long)blk * rtot + rg >= (long)blocks * rtot) ++outside;
            if (s.count && blk != s.first + i) ++moved;
          }
        };
        load(wk, wk < rtot && wk < (nfull ? taps : rounds_last));
        for (int c = 0; c < nfull + (rounds_last ? 1 : 0); ++c) {
          const int R = c < nfull ? taps : rounds_last, rg0 = c * taps;
          for (int q = wk; q < R; q += v.ks) load(split_next_round(q, wk, v.ks, R, rg0, taps), q + v.ks < R);
        }
      }
    }
    if (given != blocks) ++missing;
  }
  std::printf("%ld loads, %ld outside, %ld real ones moved, %ld shares wrong\n", loads, outside, moved, missing);
  return outside || moved || missing;
}
"""


def test_weight_loads_stay_inside(tmp_path):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(WALK)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2207_01260_amd", "csrc"), str(src),
                           "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout


def test_prune_step_of_evenly_dealt_blocks():
    """The split kernel deals its 16-filter blocks evenly to its tiles, 112 filters on a tile of 96 as 4 + 3 blocks; the
    splits the library reports are what a tile holds.  The pruning step is the same from either box."""
    seen = 0
    for v in range(B.cprune_num_tile_variants()):
        if "conv_split" not in B.cprune_tile_variant_name(v, True, B.F32):
            continue
        tile = B.cprune_tile_variant_info(v)[0] // 16
        for c_out in list(range(1, 1200, 7)) + [16, 48, 64, 96, 97, 112, 128, 512]:
            blocks = -(-c_out // 16)
            tiles = -(-blocks // tile)
            dealt = [tiles, -(-blocks // tiles)]
            assert B.cprune_variant_prune_step(v, c_out) == 16 * B.cprune_lcm_step(dealt, dealt), (v, c_out)
        seen += 1
    assert seen
