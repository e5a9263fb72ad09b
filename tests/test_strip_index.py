"""The strips of the inverted-residual kernel, walked on the host over its own index rules: every strip of a map is its own, on
maps at the edges of the reciprocal the decode multiplies by."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

WALK = r"""
#include "strip_index.hpp"
#include <cstdio>
using namespace cprune;
int main() {
  // columns and rows of strips, groups of images: 14517 x 9245 in strips of 12 columns x 2 rows, its transpose, one long row,
  // one tall column, the largest map of one strip a row, small and odd ones over many images
  const int maps[][3] = {{771, 7259, 1}, {1210, 4623, 1}, {3000000, 1, 2}, {1, 3000000, 2}, {2, 2147483, 1}, {1, 1, 2147483},
                         {3, 5, 40000}, {19, 7, 3001}, {46341, 127, 1}, {7, 1, 11}, {1, 9, 64}, {2, 28, 64}};
  long strips = 0, wrong = 0;
  for (const auto& m : maps) {
    const unsigned mx = strip_magic(m[0]), my = strip_magic(m[1]);
    int strip = 0;
    for (int g = 0; g < m[2]; ++g) for (int y = 0; y < m[1]; ++y) for (int x = 0; x < m[0]; ++x, ++strip, ++strips) {
      const StripAt at = strip_at(strip, m[0], m[1], mx, my);
      if (at.tx != x || at.ty != y || at.group != g) ++wrong;
    }
  }
  std::printf("%ld strips, %ld decoded wrong\n", strips, wrong);
  return wrong != 0;
}
"""


def test_every_strip_decodes_to_its_own_place(tmp_path):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(WALK)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2207_01260_amd", "csrc"), str(src),
                           "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout


# The largest maps of the first-layer kernels (32-bit tensors below 2^31 bytes): blocks across, down, images.  One row of 2.7e8 and
# 1.3e8 pixels in pooled strips of 14 and blocks of 16, rows of 6272 pixels over 85598 images, 2047 x 65536 in blocks of 8 x 16, 290 x 1.8 million in bands.
FIRST_LAYER = "{{9586980, 1, 1}, {8388607, 1, 1}, {224, 1, 85598}, {4096, 256, 1}, {65536, 10, 1}, {1171, 4096, 1}}"


def test_blocks_of_the_largest_first_layers(tmp_path):
    """A multiply-high without a correction puts some of these blocks behind the last image; all first-layer kernels decode by the rule
    that is walked here."""
    for across in (9586980, 8388607):
        assert (across - 1) * -(-2 ** 32 // across) >> 32 == 1
    csrc = os.path.join(ROOT, "paper_2207_01260_amd", "csrc")
    for kernel in ("conv_stem_kernel.hpp", "conv_stem7_kernel.hpp", "conv_stem7_split_kernel.hpp"):
        text = open(os.path.join(csrc, kernel)).read()
        assert "strip_at(" in text and "fast_div" not in text, kernel
    head, tail = WALK.split("const int maps[][3] = ")
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(head + "const int maps[][3] = " + FIRST_LAYER + tail[tail.index(";"):])
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I", csrc, str(src), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
