// The integer rules of the inverted-residual kernel's strips and of the first-layer kernels' pixel blocks.  Plain C++, shared by the
// kernels, the host that launches them, and a host program that walks every strip of a map.
#pragma once
#include "split_index.hpp"

namespace cprune {

// Which strip a work-group owns: column and row of strips, group of images.
struct StripAt { int tx, ty, group; };

// ceil(2^32 / d), 0 for a divisor of 1
inline unsigned strip_magic(int d) { return d > 1 ? (unsigned)((0x100000000ull + (unsigned)d - 1) / (unsigned)d) : 0u; }

// n / d for any n + d below 2^32.  The product alone is one too large for some n once n * d reaches 2^32 (a map of 14517 x 9245
// pixels has 5.6 million strips, 771 in a row), never more: its excess over n / d is below n / 2^32.
CPRUNE_HD unsigned strip_div(unsigned n, unsigned d, unsigned magic) {
  if (!magic) return n;
  const unsigned q = (unsigned)((unsigned long long)n * magic >> 32);
  return q - (q * d > n ? 1u : 0u);
}

CPRUNE_HD StripAt strip_at(int strip, int tiles_x, int tiles_y, unsigned magic_x, unsigned magic_y) {
  const int rest = (int)strip_div((unsigned)strip, (unsigned)tiles_x, magic_x);
  const int group = (int)strip_div((unsigned)rest, (unsigned)tiles_y, magic_y);
  return StripAt{strip - rest * tiles_x, rest - group * tiles_y, group};
}

}  // namespace cprune
