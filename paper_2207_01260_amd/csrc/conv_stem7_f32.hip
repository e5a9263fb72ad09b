// Instantiations of the fp32 7x7 / stride 2 first-layer kernel.
#include "conv_stem7_split_kernel.hpp"

namespace cprune {

int launch_conv_stem7_f32(int mb, int pool, dim3 grid, hipStream_t s, const StemArgs& a) {
  return launch_stem7_split(mb, pool, grid, s, a);
}

}  // namespace cprune
