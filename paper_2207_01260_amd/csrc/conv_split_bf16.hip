// Instantiations of the split convolution kernel for __bf16 data in the boundary's layout.
#include "conv_split_kernel.hpp"

namespace cprune {

int launch_conv_split_bf16(int id, dim3 grid, size_t lds, hipStream_t s, const SplitArgs& a) {
  return launch_split<__bf16, true>(id, grid, lds, s, a);
}

}  // namespace cprune
