// Instantiations of the split convolution kernel for float data, both layouts.
#include "conv_split_kernel.hpp"

namespace cprune {

int launch_conv_split_f32(int id, bool nchw, dim3 grid, size_t lds, hipStream_t s, const SplitArgs& a) {
  return nchw ? launch_split<float, true>(id, grid, lds, s, a) : launch_split<float, false>(id, grid, lds, s, a);
}

}  // namespace cprune
