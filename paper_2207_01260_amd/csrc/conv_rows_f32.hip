// Instantiations of the row-strip 3x3 convolution kernel for fp32 data.
#include "conv_rows_kernel.hpp"

namespace cprune {

int launch_conv_rows_f32(int id, dim3 grid, hipStream_t s, const RowsArgs& a) { return launch_rows3<float>(id, grid, s, a); }

}  // namespace cprune
