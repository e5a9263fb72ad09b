// Instantiations of the row-strip 3x3 convolution kernel for fp16 data.
#include "conv_rows_kernel.hpp"

namespace cprune {

int launch_conv_rows_f16(int id, dim3 grid, hipStream_t s, const RowsArgs& a) { return launch_rows<_Float16>(id, grid, s, a); }

}  // namespace cprune
