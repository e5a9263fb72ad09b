// Instantiations of the row-strip 3x3 convolution kernel for bf16 data.
#include "conv_rows_kernel.hpp"

namespace cprune {

int launch_conv_rows_bf16(int id, dim3 grid, hipStream_t s, const RowsArgs& a) { return launch_rows<__bf16>(id, grid, s, a); }

}  // namespace cprune
