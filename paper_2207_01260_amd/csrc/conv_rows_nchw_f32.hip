// Instantiations of the row-strip kernel for tensors in the boundary's layout, float data.
#include "conv_rows_nchw_kernel.hpp"

namespace cprune {

int launch_conv_rows_nchw_f32(int id, dim3 grid, hipStream_t s, const RowsArgs& a) {
  return launch_rows_nchw<float>(id, grid, s, a);
}

}  // namespace cprune
