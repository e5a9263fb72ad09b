// Instantiations of the row-strip kernel for tensors in the boundary's layout, _Float16 data.
#include "conv_rows_nchw_kernel.hpp"

namespace cprune {

int launch_conv_rows_nchw_f16(int id, dim3 grid, hipStream_t s, const RowsArgs& a) {
  return launch_rows_nchw<_Float16>(id, grid, s, a);
}

}  // namespace cprune
