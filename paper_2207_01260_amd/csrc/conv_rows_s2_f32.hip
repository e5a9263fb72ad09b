// Instantiations of the stride-2 row-strip kernel for float data.
#include "conv_rows_s2_kernel.hpp"

namespace cprune {

int launch_conv_rows_s2_f32(int id, dim3 grid, hipStream_t s, const RowsS2Args& a) {
  return launch_rows_s2<float>(id, grid, s, a);
}

}  // namespace cprune
