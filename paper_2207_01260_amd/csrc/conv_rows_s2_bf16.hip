// Instantiations of the stride-2 row-strip kernel for __bf16 data.
#include "conv_rows_s2_kernel.hpp"

namespace cprune {

int launch_conv_rows_s2_bf16(int id, dim3 grid, hipStream_t s, const RowsS2Args& a) {
  return launch_rows_s2<__bf16>(id, grid, s, a);
}

}  // namespace cprune
