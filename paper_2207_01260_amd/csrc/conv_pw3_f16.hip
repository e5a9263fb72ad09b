// Instantiations of the 1x1 kernel on the 16-bit matrix cores for _Float16 data.
#include "conv_pw3_kernel.hpp"

namespace cprune {

int launch_conv_pw3_f16(int id, dim3 grid, hipStream_t s, const Pw3Args& a) {
  return launch_pw3<_Float16>(id, grid, s, a);
}

}  // namespace cprune
