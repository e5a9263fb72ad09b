// Instantiations of the fp32 1x1 kernel on three 16-bit parts.
#include "conv_pw3_kernel.hpp"

namespace cprune {

int launch_conv_pw3_f32(int id, dim3 grid, hipStream_t s, const Pw3Args& a) {
  return launch_pw3<float>(id, grid, s, a);
}

}  // namespace cprune
