// Instantiations of the inverted-residual block kernel on three bf16 parts: 3x3 windows.
#include "mbrow3_kernel.hpp"

namespace cprune {

int launch_mbrow3_f32(int stride, int mb, int xh, int low, dim3 grid, int ks, hipStream_t s, const MbArgs& a) {
  return launch_mbrow3<float>(stride, mb, xh, low, grid, ks, s, a);
}

}  // namespace cprune
