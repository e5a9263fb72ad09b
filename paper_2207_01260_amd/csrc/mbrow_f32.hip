// Instantiations of the inverted-residual block kernel for float data: 5x5 windows, and more than 96 projection filters.
#include "mbrow_kernel.hpp"

namespace cprune {

int launch_mbrow_f32(int k, int stride, int mb, int xh, int low, dim3 grid, int ks, hipStream_t s, const MbArgs& a) {
  return mbrow_parts(k, mb) ? launch_mbrow3_f32(stride, mb, xh, low, grid, ks, s, a) : launch_mbrow<float>(k, stride, mb, xh, low, grid, ks, s, a);
}

}  // namespace cprune
