// Instantiations of the inverted-residual block kernel for Float16 data.
#include "mbrow_kernel.hpp"

namespace cprune {

int launch_mbrow_f16(int k, int stride, int mb, int xh, int low, dim3 grid, int ks, hipStream_t s, const MbArgs& a) {
  return launch_mbrow<_Float16>(k, stride, mb, xh, low, grid, ks, s, a);
}

}  // namespace cprune
