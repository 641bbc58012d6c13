// Register-streaming 2D gather: F32 box stencils.
#include "kernels_rs2d_inst.hpp"

namespace stencil {

template Kernel rs2d_of<float, true>(int R, int NC, int64_t items);
template Kernel rs2d_one<float, true>(int R, int64_t items);

}  // namespace stencil
