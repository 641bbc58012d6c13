// Register-streaming 2D gather: F64 star stencils.
#include "kernels_rs2d_inst.hpp"

namespace stencil {

template Kernel rs2d_of<double, false>(int R, int NC, int64_t items);
template Kernel rs2d_one<double, false>(int R, int64_t items);

}  // namespace stencil
