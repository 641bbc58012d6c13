// Register-streaming 2D gather, one step: the batched kernel of all F64 stencils.
#include "kernels_rs2d.hpp"

namespace stencil {

template <>
void rs2d_one_merge<double>(Kernel* k) {
  merge_into<rs2d_one_merged<double>>(k);
}

}  // namespace stencil
