// 3D gather on register rows: the batched kernel of all F64 stencils.
#include "kernels_rows3d.hpp"

namespace stencil {

template <>
void rows3d_merge<double>(Kernel* k) {
  merge_into<rows3d_merged<double>>(k);
}

}  // namespace stencil
