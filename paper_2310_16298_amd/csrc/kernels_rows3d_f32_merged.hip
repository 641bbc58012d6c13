// 3D gather on register rows: the batched kernel of all F32 stencils.
#include "kernels_rows3d.hpp"

namespace stencil {

template <>
void rows3d_merge<float>(Kernel* k) {
  merge_into<rows3d_merged<float>>(k);
}

}  // namespace stencil
