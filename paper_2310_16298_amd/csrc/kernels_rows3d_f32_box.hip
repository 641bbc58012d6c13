// 3D gather on register rows: F32 box stencils.
#include "kernels_rows3d_inst.hpp"

namespace stencil {

template Kernel rows3d_of<float, true>(int R, int NC, int J, int64_t items);

}  // namespace stencil
