// Instantiations of one (type, shape) of the 3D row gather.
#pragma once

#include "kernels_rows3d.hpp"

namespace stencil {

template <typename T, bool BOX, int R, int NC, bool TALL>
static Kernel rows3d_shape(int64_t items) {
  constexpr int J = rows3d_j((int)sizeof(T), R, NC, TALL);
  // the cuts that a grid of a batch takes
  if constexpr (J == 4 ? NC != 2 || (BOX && R >= 3) : NC != 1)
    return kernel_of<rows3d_kernel<T, R, BOX, NC, J>, rows3d_batch<T, R, BOX, NC, J>>(items);
  else
    return kernel_of<rows3d_kernel<T, R, BOX, NC, J>>(items);
}

template <typename T, bool BOX, int R>
static Kernel rows3d_order(int NC, int J, int64_t items) {
  switch (NC) {
    case 1: return J == 4 ? rows3d_shape<T, BOX, R, 1, true>(items) : rows3d_shape<T, BOX, R, 1, false>(items);
    case 2: return rows3d_shape<T, BOX, R, 2, false>(items);
    case 4: return rows3d_shape<T, BOX, R, 4, false>(items);
  }
  return Kernel{};
}

template <typename T, bool BOX>
Kernel rows3d_of(int R, int NC, int J, int64_t items) {
  switch (R) {
    case 1: return rows3d_order<T, BOX, 1>(NC, J, items);
    case 2: return rows3d_order<T, BOX, 2>(NC, J, items);
    case 3: return rows3d_order<T, BOX, 3>(NC, J, items);
    case 4: return rows3d_order<T, BOX, 4>(NC, J, items);
  }
  return Kernel{};
}

}  // namespace stencil
