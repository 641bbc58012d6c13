// Instantiations of one (type, shape) of the register-streaming kernels.
#pragma once

#include "kernels_rs2d.hpp"

namespace stencil {

template <typename T, bool BOX, int R>
static Kernel rs2d_columns(int NC, int64_t items) {
  constexpr int TS = rs2d_steps<T>(R);
  switch (NC) {
    case 1: return kernel_of<rs2d_kernel<T, R, BOX, TS, 1>, rs2d_batch<T, R, BOX, TS, 1>>(items);
    case 2: return kernel_of<rs2d_kernel<T, R, BOX, TS, 2>, rs2d_batch<T, R, BOX, TS, 2>>(items);
    case 4: return kernel_of<rs2d_kernel<T, R, BOX, TS, 4>, rs2d_batch<T, R, BOX, TS, 4>>(items);
  }
  return Kernel{};
}

template <typename T, bool BOX>
Kernel rs2d_of(int R, int NC, int64_t items) {
  switch (R) {
    case 1: return rs2d_columns<T, BOX, 1>(NC, items);
    case 2: return rs2d_columns<T, BOX, 2>(NC, items);
    case 3: return rs2d_columns<T, BOX, 3>(NC, items);
    case 4: return rs2d_columns<T, BOX, 4>(NC, items);
  }
  return Kernel{};
}

template <typename T, bool BOX>
Kernel rs2d_one(int R, int64_t items) {
  switch (R) {
    case 1: return kernel_of<rs2d_kernel<T, 1, BOX, 1, 2>, rs2d_batch<T, 1, BOX, 1, 2>>(items);
    case 2: return kernel_of<rs2d_kernel<T, 2, BOX, 1, 2>, rs2d_batch<T, 2, BOX, 1, 2>>(items);
    case 3: return kernel_of<rs2d_kernel<T, 3, BOX, 1, 2>, rs2d_batch<T, 3, BOX, 1, 2>>(items);
    case 4: return kernel_of<rs2d_kernel<T, 4, BOX, 1, 2>, rs2d_batch<T, 4, BOX, 1, 2>>(items);
  }
  return Kernel{};
}

}  // namespace stencil
