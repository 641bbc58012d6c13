// Instantiations of the time-blocked gather on LDS tiles.
#include "kernels_tb2d.hpp"

namespace stencil {

template <typename T, int R, bool BOX, int TS, int TM = 0>
static Kernel tiles(int64_t items) {
  return kernel_of<tb2d_dma_kernel<T, R, BOX, TS, TM>>(items);
}

template <>
Kernel tb2d_dma<float, true>(int R, int steps, int64_t items, bool) {
  if (R == 3) {
    if (steps == 2) return tiles<float, 3, true, 2>(items);
    if (steps == 3) return tiles<float, 3, true, 3>(items);
    return tiles<float, 3, true, 4>(items);
  }
  return steps == 2 ? tiles<float, 4, true, 2>(items) : tiles<float, 4, true, 3>(items);
}

template <>
Kernel tb2d_dma<float, false>(int, int steps, int64_t items, bool) {
  return steps == 2 ? tiles<float, 4, false, 2>(items) : tiles<float, 4, false, 3>(items);
}

template <bool BOX, int TS>
static Kernel order2_of(int64_t items, bool small_tiles) {
  return small_tiles ? tiles<double, 2, BOX, TS, kTbSmallRows>(items) : tiles<double, 2, BOX, TS>(items);
}

template <bool BOX>
static Kernel order2(int steps, int64_t items, bool small_tiles) {
  if (steps == 2) return order2_of<BOX, 2>(items, small_tiles);
  if (steps == 3) return order2_of<BOX, 3>(items, small_tiles);
  return order2_of<BOX, 4>(items, small_tiles);
}

template <>
Kernel tb2d_dma<double, true>(int R, int steps, int64_t items, bool small_tiles) {
  if (R == 2) return order2<true>(steps, items, small_tiles);
  return small_tiles ? tiles<double, 4, true, 2, kTbSmallRows>(items) : tiles<double, 4, true, 2>(items);
}

template <>
Kernel tb2d_dma<double, false>(int R, int steps, int64_t items, bool small_tiles) {
  if (R == 2) return order2<false>(steps, items, small_tiles);
  return small_tiles ? tiles<double, 4, false, 2, kTbSmallRows>(items) : tiles<double, 4, false, 2>(items);
}

}  // namespace stencil
