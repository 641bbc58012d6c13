// Instantiations of the time-blocked gather on LDS tiles.
#include "kernels_tb2d.hpp"

namespace stencil {

template <typename T, int R, bool BOX, int TS>
static Kernel tiles(int64_t items) {
  return kernel_of<tb2d_dma_kernel<T, R, BOX, TS>, tb2d_dma_batch<T, R, BOX, TS>>(items);
}

// steps 2 .. 4, or 2 .. 3 at order 4
template <typename T, int R, bool BOX>
static Kernel tiles_of(int steps, int64_t items) {
  if (steps == 2) return tiles<T, R, BOX, 2>(items);
  if constexpr (R < 4) {
    if (steps == 4) return tiles<T, R, BOX, 4>(items);
  }
  return tiles<T, R, BOX, 3>(items);
}

template <>
Kernel tb2d_dma<float, true>(int R, int steps, int64_t items, bool) {
  return R == 3 ? tiles_of<float, 3, true>(steps, items) : tiles_of<float, 4, true>(steps, items);
}

template <>
Kernel tb2d_dma<float, false>(int R, int steps, int64_t items, bool) {
  return R == 2   ? tiles_of<float, 2, false>(steps, items)
         : R == 3 ? tiles_of<float, 3, false>(steps, items)
                  : tiles_of<float, 4, false>(steps, items);
}

template <int R, bool BOX, int TS>
static Kernel small(int64_t items) {
  return kernel_of<tb2d_dma_kernel<double, R, BOX, TS, kTbSmallRows>>(items);
}

template <bool BOX>
static Kernel order2(int steps, int64_t items, bool small_tiles) {
  if (!small_tiles) return tiles_of<double, 2, BOX>(steps, items);
  if (steps == 2) return small<2, BOX, 2>(items);
  if (steps == 3) return small<2, BOX, 3>(items);
  return small<2, BOX, 4>(items);
}

template <>
Kernel tb2d_dma<double, true>(int R, int steps, int64_t items, bool small_tiles) {
  if (R == 2) return order2<true>(steps, items, small_tiles);
  return small_tiles ? small<4, true, 2>(items) : tiles<double, 4, true, 2>(items);
}

Kernel tb2d_any_box4(int64_t items, bool small_tiles) {
  return small_tiles ? kernel_of<tb2d_dma_kernel<double, 4, true, 2, kTbSmallRows, true>>(items)
                     : kernel_of<tb2d_dma_kernel<double, 4, true, 2, 0, true>>(items);
}

template <>
Kernel tb2d_dma<double, false>(int R, int steps, int64_t items, bool small_tiles) {
  if (R == 2) return order2<false>(steps, items, small_tiles);
  if (R == 3) return small_tiles ? small<3, false, 2>(items) : tiles<double, 3, false, 2>(items);
  return small_tiles ? small<4, false, 2>(items) : tiles<double, 4, false, 2>(items);
}

}  // namespace stencil
