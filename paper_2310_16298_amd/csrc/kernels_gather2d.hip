// Instantiations of the 2D gather-form baseline kernel.
#include "dma2d.hpp"
#include "kernels_2d.hpp"
#include "kernels_rs2d.hpp"
#include "launch.hpp"
#include "plan.hpp"

namespace stencil {

// Where the register-streaming walk (one step, two columns per lane) beats the
// LDS windows: on every grid that cannot take direct-to-LDS windows (1021 x 1531,
// FP32 stars 14.6-22 -> 5.5-6.9 us; 75^2 17-21 -> 3.6-7.5), and on those that can
// while both buffers stay in the last-level cache, its shorter latency and
// lack of barriers (us, windows / rows: FP32 five-point star 512^2 5.9 / 3.5, 2048^2
// 10.2 / 7.6, 4096^2 22.8 / 22.8, 6144^2 50 / 68; order-3 star 2048^2 11.8 / 9.7, 5120^2
// 38.5 / 34.6, 6144^2 60 / 72; FP64 five-point star 2048^2 14.7 / 12.9, 4096^2 41.6 /
// 42.6; order-4 star 4096^2 53 / 46).  Boxes of order 3 at any size, their FMAs
// bound them (8192^2: FP32 141 / 134, FP64 319 / 223); order 4 FP32 apart from the
// sizes where the 8-row fill is long against the chunks (512^2 9.0 / 8.8, 1024^2
// 8.9 / 11.2, 2048^2 20.1 / 18.9, 8192^2 201 / 175); order 4 FP64 never (24 / 29).
template <typename T, int R, bool BOX>
static bool row_walk_better(const KArgs& a) {
  if (a.d1 < 2) return false;  // a lane's two columns
  if (!dma2d_ok(a)) return true;
  const int64_t pts = a.d0 * a.d1;
  if (BOX && R == 4) return sizeof(T) == 4 && (pts < 500000 || pts > 2500000);
  if (BOX && R == 3) return true;
  return pts * (int64_t)sizeof(T) <= (R <= 2 ? 68000000 : 136000000);
}

template <typename T, int R, bool BOX>
static Kernel pick_gather2d(KArgs& a, int32_t chunk) {
  constexpr int TN = Gather2DDma<T>::TN;
  if (row_walk_better<T, R, BOX>(a)) {
    const bool many = a.share > 0;
    RsCut c = rs_cut(a, R, BOX, (int)sizeof(T), 1, 2, many ? a.share : kRsWaves, many);
    if (chunk > 0) {
      c.ch = chunk < a.d0 ? chunk : a.d0;
      c.chunks = (a.d0 + c.ch - 1) / c.ch;
    }
    if (rs_columns_ok(a, 2, c)) {
      a.steps = 1;
      a.tiles1 = (int32_t)c.strips;
      a.chunk = (int32_t)c.ch;
      a.nchunks = (int32_t)c.chunks;
      a.variant = 2 * R + (BOX ? 1 : 0);
      Kernel k = rs2d_one<T, BOX>(R, (c.strips * c.chunks + 3) / 4);
      rs2d_one_merge<T>(&k);
      return k;
    }
  }
  // FP32 grids at most one 64-column tile wide: the 64 x 64 tiled kernel
  // (a 256-column window would leave three quarters of its lanes idle)
  if (dma2d_ok(a) && !(sizeof(T) == 4 && a.d1 <= kTile2D))
    return kernel_of<gather2d_dma_kernel<T, R, BOX>, gather2d_dma_batch<T, R, BOX>>(
        strip_grid(a, TN, kDmaBM, 1024, dma_chunk(a, TN, R, BOX, chunk)));
  return kernel_of<gather2d_kernel<T, R, BOX>, gather2d_batch<T, R, BOX>>(strip_grid(a, kTile2D, kTile2D, 2048, chunk));
}

template <typename T, bool BOX>
static Picker pick(int R) {
  switch (R) {
    case 1: return pick_gather2d<T, 1, BOX>;
    case 2: return pick_gather2d<T, 2, BOX>;
    case 3: return pick_gather2d<T, 3, BOX>;
    case 4: return pick_gather2d<T, 4, BOX>;
  }
  return nullptr;
}

Picker find_gather2d(int dtype, int R, bool box) {
  if (dtype == STENCIL_F64) return box ? pick<double, true>(R) : pick<double, false>(R);
  return box ? pick<float, true>(R) : pick<float, false>(R);
}

}  // namespace stencil
