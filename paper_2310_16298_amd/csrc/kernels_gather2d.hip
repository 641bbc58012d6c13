// Instantiations of the 2D gather-form baseline kernel.
#include "dma2d.hpp"
#include "kernels_2d.hpp"
#include "kernels_rs2d.hpp"
#include "launch.hpp"
#include "plan.hpp"

namespace stencil {

// Where the register-streaming walk (one step, two columns per lane) beats the
// LDS windows: on every grid that cannot take direct-to-LDS windows (1021 x 1531,
// FP32 stars 14.6-22 -> 5.5-6.9 us; 75^2 17-21 -> 3.6-7.5), on FP32 grids of one
// 64-column tile, and by the rules below, whose figures are us, windows / rows.
//
// A periodic grid alone: while both buffers stay in the last-level cache, the
// walk's shorter latency and lack of barriers (FP32 five-point star 512^2 5.9 / 3.5, 2048^2
// 10.2 / 7.6, 4096^2 22.8 / 22.8, 6144^2 50 / 68; order-3 star 2048^2 11.8 / 9.7, 5120^2
// 38.5 / 34.6, 6144^2 60 / 72; FP64 five-point star 2048^2 14.7 / 12.9, 4096^2 41.6 /
// 42.6; order-4 star 4096^2 53 / 46).  Boxes of order 3 at any size, their FMAs
// bound them (8192^2: FP32 141 / 134, FP64 319 / 223); order 4 FP32 apart from the
// sizes where the 8-row fill is long against the chunks (512^2 9.0 / 8.8, 640^2 8.5 /
// 9.1, 1024^2 8.9 / 11.2, 2048^2 20.1 / 18.9, 8192^2 201 / 175); order 4 FP64 never (24 / 29).
template <typename T, int R, bool BOX>
static bool walk_periodic(const KArgs& a) {
  const int64_t pts = a.d0 * a.d1;
  if (R == 4 && a.d0 >= 16 && a.d1 > 64 * a.d0) return false;  // 24 x 8448: FP32 box 8.6 / 9.4, FP64 star 6.5 / 7.3
  if (BOX && R == 4) return sizeof(T) == 4 && (pts < 400000 || pts > 2500000);
  if (BOX && R == 3) return true;
  return pts * (int64_t)sizeof(T) <= (R <= 2 ? 68000000 : 136000000);
}

// A zero-halo grid alone: its windows do not wrap and are staged 1.2-1.6 times as fast
// as periodic ones, so below a size the walk wins only where its waves read few
// rows, its fill of 2R included (rounded up to 4): FP32 five-point star 512^2 3.7 / 3.1, 2048^2
// 7.1 / 7.2, 2560^2 10.2 / 11.3, order-2 box 768^2 4.8 / 4.2, 1024^2 (12 rows) 5.1 / 5.5, order-3 star
// 640^2 4.3 / 4.0, 768^2 4.4 / 4.7, 1280^2 5.2 / 6.0, order-3 box 1024^2 5.9 / 6.9, 2048^2 13.1 / 13.2, order-4
// star 512^2 4.1 / 4.8, 2048^2 9.1 / 10.3, 2560^2 13.8 / 13.1, box 512^2 6.2 / 8.4, 2048^2 16.5 / 18.2,
// 2560^2 25.9 / 22.6; FP64 27-point box 2048^2 13.4 / 12.8, 2560^2 18.3 / 19.7, order-2 box 1024^2
// 5.9 / 6.5, 1280^2 8.9 / 7.1, order-3 box 256^2 5.5 / 4.6, 512^2 5.6 / 6.1, 1280^2 13.5 / 11.0, star 768^2
// 5.2 / 5.5, 1280^2 9.0 / 6.8, order-4 star 64^2 3.6 / 4.9, 1024^2 5.8 / 7.8, 1280^2 9.1 / 7.8.  Few rows and
// many columns leave chunks of a row (24 x 8448: FP64 order-2 star 3.9 / 5.1, FP32 order-3
// star 4.2 / 4.5, but 3 x 100000 FP64 order-2 star 5.6 / 4.8); one strip of many rows leaves
// the windows too few items (40000 x 8: FP64 order-3 box 25 / 15, order-4 star 15 / 9.8).
template <typename T, int R, bool BOX>
static bool walk_zero_halo(const KArgs& a, const RsCut& c) {
  constexpr bool F32 = sizeof(T) == 4;
  const int64_t pts = a.d0 * a.d1, bytes = pts * (int64_t)sizeof(T);
  if (BOX && R == 4 && !F32) return false;
  if (R >= 2 && a.d0 >= 16 && a.d1 > 64 * a.d0) return false;
  const bool tall = a.d1 <= 64 && a.d0 > 10000;
  constexpr double kFewRowsBelow[2][5] = {{0, 0, 1.3e6, BOX ? 2.0e6 : 5.0e6, 5.0e6}, {0, 0, 1.3e6, 1.1e6, 1.2e6}};
  const int64_t rows = (2 * R + c.ch + 3) / 4 * 4;
  if (rows >= 12 && !tall && (double)pts < kFewRowsBelow[F32 ? 0 : 1][R]) return false;
  if (!F32 && BOX && R == 3 && a.d0 >= 16 && !tall && pts >= 100000 && pts < 1100000) return false;
  if (BOX && R >= 3) return true;
  if (R == 1) return bytes <= (F32 ? (BOX ? 68000000 : 17000000) : (BOX ? 40000000 : 68000000));
  return bytes <= (R == 2 ? 68000000 : 136000000);
}

// One of several grids of one stencil in a launch of their own: by the points of
// all of them, which say how many rounds of waves hide the walk's chain of row
// loads (us a step: zero halo, 16 grids of 256^2: FP32 five-point star 5.2 / 7.2, order-4 star
// 5.8 / 9.0, FP64 order-3 star 7.8 / 9.8; 200: 23 / 23, 29 / 26, 56 / 41; 64 of 256^2 FP32 9-point box
// 9.5 / 10.9, FP64 18 / 16; 12 of 1024^2 FP32 order-4 box 46 / 42, 200 of 256^2 49 / 58; one strip of
// up to 128 columns, 16 grids of 128^2: FP32 order-2 box 5.6 / 5.5, order-3 6.3 / 7.4, 256: 21 / 10.5,
// 22 / 14; periodic: 16 of 256^2 FP32 order-4 box 10.4 / 14, order-2 box 8.0 / 8.2, FP64 order-3 box
// 11.4 / 13.4; two of 1024^2 FP32 order-4 star 9.4 / 10.6).
template <typename T, int R, bool BOX>
static bool walk_many(const KArgs& a) {
  constexpr bool F32 = sizeof(T) == 4;
  if (BOX && R == 4 && !F32) return false;
  const double total = (double)a.d0 * (double)a.d1 * 2048.0 / a.share;
  if (a.periodic) {
    const bool few = total >= 5.0e5 && total < (F32 ? (BOX && R == 4 ? 4.5e6 : 3.0e6) : 2.0e6);
    return !(R >= 3 && a.d1 >= 128 + (F32 ? 1 : 0) && few);
  }
  if (a.d1 <= 128) return (F32 && R <= 2) || total >= 1.0e6;
  return total >= (F32 ? (BOX && R == 4 ? 1.6e7 : BOX && R == 2 ? 6.0e6 : 1.0e7) : 2.5e6);
}

// chunk > 0: rows per item asked for.  The walk goes through them one by one, and wins
// on periodic grids only (512^2, 64 rows: FP32 order-2 star zero halo 9.5 / 14,
// periodic 20 / 14; order-4 box 18 / 31, 31 / 31).
// Beside other stencils of its type (kinds > 1) the walk shares their launch, and among
// more than three classes it fills the chip with theirs (104 mixed FP32 grids, 3 steps,
// windows / walk: 181 / 154 us).
template <typename T, int R, bool BOX>
static bool row_walk_better(const KArgs& a, int32_t chunk, const RsCut& c) {
  if (a.d1 < 2) return false;  // a lane's two columns
  if (!dma2d_ok(a)) return true;
  if (sizeof(T) == 4 && a.d1 <= kTile2D) return chunk <= 16;
  if (chunk > 0) return a.periodic && !(BOX && R == 4) && walk_periodic<T, R, BOX>(a);
  if (a.share > 0 && a.kinds < 2) return walk_periodic<T, R, BOX>(a) && walk_many<T, R, BOX>(a);
  return a.periodic || a.share > 0 ? walk_periodic<T, R, BOX>(a) : walk_zero_halo<T, R, BOX>(a, c);
}

template <typename T, int R, bool BOX>
static Kernel pick_gather2d(KArgs& a, int32_t chunk) {
  constexpr int TN = Gather2DDma<T>::TN;
  const bool many = a.share > 0;
  RsCut c = rs_cut(a, R, BOX, (int)sizeof(T), 1, 2, many ? a.share : kRsWaves, many);
  if (row_walk_better<T, R, BOX>(a, chunk, c)) {
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
