// Kernel choice of the time-blocked 2D gather.
#include <algorithm>
#include <type_traits>

#include "kernels_rs2d.hpp"
#include "kernels_tb2d.hpp"
#include "launch.hpp"
#include "plan.hpp"

namespace stencil {

// The grids of one batch class (same type, order, shape and step count) share
// one kernel, so one NC: the one with the shortest class time, its work over
// the full chip or its longest wave.  index[k]: grid k's place in share.
int rs2d_batch_cut(const std::vector<const Resolved*>& grids, const int* share, const int32_t* index) {
  int columns = 0;
  double best = 0.0;
  for (int NC = 1; NC <= 4; NC *= 2) {
    double work = 0.0, longest = 0.0;
    bool ok = true;
    for (size_t k = 0; k < grids.size() && ok; ++k) {
      const Resolved& g = *grids[k];
      const RsCut c = rs_cut(g.args, g.info.radius, g.info.shape != STENCIL_STAR, g.info.dtype == STENCIL_F64 ? 8 : 4,
                             g.time_block, NC, share[index[k]], true);
      ok = rs_columns_ok(g.args, NC, c);
      const double wave = c.wave + 1500.0;  // finding the grid, its weights, the first rows
      work += wave * (double)(c.strips * c.chunks);
      longest = std::max(longest, wave);
    }
    const double t = std::max(work / kRsWaves, longest);
    if (!ok || (columns && t >= best)) continue;
    columns = NC;
    best = t;
  }
  return columns ? columns : 1;
}

// Cuts the grid (MANY: for the NC in a.columns and the share of the waves in
// a.share) and returns NC.
template <typename T, int R, bool BOX, bool MANY>
static int cut_rs2d(KArgs& a) {
  const KArgs in = a;
  int best = 0;
  double best_time = 0.0;
  for (int NC = 1; NC <= 4; NC *= 2) {
    if (MANY && NC != in.columns) continue;
    const int64_t waves_for = MANY ? in.share : kRsWaves;
    const RsCut c = rs_cut(in, R, BOX, (int)sizeof(T), in.steps, NC, waves_for, MANY);
    const double waves = (double)(c.strips * c.chunks);
    const double t = c.wave * std::max(1.0, waves / (double)waves_for);
    if (!rs_columns_ok(in, NC, c) || (best && t >= best_time)) continue;
    best = NC;
    best_time = t;
    a.tiles1 = (int32_t)c.strips;
    a.chunk = (int32_t)c.ch;
    a.nchunks = (int32_t)c.chunks;
  }
  return best;
}

// Few rows and many columns: the walk's chunks shrink to a row or two there, each
// with a pipeline fill of its own.
static bool wide(const KArgs& a) { return a.d0 >= 16 && a.d1 > 64 * a.d0; }

// The LDS tiles (direct-to-LDS windows of 64 x 64, FP64 32 x 64) for a grid
// alone that they suit better: orders 2 to 4 on grids in between, where the
// pipeline's fill of 2 R steps rows is long against the chunks of a full
// chip, and (FP64) its latency against 16-row tiles.  The tiles stage a zero halo
// faster than a periodic one, whose windows wrap.  us per launch, LDS tiles
// / register streaming, periodic: FP32 order-4 box 512^2 13.3 / 12.0, 1024^2 13.8 / 17.4,
// 2048^2 27 / 37, 4096^2 81 / 94, 6144^2 184 / 174; order-4 star 700^2 11.9 / 10.6,
// 1024^2 12.0 / 12.6, 1500^2 14.9 / 16.3, 2048^2 22.2 / 21.3; order-3 box 700^2 20.5 /
// 19.0, 1024^2 20.6 / 23.4, 1500^2 34.9 / 35.2, 2500^2 69 / 62; FP64 order-4 star
// 256^2 7.3 / 7.1, 512^2 7.1 / 8.2, 1024^2 11.7 / 11.9, 1500^2 17.5 / 16.0; order-4 box
// 64^2 10.8 / 12.5, 512^2 9.9 / 21.5, 2048^2 53 / 68, 4096^2 190 / 172.  Zero halo: FP32
// order-4 box 384^2 12.2 / 11.0, 512^2 12.2 / 12.6, 640^2 12.6 / 13.8, 24 x 8448 12.0 / 13.0;
// order-4 star 640^2 10.7 / 10.8, 768^2 10.7 / 11.4, 2048^2 20.0 / 22.2, 2560^2 29.8 / 27.3; order-3
// star 768^2 12.2 / 11.2, 1024^2 12.5 / 13.2, 1280^2 14.9 / 15.2; FP64 order-4 star 64^2 5.6 / 6.8,
// 256^2 5.9 / 7.8, 1280^2 12.6 / 13.6, 2048^2 23.1 / 21.6; order-3 star 384^2 6.2 / 6.0, 512^2 6.4 / 6.6,
// 24 x 8448 6.8 / 7.6, 768^2 9.3 / 7.6, 40000 x 8 15 / 11.  FP64 order 2, zero halo: box 256^2 8.5 / 9.1,
// 512^2 8.8 / 10.4, 48 x 4224 8.8 / 10.8, 768^2 14.2 / 11.6, star 384^2 6.8 / 7.0, 512^2 6.9 /
// 7.8, 768^2 10.6 / 8.9; periodic: box 48 x 4224 10.0 / 11.1, 512^2 9.9 / 10.7, star 24 x 8448
// 8.4 / 9.3, 48 x 4224 9.1 / 9.6, 128 x 2048 9.3 / 9.2, 512^2 9.0 / 8.4.
template <typename T, int R, bool BOX>
static bool lds_tiles_better(const KArgs& a) {
  const int64_t pts = a.d0 * a.d1;
  if constexpr (sizeof(T) == 4) {
    if (BOX && R == 4)
      return pts < 32000000 && pts >= (a.periodic || a.d0 < 16 ? 450000 : wide(a) ? 100000 : 250000);
    if (R == 4) return a.periodic ? pts >= 800000 && pts < 3000000 : pts >= 500000 && pts < 6000000;
    if (BOX && R == 3) return pts >= 800000 && pts < 2400000;
    return R == 3 && !a.periodic && a.d1 > 64 && pts >= 800000 && pts < 1700000;
  } else {
    if (BOX && R == 4) return pts < 10000000;
    if (R == 4) return a.periodic ? pts >= 100000 && pts < 1100000 : pts < 2000000;
    if (R == 3) return !BOX && !a.periodic && a.d0 >= 16 && a.d1 > 64 && pts > 200000 && pts < 450000;
    return R == 2 && pts < 480000 && (a.periodic ? pts >= 180000 && (BOX || wide(a)) : pts >= 45000);
  }
}

// Ragged extents or misaligned buffers: the FP64 order-4 box, whose walk is slowest to
// fill, on tiles staged by element.  us a step at two steps a launch, tiles / walk,
// zero halo: 64 x 66 4.7 / 6.1, 300 x 201 4.8 / 9.4, 17 x 5001 4.7 / 10.0, 1021 x 1531
// 13.5 / 15.8, 2001 x 2003 31 / 35, 3001 x 3003 65 / 59, 40000 x 5 18.0 / 17.3; periodic: 64 x 66 7.4 /
// 6.2, 300 x 65 7.1 / 6.2, 300 x 201 6.6 / 9.4, 3000 x 9 6.6 / 9.4, 901 x 777 10.5 / 12.7, 1021 x 1531
// 15.7 / 15.6, 40000 x 5 27 / 17.
template <typename T, int R, bool BOX>
static bool any_tiles_better(const KArgs& a) {
  if (sizeof(T) == 4 || R != 4 || !BOX || a.d1 <= 8) return false;
  const int64_t pts = a.d0 * a.d1;
  return a.periodic ? pts >= 25000 && pts < 1500000 : pts < 5000000;
}

// Among many grids the tiles win where all of the class's grids together are about
// one round of waves: the walk's chunks are as short as their fill then, and
// there are too few of them to hide it (us a step, tiles / walk, zero halo: 16 FP32 grids
// of 256^2, stars r = 2..4 3.1 / 3.5, 3.7 / 4.7, 4.5 / 6.1, boxes r = 3, 4 6.1 / 7.1, 8.3 / 10.7;
// 64 of 256^2 6.8 / 4.3, 11.7 / 6.3, 14.0 / 8.3, 21.3 / 13.3, 27.9 / 20.1; two FP64 ones of 512^2,
// stars 2.7 / 3.4, 4.6 / 5.8, 4.4 / 6.8, order-2 box 3.3 / 4.1; eight 5.8 / 4.6, 9.6 / 7.3, 9.1 / 9.2,
// 7.8 / 5.9; 50 FP32 order-4 stars of 96^2 4.1 / 4.6, four of 128^2 3.8 / 3.8).  Beside other
// classes (a.kinds in all) their walks fill the chip, and a class cut in two is more
// launches: 16 FP32 grids of 256^2 of 2 / 3 / 4 / 8 stencils 13.5 / 14.7, 17.2 / 16.4, 22.5 / 20.7, 30 /
// 26.5; two of 512^2 10.5 / 12.4, 10.9 / 13.4 (3), 20.7 / 19.3 (8); the 120 mixed FP64 grids, 10 steps,
// 606 / 565.
template <typename T, int R, bool BOX>
static bool lds_tiles_better_many(const KArgs& a) {
  const double total = (double)a.d0 * (double)a.d1 * 2048.0 / a.share;  // points of the class
  if (a.kinds > 3 || total >= 1.6e6 || a.kinds * total >= 3.0e6) return false;
  if constexpr (sizeof(T) == 4) {
    if (R == 4) return a.d1 > 64 ? total >= (a.periodic ? 5.0e5 : 4.0e5) : !BOX && total >= 7.0e5;
    return a.d1 > 64 && total >= (R == 3 && !BOX && !a.periodic ? 5.0e5 : 7.0e5);
  } else {
    if (BOX && R == 4) return false;
    if (R == 4 && !a.periodic) return true;
    if (R == 4) return a.d1 >= 256 && total >= 5.0e5;
    return a.d1 >= 512 && total >= 5.0e5 && total < 1.0e6;
  }
}

// MANY: the grid is one of many in a batched launch.
template <typename T, int R, bool BOX, bool MANY = false>
static Kernel pick_tb2d(KArgs& a, int32_t chunk) {
  // a launch of one step (the remainder of a run): the one-step gather
  if (a.steps <= 1) return find_gather2d(std::is_same<T, double>::value ? STENCIL_F64 : STENCIL_F32, R, BOX)(a, chunk);
  if constexpr (tb2d_dma_built<T>(R, BOX)) {
    const bool fast = tb2d_fast<T>(a) && a.zeros != nullptr;
    if (fast ? (MANY ? lds_tiles_better_many<T, R, BOX>(a) : lds_tiles_better<T, R, BOX>(a))
             : (!MANY && any_tiles_better<T, R, BOX>(a))) {
      int TM = TbDmaShape<T, R, 2>::TM;
      a.tiles1 = (int32_t)((a.d1 + 63) / 64);
      // FP64 grids of fewer tiles than CUs (launch-bound: 512^2 has 128) take
      // 16-row tiles, twice the workgroups at the cost of more halo rows
      const bool small =
          !MANY && !std::is_same<T, float>::value && (int64_t)((a.d0 + TM - 1) / TM) * a.tiles1 < 256;
      if (small) TM = kTbSmallRows;
      a.tiles0 = (int32_t)((a.d0 + TM - 1) / TM);
      const int64_t items = (int64_t)a.tiles0 * a.tiles1;
      return fast ? tb2d_dma<T, BOX>(R, a.steps, items, small) : tb2d_any_box4(items, small);
    }
  }
  const int NC = cut_rs2d<T, R, BOX, MANY>(a);
  if (NC == 0) return Kernel{};
  return rs2d_of<T, BOX>(R, NC, ((int64_t)a.tiles1 * a.nchunks + 3) / 4);
}

template <typename T, bool BOX, bool MANY>
static Picker pick(int R) {
  switch (R) {
    case 1: return pick_tb2d<T, 1, BOX, MANY>;
    case 2: return pick_tb2d<T, 2, BOX, MANY>;
    case 3: return pick_tb2d<T, 3, BOX, MANY>;
    case 4: return pick_tb2d<T, 4, BOX, MANY>;
  }
  return nullptr;
}

template <bool MANY>
static Picker find(int dtype, int R, bool box) {
  if (dtype == STENCIL_F64) return box ? pick<double, true, MANY>(R) : pick<double, false, MANY>(R);
  return box ? pick<float, true, MANY>(R) : pick<float, false, MANY>(R);
}

Picker find_tb2d(int dtype, int R, bool box) { return find<false>(dtype, R, box); }
Picker find_tb2d_batch(int dtype, int R, bool box) { return find<true>(dtype, R, box); }

int tb2d_max_steps(int dtype, int R) { return dtype == STENCIL_F64 ? rs2d_steps<double>(R) : rs2d_steps<float>(R); }

}  // namespace stencil
