// 3D gather on register rows: one step, no LDS, no alignment or size demands.
//
// A wave computes J rows of one output plane over a strip of 64 NC columns
// (lane l: columns NC l .. NC l + NC - 1).  It reads, plane by plane, the J + 2R
// input rows around them (a star's planes other than its own: the J rows), takes
// the k neighbours of a row from the lanes beside it by DPP shifts, and adds
// the taps in the order of the tiled gather (planes, then j, then k ascending; a
// star's centre plane: the j arm, then the k arm), so the results agree bit for
// bit.  Rows that several waves read come from the caches: the four waves of a
// workgroup take neighbouring row groups, an XCD a contiguous range of planes.
// Strips overlap by the R columns that go stale on each side.
//
// What bounds it: the FMAs for boxes from order 2, the caches below that.  Against
// the plane-ring kernel, whose chunks of at least 4R planes leave a small
// grid a handful of workgroups and whose ragged windows are staged without
// overlap (us a step, zero halo): 33^3 FP32 order-4 box 364 -> 14, order-1 star 22 ->
// 3.5; 71^3 FP64 order-3 box 211 -> 19; 150^3 FP64 order-4 box 838 -> 177; 203 x 150 x 177
// FP32 order-2 star 63 -> 16, FP64 27-point box 49 -> 21; 256^3 boxes FP32 order 2..4
// 100 / 426 / 810 -> 69 / 167 / 344 (outer products 97 / 237 / 432), FP64 163 / 456 / 1383 ->
// 111 / 231 / 504.
#pragma once

#include <cmath>

#include "dma3d.hpp"
#include "kernels_3d.hpp"
#include "kernels_rs2d.hpp"

namespace stencil {

template <typename T, int R, bool BOX, int NC, int J>
struct Rows3D {
  static constexpr int W = 2 * R + 1, XR = J + 2 * R;
  T acc[J][NC];
  ConstPtr<T> c;
  const T* in;
  uint32_t wcol;          // the lane's first column, wrapped / clamped into the row
  uint32_t N, plane;      // columns; elements of a plane
  uint32_t roff[XR];      // element offset of input row x in its plane (wrapped / clamped)
  bool rok[XR];           // row x lies in the grid (periodic: always)
  bool ok[NC];            // column e lies in the grid (periodic: always)
  bool periodic;

  template <int MODE>
  __device__ __forceinline__ void load_row(const T* pl, int x, T* v) {
    const T* src = pl + roff[x];
    if constexpr (MODE < 2) {
      const RsPack<T, NC> p = *reinterpret_cast<const RsPack<T, NC>*>(src + wcol);
#pragma unroll
      for (int e = 0; e < NC; ++e) v[e] = p.v[e];
    } else {
#pragma unroll
      for (int e = 0; e < NC; ++e) v[e] = src[wcol + e < N ? wcol + e : (periodic ? wcol + e - N : 0u)];
    }
  }

  // zero halo: what lies outside the grid
  template <int MODE>
  __device__ __forceinline__ void mask(int x, T* v) {
    if constexpr (MODE > 0) {
#pragma unroll
      for (int e = 0; e < NC; ++e) v[e] = rok[x] && ok[e] ? v[e] : T(0);
    }
  }

  // columns col - R .. col + NC - 1 + R of a row
  __device__ __forceinline__ void widen(const T* v, T* e) {
    constexpr int HL = (R + NC - 1) / NC;
    T s[NC];
#pragma unroll
    for (int k = 0; k < NC; ++k) e[R + k] = s[k] = v[k];
#pragma unroll
    for (int h = 0; h < HL; ++h)
#pragma unroll
      for (int k = NC - 1; k >= 0; --k) {
        const int at = k - NC * (h + 1);
        if (at < -R) continue;
        s[k] = rs_shift<true>(s[k]);
        e[R + at] = s[k];
      }
#pragma unroll
    for (int k = 0; k < NC; ++k) s[k] = v[k];
#pragma unroll
    for (int h = 0; h < HL; ++h)
#pragma unroll
      for (int k = 0; k < NC; ++k) {
        const int at = k + NC * (h + 1);
        if (at > NC - 1 + R) continue;
        s[k] = rs_shift<false>(s[k]);
        e[R + at] = s[k];
      }
  }

  template <int MODE>
  __device__ __forceinline__ void load_plane(const T* pl, T (*v)[NC]) {
#pragma unroll
    for (int x = 0; x < XR; ++x) load_row<MODE>(pl, x, v[x]);
  }

  // box: the rows v of coefficient plane a
  template <int MODE>
  __device__ __forceinline__ void box_plane(int a, T (*v)[NC]) {
    T w[W * W];
#pragma unroll
    for (int i = 0; i < W * W; ++i) {
      w[i] = vector_weight<T>(c[a * W * W + i]);
    }
#pragma unroll
    for (int x = 0; x < XR; ++x) {
      mask<MODE>(x, v[x]);
      T e[2 * R + NC];
      widen(v[x], e);
#pragma unroll
      for (int p = 0; p < J; ++p) {
        const int b = x - p;
        if (b < 0 || b > 2 * R) continue;
#pragma unroll
        for (int cc = 0; cc < W; ++cc)
#pragma unroll
          for (int k = 0; k < NC; ++k) acc[p][k] = rs_fma(w[b * W + cc], e[cc + k], acc[p][k]);
      }
    }
  }

  // in-plane arms of a star
  template <int MODE>
  __device__ __forceinline__ void star_centre(T (*v)[NC]) {
#pragma unroll
    for (int x = 0; x < XR; ++x) {
      mask<MODE>(x, v[x]);
#pragma unroll
      for (int p = 0; p < J; ++p) {
        const int b = x - p;
        if (b < 0 || b > 2 * R) continue;
        const T w = c[(R * W + b) * W + R];
#pragma unroll
        for (int k = 0; k < NC; ++k) acc[p][k] = rs_fma(w, v[x][k], acc[p][k]);
      }
    }
#pragma unroll
    for (int p = 0; p < J; ++p) {
      T e[2 * R + NC];
      widen(v[p + R], e);
#pragma unroll
      for (int cc = 0; cc < W; ++cc) {
        if (cc == R) continue;
        const T w = c[(R * W + R) * W + cc];
#pragma unroll
        for (int k = 0; k < NC; ++k) acc[p][k] = rs_fma(w, e[cc + k], acc[p][k]);
      }
    }
  }

  // plane o + d of the input, nullptr outside a zero-halo grid
  __device__ __forceinline__ const T* plane_at(int64_t o, int d, int64_t Ni) {
    int64_t g = o + d;
    if (g < 0 || g >= Ni) {
      if (!periodic) return nullptr;
      g %= Ni;
      if (g < 0) g += Ni;
    }
    return in + g * (int64_t)plane;
  }

  template <int MODE>
  __device__ __forceinline__ void point(int64_t o, int64_t Ni) {
#pragma unroll
    for (int p = 0; p < J; ++p)
#pragma unroll
      for (int k = 0; k < NC; ++k) acc[p][k] = T(0);
    const T* own = plane_at(o, 0, Ni);
    if constexpr (BOX) {
      // two planes' rows in turn: one is loaded while the other is added; a
      // plane outside the grid is read as the own one and skipped
      T va[XR][NC], vb[XR][NC];
      const T* pa = plane_at(o, -R, Ni);
      load_plane<MODE>(pa ? pa : own, va);
#pragma unroll 1
      for (int a = 0; a < W; a += 2) {
        const T* pb = a + 1 < W ? plane_at(o, a + 1 - R, Ni) : nullptr;
        load_plane<MODE>(pb ? pb : own, vb);
        if (pa) box_plane<MODE>(a, va);
        if (a + 1 >= W) break;
        pa = plane_at(o, a + 2 - R, Ni);  // a + 2 < W: W is odd
        load_plane<MODE>(pa ? pa : own, va);
        if (pb) box_plane<MODE>(a + 1, vb);
      }
    } else {
      T v[XR][NC], u[W][J][NC];
      load_plane<MODE>(own, v);
      const T* pl[W];
#pragma unroll
      for (int a = 0; a < W; ++a) {
        if (a == R) continue;
        pl[a] = plane_at(o, a - R, Ni);
#pragma unroll
        for (int p = 0; p < J; ++p) load_row<MODE>(pl[a] ? pl[a] : own, p + R, u[a][p]);
      }
#pragma unroll
      for (int a = 0; a < W; ++a) {
        if (a == R) {
          star_centre<MODE>(v);
          continue;
        }
        const T w = pl[a] ? c[(a * W + R) * W + R] : T(0);
#pragma unroll
        for (int p = 0; p < J; ++p) {
          mask<MODE>(p + R, u[a][p]);
#pragma unroll
          for (int k = 0; k < NC; ++k) acc[p][k] = pl[a] ? rs_fma(w, u[a][p][k], acc[p][k]) : acc[p][k];
        }
      }
    }
  }
};

// Work decomposition: a.tiles0 row groups, a.tiles1 strips per plane; pieces
// are numbered row group fastest, then strip, then plane; an item is four.
template <typename T, int R, bool BOX, int NC, int J>
__device__ __forceinline__ void rows3d_item(const KArgs& a, int item) {
  typedef Rows3D<T, R, BOX, NC, J> S;
  const int piece = __builtin_amdgcn_readfirstlane(item * 4 + (int)(threadIdx.x >> 6));
  const int per_plane = a.tiles0 * a.tiles1;
  const int o = piece / per_plane;
  if (o >= a.d0) return;
  const int rest = piece - o * per_plane;
  const int si = rest / a.tiles0, jt = rest - si * a.tiles0;
  const int lane = threadIdx.x & 63;
  const bool periodic = a.periodic != 0;
  const int hl = !periodic && a.d2 <= 64 * NC ? 0 : (R + NC - 1) / NC;
  S s;
  s.c = (ConstPtr<T>)a.coef;
  s.in = (const T*)a.in;
  s.periodic = periodic;
  s.N = (uint32_t)a.d2;
  s.plane = (uint32_t)(a.d1 * a.d2);
  const int64_t N = a.d2;
  const int64_t k0 = ((int64_t)si * (64 - 2 * hl) - hl) * NC;
  const int64_t col = k0 + lane * NC;
  const bool store_lane = lane >= hl && lane < 64 - hl && col < N;
  int64_t wc = col;
  if (periodic) {
    wc %= N;
    if (wc < 0) wc += N;
  } else if (wc < 0 || wc >= N) {
    wc = 0;
  }
  s.wcol = (uint32_t)wc;
#pragma unroll
  for (int e = 0; e < NC; ++e) s.ok[e] = periodic || (col + e >= 0 && col + e < N);
  const bool split = NC > 1 && __builtin_amdgcn_ballot_w64(wc + NC > N) != 0;
  const int Nj = (int)a.d1, j0 = jt * J;
#pragma unroll
  for (int x = 0; x < S::XR; ++x) {
    int r = j0 - R + x;
    s.rok[x] = true;
    if (r < 0 || r >= Nj) {
      s.rok[x] = periodic;
      r = periodic ? r % Nj : 0;
      if (r < 0) r += Nj;
    }
    s.roff[x] = (uint32_t)r * s.N;
  }
  const bool edge = !periodic && (k0 < 0 || k0 + 64 * NC > N || j0 < R || j0 + J + R > Nj);
  if (split) s.template point<2>(o, a.d0);
  else if (edge) s.template point<1>(o, a.d0);
  else s.template point<0>(o, a.d0);
  if (!store_lane) return;
  T* out = (T*)a.out + (int64_t)o * s.plane + col;
#pragma unroll
  for (int p = 0; p < J; ++p) {
    if (j0 + p >= Nj) break;
    T* dst = out + (uint32_t)(j0 + p) * s.N;
    if (col + NC <= N) {
      RsPack<T, NC> v;
#pragma unroll
      for (int k = 0; k < NC; ++k) v.v[k] = s.acc[p][k];
      *reinterpret_cast<RsPack<T, NC>*>(dst) = v;
    } else {
#pragma unroll
      for (int k = 0; k < NC; ++k)
        if (col + k < N) dst[k] = s.acc[p][k];
    }
  }
}

template <typename T, int R, bool BOX, int NC, int J>
__global__ __launch_bounds__(256) void rows3d_kernel(KArgs a) {
  rows3d_item<T, R, BOX, NC, J>(a, xcd_remap(blockIdx.x, gridDim.x));
}

template <typename T, int R, bool BOX, int NC, int J>
__global__ __launch_bounds__(256) void rows3d_batch(BatchArgs b) {
  for_each_batch_item(b, [&](const KArgs& x, int id) { rows3d_item<T, R, BOX, NC, J>(x, id); });
}

// Batched, every order and shape in one kernel (NC = 1, J = 4).  A mixed batch is
// bound by its launches: 120 FP64 grids of 64^2 .. 64^3, 10 steps, spent 150 of 178
// launches on 3D kernels of its own each.
template <typename T>
__global__ __launch_bounds__(256, sizeof(T) == 4 ? 4 : 3) void rows3d_merged(BatchArgs b) {
  for_each_batch_item(b, [&](const KArgs& x, int id) {
    switch (x.variant) {
      case 2: rows3d_item<T, 1, false, 1, 4>(x, id); break;
      case 3: rows3d_item<T, 1, true, 1, 4>(x, id); break;
      case 4: rows3d_item<T, 2, false, 1, 4>(x, id); break;
      case 5: rows3d_item<T, 2, true, 1, 4>(x, id); break;
      case 6: rows3d_item<T, 3, false, 1, 4>(x, id); break;
      case 7: rows3d_item<T, 3, true, 1, 4>(x, id); break;
      case 8: rows3d_item<T, 4, false, 1, 4>(x, id); break;
      case 9: rows3d_item<T, 4, true, 1, 4>(x, id); break;
    }
  });
}

// ------------------------------------------------------------------ host
// The shapes built, NC x J: 1 x 2, 1 x 4, 2 x 4 and 4 x 4 (FP64 orders 3 and 4: 4 x 2,
// the wider rows' registers leave one wave per SIMD otherwise: 256^3 FP64
// order-4 box 572 -> 504 us).
constexpr int rows3d_j(int es, int R, int NC, bool tall) {
  return NC == 1 ? (tall ? 4 : 2) : (NC == 4 && es == 8 && R >= 3) ? 2 : 4;
}

struct Rows3DCut {
  int NC = 0, J = 0;
  int64_t strips = 0, groups = 0, waves = 0;
  double time = 0.0;  // us, estimated
};

// One shape's cut and time: issue slots of a wave (the FMAs, FP64 ones at
// about half the FP32 rate; about three slots per halo column moved; the loads)
// over the 2048 waves that issue at once, 4 cycles each at 2.1 GHz, and the factor
// that boxes measured (256^3 FP32 order 3: 108 us of slots, 167 measured;
// order 4: 228, 344; FP64 order 3: 230, 268; order 4: 483, 504).
inline Rows3DCut rows3d_cut(const KArgs& a, int R, bool box, int es, int NC, int J) {
  Rows3DCut c;
  c.NC = NC;
  c.J = J;
  const int W = 2 * R + 1, XR = J + 2 * R;
  const int hl = !a.periodic && a.d2 <= 64 * NC ? 0 : (R + NC - 1) / NC;
  const int cols = (64 - 2 * hl) * NC;
  c.strips = (a.d2 + cols - 1) / cols;
  c.groups = (a.d1 + J - 1) / J;
  c.waves = c.strips * c.groups * a.d0;
  const double grids = a.share > 0 ? 2048.0 / a.share : 1.0;  // like this one in the launch
  const double f = es == 8 ? 1.85 : 1.0, move = 6.0 * R * (es / 4);
  const double slots = box ? W * (XR * (move + 8) + J * NC * W * W * f + (es == 4 ? W * W : 0))
                           : XR * 8.0 + 2 * R * J * 8.0 + J * move + J * NC * (6 * R + 1) * f;
  c.time = 2.5 + (es == 8 && R >= 3 ? 1.1 : 1.45) * slots * std::max(1.0, c.waves * grids / 2048.0) * 4.0 / 2100.0;
  return c;
}

// The best shape for a grid, NC = 0 when the kernel's 32-bit indices do not reach.
// Alone, and for boxes from order 3 that make up most of a launch or are among so
// many that the chip runs several rounds of their waves: the shortest estimate
// (four 128^3 grids, one column per lane or the ring / this, us a step: FP32 order-3
// and -4 boxes 162 / 113, 315 / 224, FP64 262 / 144, 433 / 273; one, order 4 111 / 57).  Else one of several: one lane column up to 200 columns, as
// each shape more is a launch more.
inline Rows3DCut rows3d_best(const KArgs& a, int R, bool box, int es) {
  Rows3DCut best;
  if (a.d1 * a.d2 >= (int64_t(1) << 31)) return best;
  const bool full =
      box && R >= 3 && (a.share > 1024 || (a.share > 0 && rows3d_cut(a, R, box, es, 1, 4).waves >= 8 * a.share));
  for (int k = 0; k < 4; ++k) {
    const int NC = k < 2 ? 1 : k == 2 ? 2 : 4;
    if (NC > a.d2) continue;
    if (a.share > 0 && (full ? k == 0 : k != (a.d2 <= 200 ? 1 : 3))) continue;
    const Rows3DCut c = rows3d_cut(a, R, box, es, NC, rows3d_j(es, R, NC, k == 1));
    if (c.waves >= (int64_t(1) << 31) - 4 || (best.NC && c.time >= best.time)) continue;
    best = c;
  }
  return best;
}

// Plane-tiles of the ring kernels (plane ring and n = 4 outer products) over the grids
// of a class: workgroups on the fullest CU, and thousands of 32 x 64 tiles filled
// by the grid in the planes a chunk walks, its 2R warm-up planes included.
struct RingLoad {
  double rounds = 0.0, planes = 0.0;
};

inline RingLoad ring_load(const KArgs& a, int R) {
  // the share is rounded down: 12 grids read back as 12.05, a round too many
  const double grids = a.share > 0 ? std::max(1.0, std::floor(2048.0 / a.share)) : 1.0;
  RingLoad l;
  l.rounds = std::ceil(grids * (double)chunk3d_items(a) / 256.0);
  l.planes = grids * (double)a.nchunks * (a.chunk + 2 * R) * (double)(a.d1 * a.d2) / 2048.0e3;
  return l;
}

// us a step of the grids of a class (2048 / share of them) on the rows: fitted to
// batches of 1 .. 2048 grids of 16^3 .. 256^3 by waves of one column and four
// rows; boxes of order 4, and FP64 ones of order 3, by the cut's own time.
inline double rows3d_many_us(const KArgs& a, const Rows3DCut& c, int R, bool box, int es) {
  constexpr double k[2][2][5][2] = {
      {{{0, 0}, {4.4, 0.648}, {4.7, 0.834}, {4.8, 1.04}, {5.1, 1.26}}, {{0, 0}, {4.6, 0.803}, {5.8, 1.81}, {7.6, 3.9}}},
      {{{0, 0}, {4.5, 0.904}, {4.8, 1.227}, {4.8, 1.83}, {5.0, 2.2}}, {{0, 0}, {4.8, 1.084}, {6.5, 2.29}}}};
  if (box && R == 4) return es == 4 ? 1.1 + (c.NC == 4 ? 1.16 : 0.953) * c.time : 5.4 + 1.003 * c.time;
  if (box && R == 3 && es == 8) return 2.5 + 1.028 * c.time;
  const double* f = k[es / 8][box ? 1 : 0][R];
  const double width = (c.NC == 1 ? 1.0 : c.NC == 2 ? 1.8 : 3.3) * c.J / 4.0;
  return f[0] + f[1] * (2048.0 / a.share) * (double)c.waves * width * 1e-3;
}

// The same on the whole-grid gather, a workgroup a grid: 1 to 256 grids take one
// round, whose time follows the grid's points (fitted to 32 .. 300 grids of 8^3 .. 20^3).
inline double whole3d_many_us(double points, int R, bool box, int es) {
  constexpr double k[2][2][5][2] = {
      {{{0, 0}, {4.2, 2.56}, {4.9, 3.36}, {5.8, 4.16}, {7.2, 4.97}}, {{0, 0}, {4.1, 3.30}, {5.4, 7.70}, {8.2, 16.9}, {12.3, 33.0}}},
      {{{0, 0}, {4.2, 2.76}, {5.2, 3.46}, {5.9, 4.36}, {7.1, 5.55}}, {{0, 0}, {4.2, 3.64}, {7.0, 9.31}, {8.4, 28.6}, {13.1, 57.7}}}};
  const double* f = k[es / 8][box ? 1 : 0][R];
  return f[0] + f[1] * points * 1e-3;
}

// The same on the plane ring and on the FP32 outer products of order 3 and 4.
inline double ring3d_many_us(const RingLoad& l, int R, bool box, int es) {
  constexpr double k[2][2][5][3] = {
      {{{0, 0, 0}, {7.2, 1.28, 1.22}, {12.7, 2.38, 1.19}, {19.5, 4.75, 0.73}, {26.3, 7.5, 0.86}},
       {{0, 0, 0}, {8.3, 2.52, 0.82}, {23.2, 14.3, 0.57}, {63.8, 57.2, 0}, {64.1, 199, 6.9}}},
      {{{0, 0, 0}, {8.1, 2.8, 2.27}, {13.2, 4.6, 2.5}, {18.2, 14.8, 1.2}, {24.5, 13.2, 2.1}},
       {{0, 0, 0}, {8.7, 4.5, 1.54}, {15.2, 25.2, 1.6}, {67, 97.7, 0}, {41, 293, 8}}}};
  const double* f = k[es / 8][box ? 1 : 0][R];
  double us = f[0] + f[1] * l.rounds + f[2] * l.planes;
  if (box && R == 2 && es == 8 && l.rounds == 3.0) us *= 0.85;  // three items a CU side by side: 81 (24^3 x 256)
  if (box && R == 3 && es == 4 && l.rounds == 1.0) us *= 1.05;  // 125-130 (32^3 x 64, 64^3 x 16)
  return us;
}
inline double mfma3d_box_many_us(const RingLoad& l, int R) {
  return R == 3 ? 38.7 + 59.9 * l.rounds + 1.0 * l.planes : 67.3 + 148.9 * l.rounds + 3.5 * l.planes;
}

// One of many aligned grids: the rows end early (a chip's waves of them in 5-25 us),
// the ring's few deep items late but at less cost a point, so the rows serve few
// or small grids and the ring many.  Ring / rows, us a step: FP32 7-point star 32^3
// x 16 8.3 / 7.1, x 64 10.5 / 13.5, 64^3 x 4 9.4 / 7.2, x 16 12.0 / 14.4, 128^3 x 2 12.5 / 18.4; order-3
// star 32^3 x 64 24 / 20, x 256 33 / 76; order-2 box 32^3 x 128 48 / 64, 24^3 x 128 45 / 36; order-3 box
// 48^3 x 64 164 / 157, 32^3 x 256 236 / 281; FP64 27-point box 128^3 x 2 22 / 29, order-4 box 32^3 x 64 363 /
// 188, x 256 650 / 742; 24^3 x 1024 2800 / 1556.
// Beside other stencils the ring's depth is hidden by their work, so a class of
// one size has the rows up to nine tenths of its time only (us a step: four FP64 96^3
// of the order-2 star and box 87 on rows, 62, with the 7-point star 109, 76; 40 mixed
// grids, 15 steps, 461 at 1.0 and 0.9, 528 at 0.85).  Of mixed sizes the small grids fill the ring's
// tiles badly (120 mixed FP64 grids, 10 steps, 572 at 1.0, 585 at 0.9).
// The server's launches (columns = 0) follow one another on one stream: there the rows
// share the merged one below fifteen rounds of waves at any rate (nine mixed requests,
// an 80^3 star among them, 1370 us, 1470 with its ring launches).
inline bool rows3d_better_many(const KArgs& a, const Rows3DCut& c, int R, bool box, int es) {
  const double width = c.NC == 1 ? 1.0 : c.NC == 2 ? 1.8 : 3.3;
  if (a.kinds > 1 && a.columns == 0 && 2048.0 / a.share * (double)c.waves * width < 30000.0) return true;
  const double ring = ring3d_many_us(ring_load(a, R), R, box, es);
  const bool one_size = (int64_t)a.columns * a.share <= 2048;
  return rows3d_many_us(a, c, R, box, es) < (a.kinds > 1 && one_size ? 0.9 : 1.0) * ring;
}

// AUTO's FP32 boxes of order 3 and 4 among many: the n = 4 outer products, whose
// rate at a full chip the gathers do not reach (us a step, best gather / outer products: order 4
// 256 grids of 32^3 442 / 339, 64 of 64^3 525 / 390, 128 of 48^3 650 / 506, 128 of 32^3 253 / 205, order 3 236 / 207,
// 257 / 226; eight and twelve of 128^3, order 4, 443 / 393, 672 / 558, four of 160^3 645 / 545; not 64 of
// 32^3, order 4 149 / 195, order 3 73 / 101, nor six of 128^3 338 / 387).
inline bool outer_products_better_many(const KArgs& a, int R) {
  const Rows3DCut c = rows3d_best(a, R, true, 4);
  if (!dma3d_ok<float>(a) || a.share <= 0 || c.NC == 0) return false;
  const RingLoad l = ring_load(a, R);
  const double gather = std::min(rows3d_many_us(a, c, R, true, 4), ring3d_many_us(l, R, true, 4));
  return mfma3d_box_many_us(l, R) < gather;
}

// A grid alone of up to 32 MB, us a step, ring / rows: on the rows, except where their
// cache reads cost more than the ring's depth.  Stars and 27-point boxes whose planes
// are a multiple of 1 MB, whose rows then meet in the same cache sets (FP32, 16 and
// 28 x 512 x 512: star r = 1 9.7 / 12.3, 13.5 / 17.5, r = 4 22 / 30, 31 / 46, box 12.6 / 14.0, 17 / 19; 12 x 600 x
// 600, r = 2 17.6 / 17.8).  FP32 of order 1 by the fitted times (periodic, whose strips
// overlap: 64 x 256 x 256 10.1 / 12.6, 160^3 10.8 / 10.2).  FP32 stars of order 3 and 4 on planes of
// more than 300000 points (12 x 600 x 600 22 / 28; 32 x 384 x 384 26.5 / 26.8), FP64 ones of order 4 of more
// than 80000 (20 x 300 x 300 23.6 / 26.2; 8 x 400 x 400 20.4 / 18.9).
inline bool rows3d_better_small(const KArgs& a, const Rows3DCut& c, int R, bool box, int es) {
  if (box && R >= 2) return true;
  const int64_t plane = a.d1 * a.d2;
  if (plane * es % (1 << 20) == 0) return false;
  if (es == 4 && R == 1) {
    const int64_t tiles = (int64_t)a.tiles0 * a.tiles1;
    double chunk = a.chunk, items = (double)chunk3d_items(a);
    if (items < 256.0) {  // one per CU, as balanced_items3d cuts a grid alone
      chunk = std::min(chunk, std::max(1.0, std::ceil((double)(a.d0 * tiles) / 256.0)));
      items = (double)tiles * std::ceil((double)a.d0 / chunk);
    }
    const double planes = items * (chunk + 2.0) * 1e-3, points = (double)c.waves * c.NC * c.J * 1e-3;
    const double rows = box ? 4.7 + 0.084 * points : 4.35 + 0.068 * points;
    const double ring = box ? 2.6 + 1.69 * planes + 0.9 * (chunk + 2.0) : 2.8 + 1.30 * planes + 0.556 * (chunk + 2.0);
    return ring > 0.9 * rows;
  }
  if (es == 4 && R >= 3) return plane < 300000;
  return !(es == 8 && R == 4 && a.d0 >= 16 && plane >= 80000);
}

// Whether the cut beats the plane ring: on ragged or misaligned grids always (the
// ring stages those without overlap); else on small grids, and for boxes from
// order 2 where the estimate is below the ring's time per point (ps) at 256^3 and
// 512^3.
// Larger stars and 27-point boxes are bound by memory, where the ring reads a
// plane once: 512^3 FP32 star 212-248 us against 311-690, 256^3 25-39 against 24-46.
// Among 2048 / share grids like this one rows3d_better_many decides instead.
template <typename T, int R, bool BOX>
inline bool rows3d_better(const KArgs& a, const Rows3DCut& c) {
  if (!dma3d_ok<T>(a)) return true;
  if (a.share > 0 && (a.share < 2048 || a.kinds > 1)) return rows3d_better_many(a, c, R, BOX, (int)sizeof(T));
  const double pts = (double)a.d0 * (double)a.d1 * (double)a.d2;
  if (pts * sizeof(T) <= 32e6) return rows3d_better_small(a, c, R, BOX, (int)sizeof(T));
  constexpr double ring_ps[2][2][5] = {{{0, 0, 4.9, 25.4, 48.3}, {0, 0, 9.7, 27.2, 82.5}},
                                       {{0, 0, 3.6, 16.2, 34.6}, {0, 0, 7.2, 20.8, 66.6}}};
  return BOX && R >= 2 && c.time < pts * ring_ps[pts < 3e7 ? 0 : 1][sizeof(T) / 8][R] * 1e-6;
}

// Whether one of many small grids, a workgroup each, beats the cut.  From 228 on
// they fill the chip.  Fewer are bound by a workgroup's latency, so the rows have
// them while they end sooner (us a step, whole / rows: 8^3 FP64 order-4 box, 64 grids
// 42 / 21, 200 43 / 54; 27-point box 128 grids 5.9 / 5.3, 200 5.9 / 7.2; 12^3 FP64
// order-3 star 64 grids 12.7 / 7.5, 150 12.8 / 15.2; 16^3 order-3 star, 128 grids
// 22 / 19, 200 22 / 28; order-4 box 32 grids 250 / 30).  Beside other stencils the
// rows share a launch.
inline bool whole3d_better(const KArgs& a, int R, bool box, int es) {
  KArgs n = a;  // by the number of grids
  if (a.columns > 0) n.share = std::max(1, 2048 / a.columns);
  if (n.share <= 8) return true;
  const Rows3DCut c = rows3d_best(n, R, box, es);
  if (a.kinds > 1 || !c.NC) return false;
  const double points = (double)a.d0 * (double)a.d1 * (double)a.d2;
  return whole3d_many_us(points, R, box, es) < rows3d_many_us(n, c, R, box, es);
}

// AUTO's choice between the cut and the n = 4 outer products for FP32 boxes of
// order 3 and 4: those take 97 / 225 us however small the grid, and 14.2 / 25.7 ps a
// point at 256^3, 11.4 / 20.9 at 320^3, 8.9 / 16.6 at 512^3 (the rows: 10.0 / 20.5 at
// 256^3, 13.4 / 28.2 at 320^3).  Up to 16^3 the outer products are the documented path
// (a plan reports it, and the paths round differently), not the faster one.
inline bool rows3d_beats_mfma(const Rows3DCut& c, int R, double pts) {
  const double ps = R == 3 ? (pts < 2e7 ? 13.5 : pts < 5e7 ? 11.0 : 8.9) : (pts < 2e7 ? 25.0 : pts < 5e7 ? 20.5 : 16.6);
  return c.NC && pts > 4096 && c.time < std::max(R == 3 ? 97.0 : 225.0, pts * ps * 1e-6);
}

// The kernel of a cut (NC x J built above).
template <typename T, bool BOX>
Kernel rows3d_of(int R, int NC, int J, int64_t items);
template <typename T>
void rows3d_merge(Kernel* k);

// Its args and kernel.
template <typename T, int R, bool BOX>
inline Kernel rows3d_kernel_for(KArgs& a, const Rows3DCut& c) {
  a.tiles0 = (int32_t)c.groups;
  a.tiles1 = (int32_t)c.strips;
  Kernel k = rows3d_of<T, BOX>(R, c.NC, c.J, (c.waves + 3) / 4);
  if (c.NC == 1 && c.J == 4) {
    a.variant = 2 * R + (BOX ? 1 : 0);
    rows3d_merge<T>(&k);
  }
  return k;
}

}  // namespace stencil
