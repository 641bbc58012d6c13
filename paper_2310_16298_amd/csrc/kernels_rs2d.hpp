// Time-blocked 2D gather in registers: up to TS Jacobi steps per launch, no LDS.
//
// A wave owns a strip of 64 NC grid columns (lane l: columns NC l .. NC l +
// NC - 1) and walks down the rows of a chunk.  Each incoming row passes
// through a pipeline of `steps` levels: level t takes row g of time t - 1,
// scatters it into the 2R + 1 output rows it reaches and hands row g - R of
// time t, complete with this row, to level t + 1.  A level keeps only the 2R
// unfinished output rows, NC values each, in registers; the update of output
// row z reads its accumulator in slot z + 1 and writes slot z, so the ring
// moves down in the FMAs themselves.  Columns of the neighbouring lanes come
// through DPP wave shifts (one move per halo column).  Rows arrive in
// ascending order and columns are taken in ascending order, the tap order of
// the one-step gather, so the results agree with it bit for bit.
//
// Strips overlap by the R steps columns that go stale on each side (rounded
// up to whole lanes), chunks by the 2 R steps rows of the pipeline's fill.
// Zero halo: strips and chunks that meet the grid's faces reset what lies
// outside it after every level.
//
// What bounds it: the FP32 FMA rate for boxes, memory for stars.  With no LDS
// and no barrier the inner loop is FMAs plus 2R moves per level (order-2 box:
// 100 FMAs and 4 DPP moves for 4 points).  A SIMD issues the vector
// instructions of two waves side by side only if they do not both read a
// scalar operand (register-only FMA chains, two waves per SIMD: 64 T FMA/s
// with vector weights, 37.5 T with scalar ones; FP64: 35 T either way), so FP32
// weights live in vector registers.  8192^2, one launch of T steps, against
// the LDS tiles of tb2d_dma_kernel: FP32 stars r = 1..4 (T = 8 / 4 / 4 / 3)
// 231 / 165 / 222 / 200 -> 132 / 132 / 163 / 162 us (537 MB: 4.1 TB/s at r = 1, 2;
// a large copy runs at 5.0), boxes (8 / 4 / 4 / 2) 323 / 292 / 556 / 331 -> 157 / 198 /
// 369 / 290 us; FP64 stars (8 / 4 / 2 / 2) 508 / 339 / 285 / 281 -> 235 / 232 / 230 /
// 232 us (1.07 GB: 4.6 TB/s), boxes (8 / 4) 615 / 506 -> 252 / 309 us.
#pragma once

#include <algorithm>

#include "device_common.hpp"
#include "launch.hpp"

namespace stencil {

// Value of the lane below (wave_shr:1) / above (wave_shl:1); 0 past the wave's ends.
__device__ __forceinline__ int rs_dpp_up(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x138, 0xf, 0xf, true); }
__device__ __forceinline__ int rs_dpp_down(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x130, 0xf, 0xf, true); }

template <bool UP>
__device__ __forceinline__ float rs_shift(float v) {
  const int b = __builtin_bit_cast(int, v);
  return __builtin_bit_cast(float, UP ? rs_dpp_up(b) : rs_dpp_down(b));
}
template <bool UP>
__device__ __forceinline__ double rs_shift(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = UP ? rs_dpp_up((int)(uint32_t)b) : rs_dpp_down((int)(uint32_t)b);
  const uint32_t hi = UP ? rs_dpp_up((int)(b >> 32)) : rs_dpp_down((int)(b >> 32));
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

__device__ __forceinline__ float rs_fma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double rs_fma(double a, double b, double c) { return __builtin_fma(a, b, c); }

// The FMA that moves an accumulator down one slot, kept in its three-address
// form: the compiler would tie result and accumulator, and then move every
// accumulator once per row (order-2 box: 64 moves beside 360 FMAs).  Its
// result must not be read by a DPP instruction within two wait states (the
// compiler does not see a vector write in the asm), so a level's outgoing row,
// which the next level shifts, ends in an ordinary FMA or in rs_out.
__device__ __forceinline__ float rs_fma3(float w, float e, float a) {
  float d;
  asm("v_fma_f32 %0, %1, %2, %3" : "=v"(d) : "v"(w), "v"(e), "v"(a));
  return d;
}
__device__ __forceinline__ double rs_fma3(double w, double e, double a) {
  double d;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "s"(w), "v"(e), "v"(a));
  return d;
}
// A star's outgoing row (one tap left), with the wait states of its DPP readers.
__device__ __forceinline__ void rs_out(float w, const float (&e)[1], const float (&a)[1], float* x) {
  float d0;
  asm("v_fma_f32 %0, %1, %2, %3\n\ts_nop 1" : "=&v"(d0) : "v"(w), "v"(e[0]), "v"(a[0]));
  x[0] = d0;
}
__device__ __forceinline__ void rs_out(double w, const double (&e)[1], const double (&a)[1], double* x) {
  double d0;
  asm("v_fma_f64 %0, %1, %2, %3\n\ts_nop 1" : "=&v"(d0) : "s"(w), "v"(e[0]), "v"(a[0]));
  x[0] = d0;
}
__device__ __forceinline__ void rs_out(float w, const float (&e)[2], const float (&a)[2], float* x) {
  float d0, d1;
  asm("v_fma_f32 %0, %2, %3, %5\n\tv_fma_f32 %1, %2, %4, %6\n\ts_nop 1"
      : "=&v"(d0), "=&v"(d1)
      : "v"(w), "v"(e[0]), "v"(e[1]), "v"(a[0]), "v"(a[1]));
  x[0] = d0;
  x[1] = d1;
}
__device__ __forceinline__ void rs_out(double w, const double (&e)[2], const double (&a)[2], double* x) {
  double d0, d1;
  asm("v_fma_f64 %0, %2, %3, %5\n\tv_fma_f64 %1, %2, %4, %6\n\ts_nop 1"
      : "=&v"(d0), "=&v"(d1)
      : "s"(w), "v"(e[0]), "v"(e[1]), "v"(a[0]), "v"(a[1]));
  x[0] = d0;
  x[1] = d1;
}
__device__ __forceinline__ void rs_out(float w, const float (&e)[4], const float (&a)[4], float* x) {
  float d0, d1, d2, d3;
  asm("v_fma_f32 %0, %4, %5, %9\n\tv_fma_f32 %1, %4, %6, %10\n\t"
      "v_fma_f32 %2, %4, %7, %11\n\tv_fma_f32 %3, %4, %8, %12\n\ts_nop 1"
      : "=&v"(d0), "=&v"(d1), "=&v"(d2), "=&v"(d3)
      : "v"(w), "v"(e[0]), "v"(e[1]), "v"(e[2]), "v"(e[3]), "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]));
  x[0] = d0;
  x[1] = d1;
  x[2] = d2;
  x[3] = d3;
}
__device__ __forceinline__ void rs_out(double w, const double (&e)[4], const double (&a)[4], double* x) {
  double d0, d1, d2, d3;
  asm("v_fma_f64 %0, %4, %5, %9\n\tv_fma_f64 %1, %4, %6, %10\n\t"
      "v_fma_f64 %2, %4, %7, %11\n\tv_fma_f64 %3, %4, %8, %12\n\ts_nop 1"
      : "=&v"(d0), "=&v"(d1), "=&v"(d2), "=&v"(d3)
      : "s"(w), "v"(e[0]), "v"(e[1]), "v"(e[2]), "v"(e[3]), "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]));
  x[0] = d0;
  x[1] = d1;
  x[2] = d2;
  x[3] = d3;
}

// NC consecutive elements at element alignment (one load or store of up to 16 bytes each).
template <typename T, int NC>
struct __attribute__((packed, aligned(sizeof(T)))) RsPack {
  T v[NC];
};

// Lanes per side of a strip that go stale over a launch's steps.  A zero-halo
// grid that fits one strip has none: the zeros the shifts bring in are its halo.
__host__ __device__ inline int rs2d_halo_lanes(const KArgs& a, int R, int NC) {
  return !a.periodic && a.d1 <= 64 * NC ? 0 : (R * a.steps + NC - 1) / NC;
}

// The levels of one wave.  Row numbers are kept modulo 2^32 (extents are below
// 2^31): r < M as unsigned says that row r lies in the grid.
template <typename T, int R, bool BOX, int TS, int NC>
struct RsWave {
  static constexpr int W = 2 * R + 1;
  static constexpr int U = TS == 1 ? 4 : 2;  // rows loaded ahead
  T acc[TS][2 * R][NC];  // level t + 1: its unfinished output rows, oldest first
  // The weights stay in registers for the whole walk.  FP32: vector registers
  // (a scalar operand would keep a second wave from issuing beside this one),
  // the order-4 box's odd columns in scalar ones (81 would cost a third of
  // the vector registers).  FP64: scalar registers for the first 25 (of a box,
  // all of column 0: rs_fma3 reads those).
  T held[W * W];
  static constexpr bool scalar_weight(int i) {
    if (sizeof(T) == 4) return BOX && R == 4 && i % W % 2 == 1;
    constexpr int NS = 25;
    return (BOX ? W * W : 2 * W - 1) <= NS || i % W == 0 || (i / W) * (W - 1) + i % W + W <= NS;
  }
  const T* in;
  T* out;
  uint32_t M, N;
  uint32_t row, wrow;  // next input row: its index and its index after wrapping
  uint32_t orow;       // next output row
  uint32_t col;        // the lane's first column (stored ones: inside the grid) ...
  uint32_t wcol;       // ... wrapped / clamped into the row
  bool periodic, store_lane;
  int turn;            // 0 or 1: the workgroup's place on its CU
  bool ok[NC];         // column col + e lies in the grid

  __device__ __forceinline__ void hold(ConstPtr<T> c) {
#pragma unroll
    for (int i = 0; i < W * W; ++i)
      if (BOX || i / W == R || i % W == R) held[i] = c[i];
#pragma unroll
    for (int i = 0; i < W * W; ++i)
      if (BOX || i / W == R || i % W == R) {
        // loaded here, once
        if (scalar_weight(i)) asm volatile("" : "+s"(held[i]));
        else asm volatile("" : "+v"(held[i]));
      }
  }

  // Input row `row` into x, and on to the next one; rows outside a zero-halo
  // grid read some row inside (mask() zeroes them).  MODE 0: inside the grid or
  // periodic, whole lanes; 1: zero halo, whole lanes; 2: some lane's columns
  // run past the row's end.  No branches on the way to the load: behind one,
  // the compiler waits for the load at once (order-4 box: 384 -> 442 GStencil/s).
  template <int MODE>
  __device__ __forceinline__ void load(T* x) {
    const T* src = in + (int64_t)wrow * N;
    if constexpr (MODE < 2) {
      const RsPack<T, NC> p = *reinterpret_cast<const RsPack<T, NC>*>(src + wcol);
#pragma unroll
      for (int e = 0; e < NC; ++e) x[e] = p.v[e];
    } else {
#pragma unroll
      for (int e = 0; e < NC; ++e) x[e] = src[wcol + e < N ? wcol + e : (periodic ? wcol + e - N : 0u)];
    }
    ++row;
    const uint32_t next = wrow + 1 == M ? 0u : wrow + 1;
    wrow = periodic ? next : (row < M ? row : 0u);
  }

  // level t + 1: row x of time t in, the row of time t + 1 it completes out
  __device__ __forceinline__ void level(int t, T* x) {
    constexpr int HL = (R + NC - 1) / NC;  // neighbour lanes reached
    T e[2 * R + NC];                       // columns col - R .. col + NC - 1 + R
    T s[NC];
#pragma unroll
    for (int k = 0; k < NC; ++k) e[R + k] = s[k] = x[k];
#pragma unroll
    for (int h = 0; h < HL; ++h)
#pragma unroll
      for (int k = NC - 1; k >= 0; --k) {
        const int at = k - NC * (h + 1);  // the column offset this value has here
        if (at < -R) continue;
        s[k] = rs_shift<true>(s[k]);
        e[R + at] = s[k];
      }
#pragma unroll
    for (int k = 0; k < NC; ++k) s[k] = x[k];
#pragma unroll
    for (int h = 0; h < HL; ++h)
#pragma unroll
      for (int k = 0; k < NC; ++k) {
        const int at = k + NC * (h + 1);
        if (at > NC - 1 + R) continue;
        s[k] = rs_shift<false>(s[k]);
        e[R + at] = s[k];
      }
#pragma unroll
    for (int z = 0; z < W; ++z) {
      const int a = 2 * R - z;  // C^g row that takes this input row to output row z
      T n[NC];
      if (!BOX && z == 0) {
        constexpr int G = NC < 4 ? NC : 4;
#pragma unroll
        for (int q = 0; q < NC; q += G) {
          T ec[G], ac[G];
#pragma unroll
          for (int k = 0; k < G; ++k) {
            ec[k] = e[R + q + k];
            ac[k] = acc[t][0][q + k];
          }
          rs_out(held[a * W + R], ec, ac, n + q);
        }
      } else {
#pragma unroll
        for (int b = 0; b < W; ++b) {
          if (!BOX && a != R && b != R) continue;
          const T w = held[a * W + b];
          const bool first = b == 0 || (!BOX && a != R);
#pragma unroll
          for (int k = 0; k < NC; ++k) {
            if (!first) n[k] = rs_fma(w, e[b + k], n[k]);
            else if (z == 2 * R) n[k] = rs_fma(w, e[b + k], T(0));
            else n[k] = rs_fma3(w, e[b + k], acc[t][z == 2 * R ? 0 : z][k]);
          }
        }
      }
#pragma unroll
      for (int k = 0; k < NC; ++k) {
        if (z == 0) x[k] = n[k];
        else acc[t][z == 0 ? 0 : z - 1][k] = n[k];
      }
    }
  }

  // row r of a level's output: 0 outside the grid
  template <int MODE>
  __device__ __forceinline__ void mask(T* x, uint32_t r) {
    if constexpr (MODE > 0) {
      if (MODE == 2 && periodic) return;
      if (r < M) {
#pragma unroll
        for (int k = 0; k < NC; ++k) x[k] = ok[k] ? x[k] : T(0);
      } else {
#pragma unroll
        for (int k = 0; k < NC; ++k) x[k] = T(0);
      }
    }
  }

  // one row through L levels, stored when `put`; nx: the row, then the one U
  // rows on, in flight behind the levels
  template <int L, int MODE>
  __device__ __forceinline__ void one(bool put, T* nx) {
    T x[NC];
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      x[k] = nx[k];
      asm volatile("" : "+v"(x[k]));  // wait for this row before the next load is issued
    }
    const uint32_t g = row - U;  // the row in x
    load<MODE>(nx);
    mask<MODE>(x, g);
#pragma unroll
    for (int t = 0; t < L; ++t) {
      level(t, x);
      if (t + 1 < L) mask<MODE>(x, g - R * (t + 1));
    }
    if (put) {
      if (store_lane) {
        T* dst = out + (int64_t)orow * N + col;
        if (MODE < 2 || ok[NC - 1]) {
          RsPack<T, NC> p;
#pragma unroll
          for (int k = 0; k < NC; ++k) p.v[k] = x[k];
          *reinterpret_cast<RsPack<T, NC>*>(dst) = p;
        } else {
#pragma unroll
          for (int k = 0; k < NC; ++k)
            if (ok[k]) dst[k] = x[k];
        }
      }
      ++orow;
    }
  }

  // n rows (a multiple of U) through L levels; rows first .. first + ch - 1 are stored
  template <int L, int MODE>
  __device__ __forceinline__ void rows(int n, int first, int ch, T (*nx)[NC]) {
#pragma unroll 1
    for (int i = 0; i < n; i += U) {
      // The two waves of a SIMD take turns at being served first, 16 rows each:
      // always the older first, it ends early and the other walks on alone
      // (8192^2 FP32 boxes r = 1, 3, 4 +5 / +2 / +3 %, 2048^2 order-2 box +4 %).
      if ((i >> 4 ^ turn) & 1) __builtin_amdgcn_s_setprio(1);
      else __builtin_amdgcn_s_setprio(0);
#pragma unroll
      for (int u = 0; u < U; ++u) one<L, MODE>(i + u >= first && i + u < first + ch, nx[u]);
    }
  }

  // fill the pipeline level by level, then stream the chunk's ch rows
  template <int L, int MODE>
  __device__ __forceinline__ void fill(int steps, int ch, T (*nx)[NC]) {
    static_assert(TS == 1 || 2 * R % U == 0, "whole rounds of rows");
    const bool last = L == TS || L == steps;
    rows<L, MODE>(last ? (2 * R + ch + U - 1) / U * U : 2 * R, last ? 2 * R : 0x40000000, last ? ch : 0, nx);
    if constexpr (L < TS) {
      if (!last) fill<L + 1, MODE>(steps, ch, nx);
    }
  }

  template <int MODE>
  __device__ __forceinline__ void walk(int steps, int ch) {
    T nx[U][NC];
#pragma unroll
    for (int u = 0; u < U; ++u) load<MODE>(nx[u]);
    fill<1, MODE>(steps, ch, nx);
  }
};

// Work decomposition: a.tiles1 strips, a.nchunks chunks of a.chunk rows; an
// item is four consecutive (chunk, strip) pieces, one per wave.
template <typename T, int R, bool BOX, int TS, int NC>
__device__ __forceinline__ void rs2d_item(const KArgs& a, int item) {
  const int piece = __builtin_amdgcn_readfirstlane(item * 4 + (int)(threadIdx.x >> 6));
  if (piece >= a.tiles1 * a.nchunks) return;
  const int ci = piece / a.tiles1, si = piece - ci * a.tiles1;
  const int lane = threadIdx.x & 63;
  const int steps = a.steps;
  const int hl = rs2d_halo_lanes(a, R, NC);  // stale lanes per side
  RsWave<T, R, BOX, TS, NC> w;
  w.hold((ConstPtr<T>)a.coef);
  w.turn = (int)(blockIdx.x >> 8) & 1;  // one workgroup per CU before the next ones
  w.in = (const T*)a.in;
  w.out = (T*)a.out;
  w.M = (uint32_t)a.d0;
  w.N = (uint32_t)a.d1;
  w.periodic = a.periodic != 0;
  const int64_t N = a.d1;
  const int64_t j0 = ((int64_t)si * (64 - 2 * hl) - hl) * NC;  // the strip's first column
  const int64_t col = j0 + lane * NC;
  w.col = (uint32_t)col;
  w.store_lane = lane >= hl && lane < 64 - hl && col < N;
  int64_t wc = col;
  if (w.periodic) {
    wc %= N;
    if (wc < 0) wc += N;
  } else if (wc < 0 || wc >= N) {
    wc = 0;
  }
  w.wcol = (uint32_t)wc;
#pragma unroll
  for (int e = 0; e < NC; ++e) w.ok[e] = col + e >= 0 && col + e < N;
  // a lane whose columns run past the row's end: element loads and stores
  const bool split = NC > 1 && __builtin_amdgcn_ballot_w64(wc + NC > N) != 0;
  const uint32_t i0 = (uint32_t)ci * (uint32_t)a.chunk;
  const int ch = (int)(w.M - i0 < (uint32_t)a.chunk ? w.M - i0 : (uint32_t)a.chunk);
  w.orow = i0;
  w.row = i0 - (uint32_t)(R * steps);
  w.wrow = w.row < w.M ? w.row : 0u;
  if (w.periodic) {
    const int64_t r = ((int64_t)i0 - R * steps) % a.d0;
    w.wrow = (uint32_t)(r < 0 ? r + a.d0 : r);
  }
#pragma unroll
  for (int t = 0; t < TS; ++t)
#pragma unroll
    for (int z = 0; z < 2 * R; ++z)
#pragma unroll
      for (int k = 0; k < NC; ++k) w.acc[t][z][k] = T(0);
  const bool edge =
      !w.periodic && (j0 < 0 || j0 + 64 * NC > N || i0 < (uint32_t)(R * steps) || i0 + ch + R * steps > w.M);
  if (split) w.template walk<2>(steps, ch);
  else if (edge) w.template walk<1>(steps, ch);
  else w.template walk<0>(steps, ch);
}

template <typename T, int R, bool BOX, int TS, int NC>
__global__ __launch_bounds__(256) void rs2d_kernel(KArgs a) {
  rs2d_item<T, R, BOX, TS, NC>(a, xcd_remap(blockIdx.x, gridDim.x));
}

template <typename T, int R, bool BOX, int TS, int NC>
__global__ __launch_bounds__(256) void rs2d_batch(BatchArgs b) {
  for_each_batch_item(b, [&](const KArgs& x, int id) { rs2d_item<T, R, BOX, TS, NC>(x, id); });
}

// Batched single steps, every order and shape in one kernel (NC = 2).
template <typename T>
__global__ __launch_bounds__(256) void rs2d_one_merged(BatchArgs b) {
  for_each_batch_item(b, [&](const KArgs& x, int id) {
    switch (x.variant) {
      case 2: rs2d_item<T, 1, false, 1, 2>(x, id); break;
      case 3: rs2d_item<T, 1, true, 1, 2>(x, id); break;
      case 4: rs2d_item<T, 2, false, 1, 2>(x, id); break;
      case 5: rs2d_item<T, 2, true, 1, 2>(x, id); break;
      case 6: rs2d_item<T, 3, false, 1, 2>(x, id); break;
      case 7: rs2d_item<T, 3, true, 1, 2>(x, id); break;
      case 8: rs2d_item<T, 4, false, 1, 2>(x, id); break;
      case 9: rs2d_item<T, 4, true, 1, 2>(x, id); break;
    }
  });
}

// Work decomposition of the register-streaming kernel: strips of 64 NC
// columns, chunks of rows.  A launch runs two waves per SIMD (kRsWaves = 2048 on
// 256 CUs), each with an issue port of its own, so a grid alone is cut into
// that many waves; a wave's time is its rows, 3/4 of the pipeline's fill
// included, times the instructions of a row, and the NC with the shortest
// time is taken.  8192^2 FP32 order-2 box, NC = 4: 1283 GStencil/s at two waves per
// SIMD, 996 at one, 1212 at four.
constexpr int kRsWaves = 2048;  // two per SIMD

struct RsCut {
  int64_t strips = 0, chunks = 0, ch = 0;
  double wave = 0.0;  // issue slots of one wave
};

// waves_for: the waves the grid is cut into; `many`: chunks of 8 to 64 rows
// (longer ones gain little and balance worse).
inline RsCut rs_cut(const KArgs& a, int R, bool box, int es, int steps, int NC, int64_t waves_for, bool many) {
  RsCut c;
  KArgs b = a;
  b.steps = steps;
  const int cols = (64 - 2 * rs2d_halo_lanes(b, R, NC)) * NC;
  c.strips = (a.d1 + cols - 1) / cols;
  int64_t chunks = std::max<int64_t>(1, std::min<int64_t>(a.d0, waves_for / c.strips));
  if (many) chunks = std::max((a.d0 + 63) / 64, std::min((a.d0 + 7) / 8, chunks));
  c.ch = (a.d0 + chunks - 1) / chunks;
  c.chunks = (a.d0 + c.ch - 1) / c.ch;
  // per row and level: the FMAs, the moves of 2R halo columns (about three
  // issue slots each), the loop's own
  const int taps = box ? (2 * R + 1) * (2 * R + 1) : 4 * R + 1;
  c.wave = (c.ch + 1.5 * R * steps) * (taps * NC + 3.0 * R * (es / 4) + 4);
  return c;
}

inline bool rs_columns_ok(const KArgs& a, int NC, const RsCut& c) {
  return NC <= a.d1 && c.strips * c.chunks <= (int64_t(1) << 30);
}

// Levels built per order: the largest step count of a time-blocked launch.
template <typename T>
constexpr int rs2d_steps(int R) {
  return sizeof(T) == 8 ? (R == 1 ? 8 : R == 2 ? 4 : 2) : (R == 1 ? 12 : R == 2 ? 6 : R == 3 ? 4 : 3);
}

// The kernel for order R and NC columns per lane.
template <typename T, bool BOX>
Kernel rs2d_of(int R, int NC, int64_t items);
// The same walk with one step (NC = 2).
template <typename T, bool BOX>
Kernel rs2d_one(int R, int64_t items);
template <typename T>
void rs2d_one_merge(Kernel* k);

}  // namespace stencil
