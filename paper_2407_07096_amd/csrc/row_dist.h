// Squared distances between gathered rows, by fp64 direct differences: four
// lanes read a row together.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace stag {
namespace {

// v of another lane of the quad (a quad permutation), all lanes active: 0x00,
// 0x55, 0xAA, 0xFF that of lane 0 .. 3, 0xB1 of lane ^ 1, 0x4E of lane ^ 2.
template <int CTRL>
__device__ inline int quad_perm(int v) {
  return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, false);
}
template <int CTRL>
__device__ inline double quad_perm(double v) {
  return __hiloint2double(quad_perm<CTRL>(__double2hiint(v)), quad_perm<CTRL>(__double2loint(v)));
}

// Sums over a quad of four values each, the sum of value r in lane r.
__device__ inline double quad_sums(const double (&v)[4]) {
  const bool b1 = threadIdx.x & 2, b0 = threadIdx.x & 1;
  const double k0 = (b1 ? v[2] : v[0]) + quad_perm<0x4E>(b1 ? v[0] : v[2]);  // values 2 b1
  const double k1 = (b1 ? v[3] : v[1]) + quad_perm<0x4E>(b1 ? v[1] : v[3]);  // values 2 b1 + 1
  return (b0 ? k1 : k0) + quad_perm<0xB1>(b0 ? k0 : k1);
}

// ||xi - x_j||^2 for the row j of each lane (rows of d floats, ld apart), by fp64
// direct differences; xi is the same in the four lanes of a quad, and all lanes
// are active.
//
// d > 8: the quad reads its four rows one after the other, each lane 16 bytes
// of every 64, and the four partial sums per row are added across the quad at
// the end.  With a lane per row every load touches 64 cache lines, and the
// rate of the L1's tag lookups bounds the gathers: 1e5 points of 64
// coordinates, 1.7e6 draws over 12 levels took 36.5 ms that way (2.0 at the
// leaves); now 20.9 (0.85), bound by the fp64 operations where a node's rows
// fit an L2 and by the misses of the first three levels.  Two pieces at a time
// leave 6 waves a SIMD; four took 25.2 with 4 waves.  d <= 8: a lane per row,
// whose line or two it reads whole (n = 2e4, d = 4, t = 4: quads 2.7 ms a
// call, a lane per row 0.9).
//
// Rows need only the alignment of a float: 16-byte loads need no more.
enum RowRead { kOwnRow, kQuad4, kQuad };  // d <= 8; d a multiple of 4; any d
inline RowRead row_read(int d) { return d <= 8 ? kOwnRow : d % 4 == 0 ? kQuad4 : kQuad; }

using RowVec = float __attribute__((ext_vector_type(4), aligned(4)));

// U 64-byte pieces from coordinate c on; PART: the last may end before 64.
template <RowRead ROWS, int U, bool PART>
__device__ __forceinline__ void row_piece(const float* __restrict__ xi, const float* const (&xj)[4], int c, int d,
                                           double (&acc)[4]) {
  const int q = threadIdx.x & 3;
  auto load = [&](const float* x, int u) {
    const int at = c + (4 * u + q) * 4;
    RowVec v = {0.f, 0.f, 0.f, 0.f};
    if (!PART || u < U - 1 || at + 4 <= d) {
      v = *reinterpret_cast<const RowVec*>(x + at);
    } else if (ROWS == kQuad && at < d) {
      v[0] = x[at];
      if (at + 1 < d) v[1] = x[at + 1];
      if (at + 2 < d) v[2] = x[at + 2];
    }
    return v;
  };
  RowVec y[4][U];
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int u = 0; u < U; ++u) y[r][u] = load(xj[r], u);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const RowVec x = load(xi, u);
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const double xd = x[w];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double t = xd - (double)y[r][u][w];
        acc[r] = fma(t, t, acc[r]);
      }
    }
  }
}

template <RowRead ROWS>
__device__ __forceinline__ double row_dist2(const float* __restrict__ xi, const float* __restrict__ X, int64_t ld,
                                            int64_t j, int d) {
  if constexpr (ROWS == kOwnRow) {
    const float* x = X + j * ld;
    double D = 0.0;
    int c = 0;
    for (; c + 4 <= d; c += 4) {
      const RowVec u = *reinterpret_cast<const RowVec*>(xi + c), v = *reinterpret_cast<const RowVec*>(x + c);
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const double t = (double)u[w] - (double)v[w];
        D = fma(t, t, D);
      }
    }
    for (; c < d; ++c) {
      const double t = (double)xi[c] - (double)x[c];
      D = fma(t, t, D);
    }
    return D;
  } else {
    const float* xj[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) xj[r] = X + (int64_t)__shfl((int)j, r, 4) * ld;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    int c = 0;
    for (; c + 32 <= d; c += 32) row_piece<ROWS, 2, false>(xi, xj, c, d, acc);
    if (d - c > 16) row_piece<ROWS, 2, true>(xi, xj, c, d, acc);
    else if (d - c > 0) row_piece<ROWS, 1, true>(xi, xj, c, d, acc);
    return quad_sums(acc);
  }
}

}  // namespace
}  // namespace stag
