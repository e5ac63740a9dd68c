// Similarity-graph edge sampling (Sec. "The MS Algorithm": sample edge (i,j)
// with probability proportional to w_F(i,j)/deg_F(i) + w_F(i,j)/deg_F(j), the
// degrees being kernel sums, so that the sampled graph keeps the cluster
// structure of the fully connected one with O~(n) edges).
//
// Mechanism (the paper leaves it open): every node i draws s neighbours
// j != i with probability k_ij / rest_i, rest_i = sum_{j != i} k_ij, and each
// draw carries weight 1 / (s (1/rest_i + 1/rest_j)), so the expected sampled
// weight of every pair is k_ij.  deg(i) = 1 + rest_i.
//
// Exact mode: one self-excluding pass of the exact tile kernel gives the
// per-chunk (4096 rows) fp64 sums and per-tile (32 rows) fp32 sums of every
// row of the kernel matrix (tile sums stored node-major, so one draw reads
// its chunk's 128 tile sums contiguously); a draw walks chunk sums, then tile sums, then
// recomputes the 32 kernel values of its tile in fp64 (direct differences,
// two lanes per row) and inverts the cumulative sum at each level, j
// ascending.  Between the tile and the row step the draws are sorted by tile
// so that draws gathering the same rows run together.
// LSH mode: the CKNS estimator's terms replace the kernel row (lsh.hip).
#include <cmath>

#include "kde_exact.h"
#include "lsh.h"
#include "row_dist.h"
#include "runtime.h"
#include "sort.h"

namespace stag {
namespace {

constexpr uint64_t kGammaS = 0x9E3779B97F4A7C15ULL;
constexpr uint64_t kTagDrawS = 0x44524157ULL;
// Rows up to this width, and data of up to so many bytes (an XCD's L2 holds 4
// MB), draw in one fused kernel, others (and all above 256 wide) through the
// tile sort: the tiles of narrow rows and small data stay in cache in any order.
// Measured by call, fused against sorted, 17 draws per node at n = 100,000: 4.72
// against 4.95 ms at d = 48, 5.29 and 5.24 at 64, 7.68 and 6.97 at 65, 10.1 and
// 8.66 at 128, 15.8 and 12.8 at 192; in us at other sizes, 146 and 181 at 5,000 x
// 128 (2.6 MB), 583 and 628 at 20,000 x 80 (6.4 MB), 269 and 282 at 8,000 x 192
// (6.1 MB), 759 and 710 at 20,000 x 100 (8.0 MB), 358 and 329 at 8,000 x 256
// (8.2 MB), 486 and 505 at 16,000 x 128 (8.2 MB), 856 and 831 at 26,000 x 80 (8.3
// MB), 546 and 507 at 12,000 x 192 (9.2 MB).
constexpr int kDrawFusedMaxDim = 64;
constexpr int64_t kDrawFusedMaxBytes = (int64_t)7 << 20;
constexpr int kChunkTiles = 128;  // 32-row tiles per 4096-row chunk
constexpr double kLog2eS = 1.4426950408889634074;

__device__ inline uint64_t mixs(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
  return z ^ (z >> 31);
}

// Inclusive sums over each half of the wave.
__device__ inline double scan32(double v) {
  const int c = threadIdx.x & 31;
#pragma unroll
  for (int o = 1; o < 32; o <<= 1) {
    const double u = __shfl_up(v, o, 32);
    if (c >= o) v += u;
  }
  return v;
}

// The lanes of this half among those where `p` holds (all lanes active).
__device__ inline uint32_t half_ballot(bool p) { return (uint32_t)(__ballot(p) >> (threadIdx.x & 32)); }

// rest_i (chunk order) and a node-major copy of the chunk sums, so that a
// draw reads its node's P sums from consecutive addresses.
// A row whose sum is below kRescueBelow sets flag[i] and the flag of its
// query tile of qtile_rows rows (underflow rescue).
__global__ void row_rest(const double* __restrict__ partial, int P, int64_t m_pad, int64_t n,
                         double* __restrict__ rest, double* __restrict__ deg, double* __restrict__ chunk_t,
                         int* __restrict__ flag, int* __restrict__ qtile_flag, int qtile_rows) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double s = 0.0;
  for (int p = 0; p < P; ++p) {
    const double v = partial[(int64_t)p * m_pad + i];
    chunk_t[i * P + p] = v;
    s += v;
  }
  rest[i] = s;
  if (deg) deg[i] = 1.0 + s;
  if (flag && s < kRescueBelow) {
    flag[i] = 1;
    qtile_flag[i / qtile_rows] = 1;
  }
}

// Rows of the rescue's second self pass: a flagged row takes its shifted
// chunk sums (the draws use them and the shifted total rest_draw), and its
// true total rest = rest_draw 2^{m_i} for the weights and degrees; other rows
// keep rest_draw = rest.
__global__ void rescue_rows(const double* __restrict__ partial, int P, int64_t m_pad, int64_t n,
                            const int* __restrict__ flag, const double* __restrict__ shift,
                            double* __restrict__ rest, double* __restrict__ rest_draw, double* __restrict__ deg,
                            double* __restrict__ chunk_t) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  if (!flag[i]) {
    rest_draw[i] = rest[i];
    return;
  }
  double s = 0.0;
  for (int p = 0; p < P; ++p) {
    const double v = partial[(int64_t)p * m_pad + i];
    chunk_t[i * P + p] = v;
    s += v;
  }
  rest_draw[i] = s;
  const double t = s * exp2(shift[i]);
  rest[i] = t;
  if (deg) deg[i] = 1.0 + t;
}

// Each half of the wave inverts a cumulative sum over `count` values (the same
// count in both) for its own `target`: 32 N values at a time, fetch(k0, v)
// giving lane c the values k0 + N c .. + N - 1 (0 past the end).  Returns the
// index and the remainder below it.  Past the total (rounding), the last
// positive value is taken with an infinite remainder so that lower levels also
// take their last element; -1 if no value is positive.  All lanes active.
template <int N, class Fetch>
__device__ inline int invert_half(int count, double target, Fetch&& fetch, double* resid_out) {
  const int c = threadIdx.x & 31;
  double running = 0.0, resid = INFINITY;
  int found = -1, last = -1;
  for (int k0 = 0; k0 < count; k0 += 32 * N) {
    double v[N], sum[N];
    fetch(k0, v);
    sum[0] = v[0];
#pragma unroll
    for (int q = 1; q < N; ++q) sum[q] = sum[q - 1] + v[q];
    const double incl = scan32(sum[N - 1]);
    double before = __shfl_up(incl, 1, 32);
    before = c == 0 ? running : running + before;
    // only a positive value can be the crossing: past the last positive value
    // the tree scan may differ from it by a rounding, and a crossing found
    // there means the target lies beyond these values
    int at = N, lastq = -1;
#pragma unroll
    for (int q = N - 1; q >= 0; --q)
      if (v[q] > 0.0) {
        lastq = lastq < 0 ? q : lastq;
        if (before + sum[q] > target) at = q;
      }
    const uint32_t pos = half_ballot(lastq >= 0), over = half_ballot(at < N);
    double below = before;  // of the crossing
    if constexpr (N > 1) {
#pragma unroll
      for (int q = 1; q < N; ++q) below = at == q ? before + sum[q - 1] : below;
    }
    const int lo = over ? __builtin_ctz(over) : 0, lp = pos ? 31 - __builtin_clz(pos) : 0;
    const int q_over = __shfl(at, lo, 32), q_last = __shfl(lastq, lp, 32);
    const double r = target - __shfl(below, lo, 32), total = __shfl(incl, 31, 32);
    if (found < 0) {
      if (over) {
        found = k0 + N * lo + q_over;
        resid = r;
      } else if (pos) {
        last = k0 + N * lp + q_last;
      }
    }
    running += total;
    if (__ballot(found < 0) == 0ull) break;
  }
  *resid_out = found >= 0 ? resid : INFINITY;
  return found >= 0 ? found : last;
}

// A draw of node i takes a chunk, then a 32-row tile within it, then a row
// within the tile, each by inversion of a cumulative sum.  The first two
// steps read only the chunk and tile sums; the last reads the 32 rows of the
// tile.  For wide rows they run as two kernels with the draws sorted by tile
// in between (stable radix sort): with the XCD-aware block order of
// `draw_row` each XCD takes a contiguous range of tiles, and the waves that
// gather the same tile run side by side and hit in that XCD's L2.  For
// narrow rows, whose tiles stay in cache anyway, one fused kernel does both.
// The order changes only where a draw runs, not what it computes.
//
// A draw is a chain of dependent loads and scans, so it is the waves in flight
// that bound it: half a wave per draw, the tile sums of a chunk in one scan of
// four a lane, and the rows of the tile read by quads of lanes.  With a wave
// per draw, two scans of 64 tile sums and two lanes a row, 1.7e6 draws at
// n = 1e5, d = 64 took 2.6 ms; now 1.8.

// The uniform of draw r of node i.
__device__ inline double draw_uniform(uint64_t seed, int64_t i, int r) {
  uint64_t ds = mixs(mixs(mixs(seed ^ kTagDrawS) ^ (uint64_t)i) ^ 0ULL);
  return (double)(mixs(ds + (uint64_t)(r + 1) * kGammaS) >> 11) * 0x1.0p-53;
}

// e / s (the 64-bit quotient is a long sequence)
__device__ inline int64_t node_of(int64_t e, int s) {
  return e < ((int64_t)1 << 31) ? (int64_t)((uint32_t)e / (uint32_t)s) : e / s;
}

// Steps 1 and 2 of a draw (half a wave): the tile (ntile when the draw finds
// none) and the remainder of the target below it.
__device__ inline int64_t draw_tile_of(int64_t i, double u, int P, int64_t ntile, int64_t tstride,
                                       const double* __restrict__ chunk_t, const float* __restrict__ tp,
                                       const double* __restrict__ rest, const double* __restrict__ rest_draw,
                                       double* resid2) {
  // rest_draw: the total in the scale of the chunk and tile sums (2^{-m_i}
  // times the true one for a row of the underflow rescue, else the same)
  const int lane32 = threadIdx.x & 31;
  const double tot = rest_draw[i];
  const bool any = rest[i] > 0.0 && tot > 0.0;
  double resid = 0.0;
  const int c = invert_half<1>(
      P, u * tot,
      [&](int k0, double (&v)[1]) { v[0] = any && k0 + lane32 < P ? chunk_t[i * P + k0 + lane32] : 0.0; }, &resid);
  const int64_t t0 = (int64_t)(c < 0 ? 0 : c) * kChunkTiles;
  const int nt = c < 0 ? 0 : (int)((ntile - t0) < kChunkTiles ? (ntile - t0) : kChunkTiles);
  static_assert(kChunkTiles == 4 * 32, "one scan of four a lane");
  const int tl = invert_half<4>(
      kChunkTiles, resid,
      [&](int, double (&v)[4]) {
        // tstride and t0 are multiples of 16: aligned, and inside the row
        const int k = 4 * lane32;
        float4 f = make_float4(0.f, 0.f, 0.f, 0.f);
        if (k < nt) f = *reinterpret_cast<const float4*>(&tp[i * tstride + t0 + k]);
        v[0] = (double)f.x;
        v[1] = k + 1 < nt ? (double)f.y : 0.0;
        v[2] = k + 2 < nt ? (double)f.z : 0.0;
        v[3] = k + 3 < nt ? (double)f.w : 0.0;
      },
      resid2);
  if (tl < 0) {
    *resid2 = 0.0;
    return ntile;
  }
  return t0 + tl;
}

// Step 3 (half a wave): the row of tile T for remainder resid2, or -1 (also
// for T = ntile).
template <RowRead ROWS>
__device__ inline int64_t draw_row_of(const float* __restrict__ X, int64_t n, int64_t ntile, int d, double a,
                                      int64_t i, int64_t T, double resid2, double sh) {
  const int64_t rb = T * 32, j = rb + (threadIdx.x & 31);
  const bool live = T < ntile && j < n && j != i;
  const double D = row_dist2<ROWS>(X + i * d, X, d, live ? j : i, d);
  // a shifted row's values are 2^{E - m_i} with E = -a log2(e) D in one
  // exponent (2^{-m_i} alone overflows for m_i < -1024, and exp(-a D) is
  // subnormal there)
  double kv = 0.0;
  if (live) kv = sh == 0.0 ? exp(-a * D) : exp2(fma(-a * kLog2eS, D, -sh));
  double resid3 = 0.0;
  const int jl = invert_half<1>(32, resid2, [&](int, double (&v)[1]) { v[0] = kv; }, &resid3);
  return jl >= 0 ? rb + jl : -1;
}

__device__ inline void draw_store(int64_t e, int64_t i, int64_t pick, int s, const double* __restrict__ rest,
                                  int64_t* __restrict__ src, int64_t* __restrict__ dst, double* __restrict__ w) {
  src[e] = i;
  dst[e] = pick;
  w[e] = pick >= 0 ? 1.0 / ((double)s * (1.0 / rest[i] + 1.0 / rest[pick])) : 0.0;
}

// Fused draw, half a wave per draw e = (node i, draw r).
template <RowRead ROWS>
__global__ __launch_bounds__(256) void draw_exact(const float* __restrict__ X, int64_t n, int d, double a, int s,
                                                  uint64_t seed, int P, int64_t ntile, int64_t tstride,
                                                  const double* __restrict__ chunk_t, const float* __restrict__ tp,
                                                  const double* __restrict__ rest,
                                                  const double* __restrict__ rest_draw,
                                                  const double* __restrict__ shift, int64_t* __restrict__ src,
                                                  int64_t* __restrict__ dst, double* __restrict__ w) {
  const int64_t e0 = (int64_t)blockIdx.x * 8 + (threadIdx.x >> 5);
  const int64_t e = e0 < n * s ? e0 : n * s - 1;  // the last wave's spare half repeats
  const int64_t i = node_of(e, s);
  double resid2 = 0.0;
  const int64_t T = draw_tile_of(i, draw_uniform(seed, i, (int)(e - i * s)), P, ntile, tstride, chunk_t, tp, rest,
                                 rest_draw, &resid2);
  const int64_t pick = draw_row_of<ROWS>(X, n, ntile, d, a, i, T, resid2, shift[i]);
  if ((threadIdx.x & 31) == 0 && e0 == e) draw_store(e, i, pick, s, rest, src, dst, w);
}

// Split draw, step 1 (half a wave per draw e): tile[e], order[e] = e and the
// remainder.
__global__ __launch_bounds__(256) void draw_tile(int64_t n, int s, uint64_t seed, int P, int64_t ntile,
                                                 int64_t tstride, const double* __restrict__ chunk_t,
                                                 const float* __restrict__ tp, const double* __restrict__ rest,
                                                 const double* __restrict__ rest_draw, uint32_t* __restrict__ tile,
                                                 uint32_t* __restrict__ order, double* __restrict__ resid_out) {
  const int64_t e0 = (int64_t)blockIdx.x * 8 + (threadIdx.x >> 5);
  const int64_t e = e0 < n * s ? e0 : n * s - 1;
  const int64_t i = node_of(e, s);
  double resid2 = 0.0;
  const int64_t T = draw_tile_of(i, draw_uniform(seed, i, (int)(e - i * s)), P, ntile, tstride, chunk_t, tp, rest,
                                 rest_draw, &resid2);
  if ((threadIdx.x & 31) == 0 && e0 == e) {
    tile[e] = (uint32_t)T;
    order[e] = (uint32_t)e;
    resid_out[e] = resid2;
  }
}

// Split draw, step 2, half a wave per draw in the order given by `order`
// (tile[k] is the tile of draw order[k]).  Workgroups go round-robin to the 8
// XCDs: block b works on logical block (b % 8) per + b / 8 (the grid is 8 per
// blocks), i.e. slots [8 L, 8 L + 8).
template <RowRead ROWS>
__global__ __launch_bounds__(256) void draw_row(const float* __restrict__ X, int64_t n, int d, double a, int s,
                                                int64_t ntile, int per, const uint32_t* __restrict__ tile,
                                                const uint32_t* __restrict__ order,
                                                const double* __restrict__ resid_in,
                                                const double* __restrict__ rest, const double* __restrict__ shift,
                                                int64_t* __restrict__ src, int64_t* __restrict__ dst,
                                                double* __restrict__ w) {
  const int b = blockIdx.x;
  const int64_t slot0 = ((int64_t)(b % 8) * per + b / 8) * 8 + (threadIdx.x >> 5);
  const int64_t slot = slot0 < n * s ? slot0 : n * s - 1;
  const int64_t e = (int64_t)order[slot];
  const int64_t i = node_of(e, s);
  const int64_t pick = draw_row_of<ROWS>(X, n, ntile, d, a, i, tile[slot], resid_in[e], shift[i]);
  if ((threadIdx.x & 31) == 0 && slot0 == slot) draw_store(e, i, pick, s, rest, src, dst, w);
}

stag_status sample_exact(const float* X, int64_t n, int d, double a, int form, int s, uint64_t seed, int64_t* src,
                         int64_t* dst, double* w, double* deg_out, hipStream_t st) {
  Workspace ws(st);
  Operands xo, qo;
  STAG_TRY(alloc_operands(form, n, d, false, ws, &xo));
  STAG_TRY(alloc_operands(form, n, d, true, ws, &qo));
  const int64_t nqt = qo.rows_pad / query_tile_rows();
  const int64_t nr = round_up(n, 64);
  int *flag = nullptr, *qflag = nullptr;
  STAG_TRY(ws.alloc(&flag, (size_t)(nr + nqt)));
  qflag = flag + nr;
  STAG_TRY(prep_operand_pair(X, X, a, xo, qo, false, flag, (size_t)(nr + nqt), st));
  const int P = (int)exact_chunks(xo.rows_pad);
  const int64_t ntile = xo.rows_pad / 32;
  const int64_t tstride = round_up(ntile, 16);
  double* partial = nullptr;
  float* tp = nullptr;
  double* rest = nullptr;
  double* chunk_t = nullptr;
  STAG_TRY(ws.alloc(&partial, (size_t)P * qo.rows_pad));
  STAG_TRY(ws.alloc(&chunk_t, (size_t)P * n));
  STAG_TRY(ws.alloc(&tp, (size_t)tstride * qo.rows_pad));
  STAG_TRY(ws.alloc(&rest, (size_t)n));
  TileExtra ex;
  ex.self = 1;
  ex.tp = tp;
  ex.ntile = tstride;
  STAG_TRY(alloc_parts(xo, qo, STAG_KERNEL_GAUSSIAN, ws, &ex));
  STAG_TRY(launch_exact_tiles(xo, qo, partial, ex, st));
  // underflow rescue: rows whose sum is below kRescueBelow get their
  // exponents shifted by their maximum over the other rows and a second self
  // pass (over their 128-row tiles only; other workgroups return at once)
  double *rest_draw = nullptr, *shift = nullptr;
  float* off2 = nullptr;
  STAG_TRY(ws.alloc(&rest_draw, (size_t)n));
  STAG_TRY(ws.alloc(&shift, (size_t)qo.rows_pad));
  STAG_TRY(ws.alloc(&off2, (size_t)qo.rows_pad));
  hipLaunchKernelGGL(row_rest, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, st, partial, P, qo.rows_pad, n, rest,
                     deg_out, chunk_t, flag, qflag, (int)query_tile_rows());
  STAG_TRY(check_launch("row_rest"));
  STAG_TRY(rescue_offsets(xo, qo, P, a, 1, flag, qflag, off2, shift, ws, st));
  Operands q2 = qo;
  q2.off = off2;
  TileExtra exr = ex;
  exr.qtile_active = qflag;
  STAG_TRY(launch_exact_tiles(xo, q2, partial, exr, st));
  hipLaunchKernelGGL(rescue_rows, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, st, partial, P, qo.rows_pad, n,
                     flag, shift, rest, rest_draw, deg_out, chunk_t);
  STAG_TRY(check_launch("rescue_rows"));
  const int64_t nd = n * s;
  const RowRead rows = row_read(d);
  auto by_rows = [&](auto own, auto quad4, auto quad) { return rows == kOwnRow ? own : rows == kQuad4 ? quad4 : quad; };
  ScopedTimer tm("simgraph_draw_exact", st);
  // the sort carries draw indices in 32 bits (the n x n/32 tile sums above
  // bound n far below this in practice)
  const bool sortable = nd < ((int64_t)1 << 31);
  const bool cached = n * d * (int64_t)sizeof(float) <= kDrawFusedMaxBytes;
  if (d <= kDrawFusedMaxDim || (d <= 256 && (cached || !sortable))) {
    hipLaunchKernelGGL(by_rows(draw_exact<kOwnRow>, draw_exact<kQuad4>, draw_exact<kQuad>),
                       dim3((unsigned)ceil_div(nd, 8)), dim3(256), 0, st, X, n, d, a, s, seed, P, ntile, tstride,
                       chunk_t, tp, rest, rest_draw, shift, src, dst, w);
    return check_launch("draw_exact");
  }
  if (!sortable) return fail(STAG_E_UNSUPPORTED, "stag_simgraph_sample: n * s >= 2^31 draws");
  uint32_t *tile = nullptr, *order = nullptr, *tile_s = nullptr, *order_s = nullptr;
  double* resid = nullptr;
  STAG_TRY(ws.alloc(&tile, (size_t)nd));
  STAG_TRY(ws.alloc(&order, (size_t)nd));
  STAG_TRY(ws.alloc(&tile_s, (size_t)nd));
  STAG_TRY(ws.alloc(&order_s, (size_t)nd));
  STAG_TRY(ws.alloc(&resid, (size_t)nd));
  hipLaunchKernelGGL(draw_tile, dim3((unsigned)ceil_div(nd, 8)), dim3(256), 0, st, n, s, seed, P, ntile, tstride,
                     chunk_t, tp, rest, rest_draw, tile, order, resid);
  STAG_TRY(check_launch("draw_tile"));
  int bits = 1;
  while (((int64_t)1 << bits) <= ntile) ++bits;  // keys 0..ntile
  STAG_TRY(radix_sort_pairs_u32(tile, order, tile_s, order_s, nd, bits, ws, st));
  const int per = (int)ceil_div(ceil_div(nd, 8), 8);
  hipLaunchKernelGGL(by_rows(draw_row<kOwnRow>, draw_row<kQuad4>, draw_row<kQuad>), dim3((unsigned)(8 * per)),
                     dim3(256), 0, st, X, n, d, a, s, ntile, per, tile_s, order_s, resid, rest, shift, src, dst, w);
  return check_launch("draw_row");
}

}  // namespace
}  // namespace stag

extern "C" int32_t stag_simgraph_draws_per_node(int64_t n, int32_t samples_per_node) {
  if (n < 1 || samples_per_node < 0 || samples_per_node > 64) return -1;
  if (samples_per_node > 0) return samples_per_node;
  int s = 0;
  while (((int64_t)1 << s) < n) ++s;  // ceil(log2 n)
  return s < 1 ? 1 : s;
}

extern "C" stag_status stag_simgraph_sample(const float* X, int64_t n, int32_t d, double a, int32_t samples_per_node,
                                            int32_t kde_mode, int32_t form, double eps, const stag_lsh_params* lsh,
                                            uint64_t seed, int64_t* src_out, int64_t* dst_out, double* w_out,
                                            double* deg_out, hipStream_t stream) {
  using namespace stag;
  if (!X || !src_out || !dst_out || !w_out) return fail(STAG_E_INVAL, "stag_simgraph_sample: NULL argument");
  if (n < 2 || d < 1 || n > 2147483647LL) return fail(STAG_E_INVAL, "stag_simgraph_sample: need 2 <= n < 2^31, d >= 1");
  if (!(a > 0.0) || !std::isfinite(a)) return fail(STAG_E_INVAL, "stag_simgraph_sample: a must be positive and finite");
  if (samples_per_node < 0 || samples_per_node > 64)
    return fail(STAG_E_INVAL, "stag_simgraph_sample: samples_per_node must be in [0, 64]");
  const int s = stag_simgraph_draws_per_node(n, samples_per_node);
  clear_error();
  if (kde_mode == STAG_SIMGRAPH_EXACT) {
    if (form < STAG_FORM_FP32 || form > STAG_FORM_BF16_SPLIT3)
      return fail(STAG_E_INVAL, "stag_simgraph_sample: unknown form %d", form);
    if (exact_padded_dim(d) == 0 || (d > 256 && form == STAG_FORM_BF16_SPLIT3))
      return fail(STAG_E_UNSUPPORTED, "stag_simgraph_sample: d = %d not supported by this form", d);
    return sample_exact(X, n, d, a, form, s, seed, src_out, dst_out, w_out, deg_out, stream);
  }
  if (kde_mode == STAG_SIMGRAPH_LSH) {
    stag_lsh_index* idx = nullptr;
    STAG_TRY(stag_lsh_index_create(X, n, d, a, eps, lsh, &idx, stream));
    const stag_status st = lsh_sample_edges(idx, s, seed, src_out, dst_out, w_out, deg_out, stream);
    (void)hipStreamSynchronize(stream);
    stag_lsh_index_destroy(idx);
    return st;
  }
  return fail(STAG_E_INVAL, "stag_simgraph_sample: unknown kde_mode %d", kde_mode);
}
