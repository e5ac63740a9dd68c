// Similarity-graph edge sampling through a KDE tree (Sec. "The MS
// Algorithm": every edge (i, j) is drawn with probability close to eq.
// (sampling_prob), the kernel sums coming from a KDE algorithm used as a
// black box; the black box here is the random-sampling estimator of Sec.
// "Kernel Density Estimation", evaluated per tree node).
//
// Tree: leaves are blocks of 32 consecutive rows (nb = ceil(n/32)); h =
// ceil(log2 nb); node (l, k) holds rows [k 32 2^(h-l), (k+1) 32 2^(h-l))
// clipped to [0, n).  No tree is stored: a node is its index range.
//
// est(i, node): P rows; P <= t: the exact sum of k_ij over its rows j != i;
// else (P/t) sum_{c<t} k_{i,j_c} [j_c != i], j_c = lo + floor(U_c P).
// Draw (i, r): at level l the children A, B get eA, eB from their own
// sample streams, u = U(i, r, l); go to A iff u (eA + eB) < eA, and if both
// are 0 to the child with more rows other than i (A on a tie).  At the leaf
// an inverse CDF over its rows' exact values (0 for j = i) on u = U(i, r, h);
// if they are all 0, the floor(u m)-th of its m rows other than i.
// Degrees: rest_i = est(i, root) with t_deg samples; deg = 1 + rest; the
// draw (i, j) gets weight 1/(s (1/rest_i + 1/rest_j)) (0 if one is 0).
//
// Randomness: SplitMix64 (Steele, Lea & Flood 2014) counter streams; output
// c of stream (seed, tag, a, b) is mix(S + (c+1) gamma) with S =
// mix(mix(mix(seed ^ tag) ^ a) ^ b).  Sample streams: tag "TREE", a = i,
// b = r << 16 | l << 1 | side; descent uniforms: tag "TRUN", a = i, b = r,
// c = l; degree samples: tag "TDEG", a = i, b = 0.  A uniform is the top 53
// bits times 2^-53 and an index is floor(u53 P / 2^53), exact in integers.
//
// Layout and work: one wave per draw and level; lanes 0-31 hold child A's
// samples (or rows), lanes 32-63 child B's (two or four draws a wave where 16
// or 8 lanes hold a child's), one kernel value per lane from
// fp64 direct differences, whose rows four lanes read together (row_dist2);
// the values of a child are summed in a fixed butterfly order.  Work per draw: h
// levels x 2t kernel values + 32 at the leaf, each d fp64 operations on a
// gathered row.  Results are deterministic; against a sequential fp64 sum
// they differ by rounding only, which moves a decision only when its target
// lies within that rounding of a boundary.
#include <utility>

#include "row_dist.h"
#include "runtime.h"
#include "sort.h"

namespace stag {
namespace {

constexpr uint64_t kTagTreeSamples = 0x54524545ULL;  // "TREE"
constexpr uint64_t kTagTreeUniform = 0x5452554EULL;  // "TRUN"
constexpr uint64_t kTagTreeDegree = 0x54444547ULL;   // "TDEG"
constexpr uint64_t kGammaTree = 0x9E3779B97F4A7C15ULL;
constexpr int kTreeLeaf = 32;
constexpr int kTreeWaves = 4;

__device__ inline uint64_t tmix(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
  return z ^ (z >> 31);
}
__device__ inline uint64_t tstream(uint64_t seed, uint64_t tag, uint64_t a, uint64_t b) {
  return tmix(tmix(tmix(seed ^ tag) ^ a) ^ b);
}
__device__ inline uint64_t tout(uint64_t st, uint64_t c) { return tmix(st + (c + 1) * kGammaTree); }
__device__ inline double tuniform(uint64_t bits) { return (double)(bits >> 11) * 0x1.0p-53; }
// floor(u P / 2^53) for the top 53 bits u of `bits`, P < 2^31: with u =
// h 2^32 + l, the bits of l P below 2^32 cannot carry.
__device__ inline uint32_t tpick(uint64_t bits, uint32_t P) {
  const uint64_t u = bits >> 11;
  return (uint32_t)(((u >> 32) * P + __umulhi((uint32_t)u, P)) >> 21);
}

// Draw e < 2^31 belongs to row e / s; the quotient as (e m) >> shift, exact
// with m = ceil(2^shift / s), shift = 31 + ceil(log2 s) (m < 2^32).
struct DivBy {
  uint32_t s, m;
  int shift;
};
inline DivBy div_by(uint32_t s) {
  int l = 0;
  while ((1ull << l) < s) ++l;
  return {s, (uint32_t)(((1ull << (31 + l)) + s - 1) / s), 31 + l};
}
__host__ __device__ inline uint32_t quotient(uint32_t e, const DivBy& q) {
  return (uint32_t)(((uint64_t)e * q.m) >> q.shift);
}

// Sum over each group of LANES lanes (fixed butterfly).
template <int LANES>
__device__ inline double lanes_sum(double v) {
#pragma unroll
  for (int o = LANES / 2; o > 2; o >>= 1) v += __shfl_xor(v, o);
  v += quad_perm<0x4E>(v);
  return v + quad_perm<0xB1>(v);
}

// rest[i] = est(i, root) with t_deg samples; one wave per row i.
template <RowRead ROWS>
__global__ __launch_bounds__(256, 4) void tree_degrees(const float* __restrict__ X, int64_t n, int d, double a,
                                                    int64_t t_deg, uint64_t seed, double* __restrict__ rest,
                                                    double* __restrict__ deg_out) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int64_t i = (int64_t)blockIdx.x * kTreeWaves + wave;
  if (i >= n) return;
  double s = 0.0;
  const bool all = n <= t_deg;
  const int64_t count = all ? n : t_deg;
  const uint64_t st = tstream(seed, kTagTreeDegree, (uint64_t)i, 0);
  for (int64_t c0 = 0; c0 < count; c0 += 64) {
    const int64_t c = c0 + lane;
    int64_t j = i;
    if (c < count) j = all ? c : tpick(tout(st, (uint64_t)c), (uint32_t)n);
    const double D = row_dist2<ROWS>(X + i * d, X, d, j, d);
    if (j != i) s += exp(-a * D);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if (n > t_deg) s = s * ((double)n / (double)t_deg);
  if (lane == 0) {
    rest[i] = s;
    if (deg_out) deg_out[i] = 1.0 + s;
  }
}

// Draws run level by level: one launch per tree level, then the draws are
// sorted (stable radix sort) by the node they reached, so that the waves of
// a launch that work in the same node are neighbours; with the XCD-aware
// block order below each XCD takes a contiguous range of nodes, and from the
// level where a node's rows fit an XCD's L2 the gathers hit in L2.  The
// order changes only where a draw runs, not what it computes.
//
// Workgroups go round-robin to the 8 XCDs: block b works on logical block
// (b % 8) per + b / 8 (the grid is 8 per blocks), i.e. slots
// [4 L, 4 L + 4) of the sorted order, one per wave.
__device__ inline int64_t tree_slot(int per) {
  const int b = blockIdx.x;
  const int64_t L = (int64_t)(b % 8) * per + b / 8;
  return L * kTreeWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
}

// perm[w] = w, node[w] = 0.
__global__ void tree_init(uint32_t* __restrict__ perm, uint32_t* __restrict__ node, int64_t total) {
  const int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (w < total) {
    perm[w] = (uint32_t)w;
    node[w] = 0;
  }
}

// One level l < h for the draw in each slot: node_in[slot] -> node_out[slot].
// LANES lanes per child (t <= LANES), 2 LANES per draw: with few samples a
// wave takes two or four draws (n = 5e4, d = 30, t = 16: one draw a wave 17.9 ms
// a call before the wider loads, two draws 10.5, and 5.4 with them).
template <RowRead ROWS, int LANES>
__global__ __launch_bounds__(256, LANES == 32 ? 6 : 5) void tree_level(
    const float* __restrict__ X, int64_t n, int d, double a, DivBy s, int t, int h, int l, uint64_t seed,
    const uint32_t* __restrict__ perm, const uint32_t* __restrict__ node_in, uint32_t* __restrict__ node_out,
    int64_t total, int per) {
  constexpr int kDraws = 32 / LANES;  // of a wave
  const int lane = threadIdx.x & 63;
  const int64_t slot0 = kDraws * tree_slot(per);
  if (slot0 >= total) return;
  // the last wave's spare lanes repeat its last draw
  const int64_t slot = kDraws == 1 ? slot0 : min(total - 1, slot0 + lane / (2 * LANES));
  const uint32_t e = perm[slot];
  const int64_t i = quotient(e, s);
  const uint32_t r = e - (uint32_t)i * s.s;
  const int side = (lane / LANES) & 1, c = lane % LANES;
  const int64_t k = node_in[slot];
  const int64_t span = (int64_t)kTreeLeaf << (h - l - 1);
  const int64_t mid = min(n, (2 * k + 1) * span);
  const int64_t lo = side ? mid : min(n, 2 * k * span), hi = side ? min(n, (2 * k + 2) * span) : mid;
  const uint32_t P = (uint32_t)(hi - lo);
  const uint64_t si = tmix(tmix(seed ^ kTagTreeSamples) ^ (uint64_t)i);
  const uint64_t b = ((uint64_t)r << 16) | ((uint64_t)l << 1);
  const uint64_t stA = tmix(si ^ b), stB = tmix(si ^ (b | 1));
  int64_t j = i;  // i itself: no value
  if (P > (uint32_t)t) {
    if (c < t) j = lo + tpick(tout(side ? stB : stA, (uint64_t)c), P);
  } else if (c < (int)P) {
    j = lo + c;
  }
  const double D = row_dist2<ROWS>(X + i * d, X, d, j, d);
  const double v = j != i ? exp(-a * D) : 0.0;
  double est = lanes_sum<LANES>(v);
  if (P > (uint32_t)t) est = est * ((double)P / (double)t);
  const double eA = __shfl(est, 0, 2 * LANES), eB = __shfl(est, LANES, 2 * LANES);
  const double u = tuniform(tout(tstream(seed, kTagTreeUniform, (uint64_t)i, (uint64_t)r), (uint64_t)l));
  const double tot = eA + eB;
  bool left;
  if (tot > 0.0) {
    left = u * tot < eA;
  } else {
    const int64_t aLo = min(n, 2 * k * span), aHi = min(n, (2 * k + 1) * span), bHi = min(n, (2 * k + 2) * span);
    const int64_t mA = (aHi - aLo) - ((i >= aLo && i < aHi) ? 1 : 0);
    const int64_t mB = (bHi - aHi) - ((i >= aHi && i < bHi) ? 1 : 0);
    left = mA >= mB;
  }
  if (lane % (2 * LANES) == 0) node_out[slot] = (uint32_t)(left ? 2 * k : 2 * k + 1);
}

// The leaf (level h) of the draw in each slot, two draws per wave (lanes 0-31
// and 32-63): inverse CDF over its rows in row order; outputs at the draw's own
// index e = i s + r.
template <RowRead ROWS>
__global__ __launch_bounds__(256, 5) void tree_leaf(const float* __restrict__ X, int64_t n, int d, double a, DivBy s,
                                                 int h, uint64_t seed, const uint32_t* __restrict__ perm,
                                                 const uint32_t* __restrict__ node, const double* __restrict__ rest,
                                                 int64_t* __restrict__ src, int64_t* __restrict__ dst,
                                                 double* __restrict__ w, int64_t total, int per) {
  const int side = (threadIdx.x >> 5) & 1, c = threadIdx.x & 31;
  const int64_t slot = 2 * tree_slot(per) + side;
  const bool active = slot < total;
  const uint32_t e = active ? perm[slot] : 0;
  const int64_t i = quotient(e, s);
  const uint32_t r = e - (uint32_t)i * s.s;
  const int64_t k = active ? node[slot] : 0;
  const int64_t lo = min(n, k * kTreeLeaf), hi = min(n, (k + 1) * kTreeLeaf);
  const int64_t j = lo + c < hi ? lo + c : i;
  const double D = row_dist2<ROWS>(X + i * d, X, d, j, d);
  const double v = j != i ? exp(-a * D) : 0.0;
  double incl = v;  // inclusive prefix over the half's lanes
#pragma unroll
  for (int o = 1; o < 32; o <<= 1) {
    const double y = __shfl_up(incl, o, 32);
    if (c >= o) incl += y;
  }
  const double T = __shfl(incl, 31, 32);
  const double u = tuniform(tout(tstream(seed, kTagTreeUniform, (uint64_t)i, (uint64_t)r), (uint64_t)h));
  int64_t pick;
  // only a row with a positive value can take the draw (the butterfly prefix
  // need not be exactly monotone where a value is 0)
  const double target = u * T;
  const uint64_t positive = __ballot(v > 0.0), above = __ballot(v > 0.0 && incl > target);
  if (T > 0.0) {
    const uint32_t pass = (uint32_t)(above >> (32 * side));
    if (pass != 0) {
      pick = lo + __builtin_ctz(pass);
    } else {  // rounding left the target above the total: the last positive value
      pick = lo + 31 - __builtin_clz((uint32_t)(positive >> (32 * side)));
    }
  } else {
    const int64_t m = (hi - lo) - ((i >= lo && i < hi) ? 1 : 0);
    const int64_t idx = (int64_t)(u * (double)m);
    pick = lo + idx;
    if (i >= lo && i < hi && pick >= i) ++pick;
  }
  if (c == 0 && active) {
    src[e] = i;
    dst[e] = pick;
    const double ri = rest[i], rj = rest[pick];
    w[e] = (ri > 0.0 && rj > 0.0) ? 1.0 / ((double)s.s * (1.0 / ri + 1.0 / rj)) : 0.0;
  }
}

}  // namespace
}  // namespace stag

extern "C" stag_status stag_simgraph_sample_tree(const float* X, int64_t n, int32_t d, double a,
                                                 int32_t samples_per_node, int32_t est_samples,
                                                 int64_t degree_samples, uint64_t seed, int64_t* src_out,
                                                 int64_t* dst_out, double* w_out, double* deg_out,
                                                 hipStream_t stream) {
  using namespace stag;
  const char* fn = "stag_simgraph_sample_tree";
  if (!X || !src_out || !dst_out || !w_out) return fail(STAG_E_INVAL, "%s: NULL argument", fn);
  if (n < 2 || n > 2147483647LL || d < 1) return fail(STAG_E_INVAL, "%s: need 2 <= n < 2^31, d >= 1", fn);
  if (d > 1024) return fail(STAG_E_UNSUPPORTED, "%s: d = %d > 1024 is not supported", fn, d);
  if (!(a > 0.0) || !std::isfinite(a)) return fail(STAG_E_INVAL, "%s: a must be positive and finite", fn);
  if (samples_per_node < 0 || samples_per_node > 64)
    return fail(STAG_E_INVAL, "%s: samples_per_node must be in [0, 64]", fn);
  if (est_samples < 1 || est_samples > 32) return fail(STAG_E_INVAL, "%s: est_samples must be in [1, 32]", fn);
  if (degree_samples < 1) return fail(STAG_E_INVAL, "%s: degree_samples must be >= 1", fn);
  const int s = stag_simgraph_draws_per_node(n, samples_per_node);
  const int64_t draws = n * s;
  if (draws >= 2147483647LL) return fail(STAG_E_INVAL, "%s: n * samples_per_node must be < 2^31", fn);
  const int64_t nb = (n + kTreeLeaf - 1) / kTreeLeaf;
  int h = 0;
  while (((int64_t)1 << h) < nb) ++h;
  clear_error();
  Workspace ws(stream);
  double* rest = nullptr;
  STAG_TRY(ws.alloc(&rest, (size_t)n));
  const RowRead rows = row_read(d);
  auto by_rows = [&](auto own, auto quad4, auto quad) { return rows == kOwnRow ? own : rows == kQuad4 ? quad4 : quad; };
  {
    ScopedTimer tm("tree_degrees", stream);
    hipLaunchKernelGGL(by_rows(tree_degrees<kOwnRow>, tree_degrees<kQuad4>, tree_degrees<kQuad>),
                       dim3((unsigned)ceil_div(n, kTreeWaves)), dim3(256), 0, stream, X, n, (int)d, a, degree_samples,
                       seed, rest, deg_out);
    STAG_TRY(check_launch("tree_degrees"));
  }
  // draws level by level, sorted by node between levels
  const DivBy by = div_by((uint32_t)s);
  const int lanes = est_samples <= 8 ? 8 : est_samples <= 16 ? 16 : 32;
  const int per = (int)ceil_div(ceil_div(draws, kTreeWaves * (32 / lanes)), 8);
  const dim3 grid((unsigned)(8 * per));
  auto level = lanes == 8    ? by_rows(tree_level<kOwnRow, 8>, tree_level<kQuad4, 8>, tree_level<kQuad, 8>)
               : lanes == 16 ? by_rows(tree_level<kOwnRow, 16>, tree_level<kQuad4, 16>, tree_level<kQuad, 16>)
                             : by_rows(tree_level<kOwnRow, 32>, tree_level<kQuad4, 32>, tree_level<kQuad, 32>);
  uint32_t *perm = nullptr, *perm2 = nullptr, *node = nullptr, *node2 = nullptr;
  STAG_TRY(ws.alloc(&perm, (size_t)draws));
  STAG_TRY(ws.alloc(&perm2, (size_t)draws));
  STAG_TRY(ws.alloc(&node, (size_t)draws));
  STAG_TRY(ws.alloc(&node2, (size_t)draws));
  hipLaunchKernelGGL(tree_init, dim3((unsigned)ceil_div(draws, 256)), dim3(256), 0, stream, perm, node, draws);
  STAG_TRY(check_launch("tree_init"));
  for (int l = 0; l < h; ++l) {
    {
      ScopedTimer tm("tree_draws", stream);
      hipLaunchKernelGGL(level, grid, dim3(256), 0, stream, X, n, (int)d, a, by, (int)est_samples, h, l, seed,
                         perm, node, node2, draws, per);
      STAG_TRY(check_launch("tree_level"));
    }
    ScopedTimer tm("tree_sort", stream);
    STAG_TRY(radix_sort_pairs_u32(node2, perm, node, perm2, draws, l + 1, ws, stream));
    std::swap(perm, perm2);
  }
  {
    ScopedTimer tm("tree_draws", stream);
    const int leaf_per = (int)ceil_div(ceil_div(draws, 2 * kTreeWaves), 8);
    hipLaunchKernelGGL(by_rows(tree_leaf<kOwnRow>, tree_leaf<kQuad4>, tree_leaf<kQuad>),
                       dim3((unsigned)(8 * leaf_per)), dim3(256), 0, stream, X, n, (int)d, a, by, h, seed, perm, node,
                       rest, src_out, dst_out, w_out, draws, leaf_per);
    STAG_TRY(check_launch("tree_leaf"));
  }
  return STAG_OK;
}
