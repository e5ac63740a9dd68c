// Exact kernel density on the gfx950 matrix cores: operand preparation, the
// cross-chunk reduction and the C ABI entry points.  The tiles themselves are
// in kde_tiles.h.
//
// S(q) = sum_i k(||q - x_i||)   (Sec. "Kernel Density Estimation": the density
// K(q) = S(q)/n; ExactGaussianKDE evaluates it naively in O(dmn)); k is the
// Gaussian exp(-a r^2), the exponential exp(-a r) or the logistic
// 4/(2 + e^{ar} + e^{-ar}) kernel.
//
// The squared distance is expanded, ||q-x||^2 = ||q||^2 + ||x||^2 - 2 q.x,
// and scaled into a base-2 exponent
//     E = -lambda ||q-x||^2 = alpha_q + beta_x + (s q).x,
// alpha = -lambda ||q||^2, beta = -lambda ||x||^2, s = 2 lambda, with
// lambda = a log2(e) for the Gaussian kernel and (a log2(e))^2 for the other
// two.  The matrix cores produce the cross term from the (split) operands on
// top of alpha + beta; the epilogue maps E to the kernel value and sums.
//
// Pipeline of one call:
//   prep_rows  (data)    fp64 norms, beta, operand copy/split, padding rows
//   prep_rows  (queries) fp64 norms, alpha, scaled operand copy/split
//   tile_*               grid = (query tile of 128) x (data chunk of 4096 rows);
//                        4 waves, each owns 32 queries held in registers as
//                        the B operand; 32-row data tiles are streamed
//                        through double-buffered LDS as the A operand; per
//                        tile each lane adds its 16 kernel values in fp32 and
//                        flushes them into an fp64 accumulator.
//   reduce               S(q) = sum over chunks in chunk order (fp64), bound.
// The value of a query depends only on its own row, X and a: chunking and
// tiling are functions of n alone, so results are identical whatever m is and
// whatever other queries share a launch.
#include <cstring>
#include <mutex>
#include <type_traits>

#include "runtime.h"
#include "kde_exact.h"
#include "kde_tiles.h"

// Scratch of stag_kde_exact_noalloc: one array per device (the runtime gives
// each device its own copy of a __device__ variable), kept until the process
// ends.  Host code never passes `scratch` itself to a kernel (on the host it
// names a stand-in, not device memory): the device address comes from
// hipGetSymbolAddress, looked up once per device with that device current.
static constexpr size_t kScratchBytes = (size_t)128 << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace stag {
namespace {

using namespace tiles;

template <int FORM>
__device__ inline void split_value(float v, unsigned short* p) {
  if constexpr (FORM == STAG_FORM_FP16_SPLIT) {
    if (!(fabsf(v) < 65504.0f)) {  // out of fp16 range: poison the result
      p[0] = 0x7E00; p[1] = 0;
      return;
    }
    p[0] = f16_rne(v);
    p[1] = f16_rne(v - f16_to_f32(p[0]));
  } else if constexpr (FORM == STAG_FORM_BF16_SPLIT) {
    p[0] = bf16_rne(v);
    p[1] = bf16_rne(v - bf16_to_f32(p[0]));
  } else {  // three bf16 parts
    p[0] = bf16_rne(v);
    float r = v - bf16_to_f32(p[0]);
    p[1] = bf16_rne(r);
    p[2] = bf16_rne(r - bf16_to_f32(p[1]));
  }
}

// One side (data or queries) of an operand preparation.  `scale` multiplies
// the operand (1 for data, 2a log2 e for queries); off = neg_a_log2e ||row||^2
// in fp32.  Rows >= n are padding; with map, row r is src row map[r] (-1:
// padding), n unused.  max_nrm_bits (null: not wanted) takes the largest norm.
struct PrepSide {
  const float* src;
  int64_t n, rows_pad;
  double scale, neg_a_log2e;
  int is_query;
  void* part[3];
  float* off;
  double* nrm;
  unsigned long long* max_nrm_bits;
  const int* map;
  int64_t blocks;  // workgroups of this side
};

// Words that the preparation clears on the way (flags read by later launches).
struct ZeroRange {
  uint32_t* p = nullptr;
  int64_t words = 0;
};
__device__ inline void clear_range(const ZeroRange& z) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < z.words; i += (int64_t)gridDim.x * 256) z.p[i] = 0u;
}

// Largest norm of a workgroup's rows, one atomic per workgroup.
__device__ inline void block_max_norm(double mx, unsigned long long* out) {
  __shared__ double wmax[4];
  for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o));
  if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = mx;
  __syncthreads();
  if (threadIdx.x == 0) {
    const double b = fmax(fmax(wmax[0], wmax[1]), fmax(wmax[2], wmax[3]));
    atomicMax(out, (unsigned long long)__double_as_longlong(b));
  }
}

// Both sides of a call in one launch, LPR lanes per row (a power of two, 8
// coordinates each), kPrepRows rows per thread with their loads in flight
// together; VEC: every row starts at 16 bytes.  Bound by the rows' traffic (X
// read once, the operands written once): 300,000 rows of 64 into the fp16
// split form take 37 us (154 MB); a wave per row with one load in flight
// took 93.
constexpr int kPrepRows = 4;
template <int FORM, int LPR, bool VEC>
__global__ __launch_bounds__(256) void prep_rows(PrepSide x, PrepSide q, int d, int dp, ZeroRange zero) {
  clear_range(zero);
  const bool second = (int64_t)blockIdx.x >= x.blocks;
  const PrepSide& side = second ? q : x;
  const int64_t blk = second ? (int64_t)blockIdx.x - x.blocks : (int64_t)blockIdx.x;
  constexpr int RPB = 256 / LPR;  // rows per round of the block
  const int l = threadIdx.x % LPR, j0 = l * 8;
  const bool act = j0 < dp;
  int64_t row[kPrepRows];
  bool real[kPrepRows];
  float v[kPrepRows][8];
#pragma unroll
  for (int k = 0; k < kPrepRows; ++k) {
    row[k] = (blk * kPrepRows + k) * RPB + threadIdx.x / LPR;
    const int64_t sr = row[k] >= side.rows_pad ? -1 : (side.map ? (int64_t)side.map[row[k]] : row[k]);
    real[k] = sr >= 0 && (side.map != nullptr || sr < side.n);
    const float* src = side.src + (real[k] ? sr : 0) * (int64_t)d;
    if (VEC && j0 + 8 <= d) {
      const f32x4 lo = real[k] ? *reinterpret_cast<const f32x4*>(src + j0) : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      const f32x4 hi = real[k] ? *reinterpret_cast<const f32x4*>(src + j0 + 4) : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[k][e] = lo[e];
        v[k][4 + e] = hi[e];
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[k][e] = real[k] && j0 + e < d ? src[j0 + e] : 0.0f;
    }
  }
  double mx = 0.0;
#pragma unroll
  for (int k = 0; k < kPrepRows; ++k) {
    double sq = 0.0;
    float w[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      sq += (double)v[k][e] * (double)v[k][e];
      w[e] = (float)((double)v[k][e] * side.scale);
    }
    if (act && row[k] < side.rows_pad) {
      const int64_t o = row[k] * dp + j0;
      if constexpr (FORM == STAG_FORM_FP32) {
        f32x4* dst = reinterpret_cast<f32x4*>(static_cast<float*>(side.part[0]) + o);
        dst[0] = f32x4{w[0], w[1], w[2], w[3]};
        dst[1] = f32x4{w[4], w[5], w[6], w[7]};
      } else {
        constexpr int NP = FORM == STAG_FORM_BF16_SPLIT3 ? 3 : 2;
        u16x8 p[3];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          unsigned short h[3] = {0, 0, 0};
          split_value<FORM>(w[e], h);
#pragma unroll
          for (int i = 0; i < NP; ++i) p[i][e] = h[i];
        }
#pragma unroll
        for (int i = 0; i < NP; ++i)
          *reinterpret_cast<u16x8*>(static_cast<unsigned short*>(side.part[i]) + o) = p[i];
      }
    }
#pragma unroll
    for (int o = LPR / 2; o > 0; o >>= 1) sq += __shfl_xor(sq, o);
    if (real[k]) mx = fmax(mx, sq);
    if (l == 0 && row[k] < side.rows_pad) {
      side.off[row[k]] = real[k] ? (float)(side.neg_a_log2e * sq) : (side.is_query ? 0.0f : kPadOffset);
      if (real[k] && side.nrm) side.nrm[row[k]] = sq;
    }
  }
  if (side.max_nrm_bits) block_max_norm(mx, side.max_nrm_bits);
}

// Wide rows (dp > 256): the same preparation into the fragment layout of
// kde_tile_wide.h.  One workgroup per 32-row tile; thread t handles row t % 32
// of the tile and every 8th 16-byte piece of its row, so that a wave writes 1
// KB of consecutive bytes (a whole fragment) and reads 64 consecutive bytes of
// each of 32 rows.  Bound by the rows' traffic (X read once, the operands
// written once): 70,000 rows of 784 in the split form took 315 us with a wave
// per row and one element per lane and load.
template <int FORM, bool VEC>
__global__ __launch_bounds__(256) void prep_wide(PrepSide x, PrepSide q, int d, int dp, ZeroRange zero) {
  clear_range(zero);
  const bool second = (int64_t)blockIdx.x >= x.blocks;
  const PrepSide& side = second ? q : x;
  constexpr int E = FORM == STAG_FORM_FP32 ? 4 : 8;  // row elements per 16-byte piece
  __shared__ double psum[8][32];
  const int tid = threadIdx.x, r = tid & 31;
  const int64_t tile = second ? (int64_t)blockIdx.x - x.blocks : (int64_t)blockIdx.x;
  const int64_t row = tile * kTileRows + r;
  const bool real = row < side.n;
  const float* srow = side.src + (real ? row : 0) * (int64_t)d;
  char* part0 = static_cast<char*>(side.part[0]);
  char* part1 = static_cast<char*>(side.part[1]);
  const double scale = side.scale;
  const int pieces = dp / E, H = dp / 2;
  const int64_t base = tile * kTileRows * dp / E;  // the tile's first piece
  double sq = 0.0;
  for (int pi = tid >> 5; pi < pieces; pi += 8) {
    // piece pi = 2 s + h of its row
    const int k0 = FORM == STAG_FORM_FP32 ? (pi & 1) * H + 4 * (pi >> 1) : 8 * pi;
    float v[E];
    if (VEC && real && k0 + E <= d) {
#pragma unroll
      for (int e = 0; e < E; e += 4) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(srow + k0 + e);
        v[e] = x.x; v[e + 1] = x.y; v[e + 2] = x.z; v[e + 3] = x.w;
      }
    } else {
#pragma unroll
      for (int e = 0; e < E; ++e) v[e] = real && k0 + e < d ? srow[k0 + e] : 0.0f;
    }
    const int64_t o = (base + (int64_t)pi * 32 + r) * 16;
    if constexpr (FORM == STAG_FORM_FP32) {
      f32x4 w;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        sq += (double)v[e] * (double)v[e];
        w[e] = (float)((double)v[e] * scale);
      }
      *reinterpret_cast<f32x4*>(part0 + o) = w;
    } else {
      u16x8 hi, lo;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        sq += (double)v[e] * (double)v[e];
        unsigned short p[3];
        split_value<FORM>((float)((double)v[e] * scale), p);
        hi[e] = p[0];
        lo[e] = p[1];
      }
      *reinterpret_cast<u16x8*>(part0 + o) = hi;
      *reinterpret_cast<u16x8*>(part1 + o) = lo;
    }
  }
  psum[tid >> 5][r] = sq;
  __syncthreads();
  if (tid < 32) {
    double s = psum[0][r];
#pragma unroll
    for (int w = 1; w < 8; ++w) s += psum[w][r];
    side.off[row] = real ? (float)(side.neg_a_log2e * s) : (side.is_query ? 0.0f : kPadOffset);
    if (real && side.nrm) side.nrm[row] = s;
    double mx = real ? s : 0.0;
    for (int o = 16; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o));
    if (tid == 0 && side.max_nrm_bits)
      atomicMax(side.max_nrm_bits, (unsigned long long)__double_as_longlong(mx));
  }
}

// S(q) = sum of chunk partials in chunk order; optional 1/n; a-priori bound.
// With flag: a sum below kRescueBelow sets flag[q] and its 128-query tile's
// flag (both zeroed beforehand).
__global__ void reduce_partials(const double* __restrict__ partial, int P, int64_t m_pad, int64_t m, double scale,
                                const double* __restrict__ qnrm, const unsigned long long* __restrict__ max_xnrm_bits,
                                BoundModel bm, const int* __restrict__ near_over, double* __restrict__ S_out,
                                double* __restrict__ bound_out, int* __restrict__ flag, int* __restrict__ qtile_flag) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= m) return;
  const double s = chunk_sum(partial + q, P, m_pad);
  if (flag && s < kRescueBelow) {
    flag[q] = 1;
    qtile_flag[q / kBQ] = 1;
  }
  S_out[q] = s * scale;
  if (bound_out) {
    const double xm = __longlong_as_double((long long)*max_xnrm_bits);
    if (near_over && near_over[q]) bm.near_y2 = 0.0;  // near pairs left in the tile sums
    bound_out[q] = relative_bound(bm, qnrm[q], xm);
  }
}

// Centred fp32 data: S(q) = sum of chunk partials in chunk order; the
// bound is (sum of the chunks' bound numerators) / S, plus its square and
// c_tail (the numerators come from computed tile sums: first-order slack),
// and infinite for S = 0.  Flags as in reduce_partials.
__global__ void reduce_centred(const double* __restrict__ partial, const double* __restrict__ bpart, int P,
                               int64_t m_pad, int64_t m, double scale, double c_tail, double* __restrict__ S_out,
                               double* __restrict__ bound_out, int* __restrict__ flag, int* __restrict__ qtile_flag) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= m) return;
  const double s = chunk_sum(partial + q, P, m_pad);
  const double b = chunk_sum(bpart + q, P, m_pad);
  if (flag && s < kRescueBelow) {
    flag[q] = 1;
    qtile_flag[q / kBQ] = 1;
  }
  S_out[q] = s * scale;
  if (bound_out) {
    const double r = b / s;
    bound_out[q] = s > 0.0 ? r + r * r + c_tail : HUGE_VAL;
  }
}

// Adaptive form, per (sorted) query: the first pass's sum S1 over its P
// chunk partials, and the threshold T below which its chunks keep their
// first-pass values.  With budget = share * S1, T is the largest of the
// candidates 4^-j budget (j = 0 .. kBudgetSteps - 1) for which the chunk
// bound numerators below it add up to at most 0.999 budget (each candidate's
// sum kept in a register, in units of the budget); the chunks left to the
// first pass then carry at most share * S1 of bound numerator between them,
// and the recomputed ones are those with the largest numerators.  T = 0 where
// the budget is 0 (S1 = 0) or outside the range its reciprocal needs, on the
// rows past m and outside qmask (where S1 is not needed and not written).
constexpr int kBudgetSteps = 16;
__global__ void adaptive_budget(const double* __restrict__ partial, const double* __restrict__ bpart, int P,
                                int64_t m_pad, int64_t m, double share, const int* __restrict__ qmask,
                                double* __restrict__ S1, double* __restrict__ T) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= m_pad) return;
  if (q >= m || (qmask && qmask[q / kBQ] == 0)) {
    T[q] = 0.0;
    return;
  }
  const double s = chunk_sum(partial + q, P, m_pad);
  S1[q] = s;
  const double budget = share * s;
  const double inv = 1.0 / budget;
  if (!(budget > 0.0) || !(inv < HUGE_VAL)) {
    T[q] = 0.0;
    return;
  }
  float acc[kBudgetSteps];
#pragma unroll
  for (int j = 0; j < kBudgetSteps; ++j) acc[j] = 0.0f;
  auto count = [&](double v) {
    if (!(v < budget)) return;  // recomputed whatever the others hold (NaN as well)
    const float r = (float)(v * inv);
    // every chunk with v < 4^-j budget is counted under candidate j (the
    // margin covers the roundings of r)
    float c = 1.000001f;
#pragma unroll
    for (int j = 0; j < kBudgetSteps; ++j) {
      acc[j] += r <= c ? r : 0.0f;
      c *= 0.25f;
    }
  };
  int p = 0;
  for (; p + 8 <= P; p += 8) {  // loads eight at a time, counted in order
    double v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = bpart[(int64_t)(p + i) * m_pad + q];
#pragma unroll
    for (int i = 0; i < 8; ++i) count(v[i]);
  }
  for (; p < P; ++p) count(bpart[(int64_t)p * m_pad + q]);
  double t = 0.0, c = 1.0;
#pragma unroll
  for (int j = 0; j < kBudgetSteps; ++j) {
    if (t == 0.0 && acc[j] <= 0.999f) t = c;
    c *= 0.25;
  }
  T[q] = t * budget;
}

// Adaptive form: a (chunk, 256-query tile) pair is recomputed in the split
// form when some query's bound numerator v of that chunk from the single-
// product pass is positive and not below the query's threshold T (cflag
// starts at zero; every writer stores 1).  Grid: (query blocks, chunks).
__global__ void adaptive_flags(const double* __restrict__ bpart, const double* __restrict__ T, int64_t m_pad,
                               int64_t m, int n_qt256, const int* __restrict__ qmask, uint8_t* __restrict__ cflag) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t c = blockIdx.y;
  if (q >= m || (qmask && qmask[q / kBQ] == 0)) return;
  const double v = bpart[c * m_pad + q];
  if (v > 0.0 && !(v < T[q])) cflag[c * n_qt256 + q / 256] = 1;
}

// Adaptive form, the estimate: every stride-th 128-query tile is sampled.
__global__ void mark_sample(int* __restrict__ qsample, int n_qt128, int stride) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n_qt128) qsample[t] = t % stride == 0 ? 1 : 0;
}

// counts[0] += selected and counts[1] += all (chunk, 256-query tile) pairs
// of the tiles that hold a sampled 128-query tile.  Grid: (tiles, chunks).
__global__ void count_selected(const uint8_t* __restrict__ cflag, int n_qt256, const int* __restrict__ qsample,
                               int n_qt128, unsigned int* __restrict__ counts) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t c = blockIdx.y;
  if (t >= n_qt256) return;
  const bool sampled = qsample[2 * t] != 0 || (2 * t + 1 < n_qt128 && qsample[2 * t + 1] != 0);
  if (!sampled) return;
  atomicAdd(counts, cflag[c * n_qt256 + t] ? 1u : 0u);
  atomicAdd(counts + 1, 1u);
}

__global__ void fill_ones(uint8_t* __restrict__ p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 1;
}

// Adaptive form: S(q) = sum of the chunk partials in chunk order (first
// pass, or the split form where the chunk was recomputed); the bound's
// numerator adds the first pass's bound numerator of a kept chunk and
// partial x the split form's a-priori relative bound of a recomputed one;
// bound = r + r^2 + c_tail with r = numerator / S.  Results in sorted order;
// rescue flags as in reduce_partials.
__global__ void reduce_adaptive(const double* __restrict__ partial, const double* __restrict__ bpart,
                                const uint8_t* __restrict__ cflag, int P, int64_t m_pad, int64_t m, int n_qt256,
                                double scale, const double* __restrict__ qnrm,
                                const unsigned long long* __restrict__ max_xnrm_bits, BoundModel bm, double c_tail,
                                double* __restrict__ S_s, double* __restrict__ B_s, int* __restrict__ flag,
                                int* __restrict__ qtile_flag) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= m) return;
  const double xm = __longlong_as_double((long long)*max_xnrm_bits);
  const double rs = relative_bound(bm, qnrm[q], xm);
  double s = 0.0, b = 0.0;
  auto add = [&](double v, uint8_t f, double w) {
    s += v;
    b += f ? v * rs : w;
  };
  const int64_t t = q / 256;
  int p = 0;
  for (; p + 8 <= P; p += 8) {  // loads eight at a time, added in order
    double v[8], w[8];
    uint8_t f[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      v[i] = partial[(int64_t)(p + i) * m_pad + q];
      w[i] = bpart[(int64_t)(p + i) * m_pad + q];
      f[i] = cflag[(int64_t)(p + i) * n_qt256 + t];
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) add(v[i], f[i], w[i]);
  }
  for (; p < P; ++p)
    add(partial[(int64_t)p * m_pad + q], cflag[(int64_t)p * n_qt256 + t], bpart[(int64_t)p * m_pad + q]);
  if (s < kRescueBelow) {
    flag[q] = 1;
    qtile_flag[q / kBQ] = 1;
  }
  S_s[q] = s * scale;
  const double r = b / s;
  B_s[q] = s > 0.0 ? r + r * r + c_tail : HUGE_VAL;
}

// Sorted results back to the queries' rows.
__global__ void scatter_results(const double* __restrict__ S_s, const double* __restrict__ B_s,
                                const int* __restrict__ perm, int64_t m_pad, double* __restrict__ S_out,
                                double* __restrict__ bound_out) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= m_pad) return;
  const int i = perm[q];
  if (i < 0) return;
  S_out[i] = S_s[q];
  if (bound_out) bound_out[i] = B_s[q];
}

// One launch over both sides (the second may be empty: rows_pad 0).
template <int FORM>
stag_status launch_prep(PrepSide x, PrepSide q, int d, int dp, const ZeroRange& zero, hipStream_t st) {
  ScopedTimer tm("kde_prep", st);
  // 16-byte row reads where every row starts at one
  const bool vec = d % 4 == 0 && (((uintptr_t)x.src | (uintptr_t)q.src) & 15u) == 0;
  auto launch = [&](auto kern, int64_t rows_per_block) {
    x.blocks = ceil_div(x.rows_pad, rows_per_block);
    q.blocks = ceil_div(q.rows_pad, rows_per_block);
    hipLaunchKernelGGL(kern, dim3((unsigned)(x.blocks + q.blocks)), dim3(256), 0, st, x, q, d, dp, zero);
    return check_launch("prep_rows");
  };
  if (dp > 256) {  // the fragment layout of the wide tile
    if constexpr (FORM == STAG_FORM_BF16_SPLIT3) {
      return fail(STAG_E_UNSUPPORTED, "d > 256 needs the fp32, fp16 split or bf16 split form");
    } else {
      if (x.map || q.map) return fail(STAG_E_UNSUPPORTED, "wide rows: no row map");
      return vec ? launch(prep_wide<FORM, true>, kTileRows) : launch(prep_wide<FORM, false>, kTileRows);
    }
  }
  auto by_lanes = [&](auto LC) {
    constexpr int lpr = decltype(LC)::value;
    return vec ? launch(prep_rows<FORM, lpr, true>, kPrepRows * 256 / lpr)
               : launch(prep_rows<FORM, lpr, false>, kPrepRows * 256 / lpr);
  };
  if (dp <= 16) return by_lanes(std::integral_constant<int, 2>());
  if (dp <= 32) return by_lanes(std::integral_constant<int, 4>());
  if (dp <= 64) return by_lanes(std::integral_constant<int, 8>());
  if (dp <= 128) return by_lanes(std::integral_constant<int, 16>());
  return by_lanes(std::integral_constant<int, 32>());
}

stag_status prep_sides(int form, const PrepSide& x, const PrepSide& q, int d, int dp, const ZeroRange& zero,
                       hipStream_t st) {
  switch (form) {
    case STAG_FORM_FP32: return launch_prep<STAG_FORM_FP32>(x, q, d, dp, zero, st);
    case STAG_FORM_BF16_SPLIT: return launch_prep<STAG_FORM_BF16_SPLIT>(x, q, d, dp, zero, st);
    case STAG_FORM_FP16_SPLIT: return launch_prep<STAG_FORM_FP16_SPLIT>(x, q, d, dp, zero, st);
    default: return launch_prep<STAG_FORM_BF16_SPLIT3>(x, q, d, dp, zero, st);
  }
}

// The side of an operand set: the scaled split of src (data or queries), or,
// plain, an unscaled copy with offset 0 (queries of centred data, whose tile
// adds -a log2(e) ||q - c||^2 itself).
PrepSide side_of(const float* src, double a, bool is_query, bool plain, const Operands& o, const int* map = nullptr) {
  PrepSide p = {src, o.rows, o.rows_pad, plain || !is_query ? 1.0 : 2.0 * a * kLog2e, plain ? 0.0 : -a * kLog2e,
                is_query ? 1 : 0, {o.part[0], o.part[1], o.part[2]}, o.off, o.nrm, o.max_nrm_bits, map, 0};
  return p;
}

constexpr int kScanRowsPerWave = 16;
constexpr int kScanRowsPerBlock = 4 * kScanRowsPerWave;

// Statistics of an input for the form choice and the finiteness check: the
// largest squared row norm (fp64 bits), the largest |element| (fp32 bits) and
// whether any element is not finite.  One wave per row, 16 rows per wave.
__global__ __launch_bounds__(256) void scan_rows(const float* __restrict__ src, int64_t rows, int d,
                                                 unsigned long long* __restrict__ max_nrm_bits,
                                                 unsigned int* __restrict__ max_abs_bits, int* __restrict__ bad) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double mx = 0.0;
  float amax = 0.0f;
  int nonfinite = 0;
  for (int rr = 0; rr < kScanRowsPerWave; ++rr) {
    const int64_t row = (int64_t)blockIdx.x * kScanRowsPerBlock + wave * kScanRowsPerWave + rr;
    if (row >= rows) break;
    double sq = 0.0;
    for (int j = lane; j < d; j += 64) {
      const float v = src[row * d + j];
      if (!(fabsf(v) <= 3.402823466e38f)) nonfinite = 1;
      else amax = fmaxf(amax, fabsf(v));
      sq += (double)v * (double)v;
    }
    for (int o = 32; o > 0; o >>= 1) sq += __shfl_xor(sq, o);
    if (sq == sq) mx = fmax(mx, sq);
  }
  for (int o = 32; o > 0; o >>= 1) {
    amax = fmaxf(amax, __shfl_xor(amax, o));
    nonfinite |= __shfl_xor(nonfinite, o);
  }
  if (lane == 0) {
    if (mx > 0.0) atomicMax(max_nrm_bits, (unsigned long long)__double_as_longlong(mx));
    if (amax > 0.0f) atomicMax(max_abs_bits, __float_as_uint(amax));
    if (nonfinite) atomicOr(bad, 1);
  }
}

}  // namespace

int exact_padded_dim(int d) {
  static const int dims[] = {16, 32, 64, 96, 128, 160, 192, 224, 256};
  for (int v : dims)
    if (d <= v) return v;
  if (d <= kWideMaxDim) return (int)round_up(d, 64);
  return 0;
}

size_t form_element_bytes(int form) { return form == STAG_FORM_FP32 ? 4 : 2; }
int form_parts(int form) {
  return form == STAG_FORM_FP32 ? 1 : (form == STAG_FORM_BF16_SPLIT3 ? 3 : 2);
}

stag_status alloc_operands(int form, int64_t rows, int d, bool is_query, Workspace& ws, Operands* out) {
  const int dp = exact_padded_dim(d);
  const int64_t rows_pad = round_up(rows, is_query ? kBQ : kTileRows);
  out->form = form;
  out->rows = rows;
  out->rows_pad = rows_pad;
  out->d = d;
  out->dp = dp;
  for (int p = 0; p < 3; ++p) out->part[p] = nullptr;
  for (int p = 0; p < form_parts(form); ++p)
    STAG_TRY(ws.alloc_bytes(&out->part[p], (size_t)rows_pad * dp * form_element_bytes(form)));
  STAG_TRY(ws.alloc(&out->off, (size_t)rows_pad));
  STAG_TRY(ws.alloc(&out->nrm, (size_t)rows));
  out->max_nrm_bits = nullptr;
  if (!is_query) STAG_TRY(ws.alloc(&out->max_nrm_bits, 1));
  return STAG_OK;
}

stag_status prep_operands(const float* src, double a, bool is_query, const Operands& o, hipStream_t st) {
  if (o.max_nrm_bits) STAG_TRY(zero_async(o.max_nrm_bits, sizeof(unsigned long long), st));
  return prep_sides(o.form, side_of(src, a, is_query, false, o), PrepSide{}, o.d, o.dp, ZeroRange(), st);
}

stag_status prep_operand_pair(const float* X, const float* Q, double a, const Operands& xo, const Operands& qo,
                              bool bound, void* zero, size_t zero_words, hipStream_t st) {
  PrepSide x = side_of(X, a, false, false, xo);
  if (bound) STAG_TRY(zero_async(xo.max_nrm_bits, sizeof(unsigned long long), st));
  else x.max_nrm_bits = nullptr;
  return prep_sides(xo.form, x, side_of(Q, a, true, false, qo), xo.d, xo.dp,
                    {static_cast<uint32_t*>(zero), (int64_t)zero_words}, st);
}

stag_status prepare_operands(int form, const float* src, int64_t rows, int d, double a, bool is_query,
                             Workspace& ws, Operands* out, hipStream_t st) {
  STAG_TRY(alloc_operands(form, rows, d, is_query, ws, out));
  return prep_operands(src, a, is_query, *out, st);
}

int64_t exact_chunks(int64_t n_pad) { return ceil_div(n_pad, kChunkRows); }

stag_status prep_query_into(int form, const float* src, int64_t rows, int d, double a, const Operands& batch,
                            int64_t row0, hipStream_t st, bool centred) {
  Operands o = batch;
  o.rows = rows;
  o.rows_pad = round_up(rows, kBQ);
  for (int p = 0; p < form_parts(form); ++p)
    o.part[p] = static_cast<char*>(batch.part[p]) + (size_t)row0 * batch.dp * form_element_bytes(form);
  o.off = batch.off + row0;
  o.nrm = batch.nrm ? batch.nrm + row0 : nullptr;
  o.max_nrm_bits = nullptr;
  // queries of centred data are kept unscaled with offset 0
  return prep_sides(form, side_of(src, a, true, centred, o), PrepSide{}, d, batch.dp, ZeroRange(), st);
}

stag_status row_stats_async(const float* A, int64_t rows, int d, unsigned long long* nrm_bits, unsigned int* abs_bits,
                            int* bad, hipStream_t st) {
  STAG_TRY(zero_async(nrm_bits, sizeof(unsigned long long), st));
  STAG_TRY(zero_async(abs_bits, sizeof(unsigned int), st));
  STAG_TRY(zero_async(bad, sizeof(int), st));
  hipLaunchKernelGGL(scan_rows, dim3((unsigned)ceil_div(rows, kScanRowsPerBlock)), dim3(256), 0, st, A, rows, d,
                     nrm_bits, abs_bits, bad);
  return check_launch("scan_rows");
}

int choose_resident_form(uint32_t resident, int d, double a, double eps, double max_nrm_q, double max_nrm_x,
                         float max_abs_q, float max_abs_x) {
  const double qscale = 2.0 * a * kLog2e;
  const bool fp16_ok = (double)max_abs_x < 65504.0 && (double)max_abs_q * qscale < 65504.0;
  const int order[3] = {STAG_FORM_FP16_SPLIT, STAG_FORM_BF16_SPLIT, STAG_FORM_BF16_SPLIT3};
  int best = -1;
  double best_b = HUGE_VAL;
  for (int f : order) {
    if (!(resident & (1u << f)) || d > 256 || (f == STAG_FORM_FP16_SPLIT && !fp16_ok)) continue;
    const double b = relative_bound(make_bound_model(f, d, a, STAG_KERNEL_GAUSSIAN), max_nrm_q, max_nrm_x);
    if (b <= eps) return f;
    if (b < best_b) {
      best_b = b;
      best = f;
    }
  }
  if (resident & (1u << STAG_FORM_FP32)) return STAG_FORM_FP32;
  return best;
}

int64_t query_tile_rows() { return kBQ; }

namespace {

// Partials of the chunks of a wide launch from the sub-chunks' sums: those of
// each accumulator in order, then the four of a query pairwise, as one
// workgroup per chunk adds them.
__global__ __launch_bounds__(256) void combine_subs(const double* __restrict__ sub, int64_t m_pad,
                                                    double* __restrict__ partial) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t c = blockIdx.y;
  if (q >= m_pad) return;
  double t[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int k = 0; k < kSubs; ++k)
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i] += sub[sub_index(c, k, 4, i, m_pad, q)];
  partial[c * m_pad + q] = (t[0] + t[1]) + (t[2] + t[3]);
}

// Partials (and bound numerators) of the chunks from the tile sums of a part
// launch, added in the order of the tiles' own loops: each lane half in tile
// order, then the halves.  KIND 0: sums alone; 1: centred fp32 form (bsum:
// each tile's bound term); 2: centred fp16 form (fp64 sum per group, scaled
// and weighted with its bound factor when the group ends).  A workgroup takes
// 32 queries of a chunk and brings 64 tiles' sums at a time to LDS, all loads
// in flight; 64 threads (query, lane half) then add them.
constexpr int kCombineTiles = 64;
template <int KIND>
__global__ __launch_bounds__(256) void combine_parts(const float* __restrict__ tsum, const float* __restrict__ bsum,
                                                     const int* __restrict__ tgroup,
                                                     const int64_t* __restrict__ n_pad_dev, int64_t n_pad_host,
                                                     int64_t m_pad, double* __restrict__ partial,
                                                     double* __restrict__ bpart) {
  __shared__ float ts[kCombineTiles][64], bs[KIND ? kCombineTiles : 1][64];
  __shared__ int tg[kCombineTiles + 1];
  __shared__ double osum[32], obound[32];
  const int tid = threadIdx.x, c = tid & 31, h = (tid >> 5) & 1;
  const int64_t q0 = (int64_t)blockIdx.x * 32;  // m_pad is a multiple of 128
  const int64_t chunk = blockIdx.y;
  const int64_t n_pad = n_pad_dev ? *n_pad_dev : n_pad_host;
  const int nt = (int)max((int64_t)0, min((int64_t)kChunkTiles, n_pad / kTileRows - chunk * kChunkTiles));
  double acc = 0.0, bacc = 0.0, seg = 0.0;
  for (int t0 = 0; t0 < nt; t0 += kCombineTiles) {
    const int k = min(kCombineTiles, nt - t0);
    float v[kCombineTiles / 4], w[kCombineTiles / 4];
#pragma unroll
    for (int i = 0; i < kCombineTiles / 4; ++i) {
      const int t = t0 + min(4 * i + (tid >> 6), k - 1);
      v[i] = tsum[tsum_index(chunk, t, h, m_pad, q0 + c)];
      if constexpr (KIND != 0) w[i] = bsum[tsum_index(chunk, t, h, m_pad, q0 + c)];
    }
    __syncthreads();  // the previous round's sums are taken
#pragma unroll
    for (int i = 0; i < kCombineTiles / 4; ++i) {
      ts[4 * i + (tid >> 6)][tid & 63] = v[i];
      if constexpr (KIND != 0) bs[4 * i + (tid >> 6)][tid & 63] = w[i];
    }
    if constexpr (KIND == 2) {
      // the groups, one past the round's tiles (-1 past the chunk's last)
      if (tid <= kCombineTiles) tg[tid] = t0 + tid < nt ? tgroup[chunk * kChunkTiles + t0 + tid] : -1;
    }
    __syncthreads();
    if (tid < 64) {
      for (int t = 0; t < k; ++t) {
        if constexpr (KIND == 2) {
          seg += (double)ts[t][tid];
          if (tg[t + 1] != tg[t]) {  // the group's last tile in the chunk
            const double s = (double)bs[t][c];
            acc = fma(seg, s, acc);
            bacc = fma(seg, s * (double)bs[t][32 + c], bacc);
            seg = 0.0;
          }
        } else {
          acc += (double)ts[t][tid];
          if constexpr (KIND == 1) bacc += (double)bs[t][tid];
        }
      }
    }
  }
  if (tid >= 32 && tid < 64) {
    osum[c] = acc;
    obound[c] = bacc;
  }
  __syncthreads();
  if (tid < 32) {
    partial[chunk * m_pad + q0 + c] = acc + osum[c];
    if (KIND != 0) bpart[chunk * m_pad + q0 + c] = bacc + obound[c];
  }
}

}  // namespace

stag_status alloc_parts(const Operands& xo, const Operands& qo, int kernel, Workspace& ws, TileExtra* ex) {
  ex->nsub = 1;
  if (!ws.pooled() || kernel == STAG_KERNEL_EXPONENTIAL) return STAG_OK;
  const int64_t P = exact_chunks(xo.rows_pad), pairs = P * (qo.rows_pad / kBQ);
  const bool wide = xo.dp > 256;
  if (pairs >= (wide ? kFewPairsWide : kFewPairs)) return STAG_OK;
  if (P == 1) {
    // one short chunk: what an eighth of a whole one holds is not shared
    int64_t unshared = kSubTiles;
    if (wide) unshared = xo.form == STAG_FORM_FP32 ? 3 * kSubTiles : 3 * kSubTiles / 2;
    if (kernel == STAG_KERNEL_GAUSSIAN && !xo.centred && xo.dp <= 32) unshared = 2 * kSubTiles;
    if (xo.form == STAG_FORM_FP16_CENTRED && xo.dp > 128) unshared = 4 * kSubTiles - 1;
    if (xo.rows_pad / kTileRows <= unshared) return STAG_OK;
  }
  int nsub = wide ? kSubs : 2;
  while (nsub < kSubs && pairs * nsub < kSplitGrid) nsub *= 2;
  if (wide) {
    STAG_TRY(ws.alloc(&ex->sub, (size_t)P * kSubs * 4 * qo.rows_pad));
  } else {
    const size_t sums = (size_t)P * kChunkTiles * 2 * qo.rows_pad;
    STAG_TRY(ws.alloc(&ex->tsum, sums));
    if (xo.centred) STAG_TRY(ws.alloc(&ex->bsum, sums));
  }
  ex->nsub = nsub;
  return STAG_OK;
}

static stag_status launch_tiles_by_mode(const Operands& xo, const Operands& qo, double* partial, const TileExtra& ex,
                                        hipStream_t st);

stag_status launch_exact_tiles(const Operands& xo, const Operands& qo, double* partial, const TileExtra& ex,
                               hipStream_t st) {
  if (ex.nsub > 1 && (ex.qtile_active || ex.max_pass || ex.cflag || ex.kernel == STAG_KERNEL_EXPONENTIAL)) {
    // launches over selected tiles, and those of the rescue: whole chunks
    TileExtra e = ex;
    e.nsub = 1;
    return launch_tiles_by_mode(xo, qo, partial, e, st);
  }
  STAG_TRY(launch_tiles_by_mode(xo, qo, partial, ex, st));
  if (ex.nsub == 1) return STAG_OK;
  const int64_t m_pad = qo.rows_pad;
  const unsigned P = (unsigned)exact_chunks(xo.rows_pad);
  if (xo.dp > 256) {
    hipLaunchKernelGGL(combine_subs, dim3((unsigned)ceil_div(m_pad, 256), P), dim3(256), 0, st, ex.sub, m_pad, partial);
    return check_launch("combine_subs");
  }
  const dim3 grid((unsigned)(m_pad / 32), P);
  auto combine = [&](auto kern) {
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, st, ex.tsum, ex.bsum, xo.tgroup, xo.n_pad_dev, xo.rows_pad, m_pad,
                       partial, ex.bpart);
  };
  if (!xo.centred) combine(combine_parts<0>);
  else if (xo.form == STAG_FORM_FP32) combine(combine_parts<1>);
  else combine(combine_parts<2>);
  return check_launch("combine_parts");
}

static stag_status launch_tiles_by_mode(const Operands& xo, const Operands& qo, double* partial, const TileExtra& ex,
                               hipStream_t st) {
  if (ex.kernel != STAG_KERNEL_GAUSSIAN && (ex.self || ex.tp))
    return fail(STAG_E_UNSUPPORTED, "tile extras need the Gaussian kernel");
  switch (tiles::tile_mode(ex)) {
    case tiles::kModeMax: return launch_tiles_max(xo, qo, partial, ex, st);
    case tiles::kModeGaussRescue: return launch_tiles_gauss_rescue(xo, qo, partial, ex, st);
    case tiles::kModeGaussExtraRescue: return launch_tiles_gauss_extra_rescue(xo, qo, partial, ex, st);
    case tiles::kModeExpShift: return launch_tiles_exp_shift(xo, qo, partial, ex, st);
    case tiles::kModeLogShift: return launch_tiles_log_shift(xo, qo, partial, ex, st);
    case tiles::kModeGauss: return launch_tiles_gauss(xo, qo, partial, ex, st);
    case tiles::kModeGaussExtra: return launch_tiles_gauss_extra(xo, qo, partial, ex, st);
    case tiles::kModeGaussPart: return launch_tiles_gauss_part(xo, qo, partial, ex, st);
    case tiles::kModeGaussExtraPart: return launch_tiles_gauss_extra_part(xo, qo, partial, ex, st);
    case tiles::kModeLogisticPart: return launch_tiles_logistic_part(xo, qo, partial, ex, st);
    case tiles::kModeExponential: return launch_tiles_exponential(xo, qo, partial, ex, st);
    default: return launch_tiles_logistic(xo, qo, partial, ex, st);
  }
}

stag_status launch_reduce(const double* partial, int P, const Operands& qo, const Operands& xo, double scale,
                          const BoundModel& bm, double* S_out, double* bound_out, hipStream_t st,
                          const int* near_over, int* flag, int* qtile_flag) {
  const int64_t m = qo.rows;
  ScopedTimer tm("kde_reduce", st);
  hipLaunchKernelGGL(reduce_partials, dim3((unsigned)ceil_div(m, 256)), dim3(256), 0, st, partial, P, qo.rows_pad, m,
                     scale, qo.nrm, xo.max_nrm_bits, bm, near_over, S_out, bound_out, flag, qtile_flag);
  return check_launch("reduce_partials");
}

double kernel_tile_a(int kernel, double a) { return kernel == STAG_KERNEL_GAUSSIAN ? a : a * a * kLog2e; }

BoundModel make_bound_model(int form, int d, double a_tile, int kernel) {
  BoundModel bm;
  const double u = 0x1.0p-24;
  bm.la = a_tile * kLog2e;
  bm.kern = kernel;
  // fp32 accumulation of the d cross products and the six offset parts,
  // probabilistic model with lambda = 6 (Higham & Mary 2019)
  bm.c_acc = 6.0 * std::sqrt((double)d + 6.0) * u;
  double c_split;
  switch (form) {
    case STAG_FORM_FP32: c_split = u; break;                          // rounding of s*q to fp32
    case STAG_FORM_FP16_SPLIT: c_split = 3.0 * 0x1.0p-22 + u; break;  // dropped lo*lo, part rounding
    case STAG_FORM_BF16_SPLIT: c_split = 3.0 * 0x1.0p-16 + u; break;
    default: c_split = 4.0 * 0x1.0p-24 + u; break;
  }
  bm.c_split = c_split;
  bm.c_off = 3.0 * u;                   // alpha, beta rounded to fp32
  bm.c_tail = 0x1.0p-22 + 16.0 * u;     // exp2 and the 16-term fp32 tile sums
  // centred fp32 tile (per term, times M_T): the MFMA accumulation and the
  // fp32 sum of the d squared differences (c_acc each), the roundings of
  // q - c, its scaling and x - c in the cross term (3u), beta, the final
  // exponent add and the offset (3u), with 2u to spare
  bm.c_cent = 2.0 * bm.c_acc + 8.0 * u;
  if (kernel == STAG_KERNEL_EXPONENTIAL) bm.near_y2 = kNearY2;
  return bm;
}

}  // namespace stag

namespace stag {

namespace {

// Underflow rescue of the Gaussian exact sum.  For a flagged query (sum
// below kRescueBelow), m_q = the largest exponent E over the data (max pass
// of the tiles); its offset becomes fl32(-a log2(e) ||q||^2 - m_q) (one
// rounding from binary64), so that its largest term is about 2^0, and the
// tiles run again on the flagged query tiles; S = (sum) 2^{m_q}.
__global__ void rescue_shift(const double* __restrict__ pmax, int P, int64_t m_pad, int64_t m,
                             const int* __restrict__ flag, const double* __restrict__ qnrm, double neg_a_l2e,
                             const float* __restrict__ off, float* __restrict__ off2, double* __restrict__ shift) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= m_pad) return;
  double mq = 0.0;
  float o = off[q];
  if (q < m && flag[q]) {
    mq = -HUGE_VAL;
    for (int p = 0; p < P; ++p) mq = fmax(mq, pmax[(int64_t)p * m_pad + q]);
    o = (float)(neg_a_l2e * qnrm[q] - mq);
  }
  off2[q] = o;
  shift[q] = mq;
}

__global__ void rescue_reduce(const double* __restrict__ partial, int P, int64_t m_pad, int64_t m,
                              const int* __restrict__ flag, const double* __restrict__ shift, double scale,
                              const double* __restrict__ qnrm, const unsigned long long* __restrict__ max_xnrm_bits,
                              BoundModel bm, double* __restrict__ S_out, double* __restrict__ bound_out) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= m || !flag[q]) return;
  const double s = chunk_sum(partial + q, P, m_pad);
  S_out[q] = s * exp2(shift[q]) * scale;
  if (bound_out) {
    const double xm = __longlong_as_double((long long)*max_xnrm_bits);
    bound_out[q] = relative_bound(bm, qnrm[q], xm, fabs(shift[q]));
  }
}

// Centred data: a flagged query's offset becomes fl32(-m_q) (the tile adds it
// to alpha'), others keep theirs (0).
__global__ void rescue_shift_centred(const double* __restrict__ pmax, int P, int64_t m_pad, int64_t m,
                                     const int* __restrict__ flag, const float* __restrict__ off,
                                     float* __restrict__ off2, double* __restrict__ shift) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= m_pad) return;
  double mq = 0.0;
  float o = off[q];
  if (q < m && flag[q]) {
    mq = -HUGE_VAL;
    for (int p = 0; p < P; ++p) mq = fmax(mq, pmax[(int64_t)p * m_pad + q]);
    o = (float)(-mq);
  }
  off2[q] = o;
  shift[q] = mq;
}

__global__ void rescue_reduce_centred(const double* __restrict__ partial, const double* __restrict__ bpart, int P,
                                      int64_t m_pad, int64_t m, const int* __restrict__ flag,
                                      const double* __restrict__ shift, double scale, double c_tail,
                                      double* __restrict__ S_out, double* __restrict__ bound_out) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= m || !flag[q]) return;
  double s = 0.0, b = 0.0;
  for (int p = 0; p < P; ++p) {
    s += partial[(int64_t)p * m_pad + q];
    b += bpart[(int64_t)p * m_pad + q];
  }
  S_out[q] = s * exp2(shift[q]) * scale;
  if (bound_out) {
    const double r = b / s;
    bound_out[q] = s > 0.0 ? r + r * r + c_tail : HUGE_VAL;
  }
}

stag_status rescue_underflow(const Operands& xo, const Operands& qo, int P, double a_tile, double scale,
                             const BoundModel& bm, const RescueBuffers& rb, double* S_out, double* bound_out,
                             hipStream_t st) {
  const int64_t m_pad = qo.rows_pad, m = qo.rows;
  STAG_TRY(rescue_offsets_into(xo, qo, P, a_tile, 0, rb.flag, rb.qflag, rb.pmax, rb.off2, rb.shift, st));
  Operands q2 = qo;
  q2.off = rb.off2;
  TileExtra exs;
  exs.qtile_active = rb.qflag;
  STAG_TRY(launch_exact_tiles(xo, q2, rb.p2, exs, st));
  hipLaunchKernelGGL(rescue_reduce, dim3((unsigned)ceil_div(m, 256)), dim3(256), 0, st, rb.p2, P, m_pad, m, rb.flag,
                     rb.shift, scale, qo.nrm, xo.max_nrm_bits, bm, S_out, bound_out);
  return check_launch("rescue_reduce");
}

// Exponential and logistic kernels: ys = sqrt(-max E) of each flagged
// query (its smallest y), 0 otherwise.
__global__ void rescue_yshift(const double* __restrict__ pmax, int P, int64_t m_pad, int64_t m,
                              const int* __restrict__ flag, float* __restrict__ yshift) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= m_pad) return;
  float ys = 0.0f;
  if (q < m && flag[q]) {
    double mq = -HUGE_VAL;
    for (int p = 0; p < P; ++p) mq = fmax(mq, pmax[(int64_t)p * m_pad + q]);
    ys = (float)sqrt(fmax(-mq, 0.0));
  }
  yshift[q] = ys;
}

__global__ void rescue_reduce_y(const double* __restrict__ partial, int P, int64_t m_pad, int64_t m,
                                const int* __restrict__ flag, const float* __restrict__ yshift, double scale,
                                const double* __restrict__ qnrm, const unsigned long long* __restrict__ max_xnrm_bits,
                                BoundModel bm, double* __restrict__ S_out, double* __restrict__ bound_out) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= m || !flag[q]) return;
  const double s = chunk_sum(partial + q, P, m_pad);
  const double ys = (double)yshift[q];
  S_out[q] = s * exp2(-ys) * scale;
  if (bound_out) {
    const double xm = __longlong_as_double((long long)*max_xnrm_bits);
    bound_out[q] = relative_bound(bm, qnrm[q], xm, ys);
  }
}

}  // namespace

stag_status rescue_offsets_into(const Operands& xo, const Operands& qo, int P, double a_tile, int self,
                                const int* flag, const int* qtile_flag, double* pmax, float* off2, double* shift,
                                hipStream_t st) {
  const int64_t m_pad = qo.rows_pad, m = qo.rows;
  TileExtra exm;
  exm.max_pass = 1;
  exm.self = self;
  exm.qtile_active = qtile_flag;
  STAG_TRY(launch_exact_tiles(xo, qo, pmax, exm, st));
  hipLaunchKernelGGL(rescue_shift, dim3((unsigned)ceil_div(m_pad, 256)), dim3(256), 0, st, pmax, P, m_pad, m, flag,
                     qo.nrm, -a_tile * kLog2e, qo.off, off2, shift);
  return check_launch("rescue_shift");
}

stag_status rescue_offsets(const Operands& xo, const Operands& qo, int P, double a_tile, int self, const int* flag,
                           const int* qtile_flag, float* off2, double* shift, Workspace& ws, hipStream_t st) {
  double* pmax = nullptr;
  STAG_TRY(ws.alloc(&pmax, (size_t)P * qo.rows_pad));
  return rescue_offsets_into(xo, qo, P, a_tile, self, flag, qtile_flag, pmax, off2, shift, st);
}

stag_status alloc_rescue(int kernel, int P, const Operands& qo, Workspace& ws, RescueBuffers* rb) {
  const int64_t m = qo.rows, m_pad = qo.rows_pad;
  *rb = RescueBuffers();
  // the flags in one buffer, cleared in one go
  const int64_t mr = round_up(m, 64);
  rb->zero_words = (size_t)(mr + m_pad / kBQ);
  if (kernel == STAG_KERNEL_EXPONENTIAL) rb->zero_words = (size_t)(2 * mr + m_pad / kBQ);
  STAG_TRY(ws.alloc(&rb->flag, rb->zero_words));
  rb->qflag = rb->flag + mr;
  if (kernel == STAG_KERNEL_EXPONENTIAL) {
    rb->near_over = rb->flag + mr;
    rb->qflag = rb->flag + 2 * mr;
  }
  STAG_TRY(ws.alloc(&rb->pmax, (size_t)P * m_pad));
  STAG_TRY(ws.alloc(&rb->p2, (size_t)P * m_pad));
  if (kernel == STAG_KERNEL_GAUSSIAN) {
    STAG_TRY(ws.alloc(&rb->shift, (size_t)m_pad));
    STAG_TRY(ws.alloc(&rb->off2, (size_t)m_pad));
  } else {
    STAG_TRY(ws.alloc(&rb->yshift, (size_t)m_pad));
  }
  return STAG_OK;
}

// launch_reduce for the exponential and logistic kernels with the underflow
// rescue: a flagged query's terms are recomputed as 2^{ys - y}, ys its
// smallest y (from the max pass), and S = (sum) 2^{-ys}.
stag_status reduce_with_rescue_y(const double* partial, int P, const Operands& qo, const Operands& xo, int kernel,
                                 double scale, const BoundModel& bm, const int* near_over, const RescueBuffers& rb,
                                 double* S_out, double* bound_out, hipStream_t st) {
  const int64_t m = qo.rows, m_pad = qo.rows_pad;
  STAG_TRY(launch_reduce(partial, P, qo, xo, scale, bm, S_out, bound_out, st, near_over, rb.flag, rb.qflag));
  TileExtra exm;
  exm.max_pass = 1;
  exm.qtile_active = rb.qflag;
  STAG_TRY(launch_exact_tiles(xo, qo, rb.pmax, exm, st));
  hipLaunchKernelGGL(rescue_yshift, dim3((unsigned)ceil_div(m_pad, 256)), dim3(256), 0, st, rb.pmax, P, m_pad, m,
                     rb.flag, rb.yshift);
  STAG_TRY(check_launch("rescue_yshift"));
  TileExtra exs;
  exs.kernel = kernel;
  exs.qtile_active = rb.qflag;
  exs.yshift = rb.yshift;
  STAG_TRY(launch_exact_tiles(xo, qo, rb.p2, exs, st));
  hipLaunchKernelGGL(rescue_reduce_y, dim3((unsigned)ceil_div(m, 256)), dim3(256), 0, st, rb.p2, P, m_pad, m, rb.flag,
                     rb.yshift, scale, qo.nrm, xo.max_nrm_bits, bm, S_out, bound_out);
  return check_launch("rescue_reduce_y");
}

stag_status reduce_with_rescue_into(const double* partial, int P, const Operands& qo, const Operands& xo,
                                    double a_tile, double scale, const BoundModel& bm, const RescueBuffers& rb,
                                    double* S_out, double* bound_out, hipStream_t st) {
  STAG_TRY(launch_reduce(partial, P, qo, xo, scale, bm, S_out, bound_out, st, nullptr, rb.flag, rb.qflag));
  return rescue_underflow(xo, qo, P, a_tile, scale, bm, rb, S_out, bound_out, st);
}

stag_status reduce_with_rescue(const double* partial, int P, const Operands& qo, const Operands& xo, double a_tile,
                               double scale, const BoundModel& bm, double* S_out, double* bound_out, Workspace& ws,
                               hipStream_t st) {
  RescueBuffers rb;
  STAG_TRY(alloc_rescue(STAG_KERNEL_GAUSSIAN, P, qo, ws, &rb));
  STAG_TRY(zero_async(rb.flag, rb.zero_words * sizeof(int), st));
  return reduce_with_rescue_into(partial, P, qo, xo, a_tile, scale, bm, rb, S_out, bound_out, st);
}

namespace {

struct InputStats {
  double max_nrm_x, max_nrm_q;
  float max_abs_x, max_abs_q;
  bool nonfinite;
};

stag_status input_stats(const float* X, int64_t n, const float* Q, int64_t m, int d, Workspace& ws,
                        InputStats* out, hipStream_t st) {
  unsigned long long* nb = nullptr;
  unsigned int* ab = nullptr;
  int* bad = nullptr;
  STAG_TRY(ws.alloc(&nb, 2));
  STAG_TRY(ws.alloc(&ab, 2));
  STAG_TRY(ws.alloc(&bad, 1));
  STAG_HIP(hipMemsetAsync(nb, 0, 2 * sizeof(unsigned long long), st));
  STAG_HIP(hipMemsetAsync(ab, 0, 2 * sizeof(unsigned int), st));
  STAG_HIP(hipMemsetAsync(bad, 0, sizeof(int), st));
  hipLaunchKernelGGL(scan_rows, dim3((unsigned)ceil_div(n, kScanRowsPerBlock)), dim3(256), 0, st, X, n, d, nb, ab,
                     bad);
  STAG_TRY(check_launch("scan_rows"));
  hipLaunchKernelGGL(scan_rows, dim3((unsigned)ceil_div(m, kScanRowsPerBlock)), dim3(256), 0, st, Q, m, d, nb + 1,
                     ab + 1, bad);
  STAG_TRY(check_launch("scan_rows"));
  unsigned long long hn[2];
  unsigned int ha[2];
  int hb = 0;
  STAG_HIP(hipMemcpyAsync(hn, nb, sizeof(hn), hipMemcpyDeviceToHost, st));
  STAG_HIP(hipMemcpyAsync(ha, ab, sizeof(ha), hipMemcpyDeviceToHost, st));
  STAG_HIP(hipMemcpyAsync(&hb, bad, sizeof(int), hipMemcpyDeviceToHost, st));
  STAG_HIP(hipStreamSynchronize(st));
  std::memcpy(&out->max_nrm_x, &hn[0], sizeof(double));
  std::memcpy(&out->max_nrm_q, &hn[1], sizeof(double));
  std::memcpy(&out->max_abs_x, &ha[0], sizeof(float));
  std::memcpy(&out->max_abs_q, &ha[1], sizeof(float));
  out->nonfinite = hb != 0;
  return STAG_OK;
}

// The cheapest form whose a-priori bound at the largest query norm is <= eps
// (the bound grows with ||q||), FP32 if none is.
int choose_form(int d, double a_tile, int kernel, double eps, const InputStats& is) {
  const double qscale = 2.0 * a_tile * kLog2e;  // the split query operand is q * qscale
  const bool fp16_ok = (double)is.max_abs_x < 65504.0 && (double)is.max_abs_q * qscale < 65504.0;
  const int order[3] = {STAG_FORM_FP16_SPLIT, STAG_FORM_BF16_SPLIT, STAG_FORM_BF16_SPLIT3};
  if (d <= 256)
    for (int f : order) {
      if (f == STAG_FORM_FP16_SPLIT && !fp16_ok) continue;
      if (relative_bound(make_bound_model(f, d, a_tile, kernel), is.max_nrm_q, is.max_nrm_x) <= eps) return f;
    }
  return STAG_FORM_FP32;
}

stag_status check_exact_args(const char* fn, const float* X, int64_t n, const float* Q, int64_t m, int32_t d,
                             int32_t kernel, double a, double eps, int32_t form, uint32_t flags, double* S_out) {
  if (!X || !Q || !S_out) return fail(STAG_E_INVAL, "%s: NULL pointer argument", fn);
  if (n < 1 || m < 1 || d < 1) return fail(STAG_E_INVAL, "%s: n, m, d must be >= 1", fn);
  if (!(a > 0.0) || !std::isfinite(a)) return fail(STAG_E_INVAL, "%s: a must be positive and finite", fn);
  if (kernel < STAG_KERNEL_GAUSSIAN || kernel > STAG_KERNEL_LOGISTIC)
    return fail(STAG_E_INVAL, "%s: unknown kernel %d", fn, kernel);
  if (form < STAG_FORM_FP32 || form > STAG_FORM_FP16_ADAPTIVE)
    return fail(STAG_E_INVAL, "%s: unknown form %d", fn, form);
  if ((form == STAG_FORM_FP16_CENTRED || form == STAG_FORM_FP16_ADAPTIVE) && kernel != STAG_KERNEL_GAUSSIAN)
    return fail(STAG_E_UNSUPPORTED, "%s: the fp16 centred forms compute Gaussian sums only", fn);
  if (form == STAG_FORM_AUTO && !(eps > 0.0))
    return fail(STAG_E_INVAL, "%s: STAG_FORM_AUTO needs a target eps > 0", fn);
  if (flags & ~(STAG_NORMALIZE | STAG_CHECK_FINITE)) return fail(STAG_E_INVAL, "%s: unknown flags 0x%x", fn, flags);
  if (d > 1024) return fail(STAG_E_UNSUPPORTED, "%s: d = %d > 1024 is not supported", fn, d);
  if (d > 256 && form != STAG_FORM_FP32 && form != STAG_FORM_AUTO && form != STAG_FORM_FP16_SPLIT &&
      form != STAG_FORM_BF16_SPLIT)
    return fail(STAG_E_UNSUPPORTED, "%s: d = %d > 256 is supported by the fp32, fp16 split and bf16 split forms only",
                fn, d);
  if ((double)n * d >= 2147483648.0 || (double)m * d >= 2147483648.0)
    return fail(STAG_E_INVAL, "%s: n*d and m*d must be < 2^31", fn);
  const double at = kernel_tile_a(kernel, a);
  if (!std::isfinite(at) || !(at > 0.0)) return fail(STAG_E_INVAL, "%s: a out of range for this kernel", fn);
  return STAG_OK;
}

// Every device buffer of one exact call, taken from one Workspace before
// any launch (so that a counting Workspace gives the call's exact need).
struct ExactBuffers {
  Operands xo, qo;
  int P = 0;
  double* partial = nullptr;
  RescueBuffers rb;
  // centred data (fp32 or fp16 centred form, Gaussian kernel, d <= 256)
  bool centred = false;
  CentreTemp ct;
  double *bpart = nullptr, *bp2 = nullptr;
  // adaptive form: the split operands (data in the grouped order, queries
  // sorted), the query order, the first pass's sums, the chunk selection
  // and the sorted results
  bool adaptive = false;
  Operands xs, qsp;
  QuerySort qs;
  double *S1 = nullptr, *T = nullptr, *Ss = nullptr, *Bs = nullptr;
  uint8_t* cflag = nullptr;
  int* qsample = nullptr;
  unsigned int* counts = nullptr;
  // records of the main tile launch where several workgroups share a chunk
  TileExtra share;
};

// The fp32 form of the Gaussian sum centres the data tile by tile (the wide
// tile of d > 256 does not); the fp16 centred form centres it group by group.
bool use_centred(int form, int kernel, int d) {
  return (form == STAG_FORM_FP32 || form == STAG_FORM_FP16_CENTRED) && kernel == STAG_KERNEL_GAUSSIAN &&
         exact_padded_dim(d) <= 256;
}

stag_status alloc_exact(int form, int kernel, int64_t n, int64_t m, int d, Workspace& ws, ExactBuffers* b) {
  if (form == STAG_FORM_FP16_ADAPTIVE) {
    b->centred = true;
    b->adaptive = true;
    STAG_TRY(alloc_centred_h_operands(n, d, ws, &b->xo));
    STAG_TRY(alloc_centre_temp(b->xo, ws, &b->ct));
    STAG_TRY(alloc_operands(STAG_FORM_FP32, m, d, true, ws, &b->qo));
    STAG_TRY(alloc_operands(STAG_FORM_FP16_SPLIT, b->xo.rows_pad, d, false, ws, &b->xs));
    STAG_TRY(alloc_operands(STAG_FORM_FP16_SPLIT, m, d, true, ws, &b->qsp));
    STAG_TRY(alloc_query_sort(m, b->qo.rows_pad, b->ct.K, ws, &b->qs));
    b->P = (int)exact_chunks(b->xo.rows_pad);
    const int64_t m_pad = b->qo.rows_pad;
    STAG_TRY(ws.alloc(&b->partial, (size_t)b->P * m_pad));
    STAG_TRY(ws.alloc(&b->bpart, (size_t)b->P * m_pad));
    STAG_TRY(ws.alloc(&b->S1, (size_t)m_pad));
    STAG_TRY(ws.alloc(&b->T, (size_t)m_pad));
    STAG_TRY(ws.alloc(&b->Ss, (size_t)m_pad));
    STAG_TRY(ws.alloc(&b->Bs, (size_t)m_pad));
    STAG_TRY(ws.alloc(&b->cflag, (size_t)b->P * ceil_div(m_pad, 256)));
    STAG_TRY(ws.alloc(&b->qsample, (size_t)(m_pad / kBQ)));
    STAG_TRY(ws.alloc(&b->counts, 2));
    STAG_TRY(alloc_parts(b->xo, b->qo, kernel, ws, &b->share));
    return alloc_rescue(kernel, b->P, b->qsp, ws, &b->rb);
  }
  if (use_centred(form, kernel, d)) {
    b->centred = true;
    if (form == STAG_FORM_FP16_CENTRED)
      STAG_TRY(alloc_centred_h_operands(n, d, ws, &b->xo));
    else
      STAG_TRY(alloc_centred_operands(n, d, ws, &b->xo));
    STAG_TRY(alloc_centre_temp(b->xo, ws, &b->ct));
    STAG_TRY(alloc_operands(STAG_FORM_FP32, m, d, true, ws, &b->qo));
    b->P = (int)exact_chunks(b->xo.rows_pad);
    STAG_TRY(ws.alloc(&b->partial, (size_t)b->P * b->qo.rows_pad));
    STAG_TRY(ws.alloc(&b->bpart, (size_t)b->P * b->qo.rows_pad));
    STAG_TRY(ws.alloc(&b->bp2, (size_t)b->P * b->qo.rows_pad));
    STAG_TRY(alloc_parts(b->xo, b->qo, kernel, ws, &b->share));
    return alloc_rescue(kernel, b->P, b->qo, ws, &b->rb);
  }
  STAG_TRY(alloc_operands(form, n, d, false, ws, &b->xo));
  STAG_TRY(alloc_operands(form, m, d, true, ws, &b->qo));
  b->P = (int)exact_chunks(b->xo.rows_pad);
  STAG_TRY(ws.alloc(&b->partial, (size_t)b->P * b->qo.rows_pad));
  STAG_TRY(alloc_parts(b->xo, b->qo, kernel, ws, &b->share));
  return alloc_rescue(kernel, b->P, b->qo, ws, &b->rb);
}

// Centred Gaussian sum (fp32, or the fp16 centred form): grouping and
// centring of X, the unscaled query copy, the centred tiles with their bound
// numerators, the reduction, and the underflow rescue (max pass, offsets
// -m_q, second pass) on the same tiles.
stag_status run_centred(const float* X, int64_t n, const float* Q, int64_t m, int32_t d, double a, uint32_t flags,
                        double* S_out, double* bound_out, const ExactBuffers& b, hipStream_t st) {
  const Operands& xo = b.xo;
  const Operands& qo = b.qo;
  const RescueBuffers& rb = b.rb;
  if (xo.form == STAG_FORM_FP16_CENTRED)
    STAG_TRY(prep_centred_h_operands(X, a, xo, b.ct, st));
  else
    STAG_TRY(prep_centred_operands(X, a, xo, b.ct, st));
  STAG_TRY(prep_sides(STAG_FORM_FP32, side_of(Q, a, true, true, qo), PrepSide{}, d, qo.dp,
                      {reinterpret_cast<uint32_t*>(rb.flag), (int64_t)rb.zero_words}, st));
  const BoundModel bm = make_bound_model(STAG_FORM_FP32, d, a, STAG_KERNEL_GAUSSIAN);
  TileExtra ex = b.share;
  ex.a = a;
  ex.bpart = b.bpart;
  ex.c_cent = (float)bm.c_cent;
  STAG_TRY(launch_exact_tiles(xo, qo, b.partial, ex, st));
  const double scale = (flags & STAG_NORMALIZE) ? 1.0 / (double)n : 1.0;
  const int64_t m_pad = qo.rows_pad;
  {
    ScopedTimer tm("kde_reduce", st);
    hipLaunchKernelGGL(reduce_centred, dim3((unsigned)ceil_div(m, 256)), dim3(256), 0, st, b.partial, b.bpart, b.P,
                       m_pad, m, scale, bm.c_tail, S_out, bound_out, rb.flag, rb.qflag);
    STAG_TRY(check_launch("reduce_centred"));
  }
  TileExtra exm;
  exm.max_pass = 1;
  exm.qtile_active = rb.qflag;
  exm.a = a;
  STAG_TRY(launch_exact_tiles(xo, qo, rb.pmax, exm, st));
  hipLaunchKernelGGL(rescue_shift_centred, dim3((unsigned)ceil_div(m_pad, 256)), dim3(256), 0, st, rb.pmax, b.P,
                     m_pad, m, rb.flag, qo.off, rb.off2, rb.shift);
  STAG_TRY(check_launch("rescue_shift_centred"));
  Operands q2 = qo;
  q2.off = rb.off2;
  TileExtra exs = ex;
  exs.qtile_active = rb.qflag;
  exs.bpart = b.bp2;
  STAG_TRY(launch_exact_tiles(xo, q2, rb.p2, exs, st));
  hipLaunchKernelGGL(rescue_reduce_centred, dim3((unsigned)ceil_div(m, 256)), dim3(256), 0, st, rb.p2, b.bp2, b.P,
                     m_pad, m, rb.flag, rb.shift, scale, bm.c_tail, S_out, bound_out);
  return check_launch("rescue_reduce_centred");
}

// Adaptive fp16 form: the single-product centred pass over all pairs with
// the queries in group order, then the fp16 split form over the (chunk,
// 256-query tile) pairs where some query's first-pass bound numerator lies
// above the part of its budget, kAdaptiveShare of its sum, that its smaller
// numerators fill (adaptive_budget), the reduction in sorted order with the
// underflow rescue in the split form, and the results back to the query rows.
// First an estimate: the single-product pass and the selection on every
// stride-th 128-query tile (about kAdaptiveSamples of them), read back with
// one synchronisation; when more than kAdaptiveMaxShare of the sampled pairs
// are selected (wide kernels: every chunk matters), the single-product pass
// is skipped and every pair runs in the split form.
constexpr double kAdaptiveShare = 1.0e-5;
constexpr int kAdaptiveSamples = 8;
constexpr double kAdaptiveMaxShare = 0.5;

stag_status run_adaptive(const float* X, int64_t n, const float* Q, int64_t m, int32_t d, double a, uint32_t flags,
                         double* S_out, double* bound_out, const ExactBuffers& b, hipStream_t st) {
  const Operands& xo = b.xo;
  const Operands& qo = b.qo;
  const int64_t m_pad = qo.rows_pad;
  const int n_qt256 = (int)ceil_div(m_pad, 256);
  STAG_TRY(prep_centred_h_operands(X, a, xo, b.ct, st));
  STAG_TRY(sort_queries(Q, m, m_pad, d, xo.dp, b.ct, b.qs, st));
  STAG_TRY(prep_sides(STAG_FORM_FP32, side_of(Q, a, true, true, qo, b.qs.perm), PrepSide{}, d, qo.dp, ZeroRange(), st));
  STAG_TRY(zero_async(b.xs.max_nrm_bits, sizeof(unsigned long long), st));
  STAG_TRY(prep_sides(STAG_FORM_FP16_SPLIT, side_of(X, a, false, false, b.xs, b.ct.map),
                      side_of(Q, a, true, false, b.qsp, b.qs.perm), d, b.xs.dp,
                      {reinterpret_cast<uint32_t*>(b.rb.flag), (int64_t)b.rb.zero_words}, st));
  // first pass: one fp16 product per pair, with the bound numerators, then
  // the selection of the pairs to recompute (on the sampled tiles: qmask)
  const BoundModel bm1 = make_bound_model(STAG_FORM_FP32, d, a, STAG_KERNEL_GAUSSIAN);
  TileExtra ex1 = b.share;
  ex1.a = a;
  ex1.bpart = b.bpart;
  ex1.c_cent = (float)bm1.c_cent;
  const int n_qt128 = (int)(m_pad / kBQ);
  const int stride = std::max(1, n_qt128 / kAdaptiveSamples);
  auto first_pass = [&](const int* qmask) -> stag_status {
    TileExtra e = ex1;
    e.qtile_active = qmask;
    e.sample = qmask ? 1 : 0;
    e.fold_alpha = 1;
    if (qmask && ceil_div(n_qt128, stride) <= TileExtra::kMaxSel) {
      // the sampled tiles (those mark_sample flags), launched alone
      for (int t = 0; t < n_qt128; t += stride) e.qsel[e.qsel_n++] = t;
    }
    STAG_TRY(launch_exact_tiles(xo, qo, b.partial, e, st));
    ScopedTimer tm("kde_adaptive_select", st);
    hipLaunchKernelGGL(adaptive_budget, dim3((unsigned)ceil_div(m_pad, 256)), dim3(256), 0, st, b.partial, b.bpart,
                       b.P, m_pad, m, kAdaptiveShare, qmask, b.S1, b.T);
    STAG_TRY(check_launch("adaptive_budget"));
    STAG_TRY(zero_async(b.cflag, (size_t)b.P * n_qt256, st));
    hipLaunchKernelGGL(adaptive_flags, dim3((unsigned)ceil_div(m, 256), (unsigned)b.P), dim3(256), 0, st, b.bpart,
                       b.T, m_pad, m, n_qt256, qmask, b.cflag);
    return check_launch("adaptive_flags");
  };
  hipLaunchKernelGGL(mark_sample, dim3((unsigned)ceil_div(n_qt128, 256)), dim3(256), 0, st, b.qsample, n_qt128,
                     stride);
  STAG_TRY(check_launch("mark_sample"));
  STAG_TRY(first_pass(stride > 1 ? b.qsample : nullptr));
  unsigned int hc[2] = {0u, 0u};
  {
    ScopedTimer tm("kde_adaptive_select", st);
    STAG_TRY(zero_async(b.counts, 2 * sizeof(unsigned int), st));
    hipLaunchKernelGGL(count_selected, dim3((unsigned)ceil_div(n_qt256, 256), (unsigned)b.P), dim3(256), 0, st,
                       b.cflag, n_qt256, b.qsample, n_qt128, b.counts);
    STAG_TRY(check_launch("count_selected"));
    STAG_HIP(hipMemcpyAsync(hc, b.counts, sizeof(hc), hipMemcpyDeviceToHost, st));
    STAG_HIP(hipStreamSynchronize(st));
  }
  if (hc[1] > 0 && (double)hc[0] > kAdaptiveMaxShare * (double)hc[1]) {
    // every pair in the split form (the partials of the sampled pass are overwritten)
    hipLaunchKernelGGL(fill_ones, dim3((unsigned)ceil_div((int64_t)b.P * n_qt256, 256)), dim3(256), 0, st, b.cflag,
                       (int64_t)b.P * n_qt256);
    STAG_TRY(check_launch("fill_ones"));
  } else if (stride > 1) {
    STAG_TRY(first_pass(nullptr));
  }
  // second pass: the split form on the selected pairs (overwrites their partials)
  TileExtra ex2;
  ex2.cflag = b.cflag;
  STAG_TRY(launch_exact_tiles(b.xs, b.qsp, b.partial, ex2, st));
  const BoundModel bm2 = make_bound_model(STAG_FORM_FP16_SPLIT, d, a, STAG_KERNEL_GAUSSIAN);
  const double scale = (flags & STAG_NORMALIZE) ? 1.0 / (double)n : 1.0;
  {
    ScopedTimer tm("kde_reduce", st);
    hipLaunchKernelGGL(reduce_adaptive, dim3((unsigned)ceil_div(m, 256)), dim3(256), 0, st, b.partial, b.bpart,
                       b.cflag, b.P, m_pad, m, n_qt256, scale, b.qsp.nrm, b.xs.max_nrm_bits, bm2, bm1.c_tail, b.Ss,
                       b.Bs, b.rb.flag, b.rb.qflag);
    STAG_TRY(check_launch("reduce_adaptive"));
  }
  // queries whose sum lies below the fp32 terms' range: recomputed in the split form
  STAG_TRY(rescue_underflow(b.xs, b.qsp, b.P, a, scale, bm2, b.rb, b.Ss, b.Bs, st));
  hipLaunchKernelGGL(scatter_results, dim3((unsigned)ceil_div(m_pad, 256)), dim3(256), 0, st, b.Ss, b.Bs, b.qs.perm,
                     m_pad, S_out, bound_out);
  return check_launch("scatter_results");
}

// The launches of one exact call into buffers from alloc_exact.
stag_status run_exact(const float* X, int64_t n, const float* Q, int64_t m, int32_t d, int32_t kernel, double a,
                      int32_t form, uint32_t flags, double* S_out, double* bound_out, const ExactBuffers& b,
                      hipStream_t stream) {
  if (b.adaptive) return run_adaptive(X, n, Q, m, d, a, flags, S_out, bound_out, b, stream);
  if (b.centred) return run_centred(X, n, Q, m, d, a, flags, S_out, bound_out, b, stream);
  const double at = kernel_tile_a(kernel, a);
  STAG_TRY(prep_operand_pair(X, Q, at, b.xo, b.qo, bound_out != nullptr, b.rb.flag, b.rb.zero_words, stream));
  TileExtra ex = b.share;
  ex.kernel = kernel;
  if (kernel == STAG_KERNEL_EXPONENTIAL) {
    ex.near_x = X;
    ex.near_q = Q;
    ex.d = d;
    ex.near_e = (float)kNearY2;
    ex.a = a;
    ex.m_rows = m;
    ex.near_over = b.rb.near_over;
  }
  STAG_TRY(launch_exact_tiles(b.xo, b.qo, b.partial, ex, stream));
  const double scale = (flags & STAG_NORMALIZE) ? 1.0 / (double)n : 1.0;
  const BoundModel bm = make_bound_model(form, d, at, kernel);
  // Gaussian: sums below kRescueBelow are recomputed with shifted exponents
  if (kernel == STAG_KERNEL_GAUSSIAN)
    return reduce_with_rescue_into(b.partial, b.P, b.qo, b.xo, at, scale, bm, b.rb, S_out, bound_out, stream);
  return reduce_with_rescue_y(b.partial, b.P, b.qo, b.xo, kernel, scale, bm, ex.near_over, b.rb, S_out, bound_out,
                              stream);
}

stag_status exact_kernel_impl(const char* fn, const float* X, int64_t n, const float* Q, int64_t m, int32_t d,
                              int32_t kernel, double a, double eps, int32_t form, uint32_t flags, double* S_out,
                              double* bound_out, hipStream_t stream) {
  STAG_TRY(check_exact_args(fn, X, n, Q, m, d, kernel, a, eps, form, flags, S_out));
  clear_error();
  Workspace ws(stream);
  if (form == STAG_FORM_AUTO || (flags & STAG_CHECK_FINITE)) {
    InputStats is;
    STAG_TRY(input_stats(X, n, Q, m, d, ws, &is, stream));
    if ((flags & STAG_CHECK_FINITE) && is.nonfinite) return fail(STAG_E_INVAL, "%s: X or Q holds NaN or Inf", fn);
    if (form == STAG_FORM_AUTO) form = choose_form(d, kernel_tile_a(kernel, a), kernel, eps, is);
  }
  ExactBuffers b;
  STAG_TRY(alloc_exact(form, kernel, n, m, d, ws, &b));
  return run_exact(X, n, Q, m, d, kernel, a, form, flags, S_out, bound_out, b, stream);
}

std::mutex g_scratch_mu;
void* g_scratch_ptr[64] = {};

stag_status scratch_on_current_device(void** out) {
  int dev = 0;
  STAG_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64) return fail(STAG_E_UNSUPPORTED, "device ordinal %d out of range", dev);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    STAG_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) return fail(STAG_E_DEVICE, "hipGetSymbolAddress gave a null scratch address");
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return STAG_OK;
}

}  // namespace
}  // namespace stag

extern "C" stag_status stag_kde_exact_noalloc(const float* X, int64_t n, const float* Q, int64_t m, int32_t d, double a,
                                              int32_t form, uint32_t flags, double* S_out, double* bound_out,
                                              hipStream_t stream) {
  using namespace stag;
  const char* fn = "stag_kde_exact_noalloc";
  if (form == STAG_FORM_AUTO) return fail(STAG_E_UNSUPPORTED, "%s: STAG_FORM_AUTO is not available here", fn);
  if (flags & STAG_CHECK_FINITE) return fail(STAG_E_UNSUPPORTED, "%s: STAG_CHECK_FINITE is not available here", fn);
  STAG_TRY(check_exact_args(fn, X, n, Q, m, d, STAG_KERNEL_GAUSSIAN, a, 0.0, form, flags, S_out));
  ExactBuffers need;
  Workspace counter{Workspace::CountTag{}};
  STAG_TRY(alloc_exact(form, STAG_KERNEL_GAUSSIAN, n, m, d, counter, &need));
  if (counter.used() > kScratchBytes)
    return fail(STAG_E_INVAL, "%s: this call needs %zu bytes of scratch, more than the %zu available", fn,
                counter.used(), kScratchBytes);
  clear_error();
  void* base = nullptr;
  STAG_TRY(scratch_on_current_device(&base));
  Workspace arena(stream, base, kScratchBytes);
  ExactBuffers b;
  STAG_TRY(alloc_exact(form, STAG_KERNEL_GAUSSIAN, n, m, d, arena, &b));
  return run_exact(X, n, Q, m, d, STAG_KERNEL_GAUSSIAN, a, form, flags, S_out, bound_out, b, stream);
}

extern "C" stag_status stag_kde_exact(const float* X, int64_t n, const float* Q, int64_t m, int32_t d, double a,
                                      double eps, int32_t form, uint32_t flags, double* S_out, double* bound_out,
                                      hipStream_t stream) {
  return stag::exact_kernel_impl("stag_kde_exact", X, n, Q, m, d, STAG_KERNEL_GAUSSIAN, a, eps, form, flags, S_out,
                                 bound_out, stream);
}

extern "C" stag_status stag_kde_exact_kernel(const float* X, int64_t n, const float* Q, int64_t m, int32_t d,
                                             int32_t kernel, double a, double eps, int32_t form, uint32_t flags,
                                             double* S_out, double* bound_out, hipStream_t stream) {
  return stag::exact_kernel_impl("stag_kde_exact_kernel", X, n, Q, m, d, kernel, a, eps, form, flags, S_out,
                                 bound_out, stream);
}
