// Spectral clustering of a weighted graph (Sec. "Fast Spectral Clustering":
// similarity graph -> bottom k eigenvectors of the Laplacian -> k-means on
// the embedded vertices).
//
// Graph.  The edge list (src, dst, w) is read as the symmetric adjacency A
// (every edge adds w at (src, dst) and at (dst, src); dst = -1 marks an empty
// draw).  Its 2E entries are keyed by row and put in row order by a stable
// radix sort, so each CSR row lists its entries in edge order and every row
// sum below is taken in a fixed order.  The Laplacian is the normalised
// N = I - D^{-1/2} A D^{-1/2}; the CSR values become the entries of
// M = D^{-1/2} A D^{-1/2} (spectrum in [-1, 1]), whose top eigenvectors are
// N's bottom ones (eigenvalue lambda = 1 - theta).
//
// Eigenvectors: Chebyshev-filtered subspace iteration (Zhou & Saad 2007) on
// a block of b = 8..64 columns (n x b, fp64, row-major, padded to a power of
// two bp):
//   filter     Y <- T_p((M - sigma) / e) V, the Chebyshev polynomial of
//              degree p that is bounded by 1 on the unwanted interval
//              [-1, c] (c = the block's smallest Ritz value) and grows fast
//              above it; three-term recurrence, one fused SpMM per degree
//   orthonormalise twice by Cholesky QR (Gram matrix V^T V = R^T R on the
//              host, V <- V R^{-1}; by its eigen-decomposition, V <- V Q L^{-1/2},
//              if a pivot fails)
//   Rayleigh-Ritz  W = M V, H = V^T W, H = Z diag(theta) Z^T on the host,
//              V <- V Z, W <- W Z (theta descending)
//   stop       when the k leading residuals ||W_j - theta_j V_j|| <= tol.
// Only b x b matrices cross to the host (cyclic Jacobi there); every n-sized
// operation is a kernel below, every reduction in a fixed order, so results
// are bitwise reproducible.
//
// k-means: Lloyd's iteration with k-means++ seeding, the decisions taken in
// the stated order (squared distances summed over coordinates in order
// without fused operations, seeding sums in blocks of 1024 points, ties to
// the lowest index; see include/stag_kde.h).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "runtime.h"
#include "scan.h"
#include "sort.h"

namespace stag {
namespace {

constexpr uint64_t kGamma = 0x9E3779B97F4A7C15ull;
constexpr uint64_t kTagSpectral = 0x53504543ull;  // "SPEC": initial block
constexpr uint64_t kTagKmeans = 0x4B4D4E53ull;    // "KMNS": k-means++ uniforms
constexpr int kKmBlock = 1024;                    // points per seeding/update block
constexpr int kMaxBlockCols = 64;
constexpr int kGramRows = 256;                    // rows per Gram workgroup

__host__ __device__ inline uint64_t sm_mix(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
// Output c of the counter stream (seed, tag): mix(state + (c+1) gamma),
// state = mix(mix(mix(seed ^ tag) ^ 0) ^ 0).
__host__ __device__ inline uint64_t stream_bits(uint64_t seed, uint64_t tag, uint64_t c) {
  const uint64_t s = sm_mix(sm_mix(sm_mix(seed ^ tag)));
  return sm_mix(s + (c + 1) * kGamma);
}

// ---------------------------------------------------------------------------
// Graph build
// ---------------------------------------------------------------------------
// Entry 2e is (row src, column dst), entry 2e+1 (row dst, column src); an
// empty draw gets the key n on both (sorted past every row).  Invalid edges
// raise *bad.
__global__ void edge_entries(const int64_t* __restrict__ src, const int64_t* __restrict__ dst,
                             const double* __restrict__ w, int64_t E, int64_t n, uint32_t* __restrict__ keys,
                             uint32_t* __restrict__ vals, int* __restrict__ bad) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= E) return;
  const int64_t s = src[e], t = dst[e];
  uint32_t k0 = (uint32_t)n, k1 = (uint32_t)n;
  const bool s_ok = s >= 0 && s < n;
  if (t == -1) {
    if (!s_ok) atomicOr(bad, 1);
  } else {
    const double we = w[e];
    if (!s_ok || t < 0 || t >= n || !(we >= 0.0) || !(we < INFINITY)) {
      atomicOr(bad, 1);
    } else {
      k0 = (uint32_t)s;
      k1 = (uint32_t)t;
    }
  }
  keys[2 * e] = k0;
  vals[2 * e] = (uint32_t)(2 * e);
  keys[2 * e + 1] = k1;
  vals[2 * e + 1] = (uint32_t)(2 * e + 1);
}

// rowptr[r] = first sorted entry with key >= r, r <= n, by bisection (counting
// the entries with atomics while they were written, then scanning, took
// 0.12 ms more at 3.4e6 entries; a thread per change of key would leave long
// runs of empty rows to one thread).
__global__ void row_starts(const uint32_t* __restrict__ sorted_keys, int64_t ne, int64_t n,
                           uint64_t* __restrict__ rowptr) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r > n) return;
  int64_t lo = 0, hi = ne;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if ((int64_t)sorted_keys[mid] < r) lo = mid + 1;
    else hi = mid;
  }
  rowptr[r] = (uint64_t)lo;
}

__global__ void csr_fill(const uint32_t* __restrict__ sorted_vals, const uint64_t* __restrict__ rowptr, int64_t n,
                         int64_t cap, const int64_t* __restrict__ src, const int64_t* __restrict__ dst,
                         const double* __restrict__ w, int32_t* __restrict__ col, double* __restrict__ val) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= cap || i >= (int64_t)rowptr[n]) return;
  const uint32_t v = sorted_vals[i];
  const int64_t e = v >> 1;
  col[i] = (int32_t)((v & 1u) ? src[e] : dst[e]);
  val[i] = w[e];
}

// deg(r) = row sum in CSR order; dinv = deg^{-1/2} (0 for an isolated vertex).
__global__ void row_dinv(const uint64_t* __restrict__ rowptr, const double* __restrict__ val, int64_t n,
                         double* __restrict__ deg, double* __restrict__ dinv) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  double s = 0.0;
  for (uint64_t i = rowptr[r]; i < rowptr[r + 1]; ++i) s += val[i];
  deg[r] = s;
  dinv[r] = s > 0.0 ? 1.0 / sqrt(s) : 0.0;
}

// One thread per entry, its row from the sorted keys.
__global__ void normalise_vals(const uint64_t* __restrict__ rowptr, const uint32_t* __restrict__ row,
                               const int32_t* __restrict__ col, const double* __restrict__ dinv, int64_t n,
                               int64_t cap, double* __restrict__ val) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= cap || i >= (int64_t)rowptr[n]) return;
  val[i] = dinv[row[i]] * val[i] * dinv[col[i]];
}

// ---------------------------------------------------------------------------
// Block operations (X [n][bp] fp64 row-major, the first b columns in use)
// ---------------------------------------------------------------------------
// Y = alpha (M X) + beta X + gamma Z; LPR lanes per row, two columns per lane.
template <int LPR>
__global__ __launch_bounds__(256) void spmm_comb(const uint64_t* __restrict__ rowptr,
                                                 const int32_t* __restrict__ col, const double* __restrict__ val,
                                                 int64_t n, const double2* __restrict__ X,
                                                 const double2* __restrict__ Z, double2* __restrict__ Y, double alpha,
                                                 double beta, double gamma) {
  constexpr int RPB = 256 / LPR;
  const int64_t r = (int64_t)blockIdx.x * RPB + threadIdx.x / LPR;
  const int c = threadIdx.x % LPR;
  if (r >= n) return;
  double ax = 0.0, ay = 0.0;
  const uint64_t e1 = rowptr[r + 1];
  for (uint64_t i = rowptr[r]; i < e1; ++i) {
    const double v = val[i];
    const double2 x = X[(int64_t)col[i] * LPR + c];
    ax = fma(v, x.x, ax);
    ay = fma(v, x.y, ay);
  }
  const double2 xr = X[r * LPR + c];
  double yx = alpha * ax + beta * xr.x;
  double yy = alpha * ay + beta * xr.y;
  if (Z) {
    const double2 z = Z[r * LPR + c];
    yx += gamma * z.x;
    yy += gamma * z.y;
  }
  Y[r * LPR + c] = make_double2(yx, yy);
}

// Partial Gram matrices A^T B over kGramRows rows per workgroup, rows in
// order; part [nblk][b][b].
__global__ __launch_bounds__(256) void gram_partial(const double* __restrict__ A, const double* __restrict__ B,
                                                    int64_t n, int bp, int b, double* __restrict__ part) {
  __shared__ __attribute__((aligned(16))) double sa[32 * kMaxBlockCols];
  __shared__ __attribute__((aligned(16))) double sb[32 * kMaxBlockCols];
  const int tid = threadIdx.x;
  const int bb = b * b;
  const int64_t r0 = (int64_t)blockIdx.x * kGramRows;
  // each thread 2 x 2 elements at a time (two 16-byte LDS reads for four
  // products; one element at a time, 1e5 x 28 took 41 us, now 28;
  // the columns past b are zero in LDS and not stored)
  const int h = (b + 1) / 2, hh = h * h;
  double acc[4][2][2];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int u = 0; u < 2; ++u) acc[q][u][0] = acc[q][u][1] = 0.0;
  for (int rr = 0; rr < kGramRows; rr += 32) {
    for (int v = tid; v < 32 * bp; v += 256) {
      const int64_t row = r0 + rr + v / bp;
      const int cc = v % bp;
      sa[(v / bp) * kMaxBlockCols + cc] = row < n ? A[row * bp + cc] : 0.0;
      sb[(v / bp) * kMaxBlockCols + cc] = row < n ? B[row * bp + cc] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int e = tid + 256 * q;
      if (e < hh) {
        const double* pa = sa + 2 * (e / h);
        const double* pb = sb + 2 * (e % h);
#pragma unroll 4
        for (int t = 0; t < 32; ++t) {
          const double2 x = *reinterpret_cast<const double2*>(pa + t * kMaxBlockCols);
          const double2 y = *reinterpret_cast<const double2*>(pb + t * kMaxBlockCols);
          acc[q][0][0] = fma(x.x, y.x, acc[q][0][0]);
          acc[q][0][1] = fma(x.x, y.y, acc[q][0][1]);
          acc[q][1][0] = fma(x.y, y.x, acc[q][1][0]);
          acc[q][1][1] = fma(x.y, y.y, acc[q][1][1]);
        }
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int e = tid + 256 * q;
    if (e < hh) {
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int w = 0; w < 2; ++w) {
          const int i = 2 * (e / h) + u, j = 2 * (e % h) + w;
          if (i < b && j < b) part[(int64_t)blockIdx.x * bb + i * b + j] = acc[q][u][w];
        }
    }
  }
}

// G[e] = sum over blocks of part[block][e], in order.  A workgroup takes
// kFinalCols elements: all its threads bring 512 partials of each to LDS, one
// thread per element adds them (with a thread reading its own partials 8 at a
// time, 391 partials of 28 x 28 took 21 us; now 7).
constexpr int kFinalCols = 8, kFinalRows = 512;
__global__ __launch_bounds__(256) void gram_final(const double* __restrict__ part, int64_t nblk, int bb,
                                                  double* __restrict__ G) {
  __shared__ double v[kFinalRows * kFinalCols];
  const int tid = threadIdx.x;
  const int e0 = blockIdx.x * kFinalCols;
  const int c = tid % kFinalCols;
  double s = 0.0;
  for (int64_t g0 = 0; g0 < nblk; g0 += kFinalRows) {
    const int rows = (int)min((int64_t)kFinalRows, nblk - g0);
    double t[kFinalRows * kFinalCols / 256];
#pragma unroll
    for (int q = 0; q < kFinalRows * kFinalCols / 256; ++q) {
      const int r = tid / kFinalCols + q * (256 / kFinalCols);
      t[q] = r < rows && e0 + c < bb ? part[(g0 + r) * bb + e0 + c] : 0.0;
    }
    __syncthreads();  // the last chunk is added
#pragma unroll
    for (int q = 0; q < kFinalRows * kFinalCols / 256; ++q) v[tid + 256 * q] = t[q];
    __syncthreads();
    if (tid < kFinalCols) {
      int r = 0;
      for (; r + 16 <= rows; r += 16) {
#pragma unroll
        for (int u = 0; u < 16; ++u) s += v[(r + u) * kFinalCols + tid];
      }
      for (; r < rows; ++r) s += v[r * kFinalCols + tid];
    }
  }
  if (tid < kFinalCols && e0 + tid < bb) G[e0 + tid] = s;
}

// Rinv (b x b row-major) = R^{-1} of the Cholesky factor G = R^T R, R upper
// triangular; *broken = 1 and Rinv unset if a pivot is not positive.  One
// workgroup: a step scales row j and updates the rows below it in parallel,
// then a thread per column substitutes backwards.  Each element sees the same
// unfused operations in the same order as the host's cholesky_inverse.  On the
// device to save the read-back and upload between two kernels (31 us against
// 66 for the two copies and the host's factor at b = 28).
constexpr int kCholLd = kMaxBlockCols + 1;
__global__ __launch_bounds__(1024) void chol_inverse(const double* __restrict__ G, int b, double* __restrict__ Rinv,
                                                     int* __restrict__ broken) {
#pragma clang fp contract(off)
  // R[i][k], i <= k, at i ld + k; X[k][c], k <= c, at (c + 1) ld + k
  __shared__ double L[kCholLd * kCholLd];
  const int tid = threadIdx.x;
  for (int v = tid; v < b * b; v += 1024)
    if (v / b <= v % b) L[v / b * kCholLd + v % b] = G[v];
  __syncthreads();
  for (int j = 0; j < b; ++j) {
    const double dj = L[j * kCholLd + j];
    if (!(dj > 0.0) || !isfinite(dj)) {  // the same in every thread
      if (tid == 0) *broken = 1;
      return;
    }
    const double rjj = sqrt(dj);
    __syncthreads();
    if (tid >= j && tid < b) L[j * kCholLd + tid] = tid == j ? rjj : L[j * kCholLd + tid] / rjj;
    __syncthreads();
    const int m = b - 1 - j;
    for (int v = tid; v < m * m; v += 1024) {
      const int r = j + 1 + v / m, i = j + 1 + v % m;
      if (r <= i)
        L[r * kCholLd + i] -= L[j * kCholLd + r] * L[j * kCholLd + i];
    }
    __syncthreads();
  }
  if (tid < b) {
    const int c = tid;
    double* X = L + (c + 1) * kCholLd;
    for (int i = c; i >= 0; --i) {
      double v = i == c ? 1.0 : 0.0;
      for (int k = i + 1; k <= c; ++k) v -= L[i * kCholLd + k] * X[k];
      X[i] = v / L[i * kCholLd + i];
    }
  }
  __syncthreads();
  for (int v = tid; v < b * b; v += 1024) {
    const int i = v / b, c = v % b;
    Rinv[v] = i <= c ? L[(c + 1) * kCholLd + i] : 0.0;
  }
}

// Y[:, :b] = X[:, :b] R (R b x b row-major), Y[:, b:bp] = 0.  A thread forms
// one column of kApplyRows rows, so that an element of R read from LDS serves
// that many products (one row a thread was bound by its two LDS reads a
// product: 1e5 x 28 by 28 took 33 us, now 23).  Does nothing if *broken (broken may be NULL).
constexpr int kApplyRows = 8;
__global__ __launch_bounds__(256) void apply_small(const double* __restrict__ X, int64_t n, int bp, int b,
                                                   const double* __restrict__ R, const int* __restrict__ broken,
                                                   double* __restrict__ Y) {
  if (broken && *broken) return;
  __shared__ double sR[kMaxBlockCols * kMaxBlockCols];
  __shared__ double sx[256 * kApplyRows];
  const int tid = threadIdx.x;
  for (int v = tid; v < b * b; v += 256) sR[v] = R[v];
  const int rpb = 256 / bp * kApplyRows;  // rows of the block
  const int64_t row0 = (int64_t)blockIdx.x * rpb;
  for (int v = tid; v < rpb * bp; v += 256) sx[v] = row0 * bp + v < n * bp ? X[row0 * bp + v] : 0.0;
  __syncthreads();
  const int g = tid / bp, j = tid % bp;
  const double* xr = &sx[g * kApplyRows * bp];
  double y[kApplyRows];
#pragma unroll
  for (int r = 0; r < kApplyRows; ++r) y[r] = 0.0;
  if (j < b) {
    for (int i = 0; i < b; ++i) {
      const double rv = sR[i * b + j];
#pragma unroll
      for (int r = 0; r < kApplyRows; ++r) y[r] = fma(xr[r * bp + i], rv, y[r]);
    }
  }
#pragma unroll
  for (int r = 0; r < kApplyRows; ++r) {
    const int64_t row = row0 + g * kApplyRows + r;
    if (row < n) Y[row * bp + j] = y[r];
  }
}

// Per kGramRows rows: the squared norms of the first b columns of
// W - V diag(theta), rows in order (storing the residual and forming its whole
// Gram matrix took 42 us at 1e5 x 28; this takes 16).
__global__ __launch_bounds__(256) void residual_norms(const double* __restrict__ W, const double* __restrict__ V,
                                                      const double* __restrict__ theta, int64_t n, int bp, int b,
                                                      double* __restrict__ part) {
  __shared__ double sr[32 * kMaxBlockCols];
  const int tid = threadIdx.x;
  const int64_t r0 = (int64_t)blockIdx.x * kGramRows;
  const double th = tid % bp < b ? theta[tid % bp] : 0.0;  // bp divides 256
  double acc = 0.0;
  for (int rr = 0; rr < kGramRows; rr += 32) {
    for (int v = tid; v < 32 * bp; v += 256) {
      const int64_t at = (r0 + rr) * bp + v;
      sr[v] = at < n * bp ? fma(-th, V[at], W[at]) : 0.0;
    }
    __syncthreads();
    if (tid < b) {
#pragma unroll 8
      for (int t = 0; t < 32; ++t) acc = fma(sr[t * bp + tid], sr[t * bp + tid], acc);
    }
    __syncthreads();
  }
  if (tid < b) part[(int64_t)blockIdx.x * b + tid] = acc;
}

__global__ void init_block(double* __restrict__ V, int64_t n, int bp, int b, uint64_t seed) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * bp) return;
  const int j = (int)(i % bp);
  const int64_t r = i / bp;
  double v = 0.0;
  if (j < b) v = (double)(stream_bits(seed, kTagSpectral, (uint64_t)(r * b + j)) >> 11) * 0x1.0p-52 - 1.0;
  V[i] = v;
}

// The larger of (v, i) and (w, j), the smaller index on ties.
__device__ inline void take_larger(double& v, int64_t& i, double w, int64_t j) {
  if (w > v || (w == v && j < i)) {
    v = w;
    i = j;
  }
}

// Column j < k: the entry of largest magnitude (lowest row on ties) per
// workgroup of 256 rows, then over workgroups.  Thread t: column t % bp.
__global__ __launch_bounds__(256) void col_absmax_partial(const double* __restrict__ V, int64_t n, int bp, int k,
                                                          double* __restrict__ pv, int64_t* __restrict__ pi) {
  __shared__ double sv[256];
  __shared__ int64_t si[256];
  const int64_t r0 = (int64_t)blockIdx.x * 256, r1 = min(n, r0 + 256);
  const int tid = threadIdx.x, j = tid % bp;
  double best = -1.0;
  int64_t bi = INT64_MAX;
  for (int64_t r = r0 + tid / bp; r < r1; r += 256 / bp) {
    const double a = fabs(V[r * bp + j]);
    if (a > best) {
      best = a;
      bi = r;
    }
  }
  sv[tid] = best;
  si[tid] = bi;
  __syncthreads();
  if (tid >= k) return;  // k <= bp: j == tid
  for (int t = tid + bp; t < 256; t += bp) take_larger(best, bi, sv[t], si[t]);
  pv[(int64_t)blockIdx.x * k + tid] = best;
  pi[(int64_t)blockIdx.x * k + tid] = bi;
}

__global__ __launch_bounds__(256) void col_sign(const double* __restrict__ pv, const int64_t* __restrict__ pi,
                                                int64_t nblk, const double* __restrict__ V, int bp, int k,
                                                double* __restrict__ sign) {
  __shared__ double sv[256];
  __shared__ int64_t si[256];
  const int j = blockIdx.x, tid = threadIdx.x;
  double best = -1.0;
  int64_t bi = INT64_MAX;
  for (int64_t g = tid; g < nblk; g += 256) take_larger(best, bi, pv[g * k + j], pi[g * k + j]);
  sv[tid] = best;
  si[tid] = bi;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (tid < o) take_larger(sv[tid], si[tid], sv[tid + o], si[tid + o]);
    __syncthreads();
  }
  if (tid != 0) return;
  const int64_t at = sv[0] >= 0.0 ? si[0] : 0;  // a column of NaN: row 0
  sign[j] = V[at * bp + j] < 0.0 ? -1.0 : 1.0;
}

__global__ void extract_embedding(const double* __restrict__ V, int64_t n, int bp, int k,
                                  const double* __restrict__ sign, double* __restrict__ U) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * k) return;
  const int64_t r = i / k;
  const int j = (int)(i % k);
  U[i] = sign[j] * V[r * bp + j];
}

__global__ void eig_out(const double* __restrict__ theta, int k, double* __restrict__ lam) {
  const int j = threadIdx.x;
  if (j < k) lam[j] = 1.0 - theta[j];
}

__global__ void fill_i32(int32_t* p, int64_t n, int32_t v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// ---------------------------------------------------------------------------
// Host dense helpers (b <= 64)
// ---------------------------------------------------------------------------
// Cyclic Jacobi eigen-decomposition of the symmetric b x b matrix A
// (row-major); eigenvalues descending in w, eigenvectors as the columns of Z.
void jacobi_eigen(std::vector<double> A, int b, std::vector<double>& w, std::vector<double>& Z) {
  Z.assign((size_t)b * b, 0.0);
  for (int i = 0; i < b; ++i) Z[(size_t)i * b + i] = 1.0;
  for (int sweep = 0; sweep < 100; ++sweep) {
    double off = 0.0, tot = 0.0;
    for (int i = 0; i < b; ++i)
      for (int j = 0; j < b; ++j) {
        const double v = A[(size_t)i * b + j] * A[(size_t)i * b + j];
        tot += v;
        if (i != j) off += v;
      }
    // relative off-diagonal size 1e-14: below it further sweeps only trade
    // rounding noise
    if (off <= 1e-28 * tot || off == 0.0) break;
    for (int p = 0; p < b - 1; ++p)
      for (int q = p + 1; q < b; ++q) {
        const double apq = A[(size_t)p * b + q];
        if (apq == 0.0) continue;
        const double app = A[(size_t)p * b + p], aqq = A[(size_t)q * b + q];
        const double tau = (aqq - app) / (2.0 * apq);
        const double t = (tau >= 0.0 ? 1.0 : -1.0) / (std::fabs(tau) + std::sqrt(1.0 + tau * tau));
        const double c = 1.0 / std::sqrt(1.0 + t * t), s = t * c;
        for (int r = 0; r < b; ++r) {  // A <- A J (columns p, q)
          const double arp = A[(size_t)r * b + p], arq = A[(size_t)r * b + q];
          A[(size_t)r * b + p] = c * arp - s * arq;
          A[(size_t)r * b + q] = s * arp + c * arq;
        }
        for (int r = 0; r < b; ++r) {  // A <- J^T A (rows p, q)
          const double apr = A[(size_t)p * b + r], aqr = A[(size_t)q * b + r];
          A[(size_t)p * b + r] = c * apr - s * aqr;
          A[(size_t)q * b + r] = s * apr + c * aqr;
        }
        A[(size_t)p * b + q] = A[(size_t)q * b + p] = 0.0;  // zero by construction of the rotation
        for (int r = 0; r < b; ++r) {
          const double zrp = Z[(size_t)r * b + p], zrq = Z[(size_t)r * b + q];
          Z[(size_t)r * b + p] = c * zrp - s * zrq;
          Z[(size_t)r * b + q] = s * zrp + c * zrq;
        }
      }
  }
  std::vector<int> ord((size_t)b);
  for (int i = 0; i < b; ++i) ord[i] = i;
  std::stable_sort(ord.begin(), ord.end(),
                   [&](int x, int y) { return A[(size_t)x * b + x] > A[(size_t)y * b + y]; });
  w.resize((size_t)b);
  std::vector<double> Zs((size_t)b * b);
  for (int c = 0; c < b; ++c) {
    w[c] = A[(size_t)ord[c] * b + ord[c]];
    for (int r = 0; r < b; ++r) Zs[(size_t)r * b + c] = Z[(size_t)r * b + ord[c]];
  }
  Z.swap(Zs);
}

// Upper-triangular R with G = R^T R (b x b, row-major), returned as R^{-1};
// false if a pivot is not positive (then the caller orthonormalises by the
// eigen-decomposition instead).
bool cholesky_inverse(const std::vector<double>& G, int b, std::vector<double>& Rinv) {
  std::vector<double> R((size_t)b * b, 0.0);
  for (int j = 0; j < b; ++j) {
    double dj = G[(size_t)j * b + j];
    for (int k = 0; k < j; ++k) dj -= R[(size_t)k * b + j] * R[(size_t)k * b + j];
    if (!(dj > 0.0) || !std::isfinite(dj)) return false;
    const double rjj = std::sqrt(dj);
    R[(size_t)j * b + j] = rjj;
    for (int i = j + 1; i < b; ++i) {
      double v = G[(size_t)j * b + i];
      for (int k = 0; k < j; ++k) v -= R[(size_t)k * b + j] * R[(size_t)k * b + i];
      R[(size_t)j * b + i] = v / rjj;
    }
  }
  // back substitution, column by column: R X = I
  Rinv.assign((size_t)b * b, 0.0);
  for (int c = 0; c < b; ++c)
    for (int i = c; i >= 0; --i) {
      double v = (i == c) ? 1.0 : 0.0;
      for (int k = i + 1; k <= c; ++k) v -= R[(size_t)i * b + k] * Rinv[(size_t)k * b + c];
      Rinv[(size_t)i * b + c] = v / R[(size_t)i * b + i];
    }
  return true;
}

// ---------------------------------------------------------------------------
// Subspace iteration driver
// ---------------------------------------------------------------------------
struct Csr {
  int64_t n = 0;
  uint64_t* rowptr = nullptr;
  int32_t* col = nullptr;
  double* val = nullptr;
};

stag_status build_normalised(int64_t n, const int64_t* src, const int64_t* dst, const double* w, int64_t E,
                             Workspace& ws, Csr* g, hipStream_t st) {
  const int64_t ne = 2 * E;
  uint32_t *keys = nullptr, *vals = nullptr, *sk = nullptr, *sv = nullptr;
  int* bad = nullptr;
  STAG_TRY(ws.alloc(&keys, (size_t)std::max<int64_t>(ne, 1)));
  STAG_TRY(ws.alloc(&vals, (size_t)std::max<int64_t>(ne, 1)));
  STAG_TRY(ws.alloc(&sk, (size_t)std::max<int64_t>(ne, 1)));
  STAG_TRY(ws.alloc(&sv, (size_t)std::max<int64_t>(ne, 1)));
  STAG_TRY(ws.alloc(&bad, 1));
  STAG_TRY(ws.alloc(&g->rowptr, (size_t)n + 1));
  STAG_TRY(ws.alloc(&g->col, (size_t)std::max<int64_t>(ne, 1)));
  STAG_TRY(ws.alloc(&g->val, (size_t)std::max<int64_t>(ne, 1)));
  double *deg = nullptr, *dinv = nullptr;
  STAG_TRY(ws.alloc(&deg, (size_t)n));
  STAG_TRY(ws.alloc(&dinv, (size_t)n));
  g->n = n;
  STAG_HIP(hipMemsetAsync(bad, 0, sizeof(int), st));
  ScopedTimer tm("graph_build", st);
  if (E > 0) {
    hipLaunchKernelGGL(edge_entries, dim3((unsigned)ceil_div(E, 256)), dim3(256), 0, st, src, dst, w, E, n, keys,
                       vals, bad);
    STAG_TRY(check_launch("edge_entries"));
  }
  int hbad = 0;
  STAG_HIP(hipMemcpyAsync(&hbad, bad, sizeof(int), hipMemcpyDeviceToHost, st));
  STAG_HIP(hipStreamSynchronize(st));
  if (hbad)
    return fail(STAG_E_INVAL, "graph: an edge has src or dst outside [0, n) (dst = -1 aside) or a negative or "
                              "non-finite weight");
  int key_bits = 1;
  while (key_bits < 32 && ((uint64_t)n >> key_bits) != 0) ++key_bits;
  if (ne > 0) STAG_TRY(radix_sort_pairs_u32(keys, vals, sk, sv, ne, key_bits, ws, st));
  hipLaunchKernelGGL(row_starts, dim3((unsigned)ceil_div(n + 1, 256)), dim3(256), 0, st, sk, ne, n, g->rowptr);
  STAG_TRY(check_launch("row_starts"));
  if (ne > 0) {
    hipLaunchKernelGGL(csr_fill, dim3((unsigned)ceil_div(ne, 256)), dim3(256), 0, st, sv, g->rowptr, n, ne, src, dst,
                       w, g->col, g->val);
    STAG_TRY(check_launch("csr_fill"));
  }
  hipLaunchKernelGGL(row_dinv, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, st, g->rowptr, g->val, n, deg, dinv);
  STAG_TRY(check_launch("row_dinv"));
  if (ne == 0) return STAG_OK;
  hipLaunchKernelGGL(normalise_vals, dim3((unsigned)ceil_div(ne, 256)), dim3(256), 0, st, g->rowptr, sk, g->col, dinv,
                     n, ne, g->val);
  return check_launch("normalise_vals");
}

class Subspace {
 public:
  Subspace(const Csr& g, int bp, int b, Workspace& ws, hipStream_t st) : g_(g), bp_(bp), b_(b), ws_(ws), st_(st) {}
  ~Subspace() {
    if (pinned_) {
      (void)hipStreamSynchronize(st_);
      (void)hipHostFree(pinned_);
    }
  }
  Subspace(const Subspace&) = delete;
  Subspace& operator=(const Subspace&) = delete;

  stag_status init() {
    // staging of the b x b uploads (matrix, Ritz values); the host rewrites
    // it only after a Gram read-back has synchronised the stream
    STAG_HIP(hipHostMalloc(reinterpret_cast<void**>(&pinned_), sizeof(double) * (kMaxBlockCols * kMaxBlockCols + kMaxBlockCols)));
    const size_t nb = (size_t)g_.n * bp_;
    for (double** p : {&V_, &W_, &Y0_, &Y1_, &T_}) STAG_TRY(ws_.alloc(p, nb));
    nblk_ = ceil_div(g_.n, kGramRows);
    STAG_TRY(ws_.alloc(&part_, (size_t)nblk_ * b_ * b_));
    STAG_TRY(ws_.alloc(&G_, (size_t)b_ * b_ + 1));
    broken_ = reinterpret_cast<int*>(G_ + (size_t)b_ * b_);
    STAG_TRY(ws_.alloc(&R_, (size_t)b_ * b_));
    STAG_TRY(ws_.alloc(&theta_, (size_t)kMaxBlockCols));
    return STAG_OK;
  }

  // Y = alpha M X + beta X + gamma Z
  stag_status spmm(const double* X, const double* Z, double* Y, double alpha, double beta, double gamma) {
    ScopedTimer tm("spectral_spmm", st_);
    const int lpr = bp_ / 2;
    const int64_t grid = ceil_div(g_.n, 256 / lpr);
    auto X2 = reinterpret_cast<const double2*>(X);
    auto Z2 = reinterpret_cast<const double2*>(Z);
    auto Y2 = reinterpret_cast<double2*>(Y);
    switch (lpr) {
      case 4:
        hipLaunchKernelGGL(spmm_comb<4>, dim3((unsigned)grid), dim3(256), 0, st_, g_.rowptr, g_.col, g_.val, g_.n, X2,
                           Z2, Y2, alpha, beta, gamma);
        break;
      case 8:
        hipLaunchKernelGGL(spmm_comb<8>, dim3((unsigned)grid), dim3(256), 0, st_, g_.rowptr, g_.col, g_.val, g_.n, X2,
                           Z2, Y2, alpha, beta, gamma);
        break;
      case 16:
        hipLaunchKernelGGL(spmm_comb<16>, dim3((unsigned)grid), dim3(256), 0, st_, g_.rowptr, g_.col, g_.val, g_.n, X2,
                           Z2, Y2, alpha, beta, gamma);
        break;
      default:
        hipLaunchKernelGGL(spmm_comb<32>, dim3((unsigned)grid), dim3(256), 0, st_, g_.rowptr, g_.col, g_.val, g_.n, X2,
                           Z2, Y2, alpha, beta, gamma);
    }
    return check_launch("spmm_comb");
  }

  // G_ <- A^T B (b x b)
  stag_status gram_dev(const double* A, const double* B) {
    ScopedTimer tm("spectral_gram", st_);
    hipLaunchKernelGGL(gram_partial, dim3((unsigned)nblk_), dim3(256), 0, st_, A, B, g_.n, bp_, b_, part_);
    STAG_TRY(check_launch("gram_partial"));
    return sum_parts(b_ * b_);
  }

  // G_[e] <- sum of the nblk_ partials, e < count
  stag_status sum_parts(int count) {
    hipLaunchKernelGGL(gram_final, dim3((unsigned)ceil_div(count, kFinalCols)), dim3(256), 0, st_, part_, nblk_, count,
                       G_);
    return check_launch("gram_final");
  }

  // host <- the first count doubles of G_
  stag_status read_back(size_t count, std::vector<double>& out) {
    out.resize(count);
    STAG_HIP(hipMemcpyAsync(out.data(), G_, sizeof(double) * count, hipMemcpyDeviceToHost, st_));
    STAG_HIP(hipStreamSynchronize(st_));
    return STAG_OK;
  }

  // host <- A^T B (b x b)
  stag_status gram(const double* A, const double* B, std::vector<double>& out) {
    STAG_TRY(gram_dev(A, B));
    return read_back((size_t)b_ * b_, out);
  }

  // device R <- host R (b x b), through the pinned staging buffer
  stag_status upload(const std::vector<double>& R) {
    std::copy(R.begin(), R.end(), pinned_);
    STAG_HIP(hipMemcpyAsync(R_, pinned_, sizeof(double) * R.size(), hipMemcpyHostToDevice, st_));
    return STAG_OK;
  }

  // Y = X R with the R on the device; nothing if *broken
  stag_status apply(const double* X, double* Y, const int* broken = nullptr) {
    ScopedTimer tm("spectral_apply", st_);
    hipLaunchKernelGGL(apply_small, dim3((unsigned)ceil_div(g_.n, 256 / bp_ * kApplyRows)), dim3(256), 0, st_, X, g_.n,
                       bp_, b_, R_, broken, Y);
    return check_launch("apply_small");
  }

  // Twice: V <- V R^{-1} from the Cholesky factor of V^T V (Cholesky QR).  A
  // factor that breaks down sets the flag behind G_'s matrix, whose copy comes
  // back with the next Gram matrix that the host reads; V_ is then untouched
  // (its two applications did nothing), and orthonormalise() has to run.
  stag_status orthonormalise_dev() {
    hipLaunchKernelGGL(fill_i32, dim3(1), dim3(64), 0, st_, broken_, (int64_t)2, 0);
    STAG_TRY(check_launch("fill_i32"));
    for (int pass = 0; pass < 2; ++pass) {
      STAG_TRY(gram_dev(V_, V_));
      hipLaunchKernelGGL(chol_inverse, dim3(1), dim3(1024), 0, st_, G_, b_, R_, broken_);
      STAG_TRY(check_launch("chol_inverse"));
      STAG_TRY(apply(V_, T_, broken_));
      std::swap(V_, T_);
    }
    return STAG_OK;
  }

  // The same with the host's factor or, if that breaks down, V <- V Q L^{-1/2}
  // from its eigen-decomposition.
  stag_status orthonormalise() {
    for (int pass = 0; pass < 2; ++pass) {
      std::vector<double> G, R;
      STAG_TRY(gram(V_, V_, G));
      if (!cholesky_inverse(G, b_, R)) {
        std::vector<double> lam, Q;
        jacobi_eigen(G, b_, lam, Q);
        const double floor_ = std::max(lam[0], 1e-300) * 1e-30;
        R.assign((size_t)b_ * b_, 0.0);
        for (int c = 0; c < b_; ++c) {
          const double sc = 1.0 / std::sqrt(std::max(lam[c], floor_));
          for (int r = 0; r < b_; ++r) R[(size_t)r * b_ + c] = Q[(size_t)r * b_ + c] * sc;
        }
      }
      STAG_TRY(upload(R));
      STAG_TRY(apply(V_, T_));
      std::swap(V_, T_);
    }
    return STAG_OK;
  }

  // V orthonormalised, W = M V, H = V^T W = Z theta Z^T, V <- V Z, W <- W Z.
  stag_status rayleigh_ritz() {
    std::vector<double> H, Z;
    STAG_TRY(orthonormalise_dev());
    for (int attempt = 0;; ++attempt) {
      STAG_TRY(spmm(V_, nullptr, W_, 1.0, 0.0, 0.0));
      STAG_TRY(gram_dev(V_, W_));
      STAG_TRY(read_back((size_t)b_ * b_ + 1, H));
      int broken[2];
      std::memcpy(broken, &H.back(), sizeof(broken));
      H.pop_back();
      if (!broken[0] || attempt) break;
      STAG_TRY(orthonormalise());
    }
    for (int i = 0; i < b_; ++i)  // symmetrise the rounding
      for (int j = i + 1; j < b_; ++j) {
        const double m = 0.5 * (H[(size_t)i * b_ + j] + H[(size_t)j * b_ + i]);
        H[(size_t)i * b_ + j] = H[(size_t)j * b_ + i] = m;
      }
    jacobi_eigen(H, b_, theta_h_, Z);
    STAG_TRY(upload(Z));
    STAG_TRY(apply(V_, T_));
    std::swap(V_, T_);
    STAG_TRY(apply(W_, T_));
    std::swap(W_, T_);
    double* th = pinned_ + kMaxBlockCols * kMaxBlockCols;
    std::copy(theta_h_.begin(), theta_h_.end(), th);
    STAG_HIP(hipMemcpyAsync(theta_, th, sizeof(double) * b_, hipMemcpyHostToDevice, st_));
    return STAG_OK;
  }

  // Largest residual norm over the first k Ritz pairs.
  stag_status max_residual(int k, double* out) {
    hipLaunchKernelGGL(residual_norms, dim3((unsigned)nblk_), dim3(256), 0, st_, W_, V_, theta_, g_.n, bp_, b_, part_);
    STAG_TRY(check_launch("residual_norms"));
    STAG_TRY(sum_parts(b_));
    std::vector<double> G;
    STAG_TRY(read_back((size_t)b_, G));
    double m = 0.0;
    for (int j = 0; j < k; ++j) m = std::max(m, std::sqrt(std::max(G[(size_t)j], 0.0)));
    *out = m;
    return STAG_OK;
  }

  // V <- T_p((M - c)/e) V by the three-term recurrence
  //   Y_0 = V, Y_1 = (M - c) V / e, Y_{j+1} = 2 (M - c) Y_j / e - Y_{j-1},
  // rotating three buffers (V_, Y1_, Y0_); the result becomes V_.
  stag_status filter(int p, double lo, double hi) {
    const double e = 0.5 * (hi - lo), c = 0.5 * (hi + lo);
    double* buf[3] = {V_, Y1_, Y0_};  // Y_{j-1}, Y_j, spare
    STAG_TRY(spmm(buf[0], nullptr, buf[1], 1.0 / e, -c / e, 0.0));
    for (int j = 2; j <= p; ++j) {
      STAG_TRY(spmm(buf[1], buf[0], buf[2], 2.0 / e, -2.0 * c / e, -1.0));
      double* t = buf[0];
      buf[0] = buf[1];
      buf[1] = buf[2];
      buf[2] = t;
    }
    V_ = buf[1];
    Y1_ = buf[0];
    Y0_ = buf[2];
    return STAG_OK;
  }

  stag_status run(int k, double tol, int max_iter, uint64_t seed, int* iters) {
    hipLaunchKernelGGL(init_block, dim3((unsigned)ceil_div(g_.n * bp_, 256)), dim3(256), 0, st_, V_, g_.n, bp_, b_,
                       seed);
    STAG_TRY(check_launch("init_block"));
    STAG_TRY(rayleigh_ritz());
    int it = 0;
    for (;;) {
      double res = 0.0;
      STAG_TRY(max_residual(k, &res));
      if (res <= tol || it >= max_iter) break;
      ++it;
      const double cut = std::min(theta_h_[b_ - 1], 1.0 - 1e-12);
      const double lo = -1.0;
      const double e = 0.5 * (cut - lo), c = 0.5 * (cut + lo);
      const double xt = (1.0 - c) / e;  // image of the spectrum's top
      int p = 30;
      if (xt > 1.0) p = (int)std::floor(std::acosh(1e6) / std::acosh(xt));
      p = std::max(2, std::min(30, p));
      STAG_TRY(filter(p, lo, cut));
      STAG_TRY(rayleigh_ritz());
    }
    *iters = it;
    return STAG_OK;
  }

  const double* V() const { return V_; }
  const double* theta() const { return theta_; }

 private:
  const Csr& g_;
  int bp_, b_;
  Workspace& ws_;
  hipStream_t st_;
  int64_t nblk_ = 0;
  double *V_ = nullptr, *W_ = nullptr, *Y0_ = nullptr, *Y1_ = nullptr, *T_ = nullptr;
  double *part_ = nullptr, *G_ = nullptr, *R_ = nullptr, *theta_ = nullptr;
  int* broken_ = nullptr;  // behind G_'s b_ x b_ matrix
  double* pinned_ = nullptr;
  std::vector<double> theta_h_;
};

// ---------------------------------------------------------------------------
// k-means kernels (fp64; distances and sums without fused operations)
// ---------------------------------------------------------------------------
__device__ inline double dist2_rn(const double* p, const double* c, int dim) {
  double s = 0.0;
  for (int j = 0; j < dim; ++j) {
    const double t = __dsub_rn(p[j], c[j]);
    s = __dadd_rn(s, __dmul_rn(t, t));
  }
  return s;
}

// D2[i] = min(D2[i], dist2(P_i, centre)) (first = 1 initialises D2) and S[b] =
// the sequential sum of D2 over block b: one workgroup per block, the values
// staged in LDS, then added in order by one thread.
__global__ __launch_bounds__(256) void km_d2_sums(const double* __restrict__ P, int64_t n, int dim,
                                                  const double* __restrict__ centre, int first,
                                                  double* __restrict__ D2, double* __restrict__ S) {
  __shared__ double v[kKmBlock];
  const int64_t base = (int64_t)blockIdx.x * kKmBlock;
  const int cnt = (int)min((int64_t)kKmBlock, n - base);
  for (int i = threadIdx.x; i < kKmBlock; i += 256) {
    double m = 0.0;
    if (i < cnt) {
      const double d = dist2_rn(P + (base + i) * dim, centre, dim);
      m = first ? d : fmin(D2[base + i], d);
      D2[base + i] = m;
    }
    v[i] = m;  // adding 0 past the end changes nothing
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  double s = 0.0;
  for (int i = 0; i < kKmBlock; i += 16) {
#pragma unroll
    for (int u = 0; u < 16; ++u) s = __dadd_rn(s, v[i + u]);
  }
  S[blockIdx.x] = s;
}

// Picks centre c (c == 0: uniform; else D^2 sampling in the blocked order,
// with the documented fallbacks) and copies its row to C.  One workgroup: all
// threads bring up to 1024 values to LDS, one thread turns them into running
// sums in order, all look for the first past the threshold.  At 1e5 points one
// thread that read, added and compared took 46 us a centre; now 20.
__global__ __launch_bounds__(256) void km_pick(const double* __restrict__ P, int64_t n, int dim,
                                               const double* __restrict__ D2, const double* __restrict__ S, int64_t nb,
                                               uint64_t seed, int c, unsigned char* chosen, double* __restrict__ C,
                                               int64_t* __restrict__ seeds) {
  __shared__ double v[kKmBlock];
  __shared__ int at;        // first running sum past the threshold
  __shared__ int64_t got;   // the point picked
  const int tid = threadIdx.x;
  const uint64_t u = stream_bits(seed, kTagKmeans, (uint64_t)c) >> 11;
  // v[i] = start + src[0] + .. + src[i], i < cnt, added from the left
  auto running = [&](const double* src, int cnt, double start) {
    __syncthreads();
    for (int i = tid; i < kKmBlock; i += 256) v[i] = i < cnt ? src[i] : 0.0;
    if (tid == 0) at = kKmBlock;
    __syncthreads();
    if (tid == 0) {
      double s = start;
      for (int i = 0; i < cnt; i += 16) {
        double t[16];
#pragma unroll
        for (int w = 0; w < 16; ++w) t[w] = v[i + w];
#pragma unroll
        for (int w = 0; w < 16; ++w) v[i + w] = s = __dadd_rn(s, t[w]);
      }
    }
    __syncthreads();
  };
  // the first i < cnt with before + v[i] > t, or kKmBlock
  auto first = [&](int cnt, double before, double t) {
    for (int i = tid; i < cnt; i += 256)
      if (__dadd_rn(before, v[i]) > t) {
        atomicMin(&at, i);
        break;
      }
    __syncthreads();
    return at;
  };
  if (tid == 0) got = -1;
  if (c == 0) {
    const uint64_t hi = __umul64hi(u, (uint64_t)n), lo = u * (uint64_t)n;
    if (tid == 0) got = (int64_t)((hi << 11) | (lo >> 53));
  } else {
    double T = 0.0;
    for (int64_t b0 = 0; b0 < nb; b0 += kKmBlock) {
      const int cnt = (int)min((int64_t)kKmBlock, nb - b0);
      running(S + b0, cnt, T);
      T = v[cnt - 1];
    }
    if (T > 0.0) {
      const double t = __dmul_rn((double)u * 0x1.0p-53, T);
      double B = 0.0;  // sum of the blocks before b
      bool found = false;
      for (int64_t b = 0; b < nb && !found;) {
        int cnt = (int)min((int64_t)kKmBlock, nb - b);
        running(S + b, cnt, B);
        const int f = first(cnt, 0.0, t);
        if (f == kKmBlock) {  // none of these blocks passes t
          B = v[cnt - 1];
          b += cnt;
          continue;
        }
        const double before = f > 0 ? v[f - 1] : B;
        B = v[f];
        b += f;
        cnt = (int)min((int64_t)kKmBlock, n - b * kKmBlock);
        running(D2 + b * kKmBlock, cnt, 0.0);
        const int i = first(cnt, before, t);
        if (i < kKmBlock) {
          if (tid == 0) got = b * kKmBlock + i;
          found = true;
        }
        ++b;
      }
      __syncthreads();
      if (tid == 0)
        for (int64_t i = n - 1; i >= 0 && got < 0; --i)
          if (D2[i] > 0.0) got = i;
    } else if (tid == 0) {
      for (int64_t i = 0; i < n && got < 0; ++i)
        if (!chosen[i]) got = i;
    }
  }
  if (tid == 0) {
    if (got < 0) got = 0;  // unreachable for finite inputs
    chosen[got] = 1;
    if (seeds) seeds[c] = got;
  }
  __syncthreads();
  for (int j = tid; j < dim; j += 256) C[(int64_t)c * dim + j] = P[got * dim + j];
}

// label = argmin over centres (ties to the lowest); *changed |= any change.
// DIM > 0: dim <= DIM, the point in registers and the centres zero-padded to
// DIM in LDS (a padding coordinate adds 0); otherwise both read as they are.
// With the point read from memory again for every centre, 1e5 points of 20
// coordinates and 20 centres took 58 us; now 21.
template <int DIM>
__global__ __launch_bounds__(256) void km_assign(const double* __restrict__ P, int64_t n, int dim,
                                                 const double* __restrict__ C, int k, int32_t* __restrict__ labels,
                                                 int* __restrict__ changed) {
  extern __shared__ double sC[];
  const int ld = DIM > 0 ? DIM : dim;
  for (int v = threadIdx.x; v < k * ld; v += blockDim.x) {
    const int c = v / ld, j = v % ld;
    sC[v] = j < dim ? C[c * dim + j] : 0.0;
  }
  __syncthreads();
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double* p = P + i * dim;
  double x[DIM > 0 ? DIM : 1];
  if constexpr (DIM > 0) {
#pragma unroll
    for (int j = 0; j < DIM; ++j) x[j] = j < dim ? p[j] : 0.0;
  }
  int best = 0;
  double bd = 0.0;
  for (int c = 0; c < k; ++c) {
    double dc;
    if constexpr (DIM > 0) {
      dc = 0.0;
#pragma unroll
      for (int j = 0; j < DIM; ++j) {
        const double t = __dsub_rn(x[j], sC[c * DIM + j]);
        dc = __dadd_rn(dc, __dmul_rn(t, t));
      }
    } else {
      dc = dist2_rn(p, sC + c * dim, dim);
    }
    if (c == 0 || dc < bd) {
      bd = dc;
      best = c;
    }
  }
  if (labels[i] != best) {
    labels[i] = best;
    atomicOr(changed, 1);
  }
}

// Per block of 1024 points: coordinate sums per cluster, points in order
// (lane j owns coordinate j of every cluster), and counts.
__global__ __launch_bounds__(64) void km_block_accum(const double* __restrict__ P, const int32_t* __restrict__ labels,
                                                     int64_t n, int dim, int k, double* __restrict__ part,
                                                     int64_t* __restrict__ cnt) {
  extern __shared__ double acc[];  // [k][dim]
  const int lane = threadIdx.x;
  for (int v = lane; v < k * dim; v += 64) acc[v] = 0.0;
  __syncthreads();
  const int64_t b = blockIdx.x;
  const int64_t e = min(n, (b + 1) * (int64_t)kKmBlock);
  for (int64_t i = b * kKmBlock; i < e; ++i) {
    const int l = labels[i];
    for (int j = lane; j < dim; j += 64) acc[l * dim + j] = __dadd_rn(acc[l * dim + j], P[i * dim + j]);
  }
  __syncthreads();
  for (int v = lane; v < k * dim; v += 64) part[b * k * dim + v] = acc[v];
  if (lane == 0) {
    for (int c = 0; c < k; ++c) cnt[b * k + c] = 0;
    for (int64_t i = b * kKmBlock; i < e; ++i) cnt[b * k + labels[i]] += 1;
  }
}

// The same sums for k <= 256 (8-bit labels): the block's points are listed by
// cluster (stable: ballot ranks within a wave, counts across waves), then each
// thread adds one (cluster, coordinate) over its cluster's points in order, so
// that the chains of a block run side by side: 1e5 points of 20 coordinates
// in 20 clusters 419 -> 12 us.
constexpr int kKmListMax = 256;
__global__ __launch_bounds__(1024) void km_list_accum(const double* __restrict__ P,
                                                      const int32_t* __restrict__ labels, int64_t n, int dim, int k,
                                                      double* __restrict__ part, int64_t* __restrict__ cnt) {
  __shared__ uint16_t wcount[16][kKmListMax];
  __shared__ uint32_t start[kKmListMax + 1];
  __shared__ uint16_t list[kKmBlock];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t b = blockIdx.x, base = b * kKmBlock;
  const bool valid = base + tid < n;
  const uint32_t key = valid ? (uint32_t)labels[base + tid] : 0u;
  for (int v = tid; v < 16 * kKmListMax; v += 1024) wcount[v / kKmListMax][v % kKmListMax] = 0;
  __syncthreads();
  uint64_t peers = __ballot(valid);
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const bool bit = (key >> q) & 1u;
    const uint64_t ones = __ballot(bit);
    peers &= bit ? ones : ~ones;
  }
  const uint32_t rank = (uint32_t)__popcll(peers & ((1ull << lane) - 1ull));
  if (valid && rank == 0) wcount[wave][key] = (uint16_t)__popcll(peers);
  __syncthreads();
  if (tid < kKmListMax) {
    uint32_t t = 0;
    for (int w = 0; w < 16; ++w) t += wcount[w][tid];
    start[tid + 1] = t;
    if (tid == 0) start[0] = 0;
    if (tid < k) cnt[b * k + tid] = (int64_t)t;
  }
  __syncthreads();
  if (wave == 0) {  // lane l: totals 4 l .. 4 l + 3
    uint32_t t[4], s = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) t[q] = s += start[4 * lane + q + 1];
    uint32_t before = s;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t v = __shfl_up(before, o);
      if (lane >= o) before += v;
    }
    before -= s;
#pragma unroll
    for (int q = 0; q < 4; ++q) start[4 * lane + q + 1] = before + t[q];
  }
  __syncthreads();
  if (valid) {
    uint32_t at = start[key] + rank;
    for (int w = 0; w < wave; ++w) at += wcount[w][key];
    list[at] = (uint16_t)tid;
  }
  __syncthreads();
  for (int v = tid; v < k * dim; v += 1024) {
    const int c = v / dim, j = v % dim;
    const uint32_t e = start[c + 1];
    const double* col = P + base * dim + j;
    double s = 0.0;
    uint32_t i = start[c];
    for (; i + 8 <= e; i += 8) {
      double t[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) t[q] = col[(int64_t)list[i + q] * dim];
#pragma unroll
      for (int q = 0; q < 8; ++q) s = __dadd_rn(s, t[q]);
    }
    for (; i < e; ++i) s = __dadd_rn(s, col[(int64_t)list[i] * dim]);
    part[b * k * dim + v] = s;
  }
}

__global__ void km_update(const double* __restrict__ part, const int64_t* __restrict__ cnt, int64_t nb, int dim, int k,
                          double* __restrict__ C) {
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= k * dim) return;
  const int c = v / dim;
  double s = 0.0;
  int64_t m = 0;
  int64_t b = 0;
  for (; b + 8 <= nb; b += 8) {
    double t[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      t[u] = part[(b + u) * k * dim + v];
      m += cnt[(b + u) * k + c];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) s = __dadd_rn(s, t[u]);
  }
  for (; b < nb; ++b) {
    s = __dadd_rn(s, part[b * k * dim + v]);
    m += cnt[b * k + c];
  }
  if (m > 0) C[v] = __ddiv_rn(s, (double)m);
}

stag_status kmeans_impl(const double* P, int64_t n, int dim, int k, uint64_t seed, int max_iter, const double* init,
                        int32_t* labels, double* C_out, int64_t* seeds, int* iters, Workspace& ws, hipStream_t st) {
  const int64_t nb = ceil_div(n, kKmBlock);
  double *C = nullptr, *D2 = nullptr, *S = nullptr, *part = nullptr;
  int64_t* cnt = nullptr;
  int* changed = nullptr;
  unsigned char* chosen = nullptr;
  STAG_TRY(ws.alloc(&C, (size_t)k * dim));
  STAG_TRY(ws.alloc(&part, (size_t)nb * k * dim));
  STAG_TRY(ws.alloc(&cnt, (size_t)nb * k));
  STAG_TRY(ws.alloc(&changed, 1));
  ScopedTimer tm("kmeans", st);
  if (init) {
    STAG_HIP(hipMemcpyAsync(C, init, sizeof(double) * (size_t)k * dim, hipMemcpyDeviceToDevice, st));
    if (seeds) {
      std::vector<int64_t> neg((size_t)k, -1);
      STAG_HIP(hipMemcpyAsync(seeds, neg.data(), sizeof(int64_t) * (size_t)k, hipMemcpyHostToDevice, st));
      STAG_HIP(hipStreamSynchronize(st));
    }
  } else {
    STAG_TRY(ws.alloc(&D2, (size_t)n));
    STAG_TRY(ws.alloc(&S, (size_t)nb));
    STAG_TRY(ws.alloc(&chosen, (size_t)n));
    STAG_HIP(hipMemsetAsync(chosen, 0, (size_t)n, st));
    for (int c = 0; c < k; ++c) {
      if (c > 0) {
        hipLaunchKernelGGL(km_d2_sums, dim3((unsigned)nb), dim3(256), 0, st, P, n, dim, C + (int64_t)(c - 1) * dim,
                           c == 1 ? 1 : 0, D2, S);
        STAG_TRY(check_launch("km_d2_sums"));
      }
      hipLaunchKernelGGL(km_pick, dim3(1), dim3(256), 0, st, P, n, dim, D2, S, nb, seed, c, chosen, C, seeds);
      STAG_TRY(check_launch("km_pick"));
    }
  }
  hipLaunchKernelGGL(fill_i32, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, st, labels, n, -1);
  STAG_TRY(check_launch("fill_i32"));
  const size_t lds_c = sizeof(double) * (size_t)k * dim;
  int it = 0;
  while (it < max_iter) {
    ++it;
    STAG_HIP(hipMemsetAsync(changed, 0, sizeof(int), st));
    auto assign = [&](auto kern, int ld) {
      hipLaunchKernelGGL(kern, dim3((unsigned)ceil_div(n, 256)), dim3(256), sizeof(double) * (size_t)k * ld, st, P, n,
                         dim, C, k, labels, changed);
    };
    // k dim <= 4096: the padded centres take at most 58 KB
    if (dim <= 1) assign(km_assign<1>, 1);
    else if (dim <= 2) assign(km_assign<2>, 2);
    else if (dim <= 4) assign(km_assign<4>, 4);
    else if (dim <= 8) assign(km_assign<8>, 8);
    else if (dim <= 16) assign(km_assign<16>, 16);
    else if (dim <= 24) assign(km_assign<24>, 24);
    else if (dim <= 32) assign(km_assign<32>, 32);
    else if (dim <= 48) assign(km_assign<48>, 48);
    else if (dim <= 64) assign(km_assign<64>, 64);
    else assign(km_assign<0>, dim);
    STAG_TRY(check_launch("km_assign"));
    int h = 0;
    STAG_HIP(hipMemcpyAsync(&h, changed, sizeof(int), hipMemcpyDeviceToHost, st));
    STAG_HIP(hipStreamSynchronize(st));
    if (!h) break;
    if (k <= kKmListMax)
      hipLaunchKernelGGL(km_list_accum, dim3((unsigned)nb), dim3(1024), 0, st, P, labels, n, dim, k, part, cnt);
    else
      hipLaunchKernelGGL(km_block_accum, dim3((unsigned)nb), dim3(64), lds_c, st, P, labels, n, dim, k, part, cnt);
    STAG_TRY(check_launch("km_block_accum"));
    hipLaunchKernelGGL(km_update, dim3((unsigned)ceil_div(k * dim, 256)), dim3(256), 0, st, part, cnt, nb, dim, k, C);
    STAG_TRY(check_launch("km_update"));
  }
  if (C_out) STAG_HIP(hipMemcpyAsync(C_out, C, sizeof(double) * (size_t)k * dim, hipMemcpyDeviceToDevice, st));
  STAG_HIP(hipStreamSynchronize(st));
  if (iters) *iters = it;
  return STAG_OK;
}

int block_cols(int k) {
  int bp = 8;
  while (bp < k + 8) bp *= 2;
  return bp;
}

stag_status check_graph_args(const char* fn, int64_t n, const int64_t* src, const int64_t* dst, const double* w,
                             int64_t E, int32_t k) {
  if (n < 1 || n >= ((int64_t)1 << 31)) return fail(STAG_E_INVAL, "%s: n must be in [1, 2^31)", fn);
  if (E < 0 || E >= ((int64_t)1 << 30)) return fail(STAG_E_INVAL, "%s: n_edges must be in [0, 2^30)", fn);
  if (E > 0 && (!src || !dst || !w)) return fail(STAG_E_INVAL, "%s: NULL edge array", fn);
  if (k < 1 || k > 56 || k > n) return fail(STAG_E_INVAL, "%s: k must be in [1, min(56, n)]", fn);
  return STAG_OK;
}

stag_status embedding_impl(int64_t n, const int64_t* src, const int64_t* dst, const double* w, int64_t E, int32_t k,
                           double tol, int32_t max_iter, uint64_t seed, double* lam_out, double* U_out,
                           int32_t* iters_out, Workspace& ws, hipStream_t st) {
  Csr g;
  STAG_TRY(build_normalised(n, src, dst, w, E, ws, &g, st));
  const int bp = block_cols(k);
  const int b = (int)std::min<int64_t>(n, bp);
  Subspace sub(g, bp, b, ws, st);
  STAG_TRY(sub.init());
  int it = 0;
  STAG_TRY(sub.run(k, tol, max_iter, seed, &it));
  // signs, embedding, eigenvalues
  const int64_t nblk = ceil_div(n, 256);
  double *pv = nullptr, *sign = nullptr;
  int64_t* pi = nullptr;
  STAG_TRY(ws.alloc(&pv, (size_t)nblk * k));
  STAG_TRY(ws.alloc(&pi, (size_t)nblk * k));
  STAG_TRY(ws.alloc(&sign, (size_t)k));
  hipLaunchKernelGGL(col_absmax_partial, dim3((unsigned)nblk), dim3(256), 0, st, sub.V(), n, bp, k, pv, pi);
  STAG_TRY(check_launch("col_absmax_partial"));
  hipLaunchKernelGGL(col_sign, dim3((unsigned)k), dim3(256), 0, st, pv, pi, nblk, sub.V(), bp, k, sign);
  STAG_TRY(check_launch("col_sign"));
  hipLaunchKernelGGL(extract_embedding, dim3((unsigned)ceil_div(n * k, 256)), dim3(256), 0, st, sub.V(), n, bp, k,
                     sign, U_out);
  STAG_TRY(check_launch("extract_embedding"));
  if (lam_out) {
    hipLaunchKernelGGL(eig_out, dim3(1), dim3(64), 0, st, sub.theta(), k, lam_out);
    STAG_TRY(check_launch("eig_out"));
  }
  STAG_HIP(hipStreamSynchronize(st));
  if (iters_out) *iters_out = it;
  return STAG_OK;
}

}  // namespace
}  // namespace stag

extern "C" stag_status stag_spectral_embedding(int64_t n, const int64_t* src, const int64_t* dst, const double* w,
                                               int64_t n_edges, int32_t k, double tol, int32_t max_iter,
                                               uint64_t seed, double* eigvals_out, double* U_out, int32_t* iters_out,
                                               hipStream_t stream) {
  using namespace stag;
  STAG_TRY(check_graph_args("stag_spectral_embedding", n, src, dst, w, n_edges, k));
  if (!U_out) return fail(STAG_E_INVAL, "stag_spectral_embedding: NULL U_out");
  if (!(tol > 0.0) || max_iter < 0) return fail(STAG_E_INVAL, "stag_spectral_embedding: tol > 0, max_iter >= 0");
  clear_error();
  Workspace ws(stream);
  return embedding_impl(n, src, dst, w, n_edges, k, tol, max_iter, seed, eigvals_out, U_out, iters_out, ws, stream);
}

extern "C" stag_status stag_kmeans(const double* P, int64_t n, int32_t dim, int32_t k, uint64_t seed,
                                   int32_t max_iter, const double* init, int32_t* labels_out, double* centroids_out,
                                   int64_t* seeds_out, int32_t* iters_out, hipStream_t stream) {
  using namespace stag;
  if (!P || !labels_out) return fail(STAG_E_INVAL, "stag_kmeans: NULL pointer argument");
  if (n < 1 || n >= ((int64_t)1 << 31) || dim < 1 || k < 1 || k > n || max_iter < 1)
    return fail(STAG_E_INVAL, "stag_kmeans: need 1 <= k <= n < 2^31, dim >= 1, max_iter >= 1");
  if ((int64_t)k * dim > 4096) return fail(STAG_E_UNSUPPORTED, "stag_kmeans: k * dim must be <= 4096");
  clear_error();
  Workspace ws(stream);
  int it = 0;
  STAG_TRY(kmeans_impl(P, n, dim, k, seed, max_iter, init, labels_out, centroids_out, seeds_out, &it, ws, stream));
  if (iters_out) *iters_out = it;
  return STAG_OK;
}

extern "C" stag_status stag_spectral_cluster(int64_t n, const int64_t* src, const int64_t* dst, const double* w,
                                             int64_t n_edges, int32_t k, uint64_t seed, int32_t* labels_out,
                                             hipStream_t stream) {
  using namespace stag;
  STAG_TRY(check_graph_args("stag_spectral_cluster", n, src, dst, w, n_edges, k));
  if (!labels_out) return fail(STAG_E_INVAL, "stag_spectral_cluster: NULL labels_out");
  clear_error();
  Workspace ws(stream);
  double* U = nullptr;
  STAG_TRY(ws.alloc(&U, (size_t)n * k));
  STAG_TRY(embedding_impl(n, src, dst, w, n_edges, k, 1e-8, 300, seed, nullptr, U, nullptr, ws, stream));
  int it = 0;
  return kmeans_impl(U, n, k, k, seed, 300, nullptr, labels_out, nullptr, nullptr, &it, ws, stream);
}
