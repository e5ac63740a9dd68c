// Exclusive prefix sum: a scan per block of 1024 with block totals, then every
// block adds the totals before it, which it sums itself (up to kScanDirect
// blocks), or whose scan it reads (more).  The scans of these calls are short
// (1e5 to 1e6 elements), so launches are what they cost: the totals' own scan,
// its grand total and the sum's were five launches, about 25 us, now two.
#include "scan.h"

namespace stag {
namespace {

constexpr int kScanBlock = 1024;  // elements per block (4 per thread)

__device__ inline uint64_t wave_incl_scan(uint64_t v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint64_t u = __shfl_up(v, o);
    if (lane >= o) v += u;
  }
  return v;
}

// Block-level exclusive scan of 1024 values (4 per thread); returns the
// block total through *total.
template <typename T>
__device__ inline void block_scan4(const T* vin, uint64_t* vout, uint64_t* total) {
  __shared__ uint64_t wsum[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint64_t loc[4], run = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    loc[k] = run;
    run += (uint64_t)vin[k];
  }
  const uint64_t incl = wave_incl_scan(run);
  if (lane == 63) wsum[wave] = incl;
  __syncthreads();
  uint64_t wbase = 0;
  for (int w = 0; w < wave; ++w) wbase += wsum[w];
  const uint64_t base = wbase + incl - run;
#pragma unroll
  for (int k = 0; k < 4; ++k) vout[k] = base + loc[k];
  *total = wsum[0] + wsum[1] + wsum[2] + wsum[3];
}

template <typename T>
__global__ __launch_bounds__(256) void scan_blocks(const T* __restrict__ in, int64_t n, uint64_t* __restrict__ out,
                                                   uint64_t* __restrict__ block_tot) {
  const int64_t base = (int64_t)blockIdx.x * kScanBlock + threadIdx.x * 4;
  T v[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = base + k < n ? in[base + k] : (T)0;
  uint64_t o[4], tot;
  block_scan4<T>(v, o, &tot);
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (base + k < n) out[base + k] = o[k];
  if (threadIdx.x == 0) {
    if (gridDim.x == 1) out[n] = tot;
    else block_tot[blockIdx.x] = tot;
  }
}

// out[i] += totals of the blocks before i's, out[n] = the grand total.  Block b
// reads b totals: at most kScanDirect / 2 x 8 bytes on average, from the cache.
constexpr int64_t kScanDirect = 4096;
__global__ __launch_bounds__(256) void add_totals(uint64_t* __restrict__ out, int64_t n,
                                                  const uint64_t* __restrict__ block_tot) {
  __shared__ uint64_t wsum[4];
  const int tid = threadIdx.x;
  uint64_t s = 0;
  for (int64_t j = tid; j < blockIdx.x; j += 256) s += block_tot[j];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if ((tid & 63) == 0) wsum[tid >> 6] = s;
  __syncthreads();
  s = wsum[0] + wsum[1] + wsum[2] + wsum[3];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int64_t i = (int64_t)blockIdx.x * kScanBlock + 256 * k + tid;
    if (i < n) out[i] += s;
  }
  if (tid == 0 && blockIdx.x == gridDim.x - 1) out[n] = s + block_tot[blockIdx.x];
}

__global__ void add_offsets(uint64_t* __restrict__ out, int64_t n, const uint64_t* __restrict__ block_off) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] += block_off[i / kScanBlock];
  if (i == n) out[n] = block_off[(n + kScanBlock - 1) / kScanBlock];
}

template <typename T>
stag_status scan_impl(const T* in, uint64_t* out, int64_t n, Workspace& ws, hipStream_t st) {
  const int64_t nb = ceil_div(n, kScanBlock);
  uint64_t* tot = nullptr;
  STAG_TRY(ws.alloc(&tot, (size_t)nb));
  hipLaunchKernelGGL(scan_blocks<T>, dim3((unsigned)nb), dim3(256), 0, st, in, n, out, tot);
  STAG_TRY(check_launch("scan_blocks"));
  if (nb == 1) return STAG_OK;
  if (nb <= kScanDirect) {
    hipLaunchKernelGGL(add_totals, dim3((unsigned)nb), dim3(256), 0, st, out, n, tot);
    return check_launch("add_totals");
  }
  uint64_t* off = nullptr;
  STAG_TRY(ws.alloc(&off, (size_t)nb + 1));
  STAG_TRY(scan_impl<uint64_t>(tot, off, nb, ws, st));
  hipLaunchKernelGGL(add_offsets, dim3((unsigned)ceil_div(n + 1, 256)), dim3(256), 0, st, out, n, off);
  return check_launch("add_offsets");
}

}  // namespace

stag_status exclusive_scan_u32(const uint32_t* in, uint64_t* out, int64_t n, Workspace& ws, hipStream_t st) {
  return scan_impl<uint32_t>(in, out, n, ws, st);
}

}  // namespace stag
