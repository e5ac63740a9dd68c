// Dense levels of the CKNS walks (internal; part of lsh.hip).
//
// The per-query walk reads the row of every candidate of every query, lane by
// lane, from the caches.  Where a level's buckets hold a good part of its
// members for most queries, the same distances are a dense (queries x
// members) problem: dense_pairs takes 128 x 128 pairs per workgroup, finds by
// their keys the first table in which each pair meets, and forms the fp64
// distances of the tile with every row staged once in LDS and an 8 x 4 block
// of chains per thread.  dense_terms turns them into the level's terms, which
// the draws read again instead of walking.
//
// Which segments (copy, level) are dense is decided once per index, from the
// index's own points: the share of (sampled member, member) pairs that meet in
// some table (find_dense).  A result therefore never depends on the queries
// that share its batch.  Measured: where every pair meets (70,000 sparse rows
// of 784 against 4,400 members) the walk took 5.2e-10 s a candidate and the
// pairs 0.9e-10 s with their terms; on mixtures the two are about even (30,000
// rows of 256 with draws: walk alone 8.1 ms, with the levels above 1/8, 1/4
// and 2/5 dense 8.6, 8.3 and 8.3 ms; queries alone at d = 200: 4.5, 3.8, 3.5
// and 4.3 ms).
#pragma once

namespace stag {
namespace {

constexpr int kDenseTile = 128;         // queries and members per workgroup
constexpr int kDenseSamples = 64;       // points whose candidates decide
constexpr double kDenseShare = 0.25;
constexpr int64_t kDenseMaxCols = 65536;               // columns of the pair matrix
// Pair buffers of one batch.  Each launch ends with a round that leaves part of
// the chip idle; 70,000 rows of 784 took 21.9 ms of pairs in 28 launches at
// 512 MB, 19.3 in 14 at 1 GB (their terms 6.8 and 7.2: the buffers leave the
// last-level cache).
constexpr int64_t kDenseMaxBytes = (int64_t)1 << 30;
constexpr int kDenseK = 8;              // coordinates staged at a time
constexpr int kDensePad = kDenseK + 2;  // LDS row stride (doubles): 8 rows' 16 bytes on distinct banks

using DensePair = double __attribute__((ext_vector_type(2)));

struct DenseTile {
  int32_t seg;  // segment
  int32_t u0;   // first member
};

// Pairs of one batch: D [rows][ncol] squared distances, then terms; F the
// first table of the pair (255: no term); any [row tile][column tile] whether
// a tile, of `rows` queries, holds a pair at all (where not, D and F are not
// written).  For draws,
// V and J hold each (row, segment)'s positive terms and their points in the
// walk's order (table, member ascending), from the segment's first column on,
// and len their number at [row][first column tile].
struct DensePairs {
  double* D = nullptr;
  uint8_t* F = nullptr;
  uint8_t* any = nullptr;
  double* V = nullptr;
  int32_t* J = nullptr;
  int32_t* len = nullptr;
  int rows = kDenseTile;
  int ncol = 0;                    // columns, kDenseTile per column tile
  const DenseTile* tiles = nullptr;  // the column tiles, segments ascending
  const int32_t* first = nullptr;  // [nseg + 1] first column tile of each segment
  const uint64_t* levels = nullptr;  // [K1] bit i - 1: level i of the copy is dense
};

// met[seg] = pairs (sample, member) of the segment that meet in some table, of
// up to kDenseSamples samples and kDenseMembers members, both evenly spaced (k
// of m: members r cnt / m), so that a sample is among the members and meets
// itself.  A workgroup per segment: thread (g, c) takes member c through every
// fourth group of kMetTables tables, against the samples' keys in LDS, their
// low halves.  The keys are the members' own and only that many members count:
// hashing 64 points of the data for the samples took 0.98 ms of the 20.9 that an
// index of 40,000 rows of 200 took to build, all its members 0.68; 0.03 as it is.
constexpr int kDenseMembers = 256, kMetTables = 4, kMetGroups = 4;
__global__ __launch_bounds__(kDenseMembers* kMetGroups) void count_met(int L, const uint64_t* __restrict__ seg_off,
                                                                       const uint64_t* __restrict__ mkeys,
                                                                       uint32_t* __restrict__ met) {
  __shared__ __attribute__((aligned(16))) uint32_t sk[kMetGroups][kMetTables][kDenseSamples];
  __shared__ unsigned long long met_by[kDenseMembers];
  __shared__ uint32_t total;
  const int c = threadIdx.x % kDenseMembers, g = threadIdx.x / kDenseMembers;
  const int64_t s0 = (int64_t)seg_off[blockIdx.x], cnt = (int64_t)seg_off[blockIdx.x + 1] - s0;
  if (threadIdx.x == 0) total = 0;
  if (g == 0) met_by[c] = 0;
  const int ns = (int)min(cnt, (int64_t)kDenseSamples), nm = (int)min(cnt, (int64_t)kDenseMembers);
  const int64_t u = cnt > 0 ? s0 + min(c, nm - 1) * cnt / nm : 0;
  const int sr = c % kDenseSamples, sl = c / kDenseSamples;  // this thread's sample and table of a group
  const int64_t us = cnt > 0 ? s0 + min(sr, ns - 1) * cnt / ns : 0;
  uint64_t hit = 0;
  for (int l0 = 0; cnt > 0 && l0 < L; l0 += kMetTables * kMetGroups) {
    const int lg = l0 + kMetTables * g;
    __syncthreads();  // the last tables' keys are used up
    if (lg + sl < L) sk[g][sl][sr] = (uint32_t)mkeys[us * L + lg + sl];
    __syncthreads();
    for (int l = 0; l < kMetTables && lg + l < L; ++l) {
      const uint32_t key = (uint32_t)mkeys[u * L + lg + l];
#pragma unroll
      for (int r = 0; r < kDenseSamples; ++r) hit |= (uint64_t)(sk[g][l][r] == key) << r;
    }
  }
  __syncthreads();
  if (c < nm) atomicOr(&met_by[c], hit & (ns < 64 ? (1ull << ns) - 1 : ~0ull));
  __syncthreads();
  if (g == 0) {
    uint32_t n = (uint32_t)__popcll(met_by[c]);
    for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o);
    if (c % 64 == 0) atomicAdd(&total, n);
  }
  __syncthreads();
  if (threadIdx.x == 0) met[blockIdx.x] = total;
}
static_assert(kDenseMembers == kDenseSamples * kMetTables && kDenseSamples == 64, "a key per thread, a bit per sample");

// One workgroup of 512 threads per (column tile, row tile).  Thread (ty, tx) =
// (tid / 32, tid % 32) holds rows ty + 16 i and columns tx + 32 j, i < 8, j <
// 4: 32 fp64 chains D = fma(e, e, D), e = (double)q - (double)x over ascending
// coordinates, fed by 8 + 4 LDS reads of 16 bytes for two coordinates (one at a
// time 22.4 ms, two 21.9 for 70,000 rows of 784 against 4,345 members).  Bound
// by the fp64 rate (a subtraction and a fused product per coordinate and pair,
// 4.65 cycles each: 14.9 ms of it).  8 x 8 chains per thread spilled.  A pair
// that the norm bounds of the walk put outside its level needs no distance; a
// tile without a pair that does is left out whole.  16 NI rows per workgroup
// (the figures are NI = 8's; the rule is in walk_rows).
template <bool QVEC, int NI>
__global__ __launch_bounds__(512, 4) void dense_pairs(IndexView ix, LevelConst lc, const float* __restrict__ Q,
                                                   int64_t ldq, int64_t qrow0, int64_t nq,
                                                   const uint64_t* __restrict__ qkeys, int64_t qs,
                                                   const double* __restrict__ qnorm, int self_excl, DensePairs dp,
                                                   int64_t* __restrict__ ncand) {
  __shared__ __attribute__((aligned(16))) union {
    uint64_t key[2][8][kDenseTile];
    double row[2][2][kDenseTile * kDensePad];  // [buffer][queries, members]
  } sh;
  __shared__ int32_t mj[kDenseTile];
  const int tid = threadIdx.x, tx = tid & 31, ty = tid >> 5;
  const DenseTile ct = dp.tiles[blockIdx.x];
  const int64_t r0 = (int64_t)blockIdx.y * 16 * NI;  // row of the batch
  const int L = ix.L, d = ix.d;
  const int lev = ct.seg % ix.J + 1;
  const int64_t s0 = (int64_t)ix.seg_off[ct.seg];
  const int mcnt = (int)min((int64_t)kDenseTile, (int64_t)ix.seg_off[ct.seg + 1] - s0 - ct.u0);
  const int rcnt = (int)min((int64_t)(16 * NI), nq - r0);
  if (tid < kDenseTile) mj[tid] = ix.members[s0 + ct.u0 + min(tid, mcnt - 1)];

  // first table of each pair: byte j of first[i] (255: none)
  uint32_t first[NI];
  uint32_t met[NI];  // tables in which the row meets this thread's members
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    first[i] = ~0u;
    met[i] = 0;
  }
  for (int l0 = 0; l0 < L; l0 += 8) {
    const int nl = min(8, L - l0);
    __syncthreads();
    for (int e = tid; e < nl * kDenseTile; e += 512) {
      const int l = e / kDenseTile, r = e % kDenseTile;
      sh.key[0][l][r] = qkeys[((int64_t)ct.seg * L + l0 + l) * qs + r0 + min(r, rcnt - 1)];
      sh.key[1][l][r] = ix.mkeys[(s0 + ct.u0 + min(r, mcnt - 1)) * L + l0 + l];
    }
    __syncthreads();
    for (int l = 0; l < nl; ++l) {
      uint64_t km[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) km[j] = sh.key[1][l][tx + 32 * j];
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const uint64_t kq = sh.key[0][l][ty + 16 * i];
        uint32_t eq = 0;  // 0xFF in the byte of every member that meets here
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const bool same = kq == km[j];
          eq |= same ? 0xFFu << (8 * j) : 0u;
          met[i] += same && tx + 32 * j < mcnt ? 1u : 0u;
        }
        // where the byte is still 255 it becomes the table (tables are below
        // 64, so bit 7 tells)
        const uint32_t open = ((first[i] >> 7) & 0x01010101u) * 0xFFu;
        const uint32_t take = eq & open;
        first[i] = (first[i] & ~take) | (take & ((uint32_t)(l0 + l) * 0x01010101u));
      }
    }
  }
  const double Tlo = lc.T[lev - 1], Thi = lc.T[lev];
  bool need = false;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int r = ty + 16 * i;
    const bool rlive = r < rcnt;
    const double sq = qnorm[r0 + min(r, rcnt - 1)];
    const int64_t self_idx = self_excl ? qrow0 + r0 + r : -1;
    uint32_t drop = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int c = tx + 32 * j;
      const int32_t m = mj[c];
      // the walk's norm bounds (see walk_copy)
      const double sx = ix.xn[m];
      const double e = 4e-12 * (sq + sx);
      const double up = sq + sx + e, dn = fmax(fabs(sq - sx) - e, 0.0);
      const bool out = up * up < Tlo || dn * dn >= Thi;
      if (!rlive || c >= mcnt || m == self_idx || out) drop |= 0xFFu << (8 * j);
    }
    first[i] |= drop;
    need = need || first[i] != ~0u;
    if (ncand && rlive) {
      uint32_t s = met[i];
#pragma unroll
      for (int o = 16; o > 0; o >>= 1) s += __shfl_xor(s, o);
      if (tx == 0 && s > 0) atomicAdd(reinterpret_cast<unsigned long long*>(ncand + qrow0 + r0 + r), (unsigned long long)s);
    }
  }
  const int any = __syncthreads_or(need);
  if (tid == 0) dp.any[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = any ? 1 : 0;
  if (!any) return;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int r = ty + 16 * i;
    uint8_t* f = dp.F + (r0 + r) * dp.ncol + (int64_t)blockIdx.x * kDenseTile + tx;
    if (r < rcnt)
#pragma unroll
      for (int j = 0; j < 4; ++j) f[32 * j] = (uint8_t)(first[i] >> (8 * j));
  }

  // rows kDenseK coordinates at a time, widened once on their way to LDS (a
  // conversion costs as much as four fp64 products): 2 x 128 rows x 2 pieces
  // of 16 bytes, one per thread; the first 256 threads take the queries
  const int side = tid >> 8, pr = (tid >> 1) & 127, pc = (tid & 1) * 4;
  const float* src = side == 0 ? Q + (qrow0 + r0 + min(pr, rcnt - 1)) * ldq : ix.X + (int64_t)mj[pr] * ix.dx;
  float4 st4;
  auto gload = [&](int k0) {
    const int c = k0 + pc;
    if (QVEC || side == 1) {
      // whole pieces: rows are at least d rounded up to 4 wide here, zero past d
      st4 = c < d ? *reinterpret_cast<const float4*>(src + c) : float4{0.0f, 0.0f, 0.0f, 0.0f};
    } else {
      st4.x = c < d ? src[c] : 0.0f;
      st4.y = c + 1 < d ? src[c + 1] : 0.0f;
      st4.z = c + 2 < d ? src[c + 2] : 0.0f;
      st4.w = c + 3 < d ? src[c + 3] : 0.0f;
    }
  };
  auto lstore = [&](int buf) {
    DensePair* o = reinterpret_cast<DensePair*>(&sh.row[buf][side][pr * kDensePad + pc]);
    o[0] = DensePair{(double)st4.x, (double)st4.y};
    o[1] = DensePair{(double)st4.z, (double)st4.w};
  };
  double D[NI][4];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) D[i][j] = 0.0;
  const int nk = (d + kDenseK - 1) / kDenseK;
  gload(0);
  lstore(0);
  for (int kb = 0; kb < nk; ++kb) {
    const int buf = kb & 1;
    if (kb + 1 < nk) gload((kb + 1) * kDenseK);
    __syncthreads();  // chunk kb is in LDS, the other buffer is free
    const double* ql = sh.row[buf][0] + ty * kDensePad;
    const double* xl = sh.row[buf][1] + tx * kDensePad;
#pragma unroll 1  // unrolled, the reads of all coordinates are held at once (spills)
    for (int k = 0; k < kDenseK; k += 2) {
      DensePair xd[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) xd[j] = *reinterpret_cast<const DensePair*>(&xl[32 * j * kDensePad + k]);
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const DensePair qd = *reinterpret_cast<const DensePair*>(&ql[16 * i * kDensePad + k]);
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const double t = qd[e] - xd[j][e];
            D[i][j] = __builtin_fma(t, t, D[i][j]);
          }
      }
    }
    if (kb + 1 < nk) lstore(buf ^ 1);
  }
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int r = ty + 16 * i;
    if (r < rcnt) {
      double* o = dp.D + (r0 + r) * dp.ncol + (int64_t)blockIdx.x * kDenseTile + tx;
#pragma unroll
      for (int j = 0; j < 4; ++j) o[32 * j] = D[i][j];
    }
  }
}

// Terms of the dense pairs and what they add to each query's copy sums, level
// masks and accepted counts.  One wave per query and copy: columns in order,
// lanes strided, one butterfly sum (one query of an index of 5,000 rows of 200:
// a wave for all copies 162 us, 7 with one for each).  LIST: the terms take their distances'
// place (table 255 outside the level) and are then listed per segment in the
// walk's order: a count per table, a scan over the tables and a second pass
// that ranks a batch's equal tables, both by ballots of the tables' bits.
template <bool LIST>
__global__ __launch_bounds__(256) void dense_terms(IndexView ix, LevelConst lc, int64_t qrow0, int64_t nq,
                                                   DensePairs dp, double* __restrict__ Scopy,
                                                   int64_t* __restrict__ nacc, uint64_t* __restrict__ levels_out) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t r = (int64_t)blockIdx.x * 4 + wave;
  if (r >= nq) return;
  const int nct = dp.ncol / kDenseTile;
  const uint8_t* any = dp.any + (r / dp.rows) * nct;
  const uint64_t below = (1ull << lane) - 1ull;
  // the column tiles in [c0, c1) that hold a pair, the next one's values
  // loaded before this one's are used (a wave's loads one after the other
  // were what the terms waited for: 7.2 ms for 70,000 rows, then 6.7; 6.2 with
  // the ranks below from ballots instead of a loop over the tables met; 5.2
  // with a wave for every copy)
  struct Piece {
    double D[kDenseTile / 64];
    uint8_t f[kDenseTile / 64];
  };
  auto each_tile = [&](int c0, int c1, auto&& use) {
    for (int cb = c0; cb < c1; cb += 64) {
      uint64_t left = __ballot(cb + lane < c1 && any[min(cb + lane, c1 - 1)]);
      Piece next;
      int64_t o = 0;
      int ct = cb;
      auto load = [&] {
        ct = cb + __builtin_ctzll(left);
        left &= left - 1;
        o = r * dp.ncol + (int64_t)ct * kDenseTile + lane;
#pragma unroll
        for (int k = 0; k < kDenseTile; k += 64) {
          next.D[k / 64] = dp.D[o + k];
          next.f[k / 64] = dp.F[o + k];
        }
      };
      bool some = left != 0;
      if (some) load();
      while (some) {
        const Piece p = next;
        const int64_t at = o;
        const int tile = ct;
        some = left != 0;
        if (some) load();
        use(tile, at, p);
      }
    }
  };
  int lbits = 0;  // of a table's number
  while ((1 << lbits) < ix.L) ++lbits;
  const int t = blockIdx.y;
  int64_t na = 0;
  double acc = 0.0;
  uint64_t hit = 0;
  for (int i = 1; i <= ix.J; ++i) {
    const int seg = t * ix.J + (i - 1);
    const int c0 = dp.first[seg], c1 = dp.first[seg + 1];
    if (c0 == c1) continue;
    const double Tlo = lc.T[i - 1], Thi = lc.T[i], ri = lc.r[i];
    uint32_t count = 0;  // lane l: positive terms of table l, then its next place
    each_tile(c0, c1, [&](int, int64_t o, const Piece& p) {
#pragma unroll
      for (int k = 0; k < kDenseTile; k += 64) {
        const double D = p.D[k / 64];
        const uint8_t f = p.f[k / 64];
        const bool in = f != 255 && D >= Tlo && D < Thi;
        const double v = in ? level_weight(ix.cheb + i * kChebRow, sqrt(D) / ri) : 0.0;
        acc += v;
        na += v > 0.0 ? 1 : 0;
        const uint64_t open = __ballot(v > 0.0);
        if (open) hit |= 1ull << (i - 1);
        if constexpr (LIST) {
          dp.D[o + k] = v;
          if (!(v > 0.0)) dp.F[o + k] = 255;
          // lane l: the terms of table l, from the ballots of the tables' bits
          uint64_t same = lane < ix.L ? open : 0ull;
          for (int q = 0; q < lbits; ++q) {
            const uint64_t ones = __ballot((f >> q) & 1);
            same &= (lane >> q) & 1 ? ones : ~ones;
          }
          count += (uint32_t)__popcll(same);
        }
      }
    });
    if constexpr (LIST) {
      uint32_t incl = count;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(incl, o);
        if (lane >= o) incl += y;
      }
      count = incl - count;
      if (lane == 63) dp.len[r * nct + c0] = (int32_t)incl;
      const int64_t s0 = (int64_t)ix.seg_off[seg];
      const int64_t out = r * dp.ncol + (int64_t)c0 * kDenseTile;
      each_tile(c0, c1, [&](int ct, int64_t, const Piece& p) {
#pragma unroll
        for (int k = 0; k < kDenseTile; k += 64) {
          const uint8_t f = p.f[k / 64];
          const uint64_t open = __ballot(f != 255);
          uint64_t same = lane < ix.L ? open : 0ull, peers = open;  // terms of table `lane`; of this term's table
          for (int q = 0; q < lbits; ++q) {
            const uint64_t ones = __ballot((f >> q) & 1);
            same &= (lane >> q) & 1 ? ones : ~ones;
            peers &= (f >> q) & 1 ? ones : ~ones;
          }
          const uint32_t place = (uint32_t)__shfl((int)count, f & 63) + (uint32_t)__popcll(peers & below);
          count += (uint32_t)__popcll(same);
          if (f != 255) {
            dp.V[out + place] = p.D[k / 64];
            dp.J[out + place] = ix.members[s0 + (int64_t)(ct - c0) * kDenseTile + k + lane];
          }
        }
      });
    }
  }
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
  if (lane == 0) {
    Scopy[r * ix.K1 + t] += acc;
    if (levels_out && hit) levels_out[(qrow0 + r) * ix.K1 + t] |= hit;
  }
  for (int o = 32; o > 0; o >>= 1) na += __shfl_xor(na, o);
  if (nacc && lane == 0 && na > 0)
    atomicAdd(reinterpret_cast<unsigned long long*>(nacc + qrow0 + r), (unsigned long long)na);
}

// A node's listed terms of one dense segment, handed to on_batch 64 at a time.
template <class F>
__device__ inline void dense_walk(const DensePairs& dp, int64_t row, int seg, int lev, F&& on_batch) {
  const int lane = threadIdx.x & 63;
  const int c0 = dp.first[seg];
  const int n = dp.len[row * (dp.ncol / kDenseTile) + c0];
  const int64_t o = row * dp.ncol + (int64_t)c0 * kDenseTile;
  for (int k = 0; k < n; k += 64) {
    const bool mine = k + lane < n;
    on_batch(mine ? dp.V[o + k + lane] : 0.0, mine ? dp.J[o + k + lane] : -1, mine, lev);
  }
}

}  // namespace
}  // namespace stag
