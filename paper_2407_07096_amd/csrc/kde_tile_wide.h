// Wide rows (256 < d <= 1024) of the exact kernel density: the matrix-core
// tile of the fp32 and the hi + lo split forms, and the operand layout it
// reads (internal; included by kde_tiles.h).
//
// Operand layout ("fragments").  Rows are stored per 32-row tile in the order
// in which a wave reads its matrix operands: fragment (tile, s) is 1 KB, 16
// bytes per lane, lane l = 32 h + r holding, of row r of the tile,
//   split forms  the 8 halfs of dimensions [16 s + 8 h, 16 s + 8 h + 8)
//   fp32         the 4 floats of dimensions h DP/2 + [4 s, 4 s + 4)
// A tile has DP/16 (split) or DP/8 (fp32) fragments; a fragment is one
// coalesced 1 KB read, lands in LDS as it is and is read back there at
// 16 bytes per lane without bank conflicts.
#pragma once

namespace stag {
namespace tiles {

constexpr int kWideRT = 8;          // 32-row data tiles per workgroup step
constexpr int kWideQT = 4;          // 32-query blocks per workgroup (kBQ queries)
constexpr int kSubTiles = 16;       // 32-row tiles per sub-chunk
constexpr int kSubs = kChunkTiles / kSubTiles;
constexpr int kWideRuns = kSubTiles / kWideRT;  // steps per sub-chunk
// Record of sub-chunk k of the chunk, accumulator c of C, query qi.
__device__ inline int64_t sub_index(int64_t chunk, int k, int C, int c, int64_t m_pad, int64_t qi) {
  return ((chunk * kSubs + k) * C + c) * m_pad + qi;
}
constexpr int kWideWinQ = 8, kWideWinC = 8;
// Launches of at most this many pairs (128 queries x chunk) that don't share
// chunks (the exponential kernel, whose near pairs are kept per chunk, the
// no-allocation call and the rescue's passes) take 32 queries a workgroup.
// fp32 is bound by the matrix products of a compute unit's one workgroup:
// 1,992 us with 128 queries and 727 with 32 at d = 784 and 64 pairs, 1,992 and
// 1,309 at 128, 2,000 and 1,890 at 192, 1,997 and 2,470 at 224 (three quarters
// of the last round of 256 compute units idle).  The split forms wait on memory
// instead, where 128 queries share a row: 653 and 470 us at 64 pairs, 652 and
// 739 at 80.
template <int FORM>
constexpr int64_t kWideNarrowPairs = FORM == STAG_FORM_FP32 ? 192 : 64;

// Workgroup b -> (query tile, chunk).  Workgroups are dealt to the 8 XCDs
// in turn; XCD x takes the x-th eighth of the list of all pairs, ordered by
// windows of 8 query tiles x 8 chunks, so that the 64 workgroups an XCD runs
// together read 8 chunks' rows and 8 tiles' queries instead of 64 different
// ones of either.  Returns false past the end of the list.
__device__ inline bool wide_tile(int64_t b, int nq, int P, int* qtile, int* chunk) {
  const int64_t total = (int64_t)nq * P, per = (total + 7) / 8;
  const int64_t i = (b % 8) * per + b / 8;
  if (b / 8 >= per || i >= total) return false;
  const int g = (int)(i / ((int64_t)kWideWinC * nq));  // chunk group
  const int cg = min(kWideWinC, P - g * kWideWinC);
  const int64_t r = i - (int64_t)g * kWideWinC * nq;  // < cg * nq
  const int w = (int)(r / (kWideWinQ * cg));
  const int qn = min(kWideWinQ, nq - w * kWideWinQ);
  const int e = (int)(r - (int64_t)w * kWideWinQ * cg);
  *chunk = g * kWideWinC + e / qn;
  *qtile = w * kWideWinQ + e % qn;
  return true;
}

template <int FORM>
constexpr int kWideParts = FORM == STAG_FORM_FP32 ? 1 : 2;
// k-steps (fragments) loaded at a time
template <int FORM, int QT>
constexpr int kWideK = QT == 1 ? (FORM == STAG_FORM_FP32 ? 4 : 2) : 1;

// A workgroup takes QT blocks of 32 queries against a 4096-row chunk, 256 data
// rows at a time, which its four waves split by row tile and query block:
//   QT = 4 (128 queries; or a share of the chunk: ex.nsub workgroups per pair,
//     each storing its sub-chunks' sums, which combine_subs adds in the same
//     order): the 8 x 4 blocks of 32 rows x 32 queries as 2 x 2, 4 row tiles x
//     2 query blocks (128 accumulators) each; wave half wr takes the tiles t
//     with (t / 2) % 2 = wr.
//   QT = 1 (32 queries): wave w takes the tiles t with t % 4 = w.  For
//     launches whose 128-query pairs leave compute units idle and that can't
//     share a chunk (see kWideNarrowPairs): four times as many workgroups with
//     a quarter of the products each.
// Per step the 8 row and QT query fragments (per part and k-step) go through
// registers to LDS, loaded from memory two steps ahead of their use (two
// buffers, one barrier per step); with QT = 4 a wave reads 12 fragments for its
// 24 products (split).  With QT = 1 a step takes several k-steps (kWideK), as
// its products no longer cover the loads: 8 queries against 70,000 rows of 784
// in the fp16 split form took 892 us a call with one k-step at a time, 495 with
// two (fp32 1,115 and 929 with four).  Products of one block come in ascending
// k with the parts in a fixed order on one accumulator, so a result has the
// same bits as with any other tiling.
// Measured at n = 70,000, d = 784 (a whole call): against 10,000 queries in the
// fp16 split form 8.2 -> 2.3 ms, in fp32 9.7 (the tile before this one kept 32
// queries per workgroup in LDS and streamed every row from the last-level cache
// for them: 0.5 TB a call).
// Sums: per lane fp64 over the tiles of a sub-chunk of a class t % 4 in order,
// classes 0 + 1 and 2 + 3, the sub-chunks in order, then lane halves, then the
// two pairs of classes.
// Near pairs (exponential kernel): the first kNearSlots tiles that hold some
// are taken of each class and lane.
template <int FORM, int MODE, int QT>
__global__ __launch_bounds__(256, 2) void tile_wide(const char* __restrict__ X0, const char* __restrict__ X1,
                                                    const float* __restrict__ Xoff, const char* __restrict__ Q0,
                                                    const char* __restrict__ Q1, const float* __restrict__ Qoff,
                                                    int nfrag, int ns, int64_t n_pad, int n_qtiles, int P,
                                                    int64_t m_pad, double* __restrict__ partial, TileExtra ex) {
  static_assert(QT == 1 || QT == kWideQT, "32 or 128 queries");
  constexpr int NP = kWideParts<FORM>;
  constexpr int NF = (kWideRT + QT) * NP;  // fragments per k-step
  constexpr int NK = kWideK<FORM, QT>;
  constexpr int NR = QT == 1 ? 2 : 4;      // row tiles of a wave and step
  constexpr int NB = QT == 1 ? 1 : 2;      // query blocks of a wave
  constexpr int NC = QT == 1 ? 1 : 2;      // tile classes of a wave: that of row tile i is i % NC
  constexpr bool NEAR = MODE == kModeExponential;
  __shared__ __attribute__((aligned(16))) char frag[2][NK * NF * 1024];
  __shared__ double wsum[2][QT][32];
  __shared__ uint32_t near_lds[NEAR ? NB * NC * kNearSlots * 256 : 1];
  // QT = 4: the sums so far of a lane's query blocks; 1: those of each sub-chunk
  constexpr int NT = QT == 1 ? kSubs : NB;
  __shared__ double total[NT][256];
  const int tid = threadIdx.x, lane = tid & 63, r32 = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = QT == 1 ? wave : wave >> 1, wq = QT == 1 ? 0 : wave & 1;
  // row tile i of this wave among the 8 of a step
  auto row_tile = [&](int i) { return QT == 1 ? wr + 4 * i : (i & 1) + 2 * wr + 4 * (i >> 1); };
  int qtile, chunk;
  // shares of a chunk are neighbours in the order of the list
  if (!wide_tile(blockIdx.x, n_qtiles, P * ex.nsub, &qtile, &chunk)) return;
  const int part = chunk % ex.nsub;
  chunk /= ex.nsub;
  if (ex.qtile_active && ex.qtile_active[qtile * QT / kWideQT] == 0) return;  // whole block
  const int nrun = kSubs / ex.nsub;  // sub-chunks of this workgroup
  const int64_t row0 = (int64_t)chunk * kChunkRows + (int64_t)part * nrun * kSubTiles * kTileRows;
  const int ntiles = (int)max((int64_t)0, min((n_pad - row0) / kTileRows, (int64_t)nrun * kSubTiles));
  const int nblk = (ntiles + kWideRT - 1) / kWideRT;
  const int64_t tile0 = row0 / kTileRows;
  int64_t col[NB], qi[NB];
  float alpha[NB], ys[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    col[j] = ((int64_t)qtile * QT + NB * wq + j) * 32;
    qi[j] = col[j] + r32;
    alpha[j] = Qoff[qi[j]];
    ys[j] = kShiftMode<MODE> ? ex.yshift[qi[j]] : 0.0f;
  }

  double acc[NB][NC];
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[j][c] = acc_init<MODE>();
#pragma unroll
  for (int j = 0; j < NT; ++j) total[j][tid] = acc_init<MODE>();
  auto end_run = [&](int k) {  // end of this workgroup's sub-chunk k
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      if constexpr (QT == 1) {
        total[k][tid] = acc[0][0];
      } else {
        const double a = acc_add<MODE>(acc[j][0], acc[j][NC - 1]);
        if (ex.nsub > 1) ex.sub[sub_index(chunk, part * nrun + k, 4, 2 * wr + h, m_pad, qi[j])] = a;
        else total[j][tid] = acc_add<MODE>(total[j][tid], a);
      }
#pragma unroll
      for (int c = 0; c < NC; ++c) acc[j][c] = acc_init<MODE>();
    }
  };
  if (ntiles == 0) {  // a share past the last row (nsub > 1)
    for (int k = 0; k < nrun; ++k) end_run(k);
    return;
  }

  // This wave's fragments of a step: row tiles 2 wave and 2 wave + 1 and, if
  // there is one, query block wave, every part (scalar addresses; past the
  // chunk's last tile the last one is read again and its results left out).
  constexpr int WA = kWideRT / 4;
  const int64_t tbytes = (int64_t)nfrag * 1024;
  f32x4 sa[NK][NP][WA], sb[NK][NP];
  auto gload = [&](int b, int s) {
#pragma unroll
    for (int u = 0; u < NK; ++u) {
#pragma unroll
      for (int p = 0; p < NP; ++p) {
#pragma unroll
        for (int k = 0; k < WA; ++k) {
          const int64_t t = tile0 + min(b * kWideRT + WA * wave + k, ntiles - 1);
          const char* src = (p == 0 ? X0 : X1) + (t * tbytes + (s + u) * 1024);
          sa[u][p][k] = *reinterpret_cast<const f32x4*>(src + lane * 16);
        }
        if (QT == kWideQT || wave < QT) {
          const char* src = (p == 0 ? Q0 : Q1) + (((int64_t)qtile * QT + wave) * tbytes + (s + u) * 1024);
          sb[u][p] = *reinterpret_cast<const f32x4*>(src + lane * 16);
        }
      }
    }
  };
  auto lstore = [&](int buf) {
    char* dst = &frag[buf][lane * 16];
#pragma unroll
    for (int u = 0; u < NK; ++u) {
#pragma unroll
      for (int p = 0; p < NP; ++p) {
#pragma unroll
        for (int k = 0; k < WA; ++k)
          *reinterpret_cast<f32x4*>(dst + (u * NF + p * kWideRT + WA * wave + k) * 1024) = sa[u][p][k];
        if (QT == kWideQT || wave < QT)
          *reinterpret_cast<f32x4*>(dst + (u * NF + NP * kWideRT + p * QT + wave) * 1024) = sb[u][p];
      }
    }
  };

  NearRec nr[NB][NC];  // [query block][tile class]
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int k = 0; k < NC; ++k) nr[j][k] = {near_lds + (NEAR ? (NC * j + k) * kNearSlots * 256 : 0), 0, false};
  // the next step to load: (block lb, k-step ls); past the last one it is
  // loaded again
  int lb = 0, ls = 0;
  auto advance = [&]() {
    gload(lb, ls);
    const bool wrap = ls + NK == ns;
    const bool end = wrap && lb + 1 == nblk;
    ls = end ? ls : (wrap ? 0 : ls + NK);
    lb = wrap && !end ? lb + 1 : lb;
  };
  advance();
  lstore(0);
  advance();
  int buf = 0;
  for (int b = 0; b < nblk; ++b) {
    f32x16 c[NR][NB];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      if constexpr (FORM == STAG_FORM_FP32) {
#pragma unroll
        for (int j = 0; j < NB; ++j) c[i][j] = f32x16{0};
      } else {
        // the accumulators start from the offsets alpha_q + beta_x
        const int64_t rb = row0 + (int64_t)min(b * kWideRT + row_tile(i), ntiles - 1) * kTileRows;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x4 bv = *reinterpret_cast<const f32x4*>(Xoff + rb + 8 * g + 4 * h);
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int j = 0; j < NB; ++j) c[i][j][4 * g + e] = alpha[j] + bv[e];
        }
      }
    }
    for (int s = 0; s < ns; s += NK) {
      __syncthreads();  // these steps' fragments are in buf; the other buffer is free
      f32x4 fa[NP][NR], fb[NP][NB];
      auto fetch = [&](int u) {
        const char* fl = &frag[buf][u * NF * 1024 + lane * 16];
#pragma unroll
        for (int p = 0; p < NP; ++p) {
#pragma unroll
          for (int j = 0; j < NB; ++j)
            fb[p][j] = *reinterpret_cast<const f32x4*>(fl + (kWideRT * NP + p * QT + NB * wq + j) * 1024);
#pragma unroll
          for (int i = 0; i < NR; ++i)
            fa[p][i] = *reinterpret_cast<const f32x4*>(fl + (p * kWideRT + row_tile(i)) * 1024);
        }
      };
      auto products = [&] {
        if constexpr (FORM == STAG_FORM_FP32) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < NR; ++i)
#pragma unroll
              for (int j = 0; j < NB; ++j)
                c[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[0][i][e], fb[0][j][e], c[i][j], 0, 0, 0);
        } else {
          // per block: hi hi, hi lo, lo hi
#pragma unroll
          for (int o = 0; o < 3; ++o)
#pragma unroll
            for (int i = 0; i < NR; ++i)
#pragma unroll
              for (int j = 0; j < NB; ++j)
                c[i][j] = mma16<FORM>(__builtin_bit_cast(u16x8, fa[o == 2 ? NP - 1 : 0][i]),
                                      __builtin_bit_cast(u16x8, fb[o == 1 ? NP - 1 : 0][j]), c[i][j]);
        }
      };
      fetch(0);
      lstore(buf ^ 1);  // the next steps' (after the last: a copy nobody reads)
      advance();
      products();
#pragma unroll
      for (int u = 1; u < NK; ++u) {
        fetch(u);
        products();
      }
      buf ^= 1;
    }
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int t = b * kWideRT + row_tile(i);
      if (t < ntiles) {  // wave-uniform
        const int64_t rb = row0 + (int64_t)t * kTileRows;
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          if constexpr (FORM == STAG_FORM_FP32) {
            // offsets by one more product: 1 * alpha (half 0) + beta * 1 (half 1)
            const float tb = Xoff[rb + r32];
            c[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(h == 0 ? 1.0f : tb, h == 0 ? alpha[j] : 1.0f, c[i][j], 0,
                                                           0, 0);
          }
          double& a = acc[j][i % NC];
          a = acc_add<MODE>(a, (double)tile_epilogue<MODE>(c[i][j], rb, col[j], r32, h, qi[j], ex, nullptr, false,
                                                           &nr[j][i % NC], t, ys[j]));
        }
      }
    }
    if (b % kWideRuns == kWideRuns - 1) end_run(b / kWideRuns);
  }
  if (nblk % kWideRuns != 0) end_run(nblk / kWideRuns);
  if (ex.nsub > 1) {
    for (int k = (nblk + kWideRuns - 1) / kWideRuns; k < nrun; ++k) end_run(k);  // runs past the last row
    return;
  }
  if constexpr (QT == 1) {
    __shared__ double near_sum[NEAR ? 256 : 1];
    if constexpr (NEAR) near_sum[tid] = near_finish(ex, nr[0][0], qi[0], h, row0, tid);
    __syncthreads();
    if (wave < 2) {  // wave w adds up the classes 2 w and 2 w + 1
      const int c0 = 128 * wave + lane, c1 = c0 + 64;
      double a = acc_init<MODE>();
#pragma unroll
      for (int k = 0; k < kSubs; ++k) a = acc_add<MODE>(a, acc_add<MODE>(total[k][c0], total[k][c1]));
      if constexpr (NEAR) {
        a += near_sum[c0];
        a += near_sum[c1];
      }
      const double other = __shfl_down(a, 32);
      if (h == 0) wsum[wave][0][r32] = acc_add<MODE>(a, other);
    }
  } else {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      double a = total[j][tid];
      if constexpr (NEAR) {
        a += near_finish(ex, nr[j][0], qi[j], h, row0, tid);
        a += near_finish(ex, nr[j][NC - 1], qi[j], h, row0, tid);
      }
      const double other = __shfl_down(a, 32);
      if (h == 0) wsum[wr][2 * wq + j][r32] = acc_add<MODE>(a, other);
    }
  }
  __syncthreads();
  if (tid < 32 * QT)
    partial[(int64_t)chunk * m_pad + (int64_t)qtile * 32 * QT + tid] =
        acc_add<MODE>(wsum[0][tid >> 5][tid & 31], wsum[1][tid >> 5][tid & 31]);
}

}  // namespace tiles
}  // namespace stag
