// Block scoring (paper Sec. IV: blocks are ranked by their l2 magnitude).
//
// score[i*nbc + j] = sum of x^2 over the valid elements of block (i,j), in
// binary64.  One streaming read of X: HBM-bound.  A workgroup owns `RB`
// consecutive block-rows and a chunk of `jc` block-columns; consecutive lanes
// read consecutive vectors of one matrix row (coalesced), row groups stride over
// the rows, and the partial sums meet in LDS where one lane per block adds them
// in a fixed order (reproducible bit for bit, no atomics).
#include "common.h"

namespace bsr {

namespace {

constexpr int kScoreThreads = 256;
constexpr int kRowClasses = 8;     // rows of a block that are eight apart are summed by one lane (score_direct_body)

struct ScoreGeom {
  int jc;    // block-columns per workgroup
  int vpbt;  // lanes across one block row (= min(vectors per block row, 256))
  int vct;   // lanes across the chunk (= jc * vpbt)
  int gb;    // row groups per block-row
  int rb;    // block-rows handled per pass
  int nchunks;
  int direct;  // score_direct_body (1; 2: its form for few tall blocks), gb lanes per vector column of a block and vpbt of
               // these in a block; nchunks = its workgroups
};

// bx, by, gy: the workgroup's place in its tensor's (chunks x passes) grid.  Threads beyond
// g.vct * g.gb * g.rb (a batched launch runs every tensor with 256) find no row group and idle.
template <typename T, int V>
__device__ __forceinline__ void score_body(
    const T *__restrict__ X, int64_t M, int64_t K, int64_t ldx, int br, int bc, int64_t nbr,
    int64_t nbc, const ScoreGeom &g, double *__restrict__ scores, uint32_t bx, uint32_t by, uint32_t gy) {
  __shared__ double part[kScoreThreads];
  const int t = threadIdx.x;
  const int lane_col = t % g.vct;          // vector column inside the chunk
  const int grp = t / g.vct;               // row group
  const int ib = grp / g.gb;               // block-row of this pass
  const int gr = grp % g.gb;               // row group inside the block-row
  const int jj = lane_col / g.vpbt;        // block-column inside the chunk
  const int vpb = bc / V;                  // vectors per block row
  const int64_t j = (int64_t)bx * g.jc + jj;
  const int64_t col0 = j * bc;

  for (int64_t pass = by; pass * g.rb < nbr; pass += gy) {
    const int64_t i = pass * g.rb + ib;
    double acc = 0.0;
    if (ib < g.rb && i < nbr && j < nbc) {
      const int64_t m0 = i * br;
      const int rows = (int)((M - m0) < br ? (M - m0) : br);
      for (int u = lane_col % g.vpbt; u < vpb; u += g.vpbt) {
        const int64_t col = col0 + (int64_t)u * V;
        if (col >= K) break;
        const T *p = X + m0 * ldx + col;
        // kInFlight loads are issued before the first of them is consumed (the
        // kernel is bound by memory latency, not arithmetic); the order of the
        // additions stays r ascending, whatever the batching
        constexpr int kInFlight = 8;
        for (int r0 = gr; r0 < rows; r0 += kInFlight * g.gb) {
          Raw<T, V> v[kInFlight];
#pragma unroll
          for (int b = 0; b < kInFlight; ++b) {
            const int r = r0 + b * g.gb;
            if (r < rows) v[b] = *reinterpret_cast<const Raw<T, V> *>(p + (int64_t)r * ldx);
          }
#pragma unroll
          for (int b = 0; b < kInFlight; ++b) {
            if (r0 + b * g.gb < rows) {
#pragma unroll
              for (int q = 0; q < V; ++q) {
                const double x = (double)raw_elem<T, V>(v[b], q);
                acc = fma(x, x, acc);
              }
            }
          }
        }
      }
    }
    part[t] = acc;
    __syncthreads();
    // one lane per (block-row, block-column) of this pass adds the partials
    if (t < g.rb * g.jc) {
      const int oib = t / g.jc, ojj = t % g.jc;
      const int64_t oi = pass * g.rb + oib, oj = (int64_t)bx * g.jc + ojj;
      if (oi < nbr && oj < nbc) {
        double s = 0.0;
        for (int a = 0; a < g.gb; ++a)
          for (int u = 0; u < g.vpbt; ++u) s += part[(oib * g.gb + a) * g.vct + ojj * g.vpbt + u];
        scores[oi * nbc + oj] = s;
      }
    }
    __syncthreads();
  }
}

// Large matrices: bc / V * RS lanes own a block -- lane (part, u) reads vector u of the rows
// part, part + RS, ... of the block, eight loads on their way at a time (consecutive lanes
// read consecutive vectors of a matrix row, whole 64-byte pieces or more).  No LDS, no barrier,
// every lane busy.  RS (1, 2, 4 or 8, g.gb) is chosen so that the tensor has enough lanes for the chip.
// The sum does not depend on it: the rows r, r + 8, ... of a vector column are added top to
// bottom, then the eight such sums pairwise (r and r + 4, r and r + 2, r and r + 1), then the vector
// columns; a step of that is an addition inside a lane or a lane exchange, depending on RS.
// TALL: few blocks of 128 rows and more, where eight lanes per vector column leave the chip idle and a lane with a
// chain of additions as long as its rows.  rs = 8 .. 64 lanes share a column, a number that follows from the matrix and the
// block alone (score_geometry), and each keeps two sums, of the even and of the odd elements.  ([4096 x 384] binary32
// in 256x16 blocks, score and select: 16.0 us through the LDS body, 7.5 so.)
// LOOSE: rows that begin at any element, block widths that are no whole vectors, a last block in part: 16 bytes at a time
// all the same (global loads need no alignment beyond the element's).  What a vector holds beyond its block or the last column is set
// to zero, a vector that would reach beyond the last element of X ends there and is shifted.  (Score and select, bf16,
// through 2- and 4-byte loads and the LDS body and so: [41298 x 805] in 14x14 blocks 102 and 32 us, [23394 x 1453] 99 and 32,
// [10307 x 1071] in 1x32 75 and 28, [30022 x 1153] in 64x64 31 and 24.)
// wg = index of the workgroup among the ceil(nbr * nbc * vpb * RS / 256) of its tensor.
template <typename T, int V, int RS, bool LOOSE>
__device__ __forceinline__ void score_direct_body(
    const T *__restrict__ X, int64_t M, int64_t K, int64_t ldx, int br, int bc, int64_t nbr,
    int64_t nbc, uint32_t vpb, int rs, double *__restrict__ scores, uint32_t wg) {
  static_assert(!LOOSE || V * sizeof(T) == 16, "whole vectors of 16 bytes");
  constexpr bool TALL = RS == 0;
  const int lanes = TALL ? rs : RS;
  constexpr int kOwn = TALL ? 2 : kRowClasses / (TALL ? 1 : RS);   // sums a lane keeps: its row classes
  // vpb: lanes across a block row, a power of two
  const uint32_t lpb = vpb * (uint32_t)lanes;              // lanes per block: a power of two, at most 64
  const uint32_t per_row = (uint32_t)nbc * lpb;            // lanes per block-row
  const uint32_t gid = wg * (uint32_t)kScoreThreads + threadIdx.x;
  const uint32_t i = gid / per_row, c = gid - i * per_row;
  const uint32_t j = c / lpb, within = c & (lpb - 1), part = within / vpb, u = within & (vpb - 1);
  const int64_t col = (int64_t)j * bc + (int64_t)u * V;
  const bool live = (int64_t)i < nbr && col < K && (!LOOSE || (int)u * V < bc);
  const int64_t m0 = (int64_t)i * br;
  const int rows = live ? (int)((M - m0) < br ? (M - m0) : br) : 0;
  const T *p = X + m0 * ldx + col;
  // LOOSE: the words of a vector that belong to the block, and whether any of the lane's vectors reaches beyond X
  RawWords<16>::type own = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu};
  const T *const end = X + (M - 1) * ldx + K;
  bool near_end = false;
  if constexpr (LOOSE) {
    int n = bc - (int)u * V < V ? bc - (int)u * V : V;
    if (K - col < n) n = (int)(K - col);
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const int in = n * (int)sizeof(T) - 4 * w;             // bytes of word w inside
      own[w] = in >= 4 ? 0xFFFFFFFFu : in > 0 ? (1u << (8 * in)) - 1u : 0u;
    }
    near_end = rows > 0 && p + (int64_t)(rows - 1) * ldx + V > end;
  }
  auto load = [&](const T *at) -> Raw<T, V> {
    if constexpr (LOOSE) {
      typedef RawWords<16>::type __attribute__((aligned(2))) Any;
      return *reinterpret_cast<const Any *>(at);
    } else {
      return load_stream(reinterpret_cast<const Raw<T, V> *>(at));
    }
  };
  double acc[kOwn];
#pragma unroll
  for (int k = 0; k < kOwn; ++k) acc[k] = 0.0;
  // (eight, not more: with sixteen the registers they need leave room for three waves per SIMD only,
  // and a workgroup has nothing in flight while it adds up.  As native vectors: loads of eight 16-bit elements under
  // a condition came one at a time; score and select of 24 tensors [25088 x 384] took 92 us so, 81 now, of
  // [6000 x 768] in 64x64 blocks 11.9 and 9.8)
  constexpr int kInFlight = 8;
  auto add = [&](Raw<T, V> v, int b) {
    if constexpr (LOOSE) v &= own;
#pragma unroll
    for (int q = 0; q < V; ++q) {
      const double x = (double)raw_elem<T, V>(v, q);
      const int k = TALL ? q % 2 : b % kOwn;
      acc[k] = fma(x, x, acc[k]);
    }
  };
  int first = (int)part;
  if constexpr (LOOSE) {
    if (__builtin_expect(near_end, 0)) {                     // one row at a time
      for (; first < rows; first += kInFlight * lanes) {
#pragma unroll
        for (int b = 0; b < kInFlight; ++b) {
          const int r = first + b * lanes;
          if (r >= rows) continue;
          const T *const at = p + (int64_t)r * ldx;
          const int over = at + V > end ? (int)(at + V - end) * (int)sizeof(T) : 0;
          RawWords<16>::type v = load(reinterpret_cast<const T *>(reinterpret_cast<const char *>(at) - over));
          uint64_t lo = ((uint64_t)v[1] << 32) | v[0], hi = ((uint64_t)v[3] << 32) | v[2];
          if (over >= 8) { lo = hi >> (8 * (over - 8)); hi = 0; }
          else if (over > 0) { lo = (lo >> (8 * over)) | (hi << (64 - 8 * over)); hi >>= 8 * over; }
          v[0] = (uint32_t)lo; v[1] = (uint32_t)(lo >> 32); v[2] = (uint32_t)hi; v[3] = (uint32_t)(hi >> 32);
          add(v, b);
          asm volatile("" ::: "memory");                     // (no loads ahead: their registers would be all lanes')
        }
      }
    }
  }
  for (int r0 = first; r0 < rows; r0 += kInFlight * lanes) {
    Raw<T, V> v[kInFlight];
#pragma unroll
    for (int b = 0; b < kInFlight; ++b)
      if (r0 + b * lanes < rows) v[b] = load(p + (int64_t)(r0 + b * lanes) * ldx);
#pragma unroll
    for (int b = 0; b < kInFlight; ++b) {
      if (r0 + b * lanes >= rows) continue;
      if constexpr (LOOSE) {
        add(v[b], b);
      } else {
        // (not through the function above: 8 registers more for bfloat16, six waves per SIMD instead of seven.  Score and select of
        // [25088 x 1536] with a pitch of 1544 in 4x96 blocks 67 us so, 62 without)
#pragma unroll
        for (int q = 0; q < V; ++q) {
          const double x = (double)raw_elem<T, V>(v[b], q);
          const int k = TALL ? q % 2 : b % kOwn;
          acc[k] = fma(x, x, acc[k]);
        }
      }
    }
  }
#pragma unroll
  for (int half = kOwn / 2; half >= 1; half /= 2)
#pragma unroll
    for (int k = 0; k < half; ++k) acc[k] += acc[k + half];
  double sum = acc[0];
  for (int o = lanes / 2; o >= 1; o /= 2) sum += __shfl_xor(sum, o * (int)vpb);
  for (uint32_t o = 1; o < vpb; o <<= 1) sum += __shfl_xor(sum, (int)o);
  if (live && within == 0) scores[(int64_t)i * nbc + j] = sum;
}

template <typename T, int V, bool LOOSE>
__device__ __forceinline__ void score_direct(
    const T *__restrict__ X, int64_t M, int64_t K, int64_t ldx, int br, int bc, int64_t nbr,
    int64_t nbc, const ScoreGeom &g, double *__restrict__ scores, uint32_t wg) {
  const uint32_t vpb = LOOSE ? (uint32_t)g.vpbt : (uint32_t)(bc / V);
  if (g.direct == 2) {
    score_direct_body<T, V, 0, LOOSE>(X, M, K, ldx, br, bc, nbr, nbc, vpb, g.gb, scores, wg);
    return;
  }
  switch (g.gb) {
    case 1: score_direct_body<T, V, 1, LOOSE>(X, M, K, ldx, br, bc, nbr, nbc, vpb, 1, scores, wg); break;
    case 2: score_direct_body<T, V, 2, LOOSE>(X, M, K, ldx, br, bc, nbr, nbc, vpb, 2, scores, wg); break;
    case 4: score_direct_body<T, V, 4, LOOSE>(X, M, K, ldx, br, bc, nbr, nbc, vpb, 4, scores, wg); break;
    default: score_direct_body<T, V, 8, LOOSE>(X, M, K, ldx, br, bc, nbr, nbc, vpb, 8, scores, wg); break;
  }
}

template <typename T, int V, bool LOOSE>
__global__ __launch_bounds__(kScoreThreads) void score_kernel(
    const T *__restrict__ X, int64_t M, int64_t K, int64_t ldx, int br, int bc, int64_t nbr,
    int64_t nbc, ScoreGeom g, double *__restrict__ scores) {
  if (LOOSE || g.direct) score_direct<T, V, LOOSE>(X, M, K, ldx, br, bc, nbr, nbc, g, scores, blockIdx.x);
  else score_body<T, V>(X, M, K, ldx, br, bc, nbr, nbc, g, scores, blockIdx.x, blockIdx.y, gridDim.y);
}

// Several tensors per launch: workgroup w belongs to the tensor whose range of
// workgroups holds w; the tensors' parameters come with the kernel arguments.
constexpr int kScoreBatchMax = 24;
struct ScoreItem {
  const void *X;
  double *scores;
  int64_t M, K, ldx, nbr, nbc;
  int br, bc;
  ScoreGeom g;
  uint32_t wg_begin, gy;
};
struct ScoreBatch {
  ScoreItem it[kScoreBatchMax];
};

template <typename T, int V, bool LOOSE>
__global__ __launch_bounds__(kScoreThreads) void score_batched_kernel(ScoreBatch b, int n) {
  int i = 0;
  while (i + 1 < n && blockIdx.x >= b.it[i + 1].wg_begin) ++i;
  const ScoreItem &it = b.it[i];
  const uint32_t local = blockIdx.x - it.wg_begin;
  if (LOOSE || it.g.direct) {
    score_direct<T, V, LOOSE>(static_cast<const T *>(it.X), it.M, it.K, it.ldx, it.br, it.bc, it.nbr, it.nbc, it.g, it.scores,
                            local);
    return;
  }
  score_body<T, V>(static_cast<const T *>(it.X), it.M, it.K, it.ldx, it.br, it.bc, it.nbr, it.nbc, it.g, it.scores,
                   local % (uint32_t)it.g.nchunks, local / (uint32_t)it.g.nchunks, it.gy);
}

// Narrow blocks (rows shorter than a 16-byte vector, e.g. 14x14 patches) and blocks
// of few rows (1 x b row segments) on contiguous matrix rows: a workgroup reads the rows of g.rb block-rows as one
// linear span into LDS, then a thread per (matrix row, block-column, piece of 32
// elements) adds that piece's squares left to right, and a thread per block adds
// the pieces row by row.  LDS layout: span | partial sums (binary64).
template <typename T, typename V>
__device__ __forceinline__ void score_span_body(const uint8_t *__restrict__ X, int64_t M, int64_t K, int bc,
                                                int64_t nbr, const SpanGeom &g, size_t span_words, int pieces,
                                                uint32_t magic_pieces, double *__restrict__ scores,
                                                uint32_t wg) {
  constexpr int kVecs = kSpanBytes / (int)sizeof(V) / 256;
  extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
  double *part = reinterpret_cast<double *>(lds + span_words);
  const int t = threadIdx.x;
  const int64_t i0 = (int64_t)wg * g.rb;
  const int nb = (int)((nbr - i0) < g.rb ? (nbr - i0) : g.rb);
  const int64_t m0 = i0 * g.br;
  const int rows = (int)((M - m0) < (int64_t)nb * g.br ? (M - m0) : (int64_t)nb * g.br);
  const int nvec = rows * g.row_words * 4 / (int)sizeof(V);
  const V *src = reinterpret_cast<const V *>(X + m0 * g.row_words * 4);
  V reg[kVecs];
  // (no load is under a condition: behind the span's end the last vector again)
#pragma unroll
  for (int k = 0; k < kVecs; ++k) reg[k] = src[t + 256 * k < nvec ? t + 256 * k : nvec - 1];
  V *sv = reinterpret_cast<V *>(lds);
#pragma unroll
  for (int k = 0; k < kVecs; ++k)
    if (t + 256 * k < nvec) sv[t + 256 * k] = reg[k];
  __syncthreads();
  const int kk = (int)K;
  // a row segment is summed in pieces of 32 elements (`pieces` per segment)
  for (int pc = t; pc < rows * g.nbc * pieces; pc += 256) {
    const uint32_t pair = span_div((uint32_t)pc, (uint32_t)pieces, magic_pieces), sub = (uint32_t)pc - pair * pieces;
    const uint32_t row = span_div(pair, (uint32_t)g.nbc, g.magic_nbc), j = pair - row * g.nbc;
    const int c0 = (int)j * bc + (int)sub * 32;
    int c1 = c0 + 32 < (int)(j + 1) * bc ? c0 + 32 : (int)(j + 1) * bc;
    if (c1 > kk) c1 = kk;
    double acc = 0.0;
    if constexpr (sizeof(T) == 2) {
      // (rows and segments are whole words here: two elements per LDS read)
      const uint32_t *p = lds + (int)row * (kk >> 1) + (c0 >> 1);
      const int n = (c1 - c0) >> 1;
#pragma unroll 4
      for (int c = 0; c < n; ++c) {
        const uint32_t v = p[c];
        const double lo = (double)__uint_as_float(v << 16), hi = (double)__uint_as_float(v & 0xFFFF0000u);
        acc = fma(lo, lo, acc);
        acc = fma(hi, hi, acc);
      }
    } else {
      const T *p = reinterpret_cast<const T *>(lds) + (int)row * kk;
      for (int c = c0; c < c1; ++c) {
        const double x = (double)elem_to_float<T>(p[c]);
        acc = fma(x, x, acc);
      }
    }
    part[pc] = acc;
  }
  __syncthreads();
  for (int bj = t; bj < nb * g.nbc; bj += 256) {
    const uint32_t b = span_div((uint32_t)bj, (uint32_t)g.nbc, g.magic_nbc), j = (uint32_t)bj - b * g.nbc;
    const int r1 = rows - (int)b * g.br < g.br ? rows - (int)b * g.br : g.br;
    double sum = 0.0;
    for (int r = 0; r < r1; ++r)
      for (int u = 0; u < pieces; ++u) sum += part[(((int)b * g.br + r) * g.nbc + (int)j) * pieces + u];
    scores[(i0 + b) * g.nbc + j] = sum;
  }
}

template <typename T, typename V>
__global__ __launch_bounds__(256) void score_span_kernel(const uint8_t *__restrict__ X, int64_t M, int64_t K,
                                                         int bc, int64_t nbr, SpanGeom g, size_t span_words,
                                                         int pieces, uint32_t magic_pieces,
                                                         double *__restrict__ scores) {
  score_span_body<T, V>(X, M, K, bc, nbr, g, span_words, pieces, magic_pieces, scores, blockIdx.x);
}

struct SpanScoreItem {
  const uint8_t *X;
  double *scores;
  int64_t M, K, nbr;
  SpanGeom g;
  uint32_t span_words, magic_pieces;
  int bc, pieces;
  uint32_t wg_begin;
};
struct SpanScoreBatch {
  SpanScoreItem it[kScoreBatchMax];
};

template <typename T, typename V>
__global__ __launch_bounds__(256) void score_span_batched_kernel(SpanScoreBatch b, int n) {
  int i = 0;
  while (i + 1 < n && blockIdx.x >= b.it[i + 1].wg_begin) ++i;
  const SpanScoreItem &it = b.it[i];
  score_span_body<T, V>(it.X, it.M, it.K, it.bc, it.nbr, it.g, it.span_words, it.pieces, it.magic_pieces, it.scores,
                        blockIdx.x - it.wg_begin);
}

// Few-row blocks whose row segments are whole 16-byte vectors (1 x b row segments):
// the same span of g.rb block-rows, but every lane keeps its vectors in registers
// and only their sums of squares go to LDS; a thread per block then adds the
// vectors of its segments left to right, row by row.
template <typename T>
__global__ __launch_bounds__(256) void score_rows_kernel(const uint8_t *__restrict__ X, int64_t M, int bc,
                                                         int64_t nbr, SpanGeom g, double *__restrict__ scores) {
  constexpr int VE = 16 / (int)sizeof(T);
  constexpr int kVecs = kSpanBytes / 16 / 256;
  __shared__ double part[kSpanBytes / 16];
  const int t = threadIdx.x;
  const int64_t i0 = (int64_t)blockIdx.x * g.rb;
  const int nb = (int)((nbr - i0) < g.rb ? (nbr - i0) : g.rb);
  const int64_t m0 = i0 * g.br;
  const int rows = (int)((M - m0) < (int64_t)nb * g.br ? (M - m0) : (int64_t)nb * g.br);
  const int rv = g.row_words / 4;                        // vectors per matrix row
  const int nvec = rows * rv;
  const Raw<T, VE> *src = reinterpret_cast<const Raw<T, VE> *>(X + m0 * g.row_words * 4);
  Raw<T, VE> reg[kVecs];
  // (no load is under a condition: behind the span's end the last vector again)
#pragma unroll
  for (int k = 0; k < kVecs; ++k) reg[k] = src[t + 256 * k < nvec ? t + 256 * k : nvec - 1];
#pragma unroll
  for (int k = 0; k < kVecs; ++k) {
    if (t + 256 * k < nvec) {
      double acc = 0.0;
#pragma unroll
      for (int q = 0; q < VE; ++q) {
        const double x = (double)raw_elem<T, VE>(reg[k], q);
        acc = fma(x, x, acc);
      }
      part[t + 256 * k] = acc;
    }
  }
  __syncthreads();
  const int vps = bc / VE;                               // vectors per row segment
  for (int bj = t; bj < nb * g.nbc; bj += 256) {
    const uint32_t b = span_div((uint32_t)bj, (uint32_t)g.nbc, g.magic_nbc), j = (uint32_t)bj - b * g.nbc;
    const int r1 = rows - (int)b * g.br < g.br ? rows - (int)b * g.br : g.br;
    const int u1 = rv - (int)j * vps < vps ? rv - (int)j * vps : vps;       // ragged last block-column
    double sum = 0.0;
    for (int r = 0; r < r1; ++r)
      for (int u = 0; u < u1; ++u) sum += part[((int)b * g.br + r) * rv + (int)j * vps + u];
    scores[(i0 + b) * g.nbc + j] = sum;
  }
}

template <typename T>
int run_score_span(const void *X, int64_t M, int64_t K, int bc, const SpanGeom &g, double *scores,
                   hipStream_t s) {
  const int64_t nbr = ceil_div(M, g.br);
  if (g.vb == 16 && g.seg_words % 4 == 0) {
    hipLaunchKernelGGL((score_rows_kernel<T>), dim3((unsigned)ceil_div(nbr, g.rb)), dim3(256), 0, s,
                       static_cast<const uint8_t *>(X), M, bc, nbr, g, scores);
    return check_launch();
  }
  const size_t span_words = align_up((size_t)g.rb * g.br * g.row_words, 4);
  const int pieces = (bc + 31) / 32;
  const uint32_t magic_pieces = (uint32_t)(((uint64_t(1) << 32) + pieces - 1) / pieces);
  const size_t lds = span_words * 4 + (size_t)g.rb * g.br * g.nbc * pieces * sizeof(double);
  const dim3 grid((unsigned)ceil_div(nbr, g.rb));
  const uint8_t *x = static_cast<const uint8_t *>(X);
  switch (g.vb) {
    case 16:
      hipLaunchKernelGGL((score_span_kernel<T, RawWords<16>::type>), grid, dim3(256), lds, s, x, M, K, bc, nbr, g, span_words, pieces, magic_pieces, scores);
      break;
    case 8:
      hipLaunchKernelGGL((score_span_kernel<T, RawWords<8>::type>), grid, dim3(256), lds, s, x, M, K, bc, nbr, g, span_words, pieces, magic_pieces, scores);
      break;
    default:
      hipLaunchKernelGGL((score_span_kernel<T, uint32_t>), grid, dim3(256), lds, s, x, M, K, bc, nbr, g, span_words, pieces, magic_pieces, scores);
      break;
  }
  return check_launch();
}

// Launch geometry of score_kernel for vectors of V elements in a launch of `tensors` tensors; *gy = passes of
// the grid.  loose: of its form for any alignment, which has the direct body only (direct == 0: not for this matrix).
ScoreGeom score_geometry(int V, int64_t M, int64_t K, int br, int bc, int tensors, int64_t *gy_out, bool loose = false) {
  const int64_t nbr = ceil_div(M, br), nbc = ceil_div(K, bc);
  ScoreGeom g;
  int vpb = bc / V;
  if (loose)
    for (vpb = 1; vpb * V < bc;) vpb *= 2;
  g.direct = 0;
  // large matrices take the direct body: rs lanes share a vector column of a block so that the
  // tensor has at least `want` lanes, and every lane still has a few rows.  A tensor on its own wants
  // 256 Ki lanes, half of what the chip holds: with 64 Ki the loads on their way (8 x 16 bytes a lane)
  // do not cover the latency of HBM ([25088 x 384] bf16, 32x32 blocks: 10.9 us with 64 Ki lanes, 8.5 with
  // 128 Ki, 6.8 with 256 Ki, 7.1 with 512 Ki; [25088 x 1536]: 22.4 / 22.8 / 16.7 / 18.7).  Tensors that
  // share a launch fill the chip together, and more lanes a block only cost exchanges there (24 tensors:
  // 188 us with 64 Ki lanes each, 202 with 128 Ki).
  if (vpb >= 1 && vpb <= 64 && (vpb & (vpb - 1)) == 0 && (loose || vpb * V == bc)) {
    int64_t want = 262144 / tensors;
    if (want < 65536) want = 65536;
    int rs = 1;
    while (nbr * nbc * vpb * rs < want && vpb * rs * 2 <= 64 && rs * 2 * 4 <= br && rs < kRowClasses) rs *= 2;
    // (tall blocks: the same rs in a launch of one tensor and of many, since it decides the order of the additions)
    const bool tall = br >= 128 && rs == kRowClasses && nbr * nbc * vpb * rs < 65536;
    while (tall && nbr * nbc * vpb * rs < 65536 && vpb * rs * 2 <= 64 && rs * 2 * 4 <= br) rs *= 2;
    const int64_t lanes = nbr * nbc * vpb * rs;
    // (loose, tall blocks: more lanes, or the LDS body, whose row groups share a block, is the faster one; [949 x 1428] in 64x64
    // blocks, 22080 lanes: score and select 9.3 us there, 11.4 so, [912 x 1299] in 14x14, 24552 lanes: 15.3 and 11.6)
    if (lanes >= (loose && br >= 64 ? 32768 : 16384) && lanes < (int64_t(1) << 31)) {
      g.direct = tall ? 2 : 1;
      g.jc = g.vct = g.rb = 1;
      g.vpbt = vpb;
      g.gb = rs;
      g.nchunks = (int)ceil_div(lanes, (int64_t)kScoreThreads);
      *gy_out = 1;
      return g;
    }
  }
  g.vpbt = vpb < kScoreThreads ? vpb : kScoreThreads;
  // about one wave across the chunk (a 1 KB row segment per load instruction), the
  // other waves of the workgroup as row groups: many workgroups, few rows per
  // thread, so that all of a thread's loads are in flight at once
  // (a matrix row of at most two waves stays in one piece)
  g.jc = g.vpbt >= 64 ? 1 : 64 / g.vpbt;
  if (nbc * g.vpbt <= 128 || g.jc > nbc) g.jc = (int)nbc;
  g.vct = g.jc * g.vpbt;
  const int groups = kScoreThreads / g.vct;      // >= 1
  g.gb = groups < br ? groups : br;
  g.rb = groups / g.gb;
  if (g.rb > nbr) g.rb = (int)nbr;
  g.nchunks = (int)ceil_div(nbc, g.jc);
  const int64_t passes = ceil_div(nbr, g.rb);
  // enough workgroups to fill 256 CUs several times over, bounded so that a
  // workgroup of a very tall matrix loops instead of flooding the dispatcher
  int64_t gy = passes;
  const int64_t cap = ceil_div(16384, g.nchunks);
  if (gy > cap) gy = cap;
  if (gy > 65535) gy = 65535;
  *gy_out = gy;
  return g;
}

template <typename T, int V, bool LOOSE>
int run_score(const void *X, int64_t M, int64_t K, int64_t ldx, int br, int bc, double *scores,
              hipStream_t s) {
  const int64_t nbr = ceil_div(M, br), nbc = ceil_div(K, bc);
  int64_t gy;
  const ScoreGeom g = score_geometry(V, M, K, br, bc, 1, &gy, LOOSE);
  dim3 grid((unsigned)g.nchunks, (unsigned)gy, 1);
  hipLaunchKernelGGL((score_kernel<T, V, LOOSE>), grid, dim3(g.direct ? kScoreThreads : g.vct * g.gb * g.rb), 0, s,
                     static_cast<const T *>(X), M, K, ldx, br, bc, nbr, nbc, g, scores);
  return check_launch();
}

// Whether the form for any alignment is the faster one, where its direct body has lanes enough; `key`: elements of the plain form's
// vectors, `direct`: which body that form takes.  A block row that is one plain load gains nothing (16 bytes, masked, for the same).  Else
// it saves loads, the more the lower the blocks: tall ones have lanes enough for loads of 2 or 4 bytes by consecutive lanes, and
// the LDS body's lanes fit widths of an odd number of vectors well.  Over 3300 pairs of heights 1 .. 128, widths 1 .. 256 and pitches
// at two sizes of either type.  Score and select, in us, plain and so: bfloat16 [25088 x 1536] in 64x1 blocks 41 and 112,
// 16x4 33 and 39, 64x5 34 and 43, 64x18 27 and 31; with a pitch of 1537: 128x4 38 and 89, 64x8 32 and 40, 32x8 38 and 37, 32x14 49 and 32;
// binary32 [25088 x 768]: 64x1 30 and 53, 64x9 36 and 40, 64x30 34 and 37, with a pitch of 769 64x14 41 and 30.
bool loose_pays(int dtype, int br, int bc, int key, bool direct) {
  if (key >= bc) return false;
  const bool spread = key == 1 || bc / key % 2 == 0;         // (rows out of step with the width, not the width itself)
  if (dtype == BSR_F32) {
    if (direct) return br >= 64 && bc >= 4;
    if (br >= 64) return bc >= 10 && spread;
    return br <= 16 || key == 1 || bc > 6;
  }
  if (direct) {
    if (br > 16) return bc >= (br < 64 ? 8 : 16);
    return bc >= 8 || (bc == 4 ? key == 1 || br <= 8 : br <= 4);
  }
  if (br >= 64) return bc >= 14 && (spread || (key == 2 && bc >= 20));
  return br <= 16 || (bc >= 5 && key < 4) || bc >= 20;
}

// Which kernel scores a tensor: 0 = score_kernel with vectors of `key` elements (kLoose: its form for any alignment),
// 1 = score_span_kernel with `key`-byte accesses, 2 = score_rows_kernel.
constexpr int kLoose = 100;
int score_kind(int dtype, const void *X, int64_t M, int64_t K, int64_t ldx, int br, int bc, SpanGeom *g, int *key) {
  // (partial sums in LDS: at most 48 KB of binary64 beside the span)
  if (span_geometry(dtype, M, K, ldx, br, bc, X, nullptr, g) &&
      (int64_t)g->rb * br * g->nbc * ((bc + 31) / 32) <= 6144) {
    *key = g->vb;
    return (g->vb == 16 && g->seg_words % 4 == 0) ? 2 : 1;
  }
  const int v = dtype == BSR_F32 ? 4 : 8;
  *key = pick_vector(v, elem_bytes(dtype), bc, K, ldx, X);
  int64_t gy;
  if (*key == v || (M - 1) * ldx + K < v || !score_geometry(v, M, K, br, bc, 1, &gy, true).direct) return 0;
  if (loose_pays(dtype, br, bc, *key, score_geometry(*key, M, K, br, bc, 1, &gy).direct != 0)) *key = kLoose;
  return 0;
}

template <typename T>
int launch_generic_batch(const ScoreBatch &b, int n, uint32_t wgs, int v, hipStream_t s) {
  const dim3 grid(wgs), block(kScoreThreads);
  if (sizeof(T) == 4) {
    switch (v) {
      case kLoose: hipLaunchKernelGGL((score_batched_kernel<float, 4, true>), grid, block, 0, s, b, n); break;
      case 4: hipLaunchKernelGGL((score_batched_kernel<float, 4, false>), grid, block, 0, s, b, n); break;
      case 2: hipLaunchKernelGGL((score_batched_kernel<float, 2, false>), grid, block, 0, s, b, n); break;
      default: hipLaunchKernelGGL((score_batched_kernel<float, 1, false>), grid, block, 0, s, b, n); break;
    }
  } else {
    switch (v) {
      case kLoose: hipLaunchKernelGGL((score_batched_kernel<uint16_t, 8, true>), grid, block, 0, s, b, n); break;
      case 8: hipLaunchKernelGGL((score_batched_kernel<uint16_t, 8, false>), grid, block, 0, s, b, n); break;
      case 4: hipLaunchKernelGGL((score_batched_kernel<uint16_t, 4, false>), grid, block, 0, s, b, n); break;
      case 2: hipLaunchKernelGGL((score_batched_kernel<uint16_t, 2, false>), grid, block, 0, s, b, n); break;
      default: hipLaunchKernelGGL((score_batched_kernel<uint16_t, 1, false>), grid, block, 0, s, b, n); break;
    }
  }
  return check_launch();
}

template <typename T>
int launch_span_batch(const SpanScoreBatch &b, int n, uint32_t wgs, size_t lds, int vb, hipStream_t s) {
  const dim3 grid(wgs), block(256);
  switch (vb) {
    case 16: hipLaunchKernelGGL((score_span_batched_kernel<T, RawWords<16>::type>), grid, block, lds, s, b, n); break;
    case 8: hipLaunchKernelGGL((score_span_batched_kernel<T, RawWords<8>::type>), grid, block, lds, s, b, n); break;
    default: hipLaunchKernelGGL((score_span_batched_kernel<T, uint32_t>), grid, block, lds, s, b, n); break;
  }
  return check_launch();
}

}  // namespace

int launch_score(const void *X, int dtype, int64_t M, int64_t K, int64_t ldx, int br, int bc,
                 double *scores, hipStream_t s) {
  if (M == 0 || K == 0) return BSR_OK;
  SpanGeom g;
  int key;
  if (score_kind(dtype, X, M, K, ldx, br, bc, &g, &key) != 0)
    return dtype == BSR_F32 ? run_score_span<float>(X, M, K, bc, g, scores, s)
                            : run_score_span<uint16_t>(X, M, K, bc, g, scores, s);
  if (dtype == BSR_F32) {
    switch (key) {
      case kLoose: return run_score<float, 4, true>(X, M, K, ldx, br, bc, scores, s);
      case 4: return run_score<float, 4, false>(X, M, K, ldx, br, bc, scores, s);
      case 2: return run_score<float, 2, false>(X, M, K, ldx, br, bc, scores, s);
      default: return run_score<float, 1, false>(X, M, K, ldx, br, bc, scores, s);
    }
  }
  switch (key) {
    case kLoose: return run_score<uint16_t, 8, true>(X, M, K, ldx, br, bc, scores, s);
    case 8: return run_score<uint16_t, 8, false>(X, M, K, ldx, br, bc, scores, s);
    case 4: return run_score<uint16_t, 4, false>(X, M, K, ldx, br, bc, scores, s);
    case 2: return run_score<uint16_t, 2, false>(X, M, K, ldx, br, bc, scores, s);
    default: return run_score<uint16_t, 1, false>(X, M, K, ldx, br, bc, scores, s);
  }
}

bool score_order(const void *X, int dtype, int64_t M, int64_t K, int64_t ldx, int br, int bc, ScoreOrder *o) {
  SpanGeom sg;
  int key;
  const int v = dtype == BSR_F32 ? 4 : 8, kind = score_kind(dtype, X, M, K, ldx, br, bc, &sg, &key);
  if (kind == 2) {                                           // score_rows_kernel: vectors of 16 bytes, row by row
    *o = ScoreOrder{br, v, bc / v, v, false};
    return true;
  }
  if (kind == 1) {                                           // score_span_body: pieces of 32 elements, row by row
    *o = ScoreOrder{br, 32, (int)ceil_div(bc, 32), v, true};
    return (M - 1) * ldx + K >= v;
  }
  if (key == kLoose) return false;
  int64_t gy;
  const ScoreGeom g = score_geometry(key, M, K, br, bc, 1, &gy);
  if (g.direct || g.vpbt * key != bc) return false;
  *o = ScoreOrder{g.gb, key, g.vpbt, key, false};            // score_body
  return true;
}

int launch_score_batched(const ScoreJob *jobs, int n, int dtype, hipStream_t s) {
  // tensors that take the same kernel instance share launches of up to kScoreBatchMax tensors
  static const int kKeys[2][5] = {{kLoose, 8, 4, 2, 1}, {16, 8, 4, 0, 0}};
  for (int kind = 0; kind < 2; ++kind) {
    for (int ki = 0; ki < 5; ++ki) {
      const int want_key = kKeys[kind][ki];
      if (want_key == 0) continue;
      ScoreBatch gb;
      SpanScoreBatch sb;
      int m = 0;
      uint32_t wgs = 0;
      size_t lds = 0;
      auto flush = [&]() -> int {
        if (m == 0) return BSR_OK;
        int rc;
        if (kind == 0)
          rc = dtype == BSR_F32 ? launch_generic_batch<float>(gb, m, wgs, want_key, s)
                                : launch_generic_batch<uint16_t>(gb, m, wgs, want_key, s);
        else
          rc = dtype == BSR_F32 ? launch_span_batch<float>(sb, m, wgs, lds, want_key, s)
                                : launch_span_batch<uint16_t>(sb, m, wgs, lds, want_key, s);
        m = 0;
        wgs = 0;
        lds = 0;
        return rc;
      };
      for (int i = 0; i < n; ++i) {
        const ScoreJob &j = jobs[i];
        if (j.M == 0 || j.K == 0) continue;
        SpanGeom g;
        int key;
        const int k = score_kind(dtype, j.X, j.M, j.K, j.ldx, j.br, j.bc, &g, &key);
        if (k == 2) {                                        // register-resident row segments: one by one
          if (kind == 0 && ki == 0) {
            const int rc = launch_score(j.X, dtype, j.M, j.K, j.ldx, j.br, j.bc, j.scores, s);
            if (rc != BSR_OK) return rc;
          }
          continue;
        }
        if (k != kind || key != want_key) continue;
        const int64_t nbr = ceil_div(j.M, j.br), nbc = ceil_div(j.K, j.bc);
        if (kind == 0) {
          ScoreItem &it = gb.it[m];
          int64_t gy;
          it.g = score_geometry(key == kLoose ? (dtype == BSR_F32 ? 4 : 8) : key, j.M, j.K, j.br, j.bc, n, &gy, key == kLoose);
          it.X = j.X;
          it.scores = j.scores;
          it.M = j.M; it.K = j.K; it.ldx = j.ldx; it.nbr = nbr; it.nbc = nbc;
          it.br = j.br; it.bc = j.bc;
          it.wg_begin = wgs;
          it.gy = (uint32_t)gy;
          wgs += (uint32_t)(it.g.nchunks * gy);
        } else {
          SpanScoreItem &it = sb.it[m];
          it.g = g;
          it.X = static_cast<const uint8_t *>(j.X);
          it.scores = j.scores;
          it.M = j.M; it.K = j.K; it.nbr = nbr;
          it.bc = j.bc;
          it.pieces = (j.bc + 31) / 32;
          it.magic_pieces = (uint32_t)(((uint64_t(1) << 32) + it.pieces - 1) / it.pieces);
          it.span_words = (uint32_t)align_up((size_t)g.rb * g.br * g.row_words, 4);
          const size_t need = (size_t)it.span_words * 4 + (size_t)g.rb * g.br * g.nbc * it.pieces * sizeof(double);
          if (need > lds) lds = need;
          it.wg_begin = wgs;
          wgs += (uint32_t)ceil_div(nbr, g.rb);
        }
        if (++m == kScoreBatchMax) {
          const int rc = flush();
          if (rc != BSR_OK) return rc;
        }
      }
      const int rc = flush();
      if (rc != BSR_OK) return rc;
    }
  }
  return BSR_OK;
}

}  // namespace bsr
