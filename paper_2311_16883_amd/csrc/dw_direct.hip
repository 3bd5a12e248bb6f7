// Weight gradient from a BSR activation, one product per launch, without shared tiles in LDS and without a barrier in the main
// loop: each wave gathers kept blocks and the rows of dY that they meet.  bfloat16 and binary32, 14x14, 16x16, 32x32 and
// 64x64 blocks, and row segments of whole 32 columns (1x32, 1x64, ...), of which a wave takes 16 kept ones at a time.
//
// A workgroup owns one strip of IW rows of dW (all of a block-column, half of a 64-wide one) and IW * NS columns, for a
// contiguous range of block-rows.  It lists the blocks that this strip keeps in its range, and its W waves take 16-row
// units of them in turn: pruned blocks cost nothing, not even their rows of dY, and a 14- or 16-wide block is skipped by
// itself (32-wide tiles hold two or three of them, of which one is kept in 75 .. 90 % of the cases at keep 0.5).  The
// waves' sums meet in LDS at the end.  Few tiles: many waves with few columns each, so that a small product needs no
// second launch; many tiles: four waves with 128 columns each, and splits of the contraction over workgroups where
// compute units would be idle.
//
// binary32: the matrix instructions contract two (32x32x2) or four (16x16x4) activation rows and want one element per
// lane and operand: lane l supplies column l % IW of row l / IW.  A kept block and rows of dY lie in memory just so,
// and which column of dW a lane's dY element stands for is free as long as the store knows it: a lane loads VQ
// consecutive columns of dY in one instruction and feeds element q to its q-th tile, so that the columns
// VQ * i + q (i = 0 .. IW - 1) form tile q, and a lane's results are VQ consecutive columns as well.  Per step a wave
// issues one 4-byte load of the activation, one 16-byte load of dY and four matrix instructions.  Small products are bound by
// latency (list, loads, sums, each a trip or two to memory: 6 us for [256 x 128 x 64], 9.7 in 128 x 128 tiles), larger ones by the
// matrix cores and by what reaches a compute unit, 48 bytes per ns; where most blocks are kept the tiles, which load less for
// each multiply-add, take those ([12544 x 768 x 768] in 16x16 blocks, keep 0.9: 144 us so, 122 there).
//
// bfloat16: a lane's operand is eight (16-wide tiles: four) elements of one column, so a unit goes through a small tile of LDS that belongs to
// the wave alone and comes back through transposing reads.  Bound by latency ([1202 x 152 x 446] 7.1 us, 12.7 in the tiles) and by
// the loads, 160 rows and columns for each 32 x 128 multiply-adds.
//
// Row segments: the rows of a unit are any 16 that keep a segment in this strip, so nothing pruned is multiplied and no re-tiled
// copy is written ([742 x 96 x 2848] in 1x64 blocks, keep 0.1: 7.9 us, 15.6 re-tiled).  Finding them takes a walk over all entries
// of the workgroup's rows.
#include <type_traits>

#include "buffer_access.h"
#include "common.h"

namespace bsr {

namespace {

typedef __attribute__((ext_vector_type(4))) short v4s;
typedef __attribute__((ext_vector_type(8))) short v8s;
typedef __attribute__((ext_vector_type(8))) __bf16 v8bf;
typedef __attribute__((ext_vector_type(4))) float v4f;
typedef __attribute__((ext_vector_type(16))) float v16f;

constexpr uint32_t kDead = 0x80000000u;     // offset in `values` that reads as zero (they stay below 2 GiB)
// block-rows of a split: its list of kept blocks is in LDS
constexpr int max_rows(int br) { return br == 1 ? 4096 : 1024; }
constexpr int kUnit = 16;                   // rows of a block that a wave takes at a time

template <int BYTES> struct Words;
template <> struct Words<16> { typedef u32x4 type; };
template <> struct Words<8> { typedef u32x2 type; };
template <> struct Words<4> { typedef uint32_t type; };

template <int WORDS>
__device__ __forceinline__ typename Words<4 * WORDS>::type load_words(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  if constexpr (WORDS == 4) return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
  else if constexpr (WORDS == 2) return __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
  else return __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
}
template <int WORDS>
__device__ __forceinline__ float word(const typename Words<4 * WORDS>::type &v, int q) {
  if constexpr (WORDS == 1) return __uint_as_float(v);
  else return __uint_as_float(v[q]);
}

// 16 bytes from any 2-byte boundary
struct __attribute__((packed, aligned(2))) LooseVec {
  u32x4 v;
};

// Columns 16-wide group by 16-wide group transposed out of an LDS tile of bfloat16: 4 rows x 16 columns for each 16 lanes.
__device__ __forceinline__ v4s read_transposed(const uint16_t *p) {
  typedef v4s __attribute__((address_space(3))) * lds_v4s;
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(p));
}
// Place of (row, col) in a wave's tile of COLS columns: the 32-byte chunks of a row are permuted so that the four rows that a
// transposing read takes lie in different banks (rows of 64 bytes and less do by themselves).
template <int COLS>
__device__ __forceinline__ int tile_place(int row, int col) {
  const int chunk = COLS == 128 ? (row & 3) << 1 : COLS == 64 ? (row >> 1) & 1 : 0;
  return row * COLS + (((col >> 4) ^ chunk) << 4 | (col & 15));
}

// WORDS consecutive floats at any 4-byte boundary
template <int WORDS>
struct __attribute__((packed, aligned(4))) Floats {
  float v[WORDS];
};

template <typename T, int BR, int BC, int NS>
struct Geo {
  static constexpr int E = (int)sizeof(T);
  static constexpr int IW = BC % 32 == 0 ? 32 : 16;     // rows and columns of a tile of dW
  static constexpr int KS = 64 / IW;                    // activation rows of one instruction
  static constexpr int STEPS = kUnit / KS;
  static constexpr int UPB = BR > kUnit ? BR / kUnit : 1;   // units of a block
  static constexpr bool SEGMENTS = BR == 1;             // row segments: a unit is 16 of them; BC stands for a part of 32 columns
  static constexpr int SPB = BC > 32 ? BC / 32 : 1;         // strips of a block-column
  // binary32: columns of a dY load, consecutive ones, and loads of a step; a lane's results are as many consecutive columns
  static constexpr int VQ = E == 2 ? 1 : NS < 4 ? NS : 4;
  static constexpr int NG = NS / VQ;
  static constexpr int REGS = IW == 32 ? 16 : 4;        // results per lane and tile
  static constexpr int COLS = IW * NS;
  // bfloat16: bytes of an activation load, dY loads of a unit, and a wave's tiles of both in LDS (elements)
  static constexpr int ABYTES = IW / 2, BLOADS = kUnit * COLS / (64 * 8);
  static constexpr int TILES = E == 2 ? kUnit * (IW + COLS) : 0;
  static_assert(BR <= kUnit || BR % kUnit == 0, "whole units");
  static_assert(BR != 1 || BC == 32, "parts of segments");
  static_assert(BC <= 16 || BC % 32 == 0, "a strip lies in one block-column");
};

struct DirectParams {
  const int32_t *row_ptr, *col_idx;
  const void *values, *dY;
  float *out;
  int64_t M, K, N, lddy, ldo, split_stride, nbr, nbc;
  int rows_per_split, strips, tiles_n, splits, accumulate, bc;
};

// D: units of a wave whose loads are on their way or being multiplied.
// ODD (bfloat16): rows of dY may start or end on odd elements.
template <typename T, int BR, int BC, int NS, int W, int D, int WAVES, bool ODD>
__global__ __launch_bounds__(64 * W, WAVES) void dw_direct_kernel(DirectParams prm) {
  typedef Geo<T, BR, BC, NS> G;
  constexpr int E = G::E;
  static_assert(!ODD || E == 2, "binary32 rows start on whole words");
  constexpr int kThreads = 64 * W, R = NS * G::REGS;
  // (results that the waves exchange at a time: 32 KB of them, so that three workgroups of four waves share a compute unit)
  constexpr int kPart = W * R * 256 > 32768 ? 32768 / (W * 256) : R;
  static_assert(R % kPart == 0 && kPart % G::VQ == 0, "whole parts of whole vectors");
  constexpr int kSumWords = W * kPart * 64 > W * G::TILES / 2 ? W * kPart * 64 : W * G::TILES / 2;
  constexpr int kMaxRows = max_rows(BR);
  __shared__ __attribute__((aligned(16))) float sSum[kSumWords > kMaxRows + 1 ? kSumWords : kMaxRows + 1];
  __shared__ uint2 sUnit[kMaxRows];          // kept blocks of the strip: offset in `values`, first row of dY
  __shared__ int sCount[4 * W];
  int32_t *const sRow = reinterpret_cast<int32_t *>(sSum);   // (until the main loop)

  // XCD x (workgroup id % 8) takes the x-th eighth of the work items, split by split: the tiles of a split read the same
  // rows, which its L2 then fetches once
  const int items = prm.strips * prm.tiles_n * prm.splits, per_xcd = (items + 7) / 8;
  const int item = (int)(blockIdx.x & 7u) * per_xcd + (int)(blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per_xcd || item >= items) return;
  const int split = item / (prm.strips * prm.tiles_n), tile = item % (prm.strips * prm.tiles_n);
  const int strip = tile % prm.strips, tile_n = tile / prm.strips;
  // block-column, first column inside it
  const int spb = G::SEGMENTS ? prm.bc / 32 : G::SPB, bc = G::SEGMENTS ? prm.bc : BC;
  const int j = strip / spb, sub = (strip % spb) * 32;
  const int64_t n0 = (int64_t)tile_n * G::COLS;
  const int64_t i_begin = (int64_t)split * prm.rows_per_split;
  int nrows = prm.rows_per_split;
  if (i_begin + nrows > prm.nbr) nrows = (int)(prm.nbr - i_begin);
  if (nrows < 0) nrows = 0;

  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int64_t last = (int64_t)__builtin_amdgcn_readfirstlane(prm.row_ptr[prm.nbr]);

  // ---- the strip's kept blocks, in the order of their rows ----
  int kept = 0;
  if constexpr (G::SEGMENTS) {
    // Many rows of few entries: all threads walk the entries together, 16 bytes at a time, and list those of this
    // block-column; which rows they are in is looked up afterwards.
    const int32_t *const rp = prm.row_ptr + i_begin;
    for (int e = t; e <= nrows; e += kThreads) sRow[e] = rp[e];
    const int32_t e0 = rp[0], e1 = rp[nrows];
    typedef int32_t __attribute__((ext_vector_type(4), aligned(4))) Entries;
    constexpr int kTogether = 4;
    for (int32_t base = e0; base < e1; base += kTogether * 4 * kThreads) {
      int32_t c[kTogether][4];
#pragma unroll
      for (int u = 0; u < kTogether; ++u) {
        const int32_t e = base + 4 * (u * kThreads + t);
        if (e + 4 <= e1) {
          const Entries v = *reinterpret_cast<const Entries *>(prm.col_idx + e);
#pragma unroll
          for (int q = 0; q < 4; ++q) c[u][q] = v[q];
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q) c[u][q] = e + q < e1 ? prm.col_idx[e + q] : -1;
        }
      }
      int mine[kTogether];                   // matches of the wave's lanes in front of this one
      const uint64_t in_front = (1ull << lane) - 1ull;
#pragma unroll
      for (int u = 0; u < kTogether; ++u) {
        int before = 0, all = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint64_t m = __ballot(c[u][q] == j);
          before += __popcll(m & in_front);
          all += __popcll(m);
        }
        mine[u] = before;
        if (lane == 0) sCount[u * W + wave] = all;
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < kTogether; ++u) {
        int at = kept;
#pragma unroll
        for (int w = 0; w < W; ++w) {
          at += w < wave ? sCount[u * W + w] : 0;
          kept += sCount[u * W + w];
        }
        at += mine[u];
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (c[u][q] == j && at < kMaxRows) sUnit[at++].x = (uint32_t)(base + 4 * (u * kThreads + t) + q);
      }
      __syncthreads();
    }
    if (kept > nrows) kept = nrows;          // (a row has a column once)
    __syncthreads();                         // (sRow, where there is no entry at all)
    for (int k = t; k < kept; k += kThreads) {
      const int32_t e = (int32_t)sUnit[k].x;
      int lo = 0, hi = nrows;                // sRow[lo] <= e < sRow[hi]
      while (hi - lo > 1) {
        const int mid = (lo + hi) / 2;
        if (sRow[mid] <= e) lo = mid;
        else hi = mid;
      }
      sUnit[k] = make_uint2((uint32_t)e * (uint32_t)(bc * E), (uint32_t)(i_begin + lo));
    }
    __syncthreads();
  } else {
    for (int e = t; e < nrows; e += kThreads) sRow[e] = -1;
    int per_row = 1;                           // lanes that share a block-row: a power of two
    while (per_row < 64 && 2 * per_row * nrows <= kThreads) per_row *= 2;
    __syncthreads();
    for (int rr = t / per_row; rr < nrows; rr += kThreads / per_row) {
      const int32_t p0 = prm.row_ptr[i_begin + rr], p1 = prm.row_ptr[i_begin + rr + 1];
      constexpr int kTogether = 4;
      for (int32_t pb = p0 + (t & (per_row - 1)); pb < p1; pb += kTogether * per_row) {
        int32_t c[kTogether];
#pragma unroll
        for (int u = 0; u < kTogether; ++u) c[u] = pb + u * per_row < p1 ? prm.col_idx[pb + u * per_row] : -1;
#pragma unroll
        for (int u = 0; u < kTogether; ++u)
          if (c[u] == j) sRow[rr] = pb + u * per_row;
      }
    }
    __syncthreads();
    for (int base = 0; base < nrows; base += kThreads) {
      const int rr = base + t;
      const int32_t at = rr < nrows ? sRow[rr] : -1;
      const uint64_t live = __ballot(at >= 0);
      if (lane == 0) sCount[wave] = __popcll(live);
      __syncthreads();
      int before = kept, all = kept;
#pragma unroll
      for (int w = 0; w < W; ++w) {
        before += w < wave ? sCount[w] : 0;
        all += sCount[w];
      }
      if (at >= 0) {
        const int e = before + __popcll(live & ((1ull << lane) - 1ull));
        sUnit[e] = make_uint2((uint32_t)at * (uint32_t)(BR * BC * E), (uint32_t)(i_begin + rr) * (uint32_t)BR);
      }
      kept = all;
      __syncthreads();
    }
  }

  // ---- main loop ----
  const int64_t stored = last < prm.nbr * prm.nbc ? last : prm.nbr * prm.nbc;
  const __amdgpu_buffer_rsrc_t rsrc_a = make_rsrc(prm.values, (uint32_t)stored * (uint32_t)(BR * bc * E));
  const uint32_t dy_bytes = (uint32_t)(((prm.M - 1) * prm.lddy + prm.N) * E);
  const __amdgpu_buffer_rsrc_t rsrc_b = make_rsrc(prm.dY, dy_bytes);
  const int i = lane % G::IW, kr = lane / G::IW;
  const uint32_t pitch = (uint32_t)prm.lddy * (uint32_t)E;
  const int units = G::SEGMENTS ? (kept + kUnit - 1) / kUnit : kept * G::UPB;

  typename std::conditional<G::IW == 32, v16f, v4f>::type acc[NS];
#pragma unroll
  for (int q = 0; q < NS; ++q)
#pragma unroll
    for (int r = 0; r < G::REGS; ++r) acc[q][r] = 0.f;

  // Loads of unit u into ring slot d, and the multiplies of a slot.  (A unit beyond the last: loads that touch no memory, so that
  // their number on the way is known.)
  auto unit_at = [&](int u, uint32_t *ea, uint32_t *row) {
    const bool live = u < units;
    const uint2 e = sUnit[live ? u / G::UPB : 0];
    const uint32_t h = (uint32_t)(u % G::UPB) * kUnit;
    *ea = live ? (uint32_t)__builtin_amdgcn_readfirstlane((int)e.x) + h * (BC * E) : kDead;
    *row = (uint32_t)__builtin_amdgcn_readfirstlane((int)e.y) + h;
    return live;
  };
  // (row segments: each lane looks up its own; beyond the last one nothing is read)
  auto segment_at = [&](int u, int r, bool *live) {
    const int k = u * kUnit + r;
    *live = k < kept;
    return sUnit[*live ? k : 0];
  };
  auto run_units = [&](auto load, auto multiply) {
    if (wave >= units) return;
#pragma unroll
    for (int d = 0; d < D - 1; ++d) load(d, wave + d * W);
    for (int u = wave; u < units; u += D * W) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        if (u + d * W < units) {
          load((d + D - 1) % D, u + (d + D - 1) * W);
          multiply(d);
        }
      }
    }
  };
  if constexpr (E == 4) {
    typedef typename Words<4 * G::VQ>::type BVec;
    const bool col_ok = BC >= G::IW || i < BC;
    const uint32_t a_lane = (uint32_t)((kr * BC + sub + i) * 4);
    const uint32_t b_lane = (uint32_t)kr * pitch + (uint32_t)(n0 + G::VQ * i) * 4u;
    const uint32_t b_step = (uint32_t)G::KS * pitch;
    uint32_t a[D][G::STEPS];
    BVec b[D][G::STEPS][G::NG];
    run_units(
        [&](int d, int u) {
          uint32_t ea = 0, row = 0;
          bool live = true;
          if constexpr (!G::SEGMENTS) live = unit_at(u, &ea, &row);
#pragma unroll
          for (int s = 0; s < G::STEPS; ++s) {
            if constexpr (G::SEGMENTS) {
              const uint2 e = segment_at(u, s * G::KS + kr, &live);
              a[d][s] = load_words<1>(rsrc_a, live ? e.x + (uint32_t)((sub + i) * 4) : kDead);
              const uint32_t at = live ? e.y * pitch + (uint32_t)(n0 + G::VQ * i) * 4u : kOutOfRange;
#pragma unroll
              for (int g = 0; g < G::NG; ++g)
                b[d][s][g] = load_words<G::VQ>(rsrc_b, g == 0 || !live ? at : at + (uint32_t)(g * G::IW * G::VQ * 4));
              continue;
            }
            // rows beyond a block of 14 belong to the next block-row
            const bool row_ok = BR % kUnit == 0 || (s + 1) * G::KS <= BR || s * G::KS + kr < BR;
            a[d][s] = load_words<1>(rsrc_a, col_ok && row_ok ? ea + a_lane + (uint32_t)(s * G::KS * BC * 4) : kDead);
            const uint32_t ob = row_ok && live ? row * pitch + b_lane + (uint32_t)s * b_step : kOutOfRange;
#pragma unroll
            for (int g = 0; g < G::NG; ++g)
              b[d][s][g] = load_words<G::VQ>(rsrc_b, g == 0 || ob == kOutOfRange ? ob : ob + (uint32_t)(g * G::IW * G::VQ * 4));
          }
        },
        [&](int d) {
#pragma unroll
          for (int s = 0; s < G::STEPS; ++s)
#pragma unroll
            for (int q = 0; q < NS; ++q) {
              const float fa = __uint_as_float(a[d][s]), fb = word<G::VQ>(b[d][s][q / G::VQ], q % G::VQ);
              if constexpr (G::IW == 32) acc[q] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa, fb, acc[q], 0, 0, 0);
              else acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa, fb, acc[q], 0, 0, 0);
            }
        });
  } else {
    // A unit goes through a tile of the wave's own in LDS, since a lane's operand is 4 or 8 elements of one column; no other
    // wave touches it, and a wave's LDS accesses are in order.
    typedef typename Chunk<G::ABYTES>::type AVec;
    constexpr int VA = G::ABYTES / 2, LPR = G::IW / VA, CPR = G::COLS / 8;    // vectors per row of either tile
    static_assert(LPR * kUnit == 64, "one activation load per unit");
    uint16_t *const tile_a = reinterpret_cast<uint16_t *>(sSum) + wave * G::TILES, *const tile_b = tile_a + kUnit * G::IW;
    const int ar = lane / LPR, ac = lane % LPR * VA;
    const uint32_t a_lane = ar < BR ? (uint32_t)((ar * BC + sub + ac) * 2) : kDead;
    AVec a[D];
    u32x4 b[D][G::BLOADS];
    uint32_t over[D][G::BLOADS];             // (ODD: bytes by which the load was held back from the end of dY)
    const char *const dy = static_cast<const char *>(prm.dY);
    const int br = lane / CPR, bcol = lane % CPR * 8;
    run_units(
        [&](int d, int u) {
          uint32_t ea = 0, row = 0;
          bool live = true;
          if constexpr (G::SEGMENTS) {
            const uint32_t at = segment_at(u, ar, &live).x;
            a[d] = buffer_load<G::ABYTES>(rsrc_a, live ? at + (uint32_t)((sub + ac) * 2) : kDead);
          } else {
            live = unit_at(u, &ea, &row);
            a[d] = buffer_load<G::ABYTES>(rsrc_a, a_lane == kDead ? kDead : ea + a_lane);
          }
#pragma unroll
          for (int it = 0; it < G::BLOADS; ++it) {
            const int r = br + it * (64 / CPR);
            if constexpr (G::SEGMENTS) row = segment_at(u, r, &live).y - (uint32_t)r;
            const bool ok = live && (G::SEGMENTS || r < (BR < kUnit ? BR : kUnit));
            const uint32_t ob = (row + (uint32_t)r) * pitch + (uint32_t)(n0 + bcol) * 2u;
            if constexpr (ODD) {
              const uint32_t end = ob + 16u < dy_bytes ? ob + 16u : dy_bytes;
              over[d][it] = ok ? ob + 16u - end : 16u;
              b[d][it] = reinterpret_cast<const LooseVec *>(dy + (ok ? end : 16u) - 16)->v;
            } else {
              b[d][it] = buffer_load<16>(rsrc_b, ok ? ob : kOutOfRange);
            }
          }
        },
        [&](int d) {
          // (columns 14 and 15 of a 14-wide block's tile hold what follows in memory; they are rows of no dW)
          *reinterpret_cast<AVec *>(tile_a + ar * G::IW + ac) = a[d];
#pragma unroll
          for (int it = 0; it < G::BLOADS; ++it) {
            u32x4 v = b[d][it];
            if constexpr (ODD) {
              if (over[d][it] > 0) {
                uint64_t lo = ((uint64_t)v[1] << 32) | v[0], hi = ((uint64_t)v[3] << 32) | v[2];
                const uint32_t sh = 8u * (over[d][it] < 16 ? over[d][it] : 16u);
                if (sh >= 64) { lo = sh >= 128 ? 0 : hi >> (sh - 64); hi = 0; }
                else { lo = (lo >> sh) | (hi << (64 - sh)); hi >>= sh; }
                v[0] = (uint32_t)lo; v[1] = (uint32_t)(lo >> 32); v[2] = (uint32_t)hi; v[3] = (uint32_t)(hi >> 32);
              }
            }
            *reinterpret_cast<u32x4 *>(tile_b + tile_place<G::COLS>(br + it * (64 / CPR), bcol)) = v;
          }
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          const int g = lane >> 4, L = lane & 15;
          if constexpr (G::IW == 32) {
            const int r0 = 8 * (g >> 1) + (L >> 2), c0 = 16 * (g & 1) + 4 * (L & 3);
            auto fragment = [&](const uint16_t *p0, const uint16_t *p1) {
              const v4s lo = read_transposed(p0), hi = read_transposed(p1);
              return __builtin_bit_cast(v8bf, (v8s){lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
            };
            const v8bf fa = fragment(tile_a + r0 * 32 + c0, tile_a + (r0 + 4) * 32 + c0);
#pragma unroll
            for (int q = 0; q < NS; ++q) {
              const v8bf fb = fragment(tile_b + tile_place<G::COLS>(r0, 32 * q + c0), tile_b + tile_place<G::COLS>(r0 + 4, 32 * q + c0));
              acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, fb, acc[q], 0, 0, 0);
            }
          } else {
            const int r0 = 4 * g + (L >> 2), c0 = 4 * (L & 3);
            const v4s fa = read_transposed(tile_a + r0 * 16 + c0);
#pragma unroll
            for (int q = 0; q < NS; ++q)
              acc[q] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(fa, read_transposed(tile_b + tile_place<G::COLS>(r0, 16 * q + c0)),
                                                                 acc[q], 0, 0, 0);
          }
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        });
    __syncthreads();                         // the tiles' place is taken by the sums
  }

  // ---- the waves' sums together, each wave its share of the results ----
  float *const o = prm.out + (int64_t)split * prm.split_stride;
#pragma unroll
  for (int part = 0; part < R / kPart; ++part) {
    if (part > 0) __syncthreads();
#pragma unroll
    for (int y = 0; y < kPart; ++y) {        // result y of the part: element y % VQ of a vector
      const int x = (part * kPart + y) / G::VQ, q = (x / G::REGS) * G::VQ + y % G::VQ;
      sSum[(wave * kPart + y) * 64 + lane] = acc[q][x % G::REGS];
    }
    __syncthreads();
    for (int v = wave; v < kPart / G::VQ; v += W) {
      const int x = part * (kPart / G::VQ) + v, g = x / G::REGS, r = x % G::REGS;
      Floats<G::VQ> sum;
#pragma unroll
      for (int q = 0; q < G::VQ; ++q) sum.v[q] = 0.f;
#pragma unroll
      for (int w = 0; w < W; ++w)
#pragma unroll
        for (int q = 0; q < G::VQ; ++q) sum.v[q] += sSum[(w * kPart + v * G::VQ + q) * 64 + lane];
      const int row = G::IW == 32 ? 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3) : 4 * (lane >> 4) + r;
      const int64_t k = (int64_t)j * bc + sub + row, n = n0 + g * G::IW * G::VQ + G::VQ * i;
      if ((BC < G::IW && row >= BC) || k >= prm.K) continue;
      float *const dst = o + k * prm.ldo + n;
      if (n + G::VQ <= prm.N) {
        if (prm.accumulate) {
          const Floats<G::VQ> old = *reinterpret_cast<const Floats<G::VQ> *>(dst);
#pragma unroll
          for (int q = 0; q < G::VQ; ++q) sum.v[q] = old.v[q] + sum.v[q];
        }
        *reinterpret_cast<Floats<G::VQ> *>(dst) = sum;
      } else {
#pragma unroll
        for (int q = 0; q < G::VQ; ++q)
          if (n + q < prm.N) dst[q] = prm.accumulate ? dst[q] + sum.v[q] : sum.v[q];
      }
    }
  }
}

// A plan's variant: 0 wide tiles .. 2 narrow ones.
constexpr int kVariants = 3;
constexpr int kWaves[kVariants] = {4, 8, 16};
inline int variant_columns(int v) { return 128 >> v; }
// workgroups that a compute unit holds (e: bytes of an element)
inline int at_a_time(int v, int e, int br, int bc) { return v == 0 ? (br == 1 ? 2 : 3) : v == 1 || (e == 4 && bc % 32 != 0) ? 2 : 1; }

// What each choice would take, in microseconds: rounds of the workgroups that the compute units hold at a time, each with a start
// and an end (list of blocks, sums) and the units of its waves, which take what their matrix instructions (bfloat16: and LDS
// accesses) need, what their loads need, or what one wave's loads are on their way; and the launch that adds up the
// splits.  Variant and splits are chosen at keep 0.6, since what is kept is not known here.  The constants are a fit to every
// variant and number of splits at 15 shapes in binary32, from [256 x 128 x 64] to [47739 x 860 x 67], and at 20 in bfloat16, up to
// [9947 x 411 x 1001] and [49035 x 658 x 32]: what is chosen takes 1.01 (bfloat16 1.03) times as long as the best one in the mean.  What
// matters most is that the workgroups fill whole rounds: binary32 [12544 x 384 x 1536] in 32x32 blocks 80 us
// in 5 splits = 720 workgroups, 99 in 4, 95 in 6.
struct DirectCosts {
  double start, unit32, unit_wide16, unit_mid16, unit_narrow16;   // of a workgroup; of a unit on a SIMD, 32 columns / 16-wide tiles of 128, 64, 32 columns
  double bytes_per_ns, on_the_way, round, reduce, reduce_per_mb;
};
constexpr DirectCosts kCostsF32 = {3.8, 0.24, 0.48, 0.24, 0.14, 48.5, 1.05, 3.4, 3.0, 0.212};
constexpr DirectCosts kCostsBf16 = {2.2, 0.086, 0.05, 0.025, 0.0125, 75.7, 0.4, 3.1, 3.6, 0.114};

// What a plan for row segments needs when `keep` of the segments of a strip are kept: rounds of workgroups, the walk through the
// entries by loads that all workgroups of a compute unit share and by a workgroup's own turns, units of the waves, splits.  A fit to 260
// products in bfloat16 and 200 in binary32, keep 0.9: within 10 % of four in five.
double segments_us(const DirectPlan &p, int dtype, int64_t tiles, int64_t K, int64_t N, int64_t nbc, double keep) {
  struct { double start[kVariants], round, walk_kb, walk_turn, unit32, unit, row, reduce, reduce_mb; } c;
  if (dtype == BSR_F32) c = {{7.7, 7.2, 9.8}, 6.3, 0.041, 0.0, 0.072, 0.57, 2.3e-3, 3.5, 0.134};
  else c = {{7.5, 6.5, 9.0}, 6.1, 0.044, 0.36, 0.0114, 0.42, 0.0, 3.6, 0.22};
  const int waves = kWaves[p.variant];
  const double rows = (double)p.rows_per_split, entries = rows * (double)nbc * keep, units = rows / kUnit * keep / waves + 0.5;
  const double on_a_cu = (double)ceil_div(tiles * p.splits, (int64_t)256);
  const double rounds = (double)ceil_div((int64_t)on_a_cu, (int64_t)(p.variant < 2 ? 2 : 1));
  return c.start[p.variant] + c.round * (rounds - 1.0) + c.walk_kb * entries * 4e-3 * on_a_cu +
         rounds * (c.walk_turn * entries / (waves * 64 * 16) + c.unit * units + c.row * rows) +
         c.unit32 * units * waves * on_a_cu * (variant_columns(p.variant) / 32) +
         (p.splits > 1 ? c.reduce + c.reduce_mb * (double)p.splits * (double)K * (double)N * 8e-6 : 0.0);
}

// The splits' sums go where the other kernels for the product have theirs, no more of them than fit (ws_bytes).
// A plan is chosen for keep 0.6; whether the kernel is taken at all goes by most_us, what the chosen plan needs when nine blocks in ten
// are kept (the other kernels take about as long whatever is kept, so a call that is no slower then is no slower at all).  That
// counts the walk through the entries of a workgroup's rows as well, which every strip does ([2000 x 30000 x 256] binary32 in 16x16
// blocks: 1875 strips, 1300 us at keep 0.9), and that a last block-column in part is the first to be pruned: of the others more is kept.
// What a variant's workgroups cost, whatever the splits.
struct VariantCosts {
  int64_t tiles;
  double unit_us, unit_kb;
  int waves, per_cu;
};

}  // namespace

// (the operands are below 2 GiB: 32-bit counts of block-rows.  A few hundred ns at the most: splits that cost more than the best plan
// by what they write alone end a variant's turn)
DirectPlan make_direct_plan(int dtype, int64_t M, int64_t K, int64_t N, int br, int bc, size_t ws_bytes) {
  const uint32_t nbr = (uint32_t)ceil_div(M, br);
  const int64_t nbc = ceil_div(K, bc), strips = bc > 16 ? ceil_div(K, 32) : nbc;
  const uint32_t kMaxRows = (uint32_t)max_rows(br);
  const int e = elem_bytes(dtype);
  const double upb = br > kUnit ? br / kUnit : br == 1 ? 1.0 / kUnit : 1.0;
  const DirectCosts &c = dtype == BSR_F32 ? kCostsF32 : kCostsBf16;
  const double split_us = (double)K * (double)N * 8e-6 * c.reduce_per_mb;
  auto costs = [&](int v) {
    const int cols = variant_columns(v);
    return VariantCosts{strips * ceil_div(N, cols),
                        bc % 32 == 0 ? c.unit32 * (cols / 32) : cols > 64 ? c.unit_wide16 : cols > 32 ? c.unit_mid16 : c.unit_narrow16,
                        kUnit * e * ((bc < 32 ? bc : 32) + cols) * 1e-3, kWaves[v], at_a_time(v, e, br, bc)};
  };
  auto estimate = [&](const VariantCosts &vc, uint32_t rows, uint32_t splits, double keep, bool walk) {
    const double units = (double)rows * upb * keep / vc.waves + 0.5;
    auto round_us = [&](int64_t n) {
      const double on_all = (double)(vc.waves * n);
      const double mult = vc.unit_us * on_all / 4, load = vc.unit_kb * on_all / c.bytes_per_ns;
      const double busy = mult > load ? mult : load;
      return c.round + (walk ? (double)rows * nbc * 4e-3 * keep * (double)n / c.bytes_per_ns : 0.0) +
             units * (busy > c.on_the_way ? busy : c.on_the_way);
    };
    const int64_t on_a_cu = (vc.tiles * splits + 255) >> 8;
    const int64_t full = vc.per_cu == 1 ? on_a_cu : vc.per_cu == 2 ? on_a_cu >> 1 : on_a_cu / 3, rest = on_a_cu - full * vc.per_cu;
    return c.start + (full > 0 ? (double)full * round_us(vc.per_cu) : 0.0) + (rest > 0 ? round_us(rest) : 0.0) +
           (splits > 1 ? c.reduce + (double)splits * split_us : 0.0);
  };
  DirectPlan best{0, 0, 0, 1, (int)(nbr < 1 ? 1 : nbr > kMaxRows ? kMaxRows : nbr)};
  bool any = false;
  const int64_t s_room = (int64_t)(ws_bytes / ((size_t)K * N * sizeof(float)));
  for (int v = 0; v < kVariants; ++v) {
    const VariantCosts vc = costs(v);
    // (splits beyond four rounds of workgroups gain nothing)
    const uint32_t s_min = (nbr + kMaxRows - 1) / kMaxRows;
    const int64_t s_full = 1024 * vc.per_cu / vc.tiles + 1;
    int64_t s_max = nbr < 64 ? nbr : 64;
    if (s_max > s_full) s_max = s_full;
    if (s_max < s_min) s_max = s_min;
    if (s_max > s_room) s_max = s_room > 1 ? s_room : 1;
    uint32_t rows_before = 0;
    for (uint32_t s = s_min; s <= s_max; ++s) {
      const uint32_t rows = (nbr + s - 1) / s;
      if (rows == rows_before) continue;
      rows_before = rows;
      const uint32_t splits = (nbr + rows - 1) / rows;
      if (any && splits > 1 && c.start + c.round + c.reduce + (double)splits * split_us > best.us) break;
      const double us = estimate(vc, rows, splits, 0.6, br == 1);   // (row segments: every workgroup walks all entries of its rows)
      if (!any || us < best.us) best = DirectPlan{us, 0, v, (int)splits, (int)rows};
      any = true;
    }
  }
  if (!any) return best;                     // (us 0: no plan)
  const int64_t whole = K / bc < 1 ? 1 : K / bc;
  double most = 0.9 * (double)nbc / (double)whole;
  if (most > 1.0) most = 1.0;
  const VariantCosts vc = costs(best.variant);
  if (br == 1) {
    best.most_us = segments_us(best, dtype, vc.tiles, K, N, nbc, most);
    return best;
  }
  best.most_us = estimate(vc, (uint32_t)best.rows_per_split, (uint32_t)best.splits, most, true);
  // (bfloat16, one workgroup of 16 waves per compute unit: with many units each, their loads take longer than the model has it,
  // [5615 x 96 x 2160] in 64x64 blocks, 22 units: 17.2 us in 128 x 128 tiles, 21.2 here, 14 by the model; [2916 x 32 x 584], 11.5: 10.3,
  // 12.4 and 9.9)
  const int64_t units = (int64_t)best.rows_per_split * br / kUnit;
  if (dtype == BSR_BF16 && bc >= 32 && best.variant == 2 && best.splits == 1 && units > 11 * kWaves[2])
    best.most_us *= units > 16 * kWaves[2] ? 2.0 : 1.15;
  return best;
}

namespace {

template <typename T, int BR, int BC, int NS, int W, int D, int WAVES>
void start(const DirectParams &prm, bool odd, hipStream_t s) {
  const int64_t items = (int64_t)prm.strips * prm.tiles_n * prm.splits;
  const dim3 grid((unsigned)(8 * ceil_div(items, 8))), block(64 * W);
  if constexpr (sizeof(T) == 2) {
    if (odd) {
      hipLaunchKernelGGL((dw_direct_kernel<T, BR, BC, NS, W, D, WAVES, true>), grid, block, 0, s, prm);
      return;
    }
  }
  hipLaunchKernelGGL((dw_direct_kernel<T, BR, BC, NS, W, D, WAVES, false>), grid, block, 0, s, prm);
}

template <typename T, int BR, int BC>
void start_variant(int v, const DirectParams &prm, bool odd, hipStream_t s) {
  constexpr int F = BC % 32 == 0 ? 1 : 2;    // 16-wide tiles: twice as many for the same columns
  if constexpr (sizeof(T) == 4) {
    if (v == 0) start<T, BR, BC, 4 * F, 4, F == 1 ? 2 : 3, BR == 1 ? 2 : 3>(prm, odd, s);
    else if (v == 1) start<T, BR, BC, 2 * F, 8, 3, 4>(prm, odd, s);
    else start<T, BR, BC, F, 16, 3, F == 1 ? 4 : 8>(prm, odd, s);
  } else {
    if (v == 0) start<T, BR, BC, 4 * F, 4, 3, BR == 1 ? 2 : 3>(prm, odd, s);
    else if (v == 1) start<T, BR, BC, 2 * F, 8, 4, 4>(prm, odd, s);
    else start<T, BR, BC, F, 16, 4, 4>(prm, odd, s);
  }
}

template <typename T>
int start_shape(int br, int v, const DirectParams &prm, bool odd, hipStream_t s) {
  if (br == 14) start_variant<T, 14, 14>(v, prm, odd, s);
  else if (br == 16) start_variant<T, 16, 16>(v, prm, odd, s);
  else if (br == 1) start_variant<T, 1, 32>(v, prm, odd, s);
  else if (br == 32) start_variant<T, 32, 32>(v, prm, odd, s);
  else start_variant<T, 64, 64>(v, prm, odd, s);
  return check_launch();
}

}  // namespace

// The operands are addressed with 32-bit byte offsets, the activation's below 2 GiB.  (bfloat16: values in whole 16-byte vectors,
// dY of one vector at least.)
bool dw_direct_supported(int dtype, int br, int bc, const void *values, int64_t M, int64_t K, int64_t N, int64_t lddy) {
  if ((dtype != BSR_F32 && dtype != BSR_BF16) || (br == 1 ? bc % 32 != 0 : br != bc || (br != 14 && br != 16 && br != 32 && br != 64)))
    return false;
  if (M < 1 || K < 1 || N < 1) return false;
  const int64_t e = elem_bytes(dtype);
  if (ceil_div(M, br) * br * ceil_div(K, bc) * bc * e >= (int64_t(1) << 31)) return false;
  if (lddy < N || lddy >= (int64_t(1) << 30) || (M + 2 * 64) * lddy * e >= (int64_t(1) << 32) - 4096) return false;
  if (dtype == BSR_BF16 && ((uintptr_t)values % 16 != 0 || (M - 1) * lddy + N < 8)) return false;
  return ceil_div(K, 16) * ceil_div(N, 32) < (int64_t(1) << 24);
}

int launch_dw_direct(int dtype, const DwJob &j, const DirectPlan &p, hipStream_t s) {
  const size_t need = p.splits > 1 ? (size_t)p.splits * j.K * j.N * sizeof(float) : 0;
  if (need > 0 && (j.ws == nullptr || j.ws_bytes < need)) return BSR_ERR_WORKSPACE;
  if (p.us == 0.0 || p.rows_per_split > max_rows(j.br)) return BSR_ERR_SHAPE;
  const bool split = p.splits > 1;
  DirectParams prm;
  prm.row_ptr = j.row_ptr; prm.col_idx = j.col_idx;
  prm.values = j.values; prm.dY = j.dY;
  prm.out = split ? static_cast<float *>(j.ws) : j.dW;
  prm.M = j.M; prm.K = j.K; prm.N = j.N; prm.lddy = j.lddy;
  prm.ldo = split ? j.N : j.lddw;
  prm.split_stride = split ? j.K * j.N : 0;
  prm.nbr = ceil_div(j.M, j.br); prm.nbc = ceil_div(j.K, j.bc);
  prm.rows_per_split = p.rows_per_split;
  prm.bc = j.bc;
  prm.strips = (int)(j.bc > 16 ? ceil_div(j.K, 32) : prm.nbc);
  prm.tiles_n = (int)ceil_div(j.N, variant_columns(p.variant));
  prm.splits = p.splits;
  prm.accumulate = split ? 0 : j.accumulate;
  const bool odd = dtype == BSR_BF16 && (j.N % 2 != 0 || j.lddy % 2 != 0 || (uintptr_t)j.dY % 4 != 0);
  const int rc = dtype == BSR_F32 ? start_shape<float>(j.br, p.variant, prm, false, s)
                                  : start_shape<uint16_t>(j.br, p.variant, prm, odd, s);
  if (rc != BSR_OK || !split) return rc;
  return launch_splitk_reduce(prm.out, prm.splits, j.K, j.N, j.dW, j.lddw, j.accumulate, s);
}

}  // namespace bsr
