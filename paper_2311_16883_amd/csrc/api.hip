// C ABI of libbsr_actprune: argument validation on the host, then kernel
// launches on the caller's stream.  See include/bsr_actprune.h for the contract
// of every entry point.
#include <cmath>
#include <vector>

#include "common.h"

namespace bsr {

static thread_local int g_last_hip_error = 0;

void set_hip_error(int e) { g_last_hip_error = e; }

int check_launch() {
  const hipError_t e = hipGetLastError();
  if (e == hipSuccess) return BSR_OK;
  g_last_hip_error = (int)e;
  return BSR_ERR_HIP;
}

namespace {

constexpr int64_t kMaxBlocks = (int64_t(1) << 31) - 1;
constexpr int kMaxBlockDim = 1 << 16;

struct Geometry {
  int64_t nbr, nbc, nblocks;
};

// Shared shape checks.  ld is the leading dimension of the dense matrix.
int check_shape(int dtype, int64_t M, int64_t K, int64_t ld, int br, int bc, Geometry *g) {
  if (dtype != BSR_F32 && dtype != BSR_BF16) return BSR_ERR_DTYPE;
  if (M < 0 || K < 0 || br < 1 || bc < 1 || br > kMaxBlockDim || bc > kMaxBlockDim) return BSR_ERR_SHAPE;
  if (ld < K) return BSR_ERR_SHAPE;
  if (M > (int64_t(1) << 40) || K > (int64_t(1) << 40) || ld > (int64_t(1) << 40)) return BSR_ERR_SHAPE;
  g->nbr = ceil_div(M, br);
  g->nbc = ceil_div(K, bc);
  if (g->nbr > kMaxBlocks || g->nbc > kMaxBlocks) return BSR_ERR_SHAPE;
  if (g->nbc != 0 && g->nbr > kMaxBlocks / g->nbc) return BSR_ERR_SHAPE;
  g->nblocks = g->nbr * g->nbc;
  if ((double)M * (double)ld * 4.0 > 9.0e18) return BSR_ERR_SHAPE;
  return BSR_OK;
}

bool misaligned(const void *p, size_t a) { return p != nullptr && (uintptr_t)p % a != 0; }

size_t scores_bytes(int64_t nblocks) { return align_up((size_t)nblocks * sizeof(double), 256); }

size_t score_select_ws(int64_t nblocks) { return scores_bytes(nblocks) + select_ws_bytes(nblocks); }

// How well a product suits the wide-tile kernel: its tiles of 384 x 128 times the ways its
// contraction can be split, i.e. the workgroups it can keep busy.  A call takes the wide
// kernel when that reaches half the compute units, and when the products are large enough (wide_work).
int64_t wide_parallelism(int64_t M, int64_t K, int64_t N, int br) {
  const int64_t nbr = ceil_div(M, br);
  return ceil_div(K, 384) * ceil_div(N, 128) * (nbr < 16 ? nbr : 16);
}

// Small square blocks and a small weight matrix (the cross-patch layers) in a batched call: the kernel whose
// workgroups own all of dW, once the contraction is long enough to split over a few of them.  (A product on
// its own would need so many splits to fill the GPU that the narrow-tile kernel is the faster one.)
bool use_narrow(int dtype, int br, int bc, const void *values, const void *dY, int64_t M, int64_t K, int64_t N,
                int64_t lddy) {
  return dw_narrow_supported(dtype, br, bc, values, dY, M, K, N, lddy) && ceil_div(M, br) >= 16;
}

// Work from which a call's products are worth the wide kernel, in units of that: its start, its write-out and its few large
// workgroups cost more than the 128 x 128 tiles until there is enough to multiply.
// A product of 32x32 or 64x64 blocks on its own (`alone`): 4.06e9 multiply-adds of whole tiles of 128 rows and whole strips of
// 32 columns of dW, which is what the other kernel would spend its time on.  Over 147 shapes of 1e9 .. 1.6e10 multiply-adds at
// five keeps that is 1.089 times as fast as wide tiles for all (geometric mean), nowhere more than 7 % slower, and 1.4 % from
// the better kernel each time; a line at 5e9 multiply-adds whatever the tiles is up to 22 % slower ([8147 x 152 x 1968], 2.4e9,
// in whole tiles 4.1e9: 20.9 us wide, 25.5 in 128 x 128 tiles; [12544 x 1536 x 256], keep 0.25: 26.8 and 31.5; on the other
// side [6272 x 384 x 1536] 27.6 and 22.3, [1095 x 1240 x 2832] 25.8 and 18.7, [10098 x 3616 x 32], keep 0.75, 26.0 and 21.2).
// Several: 5e9 multiply-adds of them all (whole tiles are no better measure there; two products [3136 x 384 x 1536] in 32x32
// blocks 29.2 wide and 24.8, [6272 x 384 x 1536] 31.4 and 32.9).
// 16x16 blocks, where the wide kernel copies by halves of a piece: 2.5e10 multiply-adds ([25088 x 1536 x 384] 48.9 wide and
// 46.7, [23896 x 880 x 2016] 111 and 126, 8 x [6272 x 384 x 1536], keep 0.25, 68 and 87), and tiles and compute units at least
// kFill16 times as well filled as 128 x 128 tiles would be (dw_wide_fill): these waste less where the wide tiles don't fit dW,
// and where workgroups of very different length share a launch ([27817 x 408 x 3440], 0.44 to 0.79, keep 0.9: 155 wide and 125;
// twelve products from [33324 x 352 x 200] to [14904 x 2880 x 112], 0.07 to 0.9, 509 and 153; but [49224 x 3160 x 264], 0.60 to
// 0.68, keep 0.1, 84 and 122).  Over 156 shapes and batches of all sizes at three to five keeps no call is more than 3 % slower
// so than in 128 x 128 tiles, and all together take 0.96 of the time; without this condition 1.00, the worst 3.7 times as long.
// Only where the 128 x 128 tiles can address the operands: the general kernel, the other choice, takes 1.1 .. 9 times as long
// ([1000 x 1000 x 4000] with a far pitch of dY 277 and 31 us, [4000 x 300000 x 8] 10.1 and 6.3 ms), or as long where there is
// next to nothing to multiply ([512 x 3072 x 8] 17 and 17, [128 x 6144 x 8] 13 and 15).
constexpr double kFill16 = 0.71;
double whole_tiles_work(int64_t M, int64_t K, int64_t N) {
  return (double)M * (double)(ceil_div(K, 128) * 128) * (double)(ceil_div(N, 128) * 128);
}
double wide_work(int64_t M, int64_t K, int64_t N, int br, bool alone) {
  if (br != 16 && alone) return (double)M * (double)(ceil_div(K, 128) * 128) * (double)(ceil_div(N, 32) * 32) / 4.06e9;
  return (double)M * (double)K * (double)N / (br == 16 ? 2.5e10 : 5.0e9);
}

// Block shapes without a kernel of their own: whether re-tiling and the matrix cores (two or three launches, 11 .. 19 us at the
// least) take less time than the general kernel, which walks the block-rows one after the other and multiplies on the
// vector units, the slower the fewer rows a block has (tall blocks: by the size of the activation alone; [700 x 100 x 300] in 128x16
// blocks 29 general and 14 re-tiled).  In us: [2543 x 26 x 60] in 1x32 blocks 63 general and 13 re-tiled, [563 x 19 x 1069] 28
// and 15, [412 x 213 x 26] in 7x5 blocks 9 and 19, [209 x 328 x 190] 14 and 21, [522 x 484 x 131] in 8x8 blocks 25 and 16,
// [158 x 26 x 932] 10 and 14.  Short and wide activations in small blocks, whose entries every workgroup of either kernel
// searches, are no different: [8 x 20000 x 10] in 1x1 blocks 28 and 57, [64 x 8000 x 8] in 2x2 24 and 32.  Of 232 shapes up to
// 20000 rows, 60000 columns of X and 4000 of dW, 30 take the slower of the two by more than 6 %: few rows in 1x32 or 1x128
// blocks ([41 x 3277 x 30] 22 and 12) and few in tall ones ([210 x 121 x 23] in 300x4 blocks 50 and 15).
double general_us(int64_t M, int64_t K, int64_t N, int br) {
  return 9.0 + 0.025 * (double)ceil_div(M, br) + 1e-6 * (double)M * (double)K * (double)N * (0.25 + 0.75 / br);
}
bool retiling_pays(int64_t M, int64_t K, int64_t N, int br) {
  if (br > 16) return M * K > 65536;
  return general_us(M, K, N, br) > 15.3;
}

// Parallelism and work of the products of a call, by block size (16, 32, 64: wide_class), since each size has a launch of its
// own.  The work of one does not carry another ([25088 x 384 x 1536] in 32x32 blocks with [3136 x 384 x 1536] in 16x16, keep
// 0.5: 62.5 us both wide, 58.5 so; [6272 x 384 x 1536] in 32x32 and 64x64: 51.0 and 42.2).  Half-filled launches of 32x32 and of
// 64x64 blocks together are better than none ([14600 x 384 x 896] in both: 54.0 wide, 61.6 in 128 x 128 tiles; two each of
// [50176 x 384 x 384], keep 0.25, 77 and 97): their parallelism counts as one.
struct WideSums {
  int n[3] = {0, 0, 0};
  int64_t par[3] = {0, 0, 0};
  double work[3] = {0.0, 0.0, 0.0}, work_alone[3] = {0.0, 0.0, 0.0};
  double plain16 = 0.0, whole16 = 0.0;         // multiply-adds, and of whole 128 x 128 tiles
  bool filled16 = false;
  void add(int64_t M, int64_t K, int64_t N, int br) {
    const int c = wide_class(br);
    ++n[c];
    par[c] += wide_parallelism(M, K, N, br);
    work[c] += wide_work(M, K, N, br, false);
    work_alone[c] += wide_work(M, K, N, br, true);
    if (c == 0) {
      plain16 += (double)M * (double)K * (double)N;
      whole16 += whole_tiles_work(M, K, N);
    }
  }
  // Once all are added (`jobs`: the products themselves); then pays() answers.
  void close(const DwJob *jobs, int count) {
    if (par[0] >= 128 && work[0] >= 1.0) filled16 = dw_wide_fill(jobs, count, 16) >= kFill16 * plain16 / whole16;
  }
  // `mfma`: the 128 x 128 tiles, the other choice, can address the operands
  bool pays(int br, bool mfma) const {
    const int c = wide_class(br);
    if ((c == 0 ? par[0] : par[1] + par[2]) < 128) return false;
    return ((n[c] == 1 ? work_alone[c] : work[c]) >= 1.0 && (c != 0 || filled16)) || !mfma;
  }
  static int wide_class(int br) { return br == 16 ? 0 : br == 32 ? 1 : 2; }
};

bool use_wide_single(int dtype, const DwJob &j) {
  if (!dw_wide_supported(dtype, j.br, j.bc, j.values, j.dY, j.M, j.K, j.N, j.lddy)) return false;
  WideSums sums;
  sums.add(j.M, j.K, j.N, j.br);
  sums.close(&j, 1);
  return sums.pays(j.br, dw_mfma_supported(dtype, j.br, j.bc, j.values, j.M, j.K, j.N, j.lddy));
}

// Whether a product on its own takes the kernel whose waves each gather the kept blocks of one strip, instead of the 128 x 128
// tiles: by both plans' estimates, for nine blocks in ten kept, where it gains least.  The lines differ by how far the estimates
// are off for a kind of call (the tiles need 0.7 of what their plan says in bfloat16, 0.8 in binary32).  Fitted to 1366 products
// of all these block shapes, of 600 others at keeps 0.1, 0.5, 0.75 and 0.9 two are more than 5 % slower than without this kernel
// ([32368 x 64 x 283] bfloat16 in 64x64, keep 0.9: 15.5 and 18.1), and all together take 1 / 1.22 .. 1 / 1.49 of the time, by type
// and keep (geometric mean).  In us, tiles and so, at keep 0.5 and 0.9.  Taken: binary32 [256 x 128 x 64] in 16x16 blocks 9.7 and
// 5.9; [1889 x 544 x 784] 31 and 18, 34 and 25; [25088 x 196 x 196] in 14x14 38 and 27, 41 and 37; [2000 x 3000 x 300] in 32x32 42
// and 32, 53 and 44; bfloat16 [1202 x 152 x 446] 12.7 and 7.1; [2000 x 1000 x 190] in 16x16 15 and 8.7, 15 and 11; [2006 x 454 x
// 1472] in 32x32 18 and 11, 18 and 15; [10000 x 196 x 196] in 14x14 15 and 12, 16 and 14.  Left to the tiles: binary32 [12544 x
// 768 x 768] in 16x16 103 and 90, 122 and 144; [1000 x 24000 x 300] in 14x14 211 and 546, 265 and 954; [20734 x 2592 x 64] in
// 64x64, keep 0.9, 69 and 91; bfloat16, rows of dY on odd elements, [9947 x 411 x 1001] in 32x32 32 and 25, 32 and 38.  (Binary32,
// much to multiply and few block-columns: there the tiles gain by what is pruned as a strip does, [25842 x 42 x 464] in 32x32 21
// and 27, 26 and 27; [37960 x 23 x 912] in 16x16 40 and 43.)
// By size: beyond these next to nothing was found that gains, and no plan has to be made.
bool direct_sizes(int dtype, int64_t M, int64_t K, int64_t N, int br) {
  const double work = (double)M * (double)K * (double)N;
  if (br == 1) return work < 4.2e8;
  if (dtype == BSR_F32) return work < 5.0e9;
  if (br < 32) return work < 4e8;
  return work < (M * K < 4000000 ? 1.1e9 : 7e8) || M * K < 2000000;
}
// Row segments of whole 32 columns, against re-tiling and the tiles, two or three launches, or the general kernel: here, too, by
// what each needs for nine segments in ten kept (for re-tiling a fit to 624 products, within 15 % of four in five).  Of 780
// products at keeps 0.1 .. 0.9 the worst is 8 % slower so than without this kernel.  In us, without and so, keep 0.1, 0.5 and 0.9:
// bfloat16 [40000 x 320 x 32] in 1x32 blocks 32 and 14, 28 and 16, 25 and 19; [1000 x 400 x 1000] 19 and 8.1, 20 and 10, 20 and
// 14; [1646 x 136 x 3104] in 1x64 19 and 8.8, 19 and 14, 19 and 16; binary32 [5711 x 376 x 78] in 1x128 28 and 16, 28 and 20, 27
// and 22. Not: wide activations, whose entries every strip walks, bfloat16 [4096 x 10000 x 8] in 1x32 42 and 43, 51 and 150, 64
// and 260; [3000 x 3000 x 46] 26 and 13, 25 and 24, 25 and 32; few rows and a small dW, which the general kernel takes as fast,
// [24 x 59 x 10] 8 and 9.
double segments_other_us(int dtype, int64_t M, int64_t K, int64_t N) {
  if (M < 64 && K < 1000 && K * N < 20000) return 0.0;
  // (the general kernel's search among a row's entries: [25 x 2688 x 32] bfloat16 14.6, 9.5 so)
  if (!retiling_pays(M, K, N, 1))
    return (dtype == BSR_F32 ? 0.85 : 0.8) * (general_us(M, K, N, 1) + 1.2e-3 * (double)(K < 4000 ? K : 4000));
  const double mb = (double)M * (double)K * elem_bytes(dtype) * 1e-6;
  const double other = (5.4 + 0.68 * dw_mfma_us(dtype, M, K, N, 32) + 0.37 * mb) * (K <= 32 ? 0.87 : 1.0);
  return (dtype == BSR_F32 ? 0.95 : 0.92) * other;
}

// The plan of a product on its own, and the time that the other kernels need for it.  A thread keeps those of its last shapes: a
// network's layers come by again and again, and a plan costs as much on the host as a third of a launch.
struct DirectChoice {
  int64_t M, K, N;
  size_t ws_bytes;
  int dtype, br, bc;
  DirectPlan plan;
  double other_us;
};
constexpr int kKeptChoices = 64;
const DirectChoice &direct_choice(int dtype, const DwJob &j) {
  static thread_local DirectChoice kept[kKeptChoices];
  uint64_t h = (uint64_t)j.M * 0x9E3779B97F4A7C15ull ^ (uint64_t)j.K * 0xC2B2AE3D27D4EB4Full ^ (uint64_t)j.N * 0x165667B19E3779F9ull;
  h = (h ^ (uint64_t)(j.br + 64 * j.bc + dtype)) * 0x9E3779B97F4A7C15ull;
  DirectChoice &c = kept[h >> 58];
  if (c.M != j.M || c.K != j.K || c.N != j.N || c.ws_bytes != j.ws_bytes || c.dtype != dtype || c.br != j.br || c.bc != j.bc)
    c = DirectChoice{j.M, j.K, j.N, j.ws_bytes, dtype, j.br, j.bc, make_direct_plan(dtype, j.M, j.K, j.N, j.br, j.bc, j.ws_bytes),
                     j.br == 1 ? segments_other_us(dtype, j.M, j.K, j.N) : dw_mfma_us(dtype, j.M, j.K, j.N, j.br)};
  return c;
}

bool use_direct(int dtype, const DwJob &j) {
  if (!dw_direct_supported(dtype, j.br, j.bc, j.values, j.M, j.K, j.N, j.lddy)) return false;
  const bool tiles = j.br == 1 || dw_mfma_supported(dtype, j.br, j.bc, j.values, j.M, j.K, j.N, j.lddy);
  if (tiles && !direct_sizes(dtype, j.M, j.K, j.N, j.br)) return false;
  const DirectChoice &c = direct_choice(dtype, j);
  if (c.plan.us == 0.0) return false;
  // (square blocks that the tiles cannot address, such as binary32 values off 16-byte boundaries: the general kernel takes 1 .. 4
  // times as long)
  if (!tiles) return true;
  if (j.br == 1) return c.plan.most_us < c.other_us;
  // (a small dW in narrow blocks, such as a cross-patch layer's: partial sums and tiles in part cost more than either plan has it)
  const bool small = j.bc < 32 && j.K * j.N < 50000 && j.N > 64;
  const bool odd = j.N % 2 != 0 || j.lddy % 2 != 0 || (uintptr_t)j.dY % 4 != 0;
  double line = j.bc >= 32 ? (odd ? 0.65 : 0.67) : odd ? 0.68 : small ? 0.75 : 0.70;
  if (dtype == BSR_F32) {
    const bool few = j.K < (j.bc < 32 ? 40 : 128) && (double)j.M * (double)j.K * (double)j.N > 3e8;
    line = few ? 0.55 : j.bc == 16 ? 1.0 : j.bc >= 32 ? 0.83 : small ? 1.32 : 0.9;
  }
  return c.plan.most_us < line * c.other_us;
}

// Workspace of a product, whatever kernel takes it (the gathering one makes do with what the others need).  (The wide tiles take
// activations that the 128 x 128 tiles don't, from 2 GiB up to 4 GiB, and rows of dY further apart.)
size_t dw_ws_bytes(int dtype, int64_t M, int64_t K, int64_t N, int br, int bc) {
  size_t a = dw_generic_ws_bytes(M, K, N, br, bc), b = 0;
  if (dw_mfma_supported(dtype, br, bc, nullptr, M, K, N, N)) b = dw_mfma_ws_bytes(dtype, M, K, N, br, bc);
  else if (dw_reblock_supported(dtype, br, bc, M, K, N, N)) b = dw_reblock_ws_bytes(dtype, M, K, N);
  if (b > a) a = b;
  if (dw_wide_supported(dtype, br, bc, nullptr, nullptr, M, K, N, N)) {
    b = dw_wide_ws_bytes(M, K, N, br);
    if (b > a) a = b;
  }
  if (dw_narrow_supported(dtype, br, bc, nullptr, nullptr, M, K, N, N)) {
    b = dw_narrow_ws_bytes(M, K, N, br);
    if (b > a) a = b;
  }
  return align_up(a, 256);
}

// The products of a batched call (their numbers) by the kernel that takes them; `single`: each by a launch of its own.
struct DwRoutes {
  std::vector<int> narrow, wide, mfma, single;
};

std::vector<DwJob> dw_pick(const std::vector<DwJob> &jobs, const std::vector<int> &which) {
  std::vector<DwJob> r;
  r.reserve(which.size());
  for (const int i : which) r.push_back(jobs[i]);
  return r;
}

DwRoutes dw_routes(int dtype, const std::vector<DwJob> &jobs, bool several) {
  DwRoutes r;
  WideSums sums;
  std::vector<int> maybe;
  for (int i = 0; i < (int)jobs.size(); ++i) {
    const DwJob &j = jobs[i];
    if (!several && !use_wide_single(dtype, j) && use_direct(dtype, j)) {
      r.single.push_back(i);
    } else if (several && use_narrow(dtype, j.br, j.bc, j.values, j.dY, j.M, j.K, j.N, j.lddy)) {
      r.narrow.push_back(i);
    } else if (dw_wide_supported(dtype, j.br, j.bc, j.values, j.dY, j.M, j.K, j.N, j.lddy)) {
      maybe.push_back(i);
      sums.add(j.M, j.K, j.N, j.br);
    } else {
      (dw_mfma_supported(dtype, j.br, j.bc, j.values, j.M, j.K, j.N, j.lddy) ? r.mfma : r.single).push_back(i);
    }
  }
  // too few tiles to fill the GPU even with a deep split, or too little to multiply: the 128 x 128 tiles suit those better,
  // where they can address the operands (half the activation that the wide tiles take)
  const std::vector<DwJob> candidates = dw_pick(jobs, maybe);
  sums.close(candidates.data(), (int)candidates.size());
  for (const int i : maybe) {
    const DwJob &j = jobs[i];
    const bool mfma = dw_mfma_supported(dtype, j.br, j.bc, j.values, j.M, j.K, j.N, j.lddy);
    (sums.pays(j.br, mfma) ? r.wide : mfma ? r.mfma : r.single).push_back(i);
  }
  return r;
}

// One product, with a workspace of dw_ws_bytes or more.
int launch_dw(int dtype, const DwJob &j, hipStream_t s) {
  if (use_wide_single(dtype, j)) return launch_dw_wide(j, s);
  if (use_direct(dtype, j)) return launch_dw_direct(dtype, j, direct_choice(dtype, j).plan, s);
  if (dw_mfma_supported(dtype, j.br, j.bc, j.values, j.M, j.K, j.N, j.lddy))
    return launch_dw_mfma(dtype, j.row_ptr, j.col_idx, j.values, j.M, j.K, j.br, j.bc, j.dY, j.N, j.lddy, j.dW, j.lddw, j.accumulate,
                          j.ws, j.ws_bytes, s);
  // other block shapes: re-tiled into 32x32 blocks for the matrix-core kernel, unless the
  // problem is so small that the single launch of the general kernel is the faster way
  if (retiling_pays(j.M, j.K, j.N, j.br) && dw_reblock_supported(dtype, j.br, j.bc, j.M, j.K, j.N, j.lddy) &&
      j.ws_bytes >= dw_reblock_ws_bytes(dtype, j.M, j.K, j.N))
    return launch_dw_reblocked(dtype, j.row_ptr, j.col_idx, j.values, j.M, j.K, j.br, j.bc, j.dY, j.N, j.lddy, j.dW, j.lddw,
                               j.accumulate, j.ws, j.ws_bytes, s);
  return launch_dw_generic(j.row_ptr, j.col_idx, j.values, dtype, j.M, j.K, j.br, j.bc, j.dY, j.N, j.lddy, j.dW, j.lddw,
                           j.accumulate, j.ws, j.ws_bytes, s);
}

}  // namespace
}  // namespace bsr

using namespace bsr;

extern "C" {

const char *bsr_version(void) { return "bsr_actprune 0.1 (gfx950)"; }

const char *bsr_error_string(int code) {
  switch (code) {
    case BSR_OK: return "BSR_OK";
    case BSR_ERR_NULL: return "BSR_ERR_NULL";
    case BSR_ERR_SHAPE: return "BSR_ERR_SHAPE";
    case BSR_ERR_DTYPE: return "BSR_ERR_DTYPE";
    case BSR_ERR_KEEP: return "BSR_ERR_KEEP";
    case BSR_ERR_WORKSPACE: return "BSR_ERR_WORKSPACE";
    case BSR_ERR_ALIGN: return "BSR_ERR_ALIGN";
    case BSR_ERR_HIP: return "BSR_ERR_HIP";
    case BSR_ERR_LIMIT: return "BSR_ERR_LIMIT";
    default: return "BSR_ERR_UNKNOWN";
  }
}

int bsr_last_hip_error(void) { return g_last_hip_error; }

int64_t bsr_keep_count(int64_t nblocks, double keep) {
  if (nblocks < 0 || !(keep >= 0.0 && keep <= 1.0)) return -1;
  const double v = std::ceil(keep * (double)nblocks);
  int64_t n = (int64_t)v;
  if (n < 0) n = 0;
  if (n > nblocks) n = nblocks;
  return n;
}

int64_t bsr_storage_bytes(int64_t M, int64_t K, int br, int bc, int64_t n_keep, int dtype) {
  Geometry g;
  if (check_shape(dtype, M, K, K, br, bc, &g) != BSR_OK) return -1;
  if (n_keep < 0 || n_keep > g.nblocks) return -1;
  return n_keep * (int64_t)br * bc * elem_bytes(dtype) + 4 * n_keep + 4 * (g.nbr + 1);
}

size_t bsr_workspace_bytes(int op, int64_t M, int64_t K, int64_t N, int br, int bc, int dtype) {
  Geometry g;
  if (check_shape(dtype, M, K, K, br, bc, &g) != BSR_OK) return 0;
  switch (op) {
    case BSR_OP_SCORE_SELECT: return score_select_ws(g.nblocks);
    case BSR_OP_COMPRESS: return compress_ws_bytes(dtype, M, K, br, bc);
    case BSR_OP_DECOMPRESS: return 0;
    case BSR_OP_T_DENSE_MATMUL:
      if (N < 0) return 0;
      return dw_ws_bytes(dtype, M, K, N, br, bc);
    case BSR_OP_AFFINE_SCALE_GRAD: return affine_ws_bytes(M, K, br, bc);
    default: return 0;
  }
}

int bsr_score_select(const void *X, int dtype, int64_t M, int64_t K, int64_t ldx, int br, int bc,
                     double keep, double *scores, uint8_t *keep_mask, void *ws, size_t ws_bytes,
                     void *stream) {
  Geometry g;
  int rc = check_shape(dtype, M, K, ldx, br, bc, &g);
  if (rc != BSR_OK) return rc;
  const int64_t n_keep = bsr_keep_count(g.nblocks, keep);
  if (n_keep < 0) return BSR_ERR_KEEP;
  if (g.nblocks == 0) return BSR_OK;
  if (X == nullptr || keep_mask == nullptr) return BSR_ERR_NULL;
  if (misaligned(X, elem_bytes(dtype)) || misaligned(scores, 8) || misaligned(ws, 16)) return BSR_ERR_ALIGN;
  const size_t need = score_select_ws(g.nblocks);
  if (ws == nullptr || ws_bytes < need) return BSR_ERR_WORKSPACE;
  hipStream_t s = static_cast<hipStream_t>(stream);
  SmallScore small;
  if (plan_score_select_small(X, dtype, M, K, ldx, br, bc, n_keep, &small))
    return launch_score_select_small(small, X, dtype, M, K, ldx, scores, keep_mask, s);
  double *sc = scores != nullptr ? scores : static_cast<double *>(ws);
  rc = launch_score(X, dtype, M, K, ldx, br, bc, sc, s);
  if (rc != BSR_OK) return rc;
  return launch_select(sc, g.nblocks, n_keep, keep_mask, static_cast<char *>(ws) + scores_bytes(g.nblocks), s);
}

int64_t bsr_grouped_keep_count(int64_t nbr, int64_t nbc, int64_t group_rows, double keep) {
  if (nbr < 0 || nbc < 0 || group_rows < 1 || !(keep >= 0.0 && keep <= 1.0)) return -1;
  if (nbr == 0 || nbc == 0) return 0;
  const int64_t groups = (nbr + group_rows - 1) / group_rows;
  const int64_t last_rows = nbr - (groups - 1) * group_rows;
  const int64_t full = groups > 1 ? bsr_keep_count(group_rows * nbc, keep) : 0;
  return (groups - 1) * full + bsr_keep_count(last_rows * nbc, keep);
}

int bsr_score_select_grouped(const void *X, int dtype, int64_t M, int64_t K, int64_t ldx, int br, int bc,
                             int64_t group_rows, double keep, double *scores, uint8_t *keep_mask,
                             void *ws, size_t ws_bytes, void *stream) {
  Geometry g;
  int rc = check_shape(dtype, M, K, ldx, br, bc, &g);
  if (rc != BSR_OK) return rc;
  if (group_rows < 1) return BSR_ERR_SHAPE;
  if (!(keep >= 0.0 && keep <= 1.0)) return BSR_ERR_KEEP;
  if (g.nblocks == 0) return BSR_OK;
  if (X == nullptr || keep_mask == nullptr) return BSR_ERR_NULL;
  if (misaligned(X, elem_bytes(dtype)) || misaligned(scores, 8) || misaligned(ws, 16)) return BSR_ERR_ALIGN;
  const size_t need = score_select_ws(g.nblocks);
  if (ws == nullptr || ws_bytes < need) return BSR_ERR_WORKSPACE;
  if (group_rows > g.nbr) group_rows = g.nbr;
  const int64_t groups = (g.nbr + group_rows - 1) / group_rows;
  const int64_t last_rows = g.nbr - (groups - 1) * group_rows;
  const int64_t n_keep_group = bsr_keep_count(group_rows * g.nbc, keep);
  const int64_t n_keep_last = bsr_keep_count(last_rows * g.nbc, keep);
  hipStream_t s = static_cast<hipStream_t>(stream);
  double *sc = scores != nullptr ? scores : static_cast<double *>(ws);
  rc = launch_score(X, dtype, M, K, ldx, br, bc, sc, s);
  if (rc != BSR_OK) return rc;
  return launch_select_grouped(sc, g.nbr, g.nbc, group_rows, n_keep_group, n_keep_last, keep_mask,
                               static_cast<char *>(ws) + scores_bytes(g.nblocks), s);
}

int bsr_compress(const void *X, int dtype, int64_t M, int64_t K, int64_t ldx, int br, int bc,
                 const uint8_t *keep_mask, int64_t n_keep, int32_t *row_ptr, int32_t *col_idx,
                 void *values, void *ws, size_t ws_bytes, void *stream) {
  Geometry g;
  int rc = check_shape(dtype, M, K, ldx, br, bc, &g);
  if (rc != BSR_OK) return rc;
  if (n_keep < 0 || n_keep > g.nblocks) return BSR_ERR_KEEP;
  const size_t need = compress_ws_bytes(dtype, M, K, br, bc);
  if (need > 0 && (ws == nullptr || ws_bytes < need)) return BSR_ERR_WORKSPACE;
  if (need > 0 && misaligned(ws, 16)) return BSR_ERR_ALIGN;
  if (row_ptr == nullptr) return BSR_ERR_NULL;
  if (g.nblocks > 0 && (X == nullptr || keep_mask == nullptr)) return BSR_ERR_NULL;
  if (n_keep > 0 && (col_idx == nullptr || values == nullptr)) return BSR_ERR_NULL;
  if (misaligned(X, elem_bytes(dtype)) || misaligned(values, elem_bytes(dtype)) ||
      misaligned(row_ptr, 4) || misaligned(col_idx, 4))
    return BSR_ERR_ALIGN;
  hipStream_t s = static_cast<hipStream_t>(stream);
  return launch_compress(keep_mask, X, dtype, M, K, ldx, br, bc, n_keep, row_ptr, col_idx, values, ws, s);
}

int bsr_decompress(const int32_t *row_ptr, const int32_t *col_idx, const void *values, int dtype,
                   int64_t M, int64_t K, int64_t ldx, int br, int bc, void *X_out, void *stream) {
  Geometry g;
  int rc = check_shape(dtype, M, K, ldx, br, bc, &g);
  if (rc != BSR_OK) return rc;
  if (g.nblocks == 0) return BSR_OK;
  if (row_ptr == nullptr || X_out == nullptr) return BSR_ERR_NULL;
  if (misaligned(X_out, elem_bytes(dtype)) || misaligned(values, elem_bytes(dtype)) ||
      misaligned(row_ptr, 4) || misaligned(col_idx, 4))
    return BSR_ERR_ALIGN;
  return launch_decompress(row_ptr, col_idx, values, dtype, M, K, ldx, br, bc, X_out,
                           static_cast<hipStream_t>(stream));
}

int bsr_t_dense_matmul(const int32_t *row_ptr, const int32_t *col_idx, const void *values, int dtype,
                       int64_t M, int64_t K, int br, int bc, const void *dY, int64_t N, int64_t lddy,
                       float *dW, int64_t lddw, int accumulate, void *ws, size_t ws_bytes,
                       void *stream) {
  Geometry g;
  int rc = check_shape(dtype, M, K, K, br, bc, &g);
  if (rc != BSR_OK) return rc;
  if (N < 0 || lddy < N || lddw < N || N > (int64_t(1) << 40)) return BSR_ERR_SHAPE;
  if (K == 0 || N == 0) return BSR_OK;
  if (dW == nullptr || row_ptr == nullptr) return BSR_ERR_NULL;
  if (M > 0 && dY == nullptr) return BSR_ERR_NULL;
  if (misaligned(values, elem_bytes(dtype)) || misaligned(dY, elem_bytes(dtype)) ||
      misaligned(dW, 4) || misaligned(row_ptr, 4) || misaligned(col_idx, 4) || misaligned(ws, 16))
    return BSR_ERR_ALIGN;
  const size_t need = bsr_workspace_bytes(BSR_OP_T_DENSE_MATMUL, M, K, N, br, bc, dtype);
  if (need > 0 && (ws == nullptr || ws_bytes < need)) return BSR_ERR_WORKSPACE;
  // (need, not ws_bytes: what is passed beyond it changes nothing)
  const DwJob job{row_ptr, col_idx, values, M, K, br, bc, dY, N, lddy, dW, lddw, accumulate, ws, need};
  return launch_dw(dtype, job, static_cast<hipStream_t>(stream));
}

int bsr_affine_scale_grad(const int32_t *row_ptr, const int32_t *col_idx, const void *values, int dtype,
                          int64_t M, int64_t K, int br, int bc, const void *dY, int64_t lddy, float *dalpha,
                          int accumulate, void *ws, size_t ws_bytes, void *stream) {
  Geometry g;
  int rc = check_shape(dtype, M, K, K, br, bc, &g);
  if (rc != BSR_OK) return rc;
  if (lddy < K) return BSR_ERR_SHAPE;
  if (K == 0) return BSR_OK;
  if (dalpha == nullptr || row_ptr == nullptr) return BSR_ERR_NULL;
  if (M > 0 && dY == nullptr) return BSR_ERR_NULL;
  if (misaligned(values, elem_bytes(dtype)) || misaligned(dY, elem_bytes(dtype)) || misaligned(dalpha, 4) ||
      misaligned(row_ptr, 4) || misaligned(col_idx, 4) || misaligned(ws, 16))
    return BSR_ERR_ALIGN;
  const size_t need = bsr_workspace_bytes(BSR_OP_AFFINE_SCALE_GRAD, M, K, 0, br, bc, dtype);
  if (need > 0 && (ws == nullptr || ws_bytes < need)) return BSR_ERR_WORKSPACE;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (M == 0) return launch_splitk_reduce(nullptr, 0, 1, K, dalpha, K, accumulate, s);
  return launch_affine_dscale(row_ptr, col_idx, values, dtype, M, K, br, bc, dY, lddy, dalpha, accumulate, ws, s);
}

size_t bsr_score_select_batched_workspace_bytes(const bsr_select_item *items, int n, int dtype) {
  if (items == nullptr || n <= 0) return 0;
  size_t total = 0;
  for (int i = 0; i < n; ++i) {
    Geometry g;
    const bsr_select_item &it = items[i];
    if (check_shape(dtype, it.M, it.K, it.ldx, it.br, it.bc, &g) != BSR_OK) return 0;
    total += align_up(score_select_ws(g.nblocks), 256);
  }
  return total;
}

int bsr_score_select_batched(const bsr_select_item *items, int n, int dtype, void *ws, size_t ws_bytes,
                             void *stream) {
  if (n < 0) return BSR_ERR_SHAPE;
  if (n == 0) return BSR_OK;
  if (items == nullptr) return BSR_ERR_NULL;
  std::vector<ScoreJob> score_jobs;
  std::vector<SelectJob> select_jobs;
  score_jobs.reserve(n);
  select_jobs.reserve(n);
  if (misaligned(ws, 16)) return BSR_ERR_ALIGN;
  size_t off = 0;
  for (int i = 0; i < n; ++i) {
    const bsr_select_item &it = items[i];
    Geometry g;
    const int rc = check_shape(dtype, it.M, it.K, it.ldx, it.br, it.bc, &g);
    if (rc != BSR_OK) return rc;
    const int64_t n_keep = bsr_keep_count(g.nblocks, it.keep);
    if (n_keep < 0) return BSR_ERR_KEEP;
    if (g.nblocks == 0) continue;
    if (it.X == nullptr || it.keep_mask == nullptr) return BSR_ERR_NULL;
    if (misaligned(it.X, elem_bytes(dtype)) || misaligned(it.scores, 8)) return BSR_ERR_ALIGN;
    const size_t need = align_up(score_select_ws(g.nblocks), 256);
    if (ws == nullptr || off + need > ws_bytes) return BSR_ERR_WORKSPACE;
    char *base = static_cast<char *>(ws) + off;
    off += need;
    double *sc = it.scores != nullptr ? it.scores : reinterpret_cast<double *>(base);
    score_jobs.push_back(ScoreJob{it.X, it.M, it.K, it.ldx, it.br, it.bc, sc});
    select_jobs.push_back(SelectJob{sc, g.nblocks, n_keep, it.keep_mask, base + scores_bytes(g.nblocks)});
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int rc = launch_score_batched(score_jobs.data(), (int)score_jobs.size(), dtype, s);
  if (rc != BSR_OK) return rc;
  return launch_select_batched(select_jobs.data(), (int)select_jobs.size(), s);
}

int bsr_score_select_grouped_batched(const bsr_select_item *items, const int64_t *group_rows, int n, int dtype,
                                     void *ws, size_t ws_bytes, void *stream) {
  if (n < 0) return BSR_ERR_SHAPE;
  if (n == 0) return BSR_OK;
  if (items == nullptr || group_rows == nullptr) return BSR_ERR_NULL;
  if (misaligned(ws, 16)) return BSR_ERR_ALIGN;
  std::vector<ScoreJob> score_jobs;
  std::vector<GroupedSelectJob> select_jobs;
  score_jobs.reserve(n);
  select_jobs.reserve(n);
  size_t off = 0;
  for (int i = 0; i < n; ++i) {
    const bsr_select_item &it = items[i];
    Geometry g;
    const int rc = check_shape(dtype, it.M, it.K, it.ldx, it.br, it.bc, &g);
    if (rc != BSR_OK) return rc;
    if (group_rows[i] < 1) return BSR_ERR_SHAPE;
    if (!(it.keep >= 0.0 && it.keep <= 1.0)) return BSR_ERR_KEEP;
    if (g.nblocks == 0) continue;
    if (it.X == nullptr || it.keep_mask == nullptr) return BSR_ERR_NULL;
    if (misaligned(it.X, elem_bytes(dtype)) || misaligned(it.scores, 8)) return BSR_ERR_ALIGN;
    const size_t need = align_up(score_select_ws(g.nblocks), 256);
    if (ws == nullptr || off + need > ws_bytes) return BSR_ERR_WORKSPACE;
    char *base = static_cast<char *>(ws) + off;
    off += need;
    double *sc = it.scores != nullptr ? it.scores : reinterpret_cast<double *>(base);
    const int64_t rows = group_rows[i] > g.nbr ? g.nbr : group_rows[i];
    const int64_t groups = (g.nbr + rows - 1) / rows;
    const int64_t last_rows = g.nbr - (groups - 1) * rows;
    score_jobs.push_back(ScoreJob{it.X, it.M, it.K, it.ldx, it.br, it.bc, sc});
    select_jobs.push_back(GroupedSelectJob{sc, g.nbr, g.nbc, rows, bsr_keep_count(rows * g.nbc, it.keep),
                                           bsr_keep_count(last_rows * g.nbc, it.keep), it.keep_mask,
                                           base + scores_bytes(g.nblocks)});
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int rc = launch_score_batched(score_jobs.data(), (int)score_jobs.size(), dtype, s);
  if (rc != BSR_OK) return rc;
  return launch_select_grouped_batched(select_jobs.data(), (int)select_jobs.size(), s);
}

size_t bsr_t_dense_matmul_batched_workspace_bytes(const bsr_matmul_item *items, int n, int dtype) {
  if (items == nullptr || n <= 0) return 0;
  size_t total = 0;
  for (int i = 0; i < n; ++i) {
    const bsr_matmul_item &it = items[i];
    Geometry g;
    if (check_shape(dtype, it.M, it.K, it.K, it.br, it.bc, &g) != BSR_OK || it.N < 0) return 0;
    total += dw_ws_bytes(dtype, it.M, it.K, it.N, it.br, it.bc);
  }
  return total;
}

int bsr_t_dense_matmul_batched(const bsr_matmul_item *items, int n, int dtype, void *ws, size_t ws_bytes,
                               void *stream) {
  if (n < 0) return BSR_ERR_SHAPE;
  if (n == 0) return BSR_OK;
  if (items == nullptr) return BSR_ERR_NULL;
  if (misaligned(ws, 16)) return BSR_ERR_ALIGN;
  std::vector<DwJob> jobs;
  jobs.reserve(n);
  size_t off = 0;
  for (int i = 0; i < n; ++i) {
    const bsr_matmul_item &it = items[i];
    Geometry g;
    const int rc = check_shape(dtype, it.M, it.K, it.K, it.br, it.bc, &g);
    if (rc != BSR_OK) return rc;
    if (it.N < 0 || it.lddy < it.N || it.lddw < it.N || it.N > (int64_t(1) << 40)) return BSR_ERR_SHAPE;
    if (it.K == 0 || it.N == 0) continue;
    if (it.dW == nullptr || it.row_ptr == nullptr) return BSR_ERR_NULL;
    if (it.M > 0 && it.dY == nullptr) return BSR_ERR_NULL;
    if (misaligned(it.values, elem_bytes(dtype)) || misaligned(it.dY, elem_bytes(dtype)) || misaligned(it.dW, 4) ||
        misaligned(it.row_ptr, 4) || misaligned(it.col_idx, 4))
      return BSR_ERR_ALIGN;
    const size_t need = dw_ws_bytes(dtype, it.M, it.K, it.N, it.br, it.bc);
    if (need > 0 && (ws == nullptr || off + need > ws_bytes)) return BSR_ERR_WORKSPACE;
    jobs.push_back(DwJob{it.row_ptr, it.col_idx, it.values, it.M, it.K, it.br, it.bc, it.dY, it.N, it.lddy, it.dW, it.lddw,
                         it.accumulate, need > 0 ? static_cast<char *>(ws) + off : nullptr, need});
    off += need;
  }
  const DwRoutes r = dw_routes(dtype, jobs, n > 1);
  const std::vector<DwJob> wide = dw_pick(jobs, r.wide), narrow = dw_pick(jobs, r.narrow), mfma = dw_pick(jobs, r.mfma);
  hipStream_t s = static_cast<hipStream_t>(stream);
  // the partial tiles of both kinds of products are added up by one launch behind the two kernels
  std::vector<ReduceJob> reductions;
  int rc = launch_dw_wide_batched(wide.data(), (int)wide.size(), s, &reductions);
  if (rc == BSR_OK) rc = launch_dw_narrow_batched(narrow.data(), (int)narrow.size(), s, &reductions);
  if (rc == BSR_OK && !reductions.empty()) rc = launch_splitk_reduce_batched(reductions.data(), (int)reductions.size(), s);
  if (rc == BSR_OK) rc = launch_dw_mfma_batched(dtype, mfma.data(), (int)mfma.size(), s);
  for (size_t i = 0; rc == BSR_OK && i < r.single.size(); ++i) rc = launch_dw(dtype, jobs[r.single[i]], s);
  return rc;
}

size_t bsr_compress_batched_workspace_bytes(const bsr_compress_item *items, int n, int dtype) {
  if (items == nullptr || n <= 0) return 0;
  size_t total = 0;
  for (int i = 0; i < n; ++i) {
    const bsr_compress_item &it = items[i];
    Geometry g;
    if (check_shape(dtype, it.M, it.K, it.ldx, it.br, it.bc, &g) != BSR_OK) return 0;
    total += align_up(compress_ws_bytes(dtype, it.M, it.K, it.br, it.bc), 256);
  }
  return total;
}

int bsr_compress_batched(const bsr_compress_item *items, int n, int dtype, void *ws, size_t ws_bytes,
                         void *stream) {
  if (n < 0) return BSR_ERR_SHAPE;
  if (n == 0) return BSR_OK;
  if (items == nullptr) return BSR_ERR_NULL;
  if (misaligned(ws, 16)) return BSR_ERR_ALIGN;
  std::vector<CompressJob> jobs;
  jobs.reserve((size_t)n);
  size_t off = 0;
  for (int i = 0; i < n; ++i) {
    const bsr_compress_item &it = items[i];
    Geometry g;
    const int rc = check_shape(dtype, it.M, it.K, it.ldx, it.br, it.bc, &g);
    if (rc != BSR_OK) return rc;
    if (it.n_keep < 0 || it.n_keep > g.nblocks) return BSR_ERR_KEEP;
    const size_t need = align_up(compress_ws_bytes(dtype, it.M, it.K, it.br, it.bc), 256);
    if (need > 0 && (ws == nullptr || off + need > ws_bytes)) return BSR_ERR_WORKSPACE;
    if (it.row_ptr == nullptr) return BSR_ERR_NULL;
    if (g.nblocks > 0 && (it.X == nullptr || it.keep_mask == nullptr)) return BSR_ERR_NULL;
    if (it.n_keep > 0 && (it.col_idx == nullptr || it.values == nullptr)) return BSR_ERR_NULL;
    if (misaligned(it.X, elem_bytes(dtype)) || misaligned(it.values, elem_bytes(dtype)) ||
        misaligned(it.row_ptr, 4) || misaligned(it.col_idx, 4))
      return BSR_ERR_ALIGN;
    jobs.push_back(CompressJob{it.keep_mask, it.X, it.M, it.K, it.ldx, it.br, it.bc, it.n_keep, it.row_ptr,
                               it.col_idx, it.values, need > 0 ? static_cast<char *>(ws) + off : nullptr});
    off += need;
  }
  return launch_compress_batched(jobs.data(), (int)jobs.size(), dtype, static_cast<hipStream_t>(stream));
}

int bsr_decompress_batched(const bsr_decompress_item *items, int n, int dtype, void *stream) {
  if (n < 0) return BSR_ERR_SHAPE;
  if (n == 0) return BSR_OK;
  if (items == nullptr) return BSR_ERR_NULL;
  std::vector<DecompressJob> jobs;
  jobs.reserve((size_t)n);
  for (int i = 0; i < n; ++i) {
    const bsr_decompress_item &it = items[i];
    Geometry g;
    const int rc = check_shape(dtype, it.M, it.K, it.ldx, it.br, it.bc, &g);
    if (rc != BSR_OK) return rc;
    if (g.nblocks == 0) continue;
    if (it.row_ptr == nullptr || it.X_out == nullptr) return BSR_ERR_NULL;
    if (misaligned(it.X_out, elem_bytes(dtype)) || misaligned(it.values, elem_bytes(dtype)) ||
        misaligned(it.row_ptr, 4) || misaligned(it.col_idx, 4))
      return BSR_ERR_ALIGN;
    jobs.push_back(DecompressJob{it.row_ptr, it.col_idx, it.values, it.M, it.K, it.ldx, it.br, it.bc, it.X_out});
  }
  return launch_decompress_batched(jobs.data(), (int)jobs.size(), dtype, static_cast<hipStream_t>(stream));
}

}  // extern "C"
