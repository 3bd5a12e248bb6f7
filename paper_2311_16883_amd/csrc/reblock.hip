// dW for block shapes the matrix-core kernel has no variant of (1 x b row segments
// -- the shape the paper's Table II overheads imply --, b = K whole-row pruning,
// rectangular or odd blocks): the BSR operand is re-tiled into 32x32 blocks in the
// workspace and the 32x32 kernel runs on that.
//
// A matrix-core instruction contracts 16 rows of a 32-column strip at once, so it
// can only skip work where all of those 16 x 32 positions are pruned; with row
// segments that practically never happens, and the arithmetic of the re-tiled
// operand (every 32x32 block present, pruned positions +0.0) is what any
// matrix-core formulation does.  What the BSR form still saves is the memory the
// activation occupies between forward and backward pass (paper Sec. III).
//
// reblock_kernel: a workgroup owns 32 matrix rows x a chunk of columns.  A table in LDS says which stored block
// holds each block position of that part of the matrix (the entries of a block-row may stand in any order); then every
// thread puts together 16-byte vectors of the re-tiled operand, from loads of as many elements as block widths and
// `values` allow, and stores them where they belong.  Bound by memory: the kept values are read once, the re-tiled
// operand is written once, and nothing passes through LDS.  ([25088 x 384] bfloat16 in 1x32 blocks, keep 0.5: 11.0 us,
// where staging the tile in LDS word by word took 14.8; [20322 x 2944] in 1x64 blocks, keep 0.25: 32 us, 134 where each
// of six column chunks walked all entries element by element.)
#include "common.h"

namespace bsr {

namespace {

constexpr int kRbTable = 4096;            // block positions in the table of a workgroup
constexpr int kRbInFlight = 4;            // vectors a thread puts together at a time
constexpr int kRbOnce = 4096;             // blocks longer than this: at most one boundary in 32 rows or in a chunk

// w / d for rows and columns counted from the start of a block: w < d + 512.
__device__ __forceinline__ uint32_t place_div(uint32_t w, uint32_t d, uint32_t magic) {
  return d > (uint32_t)kRbOnce ? (w >= d ? 1u : 0u) : span_div(w, d, magic);
}

// V = elements per load of `values`: a divisor of bc.
template <typename T, int V>
__global__ __launch_bounds__(256) void reblock_kernel(
    const int32_t *__restrict__ row_ptr, const int32_t *__restrict__ col_idx, const T *__restrict__ values, int br,
    int bc, int64_t nbr, int64_t nbc, int64_t nbr2, int64_t nbc2, int kc, int tcols, uint32_t magic_br, uint32_t magic_bc,
    int32_t *__restrict__ rp2, int32_t *__restrict__ ci2, T *__restrict__ values2) {
  __shared__ int32_t slot[kRbTable];        // [block-row][block-column of the chunk]: stored block, -1 if pruned
  const int t = threadIdx.x;
  constexpr int kVec = 16 / (int)sizeof(T);                                     // elements of a vector
  constexpr int kPieces = kVec / V;
  typedef Vec<T, V> Piece;
  const int64_t k0 = (int64_t)blockIdx.x * kc;
  const int64_t j0 = k0 / bc;
  const int c0 = (int)(k0 - j0 * bc);                                           // of the chunk's first column inside its block
  const int ncols = (int)(nbc - j0 < tcols ? nbc - j0 : tcols);
  const int64_t J0 = k0 / 32;
  const int jb = (int)(nbc2 - J0 < kc / 32 ? nbc2 - J0 : kc / 32);              // 32x32 blocks of the chunk
  const int nvec = jb * 32 * (32 / kVec);
  for (int64_t I = blockIdx.y; I < nbr2; I += gridDim.y) {
    const int64_t m0 = I * 32;
    const int64_t i_first = m0 / br;
    const int r0 = (int)(m0 - i_first * br);                                    // of the first row inside its block-row
    int64_t i_last = (m0 + 31) / br;
    if (i_last > nbr - 1) i_last = nbr - 1;
    const int ni = (int)(i_last - i_first + 1);                                 // source block-rows: 1 .. 32
    // the entries of a block-row are dealt to a few lanes (256 / 32 at least)
    int per_row = 8;
    while (2 * per_row * ni <= 256) per_row *= 2;
    const int rr = t / per_row, sub = t & (per_row - 1);
    const int32_t p0 = rr < ni ? row_ptr[i_first + rr] : 0, p1 = rr < ni ? row_ptr[i_first + rr + 1] : 0;
    for (int e = t; e < ni * tcols; e += 256) slot[e] = -1;
    __syncthreads();
    constexpr int kTogether = 4;                                                // entries a lane requests at a time
    for (int32_t pb = p0 + sub; pb < p1; pb += kTogether * per_row) {
      int64_t j[kTogether];
#pragma unroll
      for (int u = 0; u < kTogether; ++u) j[u] = pb + u * per_row < p1 ? (int64_t)col_idx[pb + u * per_row] - j0 : -1;
#pragma unroll
      for (int u = 0; u < kTogether; ++u)
        if (j[u] >= 0 && j[u] < ncols) slot[rr * tcols + (int)j[u]] = pb + u * per_row;
    }
    __syncthreads();
    // ---- the 32x32 blocks of the chunk, vector after vector ----
    T *const out = values2 + (I * nbc2 + J0) * 1024;
    for (int v0 = t; v0 < nvec; v0 += 256 * kRbInFlight) {
      Piece x[kRbInFlight][kPieces];
#pragma unroll
      for (int k = 0; k < kRbInFlight; ++k) {
        const uint32_t v = (uint32_t)(v0 + 256 * k);
        const uint32_t r = (v / (32 / kVec)) % 32, c = (v / 32) / (32 / kVec) * 32 + v % (32 / kVec) * kVec;
        const uint32_t br_row = (uint32_t)r0 + r, brr = place_div(br_row, (uint32_t)br, magic_br);
        const uint32_t in_row = br_row - brr * (uint32_t)br;
        const bool live = (int)v < nvec && (int)brr < ni;
#pragma unroll
        for (int q = 0; q < kPieces; ++q) {
          const uint32_t col = (uint32_t)c0 + c + (uint32_t)(q * V), jl = place_div(col, (uint32_t)bc, magic_bc);
          const int32_t p = live && (int)jl < ncols ? slot[brr * (uint32_t)tcols + jl] : -1;
          if (p >= 0) {
            x[k][q] = *reinterpret_cast<const Piece *>(values + ((int64_t)p * br + in_row) * bc + (col - jl * (uint32_t)bc));
          } else {
#pragma unroll
            for (int i = 0; i < V; ++i) x[k][q].e[i] = (T)0;
          }
        }
      }
#pragma unroll
      for (int k = 0; k < kRbInFlight; ++k) {
        const int v = v0 + 256 * k;
        if (v < nvec) {
          Vec<T, kVec> y;
#pragma unroll
          for (int q = 0; q < kPieces; ++q)
#pragma unroll
            for (int i = 0; i < V; ++i) y.e[q * V + i] = x[k][q].e[i];
          *reinterpret_cast<Vec<T, kVec> *>(out + (int64_t)v * kVec) = y;
        }
      }
    }
    if (blockIdx.x == 0) {
      for (int64_t J = t; J < nbc2; J += 256) ci2[I * nbc2 + J] = (int32_t)(J);
      if (t == 0) {
        rp2[I] = (int32_t)(I * nbc2);
        if (I == nbr2 - 1) rp2[nbr2] = (int32_t)(nbr2 * nbc2);
      }
    }
    __syncthreads();                        // the table is free for the next rows
  }
}

struct ReblockPlan {
  int64_t nbr2, nbc2;
  size_t values_off, rp_off, ci_off, inner_off, total;
};

ReblockPlan reblock_plan(int dtype, int64_t M, int64_t K, int64_t N) {
  ReblockPlan p;
  p.nbr2 = ceil_div(M, 32);
  p.nbc2 = ceil_div(K, 32);
  p.values_off = 0;
  p.rp_off = align_up((size_t)p.nbr2 * p.nbc2 * 1024 * elem_bytes(dtype), 256);
  p.ci_off = p.rp_off + align_up((size_t)(p.nbr2 + 1) * 4, 256);
  p.inner_off = p.ci_off + align_up((size_t)p.nbr2 * p.nbc2 * 4, 256);
  p.total = p.inner_off + align_up(dw_mfma_ws_bytes(dtype, M, K, N, 32, 32), 256);
  return p;
}

}  // namespace

bool dw_reblock_supported(int dtype, int br, int bc, int64_t M, int64_t K, int64_t N, int64_t lddy) {
  if (M <= 0 || K <= 0 || N <= 0) return false;
  if (ceil_div(M, 32) * ceil_div(K, 32) >= (int64_t(1) << 31)) return false;
  (void)br;
  (void)bc;
  return dw_mfma_supported(dtype, 32, 32, nullptr, M, K, N, lddy);
}

size_t dw_reblock_ws_bytes(int dtype, int64_t M, int64_t K, int64_t N) { return reblock_plan(dtype, M, K, N).total; }

int launch_dw_reblocked(int dtype, const int32_t *row_ptr, const int32_t *col_idx, const void *values, int64_t M,
                        int64_t K, int br, int bc, const void *dY, int64_t N, int64_t lddy, float *dW,
                        int64_t lddw, int accumulate, void *ws, size_t ws_bytes, hipStream_t s) {
  const ReblockPlan p = reblock_plan(dtype, M, K, N);
  if (ws_bytes < p.total) return BSR_ERR_WORKSPACE;
  char *w = static_cast<char *>(ws);
  int32_t *rp2 = reinterpret_cast<int32_t *>(w + p.rp_off);
  int32_t *ci2 = reinterpret_cast<int32_t *>(w + p.ci_off);
  const int e = elem_bytes(dtype);
  const int64_t k2 = p.nbc2 * 32;
  const int64_t nbr = ceil_div(M, br), nbc = ceil_div(K, bc);
  // Columns of a chunk: as many as give a thread eight vectors (fewer workgroups scan a row's entries then), or fewer
  // where the table of very small blocks would not fit.  Chunks start on multiples of 32 columns, tiles on multiples of
  // 32 rows: blocks that do not divide 32 may reach over both ends.
  auto spanned = [](int64_t n, int64_t b) { return 32 % b == 0 ? n / b : (n + b - 2) / b + 1; };
  const int64_t table_rows = spanned(32, br);
  auto table_cols = [&](int64_t c) { return spanned(c, bc); };
  int64_t kc = 16384 / e / 16;
  while (kc > 32 && table_rows * table_cols(kc) > kRbTable) kc -= 32;
  if (kc > k2) kc = k2;
  const int tcols = (int)table_cols(kc);
  const dim3 grid((unsigned)ceil_div(k2, kc), (unsigned)(p.nbr2 < 65535 ? p.nbr2 : 65535));
  auto magic = [](uint32_t d) { return (uint32_t)(((uint64_t(1) << 32) + d - 1) / d); };
#define BSR_REBLOCK(T, V)                                                                                   \
  hipLaunchKernelGGL((reblock_kernel<T, V>), grid, dim3(256), 0, s, row_ptr, col_idx,                       \
                     static_cast<const T *>(values), br, bc, nbr, nbc, p.nbr2, p.nbc2, (int)kc, tcols,      \
                     magic((uint32_t)br), magic((uint32_t)bc), rp2, ci2, reinterpret_cast<T *>(w + p.values_off))
  const int v = pick_vector(16 / e, e, bc, bc, bc, values);
  if (dtype == BSR_F32) {
    switch (v) {
      case 4: BSR_REBLOCK(float, 4); break;
      case 2: BSR_REBLOCK(float, 2); break;
      default: BSR_REBLOCK(float, 1); break;
    }
  } else {
    switch (v) {
      case 8: BSR_REBLOCK(uint16_t, 8); break;
      case 4: BSR_REBLOCK(uint16_t, 4); break;
      case 2: BSR_REBLOCK(uint16_t, 2); break;
      default: BSR_REBLOCK(uint16_t, 1); break;
    }
  }
#undef BSR_REBLOCK
  const int rc = check_launch();
  if (rc != BSR_OK) return rc;
  return launch_dw_mfma(dtype, rp2, ci2, w + p.values_off, M, K, 32, 32, dY, N, lddy, dW, lddw, accumulate,
                        w + p.inner_off, ws_bytes - p.inner_off, s);
}

}  // namespace bsr
