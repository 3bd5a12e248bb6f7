// Top-k block selection (paper Sec. IV: the k lowest-ranked blocks are pruned).
//
// Exact selection of the n_keep best blocks in the total order
//   (score descending, linear block index ascending)
// without sorting everything and without a host round trip.  key is the bit
// pattern of the non-negative binary64 score (orders like the value; any NaN
// becomes one quiet-NaN pattern above +inf), so all arithmetic is integer and
// the result is the same on every run.
//
// Building blocks.  radix_select: one workgroup, most-significant-digit-first
// radix select (12-bit digits) on the 96-bit rank value
// C = key * 2^32 + (nblocks-1-index): histogram of the current digit over the
// elements that still match the chosen prefix, suffix scan for the digit holding
// the n_keep-th element, repeat; once the matching set fits in LDS it is ranked
// exactly by counting, which settles ties through the index part of C.  It works
// for any input and is the fallback of bracketed_select, which is much faster
// when the caller can bracket the threshold's key (see there).
//
// Small inputs (<= 12288 blocks) and per-group selection: one workgroup per
// ranking group.  Keys are read once, four consecutive ones per thread, and stay
// in registers; bracketed_select between the group's smallest and largest key.
//
// Large inputs: two grid-wide passes, two launches.
//   pass 1  every workgroup draws the same small sample, takes from it two order
//           statistics lo <= hi that bracket the rank of the threshold, and
//           counts its slice of the keys into 256 buckets: bucket 0 below lo, the
//           last bucket above hi, equal-width buckets in between -- those on
//           either side of a gap, where the sample shows that nothing lies in most
//           of [lo, hi] (any monotone bucketing keeps the selection exact; a good
//           one only makes the threshold bucket small).  Each workgroup stores its
//           own counts: no atomics, nothing to clear.
//   pass 2  every workgroup adds up the counts, finds the bucket that holds the
//           n_keep-th largest key, keeps the buckets above it, prunes the ones
//           below and lists the keys inside it, at places that follow from the
//           counts (no atomics on memory).  The workgroup that finishes last selects among the
//           candidates exactly, with the bucket's key range as a bracket: 32-bit
//           codes linear in the key, one radix pass as a rule, then a ranking of
//           the handful that share the threshold's code through lane reads.  The
//           general radix select remains the fallback when a bracket misses or
//           too many keys are equal.
//
// What bounds it is latency: a launch, a trip to memory, a handful of barriers.
// So lane exchanges inside a wave are DPP moves (no LDS round trips), a key is
// read once per pass with 16-byte loads, and mask bytes leave four at a time.
#include <cmath>

#include "common.h"

namespace bsr {

namespace {

constexpr int kDigitBits = 12;
constexpr int kBins = 1 << kDigitBits;
constexpr int kCap = 1024;       // candidates ranked in LDS
constexpr int kSample = 128;
constexpr int kGridThreads = 1024;
constexpr int kBuckets = 256;    // buckets of the grid-wide passes
constexpr int kMaxGridWgs = 256; // workgroups of the grid-wide passes, at most
constexpr int kFinishBits = 10;  // digit of the selection among up to kCap candidates: a bin per thread
constexpr int kRankedAtOnce = 96;   // candidates that are ranked without a radix pass, at most
constexpr int kFinishKeys = 8;   // of longer lists, candidates per thread that are taken into registers

typedef unsigned __int128 u128;

__device__ __forceinline__ uint64_t score_key(double s) {
  if (s != s) return 0x7FF8000000000000ull;
  return (uint64_t)__double_as_longlong(s);
}

__device__ __forceinline__ u128 rank_value(uint64_t key, uint32_t inv_idx) {
  return ((u128)key << 32) | (u128)inv_idx;
}

// Where the elements to select from live: all scores, or a candidate list.
struct AllScores {
  const double *scores;
  __device__ __forceinline__ uint64_t key(uint32_t e) const { return score_key(scores[e]); }
  __device__ __forceinline__ uint32_t idx(uint32_t e) const { return e; }
};
// (written by workgroups of the same launch, see store_shared)
struct Candidates {
  const uint64_t *keys;
  const uint32_t *idxs;
  __device__ __forceinline__ uint64_t key(uint32_t e) const {
    return __hip_atomic_load(&keys[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ uint32_t idx(uint32_t e) const {
    return __hip_atomic_load(&idxs[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
};

struct Staged {
  const uint64_t *keys;
  const uint32_t *idxs;
  __device__ __forceinline__ uint64_t key(uint32_t e) const { return keys[e]; }
  __device__ __forceinline__ uint32_t idx(uint32_t e) const { return idxs[e]; }
};

// Values that one workgroup hands to another of the same launch: relaxed agent-scope atomic stores go
// through the L2 of their XCD to where every XCD sees them.  Once a wave has waited for its stores
// (stores_done), a flag it raises afterwards tells a reader -- which uses agent-scope atomic loads --
// that they are there.  A release fence would do the same by writing the whole L2 back.
template <typename U>
__device__ __forceinline__ void store_shared(U *p, U v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// ---- lane exchanges inside a wave by DPP: rows of 16 lanes shifted by 1, 2, 4, 8, then the last lane
// of a row broadcast to the next row (0x142), that of lane 31 to the upper half (0x143) ----
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp(uint32_t identity, uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)identity, (int)v, CTRL, ROWS, 0xF, false);
}
// inclusive prefix sum over the 64 lanes
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
  v += dpp<0x111, 0xF>(0u, v);
  v += dpp<0x112, 0xF>(0u, v);
  v += dpp<0x114, 0xF>(0u, v);
  v += dpp<0x118, 0xF>(0u, v);
  v += dpp<0x142, 0xA>(0u, v);
  v += dpp<0x143, 0xC>(0u, v);
  return v;
}
__device__ __forceinline__ uint32_t lane_value(uint32_t v, int lane) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) { return lane_value(wave_scan(v), 63); }
template <bool MAX>
__device__ __forceinline__ uint32_t pick(uint32_t a, uint32_t b) { return MAX ? (a > b ? a : b) : (a < b ? a : b); }
// largest / smallest of the 64 lanes, in every lane
template <bool MAX>
__device__ __forceinline__ uint32_t wave_extreme(uint32_t v) {
  constexpr uint32_t id = MAX ? 0u : 0xFFFFFFFFu;
  v = pick<MAX>(v, dpp<0x111, 0xF>(id, v));
  v = pick<MAX>(v, dpp<0x112, 0xF>(id, v));
  v = pick<MAX>(v, dpp<0x114, 0xF>(id, v));
  v = pick<MAX>(v, dpp<0x118, 0xF>(id, v));
  v = pick<MAX>(v, dpp<0x142, 0xA>(id, v));
  v = pick<MAX>(v, dpp<0x143, 0xC>(id, v));
  return lane_value(v, 63);
}

// Keys of elements e .. e + 3 (0 beyond n).  `wide`: scores is 16-byte aligned (e is a multiple of four).
__device__ __forceinline__ void load_keys4(const double *__restrict__ scores, uint32_t e, uint32_t n, bool wide,
                                           uint64_t *k) {
  if (wide && e + 4 <= n) {
    const double2 a = *reinterpret_cast<const double2 *>(scores + e), b = *reinterpret_cast<const double2 *>(scores + e + 2);
    k[0] = score_key(a.x); k[1] = score_key(a.y); k[2] = score_key(b.x); k[3] = score_key(b.y);
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q) k[q] = e + q < n ? score_key(scores[e + q]) : 0ull;
  }
}
// Mask bytes of elements e .. e + 3: the bytes of `word` whose bit in `own` is set (all four leave in one
// store when mask is 4-byte aligned, `wide`).
__device__ __forceinline__ void store_mask4(uint8_t *__restrict__ mask, uint32_t e, bool wide, uint32_t own, uint32_t word) {
  if (wide && own == 0xFu) {
    *reinterpret_cast<uint32_t *>(mask + e) = word;
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (own & (1u << q)) mask[e + q] = (uint8_t)(word >> (8 * q));
  }
}

struct SelectShared {
  __attribute__((aligned(16))) uint32_t hist[kBins];
  uint64_t ckey[kCap];
  uint32_t cidx[kCap];
  uint32_t wave_tot[16];
  uint32_t digit, above, count, n;
};

// Exclusive prefix sum over the THREADS threads of the block.
template <int THREADS>
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *wave_tot) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t incl = wave_scan(v);
  if (lane == 63) wave_tot[wave] = incl;
  __syncthreads();
  const uint32_t tot = wave_tot[lane & (THREADS / 64 - 1)];
  const uint32_t upto = wave_scan(lane < THREADS / 64 ? tot : 0u);
  const uint32_t base = wave > 0 ? lane_value(upto, __builtin_amdgcn_readfirstlane(wave > 0 ? wave - 1 : 0)) : 0u;
  __syncthreads();
  return base + incl - v;
}

template <int THREADS>
__device__ __forceinline__ void rank_candidates(SelectShared &sh, uint32_t m, uint32_t want,
                                                uint8_t *__restrict__ mask);

// One workgroup marks the `want` best of the n elements of `src` in mask
// (1 = kept, 0 = pruned); every element of src gets its byte written.
template <int THREADS, typename Source>
__device__ void radix_select(const Source &src, uint32_t n, uint32_t want, uint32_t nblocks,
                             uint8_t *__restrict__ mask, SelectShared &sh) {
  const int t = threadIdx.x;
  constexpr int kPerThread = kBins / THREADS;
  u128 prefix = 0;          // the top 12*level bits every candidate shares
  int level = 0;
  uint32_t n_cand = n;

  while (n_cand > (uint32_t)kCap) {   // distinct C: at most one candidate is left after all 8 digits
    for (int b = t; b < kBins; b += THREADS) sh.hist[b] = 0;
    __syncthreads();
    const int shift_prefix = 96 - kDigitBits * level;
    const int shift_digit = shift_prefix - kDigitBits;
    for (uint32_t e = t; e < n; e += THREADS) {
      const u128 c = rank_value(src.key(e), nblocks - 1 - src.idx(e));
      if (level == 0 || (c >> shift_prefix) == prefix)
        atomicAdd(&sh.hist[(uint32_t)(c >> shift_digit) & (kBins - 1)], 1u);
    }
    __syncthreads();
    // thread t owns kPerThread bins, descending digits
    uint32_t h[kPerThread], own = 0;
#pragma unroll
    for (int u = 0; u < kPerThread; ++u) {
      h[u] = sh.hist[kBins - 1 - (kPerThread * t + u)];
      own += h[u];
    }
    uint32_t above = block_exclusive_scan<THREADS>(own, sh.wave_tot);
#pragma unroll
    for (int u = 0; u < kPerThread; ++u) {
      if (above < want && want <= above + h[u]) {
        sh.digit = (uint32_t)(kBins - 1 - (kPerThread * t + u));
        sh.above = above;
        sh.count = h[u];
      }
      above += h[u];
    }
    __syncthreads();
    prefix = (prefix << kDigitBits) | (u128)sh.digit;
    want -= sh.above;
    n_cand = sh.count;
    ++level;
    __syncthreads();
  }

  // Everything above the prefix is kept, everything below pruned, the
  // candidates that match it are ranked in LDS.
  if (t == 0) sh.n = 0;
  __syncthreads();
  const int shift_prefix = 96 - kDigitBits * level;
  for (uint32_t e = t; e < n; e += THREADS) {
    const uint64_t key = src.key(e);
    const uint32_t idx = src.idx(e);
    bool inside = true;
    if (level > 0) {
      const u128 top = rank_value(key, nblocks - 1 - idx) >> shift_prefix;
      if (top != prefix) {
        inside = false;
        mask[idx] = top > prefix ? 1 : 0;
      }
    }
    if (inside) {
      const uint32_t pos = atomicAdd(&sh.n, 1u);
      sh.ckey[pos] = key;
      sh.cidx[pos] = idx;
    }
  }
  __syncthreads();
  rank_candidates<THREADS>(sh, sh.n, want, mask);
}

// Selection with a bracket.  The caller knows (or hopes) that the want-th best
// of the n elements of `src` has its key inside [lo, hi].  Thread t holds the keys of
// elements 4 (t + g THREADS) + 0 .. 3 in registers (g = 0 .. KPT / 4 - 1).  Keys above hi
// are only counted; keys inside get a 32-bit code, 1 + ((key - lo) >> shift), for the
// radix passes that find the code of the threshold: the codes spread evenly over the
// bracket, so usually one pass with next to no bin shared.  key -> code is monotone, so
// a larger (smaller) code than the threshold's means kept (pruned) for certain;
// the few elements that share the threshold's code are ranked exactly on their
// full keys and indices.  If the bracket misses the threshold or more than kCap
// elements share its code (e.g. very many all-zero blocks), the general radix
// select takes over.  Every element of src gets its mask byte written.
struct BracketShared {
  uint32_t wave_cnt[2][16];
};

// Exact ranking of the m candidates listed in sh.ckey / sh.cidx: the `want` best
// in (key descending, index ascending) order are kept.  Up to 64 candidates sit
// one per lane of the first wave and are compared through lane reads (no LDS
// round trip per comparison); longer lists (many equal keys) go through LDS.
template <int THREADS>
__device__ __forceinline__ void rank_candidates(SelectShared &sh, uint32_t m, uint32_t want,
                                                uint8_t *__restrict__ mask) {
  const int t = threadIdx.x;
  if (m <= 64u) {
    if (t < 64) {
      const bool live = (uint32_t)t < m;
      const uint64_t k = live ? sh.ckey[t] : 0ull;
      const uint32_t idx = live ? sh.cidx[t] : 0u;
      const uint32_t klo = (uint32_t)k, khi = (uint32_t)(k >> 32);
      uint32_t better = 0;   // candidates that rank strictly before this one
      for (uint32_t o = 0; o < m; ++o) {
        const uint64_t ok = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)khi, (int)o) << 32) |
                            (uint32_t)__builtin_amdgcn_readlane((int)klo, (int)o);
        const uint32_t oidx = (uint32_t)__builtin_amdgcn_readlane((int)idx, (int)o);
        better += (ok > k || (ok == k && oidx < idx)) ? 1u : 0u;
      }
      if (live) mask[idx] = better < want ? 1 : 0;
    }
    return;
  }
  if (m <= (uint32_t)THREADS) {
    // the m x m comparisons are spread over all threads: `parts` threads share one
    // candidate, each counts over its own range of opponents
    const uint32_t parts = (uint32_t)THREADS / m, chunk = (m + parts - 1) / parts;
    for (uint32_t c = t; c < m; c += THREADS) sh.hist[c] = 0;
    __syncthreads();
    const uint32_t c = (uint32_t)t % m, part = (uint32_t)t / m;
    if (part < parts) {
      const uint64_t k = sh.ckey[c];
      const uint32_t idx = sh.cidx[c];
      const uint32_t o0 = part * chunk, o1 = (o0 + chunk) < m ? (o0 + chunk) : m;
      uint32_t better = 0;
#pragma unroll 4
      for (uint32_t o = o0; o < o1; ++o) {
        const uint64_t ok = sh.ckey[o];
        better += (ok > k || (ok == k && sh.cidx[o] < idx)) ? 1u : 0u;
      }
      if (better) atomicAdd(&sh.hist[c], better);
    }
    __syncthreads();
    if ((uint32_t)t < m) mask[sh.cidx[t]] = sh.hist[t] < want ? 1 : 0;
    return;
  }
  for (uint32_t c = t; c < m; c += THREADS) {
    const uint64_t k = sh.ckey[c];
    const uint32_t idx = sh.cidx[c];
    uint32_t better = 0;
#pragma unroll 8
    for (uint32_t o = 0; o < m; ++o) {
      const uint64_t ok = sh.ckey[o];
      better += (ok > k || (ok == k && sh.cidx[o] < idx)) ? 1u : 0u;
    }
    mask[idx] = better < want ? 1 : 0;
  }
}

// DB = bits per radix pass: the pass costs one histogram of 2^DB bins (zeroed,
// filled, scanned by THREADS threads), so small workgroups take small digits.
// ALL: the bracket is known to hold every element.  The caller has zeroed sh.hist[0, 2^DB)
// and passed a barrier since.  wide: src is in linear order and mask is 4-byte aligned.
template <int THREADS, int KPT, int DB, bool ALL, typename Source>
__device__ __forceinline__ void bracketed_select(const uint64_t (&key)[KPT], const Source &src, uint32_t n,
                                                 uint32_t want_total, uint64_t lo, uint64_t hi, uint32_t nblocks,
                                                 bool wide, uint8_t *__restrict__ mask, SelectShared &sh,
                                                 BracketShared &bs) {
  constexpr int kLocalBins = 1 << DB;
  constexpr int kPerThread = kLocalBins / THREADS;
  static_assert(kPerThread >= 1 && kLocalBins <= kBins && KPT % 4 == 0, "one bin per thread at least");
  constexpr uint32_t kAbove = 0xFFFFFFFFu, kBelow = 0u;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const uint64_t range = hi - lo;
  // smallest shift with 1 + (range >> shift) <= 0xFFFFFFFE
  int shift = range == 0 ? 0 : 64 - __clzll((long long)range);          // bit length of range
  shift = shift > 31 ? shift - 31 : 0;

  uint32_t code[KPT];
  uint32_t n_above = 0, n_inside = 0;
#pragma unroll
  for (int i = 0; i < KPT; ++i) {
    const uint32_t e = 4u * (uint32_t)(t + (i >> 2) * THREADS) + (uint32_t)(i & 3);
    uint32_t c = 1u + (uint32_t)((key[i] - lo) >> shift);
    if constexpr (!ALL) c = key[i] > hi ? kAbove : (key[i] < lo ? kBelow : c);
    if (e >= n) c = kBelow;
    if constexpr (!ALL) {
      n_above += c == kAbove ? 1u : 0u;
      n_inside += (c != kAbove && c != kBelow) ? 1u : 0u;
    }
    code[i] = c;
  }
  if constexpr (ALL) {
    n_inside = n;
  } else {
    n_above = wave_sum(n_above);
    n_inside = wave_sum(n_inside);
    if (lane == 0) { bs.wave_cnt[0][wave] = n_above; bs.wave_cnt[1][wave] = n_inside; }
    __syncthreads();
    n_above = wave_sum(lane < THREADS / 64 ? bs.wave_cnt[0][lane & (THREADS / 64 - 1)] : 0u);
    n_inside = wave_sum(lane < THREADS / 64 ? bs.wave_cnt[1][lane & (THREADS / 64 - 1)] : 0u);
  }

  // bits [ctop, 32) of the threshold's code are settled and equal cprefix
  int ctop = 32;
  // (codes reach no further up than the bit length of the largest one)
  if constexpr (ALL) {
    const uint32_t top = 1u + (uint32_t)(range >> shift);
    ctop = 32 - __clz((int)top);
  }
  const int ctop0 = ctop;
  uint32_t cprefix = 0, want = want_total - n_above, n_cand = n_inside;
  const bool bracketed = want_total > n_above && want <= n_inside;
  while (bracketed && n_cand > 64u && ctop > 0) {
    const int dshift = ctop > DB ? ctop - DB : 0;
    const uint32_t dmask = (1u << (ctop - dshift)) - 1u;
    if (ctop != ctop0) {                                     // (the first histogram was zeroed by the caller)
      for (int b = t; b < kLocalBins; b += THREADS) sh.hist[b] = 0;
      __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < KPT; ++i) {
      const uint32_t c = code[i];
      if (c != kAbove && c != kBelow && (ctop == ctop0 || (c >> ctop) == cprefix))
        atomicAdd(&sh.hist[(c >> dshift) & dmask], 1u);
    }
    __syncthreads();
    uint32_t h[kPerThread], own = 0;
#pragma unroll
    for (int u = 0; u < kPerThread; ++u) {
      h[u] = sh.hist[kLocalBins - 1 - (kPerThread * t + u)];
      own += h[u];
    }
    uint32_t above = block_exclusive_scan<THREADS>(own, sh.wave_tot);
#pragma unroll
    for (int u = 0; u < kPerThread; ++u) {
      if (above < want && want <= above + h[u]) {
        sh.digit = (uint32_t)(kLocalBins - 1 - (kPerThread * t + u));
        sh.above = above;
        sh.count = h[u];
      }
      above += h[u];
    }
    if (t == 0) sh.n = 0;
    __syncthreads();
    cprefix = ctop == ctop0 ? sh.digit : ((cprefix << (ctop - dshift)) | sh.digit);
    want -= sh.above;
    n_cand = sh.count;
    ctop = dshift;
    if (n_cand > 64u && ctop > 0) __syncthreads();           // (another pass writes what was just read)
  }
  if (!bracketed || n_cand > (uint32_t)kCap) {
    __syncthreads();
    radix_select<THREADS>(src, n, want_total, nblocks, mask, sh);
    return;
  }

  // larger code: kept; smaller: pruned; equal: ranked exactly on the full keys
  if (ctop == ctop0) {                                       // no pass was run: sh.n is not set yet
    if (t == 0) sh.n = 0;
    __syncthreads();
  }
#pragma unroll
  for (int g = 0; g < KPT / 4; ++g) {
    const uint32_t e = 4u * (uint32_t)(t + g * THREADS);
    if (e >= n) continue;
    uint32_t own = 0, word = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (e + q < n) {
        const uint32_t c = code[4 * g + q];
        const bool inside = c != kAbove && c != kBelow;
        // with no pass run every element inside the bracket is a candidate
        const uint32_t chi = ctop == ctop0 ? 0u : c >> ctop;
        if (inside && chi == cprefix) {
          const uint32_t pos = atomicAdd(&sh.n, 1u);
          sh.ckey[pos] = key[4 * g + q];
          sh.cidx[pos] = src.idx(e + q);
        } else {
          const uint32_t kept = (c == kAbove || (inside && chi > cprefix)) ? 1u : 0u;
          if (!wide) mask[src.idx(e + q)] = (uint8_t)kept;
          else word |= kept << (8 * q);
        }
        own |= 1u << q;      // (a candidate's byte is written again below, behind the barrier)
      }
    }
    if (wide) store_mask4(mask, e, true, own, word);
  }
  __syncthreads();
  rank_candidates<THREADS>(sh, sh.n, want, mask);
}

// Per-group selection (paper Sec. IV: blocks are only compared inside one
// activation of the mini-batch): a ranking group is `group_blocks` consecutive
// blocks in linear order (whole block-rows); workgroup g selects inside group g
// with indices local to the group.  The group's smallest and largest key serve
// as the bracket of bracketed_select: codes linear in the key, a radix pass or
// two, exact ranking of what shares the threshold's code.  The last group may be
// shorter (last_blocks, keeping n_keep_last).
// One workgroup selects the `want` best of the n scores at `scores` into gmask.
// (12288 scores take 7.5 us, 13 before keys were kept in registers and lane exchanges became DPP moves.)
template <int THREADS, int KPT, int DB>
__device__ __forceinline__ void select_one_group(const double *__restrict__ scores, uint32_t n, uint32_t want,
                                                 uint8_t *__restrict__ gmask, SelectShared &sh, BracketShared &bs) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  if (want == 0 || want >= n) {
    for (uint32_t e = t; e < n; e += THREADS) gmask[e] = want > 0 ? 1 : 0;
    return;
  }
  const bool wide_in = (uintptr_t)scores % 16 == 0, wide_out = (uintptr_t)gmask % 4 == 0;
  uint64_t key[KPT];
#pragma unroll
  for (int g = 0; g < KPT / 4; ++g) load_keys4(scores, 4u * (uint32_t)(t + g * THREADS), n, wide_in, &key[4 * g]);
  for (int b = t; b < (1 << DB); b += THREADS) sh.hist[b] = 0;
  // the bracket: smallest and largest high word
  uint32_t mn = 0xFFFFFFFFu, mx = 0u;
#pragma unroll
  for (int i = 0; i < KPT; ++i) {
    const uint32_t e = 4u * (uint32_t)(t + (i >> 2) * THREADS) + (uint32_t)(i & 3);
    const uint32_t h = (uint32_t)(key[i] >> 32);
    mn = pick<false>(mn, e < n ? h : 0xFFFFFFFFu);
    mx = pick<true>(mx, h);
  }
  mn = wave_extreme<false>(mn);
  mx = wave_extreme<true>(mx);
  if (lane == 0) { bs.wave_cnt[0][wave] = mn; bs.wave_cnt[1][wave] = mx; }
  __syncthreads();
  mn = wave_extreme<false>(bs.wave_cnt[0][lane & (THREADS / 64 - 1)]);
  mx = wave_extreme<true>(bs.wave_cnt[1][lane & (THREADS / 64 - 1)]);
  bracketed_select<THREADS, KPT, DB, true>(key, AllScores{scores}, n, want, (uint64_t)mn << 32,
                                           ((uint64_t)mx << 32) | 0xFFFFFFFFull, n, wide_out, gmask, sh, bs);
}

template <int THREADS, int KPT, int DB>
__global__ __launch_bounds__(THREADS) void select_groups_kernel(
    const double *__restrict__ scores, uint32_t group_blocks, uint32_t n_keep_group, uint32_t last_blocks,
    uint32_t n_keep_last, uint8_t *__restrict__ mask) {
  __shared__ SelectShared sh;
  __shared__ BracketShared bs;
  const bool last = blockIdx.x == gridDim.x - 1;
  const size_t off = (size_t)blockIdx.x * group_blocks;
  select_one_group<THREADS, KPT, DB>(scores + off, last ? last_blocks : group_blocks,
                                     last ? n_keep_last : n_keep_group, mask + off, sh, bs);
}

// Per-group selection of several tensors in one launch: tensor k owns the workgroups
// [wg_begin_k, wg_begin_k + groups_k), one workgroup per group.
constexpr int kGroupBatchMax = 24;
struct GroupItem {
  const double *scores;
  uint8_t *mask;
  uint32_t group_blocks, n_keep_group, last_blocks, n_keep_last, groups, wg_begin;
};
struct GroupBatch {
  GroupItem it[kGroupBatchMax];
};
template <int THREADS, int KPT, int DB>
__global__ __launch_bounds__(THREADS) void select_groups_batched_kernel(GroupBatch b, int n) {
  __shared__ SelectShared sh;
  __shared__ BracketShared bs;
  int k = 0;
  while (k + 1 < n && blockIdx.x >= b.it[k + 1].wg_begin) ++k;
  const GroupItem &it = b.it[k];
  const uint32_t g = blockIdx.x - it.wg_begin;
  const bool last = g == it.groups - 1;
  const size_t off = (size_t)g * it.group_blocks;
  select_one_group<THREADS, KPT, DB>(it.scores + off, last ? it.last_blocks : it.group_blocks,
                                     last ? it.n_keep_last : it.n_keep_group, it.mask + off, sh, bs);
}

// Control block shared by the two grid-wide passes (lives in the workspace;
// written by workgroup 0 of pass 1).
// The bucketing of the keys: 0 below lo, kBuckets - 1 above hi, between them buckets 2^shift wide.  mid != 0: the
// keys in [lo, mid) go to buckets 1 .. kGapBucket, the last of which takes all of the gap in front of mid, those in
// [mid, hi] to the buckets behind them, 2^shift_mid wide.
struct Buckets {
  uint64_t lo, hi, mid;
  uint32_t shift, shift_mid;
};
constexpr uint32_t kGapBucket = kBuckets / 2;
struct SelectCtrl {
  Buckets buckets;
  uint32_t done;            // workgroups of pass 2 that have listed their candidates
};

__device__ __forceinline__ uint32_t bucket_of(uint64_t key, const Buckets &b) {
  if (key < b.lo) return 0u;
  if (key > b.hi) return (uint32_t)kBuckets - 1u;
  if (__builtin_expect(b.mid != 0, 0)) {                                  // (the same in all lanes)
    if (key >= b.mid) return kGapBucket + 1u + (uint32_t)((key - b.mid) >> b.shift_mid);
    const uint64_t at = (key - b.lo) >> b.shift;
    return at < (uint64_t)(kGapBucket - 1u) ? 1u + (uint32_t)at : kGapBucket;
  }
  return 1u + (uint32_t)((key - b.lo) >> b.shift);
}
// Smallest shift with (range >> shift) <= last, last < 2^bits and as few of them as possible.
__device__ __forceinline__ uint32_t bucket_shift(uint64_t range, uint32_t bits, uint32_t last) {
  uint32_t shift = range == 0 ? 0u : (uint32_t)(64 - __clzll((long long)range));   // bit length of range
  shift = shift > bits ? shift - bits : 0u;
  return (range >> shift) > (uint64_t)last ? shift + 1u : shift;
}

// What one selection needs in the kernel arguments.  wgs == 0: the one-workgroup selection.
struct SelectItem {
  const double *scores;
  uint8_t *mask;
  uint32_t nblocks, n_keep, per_wg, wgs;
  uint32_t rank_lo, rank_hi;    // order statistics of the sample that bracket the threshold (pass 1)
  uint32_t *counts;
  SelectCtrl *ctrl;
  uint64_t *cand_key;
  uint32_t *cand_idx;
};

// Pass 1 of workgroup `wg` of a selection.  Its slice is per_wg blocks (a multiple of four).
__device__ __forceinline__ void select_count_body(const SelectItem &it, const uint32_t wg) {
  __shared__ uint32_t hist[kBuckets];
  __shared__ __attribute__((aligned(16))) uint32_t sample[kSample];
  __shared__ uint32_t ranks[kSample], sorted[kSample];
  const int t = threadIdx.x;
  const double *__restrict__ scores = it.scores;
  const uint32_t nblocks = it.nblocks;
  const bool wide = (uintptr_t)scores % 16 == 0;
  const uint32_t e0 = wg * it.per_wg;
  const uint32_t e1 = (e0 + it.per_wg) < nblocks ? (e0 + it.per_wg) : nblocks;

  // the same sample in every workgroup: a key from each of kSample equal stretches, at a scattered place
  // of its stretch (even spacing would meet the same few block-columns again and again), of each the upper 25 bits (more than
  // enough for a bracket) and its position below them, which makes them distinct; and the first four
  // keys per thread of the slice, on their way while the sample is ranked
  constexpr uint32_t kPosBits = kSample - 1;
  if (t < kSample) {
    const uint32_t stretch = nblocks / kSample, at = (uint32_t)((uint64_t)t * nblocks / kSample);
    const uint32_t e = at + __umulhi((uint32_t)t * 2654435769u, stretch);
    sample[t] = ((uint32_t)(score_key(scores[e]) >> 32) & ~kPosBits) | (uint32_t)t;
    ranks[t] = 0;
  }
  if (t < kBuckets) hist[t] = 0;
  uint64_t key[4];
  load_keys4(scores, e0 + 4u * (uint32_t)t, e1, wide, key);
  __syncthreads();
  {
    // ascending rank of every sample key: eight threads share a key, each compares it with an eighth of
    // the others (256 samples made it 0.7 us more per workgroup, on whole 64-bit keys 3 us)
    constexpr int kShare = kSample * kSample / kGridThreads;
    const uint4 *others = reinterpret_cast<const uint4 *>(&sample[(t / kSample) * kShare]);
    const uint32_t me = sample[t & (kSample - 1)];
    uint32_t rank = 0;
#pragma unroll
    for (int o = 0; o < kShare / 4; ++o) {
      const uint4 k = others[o];
      rank += (k.x < me ? 1u : 0u) + (k.y < me ? 1u : 0u) + (k.z < me ? 1u : 0u) + (k.w < me ? 1u : 0u);
    }
    atomicAdd(&ranks[t & (kSample - 1)], rank);
  }
  __syncthreads();
  if (t < kSample) sorted[ranks[t]] = sample[t];
  __syncthreads();
  // lo and hi: the two order statistics around the threshold's expected position (rank_lo, rank_hi).  Where the
  // keys lie in two heaps -- all-zero blocks beside others, hot channels -- and the bracket spans both, equal-width
  // buckets would all stand in the gap between them and each heap share one (score + select of 301056 blocks, a
  // third of them zero: 220 us, 42 with both sides' buckets).  So where a gap of the sample takes more than half of
  // the bracket, the buckets are dealt out on its two sides; they are no wider then than without the gap.
  Buckets bk;
  {
    const uint32_t lane = (uint32_t)t & 63u;
    const uint32_t v0 = sorted[lane], v1 = sorted[lane + 64];
    static_assert(kSample == 128, "two keys of the sample per lane");
    auto nth = [&](uint32_t r) { return lane_value(r < 64u ? v0 : v1, (int)(r & 63u)); };
    const uint32_t low = nth(it.rank_lo), high = nth(it.rank_hi);
    bk.lo = (uint64_t)(low & ~kPosBits) << 32;
    bk.hi = ((uint64_t)(high | kPosBits) << 32) | 0xFFFFFFFFull;
    bk.mid = 0;
    bk.shift_mid = 0;
    // (such a gap holds the middle of the bracket)
    const uint32_t middle = low + (high - low) / 2;
    const uint32_t upto = (uint32_t)(__popcll(__ballot(v0 <= middle)) + __popcll(__ballot(v1 <= middle)));
    const uint32_t below = nth(upto - 1u), above = nth(upto < (uint32_t)kSample ? upto : upto - 1u);
    const uint32_t gap = above / kSample - below / kSample;
    if (__builtin_expect((gap >= 2) & (2 * gap > high / kSample - low / kSample), 0)) {
      bk.mid = (uint64_t)(above & ~kPosBits) << 32;
      bk.shift = bucket_shift((((uint64_t)(below | kPosBits) << 32) | 0xFFFFFFFFull) - bk.lo, 7, kGapBucket - 2);
      bk.shift_mid = bucket_shift(bk.hi - bk.mid, 7, kBuckets - kGapBucket - 3);
    } else {
      bk.shift = bucket_shift(bk.hi - bk.lo, 8, kBuckets - 3);
    }
  }
  if (wg == 0 && t == 0) {
    it.ctrl->done = 0;
    it.ctrl->buckets = bk;
  }
  for (uint32_t e = e0 + 4u * (uint32_t)t; e < e1; e += 4 * kGridThreads) {
    uint64_t next[4];
    load_keys4(scores, e + 4 * kGridThreads, e1, wide, next);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (e + q < e1) atomicAdd(&hist[bucket_of(key[q], bk)], 1u);
      key[q] = next[q];
    }
  }
  __syncthreads();
  if (t < kBuckets) it.counts[wg * kBuckets + t] = hist[t];
}

// Pass 2 of workgroup `wg`; the last workgroup of the selection to finish selects among the candidates.
__device__ __forceinline__ void select_classify_body(const SelectItem &it, const uint32_t wg, SelectShared &sh,
                                                     BracketShared &bs) {
  __shared__ uint32_t wg_cand, is_last;
  const int t = threadIdx.x;
  const double *__restrict__ scores = it.scores;
  uint8_t *__restrict__ mask = it.mask;
  SelectCtrl *ctrl = it.ctrl;
  const uint32_t nblocks = it.nblocks, nwgs = it.wgs;
  const bool wide_in = (uintptr_t)scores % 16 == 0, wide_out = (uintptr_t)mask % 4 == 0;
  const Buckets bk = ctrl->buckets;
  const uint32_t e0 = wg * it.per_wg;
  const uint32_t e1 = (e0 + it.per_wg) < nblocks ? (e0 + it.per_wg) : nblocks;
  uint64_t key[4];
  load_keys4(scores, e0 + 4u * (uint32_t)t, e1, wide_in, key);

  // the bucket that holds the n_keep-th largest key (same answer in every workgroup): four threads
  // share a bucket, each adds up a quarter of the workgroups' counts
  uint32_t own = 0;
  {
    constexpr uint32_t kParts = kGridThreads / kBuckets;
    const uint32_t bkt = (uint32_t)t & (kBuckets - 1), part = (uint32_t)t / kBuckets;
#pragma unroll 8
    for (uint32_t w = part; w < nwgs; w += kParts) own += it.counts[w * kBuckets + bkt];
    if (t < kBuckets) sh.hist[t] = 0;
    if (t == 0) { wg_cand = 0; is_last = 0; }
    __syncthreads();
    atomicAdd(&sh.hist[bkt], own);
    __syncthreads();
  }
  own = t < kBuckets ? sh.hist[kBuckets - 1 - t] : 0u;       // the scan runs from the top
  const uint32_t above_me = block_exclusive_scan<kGridThreads>(own, sh.wave_tot);
  if (above_me < it.n_keep && it.n_keep <= above_me + own) {
    sh.digit = (uint32_t)(kBuckets - 1 - t);
    sh.above = above_me;
    sh.count = own;
  }
  __syncthreads();
  const uint32_t bucket = sh.digit, above = sh.above, n = sh.count;

  // Other buckets: mask bytes.  The threshold's bucket: the n candidates, whose mask bytes are the last
  // workgroup's to write.  As a rule they are few: every workgroup lists its own at its slice's place in
  // the list (how many they are stands in counts).  Else the list has no holes: a workgroup's part begins
  // where those in front of it have theirs.  No atomic on memory either way.
  const bool few = n <= (uint32_t)kCap;
  uint32_t list_at = e0;
  if (!few) {
    const uint32_t in_front = wave_sum((uint32_t)t < wg ? it.counts[(uint32_t)t * kBuckets + bucket] : 0u);
    if ((t & 63) == 0) sh.wave_tot[t >> 6] = in_front;
    __syncthreads();
    list_at = wave_sum((t & 63) < kGridThreads / 64 ? sh.wave_tot[t & 63] : 0u);
  }
  for (uint32_t e = e0 + 4u * (uint32_t)t; e < e1; e += 4 * kGridThreads) {
    uint64_t next[4];
    load_keys4(scores, e + 4 * kGridThreads, e1, wide_in, next);
    uint32_t own4 = 0, word = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (e + q < e1) {
        const uint32_t b = bucket_of(key[q], bk);
        if (b != bucket) {
          own4 |= 1u << q;
          word |= (b > bucket ? 1u : 0u) << (8 * q);
        } else {
          const uint32_t at = list_at + atomicAdd(&wg_cand, 1u);
          store_shared(&it.cand_key[at], key[q]);
          store_shared(&it.cand_idx[at], e + q);
        }
      }
      key[q] = next[q];
    }
    store_mask4(mask, e, wide_out, own4, word);
  }
  stores_done();                                 // this wave's part of the list is where every workgroup sees it
  __syncthreads();
  if (t == 0)
    is_last = __hip_atomic_fetch_add(&ctrl->done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == nwgs - 1 ? 1u : 0u;
  uint32_t wg_has = 0;                           // candidates of workgroup t's slice (nwgs <= kMaxGridWgs)
  if (few && (uint32_t)t < nwgs) wg_has = it.counts[(uint32_t)t * kBuckets + bucket];
  __syncthreads();
  if (is_last == 0) return;

  // the candidates all lie in the threshold bucket's key range,
  // which serves as the bracket of their exact selection
  const Candidates src{it.cand_key, it.cand_idx};
  uint64_t blo, bhi;
  if (bucket == 0) {
    blo = 0;
    bhi = bk.lo - 1;               // (bucket 0 is empty if lo == 0: never the threshold's)
  } else if (bucket == (uint32_t)kBuckets - 1) {
    blo = bk.hi + 1;
    bhi = ~0ull;
  } else {
    const bool behind = bk.mid != 0 && bucket > kGapBucket;
    const uint32_t width = behind ? bk.shift_mid : bk.shift;
    const uint64_t last = bk.mid != 0 && !behind ? bk.mid - 1 : bk.hi;
    blo = behind ? bk.mid + ((uint64_t)(bucket - kGapBucket - 1u) << width) : bk.lo + ((uint64_t)(bucket - 1u) << width);
    bhi = blo + ((1ull << width) - 1ull);
    if (bhi > last || (bk.mid != 0 && bucket == kGapBucket)) bhi = last;
  }
  if (few) {
    // the slices' candidates side by side in LDS, selected from there
    __shared__ __attribute__((aligned(16))) uint64_t skey[kCap];
    __shared__ uint32_t sidx[kCap];
    __shared__ uint32_t slice_at[kMaxGridWgs], slice_has[kMaxGridWgs];
    const uint32_t at = block_exclusive_scan<kGridThreads>(wg_has, sh.wave_tot);
    if ((uint32_t)t < nwgs) { slice_at[t] = at; slice_has[t] = wg_has; }
    __syncthreads();
    constexpr uint32_t kWaves = kGridThreads / 64, kTogether = 4;     // slices a wave reads at a time
    const uint32_t lane = (uint32_t)t & 63u;
    for (uint32_t w0 = (uint32_t)t >> 6; w0 < nwgs; w0 += kWaves * kTogether) {
      uint64_t k[kTogether];
      uint32_t x[kTogether];
#pragma unroll
      for (uint32_t u = 0; u < kTogether; ++u) {
        const uint32_t w = w0 + u * kWaves;
        const bool live = w < nwgs && lane < slice_has[w < nwgs ? w : 0u];
        const uint32_t from = (live ? w : 0u) * it.per_wg + (live ? lane : 0u);
        k[u] = src.key(from);
        x[u] = src.idx(from);
      }
#pragma unroll
      for (uint32_t u = 0; u < kTogether; ++u) {
        const uint32_t w = w0 + u * kWaves;
        if (w >= nwgs) continue;
        const uint32_t to = slice_at[w], has = slice_has[w];
        if (lane < has) { skey[to + lane] = k[u]; sidx[to + lane] = x[u]; }
        for (uint32_t c = lane + 64u; c < has; c += 64u) {
          skey[to + c] = src.key(w * it.per_wg + c);
          sidx[to + c] = src.idx(w * it.per_wg + c);
        }
      }
    }
    for (int b = t; b < (1 << kFinishBits); b += kGridThreads) sh.hist[b] = 0;
    __syncthreads();
    // (a few: ranked right away, the comparisons of a candidate with all others shared by kGridThreads / n threads; a radix pass and
    // the ranking of what it leaves are four barriers and a scan more.  Score and select, with the pass and so: [12544 x 1536] in 32x32
    // blocks 22.3 and 19.5 us, [49152 x 196] in 14x14 21.7 and 20.7, [1416 x 790] in 1x32 19.2 and 16.0; some 150 candidates, [40827 x 161] in
    // 1x64, keep 0.1, 24.5 and 26.4)
    if (n <= (uint32_t)kRankedAtOnce) {
      const uint32_t parts = (uint32_t)kGridThreads / n, chunk = (n + parts - 1) / parts;
      const uint32_t part = (uint32_t)t / n, c = (uint32_t)t - part * n;
      if (part < parts) {
        const uint64_t k = skey[c];
        const uint32_t idx = sidx[c];
        const uint32_t o0 = part * chunk, o1 = o0 + chunk < n ? o0 + chunk : n;
        uint32_t better = 0;
#pragma unroll 4
        for (uint32_t o = o0; o < o1; ++o) {
          const uint64_t ok = skey[o];
          better += (ok > k || (ok == k && sidx[o] < idx)) ? 1u : 0u;
        }
        if (better) atomicAdd(&sh.hist[c], better);
      }
      __syncthreads();
      if ((uint32_t)t < n) mask[sidx[t]] = sh.hist[t] < it.n_keep - above ? 1 : 0;
      return;
    }
    uint64_t ckey[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) ckey[i] = 4u * (uint32_t)t + i < n ? skey[4 * t + i] : 0ull;
    bracketed_select<kGridThreads, 4, kFinishBits, false>(ckey, Staged{skey, sidx}, n, it.n_keep - above, blo, bhi, nblocks,
                                                          false, mask, sh, bs);
  } else if (n <= (uint32_t)(kFinishKeys * kGridThreads)) {
    uint64_t ckey[kFinishKeys];
#pragma unroll
    for (int i = 0; i < kFinishKeys; ++i) {
      const uint32_t c = 4u * (uint32_t)(t + (i >> 2) * kGridThreads) + (uint32_t)(i & 3);
      ckey[i] = c < n ? src.key(c) : 0ull;
    }
    for (int b = t; b < kBins; b += kGridThreads) sh.hist[b] = 0;
    __syncthreads();
    bracketed_select<kGridThreads, kFinishKeys, kDigitBits, false>(ckey, src, n, it.n_keep - above, blo, bhi, nblocks,
                                                                   false, mask, sh, bs);
  } else {
    radix_select<kGridThreads>(src, n, it.n_keep - above, nblocks, mask, sh);
  }
}

// ---- the launches: blockIdx.y names the selection of the batch, its parameters come with the kernel
// arguments.  Selection is bound by launches and latency, not by work, so a batch costs about as much as
// one selection, and tensors small enough for one workgroup ride along in the launch of pass 2. ----
constexpr int kBatchMax = 40;
template <int N>
struct SelectBatch {
  SelectItem it[N];
};

template <int N>
__global__ __launch_bounds__(kGridThreads) void select_count_kernel(SelectBatch<N> b) {
  const SelectItem &it = b.it[blockIdx.y];
  if (blockIdx.x >= it.wgs) return;
  select_count_body(it, blockIdx.x);
}

template <int N>
__global__ __launch_bounds__(kGridThreads) void select_kernel(SelectBatch<N> b) {
  __shared__ SelectShared sh;
  __shared__ BracketShared bs;
  const SelectItem &it = b.it[blockIdx.y];
  if (it.wgs != 0) {
    if (blockIdx.x < it.wgs) select_classify_body(it, blockIdx.x, sh, bs);
    return;
  }
  if (blockIdx.x != 0) return;
  if (it.nblocks <= 4096) select_one_group<kGridThreads, 4, kDigitBits>(it.scores, it.nblocks, it.n_keep, it.mask, sh, bs);
  else select_one_group<kGridThreads, 12, kDigitBits>(it.scores, it.nblocks, it.n_keep, it.mask, sh, bs);
}

// at most 1024 blocks: a workgroup of 256 threads
template <int N>
__global__ __launch_bounds__(256) void select_small_kernel(SelectBatch<N> b) {
  __shared__ SelectShared sh;
  __shared__ BracketShared bs;
  const SelectItem &it = b.it[blockIdx.x];
  select_one_group<256, 4, 8>(it.scores, it.nblocks, it.n_keep, it.mask, sh, bs);
}

// Small matrices in few blocks: scored and selected by one workgroup, one launch.  Such calls are bound by what a launch costs on the
// host, about 2.5 us, and by latency on the GPU; a compute unit takes in 128 KB in about 2 us, as long as a second launch.
// The scores are those of launch_score, bit for bit (other calls rank the same matrix by those): a thread adds up one part of a block
// after the other as ScoreOrder says -- the rows a, a + groups, ... of a slice of columns -- all its loads on their way together, then a
// thread per block adds its parts in order.  LOOSE: slices of any width at any element, in vectors of 16 bytes; what a vector holds
// beyond its slice counts as zero, one that would reach beyond X ends there and is shifted.
constexpr int kFusedThreads = 1024;
constexpr int kFusedLoads = 8;               // vectors that a thread loads, at most
constexpr int kFusedParts = 9216;            // sums of parts in LDS, a block's an odd number of places from the next one's
template <typename T, int V, bool LOOSE>
__global__ __launch_bounds__(kFusedThreads) void score_select_small_kernel(
    const T *__restrict__ X, int64_t M, int64_t K, int64_t ldx, SmallScore g, double *__restrict__ scores_out,
    uint8_t *__restrict__ mask) {
  typedef Raw<T, V> W;
  static_assert(!LOOSE || sizeof(W) == 16, "whole vectors of 16 bytes");
  __shared__ SelectShared sh;
  __shared__ BracketShared bs;
  __shared__ __attribute__((aligned(16))) double score[1024];
  __shared__ double part[kFusedParts];
  const uint32_t t = threadIdx.x, pitch = g.block_parts | 1u;
  const T *const end = X + (M - 1) * ldx + K;
  // A thread keeps to one part of a block, q = (row group a, slice u), and goes from block to block, g.per_round at a time.
  const uint32_t b0 = span_div(t, g.block_parts, g.magic_block_parts), q0 = t - b0 * g.block_parts;
  const uint32_t a = span_div(q0, g.slices, g.magic_slices), u = q0 - a * g.slices;
  const uint32_t first = b0 < g.per_round ? b0 : g.nblocks;
  uint32_t i = span_div(first, g.nbc, g.magic_nbc), j = first - i * g.nbc, block = first;
  const int wide = g.bc - (int)u * g.slice < g.slice ? g.bc - (int)u * g.slice : g.slice;
  const T *from = nullptr;                   // of the part that is being loaded: first element, rows below it, columns
  int below = 0, cols = 0, row = 0, vec = 0;
  auto locate = [&]() {
    const int m = (int)(i * (uint32_t)g.br + a), col = (int)(j * (uint32_t)g.bc) + (int)u * g.slice;
    below = (int)M - m < g.br - (int)a ? (int)M - m : g.br - (int)a;
    cols = (int)K - col < wide ? (int)K - col : wide;
    if (block >= g.nblocks) below = 0;
    from = X + (int64_t)m * ldx + col;
  };
  locate();
  uint32_t out = first * pitch + q0;         // place of the part that is being added
  int added = 0;
  double acc = 0.0;
  W v[kFusedLoads];
  int n[kFusedLoads], over[kFusedLoads];       // elements of a vector that count, bytes by which it was held back
#pragma unroll
  for (int k = 0; k < kFusedLoads; ++k) {
    n[k] = over[k] = 0;
    if (k >= g.loads) continue;
    const int left = row * g.groups < below ? cols - vec * V : 0;
    if (left > 0) {
      const T *const at = from + (int64_t)(row * g.groups) * ldx + vec * V;
      n[k] = left < V ? left : V;
      if constexpr (LOOSE) {
        typedef W __attribute__((aligned(2))) Any;
        over[k] = at + V > end ? (int)(at + V - end) * (int)sizeof(T) : 0;
        v[k] = *reinterpret_cast<const Any *>(reinterpret_cast<const char *>(at) - over[k]);
      } else {
        v[k] = *reinterpret_cast<const W *>(at);
      }
    }
    if (++vec == g.vectors) {
      vec = 0;
      if (++row == g.rows) {
        row = 0;
        block += g.per_round;
        i += g.step_i;
        j += g.step_j;
        if (j >= g.nbc) { j -= g.nbc; ++i; }
        locate();
      }
    }
  }
#pragma unroll
  for (int k = 0; k < kFusedLoads; ++k) {
    if (k >= g.loads) continue;
    if (n[k] > 0) {
      if constexpr (LOOSE) {
        if (over[k] > 0) {
          uint64_t lo = ((uint64_t)v[k][1] << 32) | v[k][0], hi = ((uint64_t)v[k][3] << 32) | v[k][2];
          if (over[k] >= 8) { lo = hi >> (8 * (over[k] - 8)); hi = 0; }
          else { lo = (lo >> (8 * over[k])) | (hi << (64 - 8 * over[k])); hi >>= 8 * over[k]; }
          v[k][0] = (uint32_t)lo; v[k][1] = (uint32_t)(lo >> 32); v[k][2] = (uint32_t)hi; v[k][3] = (uint32_t)(hi >> 32);
        }
      }
#pragma unroll
      for (int q = 0; q < V; ++q) {
        const double x = !LOOSE || q < n[k] ? (double)raw_elem<T, V>(v[k], q) : 0.0;
        acc = fma(x, x, acc);
      }
    }
    if (++added == g.rows * g.vectors) {
      added = 0;
      if (out < g.nblocks * pitch) part[out] = acc;
      out += g.per_round * pitch;
      acc = 0.0;
    }
  }
  __syncthreads();
  if (t < g.nblocks) {
    const double *const mine = part + t * pitch;
    double sum = 0.0;
#pragma unroll 8
    for (uint32_t q = 0; q < g.block_parts; ++q) sum += mine[q];
    score[t] = sum;
    if (scores_out != nullptr) scores_out[t] = sum;
  }
  __syncthreads();
  select_one_group<kFusedThreads, 4, kFinishBits>(score, g.nblocks, g.n_keep, mask, sh, bs);
}

__global__ void fill_u8_kernel(uint8_t *p, int64_t n, uint8_t v) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

constexpr int64_t kSmallLimit = 12288;     // one workgroup (up to 12 keys per thread)
constexpr int64_t kRideAlong = 4096;       // smallest tensor that the grid-wide passes of a batched call take along

constexpr int64_t kBlocksPerWg = 4096;     // slice of a workgroup of the grid-wide passes: four keys per thread

struct SelectPlan {
  size_t counts_off, ctrl_off, key_off, idx_off, total;
};

SelectPlan select_plan(int64_t nblocks) {
  SelectPlan p;
  p.counts_off = 0;
  p.ctrl_off = align_up((size_t)kMaxGridWgs * kBuckets * sizeof(uint32_t), 256);
  p.key_off = p.ctrl_off + align_up(sizeof(SelectCtrl), 256);
  p.idx_off = p.key_off + align_up((size_t)nblocks * sizeof(uint64_t), 256);
  p.total = p.idx_off + align_up((size_t)nblocks * sizeof(uint32_t), 256);
  return p;
}

}  // namespace

// (tensors of more than kRideAlong blocks may join the grid-wide passes of a batched call)
size_t select_ws_bytes(int64_t nblocks) {
  return nblocks > kRideAlong ? select_plan(nblocks).total : 0;
}

namespace {

// One selection's kernel parameters; grid_wide: with the workgroups and the workspace of the two passes.
SelectItem select_item(const SelectJob &j, bool grid_wide) {
  SelectItem it{j.scores, j.mask, (uint32_t)j.nblocks, (uint32_t)j.n_keep, 0u, 0u, 0u, 0u, nullptr, nullptr, nullptr, nullptr};
  if (!grid_wide) return it;
  // the threshold's expected position in the sorted sample, and seven standard deviations around it
  const double frac = 1.0 - (double)it.n_keep / (double)it.nblocks;    // threshold's quantile from below
  const int pos = (int)(frac * kSample);
  const int delta = 3 + (int)(3.5 * std::sqrt(kSample * frac * (1.0 - frac)));
  it.rank_lo = (uint32_t)(pos - delta < 0 ? 0 : pos - delta);
  it.rank_hi = (uint32_t)(pos + delta > kSample - 1 ? kSample - 1 : pos + delta);
  const SelectPlan p = select_plan(j.nblocks);
  char *base = static_cast<char *>(j.ws);
  it.counts = reinterpret_cast<uint32_t *>(base + p.counts_off);
  it.ctrl = reinterpret_cast<SelectCtrl *>(base + p.ctrl_off);
  it.cand_key = reinterpret_cast<uint64_t *>(base + p.key_off);
  it.cand_idx = reinterpret_cast<uint32_t *>(base + p.idx_off);
  int64_t wgs = ceil_div(j.nblocks, kBlocksPerWg);
  if (wgs > kMaxGridWgs) wgs = kMaxGridWgs;
  it.per_wg = (uint32_t)(ceil_div(ceil_div(j.nblocks, wgs), 4) * 4);
  it.wgs = (uint32_t)ceil_div(j.nblocks, (int64_t)it.per_wg);
  return it;
}

// The launches of the m selections in b: pass 1 if any of them is grid-wide, then pass 2.
template <int N>
int run_select(const SelectBatch<N> &b, int m, uint32_t max_wgs, hipStream_t s) {
  if (max_wgs > 0) {
    hipLaunchKernelGGL(select_count_kernel<N>, dim3(max_wgs, m), dim3(kGridThreads), 0, s, b);
    const int rc = check_launch();
    if (rc != BSR_OK) return rc;
  }
  hipLaunchKernelGGL(select_kernel<N>, dim3(max_wgs > 0 ? max_wgs : 1u, m), dim3(kGridThreads), 0, s, b);
  return check_launch();
}

}  // namespace

int launch_select(const double *scores, int64_t nblocks, int64_t n_keep, uint8_t *keep_mask, void *ws,
                  hipStream_t s) {
  if (nblocks == 0) return BSR_OK;
  if (n_keep <= 0 || n_keep >= nblocks) {
    const int grid = (int)(ceil_div(nblocks, 256) < 1024 ? ceil_div(nblocks, 256) : 1024);
    hipLaunchKernelGGL(fill_u8_kernel, dim3(grid), dim3(256), 0, s, keep_mask, nblocks,
                       (uint8_t)(n_keep > 0 ? 1 : 0));
    return check_launch();
  }
  SelectBatch<1> b;
  b.it[0] = select_item(SelectJob{scores, nblocks, n_keep, keep_mask, ws}, nblocks > kSmallLimit);
  if (nblocks <= 1024) {
    hipLaunchKernelGGL(select_small_kernel<1>, dim3(1), dim3(256), 0, s, b);
    return check_launch();
  }
  return run_select<1>(b, 1, b.it[0].wgs, s);
}

// Which matrices: what a thread has to do for its vectors, next to what another launch takes, and how many blocks there are to rank.
// (Score and select back to back, two launches and one, in us: of 330 matrices up to 1.4 times the line none is slower so, 1.47 times as
// fast in the geometric mean -- binary32 [256 x 128] in 16x16 blocks 7.4 and 7.2 (50 by this count; of that the host's part 7.3 and 4.7),
// [32 x 64] 7.9 and 5.0, bfloat16 [256 x 128] 7.4 and 6.6; beyond, [250 x 250] bfloat16 in 16x16 (96) 7.9 and 9.5, [1000 x 32] binary32 in
// 8x8 (56) 6.9 and 7.7, [600 x 100] bfloat16 in 32x32 (144) 8.1 and 11.)
bool plan_score_select_small(const void *X, int dtype, int64_t M, int64_t K, int64_t ldx, int br, int bc, int64_t n_keep, SmallScore *g) {
  const int64_t nbr = ceil_div(M, br), nbc = ceil_div(K, bc);
  if (nbr > 1024 || nbc > 1024 || nbr * nbc > 1024) return false;
  ScoreOrder o;
  if (!score_order(X, dtype, M, K, ldx, br, bc, &o)) return false;
  const int64_t nblocks = nbr * nbc, block_parts = (int64_t)o.groups * o.slices;
  if (block_parts > kFusedThreads || nblocks * (block_parts | 1) > kFusedParts || M * K >= (int64_t(1) << 30)) return false;
  const int64_t vectors = ceil_div(o.slice < bc ? o.slice : bc, o.vec), rows = ceil_div(M < br ? M : br, o.groups);
  const int64_t per_round = kFusedThreads / block_parts;
  const int64_t loads = ceil_div(nblocks, per_round) * rows * vectors;
  if (loads > kFusedLoads || loads * (2 + o.vec + (o.loose ? 2 : 0)) * 64 + nblocks > 50 * 64) return false;
  auto magic = [](int64_t d) { return (uint32_t)(((uint64_t(1) << 32) + d - 1) / d); };
  *g = SmallScore{br, bc, o.groups, o.slice, o.vec, o.loose, (int)vectors, (int)rows, (int)loads, (uint32_t)nblocks, (uint32_t)nbc,
                  (uint32_t)block_parts, (uint32_t)o.slices, (uint32_t)per_round, (uint32_t)(per_round / nbc), (uint32_t)(per_round % nbc), (uint32_t)n_keep,
                  magic(nbc), magic(block_parts), magic(o.slices)};
  return true;
}

int launch_score_select_small(const SmallScore &g, const void *X, int dtype, int64_t M, int64_t K, int64_t ldx, double *scores,
                              uint8_t *keep_mask, hipStream_t s) {
#define BSR_SMALL(T, V, LOOSE)                                                                                                   \
  hipLaunchKernelGGL((score_select_small_kernel<T, V, LOOSE>), dim3(1), dim3(kFusedThreads), 0, s, static_cast<const T *>(X), M, \
                     K, ldx, g, scores, keep_mask)
  if (dtype == BSR_F32) {
    if (g.loose) BSR_SMALL(float, 4, true);
    else if (g.vec == 4) BSR_SMALL(float, 4, false);
    else if (g.vec == 2) BSR_SMALL(float, 2, false);
    else BSR_SMALL(float, 1, false);
  } else {
    if (g.loose) BSR_SMALL(uint16_t, 8, true);
    else if (g.vec == 8) BSR_SMALL(uint16_t, 8, false);
    else if (g.vec == 4) BSR_SMALL(uint16_t, 4, false);
    else if (g.vec == 2) BSR_SMALL(uint16_t, 2, false);
    else BSR_SMALL(uint16_t, 1, false);
  }
#undef BSR_SMALL
  return check_launch();
}

int launch_select_grouped(const double *scores, int64_t nbr, int64_t nbc, int64_t group_rows,
                          int64_t n_keep_group, int64_t n_keep_last, uint8_t *keep_mask, void *ws,
                          hipStream_t s) {
  if (nbr == 0 || nbc == 0) return BSR_OK;
  const int64_t groups = ceil_div(nbr, group_rows);
  const int64_t group_blocks = group_rows * nbc;
  const int64_t last_blocks = (nbr - (groups - 1) * group_rows) * nbc;
  if (groups == 1) return launch_select(scores, last_blocks, n_keep_last, keep_mask, ws, s);
  if (group_blocks > kSmallLimit) {
    // large groups: the grid-wide selection, one group after the other on the stream
    for (int64_t g = 0; g < groups; ++g) {
      const bool last = g == groups - 1;
      const int rc = launch_select(scores + g * group_blocks, last ? last_blocks : group_blocks,
                                   last ? n_keep_last : n_keep_group, keep_mask + g * group_blocks, ws, s);
      if (rc != BSR_OK) return rc;
    }
    return BSR_OK;
  }
  if (group_blocks <= 1024)
    hipLaunchKernelGGL((select_groups_kernel<256, 4, 8>), dim3((unsigned)groups), dim3(256), 0, s, scores,
                       (uint32_t)group_blocks, (uint32_t)n_keep_group, (uint32_t)last_blocks,
                       (uint32_t)n_keep_last, keep_mask);
  else if (group_blocks <= 8192)
    hipLaunchKernelGGL((select_groups_kernel<1024, 8, kDigitBits>), dim3((unsigned)groups), dim3(1024), 0, s,
                       scores, (uint32_t)group_blocks, (uint32_t)n_keep_group, (uint32_t)last_blocks,
                       (uint32_t)n_keep_last, keep_mask);
  else
    hipLaunchKernelGGL((select_groups_kernel<1024, 12, kDigitBits>), dim3((unsigned)groups), dim3(1024), 0, s,
                       scores, (uint32_t)group_blocks, (uint32_t)n_keep_group, (uint32_t)last_blocks,
                       (uint32_t)n_keep_last, keep_mask);
  return check_launch();
}

int launch_select_batched(const SelectJob *jobs, int n, hipStream_t s) {
  // The launches run one after the other and each is bound by latency, not work: one pass-1 launch for
  // the grid-wide tensors, and one launch for everything else.  When pass 1 runs anyway, mid-sized
  // tensors take part in it instead of having one workgroup read all their scores.
  bool grid_wide_runs = false, only_tiny = true;
  for (int i = 0; i < n; ++i) {
    const SelectJob &j = jobs[i];
    if (j.nblocks == 0 || j.n_keep <= 0 || j.n_keep >= j.nblocks) continue;
    if (j.nblocks > kSmallLimit) grid_wide_runs = true;
    if (j.nblocks > 1024) only_tiny = false;
  }
  SelectBatch<kBatchMax> b;
  int m = 0;
  uint32_t max_wgs = 0;
  auto flush = [&]() -> int {
    if (m == 0) return BSR_OK;
    int rc;
    if (only_tiny) {
      hipLaunchKernelGGL(select_small_kernel<kBatchMax>, dim3(m), dim3(256), 0, s, b);
      rc = check_launch();
    } else {
      rc = run_select<kBatchMax>(b, m, max_wgs, s);
    }
    m = 0;
    max_wgs = 0;
    return rc;
  };
  for (int i = 0; i < n; ++i) {
    const SelectJob &j = jobs[i];
    if (j.nblocks == 0) continue;
    if (j.n_keep <= 0 || j.n_keep >= j.nblocks) {            // all kept / none kept: a fill
      const int rc = launch_select(j.scores, j.nblocks, j.n_keep, j.mask, j.ws, s);
      if (rc != BSR_OK) return rc;
      continue;
    }
    b.it[m] = select_item(j, j.nblocks > kSmallLimit || (grid_wide_runs && j.nblocks > kRideAlong));
    if (b.it[m].wgs > max_wgs) max_wgs = b.it[m].wgs;
    if (++m == kBatchMax) {
      const int rc = flush();
      if (rc != BSR_OK) return rc;
    }
  }
  return flush();
}

int launch_select_grouped_batched(const GroupedSelectJob *jobs, int n, hipStream_t s) {
  // classes by blocks per group: 0 <= 1024, 1 <= 8192, 2 <= kSmallLimit (one workgroup per group, the
  // tensors of a class share launches); a tensor of one group or of larger groups goes on its own
  for (int cls = 0; cls < 3; ++cls) {
    GroupBatch b;
    int m = 0;
    uint32_t wgs = 0;
    auto flush = [&]() -> int {
      if (m == 0) return BSR_OK;
      if (cls == 0)
        hipLaunchKernelGGL((select_groups_batched_kernel<256, 4, 8>), dim3(wgs), dim3(256), 0, s, b, m);
      else if (cls == 1)
        hipLaunchKernelGGL((select_groups_batched_kernel<1024, 8, kDigitBits>), dim3(wgs), dim3(1024), 0, s, b, m);
      else
        hipLaunchKernelGGL((select_groups_batched_kernel<1024, 12, kDigitBits>), dim3(wgs), dim3(1024), 0, s, b, m);
      m = 0;
      wgs = 0;
      return check_launch();
    };
    for (int i = 0; i < n; ++i) {
      const GroupedSelectJob &j = jobs[i];
      if (j.nbr == 0 || j.nbc == 0) continue;
      const int64_t groups = ceil_div(j.nbr, j.group_rows);
      const int64_t group_blocks = j.group_rows * j.nbc;
      const int c = groups == 1 || group_blocks > kSmallLimit ? -1 : (group_blocks <= 1024 ? 0 : (group_blocks <= 8192 ? 1 : 2));
      if (c == -1) {
        if (cls == 0) {
          const int rc = launch_select_grouped(j.scores, j.nbr, j.nbc, j.group_rows, j.n_keep_group, j.n_keep_last,
                                               j.mask, j.ws, s);
          if (rc != BSR_OK) return rc;
        }
        continue;
      }
      if (c != cls) continue;
      GroupItem &it = b.it[m];
      it.scores = j.scores;
      it.mask = j.mask;
      it.group_blocks = (uint32_t)group_blocks;
      it.n_keep_group = (uint32_t)j.n_keep_group;
      it.last_blocks = (uint32_t)((j.nbr - (groups - 1) * j.group_rows) * j.nbc);
      it.n_keep_last = (uint32_t)j.n_keep_last;
      it.groups = (uint32_t)groups;
      it.wg_begin = wgs;
      wgs += (uint32_t)groups;
      if (++m == kGroupBatchMax) {
        const int rc = flush();
        if (rc != BSR_OK) return rc;
      }
    }
    const int rc = flush();
    if (rc != BSR_OK) return rc;
  }
  return BSR_OK;
}

}  // namespace bsr
