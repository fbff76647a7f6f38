// Offline phrase-table construction on the GPU: the most frequent distinct
// n-grams of a token stream (Sec. 4.2: candidate phrases selected by corpus
// frequency; n-gram extraction dominates the construction time reported in
// the evaluation).
//
// Only the selected n-grams have to come out in order, so nothing else is
// sorted: the windows are grouped by hash, counted in LDS, and the few that
// are selected are ranked.  Steps, all on the device:
//   1. every window of n valid tokens becomes a partition number (up to 12
//      bits) and a remainder word (32 bits for n <= 2, else 64) that
//      together determine the tuple (a bijection, so remainders are compared
//      instead of tuples); a histogram per tile, one exclusive scan and a
//      scatter group the remainders by partition, in no particular order;
//   2. each partition's remainders are counted in an LDS hash table by one
//      block (slices of a partition that heavy repetition made long are
//      counted by several blocks, whose partial counts a second launch adds
//      up; a slice that fills the table is regrouped by hash into parts that
//      do not);
//   3. the (skip + top)-th largest count c* from a histogram of the counts;
//   4. the n-grams with count >= c* become records that compare in rank
//      order: count descending, then tuple (when far more n-grams have
//      count c* than are needed, a radix select over their tuples first
//      cuts off most of the others);
//   5. the records are ranked by one bucket sort (splitters from a sample,
//      LDS sorts), which writes ranks [skip, skip + top) as tuples and
//      counts; of more than a million records only the few with counts above
//      511, the others, packed tighter, by a radix sort.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <mutex>
#include <type_traits>
#include <vector>

#include "../../include/tfe.h"
#include "tfe_internal.h"

namespace tfe {
namespace {

constexpr int kScanThreads = 1024;
constexpr int kScanItems = 16;
constexpr int kScanBlock = kScanThreads * kScanItems;

// ---- 1. windows -> partitions ---------------------------------------------------

constexpr int kPartThreads = 1024;
constexpr int kMinPartBits = 9;   // keeps 4-gram remainders below 2^63
constexpr int kMaxPartBits = 12;
constexpr uint32_t kMaxParts = 1u << kMaxPartBits;
constexpr uint32_t kTok = 0x3FFFFu;  // token fields are 18 bits

struct TokSrc {
  const int32_t* tok;
  int n;
  int32_t vocab;
  int pbits;  // log2 of the number of partitions
};

// Remainder word of an n-gram.
template <int NG>
using Rem = typename std::conditional<(NG <= 2), uint32_t, uint64_t>::type;

// Windows per scatter thread and tile.  32-bit remainders: 14336 windows
// (57 KB of LDS with their staged tokens, 73 KB with the 2048-bin counts: two
// tiles per CU), 7 per partition and tile on average; 64-bit ones: 8192.
template <int NG>
constexpr int part_items() { return NG <= 2 ? 14 : 8; }
template <int NG>
constexpr int part_tile() { return kPartThreads * part_items<NG>(); }

// Tokens a tile of windows [w0, w0 + TILE) needs: [w0, w0 + TILE + 3),
// clipped to the stream (n windows of `ts.n` tokens: n + ts.n - 1 tokens),
// staged in LDS with coalesced loads (16 bytes per lane when the stream is
// 16-byte aligned) so that each window's tokens are read from LDS instead of
// with one global load per token and window.  Past the stream: -1.
template <int TILE, int NT>
__device__ __forceinline__ void stage_tokens(const TokSrc& ts, uint64_t n, uint64_t w0,
                                             int32_t* s_tok) {
  constexpr int CNT = TILE + 3;
  const uint64_t ntok = n + (uint64_t)ts.n - 1;
  const uint64_t avail = ntok > w0 ? ntok - w0 : 0;
  const int32_t* src = ts.tok + w0;
  if ((((uintptr_t)src) & 15u) == 0) {
    typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
    for (int v = threadIdx.x; v < (CNT + 3) / 4; v += NT) {
      const uint64_t e = 4ull * (uint64_t)v;
      if (e + 4 <= avail) {
        const i32x4 x = *(const i32x4*)(src + e);
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (e + q < (uint64_t)CNT) s_tok[e + q] = x[q];
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (e + q < (uint64_t)CNT) s_tok[e + q] = e + q < avail ? src[e + q] : -1;
      }
    }
  } else {
    for (int e = threadIdx.x; e < CNT; e += NT) s_tok[e] = (uint64_t)e < avail ? src[e] : -1;
  }
}

// Tile of this block.  Workgroups are dispatched round-robin over the
// 8 XCDs (each with its own L2); giving every XCD a contiguous range of
// tiles keeps the 32 tiles that share a 128-byte line of the digit-major
// histogram matrix on one XCD, so each line is written and read through
// one L2 instead of eight.  A bijection of [0, G) for any G.
__device__ __forceinline__ uint32_t xcd_tile(uint32_t b, uint32_t G) {
  const uint32_t q = G >> 3, r = G & 7u, x = b & 7u;
  return x * q + min(x, r) + (b >> 3);
}


// Hash of the tokens after the oldest one (18 bits).  24-bit multiplies run
// at full rate.
__device__ __forceinline__ uint32_t tail_hash(uint32_t t1, uint32_t t2, uint32_t t3) {
  uint32_t h = __umul24(t1, 0xC2B2ADu) + __umul24(t2, 0x9E3779u) + __umul24(t3, 0x85EBCBu);
  h ^= h >> 16;
  h = __umul24(h & 0xFFFFFFu, 0xD35A2Du);
  return h >> 14;
}

// The oldest token is scrambled by an odd multiplier modulo 2^18, which kMixInv
// undoes, and masked with the hash of the others: m's top bits are the
// partition, its other bits and the other tokens the remainder.
constexpr uint32_t kMix = 0x2E5B5u;
constexpr uint32_t mix_inverse() {
  uint32_t x = kMix;  // Newton's iteration: x kMix = 1 modulo 8, 64, ..., 2^18
  for (int i = 0; i < 4; ++i) x *= 2u - kMix * x;
  return x & kTok;
}
constexpr uint32_t kMixInv = mix_inverse();
static_assert(((kMix * kMixInv) & kTok) == 1u, "inverse modulo 2^18");

// Partition and remainder of the window t[0 .. NG) (oldest first); false if
// a token lies outside [0, vocab).
template <int NG>
__device__ __forceinline__ bool split_window(const int32_t* t, const TokSrc& ts, uint32_t* part,
                                             Rem<NG>* rem) {
  uint32_t x[4] = {0u, 0u, 0u, 0u};
  bool ok = true;
#pragma unroll
  for (int q = 0; q < NG; ++q) {
    x[q] = (uint32_t)t[q];
    ok = ok && x[q] < (uint32_t)ts.vocab;
  }
  uint32_t m = __umul24(x[0] & kTok, kMix) & kTok;
  if (NG > 1) m ^= tail_hash(x[1] & kTok, x[2] & kTok, x[3] & kTok);
  const int low = 18 - ts.pbits;
  *part = m >> low;
  Rem<NG> r = (Rem<NG>)(m & ((1u << low) - 1u));
#pragma unroll
  for (int q = 1; q < NG; ++q) r = (r << 18) | (Rem<NG>)(x[q] & kTok);
  *rem = r;
  return ok;
}

// The tuple of a remainder.
template <int NG>
__device__ __forceinline__ void join_window(uint32_t part, Rem<NG> rem, int pbits, uint32_t* x) {
  x[0] = x[1] = x[2] = x[3] = 0u;
#pragma unroll
  for (int q = NG - 1; q >= 1; --q) {
    x[q] = (uint32_t)rem & kTok;
    rem >>= 18;
  }
  uint32_t m = (part << (18 - pbits)) | (uint32_t)rem;
  if (NG > 1) m ^= tail_hash(x[1], x[2], x[3]);
  x[0] = __umul24(m, kMixInv) & kTok;
}

// ---- device-wide exclusive scan of uint32 (totals below 2^32) ----------------

template <int NT>
__device__ uint32_t block_scan_excl(uint32_t v, uint32_t* s_wave, uint32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  if (lane == 63) s_wave[wave] = x;
  __syncthreads();
  uint32_t off = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) {
    off += w < wave ? s_wave[w] : 0u;
    tot += s_wave[w];
  }
  __syncthreads();
  *total = tot;
  return x - v + off;
}

// Pass 1: per-block sums.
__global__ __launch_bounds__(kScanThreads) void k_scan_reduce(const uint32_t* in, uint64_t n,
                                                              uint32_t* part) {
  __shared__ uint32_t s_wave[kScanThreads / 64];
  const uint64_t base = (uint64_t)blockIdx.x * kScanBlock;
  // All loads first (masked past n), then the sum: one round trip.
  uint32_t v[kScanItems];
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const uint64_t i = base + (uint64_t)k * kScanThreads + threadIdx.x;
    v[k] = i < n ? in[i] : 0u;
  }
  uint32_t s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) s += v[k];
  uint32_t tot;
  (void)block_scan_excl<kScanThreads>(s, s_wave, &tot);
  if (threadIdx.x == 0) part[blockIdx.x] = tot;
}
// Inclusive sum over the lanes up to this one: DPP shifts within each
// 16-lane row, then the totals of the rows below (read out as scalars).
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x) {
  const int lane = threadIdx.x & 63;
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, false);  // row_shr:1
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, false);  // row_shr:2
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, false);  // row_shr:4
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, false);  // row_shr:8
  const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)x, 15);
  const uint32_t r1 = (uint32_t)__builtin_amdgcn_readlane((int)x, 31);
  const uint32_t r2 = (uint32_t)__builtin_amdgcn_readlane((int)x, 47);
  const int row = lane >> 4;
  return x + (row >= 1 ? r0 : 0u) + (row >= 2 ? r1 : 0u) + (row >= 3 ? r2 : 0u);
}

// Pass 3: scan within blocks plus the block offset.  Wave w of a block scans
// its contiguous kScanItems x 64 elements in rounds of 64 (coalesced), with
// a running carry; one exchange of wave totals places the waves.  part
// holds the blocks' sums as pass 1 left them: each block adds up those of
// the blocks before it itself (at most kScanItems per thread, from L2),
// which saves a one-block scan launch.
__global__ __launch_bounds__(kScanThreads) void k_scan_down(const uint32_t* in, uint64_t n,
                                                            const uint32_t* part, uint32_t* out) {
  __shared__ uint32_t s_tot[kScanThreads / 64];
  __shared__ uint32_t s_red[kScanThreads / 64];
  uint32_t off = 0;
  {
    uint32_t b = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      const uint32_t j = (uint32_t)k * kScanThreads + threadIdx.x;
      b += j < blockIdx.x ? part[j] : 0u;
    }
    (void)block_scan_excl<kScanThreads>(b, s_red, &off);
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t base = (uint64_t)blockIdx.x * kScanBlock + (uint64_t)wave * (64 * kScanItems);
  uint32_t v[kScanItems];
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const uint64_t i = base + (uint64_t)k * 64 + lane;
    v[k] = i < n ? in[i] : 0u;
  }
  uint32_t carry = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const uint32_t inc = wave_incl_scan(v[k]);
    const uint32_t ex = carry + inc - v[k];
    carry += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
    v[k] = ex;
  }
  if (lane == 0) s_tot[wave] = carry;
  __syncthreads();
  for (int w = 0; w < wave; ++w) off += s_tot[w];
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const uint64_t i = base + (uint64_t)k * 64 + lane;
    if (i < n) out[i] = off + v[k];
  }
}

// Windows of one tile per partition.
template <int NG, uint32_t PMAX>
__global__ __launch_bounds__(kPartThreads) void k_part_hist(TokSrc ts, uint64_t nwin,
                                                            uint32_t* hist, uint32_t ntiles) {
  constexpr int IT = part_items<NG>(), TILE = part_tile<NG>();
  __shared__ uint32_t cnt[PMAX];
  __shared__ int32_t s_tok[TILE + 4];
  const uint32_t P = 1u << ts.pbits;
  const uint32_t tile = xcd_tile(blockIdx.x, gridDim.x);
  const uint64_t base = (uint64_t)tile * TILE;
  for (uint32_t e = threadIdx.x; e < P; e += kPartThreads) cnt[e] = 0u;
  stage_tokens<TILE, kPartThreads>(ts, nwin, base, s_tok);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < IT; ++r) {
    const uint32_t j = (uint32_t)r * kPartThreads + threadIdx.x;
    uint32_t part;
    Rem<NG> rem;
    const bool ok = split_window<NG>(s_tok + j, ts, &part, &rem);
    if (ok && base + j < nwin) atomicAdd(&cnt[part], 1u);
  }
  __syncthreads();
  for (uint32_t e = threadIdx.x; e < P; e += kPartThreads) hist[(size_t)e * ntiles + tile] = cnt[e];
}

// Scatter of one tile.  The order inside a partition is free, so a window's
// place among the tile's windows of its partition is what its LDS atomic
// returns; the remainders are regrouped in LDS and each partition's run is
// written by a few consecutive lanes (then by whole waves, for the runs
// that heavy repetition made long).
template <int NG, uint32_t PMAX>
__global__ __launch_bounds__(kPartThreads) void k_part_scatter(TokSrc ts, uint64_t nwin,
                                                               const uint32_t* offs,
                                                               uint32_t ntiles, Rem<NG>* out) {
  using K = Rem<NG>;
  constexpr int IT = part_items<NG>(), TILE = part_tile<NG>();
  constexpr int PER = PMAX / kPartThreads;
  constexpr int LG = NG <= 2 ? 8 : 4;  // lanes per run
  __shared__ K buf[TILE + (sizeof(K) == 4 ? 4 : 0)];  // the staged tokens, then the remainders
  __shared__ uint32_t loc[PMAX + 1], dlt[PMAX];
  __shared__ uint32_t s_wave[kPartThreads / 64];
  static_assert((TILE + 3) * 4 <= (int)sizeof(buf), "token staging fits");
  const uint32_t P = 1u << ts.pbits;
  const uint32_t tile = xcd_tile(blockIdx.x, gridDim.x);
  const uint64_t base = (uint64_t)tile * TILE;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint32_t glob[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const uint32_t p = (uint32_t)tid * PER + k;
    glob[k] = p < P ? offs[(size_t)p * ntiles + tile] : 0u;
    loc[p] = 0u;
  }
  int32_t* s_tok = (int32_t*)buf;
  stage_tokens<TILE, kPartThreads>(ts, nwin, base, s_tok);
  __syncthreads();
  K rem[IT];
  uint32_t at[IT];  // partition << 16 | place in the tile's run; ~0: no window
#pragma unroll
  for (int r = 0; r < IT; ++r) {
    const uint32_t j = (uint32_t)r * kPartThreads + tid;
    uint32_t part;
    const bool ok = split_window<NG>(s_tok + j, ts, &part, &rem[r]);
    at[r] = ok && base + j < nwin ? (part << 16) | atomicAdd(&loc[part], 1u) : 0xFFFFFFFFu;
  }
  __syncthreads();
  uint32_t c[PER], sum = 0;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    c[k] = loc[tid * PER + k];
    sum += c[k];
  }
  uint32_t total;
  uint32_t run = block_scan_excl<kPartThreads>(sum, s_wave, &total);
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    loc[tid * PER + k] = run;
    dlt[tid * PER + k] = glob[k] - run;
    run += c[k];
  }
  if (tid == 0) loc[PMAX] = total;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < IT; ++r)
    if (at[r] != 0xFFFFFFFFu) buf[loc[at[r] >> 16] + (at[r] & 0xFFFFu)] = rem[r];
  __syncthreads();
  constexpr uint32_t GR = 64 / LG;      // runs per wave and round
  constexpr uint32_t LONG = 16 * LG;    // a run's part beyond this is left to the whole wave
  for (uint32_t b0 = wave * GR; b0 < P; b0 += (kPartThreads / 64) * GR) {
    const uint32_t bin = b0 + lane / LG;  // P is a multiple of GR
    const uint32_t s = loc[bin], e = loc[bin + 1], d = dlt[bin];
    const uint32_t e1 = min(e, s + LONG);
    for (uint32_t q = s + lane % LG; q < e1; q += LG) out[(uint32_t)(q + d)] = buf[q];
    uint64_t more = __builtin_amdgcn_ballot_w64(e > e1 && lane % LG == 0);
    while (more) {
      const int l = __builtin_ctzll(more);
      more &= more - 1;
      const uint32_t ls = (uint32_t)__builtin_amdgcn_readlane((int)e1, l);
      const uint32_t le = (uint32_t)__builtin_amdgcn_readlane((int)e, l);
      const uint32_t ld = (uint32_t)__builtin_amdgcn_readlane((int)d, l);
      for (uint32_t q = ls + lane; q < le; q += 64) out[(uint32_t)(q + ld)] = buf[q];
    }
  }
}

// ---- 2. counting -------------------------------------------------------------------

// Where everything lies, in one small device buffer (plan_words words).
constexpr int kSelBins = 4096;
constexpr uint32_t kMaxBuckets = 1024;
struct Plan {
  uint32_t* start;   // [P + 1]: partition p holds remainders [start[p], start[p + 1])
  uint32_t* first;   // [P + 1]: its slices are [first[p], first[p + 1])
  uint32_t* part;    // [slices]: partition of a slice
  uint32_t* nslice;  // [slices]: distinct n-grams a slice's block found
  uint32_t* nuniq;   // [P]: distinct n-grams of a partition
  uint32_t* bins;    // [kSelBins]: n-grams with count min(i, kSelBins - 1)
  uint32_t* tie;     // [512]: digit histogram of the tie selection
  uint32_t* bcnt;    // [kMaxBuckets]: records per bucket
  uint32_t* bcur;    // [kMaxBuckets]: records placed so far
  uint32_t* bstart;  // [kMaxBuckets + 1]
  uint64_t* state;   // [16], below
};
enum {
  kStCstar, kStR, kStNeed, kStAbove, kStEqual, kStU,  // k_sel_small
  kStPlaced, kStPlacedLow,                            // records gathered so far
  kStHigh,                                            // n-grams with count above kLowMax
  kStTieHi, kStTieLo, kStTieNeed,                     // tie selection: key prefix, rank in it
  kStTieDone,                                         // 0, or how many records it leaves
  kStFault,
  kStWords = 16
};
size_t plan_words(uint32_t P, uint32_t slices) {
  return 2 * ((size_t)P + 1) + 2 * (size_t)slices + P + kSelBins + 512 + 3 * (size_t)kMaxBuckets +
         1 + 2 * kStWords + 2;
}
Plan plan_at(uint32_t* w, uint32_t P, uint32_t slices) {
  Plan a;
  a.state = (uint64_t*)w;
  w += 2 * kStWords;
  a.start = w;
  a.first = a.start + P + 1;
  a.part = a.first + P + 1;
  a.nslice = a.part + slices;
  a.nuniq = a.nslice + slices;
  a.bins = a.nuniq + P;
  a.tie = a.bins + kSelBins;
  a.bcnt = a.tie + 512;
  a.bcur = a.bcnt + kMaxBuckets;
  a.bstart = a.bcur + kMaxBuckets;
  return a;
}

// Partition starts from the scanned histogram (offs[P ntiles] is the number
// of windows), slices of at most S remainders, and cleared counters.  One
// block.
__global__ __launch_bounds__(1024) void k_plan(Plan a, const uint32_t* offs, uint32_t ntiles,
                                               uint32_t P, uint32_t S) {
  __shared__ uint32_t s_wave[16];
  const uint32_t tid = threadIdx.x;
  for (uint32_t e = tid; e < kSelBins; e += 1024) a.bins[e] = 0u;
  for (uint32_t e = tid; e < 512; e += 1024) a.tie[e] = 0u;
  for (uint32_t e = tid; e < kMaxBuckets; e += 1024) a.bcnt[e] = a.bcur[e] = 0u;
  if (tid < kStWords) a.state[tid] = 0ull;
  constexpr int PER = kMaxParts / 1024;
  uint32_t beg[PER], ns[PER], sum = 0;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const uint32_t p = tid * PER + k;
    beg[k] = p < P ? offs[(size_t)p * ntiles] : 0u;
    const uint32_t end = p < P ? offs[(size_t)(p + 1) * ntiles] : 0u;
    ns[k] = (uint32_t)(((uint64_t)(end - beg[k]) + S - 1) / S);
    sum += ns[k];
  }
  uint32_t total;
  uint32_t run = block_scan_excl<1024>(sum, s_wave, &total);
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const uint32_t p = tid * PER + k;
    if (p >= P) break;
    a.start[p] = beg[k];
    a.first[p] = run;
    for (uint32_t j = 0; j < ns[k]; ++j) a.part[run + j] = p;
    run += ns[k];
  }
  if (tid == 0) {
    a.start[P] = offs[(size_t)P * ntiles];
    a.first[P] = total;
  }
}

// Hash of a remainder: its top bits pick the bucket, bits 6 to 17 the step, its
// low 16 bits the part that a remainder of too full a table falls into.
__device__ __forceinline__ uint32_t rem_hash(uint32_t r) {
  uint32_t h = r * 0x9E3779B1u;
  h ^= h >> 15;
  h *= 0x85EBCA77u;
  return h ^ (h >> 13);
}
__device__ __forceinline__ uint32_t rem_hash(uint64_t r) {
  uint32_t h = (uint32_t)r * 0x9E3779B1u;
  h ^= ((uint32_t)(r >> 32) * 0x85EBCA77u);
  h ^= h >> 15;
  h *= 0xC2B2AE3Du;
  return h ^ (h >> 13);
}

__device__ __forceinline__ uint32_t lane_of(uint32_t x, int l) {
  return (uint32_t)__builtin_amdgcn_readlane((int)x, l);
}
__device__ __forceinline__ uint64_t lane_of(uint64_t x, int l) {
  return ((uint64_t)lane_of((uint32_t)(x >> 32), l) << 32) | lane_of((uint32_t)x, l);
}

// LDS table: 16384 entries of 32-bit remainders (128 KB) or 8192 of 64-bit
// ones (96 KB), in buckets of four that are read whole: at the loads of real
// streams (up to 3/4) the slowest lane of a wave needs some 20 single entries
// but 5 buckets.
template <class K>
constexpr uint32_t agg_slots() { return sizeof(K) == 4 ? 16384u : 8192u; }
template <class K>
struct Agg {
  alignas(16) K key[agg_slots<K>()];
  uint32_t cnt[agg_slots<K>()];
  uint32_t over;  // 0, or how much had been fed when the table was given up as full
  uint32_t out;
};
// Looks; a remainder that needs more gives the table up as full, at about 17
// of 20 entries taken (with steps of one bucket instead of the remainder's own,
// at 14).  Every look beyond costs the wave: filling tables on to 19 of 20, with
// 24 looks, took the 3-grams of 2^26 Zipf tokens from 2.96 to 3.24 ms a call;
// asking at every look whether another wave has given up, the 2-grams from 1.04
// to 1.06.
constexpr uint32_t kMaxLooks = 14;

// A word of LDS that other waves write meanwhile.
__device__ __forceinline__ uint32_t read_word(const uint32_t* p) {
  return *(const volatile __attribute__((address_space(3))) uint32_t*)p;
}
// The four keys of a bucket.  Each is read as it was at some moment; a key
// never changes once it is set.
__device__ __forceinline__ void read_bucket(const uint32_t* p, uint32_t* k) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  typedef const volatile __attribute__((address_space(3))) u32x4 lds_u32x4;
  const u32x4 v = *(lds_u32x4*)p;
#pragma unroll
  for (int q = 0; q < 4; ++q) k[q] = v[q];
}
__device__ __forceinline__ void read_bucket(const uint64_t* p, uint64_t* k) {
  typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
  typedef const volatile __attribute__((address_space(3))) u64x2 lds_u64x2;
  const u64x2 a = *(lds_u64x2*)p, b = *(lds_u64x2*)(p + 2);
  k[0] = a[0];
  k[1] = a[1];
  k[2] = b[0];
  k[3] = b[1];
}

// The remainders that a (re)try takes: those whose selection string (the 16
// low hash bits, then the remainder's own bits from the lowest) starts with
// the `len` bits (vh, vr).  Different remainders have different strings, so
// splitting ends.
struct Part2 {
  int len;
  uint32_t vh;
  uint64_t vr;
};
template <class K>
__device__ __forceinline__ bool taken(const Part2& s, uint32_t h, K r) {
  if (s.len == 0) return true;
  const int lh = min(s.len, 16), lr = s.len - lh;
  return (h & ((1u << lh) - 1u)) == s.vh &&
         (lr == 0 || ((uint64_t)r & ((1ull << lr) - 1ull)) == s.vr);
}
__device__ __forceinline__ void set_bit(Part2& s, int i, bool v) {
  if (i < 16) s.vh = (s.vh & ~(1u << i)) | (v ? 1u << i : 0u);
  else s.vr = (s.vr & ~(1ull << (i - 16))) | (v ? 1ull << (i - 16) : 0ull);
}
__device__ __forceinline__ bool get_bit(const Part2& s, int i) {
  return i < 16 ? (s.vh >> i) & 1u : (s.vr >> (i - 16)) & 1ull;
}

// One look at bucket s of the table for remainder r: true once w is added to
// its count; otherwise s is where to look next (an odd number of buckets on,
// which every remainder has of its own).  A bucket's entries are taken
// from its first one on, so a remainder is in the first bucket from its own
// that had room for it, and in one entry: a lane that loses an entry to
// another remainder reads the bucket again (at most four times: each time an
// entry more is taken).
template <class K>
__device__ __forceinline__ bool agg_step(Agg<K>& L, uint32_t mask, K r, uint32_t w, uint32_t step,
                                         uint32_t& s) {
  const K none = (K)~(K)0;
  K k[4];
  read_bucket(&L.key[s], k);
  int at = -1, room = -1;
#pragma unroll
  for (int q = 3; q >= 0; --q) {
    at = k[q] == r ? q : at;
    room = k[q] == none ? q : room;
  }
  if (at < 0 && room >= 0) {
    K old = none;
    if (__hip_atomic_compare_exchange_strong(&L.key[s + (uint32_t)room], &old, r, __ATOMIC_RELAXED,
                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) ||
        old == r)
      at = room;
  }
  if (at >= 0) atomicAdd(&L.cnt[s + (uint32_t)at], w);
  else if (room < 0) s = (s + step) & mask;
  return at >= 0;
}
// Hash bits for the step: neither those of the home bucket nor the lowest,
// which parts of a partition have in common.
__device__ __forceinline__ uint32_t step_bits(uint32_t h) { return (h >> 6) & 0xFFFu; }

// Adds w to the count of r, in the lanes with act.  fed (> 0): how much the
// feed has been through.
template <class K>
__device__ __forceinline__ void agg_add(Agg<K>& L, const Part2& sel, uint32_t mask, int hshift,
                                        K r, uint32_t w, bool act, uint32_t fed) {
  const uint32_t h = rem_hash(r);
  if (!act || !taken(sel, h, r)) return;
  const uint32_t step = (step_bits(h) | 1u) << 2;
  uint32_t s = (h >> hshift) & mask & ~3u, n = 0;
  while (!agg_step(L, mask, r, w, step, s))
    if (++n == kMaxLooks) {
      L.over = fed;
      return;
    }
}

// Counts r[u] once in the lanes with act bit u, U remainders per lane.  The
// lanes of a wave that hold the first one's remainder add up first (heavily
// repeated n-grams).  Each lane works through its own remainders, a look per
// turn: waiting for the slowest lane at every remainder took 5 looks a
// remainder, this way about 2.  Counting the 2-grams of 2^26 Zipf tokens took
// 425 us with single entries, 386 with buckets and takes 332 with turns; the
// 4-grams of 20M (4900 windows a partition, where starting a block weighs
// more) 267, 234 and 230, 209 with steps of the remainder's own.
template <class K, int U>
__device__ __forceinline__ void agg_count_each(Agg<K>& L, const Part2& sel, uint32_t mask,
                                               int hshift, K (&r)[U], uint32_t act, uint32_t fed) {
  const int lane = threadIdx.x & 63;
  uint32_t q[U];  // home bucket << 20 | step bits << 8 | weight
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t h = rem_hash(r[u]);
    const bool in = ((act >> u) & 1u) && taken(sel, h, r[u]);
    uint32_t w = in ? 1u : 0u;
    const uint64_t am = __builtin_amdgcn_ballot_w64(in);
    if (am) {
      const int f = __builtin_ctzll(am);
      const uint64_t same = __builtin_amdgcn_ballot_w64(in && r[u] == lane_of(r[u], f));
      if ((same >> lane) & 1ull) w = lane == f ? (uint32_t)__builtin_popcountll(same) : 0u;
    }
    q[u] = (((h >> hshift) & mask) >> 2 << 20) | (step_bits(h) << 8) | w;
  }
  uint32_t s = q[0] >> 20 << 2, n = 0;
  for (int left = U; left > 0;) {
    const uint32_t w = q[0] & 255u;
    bool next = w == 0;
    if (!next) {
      next = agg_step(L, mask, r[0], w, ((q[0] >> 6) & 0x3FFCu) | 4u, s);
      if (!next && ++n == kMaxLooks) {
        L.over = fed;
        next = true;
      }
    }
    if (next) {
      --left;
      n = 0;
#pragma unroll
      for (int u = 0; u + 1 < U; ++u) {
        r[u] = r[u + 1];
        q[u] = q[u + 1];
      }
      s = q[0] >> 20 << 2;
    }
  }
}

// Entries that the table uses for at most len remainders.
struct TableSize {
  uint32_t slots;
  int hshift;
};
template <class K>
__device__ __forceinline__ TableSize agg_table(uint32_t len) {
  TableSize t{agg_slots<K>(), sizeof(K) == 4 ? 18 : 19};
  static_assert(agg_slots<uint32_t>() == 1u << 14 && agg_slots<uint64_t>() == 1u << 13, "shift");
  while (t.slots > 64 && t.slots / 2 >= 2 * (uint64_t)len) {
    t.slots /= 2;
    ++t.hshift;
  }
  return t;
}

// Counts, in a cleared table (or on in one, with `on`), the remainders that sel
// takes among those that feed(count, full) has count(f) add (f is called by
// whole waves with the table's parameters; full() is true once the table has
// overflowed).  Returns 0, or how much had been fed when the table was given up
// (block-uniform).
template <class K, class Feed>
__device__ __forceinline__ uint32_t agg_walk(Agg<K>& L, const Part2& sel, const TableSize& t,
                                             Feed feed, bool on = false) {
  if (!on) {
    for (uint32_t e = threadIdx.x; e < t.slots; e += 1024) {
      L.key[e] = (K)~(K)0;
      L.cnt[e] = 0u;
    }
    if (threadIdx.x == 0) L.over = 0u;
    __syncthreads();
  }
  feed([&](auto f) { f(sel, t.slots - 1, t.hshift); },
       [&] { return read_word(&L.over) != 0u; });
  __syncthreads();
  const uint32_t over = L.over;
  __syncthreads();  // over is read before it is cleared
  return over;
}

// Appends the table's remainders and counts to okey / ocnt (L.out so far).
template <class K>
__device__ __forceinline__ void agg_emit(Agg<K>& L, const TableSize& t, K* okey, uint32_t* ocnt) {
  const int lane = threadIdx.x & 63;
  const uint64_t lt = (1ull << lane) - 1ull;
  for (uint32_t e = threadIdx.x; e < t.slots; e += 1024) {
    const uint32_t c = L.cnt[e];
    const uint64_t m = __builtin_amdgcn_ballot_w64(c != 0u);
    uint32_t o = 0;
    if (m && lane == 0) o = atomicAdd(&L.out, (uint32_t)__builtin_popcountll(m));
    o = __builtin_amdgcn_readfirstlane(o) + (uint32_t)__builtin_popcountll(m & lt);
    if (c != 0u) {
      okey[o] = L.key[e];
      ocnt[o] = c;
    }
  }
  __syncthreads();
}

// Bits to select parts by after a table was given up at `over` of len fed: as
// many as keep a part at 3/4 of the entries if the rest of the feed holds as
// many distinct remainders.
constexpr int kMaxSplit = 6;
__device__ __forceinline__ int split_bits(uint32_t len, uint32_t over) {
  int b = 1;
  while (b < kMaxSplit && 7 * (uint64_t)len > (6 * (uint64_t)over) << b) ++b;
  return b;
}

// Counts the remainders of root among those fed (at most len), in parts if
// the table fills up, each of which walks the feed.
template <class K, class Feed>
__device__ __forceinline__ void agg_count(Agg<K>& L, const Part2& root, uint32_t len, Feed feed,
                                          K* okey, uint32_t* ocnt, uint64_t* fault) {
  const TableSize t = agg_table<K>(len);
  Part2 sel = root;
  int depth = root.len;  // bits that every part is selected by; more where one still overflows
  for (;;) {
    const uint32_t over = agg_walk(L, sel, t, feed);
    if (over && sel.len < 16 + 63 - kMaxSplit) {
      const bool first = sel.vh == root.vh && sel.vr == root.vr;
      for (int b = sel.len == root.len ? split_bits(len, over) : 1; b > 0; --b)
        set_bit(sel, sel.len++, false);
      if (first) depth = sel.len;
      continue;
    }
    if (over && threadIdx.x == 0) *fault = 1ull;  // not reached: such a part holds one remainder
    agg_emit(L, t, okey, ocnt);
    while (sel.len > root.len && get_bit(sel, sel.len - 1)) set_bit(sel, --sel.len, false);
    if (sel.len == root.len) break;
    set_bit(sel, sel.len - 1, true);
    while (sel.len < depth) set_bit(sel, sel.len++, false);
  }
}

// Adds the remainders of src[0, len), U of each thread at a time.
template <class K, class Count, class Full>
__device__ __forceinline__ void feed_rems(Agg<K>& L, const K* src, uint32_t len, Count count,
                                          Full full) {
  constexpr uint32_t U = 4;
  for (uint32_t b = 0; b < len; b += 1024 * U) {
    if (full()) break;
    K r[U];
    uint32_t act = 0;
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      const uint32_t i = b + u * 1024 + threadIdx.x;
      r[u] = src[i < len ? i : 0u];
      act |= i < len ? 1u << u : 0u;
    }
    count([&](const Part2& sel, uint32_t mask, int hshift) {
      agg_count_each<K, U>(L, sel, mask, hshift, r, act, b + 1024 * U);
    });
  }
}

// Regroups src[0, len) into dst by the low `bits` bits of the hash: part q at
// [at[q], at[q + 1]).  cur: as many words of LDS.
template <class K>
__device__ void regroup(const K* src, uint32_t len, int bits, K* dst, uint32_t* at, uint32_t* cur) {
  const uint32_t tid = threadIdx.x, parts = 1u << bits;
  const uint64_t lt = (1ull << (tid & 63)) - 1ull;
  constexpr uint32_t U = 4;
  // use(remainder, part, lanes of the wave with the same part), by whole waves.
  auto walk = [&](auto use) {
    for (uint32_t b = 0; b < len; b += 1024 * U) {
      K r[U];
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const uint32_t i = b + u * 1024 + tid;
        r[u] = src[i < len ? i : 0u];
      }
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const bool in = b + u * 1024 + tid < len;
        const uint32_t q = rem_hash(r[u]) & (parts - 1u);
        uint64_t m = __builtin_amdgcn_ballot_w64(in);
        for (int k = 0; k < bits; ++k) {
          const uint64_t one = __builtin_amdgcn_ballot_w64((q >> k) & 1u);
          m &= (q >> k) & 1u ? one : ~one;
        }
        use(r[u], q, in ? m : 0ull);
      }
    }
  };
  if (tid < parts) cur[tid] = 0u;
  __syncthreads();
  walk([&](K, uint32_t q, uint64_t m) {
    if (m && (m & lt) == 0) atomicAdd(&cur[q], (uint32_t)__builtin_popcountll(m));
  });
  __syncthreads();
  if (tid == 0) {
    uint32_t run = 0;
    for (uint32_t q = 0; q < parts; ++q) {
      const uint32_t c = cur[q];
      at[q] = cur[q] = run;
      run += c;
    }
    at[parts] = run;
  }
  __syncthreads();
  walk([&](K r, uint32_t q, uint64_t m) {
    uint32_t o = 0;
    if (m && (m & lt) == 0) o = atomicAdd(&cur[q], (uint32_t)__builtin_popcountll(m));
    o = (uint32_t)__shfl((int)o, m ? __builtin_ctzll(m) : 0);
    if (m) dst[o + (uint32_t)__builtin_popcountll(m & lt)] = r;
  });
  __syncthreads();
}

// One slice of a partition.  A slice with more distinct remainders than the
// table takes is regrouped by hash (through ukey's share of it, which holds
// nothing yet) and counted part by part; the parts' n-grams gather where the
// remainders were.  The table is given up as soon as probes get long, and how
// far the walk had come says how many parts there have to be.  (Halving, with a
// walk over the slice for each part and for each level above them, took 10.1 ms
// a call for the 3-grams of 2^26 Zipf tokens, 33.6 and 58.5 for the 3- and 4-grams
// of 200M; a walk for each of the right number of parts 3.4, 11.1 and 14; this
// way 2.8, 6.9 and 7.1.)
template <class K>
__global__ __launch_bounds__(1024) void k_count_slices(Plan a, K* rem, uint32_t P, uint32_t S,
                                                       K* ukey, uint32_t* ucnt) {
  __shared__ Agg<K> L;
  __shared__ uint32_t s_at[(1 << kMaxSplit) + 1], s_cur[1 << kMaxSplit];
  if (blockIdx.x >= a.first[P]) return;
  const uint32_t p = a.part[blockIdx.x];
  const uint32_t beg = a.start[p] + (blockIdx.x - a.first[p]) * S;
  const uint32_t len = min(S, a.start[p + 1] - beg);
  rem += beg;
  ukey += beg;
  ucnt += beg;
  if (threadIdx.x == 0) L.out = 0u;
  const TableSize t = agg_table<K>(len);
  const Part2 all{0, 0u, 0ull};
  // Most 3- and 4-grams of long streams are distinct: where the first windows
  // are (3/4 of them), and say that 7/8 of the slice's fill the table, the rest of
  // the filling is left out (3-grams of 2^26 Zipf tokens 3.0 -> 2.8 ms, drawn evenly
  // 3.9 -> 3.2).
  const uint32_t first = sizeof(K) == 8 && len > t.slots / 8 * 7 ? 4096u : 0u;
  uint32_t over = 0;
  if (first) {
    if (threadIdx.x == 0) s_cur[0] = 0u;
    agg_walk(L, all, t, [&](auto count, auto full) { feed_rems(L, rem, first, count, full); });
    uint32_t n = 0;
    for (uint32_t e = threadIdx.x; e < t.slots; e += 1024)
      n += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(L.cnt[e] != 0u));
    if ((threadIdx.x & 63) == 0) atomicAdd(&s_cur[0], n);
    __syncthreads();
    const uint32_t fills = (uint32_t)((uint64_t)(t.slots / 8 * 7) * first / s_cur[0]);
    if (s_cur[0] >= first / 4 * 3 && fills <= len / 8 * 7) over = fills;
    __syncthreads();  // s_cur is read before the regrouping clears it
  }
  if (!over) {
    over = agg_walk(L, all, t, [&](auto count, auto full) {
      feed_rems(L, rem + first, len - first, count, full);
    }, first != 0);
    if (over) over += first;
  }
  if (!over) {
    agg_emit(L, t, ukey, ucnt);
  } else {
    const int bits = split_bits(len, over);
    regroup(rem, len, bits, ukey, s_at, s_cur);
    for (uint32_t q = 0; q < 1u << bits; ++q) {
      const uint32_t b = s_at[q], n = s_at[q + 1] - b;
      if (n == 0) continue;
      agg_count(L, Part2{bits, q, 0ull}, n, [&](auto count, auto full) {
        feed_rems(L, ukey + b, n, count, full);
      }, rem, ucnt, a.state + kStFault);
    }
    for (uint32_t e = threadIdx.x; e < L.out; e += 1024) ukey[e] = rem[e];
  }
  if (threadIdx.x == 0) a.nslice[blockIdx.x] = L.out;
}

// The partial counts of a partition counted in several slices, added up
// (one block per partition; the others only pass their number on).
template <class K>
__global__ __launch_bounds__(1024) void k_count_merge(Plan a, const K* ukey, const uint32_t* ucnt,
                                                      uint32_t S, K* mkey, uint32_t* mcnt) {
  __shared__ Agg<K> L;
  __shared__ uint32_t s_len;
  const uint32_t p = blockIdx.x, f = a.first[p], ns = a.first[p + 1] - f, beg = a.start[p];
  if (ns <= 1) {
    if (threadIdx.x == 0) a.nuniq[p] = ns ? a.nslice[f] : 0u;
    return;
  }
  if (threadIdx.x == 0) s_len = 0u;
  __syncthreads();
  for (uint32_t j = threadIdx.x; j < ns; j += 1024) atomicAdd(&s_len, a.nslice[f + j]);
  __syncthreads();
  const uint32_t len = s_len;
  auto feed = [&](auto count, auto full) {
    uint32_t fed = 0;
    for (uint32_t j = 0; j < ns; ++j) {
      const uint32_t n = a.nslice[f + j], s = beg + j * S;
      for (uint32_t b = 0; b < n; b += 1024) {
        if (full()) return;
        const uint32_t i = b + threadIdx.x;
        const uint32_t q = s + (i < n ? i : 0u);
        const K r = ukey[q];
        const uint32_t w = ucnt[q];
        count([&](const Part2& sel, uint32_t mask, int hshift) {
          agg_add<K>(L, sel, mask, hshift, r, w, i < n, fed + b + 1024);
        });
      }
      fed += n;
    }
  };
  if (threadIdx.x == 0) L.out = 0u;
  agg_count(L, Part2{0, 0u, 0ull}, len, feed, mkey + beg, mcnt + beg, a.state + kStFault);
  if (threadIdx.x == 0) a.nuniq[p] = L.out;
}

// The distinct n-grams: partition p's nuniq[p] keys and counts, in one of two
// pairs of arrays.
template <class K>
struct Uniq {
  Plan a;
  const K *key, *mkey;          // counted in one slice; in several
  const uint32_t *cnt, *mcnt;
  uint32_t P;
  __device__ __forceinline__ uint32_t at(uint32_t p, const K** k, const uint32_t** c) const {
    const bool one = a.first[p + 1] - a.first[p] <= 1;
    *k = (one ? key : mkey) + a.start[p];
    *c = (one ? cnt : mcnt) + a.start[p];
    return a.nuniq[p];
  }
};

// ---- 3. selection -----------------------------------------------------------

// The walks over the distinct n-grams wait for memory, not for its bandwidth:
// a thread requests kWalk counts together (0 past the last).  The histogram and
// the records of the 2-grams of 2^26 tokens took 33 and 62 us one at a time,
// 28 and 56 so; of the 4-grams of 20M 32 and 71, 25 and 62.
constexpr uint32_t kWalk = 6;
__device__ __forceinline__ void load_counts(const uint32_t* c, uint32_t n, uint32_t b,
                                            uint32_t (&v)[kWalk]) {
#pragma unroll
  for (uint32_t q = 0; q < kWalk; ++q) {
    const uint32_t i = b + q * 1024 + threadIdx.x;
    v[q] = c[min(i, n - 1)];
  }
#pragma unroll
  for (uint32_t q = 0; q < kWalk; ++q)
    if (b + q * 1024 + threadIdx.x >= n) v[q] = 0u;
}

// Histogram of min(count, kSelBins - 1).  Most counts are small, so the
// lanes holding the first lane's bin add their number with one atomic.
template <class K>
__global__ __launch_bounds__(1024) void k_sel_hist(Uniq<K> u) {
  __shared__ uint32_t h[kSelBins];
  for (uint32_t e = threadIdx.x; e < (uint32_t)kSelBins; e += 1024) h[e] = 0u;
  __syncthreads();
  const uint64_t lt = (1ull << (threadIdx.x & 63)) - 1ull;
  for (uint32_t p = blockIdx.x; p < u.P; p += gridDim.x) {
    const K* k;
    const uint32_t* c;
    const uint32_t n = u.at(p, &k, &c);
    for (uint32_t b = 0; b < n; b += 1024 * kWalk) {
      uint32_t v[kWalk];
      load_counts(c, n, b, v);
#pragma unroll
      for (uint32_t q = 0; q < kWalk; ++q) {
        const bool in = b + q * 1024 + threadIdx.x < n;
        const uint32_t bin = min(v[q], (uint32_t)kSelBins - 1u);
        const uint32_t b0 = __builtin_amdgcn_readfirstlane(bin);
        const uint64_t m = __builtin_amdgcn_ballot_w64(in && bin == b0);
        if (in && bin != b0)
          atomicAdd(&h[bin], 1u);
        else if (in && (m & lt) == 0)
          atomicAdd(&h[b0], (uint32_t)__builtin_popcountll(m));
      }
    }
  }
  __syncthreads();
  for (uint32_t e = threadIdx.x; e < (uint32_t)kSelBins; e += 1024)
    if (h[e]) atomicAdd(&u.a.bins[e], h[e]);
}

// One block: U distinct n-grams, R = min(want, U) ranks, c* = the R-th
// largest count, the number above it, how many n-grams of count c* belong to
// the R ranks and how many there are.  c* = kSelBins - 1 stands for every
// count from there on.
constexpr uint32_t kLowMax = 511;  // largest count of a packed record (below)
__global__ __launch_bounds__(1024) void k_sel_small(Plan a, uint64_t want) {
  __shared__ uint32_t s_wave[16];
  const uint32_t t = threadIdx.x;
  uint32_t v[4], sum = 0;
  for (int k = 0; k < 4; ++k) {
    v[k] = a.bins[kSelBins - 1 - (4 * t + k)];  // bins in descending count order
    sum += v[k];
  }
  uint32_t U;
  uint32_t ex = block_scan_excl<1024>(sum, s_wave, &U);
  const uint32_t R = (uint32_t)min(want, (uint64_t)U);
  if (t == 0) {
    a.state[kStU] = U;
    a.state[kStR] = R;
  }
  static_assert((kSelBins - 1 - kLowMax) % 4 == 0, "the first bin of a thread");
  if (t == (kSelBins - 1 - kLowMax) / 4) a.state[kStHigh] = ex;
  for (int k = 0; k < 4; ++k) {
    if (ex < R && R <= ex + v[k]) {
      a.state[kStCstar] = kSelBins - 1 - (4 * t + k);
      a.state[kStNeed] = R - ex;
      a.state[kStTieNeed] = R - ex;
      a.state[kStAbove] = ex;
      a.state[kStEqual] = v[k];
    }
    ex += v[k];
  }
}

// ---- 4. records ---------------------------------------------------------------

// A record compares in rank order (smaller = earlier): 2^28 - count (28
// bits) and the two oldest tokens, then the two newest.
struct Rec1 {
  uint64_t hi;
};
struct Rec2 {
  uint64_t hi, lo;
};
__device__ __forceinline__ bool before(const Rec1& x, const Rec1& y) { return x.hi < y.hi; }
__device__ __forceinline__ bool before(const Rec2& x, const Rec2& y) {
  return x.hi < y.hi || (x.hi == y.hi && x.lo < y.lo);
}
template <int NG>
using Rec = typename std::conditional<(NG <= 2), Rec1, Rec2>::type;
template <class R>
__device__ __forceinline__ R last_rec();
template <>
__device__ __forceinline__ Rec1 last_rec<Rec1>() { return Rec1{~0ull}; }
template <>
__device__ __forceinline__ Rec2 last_rec<Rec2>() { return Rec2{~0ull, ~0ull}; }

__device__ __forceinline__ uint64_t key_hi(const uint32_t* x) { return ((uint64_t)x[0] << 18) | x[1]; }
__device__ __forceinline__ uint64_t key_lo(const uint32_t* x) { return ((uint64_t)x[2] << 18) | x[3]; }
__device__ __forceinline__ void make_rec(Rec1* r, uint32_t c, const uint32_t* x) {
  r->hi = ((uint64_t)((1u << 28) - c) << 36) | key_hi(x);
}
__device__ __forceinline__ void make_rec(Rec2* r, uint32_t c, const uint32_t* x) {
  r->hi = ((uint64_t)((1u << 28) - c) << 36) | key_hi(x);
  r->lo = key_lo(x);
}

__device__ __forceinline__ void write_rank(const Rec1& r, int n, int32_t* t, int64_t* c) {
  *c = (int64_t)((1u << 28) - (uint32_t)(r.hi >> 36));
  t[0] = (int32_t)((r.hi >> 18) & kTok);
  if (n == 2) t[1] = (int32_t)(r.hi & kTok);
}
__device__ __forceinline__ void write_rank(const Rec2& r, int n, int32_t* t, int64_t* c) {
  *c = (int64_t)((1u << 28) - (uint32_t)(r.hi >> 36));
  t[0] = (int32_t)((r.hi >> 18) & kTok);
  t[1] = (int32_t)(r.hi & kTok);
  t[2] = (int32_t)((r.lo >> 18) & kTok);
  if (n == 4) t[3] = (int32_t)(r.lo & kTok);
}

// Tie selection, digit d (9 bits, from the oldest token's high bits) of the
// tuples with count c* whose earlier digits are the ones decided.  Nothing
// once the selection is done.
template <int NG>
__global__ __launch_bounds__(1024) void k_tie_hist(Uniq<Rem<NG>> u, int pbits, int d) {
  __shared__ uint32_t h[512];
  if (u.a.state[kStTieDone]) return;
  if (threadIdx.x < 512) h[threadIdx.x] = 0u;
  __syncthreads();
  const uint32_t cstar = (uint32_t)u.a.state[kStCstar];
  const uint64_t ph = u.a.state[kStTieHi], pl = u.a.state[kStTieLo];
  const int sh = 27 - 9 * (d & 3);  // of the digit in its 36-bit half
  for (uint32_t p = blockIdx.x; p < u.P; p += gridDim.x) {
    const Rem<NG>* k;
    const uint32_t* c;
    const uint32_t n = u.at(p, &k, &c);
    for (uint32_t i = threadIdx.x; i < n; i += 1024) {
      if (c[i] != cstar) continue;
      uint32_t x[4];
      join_window<NG>(p, k[i], pbits, x);
      const uint64_t hi = key_hi(x), lo = key_lo(x);
      const bool in = d < 4 ? (hi >> (sh + 9)) == (ph >> (sh + 9))
                            : hi == ph && (lo >> (sh + 9)) == (pl >> (sh + 9));
      if (in) atomicAdd(&h[((d < 4 ? hi : lo) >> sh) & 511u], 1u);
    }
  }
  __syncthreads();
  if (threadIdx.x < 512 && h[threadIdx.x]) atomicAdd(&u.a.tie[threadIdx.x], h[threadIdx.x]);
}

// One block: the digit that holds the needed tuple; clears the histogram.
// Once at most `slack` tuples share the digits decided, all of them are taken
// (the ranking sorts out which are needed): every pass reads all the counts
// and keys at c*, and the six for the 3-grams of 2^26 tokens drawn evenly took
// 1.13 ms of 4.45, where one is enough.
__global__ __launch_bounds__(512) void k_tie_pick(Plan a, int d, uint32_t slack) {
  __shared__ uint32_t s_wave[8];
  if (a.state[kStTieDone]) return;
  const uint32_t t = threadIdx.x;
  const uint64_t need = a.state[kStTieNeed];
  const uint32_t v = a.tie[t];
  uint32_t tot;
  const uint64_t ex = block_scan_excl<512>(v, s_wave, &tot);
  a.tie[t] = 0u;
  if (ex < need && need <= ex + v) {
    const int sh = 27 - 9 * (d & 3);
    const bool done = v <= slack;
    const uint64_t rest = done ? (1ull << sh) - 1ull : 0ull;
    a.state[d < 4 ? kStTieHi : kStTieLo] |= (uint64_t)t << sh | rest;
    if (done && d < 4) a.state[kStTieLo] = (1ull << 36) - 1ull;
    a.state[kStTieNeed] = need - ex;
    if (done) a.state[kStTieDone] = a.state[kStAbove] + (a.state[kStNeed] - (need - ex)) + v;
  }
}

// Goes twice through the distinct n-grams, once to count and once to place
// them: use(second, partition, remainders, index, count, kept), by whole waves.
// Kept are those with count above c* and those at c* (every one; with `tie`, up
// to the selected prefix).  between() stands between the two.
template <int NG, class Use, class Between>
__device__ __forceinline__ void gather_walk(const Uniq<Rem<NG>>& u, int pbits, uint32_t tie, Use use,
                                            Between between) {
  const uint32_t cstar = (uint32_t)u.a.state[kStCstar];
  const uint64_t th = u.a.state[kStTieHi], tl = u.a.state[kStTieLo];
  auto walk = [&](auto second) {
    for (uint32_t p = blockIdx.x; p < u.P; p += gridDim.x) {
      const Rem<NG>* k;
      const uint32_t* c;
      const uint32_t n = u.at(p, &k, &c);
      for (uint32_t b = 0; b < n; b += 1024 * kWalk) {
        uint32_t v[kWalk];
        load_counts(c, n, b, v);
#pragma unroll
        for (uint32_t q = 0; q < kWalk; ++q) {
          const uint32_t i = b + q * 1024 + threadIdx.x, ci = v[q];
          bool keep = ci >= cstar && ci != 0u;
          uint32_t x[4] = {0u, 0u, 0u, 0u};
          if (keep && tie && ci == cstar) {
            join_window<NG>(p, k[i], pbits, x);
            const uint64_t hi = key_hi(x);
            keep = hi < th || (hi == th && key_lo(x) <= tl);
          }
          use(second, p, k, i, ci, keep);
        }
      }
    }
  };
  walk(std::false_type{});
  between();
  walk(std::true_type{});
}

// The places of a wave's kept lanes behind *n (LDS).
__device__ __forceinline__ uint32_t append(uint32_t* n, bool keep) {
  const int lane = threadIdx.x & 63;
  const uint64_t m = __builtin_amdgcn_ballot_w64(keep);
  uint32_t o = 0;
  if (m && lane == 0) o = atomicAdd(n, (uint32_t)__builtin_popcountll(m));
  return __builtin_amdgcn_readfirstlane(o) + (uint32_t)__builtin_popcountll(m & ((1ull << lane) - 1ull));
}
// A block's share *n becomes its first place among all of them.
__device__ __forceinline__ void take_places(uint32_t* n, uint64_t* placed) {
  *n = (uint32_t)atomicAdd((unsigned long long*)placed, (unsigned long long)*n);
}

// Records of the kept n-grams, in no particular order.  A block counts its
// share first and takes its places with one atomic.
template <int NG>
__global__ __launch_bounds__(1024) void k_gather(Uniq<Rem<NG>> u, int pbits, uint32_t tie,
                                                 Rec<NG>* out, uint32_t cap) {
  __shared__ uint32_t s_n;
  if (threadIdx.x == 0) s_n = 0u;
  __syncthreads();
  gather_walk<NG>(
      u, pbits, tie,
      [&](auto second, uint32_t p, const Rem<NG>* k, uint32_t i, uint32_t ci, bool keep) {
        const uint32_t o = append(&s_n, keep);
        if (decltype(second)::value && keep && o < cap) {
          uint32_t x[4];
          join_window<NG>(p, k[i], pbits, x);
          make_rec(&out[o], ci, x);
        }
      },
      [&] {
        __syncthreads();
        if (threadIdx.x == 0) take_places(&s_n, u.a.state + kStPlaced);
        __syncthreads();
      });
}

// The same for long rankings: records of the n-grams with count above kLowMax,
// and the others packed: kLowMax - count (9 bits) and up to three tokens in a
// word, the fourth in one of its own.
template <int NG>
constexpr int packed_tokens() { return 18 * (NG < 3 ? NG : 3); }
template <int NG>
__global__ __launch_bounds__(1024) void k_gather_long(Uniq<Rem<NG>> u, int pbits, uint32_t tie,
                                                      Rec<NG>* high, uint32_t nhigh, uint64_t* low,
                                                      uint32_t* low3, uint32_t nlow) {
  __shared__ uint32_t s_n[2];
  if (threadIdx.x < 2) s_n[threadIdx.x] = 0u;
  __syncthreads();
  gather_walk<NG>(
      u, pbits, tie,
      [&](auto second, uint32_t p, const Rem<NG>* k, uint32_t i, uint32_t ci, bool keep) {
        const bool hi = keep && ci > kLowMax, lo = keep && ci <= kLowMax;
        const uint32_t oh = append(&s_n[0], hi), ol = append(&s_n[1], lo);
        if (!decltype(second)::value) return;
        uint32_t x[4];
        if (hi && oh < nhigh) {
          join_window<NG>(p, k[i], pbits, x);
          make_rec(&high[oh], ci, x);
        } else if (lo && ol < nlow) {
          join_window<NG>(p, k[i], pbits, x);
          uint64_t w = kLowMax - ci;
#pragma unroll
          for (int q = 0; q < (NG < 3 ? NG : 3); ++q) w = (w << 18) | x[q];
          low[ol] = w;
          if (NG == 4) low3[ol] = x[3];
        }
      },
      [&] {
        __syncthreads();
        if (threadIdx.x < 2) take_places(&s_n[threadIdx.x], u.a.state + kStPlaced + threadIdx.x);
        __syncthreads();
      });
}

// ---- 5. ranking ------------------------------------------------------------------

// Bucket sort: splitters from a sorted sample (4 records per bucket), each
// record's bucket by binary search, then one LDS sort per bucket, which
// writes the ranks asked for.  A bucket holds about kBucketMean records, at
// most kBucketCap in LDS; a larger one (eight times the mean, between five
// samples taken at even distances from records in no order: one in 10^10) is
// sorted in memory.
constexpr uint32_t kBucketMean = 1024;
constexpr uint32_t kBucketCap = 8192;
// Most records the bucket sort takes.  Beyond, the radix sort of packed records
// is faster.  All the n-grams of N evenly drawn tokens, bucket sort / radix sort,
// us a call: 2-grams 263 / 263 at N = 800000, 359 / 289 at 1.4M; 3-grams
// 333 / 314, 492 / 351; 4-grams 335 / 386, 493 / 419.
constexpr uint64_t kBucketSortMax = (uint64_t)kBucketMean * kMaxBuckets;

// Bitonic sort of a[0, m), ascending, in LDS or in memory.  Every comparison
// puts the smaller record first (the first step of a merge compares mirrored
// places), so the places from m to the next power of two, which would hold
// larger records than all others, need not exist.  (Block barriers only where a
// step leaves a wave's 128 elements changed nothing in the bucket sorts and
// took 4 of 41 us off the sample's.)
template <class R>
__device__ __forceinline__ void bitonic_sort(R* a, uint32_t m) {
  uint32_t N2 = 2;
  while (N2 < m) N2 <<= 1;
  for (uint32_t size = 2; size <= N2; size <<= 1) {
    for (uint32_t stride = size >> 1; stride > 0; stride >>= 1) {
      __syncthreads();
      for (uint32_t e = threadIdx.x; e < N2 / 2; e += 1024) {
        const uint32_t i = 2 * e - (e & (stride - 1));
        const uint32_t j = stride == size >> 1 ? i ^ (size - 1) : i + stride;
        if (j >= m) continue;
        const R x = a[i], y = a[j];
        if (before(y, x)) {
          a[i] = y;
          a[j] = x;
        }
      }
    }
  }
  __syncthreads();
}

// nb - 1 splitters (nb a power of two): every fourth of 4 nb sampled records.
template <class R>
__global__ __launch_bounds__(1024) void k_bk_sample(const R* rec, uint64_t K, uint32_t nb,
                                                    R* split) {
  __shared__ R s[4 * kMaxBuckets];
  const uint32_t ns = 4 * nb;
  for (uint32_t e = threadIdx.x; e < ns; e += 1024) s[e] = rec[(uint64_t)e * K / ns];
  bitonic_sort(s, ns);
  for (uint32_t b = 1 + threadIdx.x; b < nb; b += 1024) split[b - 1] = s[4 * b];
}

constexpr uint32_t kBkTile = 4096;

// Bucket of every record: the number of splitters at or before it.
template <class R>
__global__ __launch_bounds__(1024) void k_bk_hist(Plan a, const R* rec, uint64_t K, uint32_t nb,
                                                  const R* split, uint16_t* bkt) {
  __shared__ R s[kMaxBuckets];
  __shared__ uint32_t c[kMaxBuckets];
  for (uint32_t e = threadIdx.x; e < nb; e += 1024) {
    s[e] = e + 1 < nb ? split[e] : last_rec<R>();
    c[e] = 0u;
  }
  __syncthreads();
#pragma unroll
  for (uint32_t q = 0; q < kBkTile / 1024; ++q) {
    const uint64_t i = (uint64_t)blockIdx.x * kBkTile + q * 1024 + threadIdx.x;
    if (i < K) {
      const R x = rec[i];
      uint32_t lo = 0;
      for (uint32_t h = nb >> 1; h; h >>= 1)
        if (!before(x, s[lo + h - 1])) lo += h;
      atomicAdd(&c[lo], 1u);
      bkt[i] = (uint16_t)lo;
    }
  }
  __syncthreads();
  for (uint32_t e = threadIdx.x; e < nb; e += 1024)
    if (c[e]) atomicAdd(&a.bcnt[e], c[e]);
}

template <class R>
__global__ __launch_bounds__(1024) void k_bk_scatter(Plan a, const R* rec, uint64_t K, uint32_t nb,
                                                     const uint16_t* bkt, R* out) {
  __shared__ uint32_t c[kMaxBuckets], base[kMaxBuckets];
  __shared__ uint32_t s_wave[16];
  constexpr uint32_t PER = kMaxBuckets / 1024;
  const uint32_t tid = threadIdx.x;
  uint32_t n[PER], sum = 0;
#pragma unroll
  for (uint32_t k = 0; k < PER; ++k) {
    const uint32_t b = tid * PER + k;
    n[k] = b < nb ? a.bcnt[b] : 0u;
    sum += n[k];
    c[b] = 0u;
  }
  uint32_t tot;
  uint32_t run = block_scan_excl<1024>(sum, s_wave, &tot);
#pragma unroll
  for (uint32_t k = 0; k < PER; ++k) {
    const uint32_t b = tid * PER + k;
    base[b] = run;
    if (blockIdx.x == 0 && b <= nb) a.bstart[b] = run;
    run += n[k];
  }
  if (blockIdx.x == 0 && tid == 0) a.bstart[nb] = tot;
  __syncthreads();
  uint32_t at[kBkTile / 1024], b[kBkTile / 1024];
#pragma unroll
  for (uint32_t q = 0; q < kBkTile / 1024; ++q) {
    const uint64_t i = (uint64_t)blockIdx.x * kBkTile + q * 1024 + tid;
    b[q] = i < K ? bkt[i] : 0u;
    at[q] = i < K ? atomicAdd(&c[b[q]], 1u) : 0u;
  }
  __syncthreads();
  for (uint32_t e = tid; e < nb; e += 1024)
    if (c[e]) base[e] += atomicAdd(&a.bcur[e], c[e]);
  __syncthreads();
#pragma unroll
  for (uint32_t q = 0; q < kBkTile / 1024; ++q) {
    const uint64_t i = (uint64_t)blockIdx.x * kBkTile + q * 1024 + tid;
    if (i < K) out[base[b[q]] + at[q]] = rec[i];
  }
}

// Sorts one bucket (whole > 0: all of the records, the only one) and writes its
// ranks in [skip, ranks).
template <class R>
__global__ __launch_bounds__(1024) void k_bk_sort(Plan a, R* rec, uint32_t whole, uint64_t skip,
                                                  uint64_t ranks, int n, int32_t* tuples,
                                                  int64_t* counts) {
  __shared__ R s[kBucketCap];
  const uint32_t beg = whole ? 0u : a.bstart[blockIdx.x];
  const uint32_t m = whole ? whole : a.bstart[blockIdx.x + 1] - beg;
  if (m == 0 || beg >= ranks || (uint64_t)beg + m <= skip) return;
  rec += beg;
  const bool lds = m <= kBucketCap;
  if (lds) {
    for (uint32_t e = threadIdx.x; e < m; e += 1024) s[e] = rec[e];
    bitonic_sort(s, m);
  } else {
    bitonic_sort(rec, m);
  }
  for (uint32_t e = threadIdx.x; e < m; e += 1024) {
    const R r = lds ? s[e] : rec[e];
    const uint64_t rank = (uint64_t)beg + e;
    if (rank >= skip && rank < ranks)
      write_rank(r, n, tuples + (rank - skip) * n, counts + (rank - skip));
  }
}

// Tiles of the radix sort: 512 threads (one per digit), 8 keys per thread
// for keys alone (4096 keys: 52 KB of LDS, three tiles per CU) and 6 with a
// payload.  The histogram of a tile is counted by 1024 threads.
constexpr int kTileThreads = 512;
constexpr int kTileWaves = kTileThreads / 64;
constexpr int kHistThreads = 1024;
template <class K, bool PAIRS, class V>
constexpr int tile_items() { return (sizeof(K) + (PAIRS ? sizeof(V) : 0)) > 8 ? 6 : 8; }
template <class K, bool PAIRS, class V>
constexpr int tile_keys() { return kTileThreads * tile_items<K, PAIRS, V>(); }
constexpr int kDigitBits = 9;
constexpr uint32_t kBins = 1u << kDigitBits;
static_assert(kBins <= (uint32_t)kTileThreads, "one scatter thread per digit");

// ---- 6. long rankings: stable LSD radix sort (9-bit digits) -----------------
//
// Packed records, where more than the bucket sort takes are ranked (millions of
// ranks asked for).

template <class K>
__device__ __forceinline__ uint32_t digit_of(K k, int shift) {
  return (uint32_t)(k >> shift) & (kBins - 1u);
}

// Lanes of the wave whose digit equals this lane's (active lanes only).
__device__ __forceinline__ uint64_t match_digit(uint32_t d, bool active) {
  uint64_t m = __builtin_amdgcn_ballot_w64(active);
#pragma unroll
  for (int b = 0; b < kDigitBits; ++b) {
    const uint64_t bb = __builtin_amdgcn_ballot_w64(active && ((d >> b) & 1u));
    m &= ((d >> b) & 1u) ? bb : ~bb;
  }
  return m;
}

// Digit histogram of one tile of TILE keys (kHistThreads threads; the keys
// are loaded first).  Per round, the lanes holding the first lane's digit
// add their number with one atomic and the others add 1 each: Zipf-skewed
// digits (high bits of frequent tokens are mostly 0) would otherwise pile
// same-address LDS atomics onto one bin; measured on MI355X this beats both
// plain atomics and counting every group of equal digits once.
template <class K, int TILE>
__global__ __launch_bounds__(kHistThreads) void k_rs_hist(const K* keys, uint64_t n, int shift,
                                                          uint32_t* hist, uint32_t ntiles) {
  constexpr int ITEMS = TILE / kHistThreads;
  __shared__ uint32_t h[kBins];
  for (int e = threadIdx.x; e < (int)kBins; e += kHistThreads) h[e] = 0u;
  const uint32_t tile = xcd_tile(blockIdx.x, gridDim.x);
  const uint64_t base = (uint64_t)tile * TILE;
  K kk[ITEMS];
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const uint64_t i = base + (uint64_t)k * kHistThreads + threadIdx.x;
    kk[k] = i < n ? keys[i] : (K)0;
  }
  __syncthreads();
  const uint64_t lt = (1ull << (threadIdx.x & 63)) - 1ull;
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const bool act = base + (uint64_t)k * kHistThreads + threadIdx.x < n;
    const uint32_t d = digit_of(kk[k], shift);
    const uint32_t d0 = __builtin_amdgcn_readfirstlane(d);
    const uint64_t m = __builtin_amdgcn_ballot_w64(act && d == d0);
    if (act && d == d0) {
      if ((m & lt) == 0) atomicAdd(&h[d0], (uint32_t)__builtin_popcountll(m));
    } else if (act) {
      atomicAdd(&h[d], 1u);
    }
  }
  __syncthreads();
  for (int e = threadIdx.x; e < (int)kBins; e += kHistThreads)
    hist[(size_t)e * ntiles + tile] = h[e];
}

// Scatter of one tile.  Wave w ranks the keys [w 64 ITEMS, (w+1) 64 ITEMS)
// of the tile in ITEMS rounds of 64 consecutive keys: the rank of a key
// among the wave's earlier keys of its digit is the wave's running count
// plus the matching lanes below it; the first lane of each digit group
// advances the count.  Tile positions follow (digit, wave, rank), i.e. the
// stable order; the tile is reordered in LDS and written in digit runs.
template <class K, class V, bool PAIRS, int ITEMS>
__global__ __launch_bounds__(kTileThreads) void k_rs_scatter(const K* keys, const V* vals,
                                                             uint64_t n, int shift,
                                                             const uint32_t* offs,
                                                             uint32_t ntiles, K* keys_out,
                                                             V* vals_out) {
  constexpr int TILE = kTileThreads * ITEMS;
  __shared__ uint32_t wcnt[kTileWaves][kBins];
  __shared__ uint32_t s_loc[kBins];   // tile-local start of each digit
  __shared__ uint32_t s_glob[kBins];  // global start of each digit's run of this tile
  __shared__ uint32_t s_wave[kTileWaves];
  __shared__ K s_keys[TILE];
  __shared__ V s_vals[PAIRS ? TILE : 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int e = threadIdx.x; e < kTileWaves * (int)kBins; e += kTileThreads) (&wcnt[0][0])[e] = 0u;
  const uint32_t tile = xcd_tile(blockIdx.x, gridDim.x);
  const uint64_t base = (uint64_t)tile * TILE + (uint64_t)wave * (64 * ITEMS);
  const uint64_t lt = (1ull << lane) - 1ull;
  K kk[ITEMS];
  V vv[PAIRS ? ITEMS : 1];
  uint32_t rank[ITEMS];
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const uint64_t i = base + (uint64_t)r * 64 + lane;
    kk[r] = i < n ? keys[i] : (K)0;
    if (PAIRS) vv[PAIRS ? r : 0] = i < n ? vals[i] : (V)0;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const bool act = base + (uint64_t)r * 64 + lane < n;
    const uint32_t d = digit_of(kk[r], shift);
    const uint64_t m = match_digit(d, act);
    const uint32_t before = wcnt[wave][d];
    rank[r] = before + (uint32_t)__builtin_popcountll(m & lt);
    // The lowest matching lane advances the wave's count of this digit.
    if (act && (m & lt) == 0) wcnt[wave][d] = before + (uint32_t)__builtin_popcountll(m);
  }
  __syncthreads();
  // Per digit (one thread each): counts of earlier waves, the tile's digit
  // starts.
  const uint32_t d = threadIdx.x;
  uint32_t tot = 0;
  if (d < kBins) {
    for (int w = 0; w < kTileWaves; ++w) {
      const uint32_t c = wcnt[w][d];
      wcnt[w][d] = tot;  // becomes the offset of wave w within the digit
      tot += c;
    }
  }
  uint32_t all;
  const uint32_t loc = block_scan_excl<kTileThreads>(tot, s_wave, &all);
  if (d < kBins) {
    s_loc[d] = loc;
    s_glob[d] = offs[(size_t)d * ntiles + tile];
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const uint64_t i = base + (uint64_t)r * 64 + lane;
    if (i < n) {
      const uint32_t dd = digit_of(kk[r], shift);
      const uint32_t pos = s_loc[dd] + wcnt[wave][dd] + rank[r];
      s_keys[pos] = kk[r];
      if (PAIRS) s_vals[PAIRS ? pos : 0] = vv[PAIRS ? r : 0];
    }
  }
  __syncthreads();
  const uint64_t tile0 = (uint64_t)tile * TILE;
  const uint32_t cnt = (uint32_t)min((uint64_t)TILE, n - tile0);
  for (uint32_t p = threadIdx.x; p < cnt; p += kTileThreads) {
    const K k = s_keys[p];
    const uint32_t dd = digit_of(k, shift);
    const uint64_t dst = (uint64_t)s_glob[dd] + (p - s_loc[dd]);
    keys_out[dst] = k;
    if (PAIRS) vals_out[dst] = s_vals[PAIRS ? p : 0];
  }
}

// Sorted packed records as ranks: record i is rank at + i - skip of the outputs.
template <int NG>
__global__ __launch_bounds__(256) void k_unpack(const uint64_t* low, const uint32_t* low3,
                                                uint64_t from, uint64_t to, uint64_t at,
                                                uint64_t skip, int32_t* tuples, int64_t* counts) {
  const uint64_t i = from + (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= to) return;
  uint64_t w = low[i];
  const uint64_t rank = at + i - skip;
  int32_t* t = tuples + rank * NG;
#pragma unroll
  for (int q = (NG < 3 ? NG : 3) - 1; q >= 0; --q) {
    t[q] = (int32_t)(w & kTok);
    w >>= 18;
  }
  if (NG == 4) t[3] = (int32_t)low3[i];
  counts[rank] = (int64_t)(kLowMax - (uint32_t)w);
}

uint32_t blocks_for(uint64_t n, uint64_t per) { return (uint32_t)((n + per - 1) / per); }

// Exclusive scan of n uint32 values (in may equal out).
hipError_t scan_u32(const uint32_t* in, uint32_t* out, uint64_t n, uint32_t* part,
                    hipStream_t s) {
  const uint32_t nb = blocks_for(n, kScanBlock);
  if (nb == 0) return hipSuccess;
  if (nb > (uint32_t)kScanBlock) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_scan_reduce, dim3(nb), dim3(kScanThreads), 0, s, in, n, part);
  hipLaunchKernelGGL(k_scan_down, dim3(nb), dim3(kScanThreads), 0, s, in, n, part, out);
  return hipGetLastError();
}

// Stable LSD sort of n keys (and payloads) by their low `bits` bits.  hist
// holds kBins x ceil(n / tile) entries.
template <bool PAIRS, class K, class V>
hipError_t radix_sort(K*& keys, K*& keys_alt, V*& vals, V*& vals_alt, uint64_t n, int bits,
                      uint32_t* hist, uint32_t* part, hipStream_t s) {
  constexpr int ITEMS = tile_items<K, PAIRS, V>();
  constexpr int TILE = tile_keys<K, PAIRS, V>();
  const uint32_t ntiles = blocks_for(n, TILE);
  for (int shift = 0; shift < bits; shift += kDigitBits) {
    hipLaunchKernelGGL((k_rs_hist<K, TILE>), dim3(ntiles), dim3(kHistThreads), 0, s, keys, n, shift,
                       hist, ntiles);
    const hipError_t e = scan_u32(hist, hist, (uint64_t)kBins * ntiles, part, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_rs_scatter<K, V, PAIRS, ITEMS>), dim3(ntiles), dim3(kTileThreads), 0, s,
                       keys, vals, n, shift, hist, ntiles, keys_alt, vals_alt);
    std::swap(keys, keys_alt);
    if (PAIRS) std::swap(vals, vals_alt);
  }
  return hipGetLastError();
}

// Scratch of the construction: device buffers kept for reuse by later calls
// (a hipMalloc / hipFree pair costs about 25 / 150 us per buffer and
// synchronises the device; a construction takes a dozen buffers) until
// tfe_ngram_release.  A request takes the smallest idle buffer of the device
// that holds it without wasting more than half; on a miss the device's idle
// buffers are returned first, so the cache never holds more than the calls
// in flight plus the buffers of one call.
struct CachedBuf {
  void* p;
  size_t bytes;
  int device;
  bool used;
};
std::mutex g_cache_mu;
std::vector<CachedBuf> g_cache;

void* cache_get(int device, size_t bytes) {
  constexpr size_t kGrain = (size_t)2 << 20;
  std::lock_guard<std::mutex> lock(g_cache_mu);
  int best = -1;
  for (size_t i = 0; i < g_cache.size(); ++i) {
    const CachedBuf& c = g_cache[i];
    if (!c.used && c.device == device && c.bytes >= bytes && c.bytes <= 2 * bytes + kGrain &&
        (best < 0 || c.bytes < g_cache[(size_t)best].bytes))
      best = (int)i;
  }
  if (best >= 0) {
    g_cache[(size_t)best].used = true;
    return g_cache[(size_t)best].p;
  }
  for (size_t i = 0; i < g_cache.size();) {
    if (!g_cache[i].used && g_cache[i].device == device) {
      dev_free(g_cache[i].p);
      g_cache[i] = g_cache.back();
      g_cache.pop_back();
    } else {
      ++i;
    }
  }
  const size_t rounded = (bytes + kGrain - 1) / kGrain * kGrain;
  void* p = nullptr;
  if (dev_malloc(&p, rounded) != hipSuccess) return nullptr;
  g_cache.push_back(CachedBuf{p, rounded, device, true});
  return p;
}

void cache_put(void* p) {
  std::lock_guard<std::mutex> lock(g_cache_mu);
  for (CachedBuf& c : g_cache)
    if (c.p == p) c.used = false;
}

struct Scratch {
  hipStream_t s;
  int device = 0;
  std::vector<void*> bufs;
  explicit Scratch(hipStream_t stream) : s(stream) { (void)hipGetDevice(&device); }
  ~Scratch() {
    // Idle only once the stream is done with them (error paths return early).
    (void)hipStreamSynchronize(s);
    for (void* p : bufs) cache_put(p);
  }
  template <class T>
  T* get(uint64_t count) {
    void* p = cache_get(device, std::max<uint64_t>(count, 1) * sizeof(T));
    if (p) bufs.push_back(p);
    return (T*)p;
  }
};

#define BUILD_HIP(call, what)                                                        \
  do {                                                                               \
    hipError_t e_ = (call);                                                          \
    if (e_ != hipSuccess) return fail(TFE_ERR_HIP, "%s: %s", what, hipGetErrorString(e_)); \
  } while (0)
// Partitions for nwin windows: as many as let a partition's distinct n-grams
// fit the LDS table (6000 windows against 8192 64-bit entries; for n <= 2,
// where most windows repeat, 32768 against 16384), within what the scatter's
// LDS counters allow.  Beyond (from 24.6M windows for n > 2), and where few
// 2-grams repeat, a partition's block splits it further.
int part_bits(uint64_t nwin, int n) {
  const uint64_t mean = n <= 2 ? 32768 : 6000;
  int b = kMinPartBits;
  while (b < kMaxPartBits && (nwin >> b) > mean) ++b;
  return b;
}

template <int NG>
tfe_status ngram_top_n(const int32_t* tokens, uint64_t nwin, int32_t vocab, uint64_t skip,
                       uint64_t top, int32_t* out_tuples, int64_t* out_counts, int64_t* written,
                       hipStream_t s) {
  using K = Rem<NG>;
  using R = Rec<NG>;
  Scratch sc(s);
  const TokSrc ts{tokens, NG, vocab, part_bits(nwin, NG)};
  const uint32_t P = 1u << ts.pbits;
  const uint32_t ntiles = blocks_for(nwin, part_tile<NG>());
  const uint64_t nhist = (uint64_t)P * ntiles;
  // Slices of twice the mean partition, so that only heavily repeated
  // n-grams make a partition span several.
  const uint32_t S = (uint32_t)std::max<uint64_t>(16384, 2 * (nwin / P + 1));
  const uint32_t slices = P + (uint32_t)(nwin / S) + 1;
  uint32_t* hist = sc.get<uint32_t>(nhist + 1);
  uint32_t* part = sc.get<uint32_t>(kScanBlock);
  uint32_t* words = sc.get<uint32_t>(plan_words(P, slices));
  K* rem = sc.get<K>(nwin);
  K* ukey = sc.get<K>(nwin);
  uint32_t* ucnt = sc.get<uint32_t>(nwin);
  uint32_t* mcnt = sc.get<uint32_t>(nwin);
  if (!hist || !part || !words || !rem || !ukey || !ucnt || !mcnt)
    return fail(TFE_ERR_OOM, "n-gram scratch for %llu windows", (unsigned long long)nwin);
  const Plan a = plan_at(words, P, slices);
  // 1. Remainders grouped by partition.
  BUILD_HIP(hipMemsetAsync(hist + nhist, 0, sizeof(uint32_t), s), "memset");
  if (P <= 2048)
    hipLaunchKernelGGL((k_part_hist<NG, 2048>), dim3(ntiles), dim3(kPartThreads), 0, s, ts, nwin,
                       hist, ntiles);
  else
    hipLaunchKernelGGL((k_part_hist<NG, 4096>), dim3(ntiles), dim3(kPartThreads), 0, s, ts, nwin,
                       hist, ntiles);
  BUILD_HIP(scan_u32(hist, hist, nhist + 1, part, s), "partition scan");
  hipLaunchKernelGGL(k_plan, dim3(1), dim3(1024), 0, s, a, hist, ntiles, P, S);
  if (P <= 2048)
    hipLaunchKernelGGL((k_part_scatter<NG, 2048>), dim3(ntiles), dim3(kPartThreads), 0, s, ts, nwin,
                       hist, ntiles, rem);
  else
    hipLaunchKernelGGL((k_part_scatter<NG, 4096>), dim3(ntiles), dim3(kPartThreads), 0, s, ts, nwin,
                       hist, ntiles, rem);
  BUILD_HIP(hipGetLastError(), "partition launches");
  // 2. Counts.  (A merged partition's n-grams take the place of its
  // remainders.)
  hipLaunchKernelGGL(k_count_slices<K>, dim3(slices), dim3(1024), 0, s, a, rem, P, S, ukey, ucnt);
  hipLaunchKernelGGL(k_count_merge<K>, dim3(P), dim3(1024), 0, s, a, ukey, ucnt, S, rem, mcnt);
  // 3. Selection.
  const Uniq<K> u{a, ukey, rem, ucnt, mcnt, P};
  const uint32_t walkers = std::min<uint32_t>(P, 512);
  hipLaunchKernelGGL(k_sel_hist<K>, dim3(walkers), dim3(1024), 0, s, u);
  hipLaunchKernelGGL(k_sel_small, dim3(1), dim3(1024), 0, s, a, skip + top);
  BUILD_HIP(hipGetLastError(), "count launches");
  uint64_t st[kStWords];
  BUILD_HIP(hipMemcpyAsync(st, a.state, sizeof st, hipMemcpyDeviceToHost, s), "copy");
  BUILD_HIP(hipStreamSynchronize(s), "sync");
  if (st[kStFault]) return fail(TFE_ERR_HIP, "n-gram count table");
  const uint64_t ranks = st[kStR];
  if (ranks <= skip) return TFE_OK;
  // 4. Records.  Many more ties at c* than needed: select among them first,
  // digit by digit; few: they are ranked with the rest.
  const bool tie = st[kStCstar] < (uint64_t)kSelBins - 1 &&
                   st[kStEqual] > 4 * st[kStNeed] + (1u << 20);
  uint64_t nrec = st[kStAbove] + st[kStEqual];
  if (tie) {
    // Tuples that share all tokens but the newest are 2^18 at most: the digits
    // before it always reach the slack.
    const uint32_t slack = (1u << 18) + (uint32_t)(ranks / 4);
    for (int d = 0; d < 2 * (NG - 1); ++d) {
      hipLaunchKernelGGL(k_tie_hist<NG>, dim3(walkers), dim3(1024), 0, s, u, ts.pbits, d);
      hipLaunchKernelGGL(k_tie_pick, dim3(1), dim3(512), 0, s, a, d, slack);
    }
    BUILD_HIP(hipGetLastError(), "tie launches");
    BUILD_HIP(hipMemcpyAsync(&nrec, a.state + kStTieDone, sizeof nrec, hipMemcpyDeviceToHost, s),
              "copy");
    BUILD_HIP(hipStreamSynchronize(s), "sync");
    if (nrec < ranks) return fail(TFE_ERR_HIP, "tie selection");
  }
  // 5. Ranks [skip, ranks).  The remainders and their counts are not needed
  // once gathered: their arrays (nwin >= nrec entries each) are the ranking's
  // scratch.  Ranks of n records from rank 0 on by the bucket sort:
  auto rank_records = [&](R* rec, R* rec2, uint64_t n) {
    if (n <= kBucketCap / 2) {
      hipLaunchKernelGGL(k_bk_sort<R>, dim3(1), dim3(1024), 0, s, a, rec, (uint32_t)n, skip, ranks,
                         NG, out_tuples, out_counts);
      return;
    }
    uint32_t nb = 2;
    while (nb < kMaxBuckets && n / nb > kBucketMean) nb <<= 1;
    R* split = (R*)mcnt;  // fewer than n / 512 + 2 of at most 16 bytes
    uint16_t* bkt = (uint16_t*)ucnt;
    const uint32_t tiles = blocks_for(n, kBkTile);
    hipLaunchKernelGGL(k_bk_sample<R>, dim3(1), dim3(1024), 0, s, rec, n, nb, split);
    hipLaunchKernelGGL(k_bk_hist<R>, dim3(tiles), dim3(1024), 0, s, a, rec, n, nb, split, bkt);
    hipLaunchKernelGGL(k_bk_scatter<R>, dim3(tiles), dim3(1024), 0, s, a, rec, n, nb, bkt, rec2);
    hipLaunchKernelGGL(k_bk_sort<R>, dim3(nb), dim3(1024), 0, s, a, rec2, 0u, skip, ranks, NG,
                       out_tuples, out_counts);
  };
  const uint64_t m = ranks - skip;
  if (NG == 1 || nrec <= kBucketSortMax) {
    R* rec = sc.get<R>(nrec);
    R* rec2 = sc.get<R>(nrec);
    if (!rec || !rec2) return fail(TFE_ERR_OOM, "rank arrays");
    hipLaunchKernelGGL(k_gather<NG>, dim3(walkers), dim3(1024), 0, s, u, ts.pbits, tie ? 1u : 0u,
                       rec, (uint32_t)nrec);
    rank_records(rec, rec2, nrec);
  } else {
    // At most nwin / (kLowMax + 1) n-grams are above kLowMax (and c* is not: more
    // n-grams reach it).
    const uint64_t nhigh = st[kStHigh], nlow = nrec - nhigh;
    R* rec = sc.get<R>(nhigh);
    R* rec2 = sc.get<R>(nhigh);
    uint64_t* low = sc.get<uint64_t>(nlow);
    uint64_t* low_alt = sizeof(K) == 8 ? (uint64_t*)ukey : sc.get<uint64_t>(nlow);
    uint32_t* low3 = NG == 4 ? sc.get<uint32_t>(nlow) : nullptr;
    uint32_t* low3_alt = ucnt;
    if (!rec || !rec2 || !low || !low_alt || (NG == 4 && !low3))
      return fail(TFE_ERR_OOM, "rank arrays");
    hipLaunchKernelGGL(k_gather_long<NG>, dim3(walkers), dim3(1024), 0, s, u, ts.pbits, tie ? 1u : 0u,
                       rec, (uint32_t)nhigh, low, low3, (uint32_t)nlow);
    if (nhigh > skip) rank_records(rec, rec2, nhigh);
    // Histograms of kBins words per tile of at least 3072 records: below 4 bytes
    // a record.
    static_assert(kBins < tile_keys<uint64_t, true, uint32_t>(), "mcnt holds the histograms");
    if (NG == 4) {
      BUILD_HIP(radix_sort<true>(low3, low3_alt, low, low_alt, nlow, 18, mcnt, part, s), "rank sort");
      BUILD_HIP(radix_sort<true>(low, low_alt, low3, low3_alt, nlow, packed_tokens<NG>() + 9, mcnt,
                                 part, s),
                "rank sort");
    } else {
      BUILD_HIP(radix_sort<false>(low, low_alt, low3, low3_alt, nlow, packed_tokens<NG>() + 9, mcnt,
                                  part, s),
                "rank sort");
    }
    const uint64_t from = skip > nhigh ? skip - nhigh : 0, to = ranks - nhigh;
    hipLaunchKernelGGL(k_unpack<NG>, dim3(blocks_for(to - from, 256)), dim3(256), 0, s, low, low3, from,
                       to, nhigh, skip, out_tuples, out_counts);
  }
  BUILD_HIP(hipGetLastError(), "rank launches");
  BUILD_HIP(hipStreamSynchronize(s), "sync");
  *written = (int64_t)m;
  return TFE_OK;
}

tfe_status ngram_top(const int32_t* tokens, int64_t N, int32_t vocab, int32_t n, int64_t skip,
                     int64_t top, int32_t* out_tuples, int64_t* out_counts, int64_t* written,
                     hipStream_t s) {
  if (!written) return fail(TFE_ERR_INVALID_ARG, "null written");
  *written = 0;
  // The two-level scans cover up to 2^28 elements, a record 28-bit counts.
  if (N < 0 || N > (1ll << 28)) return fail(TFE_ERR_INVALID_ARG, "N outside [0, 2^28]");
  if (vocab < 1 || vocab > (1 << 18)) return fail(TFE_ERR_INVALID_ARG, "vocab outside [1, 2^18]");
  if (n < 1 || n > 4) return fail(TFE_ERR_UNSUPPORTED, "n = %d (1..4 supported)", n);
  if (skip < 0 || top < 0) return fail(TFE_ERR_INVALID_ARG, "negative skip or top");
  if (N < n || top == 0) return TFE_OK;
  if (!tokens || !out_tuples || !out_counts)
    return fail(TFE_ERR_INVALID_ARG, "null tokens or outputs");
  // Allocates scratch and waits for the stream: not capturable.
  {
    const tfe_status st = refuse_capture(s, "tfe_ngram_top");
    if (st != TFE_OK) return st;
  }
  const uint64_t nwin = (uint64_t)(N - n + 1);
  // Ranks beyond the number of windows do not exist (and the sum cannot
  // overflow).
  if ((uint64_t)skip >= nwin) return TFE_OK;
  const uint64_t t = std::min<uint64_t>((uint64_t)top, nwin);
  switch (n) {
    case 1: return ngram_top_n<1>(tokens, nwin, vocab, skip, t, out_tuples, out_counts, written, s);
    case 2: return ngram_top_n<2>(tokens, nwin, vocab, skip, t, out_tuples, out_counts, written, s);
    case 3: return ngram_top_n<3>(tokens, nwin, vocab, skip, t, out_tuples, out_counts, written, s);
    default: return ngram_top_n<4>(tokens, nwin, vocab, skip, t, out_tuples, out_counts, written, s);
  }
}

}  // namespace
}  // namespace tfe

extern "C" tfe_status tfe_ngram_release(void) {
  tfe::begin_call();
  std::lock_guard<std::mutex> lock(tfe::g_cache_mu);
  int cur = 0;
  (void)hipGetDevice(&cur);
  for (size_t i = 0; i < tfe::g_cache.size();) {
    if (!tfe::g_cache[i].used) {
      (void)hipSetDevice(tfe::g_cache[i].device);
      tfe::dev_free(tfe::g_cache[i].p);
      tfe::g_cache[i] = tfe::g_cache.back();
      tfe::g_cache.pop_back();
    } else {
      ++i;
    }
  }
  (void)hipSetDevice(cur);
  return TFE_OK;
}

extern "C" tfe_status tfe_ngram_top(const int32_t* tokens, int64_t n_tokens, int32_t vocab,
                                    int32_t n, int64_t skip, int64_t top, int32_t* out_tuples,
                                    int64_t* out_counts, int64_t* written, void* stream) {
  tfe::begin_call();
  return tfe::ngram_top(tokens, n_tokens, vocab, n, skip, top, out_tuples, out_counts, written,
                        (hipStream_t)stream);
}
