// The stable radix sort of up to kSmallSort items by one workgroup, and what it
// shares with the larger sort.
#pragma once

#include "dcem_internal.h"

namespace dcem {
namespace {

constexpr int kDigits = 256;

// Digit pass p of a sort on `bits` key bits of which the low word holds
// low_bits: its word (from the least significant) and shift.
struct Passes {
  int n, n_low;   // passes; those in the least significant word
  __host__ __device__ Passes(int bits, int low_bits) {
    const int low = (min_(min_(bits, low_bits), 32) + 7) / 8;
    n_low = low < 0 ? 0 : low;
    n = n_low + (bits > 32 ? (bits - 32 + 7) / 8 : 0);
  }
  __host__ __device__ static int min_(int a, int b) { return a < b ? a : b; }
  __host__ __device__ int bit(int p) const { return p < n_low ? 8 * p : 32 + 8 * (p - n_low); }
};

// Lanes of the wavefront with this lane's digit d (among the lanes of `valid`).
__device__ inline uint64_t digit_peers(uint64_t valid, uint32_t d) {
  uint64_t peers = valid;
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    const uint64_t m = __ballot((d >> b) & 1u);
    peers &= ((d >> b) & 1u) ? m : ~m;
  }
  return peers;
}

// Rank this lane's item among its wavefront's items of digit d so far; cnt:
// the wavefront's running digit counts in LDS.
__device__ inline uint32_t rank_digit(bool valid, uint32_t d, volatile uint32_t* cnt) {
  const int lane = threadIdx.x & (kWave - 1);
  const uint64_t peers = digit_peers(__ballot(valid), d);
  const uint64_t below = peers & ((1ull << lane) - 1ull);
  uint32_t before = 0;
  if (valid) before = cnt[d];
  wave_sync();
  if (valid && below == 0) cnt[d] = before + (uint32_t)__popcll(peers);
  wave_sync();
  return before + (uint32_t)__popcll(below);
}

// Exclusive prefix of v over the first kDigits threads of the block (threads
// beyond pass 0); tmp: kDigits / kWave words of LDS.
__device__ inline uint32_t digit_prefix(uint32_t v, uint32_t* tmp) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  uint32_t incl = v;
  for (int off = 1; off < kWave; off <<= 1) {
    const uint32_t t = __shfl_up(incl, off);
    if (lane >= off) incl += t;
  }
  if (lane == kWave - 1 && wave < kDigits / kWave) tmp[wave] = incl;
  __syncthreads();
  uint32_t before = 0;
  for (int w = 0; w < wave && w < kDigits / kWave; ++w) before += tmp[w];
  return before + incl - v;
}

constexpr int kSmallThreads = 1024, kSmallWaves = kSmallThreads / kWave;
constexpr int kSmallRounds = 16;                            // items per thread at most
constexpr int kSmallSort = kSmallThreads * kSmallRounds;

// LDS of the one-workgroup sort (144 KB): the permutation, the keys' current
// word, digit counts.
struct SmallSort {
  uint32_t idx[kSmallSort], key[kSmallSort];
  uint32_t cnt[kSmallWaves][kDigits], tmp[kDigits / kWave];
};

// Sort n <= kSmallSort items of word-major keys [W][stride] by the digits of
// `passes`; the permutation is left in s.idx.  By a block of kSmallThreads.  7
// passes over 2200 items take 32 us, in launches per pass 46 us and eight launch
// gaps.
__device__ __forceinline__ void sort_small(const uint32_t* __restrict__ keys, int64_t stride, int W,
                                           const Passes& passes, uint32_t n, SmallSort& s) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int rounds = (int)((n + kSmallThreads - 1) / kSmallThreads);
  const uint32_t base = wave * rounds * kWave + lane;   // this lane's items: every 64th from here
  if (passes.n == 0)
    for (uint32_t i = tid; i < n; i += kSmallThreads) s.idx[i] = i;
  for (int p = 0; p < passes.n; ++p) {
    const int bit = passes.bit(p), shift = bit & 31;
    const uint32_t* word = keys + (W - 1 - bit / 32) * stride;
    const bool fresh = p == 0 || passes.bit(p - 1) / 32 != bit / 32;   // the word is not in LDS yet
    for (int i = tid; i < kSmallWaves * kDigits; i += kSmallThreads) s.cnt[0][i] = 0;
    uint32_t item[kSmallRounds], key[kSmallRounds];   // index, and in the high half the rank
    static_assert(kSmallSort <= 1 << 16 && kSmallRounds * kWave <= 1 << 16, "packed");
#pragma unroll
    for (int r = 0; r < kSmallRounds; ++r) {
      const uint32_t i = base + r * kWave;
      item[r] = key[r] = 0;
      if (r >= rounds || i >= n) continue;
      item[r] = p == 0 ? i : s.idx[i];
      key[r] = fresh ? word[item[r]] : s.key[i];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSmallRounds; ++r) {
      if (r >= rounds) continue;
      item[r] |= rank_digit(base + r * kWave < n, (key[r] >> shift) & 255u, s.cnt[wave]) << 16;
    }
    __syncthreads();
    // offsets of (digit, wavefront): the digit's first place, then the wavefronts in order
    uint32_t c[kSmallWaves], total = 0;
    if (tid < kDigits)
      for (int w = 0; w < kSmallWaves; ++w) total += c[w] = s.cnt[w][tid];
    uint32_t at = digit_prefix(total, s.tmp);
    if (tid < kDigits)
      for (int w = 0; w < kSmallWaves; ++w) {
        s.cnt[w][tid] = at;
        at += c[w];
      }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSmallRounds; ++r) {
      if (r >= rounds || base + r * kWave >= n) continue;
      const uint32_t to = s.cnt[wave][(key[r] >> shift) & 255u] + (item[r] >> 16);
      s.idx[to] = item[r] & 0xffffu;
      s.key[to] = key[r];
    }
    __syncthreads();
  }
}

}  // namespace
}  // namespace dcem
