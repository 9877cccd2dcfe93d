// Stable LSD radix sort of multi-word keys into a permutation, 8 bits a pass.
//
// Keys are read through the source permutation; only the permutation moves.
// A wavefront ranks 64 items at a time with ballots: the lanes holding the same
// digit are found by intersecting one ballot per digit bit, and a lane's rank
// is the number of such peers below it plus the wavefront's running count of
// the digit.  Every wavefront owns consecutive items and runs through them on
// counters of its own, so a pass synchronises its block only between counting
// and placing.
//
// Up to kSmallSort items are sorted by one workgroup in one launch.  More take
// one launch per pass: the digit totals of all passes are counted once, in
// item order, and the blocks of a pass find their offsets by looking back at
// the counts of the blocks before them.
//
// Bound by latency, not bandwidth: a pass over 32768 items moves 0.4 MB and takes
// 9 us, most of it the ticket, two dependent gathers and the look-back.  It was
// three launches of 19 us together (counts, their scan, placing), and 34 to 40 us
// on 100000 items, now 12; 8000 items of 7 passes took 110 us, now 32 in one
// launch.
#include "dcem_internal.h"

namespace dcem {
namespace {

constexpr int kDigits = 256;

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

// The whole sort in one workgroup, the permutation and the keys' current word
// in LDS (144 KB).  7 passes over 2200 items of a list sized for 8500 take 32 us,
// in launches per pass 46 us and eight launch gaps.
__global__ __launch_bounds__(kSmallThreads) void k_sort_small(const uint32_t* __restrict__ keys, int64_t stride, int W,
                                                              int passes, const uint32_t* __restrict__ n_dev,
                                                              uint32_t n_max, uint32_t* __restrict__ perm) {
  __shared__ uint32_t sidx[kSmallSort], skey[kSmallSort];
  __shared__ uint32_t cnt[kSmallWaves][kDigits], tmp[kDigits / kWave];
  const uint32_t n = min(min(*n_dev, n_max), (uint32_t)kSmallSort);
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int rounds = (int)((n + kSmallThreads - 1) / kSmallThreads);
  const uint32_t base = wave * rounds * kWave + lane;   // this lane's items: every 64th from here
  for (int p = 0; p < passes; ++p) {
    const int bit = 8 * p, shift = bit & 31;
    const uint32_t* word = keys + (W - 1 - bit / 32) * stride;
    const bool fresh = p == 0 || 8 * (p - 1) / 32 != bit / 32;   // the word is not in LDS yet
    for (int i = tid; i < kSmallWaves * kDigits; i += kSmallThreads) cnt[0][i] = 0;
    uint32_t idx[kSmallRounds], key[kSmallRounds], rank[kSmallRounds];
#pragma unroll
    for (int r = 0; r < kSmallRounds; ++r) {
      const uint32_t i = base + r * kWave;
      idx[r] = key[r] = 0;
      if (r >= rounds || i >= n) continue;
      idx[r] = p == 0 ? i : sidx[i];
      key[r] = fresh ? word[idx[r]] : skey[i];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSmallRounds; ++r) {
      if (r >= rounds) continue;
      rank[r] = rank_digit(base + r * kWave < n, (key[r] >> shift) & 255u, cnt[wave]);
    }
    __syncthreads();
    // offsets of (digit, wavefront): the digit's first place, then the wavefronts in order
    uint32_t c[kSmallWaves], total = 0;
    if (tid < kDigits)
      for (int w = 0; w < kSmallWaves; ++w) total += c[w] = cnt[w][tid];
    uint32_t at = digit_prefix(total, tmp);
    if (tid < kDigits)
      for (int w = 0; w < kSmallWaves; ++w) {
        cnt[w][tid] = at;
        at += c[w];
      }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSmallRounds; ++r) {
      if (r >= rounds || base + r * kWave >= n) continue;
      const uint32_t to = cnt[wave][(key[r] >> shift) & 255u] + rank[r];
      sidx[to] = idx[r];
      skey[to] = key[r];
    }
    __syncthreads();
  }
  for (uint32_t i = tid; i < n; i += kSmallThreads) perm[i] = passes ? sidx[i] : i;
}

constexpr int kThreads = 256, kWaves = kThreads / kWave;

// Scratch of a larger sort, all zero at first: the digit totals and the ticket
// of every pass, then the tiles' look-back words, which carry their pass.
struct SortScratch {
  uint32_t* totals;   // [passes][kDigits]
  uint32_t* ticket;   // [passes]
  uint64_t* state;    // [tiles][kDigits]
  __host__ SortScratch(void* p, int passes) {
    totals = static_cast<uint32_t*>(p);
    ticket = totals + (size_t)passes * kDigits;
    state = reinterpret_cast<uint64_t*>(ticket + (passes + 1) / 2 * 2);
  }
  static size_t words(int passes, int64_t tiles) {
    return (size_t)passes * kDigits + (passes + 1) / 2 * 2 + 2 * (size_t)tiles * kDigits;
  }
};

// Digit totals of every pass, in item order: one pass over the keys.  Every block
// adds its counts to the same few thousand words, so few, large blocks: 128 to 256
// of 1024 threads count 100000 items of 7 passes in 7 us, 400 of 256 in 9, 245000 of 5
// in 9 and 12.5.
constexpr int kTotalThreads = 1024;

__global__ __launch_bounds__(kTotalThreads) void k_digit_totals(const uint32_t* __restrict__ keys, int64_t stride, int W,
                                                           int passes, const uint32_t* __restrict__ n_dev,
                                                           uint32_t n_max, uint32_t* __restrict__ totals) {
  extern __shared__ uint32_t cnt[];   // [passes][kDigits]
  const uint32_t n = min(*n_dev, n_max);
  const int lane = threadIdx.x & (kWave - 1);
  for (int i = threadIdx.x; i < passes * kDigits; i += kTotalThreads) cnt[i] = 0;
  __syncthreads();
  for (uint64_t i0 = (uint64_t)blockIdx.x * kTotalThreads; i0 < n; i0 += (uint64_t)gridDim.x * kTotalThreads) {
    const uint64_t i = i0 + threadIdx.x;
    const bool valid = i < n;
    int have = -1;
    uint32_t key = 0;
    for (int p = 0; p < passes; ++p) {
      const int bit = 8 * p;
      if (bit / 32 != have) {
        have = bit / 32;
        key = valid ? keys[(W - 1 - have) * stride + i] : 0u;
      }
      const uint32_t d = (key >> (bit & 31)) & 255u;
      // a digit that all lanes share is one addition
      const uint64_t m = __ballot(valid);
      const uint32_t d0 = __builtin_amdgcn_readfirstlane(d);
      if (__ballot(valid && d != d0) == 0 && (m & 1ull)) {
        if (lane == 0) atomicAdd(&cnt[p * kDigits + d0], (uint32_t)__popcll(m));
      } else if (valid) {
        atomicAdd(&cnt[p * kDigits + d], 1u);
      }
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < passes * kDigits; i += kTotalThreads)
    if (cnt[i]) atomicAdd(&totals[i], cnt[i]);
}

// A tile's look-back word for one digit: its own count or, with kUpTo, the
// count of all tiles up to it (low half), and from bit 33 the pass (from 1).
constexpr uint64_t kUpTo = 1ull << 32;
constexpr int kPassBit = 33;

__device__ inline uint64_t load_state(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void store_state(uint64_t* p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One pass.  Tiles are taken by ticket, so a block waits only for tiles whose
// blocks are already running; each of those stores its counts before it waits
// for any other, so every wait ends.  (A word carries its own flag: relaxed
// order is enough.)  Thread d looks back for digit d, kBack tiles at a time.
template <int R>
__global__ __launch_bounds__(kThreads) void k_sort_pass(const uint32_t* __restrict__ keys, int shift,
                                                        const uint32_t* __restrict__ src, uint32_t* __restrict__ dst,
                                                        const uint32_t* __restrict__ n_dev, uint32_t n_max,
                                                        const uint32_t* __restrict__ totals,
                                                        uint32_t* __restrict__ ticket, uint64_t* __restrict__ state,
                                                        uint64_t pass) {
  constexpr int kBack = 8;
  __shared__ uint32_t cnt[kWaves][kDigits], tmp[kDigits / kWave], my_tile;
  const uint32_t n = min(*n_dev, n_max);
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  if (tid == 0) my_tile = atomicAdd(ticket, 1u);
  for (int w = 0; w < kWaves; ++w) cnt[w][tid] = 0;
  const uint32_t total = totals[tid];
  __syncthreads();
  const uint32_t tile = my_tile;
  const uint64_t first = (uint64_t)tile * (R * kThreads);
  if (first >= n) return;   // (so are all tiles after it)
  const uint64_t base = first + wave * (R * kWave) + lane;
  uint32_t idx[R], key[R], rank[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint64_t i = base + r * kWave;
    idx[r] = i < n ? (src ? src[i] : (uint32_t)i) : 0u;
  }
#pragma unroll
  for (int r = 0; r < R; ++r) key[r] = base + r * kWave < n ? (keys[idx[r]] >> shift) & 255u : 0u;
#pragma unroll
  for (int r = 0; r < R; ++r) rank[r] = rank_digit(base + r * kWave < n, key[r], cnt[wave]);
  __syncthreads();
  uint32_t c[kWaves], own = 0;
  for (int w = 0; w < kWaves; ++w) own += c[w] = cnt[w][tid];
  uint64_t* mine = state + (size_t)tile * kDigits + tid;
  const uint64_t tag = pass << kPassBit;
  store_state(mine, tag | (tile == 0 ? kUpTo : 0) | own);
  uint32_t before = 0;
  for (int64_t t = (int64_t)tile - 1; t >= 0;) {
    uint64_t s[kBack];
#pragma unroll
    for (int j = 0; j < kBack; ++j) s[j] = t - j >= 0 ? load_state(state + (size_t)(t - j) * kDigits + tid) : tag | kUpTo;
    bool done = false;
    int used = 0;
#pragma unroll
    for (int j = 0; j < kBack; ++j) {
      if (done || used < j || s[j] >> kPassBit != pass) continue;   // not stored yet: asked for again
      before += (uint32_t)s[j];
      used = j + 1;
      done = (s[j] & kUpTo) != 0;
    }
    if (done) break;
    t -= used;
  }
  if (tile > 0) store_state(mine, tag | kUpTo | (uint64_t)(before + own));
  uint32_t at = digit_prefix(total, tmp) + before;
  for (int w = 0; w < kWaves; ++w) {
    cnt[w][tid] = at;
    at += c[w];
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (base + r * kWave < n) dst[cnt[wave][key[r]] + rank[r]] = idx[r];
}

// Items per thread of a pass: few while that leaves compute units idle, then
// more tiles than the look-back wants.  Per pass with 4, 8 and 16: 245000 items
// (240, 120, 60 tiles) 17.7, 14.7 and 18.0 us; 400000 items 26, 20 and 21 us; at
// 32768 items 2 and 4 take 9.3 and 9.0 us.
int sort_rounds(int64_t n_max) { return n_max <= (int64_t)4 * kThreads * 256 ? 4 : 8; }

int64_t sort_tiles(int64_t n_max) {
  const int64_t tile = (int64_t)sort_rounds(n_max) * kThreads;
  return (n_max + tile - 1) / tile;
}

hipError_t ensure_scratch(dcem_ctx* c, int passes, int64_t n_max) {
  if (n_max <= kSmallSort) return hipSuccess;
  return ensure(c->sort_hist, sizeof(uint32_t) * SortScratch::words(passes, sort_tiles(n_max)));
}

}  // namespace

hipError_t prepare_sort(dcem_ctx* c, int bits, int64_t n_max) {
  return ensure_scratch(c, (bits + 7) / 8, n_max);
}

hipError_t radix_sort_perm(dcem_ctx* c, const uint32_t* keys, int W, int bits, const uint32_t* n_dev,
                           int64_t n_max, uint32_t* perm, uint32_t* perm_tmp, hipStream_t s, int64_t stride) {
  if (n_max <= 0) return hipSuccess;
  if (stride < 0) stride = n_max;
  const int passes = (bits + 7) / 8;
  if (n_max <= kSmallSort) {
    hipLaunchKernelGGL(k_sort_small, dim3(1), dim3(kSmallThreads), 0, s, keys, stride, W, passes, n_dev,
                       (uint32_t)n_max, perm);
    return hipGetLastError();
  }
  const int64_t tiles = sort_tiles(n_max);
  hipError_t e = ensure_scratch(c, passes, n_max);
  if (e != hipSuccess) return e;
  const SortScratch sc(c->sort_hist.p, passes);
  fill_u32(sc.totals, 0u, SortScratch::words(passes, tiles), s);
  const unsigned blocks = (unsigned)std::min<int64_t>((n_max + kTotalThreads - 1) / kTotalThreads, 256);
  hipLaunchKernelGGL(k_digit_totals, dim3(blocks), dim3(kTotalThreads), sizeof(uint32_t) * kDigits * passes, s, keys,
                     stride, W, passes, n_dev, (uint32_t)n_max, sc.totals);
  const uint32_t* src = nullptr;
  for (int p = 0; p < passes; ++p) {
    uint32_t* dst = (passes - 1 - p) % 2 == 0 ? perm : perm_tmp;
    const int bit = 8 * p;
    const auto pass = sort_rounds(n_max) == 4 ? k_sort_pass<4> : k_sort_pass<8>;
    hipLaunchKernelGGL(pass, dim3((unsigned)tiles), dim3(kThreads), 0, s, keys + (W - 1 - bit / 32) * stride, bit & 31,
                       src, dst, n_dev, (uint32_t)n_max, sc.totals + (size_t)p * kDigits, sc.ticket + p,
                       sc.state, (uint64_t)p + 1);
    src = dst;
  }
  return hipGetLastError();
}

}  // namespace dcem
