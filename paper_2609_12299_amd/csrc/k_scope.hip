// k_scope.hip -- iteration ordinals and scoped per-region statistics.
//
// The paper's Section 3.2 separates a region (the code a developer changes)
// from its scope (which dynamic executions are reported: a warp role, an
// iteration window, an SM subset), and Section 3.3 specialises probes to one
// iteration of a loop region.  The iteration of an instance is its ordinal
// among the instances of its context with the same BEGIN region, in
// canonical (context, begin time) order.
//
// Ordinals: the instance array is already ordered by context, so within any
// stretch of it a stable sort by region alone yields (region, context,
// canonical) order, in which the instances of one (context, region) form a
// run; an instance's ordinal among them is its distance from the start of
// its run.  Up to kSoMaxRegions regions, this is done per chunk of 4096
// consecutive instances, in LDS: each chunk's ordinals are exact except for
// the context that enters it from earlier chunks, whose counts per region
// (the carry) come from a scan over the chunks' counts of their last
// context, and are added where the statistics read the ordinals.  With more
// regions the whole array is sorted: an LSD radix sort over the region's
// 8-bit digits (per 4096-element tile a digit histogram, one exclusive scan
// over the digit-major histograms, then a stable scatter that ranks each
// tile's elements with eight ballots per wave), run starts from a wave
// max-scan of the run heads with one binary search per wave for a run that
// began before it, and the ordinals scattered back to canonical order.  The
// scoped statistics are taken in canonical order.
#include <string.h>

#include <algorithm>
#include <mutex>

#include "radix_tile.h"

namespace argus {

constexpr int kScThreads = 256;
constexpr int kScRounds = 16;
constexpr uint32_t kScTile = kScThreads * kScRounds;  // 4096 elements
constexpr uint32_t kScScanBlock = 4096;                // entries per scan block
// Ordinals reach their instances in two steps: (index, ordinal) pairs are
// gathered per bucket of 2^18 consecutive instance indices, then each bucket
// is written by blocks of one XCD, whose L2 holds the bucket's 1 MiB of
// output while they write it.
constexpr uint32_t kOrdBucketBits = 18;
constexpr uint32_t kOrdMaxBuckets = 1u << (31 - kOrdBucketBits);  // instances < 2^31
constexpr uint32_t kOrdSlices = 128;                              // blocks per bucket

// A stable LSD radix sort over 8-bit digits of 16-byte elements (two u64
// words, ping-pong buffers).  The first pass may read the instance array
// instead (word a = BEGIN region, word b = context << 32 | index).
struct SortBufs {
  uint64_t* a[2];
  uint64_t* b[2];
  uint32_t* hist;  // [256][tiles_max], digit-major
  uint32_t* bsum;  // scan block sums
  uint64_t tiles_max;
  const uint64_t* count_ptr;  // device element count (clamped to count_max), or NULL
  uint64_t count_max;
  const argus_instance* inst;  // source of the SRC_INST passes
};
enum { kSrcBuf = 0, kSrcInst = 1 };

__device__ __forceinline__ uint64_t sb_count(const SortBufs& s) {
  if (!s.count_ptr) return s.count_max;
  const uint64_t v = *s.count_ptr;
  return v < s.count_max ? v : s.count_max;
}

template <int SRC>
__device__ __forceinline__ void sb_load(const SortBufs& s, int in, uint64_t e, uint64_t* a,
                                        uint64_t* b) {
  if (SRC == kSrcInst) {
    const uint4 h1 = reinterpret_cast<const uint4*>(s.inst)[2 * e + 1];
    *a = h1.w & 0xFFFFu;
    *b = ((uint64_t)h1.x << 32) | e;
  } else {
    *a = s.a[in][e];
    *b = s.b[in][e];
  }
}

// Per tile: counts of each digit, written digit-major (zeros for tiles past
// the element count, so that the scan sees a complete table).
template <int SRC>
__global__ __launch_bounds__(kScThreads) void k_sort_hist(SortBufs s, int in, int word, int shift) {
  __shared__ uint32_t s_cnt[256];
  const uint64_t n = sb_count(s);
  const uint64_t tile = blockIdx.x;
  s_cnt[threadIdx.x] = 0;
  __syncthreads();
  const uint64_t base = tile * kScTile;
  for (uint32_t j = 0; j < kScRounds; ++j) {
    const uint64_t e = base + (uint64_t)j * kScThreads + threadIdx.x;
    if (e < n) {
      uint64_t a, b;
      sb_load<SRC>(s, in, e, &a, &b);
      atomicAdd(&s_cnt[((word ? b : a) >> shift) & 0xFFu], 1u);
    }
  }
  __syncthreads();
  s.hist[(uint64_t)threadIdx.x * s.tiles_max + tile] = s_cnt[threadIdx.x];
}

// Exclusive scan of a u32 array in three launches: block sums, their scan
// (one block), then each block's scan plus its base.
__global__ __launch_bounds__(kScThreads) void k_scan_sums(uint32_t* data, uint64_t total,
                                                          uint32_t* bsum) {
  __shared__ uint32_t s_part[kScThreads / 64];
  const uint64_t base = (uint64_t)blockIdx.x * kScScanBlock;
  uint32_t v = 0;
  for (uint32_t j = threadIdx.x; j < kScScanBlock; j += kScThreads)
    if (base + j < total) v += data[base + j];
  v = rows_sum32(row_sum32(v));
  if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) bsum[blockIdx.x] = s_part[0] + s_part[1] + s_part[2] + s_part[3];
}

// Exclusive scan of v over the block; *carry (LDS) holds the running total
// across calls.  Every thread of the block must call it.
template <int NT>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* s_w, uint32_t* carry) {
  const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = __shfl_up(x, d);
    if (lane >= (uint32_t)d) x += y;
  }
  if (lane == 63) s_w[w] = x;
  __syncthreads();
  uint32_t wpre = 0;
  for (uint32_t k = 0; k < w; ++k) wpre += s_w[k];
  const uint32_t c = *carry;
  __syncthreads();
  if (threadIdx.x == NT - 1) *carry = c + wpre + x;
  __syncthreads();
  return c + wpre + x - v;
}

__global__ __launch_bounds__(1024) void k_scan_top(uint32_t* bsum, uint32_t blocks) {
  __shared__ uint32_t s_carry;
  __shared__ uint32_t s_w[16];
  if (threadIdx.x == 0) s_carry = 0;
  __syncthreads();
  for (uint32_t b0 = 0; b0 < blocks; b0 += 1024) {
    const uint32_t b = b0 + threadIdx.x;
    const uint32_t v = b < blocks ? bsum[b] : 0u;
    const uint32_t ex = block_excl_scan<1024>(v, s_w, &s_carry);
    if (b < blocks) bsum[b] = ex;
  }
}

__global__ __launch_bounds__(kScThreads) void k_scan_apply(uint32_t* data, uint64_t total,
                                                           const uint32_t* bsum) {
  __shared__ uint32_t s_w[kScThreads / 64];
  __shared__ uint32_t s_carry;
  const uint64_t base = (uint64_t)blockIdx.x * kScScanBlock;
  if (threadIdx.x == 0) s_carry = bsum[blockIdx.x];
  __syncthreads();
  for (uint32_t j0 = 0; j0 < kScScanBlock; j0 += kScThreads) {
    const uint64_t i = base + j0 + threadIdx.x;
    const uint32_t v = i < total ? data[i] : 0u;
    const uint32_t ex = block_excl_scan<kScThreads>(v, s_w, &s_carry);
    if (i < total) data[i] = ex;
  }
}

// A small table scanned by one block: staged in LDS with coalesced loads,
// each of 1024 threads sums a stretch of consecutive entries, one block scan
// places the stretches, each thread writes its stretch's exclusive prefixes
// in LDS, and the table goes back with coalesced stores.
constexpr uint64_t kScSmallMax = 32768;
__global__ __launch_bounds__(1024) void k_scan_small(uint32_t* data, uint64_t total) {
  __shared__ uint32_t s_d[kScSmallMax];
  __shared__ uint32_t s_carry;
  __shared__ uint32_t s_w[16];
  const uint32_t t = threadIdx.x, n = (uint32_t)total;
  for (uint32_t i = t; i < n; i += 1024) s_d[i] = data[i];
  if (t == 0) s_carry = 0;
  __syncthreads();
  const uint32_t per = (n + 1023) / 1024, b = t * per;
  uint32_t v = 0;
  for (uint32_t k = 0; k < per; ++k)
    if (b + k < n) v += s_d[b + k];
  uint32_t run = block_excl_scan<1024>(v, s_w, &s_carry);
  for (uint32_t k = 0; k < per; ++k) {
    if (b + k >= n) break;
    const uint32_t d = s_d[b + k];
    s_d[b + k] = run;
    run += d;
  }
  __syncthreads();
  for (uint32_t i = t; i < n; i += 1024) data[i] = s_d[i];
}

// Stable scatter of one tile.  Each wave takes 1024 consecutive elements
// (16 rounds of 64 lanes, all loaded up front) and ranks each among the
// wave's earlier elements of its digit: eight ballots find the lanes that
// share it, and per-wave digit counters in LDS carry the earlier rounds
// (wave barriers only).  One block barrier later the waves' counts give
// each digit's offset per wave and the tile-local digit starts; the tile is
// staged in LDS in digit order and written out so that a run of equal
// digits goes to consecutive addresses.
constexpr size_t kScStageBytes = 2 * sizeof(uint64_t) * kScTile;  // dynamic LDS of k_sort_scatter
template <int SRC>
__global__ __launch_bounds__(kScThreads) void k_sort_scatter(SortBufs s, int in, int out, int word,
                                                             int shift) {
  extern __shared__ __align__(16) uint8_t sc_stage[];
  uint64_t* s_ta = reinterpret_cast<uint64_t*>(sc_stage);
  uint64_t* s_tb = s_ta + kScTile;
  __shared__ uint32_t s_wave[4][256];  // per-wave digit counts, then each wave's offset in the digit
  __shared__ uint32_t s_base[256];
  __shared__ uint32_t s_lstart[256];
  __shared__ uint32_t s_w[kScThreads / 64];
  __shared__ uint32_t s_carry;
  const uint64_t n = sb_count(s);
  const uint64_t tile = blockIdx.x;
  const uint32_t tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
#pragma unroll
  for (int q = 0; q < 4; ++q) s_wave[q][tid] = 0;
  s_base[tid] = s.hist[(uint64_t)tid * s.tiles_max + tile];
  if (tid == 0) s_carry = 0;
  uint64_t av[kScRounds], bv[kScRounds];
  uint32_t dg[kScRounds], rk[kScRounds];
  const uint64_t e0 = tile * kScTile + (uint64_t)w * (kScRounds * 64) + lane;
#pragma unroll
  for (int r = 0; r < kScRounds; ++r) {
    const uint64_t e = e0 + (uint64_t)r * 64;
    av[r] = 0;
    bv[r] = 0;
    if (e < n) sb_load<SRC>(s, in, e, &av[r], &bv[r]);
  }
  __syncthreads();  // counters cleared
  const uint64_t lt = lanemask_lt();
#pragma unroll
  for (int r = 0; r < kScRounds; ++r) {
    const bool valid = e0 + (uint64_t)r * 64 < n;
    const uint32_t d = (uint32_t)(((word ? bv[r] : av[r]) >> shift) & 0xFFu);
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) {
      const uint64_t bal = __ballot((d >> bit) & 1u);
      peers &= ((d >> bit) & 1u) ? bal : ~bal;
    }
    uint32_t rank = 0;
    if (valid) {
      const uint32_t old = s_wave[w][d];
      rank = old + (uint32_t)__popcll(peers & lt);
      __builtin_amdgcn_wave_barrier();
      if ((peers >> lane) == 1ull) s_wave[w][d] = old + (uint32_t)__popcll(peers);
    }
    __builtin_amdgcn_wave_barrier();
    dg[r] = valid ? d : 256u;
    rk[r] = rank;
  }
  __syncthreads();
  // thread tid owns digit tid: the waves' offsets within it, the tile's count
  // of it, and (scanned) where it starts in the staged tile
  uint32_t cnt = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t c = s_wave[q][tid];
    s_wave[q][tid] = cnt;
    cnt += c;
  }
  s_lstart[tid] = block_excl_scan<kScThreads>(cnt, s_w, &s_carry);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kScRounds; ++r) {
    const uint32_t d = dg[r];
    if (d >= 256u) continue;
    const uint32_t slot = s_lstart[d] + s_wave[w][d] + rk[r];
    if (slot < kScTile) {
      s_ta[slot] = av[r];
      s_tb[slot] = bv[r];
    }
  }
  __syncthreads();
  const uint32_t total = s_carry;  // the tile's elements
  uint64_t* da = s.a[out];
  uint64_t* db = s.b[out];
  for (uint32_t i = tid; i < total && i < kScTile; i += kScThreads) {
    const uint64_t a = s_ta[i], b = s_tb[i];
    const uint32_t d = (uint32_t)(((word ? b : a) >> shift) & 0xFFu);
    const uint64_t dst = (uint64_t)s_base[d] + (i - s_lstart[d]);
    if (dst < n) {
      da[dst] = a;
      db[dst] = b;
    }
  }
}

// Scope counters: slot 7 holds internal-error bits (zero unless a
// consistency check inside the library fails).
__device__ __forceinline__ void sc_flag(uint64_t* counters, uint64_t code) {
  atomicOr((unsigned long long*)&counters[ARGUS_SC_INTERNAL], (unsigned long long)code);
}

// Chunk-local ordinals (up to kSoMaxRegions regions).
constexpr uint32_t kSoMaxRegions = 4096;
constexpr uint32_t kSoCont = 1;    // the chunk's last context continues into the next chunk
constexpr uint32_t kSoWhole = 2;   // the chunk holds one context
constexpr uint32_t kSoPcont = 4;   // the chunk's first context began in an earlier chunk
constexpr uint32_t kSoPending = 0x80000000u;  // ordinal still lacks its chunk's carry: region << 12 | local
constexpr uint32_t kSoMaskShift = 16;         // bits 16..31: the chunk's granules that may hold instances in scope
constexpr uint32_t kSoGranule = kScTile / 16; // 256 instances
static_assert(kSoMaxRegions <= 4096 && kScTile <= 4096, "12 bits each in a pending ordinal");
constexpr uint32_t kSoSeg = 256;   // chunks per segment of the carry scan
// Up to this capacity of the instance buffer the granules are not marked and
// all are read: marking costs the ordinal pass, whose waves walk a chunk in 64
// dependent rounds, 6 us (12 with a region set), and what it saves is less
// (iterations 0..15, 1024 regions, buffers half full: capacity 2^21 251 us
// unmarked, 256 marked; 2^22 278, 282; 2^23 298 each; 2^24 362, 354).
constexpr uint64_t kSoMarkMin = 1ull << 22;

struct ScopeArgs {
  const argus_instance* inst;
  const uint64_t* excl;
  uint32_t R;
  argus_scope sc;
  const uint8_t* region_mask;
  uint32_t* ordinal;
  uint64_t* stats;
  uint64_t* counters;
  SortBufs s;         // count = the instances
  uint32_t* octr;     // [kOrdMaxBuckets] pairs gathered per bucket so far
  uint64_t* pairs;    // [count] ordinal << 32 | index, by bucket (a free sort buffer)
  uint32_t* hkey;     // [count] histogram keys (a free sort buffer): one per instance, or (fast) those
                      // of each granule's matched instances in scope, from the granule's start
  uint16_t* gcnt;     // [granules] histogram keys of each granule (a free sort buffer)
  uint32_t* cneed;    // [chunks] 1: a chunk inside one context whose ordinals reach the window (ditto)
  // chunk-local ordinals
  uint32_t fast;      // 1: k_so_local wrote the ordinals; k_sc_stats adds the carries
  uint32_t* tail;     // [chunks][R] counts of the chunk's last context per region, then
                      // the carry entering each chunk whose first context began earlier
  uint32_t* cflag;    // [chunks] kSoCont | kSoWhole | kSoPcont, and the granules' bits
  uint32_t* segb;     // [segments][R] segment composites, then the carry entering each
  uint32_t* segm;     // [segments] 1: the segment passes its entering carry on
  uint32_t hslice, hslices, hranges;  // k_sc_hist: regions per slice, slices, ranges of granules
  uint32_t hper;                      // granules a wave takes at a time (1..64)
};

// Fill kernel for the outputs that are accumulated.
__global__ __launch_bounds__(kScThreads) void k_sc_init(ScopeArgs a) {
  const uint64_t total = (uint64_t)a.R * ARGUS_RS_WIDTH;
  for (uint64_t i = (uint64_t)blockIdx.x * kScThreads + threadIdx.x; i < total;
       i += (uint64_t)gridDim.x * kScThreads) {
    const uint32_t col = (uint32_t)(i % ARGUS_RS_WIDTH);
    a.stats[i] = (col == ARGUS_RS_INCL_MIN || col == ARGUS_RS_EXCL_MIN) ? kU64Max : 0ull;
  }
  if (blockIdx.x == 0 && threadIdx.x < ARGUS_SC_NUM_COUNTERS) a.counters[threadIdx.x] = 0;
  for (uint64_t i = (uint64_t)blockIdx.x * kScThreads + threadIdx.x; i < kOrdMaxBuckets;
       i += (uint64_t)gridDim.x * kScThreads)
    a.octr[i] = 0;
}

// Start of the (key, ctx) run that holds sorted element e, by one wave:
// lane k probes e - 2^k (one round trip brackets the start), then 64 probes
// per step narrow the bracket.
__device__ __forceinline__ uint64_t run_start_wave(const uint64_t* ka, const uint64_t* kb, uint64_t e,
                                                   uint64_t key, uint32_t ctx) {
  const uint32_t lane = threadIdx.x & 63;
  auto same = [&](uint64_t p) { return ka[p] == key && (uint32_t)(kb[p] >> 32) == ctx; };
  // p = e - 2^lane; "outside" when p < 0 or its element is of another run
  const bool in = lane < 63 && (1ull << lane) <= e && same(e - (1ull << lane));
  const uint64_t out = __ballot(!in);
  const uint32_t j = (uint32_t)__ffsll((unsigned long long)out) - 1;  // first lane outside
  if (j == 0) return e;  // e - 1 is outside: e starts its run
  // the start lies in (e - 2^j, e - 2^(j-1)]: the first position whose element is in the run
  uint64_t lo = (1ull << j) <= e ? e - (1ull << j) + 1 : 0;  // lo .. hi may hold the start
  uint64_t hi = e - (1ull << (j - 1));
  while (lo < hi) {
    const uint64_t span = hi - lo;
    const uint64_t p = lo + span * lane / 64;
    const bool ok = same(p);
    // the smallest probe inside the run bounds the start from above; the
    // largest probe outside from below
    const uint64_t ins = __ballot(ok);
    const uint64_t outs = __ballot(!ok);
    if (ins) {
      const uint32_t f = (uint32_t)__ffsll((unsigned long long)ins) - 1;
      const uint64_t pf = lo + span * f / 64;
      uint64_t nlo = lo;
      if (outs & ((1ull << f) - 1ull)) {
        const uint32_t g = 63u - (uint32_t)__clzll(outs & ((1ull << f) - 1ull));
        nlo = lo + span * g / 64 + 1;
      }
      lo = nlo;
      hi = pf;
    } else {
      lo = lo + span * 63 / 64 + 1;
    }
  }
  return lo;
}

// Ordinal of each sorted element: its distance from the start of its
// (region, context) run.  A block takes 4096 sorted elements (16 rounds of
// 64 per wave, chunk c = 4 * round + wave).  The start of a run that began
// before an element's chunk is the last head of the chunks before it, or
// (before the tile's first head) the start of the run holding the tile's
// first element.  The (index, ordinal) pairs go to the buckets of their
// indices, each block reserving its share of a bucket once.
__global__ __launch_bounds__(kScThreads) void k_sc_ordinal(ScopeArgs a, int buf) {
  __shared__ uint32_t s_cnt[kOrdMaxBuckets];  // per bucket: count, then global base
  __shared__ int64_t s_last[4 * kScRounds];   // last head in each chunk, then the run start entering it
  __shared__ uint64_t s_tstart;
  const uint64_t n = sb_count(a.s);
  const uint64_t* ka = a.s.a[buf];
  const uint64_t* kb = a.s.b[buf];
  const uint32_t tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const uint32_t nbk = (uint32_t)((n + (1ull << kOrdBucketBits) - 1) >> kOrdBucketBits);
  uint32_t best = 0;
  for (uint64_t tile = blockIdx.x; tile * kScTile < n; tile += gridDim.x) {
    const uint64_t t0 = tile * kScTile;
    for (uint32_t b = tid; b < nbk; b += kScThreads) s_cnt[b] = 0;
    if (w == 0) {
      const uint64_t st = run_start_wave(ka, kb, t0, ka[t0], (uint32_t)(kb[t0] >> 32));
      if (lane == 0) s_tstart = st;
    }
    // heads, and the last head at or before each lane within its chunk
    int64_t h[kScRounds];
    uint32_t idx[kScRounds];
#pragma unroll
    for (int r = 0; r < kScRounds; ++r) {
      const uint64_t e = t0 + (uint64_t)r * kScThreads + (uint64_t)w * 64 + lane;
      const bool valid = e < n;
      bool head = false;
      idx[r] = 0xFFFFFFFFu;
      if (valid) {
        const uint64_t key = ka[e];
        const uint64_t vv = kb[e];
        idx[r] = (uint32_t)vv;
        head = e == 0 || ka[e - 1] != key || (uint32_t)(kb[e - 1] >> 32) != (uint32_t)(vv >> 32);
      }
      int64_t x = head ? (int64_t)e : -1;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int64_t o = __shfl_up(x, d);
        if (lane >= (uint32_t)d && o > x) x = o;
      }
      h[r] = x;
      if (lane == 63) s_last[4 * r + w] = x;
    }
    __syncthreads();
    if (tid == 0) {
      int64_t run = (int64_t)s_tstart;
      for (uint32_t c = 0; c < 4 * kScRounds; ++c) {
        const int64_t l = s_last[c];
        s_last[c] = run;  // the run start entering chunk c
        if (l >= 0) run = l;
      }
    }
    __syncthreads();
    uint64_t pr[kScRounds];
    uint32_t bk[kScRounds], slot[kScRounds];
#pragma unroll
    for (int r = 0; r < kScRounds; ++r) {
      const uint64_t e = t0 + (uint64_t)r * kScThreads + (uint64_t)w * 64 + lane;
      bk[r] = 0xFFFFFFFFu;
      if (e >= n) continue;
      const int64_t hs = h[r] >= 0 ? h[r] : s_last[4 * r + w];
      if (idx[r] < n && hs >= 0 && (uint64_t)hs <= e) {
        const uint32_t ord = (uint32_t)(e - (uint64_t)hs);
        best = best > ord + 1 ? best : ord + 1;
        bk[r] = idx[r] >> kOrdBucketBits;
        slot[r] = atomicAdd(&s_cnt[bk[r]], 1u);
        pr[r] = ((uint64_t)ord << 32) | idx[r];
      } else {
        sc_flag(a.counters, 1);
      }
    }
    __syncthreads();
    for (uint32_t b = tid; b < nbk; b += kScThreads) {
      const uint32_t c = s_cnt[b];
      if (c) s_cnt[b] = atomicAdd(&a.octr[b], c);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kScRounds; ++r) {
      if (bk[r] == 0xFFFFFFFFu) continue;
      const uint64_t at = ((uint64_t)bk[r] << kOrdBucketBits) + s_cnt[bk[r]] + slot[r];
      if (at < n) a.pairs[at] = pr[r];
      else sc_flag(a.counters, 1);
    }
    __syncthreads();
  }
  // wave maximum, one atomic per wave
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    const uint32_t o = __shfl_xor(best, d);
    best = best > o ? best : o;
  }
  if (lane == 0 && best)
    atomicMax((unsigned long long*)&a.counters[ARGUS_SC_N_ITERATIONS], (unsigned long long)best);
}

// Each bucket's pairs written to their instances: block k serves XCD k % 8
// (blocks are dispatched to XCDs round-robin), buckets b with b % 8 == k % 8,
// one of kOrdSlices slices of the bucket each.
__global__ __launch_bounds__(kScThreads) void k_sc_ord_place(ScopeArgs a) {
  const uint64_t n = sb_count(a.s);
  const uint32_t k = blockIdx.x, x = k % 8, j = k / 8;
  const uint64_t b = x + 8ull * (j / kOrdSlices);
  const uint32_t sl = j % kOrdSlices;
  const uint64_t b0 = b << kOrdBucketBits;
  if (b0 >= n) return;
  const uint64_t size = n - b0 < (1ull << kOrdBucketBits) ? n - b0 : (1ull << kOrdBucketBits);
  const uint64_t lo = b0 + size * sl / kOrdSlices, hi = b0 + size * (sl + 1) / kOrdSlices;
  for (uint64_t i = lo + threadIdx.x; i < hi; i += kScThreads) {
    const uint64_t pr = a.pairs[i];
    const uint32_t idx = (uint32_t)pr;
    if (idx >= b0 && idx < b0 + size) a.ordinal[idx] = (uint32_t)(pr >> 32);
    else sc_flag(a.counters, 1);
  }
}


// Inclusive maximum over the wave (unsigned; lanes past a row edge see 0).
__device__ __forceinline__ uint32_t wave_incl_max32(uint32_t v) {
  v = max(v, dpp32<kDppRowShr + 1>(v));
  v = max(v, dpp32<kDppRowShr + 2>(v));
  v = max(v, dpp32<kDppRowShr + 4>(v));
  v = max(v, dpp32<kDppRowShr + 8>(v));
  v = max(v, dpp32<kDppBcast15, 0xA>(v));
  v = max(v, dpp32<kDppBcast31, 0xC>(v));
  return v;
}

// Ordinals of one chunk of 4096 consecutive instances, exact except for the
// context that entered the chunk from earlier ones (those are written with
// kSoPending and completed in k_sc_stats), and, when the chunk's last
// context continues into the next chunk, that context's counts per region.
// One wave per chunk walks it in order, 64 elements per round.  An element's
// local ordinal is the count its (context, region) reached before the round,
// kept per region in the wave's LDS row, plus its rank among the lanes of
// the round with the same context and region (contexts are contiguous, so
// the lanes of one context form a range; the region by one ballot per
// region bit).  A counter keeps the chunk position where its context starts
// beside the count, so a context that starts inside the chunk counts from
// zero.  The loads of kSoBatch rounds are issued together.
constexpr int kSoBatch = 16;

__device__ __forceinline__ bool in_range32(uint64_t v, uint32_t lo, uint32_t hi) {
  return lo <= v && v <= hi;
}
// The context's part of a scope: warp role and group.
__device__ __forceinline__ bool in_scope_ctx(const argus_scope& sc, uint32_t ctx) {
  const uint64_t group = sc.group_shift >= 32 ? 0ull : (uint64_t)(ctx >> sc.group_shift);
  return in_range32(ctx & sc.role_mask, sc.role_lo, sc.role_hi) && in_range32(group, sc.group_lo, sc.group_hi);
}

template <bool MARK>
__global__ __launch_bounds__(kScThreads) void k_so_local(ScopeArgs a) {
  extern __shared__ uint32_t so_cnt[];  // [4 waves][R]: context start << 16 | count
  const uint64_t n = sb_count(a.s);
  const uint4* inst = reinterpret_cast<const uint4*>(a.inst);
  const uint32_t w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  uint32_t* cr = so_cnt + (uint64_t)w * a.R;
  const uint32_t rbits = a.R > 1 ? 32u - (uint32_t)__clz(a.R - 1) : 1u;
  const uint64_t lt = lanemask_lt();
  const uint64_t above = lane == 63 ? 0ull : (~0ull << (lane + 1));  // lanes after this one
  const uint64_t chunks = (n + kScTile - 1) / kScTile;
  bool bad = false;
  for (uint64_t c = (uint64_t)blockIdx.x * 4 + w; c < chunks; c += (uint64_t)gridDim.x * 4) {
    const uint64_t base = c * kScTile;
    const uint32_t cnt = n - base < (uint64_t)kScTile ? (uint32_t)(n - base) : kScTile;
    // the chunk's first and last contexts and their neighbours outside it
    const uint32_t F = inst[2 * base + 1].x, L = inst[2 * (base + cnt - 1) + 1].x;
    const uint32_t ctx_before = inst[2 * (base > 0 ? base - 1 : 0) + 1].x;
    const uint32_t ctx_after = inst[2 * (base + cnt < n ? base + cnt : base) + 1].x;
    uint32_t f = F == L ? kSoWhole : 0u;
    if (base > 0 && ctx_before == F) f |= kSoPcont;
    if (base + cnt < n && ctx_after == L) f |= kSoCont;
    uint32_t maybe = MARK ? 0u : 0xFFFFu;  // granules that may hold instances in scope
    for (uint32_t r = lane; r < a.R; r += 64) cr[r] = 0;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    uint32_t seg1 = 0;  // 1 + the context start of the element before the round
    uint32_t pctx = F;  // the context of that element (the first element starts one anyway)
    for (uint32_t b0 = 0; b0 < cnt; b0 += 64u * kSoBatch) {
      uint32_t cx[kSoBatch], rw[kSoBatch];
#pragma unroll
      for (int k = 0; k < kSoBatch; ++k) {
        const uint32_t e = b0 + 64u * k + lane;
        const uint4 h1 = inst[2 * (base + (e < cnt ? e : cnt - 1)) + 1];
        cx[k] = h1.x;
        rw[k] = h1.w;
      }
#pragma unroll
      for (int k = 0; k < kSoBatch; ++k) {
        const uint32_t r0 = b0 + 64u * k;  // the round's first element
        if (r0 < cnt) {
        const uint32_t e = r0 + lane;
        const bool in = e < cnt;
        const uint32_t ctx = cx[k], reg = rw[k] & 0xFFFFu;
        bad |= in && reg >= a.R;
        const bool ok = in && reg < a.R;
        const bool head = in && (e == 0 || lane_prev(ctx, pctx) != ctx);
        uint32_t x = wave_incl_max32(head ? e + 1 : 0u);
        x = x > seg1 ? x : seg1;
        const uint32_t seg = x - 1u;  // where this element's context starts in the chunk
        seg1 = (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
        pctx = (uint32_t)__builtin_amdgcn_readlane((int)ctx, 63);
        // the lanes of this context in the round, then those of this region
        const uint64_t nxt = __ballot(head) & above;
        const uint32_t hi = nxt ? (uint32_t)__builtin_ctzll(nxt) : 64u;
        const uint32_t lo = seg > r0 ? seg - r0 : 0u;
        uint64_t peers = __ballot(ok) & (hi == 64u ? ~0ull : ((1ull << hi) - 1ull)) & (~0ull << lo);
        for (uint32_t bit = 0; bit < rbits; ++bit) {
          const bool set = (reg >> bit) & 1u;
          const uint64_t bal = __ballot(set);
          peers &= set ? bal : ~bal;
        }
        const uint32_t rc = ok ? reg : 0u;
        const uint32_t ent = ok ? cr[rc] : 0u;
        const uint32_t prior = (ent >> 16) == seg ? (ent & 0xFFFFu) : 0u;
        const uint32_t local = ok ? prior + (uint32_t)__popcll(peers & lt) : 0u;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // the last lane of each (context, region) group carries its count on
        if (ok && (peers >> lane) == 1ull) cr[rc] = (seg << 16) | (prior + (uint32_t)__popcll(peers));
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // the chunk's first context starts at position 0
        const bool pending = ok && (f & kSoPcont) && seg == 0;
        if (in) a.ordinal[base + e] = pending ? (kSoPending | (reg << 12) | local) : local;
        if (MARK) {
          // (a pending ordinal only grows by its carry)
          const bool cand = ok && in_scope_ctx(a.sc, ctx) && local <= a.sc.iter_hi &&
                            (pending || local >= a.sc.iter_lo) && (!a.region_mask || a.region_mask[rc] != 0);
          if (__ballot(cand)) maybe |= 1u << (r0 / kSoGranule);
        }
        }
      }
    }
    if (lane == 0) {
      a.cflag[c] = f | (maybe << kSoMaskShift);
      a.cneed[c] = MARK ? 0u : 1u;
    }
    if (f & kSoCont) {
      // the last context's counts (its start: the last element's)
      const uint32_t ls = seg1 - 1u;
      uint32_t* tail = a.tail + c * (uint64_t)a.R;
      for (uint32_t r = lane; r < a.R; r += 64) {
        const uint32_t ent = cr[r];
        tail[r] = (ent >> 16) == ls ? (ent & 0xFFFFu) : 0u;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();  // the row is cleared for the next chunk after these reads
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  if (__ballot(bad) && lane == 0) sc_flag(a.counters, 2);  // regions must lie below num_regions
}

__device__ __forceinline__ uint64_t so_chunks(uint64_t n) { return (n + kScTile - 1) / kScTile; }

// The carry entering chunk c (per region): x_{c+1} = m_c x_c + b_c, with
// m_c = 1 when the chunk is one context that continues from the chunk before
// and into the next, b_c = the chunk's last-context counts when that context
// continues (else 0); x_0 = 0.  A three-phase scan: the composite of each
// segment of kSoSeg chunks, a sequential pass over the segments per region,
// then each segment's carries.
__global__ __launch_bounds__(kScThreads) void k_so_seg(ScopeArgs a) {
  const uint64_t chunks = so_chunks(sb_count(a.s));
  const uint64_t nseg = (chunks + kSoSeg - 1) / kSoSeg;
  const uint64_t i = (uint64_t)blockIdx.x * kScThreads + threadIdx.x;
  const uint64_t sg = i / a.R;
  const uint32_t r = (uint32_t)(i % a.R);
  if (sg >= nseg) return;
  uint32_t M = 1, B = 0;
  const uint64_t c1 = (sg + 1) * kSoSeg < chunks ? (sg + 1) * kSoSeg : chunks;
  // branch-free steps, eight chunks' loads at a time (a count slot of a chunk
  // whose last context ends in it holds no count and is not used)
  for (uint64_t c0 = sg * kSoSeg; c0 < c1; c0 += 8) {
    uint32_t f[8], t[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const uint64_t c = c0 + u;
      f[u] = c < c1 ? a.cflag[c] : kSoCont | kSoWhole | kSoPcont;
      t[u] = c < c1 ? a.tail[c * a.R + r] : 0u;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const uint32_t tv = (f[u] & kSoCont) ? t[u] : 0u;
      const bool keep = (f[u] & (kSoCont | kSoWhole | kSoPcont)) == (kSoCont | kSoWhole | kSoPcont);
      M = keep ? M : 0u;
      B = keep ? B + tv : tv;
    }
  }
  a.segb[sg * a.R + r] = B;
  if (r == 0) a.segm[sg] = M;
}

__global__ __launch_bounds__(kScThreads) void k_so_top(ScopeArgs a) {
  const uint64_t chunks = so_chunks(sb_count(a.s));
  const uint64_t nseg = (chunks + kSoSeg - 1) / kSoSeg;
  const uint32_t r = blockIdx.x * kScThreads + threadIdx.x;
  if (r >= a.R) return;
  uint32_t X = 0;
  for (uint64_t sg = 0; sg < nseg; ++sg) {
    const uint32_t B = a.segb[sg * a.R + r];
    a.segb[sg * a.R + r] = X;  // the carry entering the segment
    X = a.segm[sg] ? X + B : B;
  }
}

__global__ __launch_bounds__(kScThreads) void k_so_down(ScopeArgs a) {
  const uint64_t chunks = so_chunks(sb_count(a.s));
  const uint64_t nseg = (chunks + kSoSeg - 1) / kSoSeg;
  const uint64_t i = (uint64_t)blockIdx.x * kScThreads + threadIdx.x;
  const uint64_t sg = i / a.R;
  const uint32_t r = (uint32_t)(i % a.R);
  if (sg >= nseg) return;
  uint32_t x = a.segb[sg * a.R + r];
  const uint64_t c1 = (sg + 1) * kSoSeg < chunks ? (sg + 1) * kSoSeg : chunks;
  for (uint64_t c0 = sg * kSoSeg; c0 < c1; c0 += 8) {
    uint32_t f[8], t[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const uint64_t c = c0 + u;
      f[u] = c < c1 ? a.cflag[c] : 0u;
      t[u] = c < c1 ? a.tail[c * a.R + r] : 0u;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const uint64_t c = c0 + u;
      if (f[u] & kSoPcont) a.tail[c * a.R + r] = x;  // the carry entering chunk c
      const uint32_t tv = (f[u] & kSoCont) ? t[u] : 0u;
      const bool keep = (f[u] & (kSoCont | kSoWhole | kSoPcont)) == (kSoCont | kSoWhole | kSoPcont);
      // the region's ordinals in a chunk inside one context: [x, x + tv)
      if (keep && tv && x <= a.sc.iter_hi && x + tv > a.sc.iter_lo) a.cneed[c] = 1;
      x = keep ? x + tv : tv;
    }
  }
}

// Scoped statistics in canonical order.  With LDS_ROWS, each block keeps
// the twelve scalar columns of every region in LDS (LDS atomics), and adds
// them to the output once at the end; without, every column goes straight
// to the output with global atomics.  The histograms are counted afterwards
// from the keys of the matched instances in scope (k_sc_hist).
//
// A wave takes granules of 256 instances.  The ordinal pass has marked the
// granules that may hold instances in scope (and the carry scan the chunks
// inside one context whose ordinals reach the iteration window); elsewhere
// only the ordinals are completed, from the 4-byte words that hold what is
// needed for it, and the 32-byte instances are not read: 0.68 -> 0.38 ms on 67 M
// instances (iterations 0..15 of half the groups).
constexpr uint32_t kScLdsRegions = 1024;  // 12 x 8 B x 1024 = 96 KiB of LDS
constexpr int kScStatThreads = 1024;
constexpr int kScCols = 12;               // ARGUS_RS_COUNT .. ARGUS_RS_SELF_NESTED
constexpr uint32_t kScHistLds = 150 * 1024;

struct ScCounts {
  uint32_t in, m, mm, u, s, best;
};

// Adds one instance in scope (h0, h1: its halves; ex: its exclusive time;
// preg: its parent's region) to the statistics; its histogram key, or none.
template <class ColPtr>
__device__ __forceinline__ uint32_t sc_add(const ScopeArgs& a, const uint4& h0, const uint4& h1, uint64_t ex,
                                           uint32_t preg, ScCounts& c, ColPtr col_ptr) {
  const uint32_t reg = h1.w & 0xFFFFu, ereg = h1.w >> 16;
  c.in += 1;
  if (ereg == kNoEnd) {
    c.u += 1;
    atomicAdd(col_ptr(reg, ARGUS_RS_UNCLOSED), 1ull);
    return 0xFFFFFFFFu;
  }
  if (ereg != reg) {
    c.mm += 1;
    atomicAdd(col_ptr(reg, ARGUS_RS_MISM_AS_BEGIN), 1ull);
    if (ereg < a.R) atomicAdd(col_ptr(ereg, ARGUS_RS_MISM_AS_END), 1ull);
    return 0xFFFFFFFFu;
  }
  c.m += 1;
  const uint64_t tb = (uint64_t)h0.x | ((uint64_t)h0.y << 32), te = (uint64_t)h0.z | ((uint64_t)h0.w << 32);
  const uint64_t d = te - tb;
  atomicAdd(col_ptr(reg, ARGUS_RS_COUNT), 1ull);
  atomicAdd(col_ptr(reg, ARGUS_RS_INCL_SUM), (unsigned long long)d);
  atomicAdd(col_ptr(reg, ARGUS_RS_EXCL_SUM), (unsigned long long)ex);
  atomicMin(col_ptr(reg, ARGUS_RS_INCL_MIN), (unsigned long long)d);
  atomicMax(col_ptr(reg, ARGUS_RS_INCL_MAX), (unsigned long long)d);
  atomicMin(col_ptr(reg, ARGUS_RS_EXCL_MIN), (unsigned long long)ex);
  atomicMax(col_ptr(reg, ARGUS_RS_EXCL_MAX), (unsigned long long)ex);
  if (preg == reg) {
    c.s += 1;
    atomicAdd(col_ptr(reg, ARGUS_RS_SELF_NESTED), 1ull);
  }
  return (reg << 16) | (bit_width64(d) << 8) | bit_width64(ex);
}

// The counters, once per block (an atomic per wave on one counter takes 5 ns
// each, one after another).  Every thread of the block calls it.
__device__ __forceinline__ void sc_counters(const ScopeArgs& a, const ScCounts& c, uint64_t n) {
  __shared__ uint32_t s_cnt[6][kScStatThreads / 64];
  const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint32_t v[5] = {c.in, c.m, c.mm, c.u, c.s};
#pragma unroll
  for (int q = 0; q < 5; ++q) {
    const uint32_t t = rows_sum32(row_sum32(v[q]));
    if (lane == 0) s_cnt[q][w] = t;
  }
  uint32_t best = c.best;
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    const uint32_t o = __shfl_xor(best, d);
    best = best > o ? best : o;
  }
  if (lane == 0) s_cnt[5][w] = best;
  __syncthreads();
  if (threadIdx.x < 6) {
    constexpr int slot[6] = {ARGUS_SC_N_IN_SCOPE, ARGUS_SC_N_MATCHED,     ARGUS_SC_N_MISMATCHED,
                             ARGUS_SC_N_UNCLOSED, ARGUS_SC_N_SELF_NESTED, ARGUS_SC_N_ITERATIONS};
    unsigned long long t = 0;
    for (uint32_t q = 0; q < kScStatThreads / 64; ++q) {
      const uint32_t x = s_cnt[threadIdx.x][q];
      t = threadIdx.x < 5 ? t + x : (t > x ? t : x);
    }
    unsigned long long* dst = (unsigned long long*)&a.counters[slot[threadIdx.x]];
    if (t && threadIdx.x < 5) atomicAdd(dst, t);
    else if (t) atomicMax(dst, t);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) a.counters[ARGUS_SC_N_INSTANCES] = n;
}

template <bool LDS_ROWS>
__global__ __launch_bounds__(kScStatThreads) void k_sc_stats(ScopeArgs a) {
  extern __shared__ __align__(16) uint8_t sc_smem[];
  unsigned long long* srow = reinterpret_cast<unsigned long long*>(sc_smem);
  const uint64_t n = sb_count(a.s);
  const uint4* inst = reinterpret_cast<const uint4*>(a.inst);
  if (LDS_ROWS) {
    for (uint32_t i = threadIdx.x; i < a.R * kScCols; i += kScStatThreads) {
      const uint32_t col = i % kScCols;
      srow[i] = (col == ARGUS_RS_INCL_MIN || col == ARGUS_RS_EXCL_MIN) ? ~0ull : 0ull;
    }
    __syncthreads();
  }
  auto col_ptr = [&](uint32_t reg, uint32_t col) -> unsigned long long* {
    return LDS_ROWS ? &srow[(uint64_t)reg * kScCols + col]
                    : (unsigned long long*)(a.stats + (uint64_t)reg * ARGUS_RS_WIDTH + col);
  };
  ScCounts cc{};
  constexpr int IT = kSoGranule / 64;
  const uint32_t lane = threadIdx.x & 63;
  const uint64_t lt = lanemask_lt();
  const uint64_t granules = (n + kSoGranule - 1) / kSoGranule;
  const uint64_t step = (uint64_t)gridDim.x * (kScStatThreads / 64);
  // blocks take neighbouring granules in the same step, so that the chunks
  // that hold instances in scope spread over the chip
  uint64_t g = (uint64_t)(threadIdx.x >> 6) * gridDim.x + blockIdx.x;
  uint32_t pord[IT], pflag = 0, pneed = 0;
  auto issue = [&](uint64_t gi) {  // one granule ahead
    const uint64_t c = gi / (kScTile / kSoGranule);
    pflag = a.cflag[c];
    pneed = a.cneed[c];
#pragma unroll
    for (int j = 0; j < IT; ++j) {
      const uint64_t x = gi * kSoGranule + 64u * j + lane;
      pord[j] = a.ordinal[x < n ? x : n - 1];
    }
  };
  if (g < granules) issue(g);
  for (; g < granules; g += step) {
    const uint64_t x0 = g * kSoGranule + lane, c = g / (kScTile / kSoGranule);
    const uint32_t f = pflag, need_chunk = pneed;
    uint32_t ord[IT];
#pragma unroll
    for (int j = 0; j < IT; ++j) ord[j] = pord[j];
    constexpr uint32_t kInside = kSoCont | kSoWhole | kSoPcont;
    const bool need = ((f >> (kSoMaskShift + (uint32_t)(g % (kScTile / kSoGranule)))) & 1u) &&
                      ((f & kInside) != kInside || need_chunk);
    // chunk-local ordinals: add the carry of the context entering the chunk
    uint32_t carry[IT];
#pragma unroll
    for (int j = 0; j < IT; ++j)
      carry[j] = (ord[j] & kSoPending) ? a.tail[c * a.R + ((ord[j] >> 12) & 0xFFFu)] : 0u;
    uint4 h0[IT], h1[IT];
    if (need) {
#pragma unroll
      for (int j = 0; j < IT; ++j) {
        const uint64_t x = x0 + 64u * j;
        const uint64_t xc = x < n ? x : n - 1;
        h0[j] = inst[2 * xc];
        h1[j] = inst[2 * xc + 1];
      }
    }
    if (g + step < granules) issue(g + step);
#pragma unroll
    for (int j = 0; j < IT; ++j) {
      const uint64_t x = x0 + 64u * j;
      if (x < n) {
        if (ord[j] & kSoPending) {
          ord[j] = (ord[j] & 0xFFFu) + carry[j];
          a.ordinal[x] = ord[j];
        }
        cc.best = cc.best > ord[j] + 1 ? cc.best : ord[j] + 1;
      }
    }
    uint32_t keys = 0;
    if (need) {
      bool in[IT];
      uint64_t exv[IT];
      uint32_t preg[IT];
#pragma unroll
      for (int j = 0; j < IT; ++j) {
        const uint64_t x = x0 + 64u * j;
        const uint32_t reg = h1[j].w & 0xFFFFu, ereg = h1[j].w >> 16;
        in[j] = x < n && in_scope_ctx(a.sc, h1[j].x) && in_range32(ord[j], a.sc.iter_lo, a.sc.iter_hi) &&
                reg < a.R && (!a.region_mask || a.region_mask[reg] != 0);
        const bool mt = in[j] && ereg == reg;
        exv[j] = mt ? a.excl[x] : 0ull;
        const uint32_t par = h1[j].y;
        preg[j] = mt && par != kNoParent && par < n ? (inst[2 * (uint64_t)par + 1].w & 0xFFFFu)
                                                    : 0xFFFFFFFFu;
      }
#pragma unroll
      for (int j = 0; j < IT; ++j) {
        uint32_t hk = 0xFFFFFFFFu;
        if (in[j]) hk = sc_add(a, h0[j], h1[j], exv[j], preg[j], cc, col_ptr);
        const uint64_t m = __ballot(hk != 0xFFFFFFFFu);
        if (hk != 0xFFFFFFFFu) a.hkey[g * kSoGranule + keys + (uint32_t)__popcll(m & lt)] = hk;
        keys += (uint32_t)__popcll(m);
      }
    }
    if (lane == 0) a.gcnt[g] = (uint16_t)keys;
  }
  if (LDS_ROWS) {
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < a.R * kScCols; i += kScStatThreads) {
      const uint32_t col = i % kScCols, reg = i / kScCols;
      const unsigned long long v = srow[i];
      unsigned long long* dst = (unsigned long long*)(a.stats + (uint64_t)reg * ARGUS_RS_WIDTH + col);
      if (col == ARGUS_RS_INCL_MIN || col == ARGUS_RS_EXCL_MIN) {
        if (v != ~0ull) atomicMin(dst, v);
      } else if (col == ARGUS_RS_INCL_MAX || col == ARGUS_RS_EXCL_MAX) {
        if (v) atomicMax(dst, v);
      } else if (v) {
        atomicAdd(dst, v);
      }
    }
  }
  sc_counters(a, cc, n);
}

// The log2 histograms from the granules' keys: each block covers one slice of
// regions in LDS over one range of the granules (the slices of a range are 8
// blocks apart: on one XCD, whose L2 they share).  A wave takes up to 64
// granules at a time (fewer where there are not 64 for each: 2^15 instances
// took 28 us in the two waves that had any, 8 with one per wave) and,
// of those with keys, eight at once: a granule's keys are one 16-byte load per
// lane.
__global__ __launch_bounds__(kScStatThreads) void k_sc_hist(ScopeArgs a) {
  extern __shared__ __align__(16) uint8_t sc_smem[];
  uint32_t* s_h = reinterpret_cast<uint32_t*>(sc_smem);
  const uint32_t b = blockIdx.x, grp = b / (8 * a.hslices), rem = b % (8 * a.hslices);
  const uint32_t range = grp * 8 + rem % 8, r0 = rem / 8 * a.hslice;
  if (range >= a.hranges || r0 >= a.R) return;
  const uint32_t nr = (r0 + a.hslice < a.R ? r0 + a.hslice : a.R) - r0;
  for (uint32_t i = threadIdx.x; i < nr * 130; i += kScStatThreads) s_h[i] = 0;
  __syncthreads();
  const uint64_t granules = (sb_count(a.s) + kSoGranule - 1) / kSoGranule;
  const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  // four of a granule's n keys, those from 4 lane on
  auto add = [&](const uint4& v, uint32_t n) {
    const uint32_t k[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (uint32_t e = 0; e < 4; ++e) {
      const uint32_t r = k[e] >> 16;
      if (4 * lane + e >= n || r < r0 || r - r0 >= nr) continue;
      atomicAdd(&s_h[(r - r0) * 130 + ((k[e] >> 8) & 0xFFu)], 1u);
      atomicAdd(&s_h[(r - r0) * 130 + 65 + (k[e] & 0xFFu)], 1u);
    }
  };
  const uint4* keys = reinterpret_cast<const uint4*>(a.hkey);
  const uint64_t step = (uint64_t)a.hranges * (kScStatThreads / 64) * a.hper;
  for (uint64_t g0 = ((uint64_t)w * a.hranges + range) * a.hper; g0 < granules; g0 += step) {
    if (a.hper == 1) {
      // its keys and how many there are, together (the buffer goes on past the
      // last granule's keys; what lies there is not counted)
      const uint4 v = keys[g0 * (kSoGranule / 4) + lane];
      add(v, a.gcnt[g0]);
      continue;
    }
    const uint32_t cnt = lane < a.hper && g0 + lane < granules ? a.gcnt[g0 + lane] : 0u;
    uint64_t left = __ballot(cnt != 0);
    while (left) {
      uint4 v[8];
      uint32_t kn[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        kn[u] = 0;
        v[u] = make_uint4(0, 0, 0, 0);
        if (left) {
          const uint32_t q = (uint32_t)__builtin_ctzll(left);
          left &= left - 1;
          kn[u] = (uint32_t)__builtin_amdgcn_readlane((int)cnt, (int)q);
          if (4 * lane < kn[u]) v[u] = keys[(g0 + q) * (kSoGranule / 4) + lane];
        }
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) add(v[u], kn[u]);
    }
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < nr * 130; i += kScStatThreads) {
    const uint32_t h = s_h[i];
    if (h)
      atomicAdd((unsigned long long*)&a.stats[(uint64_t)(r0 + i / 130) * ARGUS_RS_WIDTH + ARGUS_RS_HIST_INCL + i % 130],
                (unsigned long long)h);
  }
}

// More than kSoMaxRegions regions: the ordinals are final, and every
// instance is read; one histogram key each.  (With the next
// instances loaded ahead and counters per wave the call took 530 us on 2^19
// instances of 20000 regions, this way 340.)
__global__ __launch_bounds__(kScStatThreads) void k_sc_stats_sorted(ScopeArgs a) {
  const uint64_t n = sb_count(a.s);
  const uint4* inst = reinterpret_cast<const uint4*>(a.inst);
  ScCounts cc{};
  auto col_ptr = [&](uint32_t reg, uint32_t col) -> unsigned long long* {
    return (unsigned long long*)(a.stats + (uint64_t)reg * ARGUS_RS_WIDTH + col);
  };
  for (uint64_t x = (uint64_t)blockIdx.x * kScStatThreads + threadIdx.x; x < n;
       x += (uint64_t)gridDim.x * kScStatThreads) {
    const uint4 h0 = inst[2 * x], h1 = inst[2 * x + 1];
    const uint32_t ord = a.ordinal[x], reg = h1.w & 0xFFFFu;
    uint32_t hk = 0xFFFFFFFFu;
    if (in_scope_ctx(a.sc, h1.x) && in_range32(ord, a.sc.iter_lo, a.sc.iter_hi) && reg < a.R &&
        (!a.region_mask || a.region_mask[reg] != 0)) {
      const bool mt = (h1.w >> 16) == reg;
      const uint64_t ex = mt ? a.excl[x] : 0ull;
      const uint32_t preg = mt && h1.y != kNoParent && h1.y < n ? (inst[2 * (uint64_t)h1.y + 1].w & 0xFFFFu)
                                                                : 0xFFFFFFFFu;
      hk = sc_add(a, h0, h1, ex, preg, cc, col_ptr);
    }
    a.hkey[x] = hk;
  }
  sc_counters(a, cc, n);
}

// ------------------------------------------------ probe <-> reference join
// Section 3.3: a probe's interval (the exposed latency of one operation at
// one iteration) is joined to the same operation's issue in the same
// iteration of the reference trace, by identity and scope rather than by
// timestamp: the joined instance is the iteration-th instance of the probe's
// context with the operation's region.  Joined probes are then sorted by
// (instance, latency), so each group is a run in latency order and its
// nearest-rank percentiles are read off by position.
//
// Up to kPrIndexRegions regions, an index of the reference is enough to find
// that instance: per tile of 4096 instances the places of each region's
// instances (one 16-bit list, in region order) and, per region, the count
// before each tile.  The instances are in context order, so those of a
// (context, region) are consecutive among the region's.  The index reads the
// upper half of every instance once and writes 2 bytes for it; sorting the
// instances by region, as is done for more regions, reads them twice and
// writes 16 (on 8.4 M instances 0.07 + 0.03 + 0.12 ms).

constexpr uint32_t kPrIndexRegions = 256;  // one counter per thread of a tile's block
constexpr uint32_t kPrJoinThreads = 512;
constexpr uint32_t kPrJoinBlocks = 2048;
constexpr uint32_t kPrTile = 1024;    // sorted probes per tile of k_pr_groups
constexpr uint32_t kPrDigits = 12;    // latency bytes 0..7, instance code bytes 0..3
constexpr uint32_t kPrPhGroups = kPrDigits;  // phase counters: one per sort pass, then the groups' tiles
constexpr uint32_t kPrCtrWords = kPhaseBase + (kPrDigits + 1) * kPhaseWords;

struct ProbeArgs {
  const argus_instance* inst;
  const uint4* probes;  // two uint4 per 32-byte probe
  uint64_t np;
  uint32_t R;
  uint64_t none;        // instance code of a probe that joined nothing (= max instances)
  SortBufs ref;         // R > kPrIndexRegions: the reference sorted by (region, context)
  int ref_buf;
  // the index of the reference; its counts [R][ref.tiles_max] are in ref.hist
  uint16_t* list;       // [tiles][4096] places in the tile, in region order
  uint16_t* lstart;     // [tiles][R] where each region starts in the tile's list
  uint32_t* tctx;       // [tiles] first context
  uint32_t* rtot;       // [R] instances of each region
  // the probes' sort: key = latency, ctxw = instance code
  RadixArgs r;
  uint32_t* dig;        // [kPrDigits][256] digit counts
  uint64_t* scan;       // [tiles of k_pr_groups] look-back words
  uint32_t* bcnt;       // [join blocks][4] bad, joined, unjoined
  uint32_t jblocks;
  uint32_t* ref_out;
  uint64_t* completion;
  uint64_t* groups;     // [np][ARGUS_PG_WIDTH]
  double* mean;
  uint64_t* counters;
};

__global__ __launch_bounds__(kScThreads) void k_pr_init(ProbeArgs a) {
  const uint64_t i0 = (uint64_t)blockIdx.x * kScThreads + threadIdx.x, stride = (uint64_t)gridDim.x * kScThreads;
  if (i0 < ARGUS_PR_NUM_COUNTERS) a.counters[i0] = 0;
  if (a.np == 0) return;
  if (i0 < 32) a.r.counters[i0] = 0;
  for (uint64_t i = i0; i < kPrDigits * kRadixBins; i += stride) a.dig[i] = 0;
  for (uint64_t i = i0; i < kPrCtrWords; i += stride) a.r.ctrs[i] = 0;
  for (uint64_t i = i0; i < ceil_div(a.np, kPrTile); i += stride) a.scan[i] = 0;
  for (uint64_t i = i0; i < ceil_div(a.np, kSortTile) * kRadixBins; i += stride) a.r.lb[i] = 0;
}

// One tile of the index: ranked like a radix pass on the region (each wave
// takes 1024 consecutive instances), the list staged in LDS.
__global__ __launch_bounds__(kScThreads) void k_pr_index(ProbeArgs a) {
  __shared__ uint32_t s_wave[4][256];
  __shared__ uint32_t s_lstart[256];
  __shared__ uint32_t s_w[kScThreads / 64];
  __shared__ uint32_t s_carry;
  __shared__ __align__(16) uint16_t s_list[kScTile];
  const uint64_t n = sb_count(a.ref), tile = blockIdx.x, base = tile * kScTile;
  if (base >= n) return;
  const uint32_t cnt = n - base < (uint64_t)kScTile ? (uint32_t)(n - base) : kScTile;
  const uint4* inst = reinterpret_cast<const uint4*>(a.inst);
  const uint32_t tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  uint32_t reg[kScRounds], rk[kScRounds];
  const uint32_t e0 = w * (kScRounds * 64) + lane;
#pragma unroll
  for (int r = 0; r < kScRounds; ++r) {
    const uint32_t e = e0 + (uint32_t)r * 64;
    const uint4 h1 = inst[2 * (base + (e < cnt ? e : cnt - 1)) + 1];
    reg[r] = h1.w & 0xFFFFu;
    if (r == 0 && tid == 0) a.tctx[tile] = h1.x;
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) s_wave[q][tid] = 0;
  if (tid == 0) s_carry = 0;
  __syncthreads();
  const uint32_t rbits = a.R > 1 ? 32u - (uint32_t)__clz(a.R - 1) : 1u;
  const uint64_t lt = lanemask_lt();
#pragma unroll
  for (int r = 0; r < kScRounds; ++r) {
    // an instance of another R (its region is not below this one) is in no list
    const bool valid = e0 + (uint32_t)r * 64 < cnt && reg[r] < a.R;
    const uint32_t d = valid ? reg[r] : 0u;
    uint64_t peers = __ballot(valid);
    for (uint32_t bit = 0; bit < rbits; ++bit) {
      const bool set = (d >> bit) & 1u;
      const uint64_t bal = __ballot(set);
      peers &= set ? bal : ~bal;
    }
    uint32_t rank = 0;
    if (valid) {
      const uint32_t old = s_wave[w][d];
      rank = old + (uint32_t)__popcll(peers & lt);
      __builtin_amdgcn_wave_barrier();
      if ((peers >> lane) == 1ull) s_wave[w][d] = old + (uint32_t)__popcll(peers);
    }
    __builtin_amdgcn_wave_barrier();
    rk[r] = valid ? rank : 0xFFFFFFFFu;
  }
  __syncthreads();
  uint32_t c = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t v = s_wave[q][tid];
    s_wave[q][tid] = c;
    c += v;
  }
  const uint32_t ls = block_excl_scan<kScThreads>(c, s_w, &s_carry);
  s_lstart[tid] = ls;
  if (tid < a.R) {
    a.ref.hist[(uint64_t)tid * a.ref.tiles_max + tile] = c;
    a.lstart[tile * a.R + tid] = (uint16_t)ls;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kScRounds; ++r)
    if (rk[r] != 0xFFFFFFFFu) s_list[s_lstart[reg[r]] + s_wave[w][reg[r]] + rk[r]] = (uint16_t)(e0 + (uint32_t)r * 64);
  __syncthreads();
  // (the list's end past the tile's valid instances, up to seven of a last
  // request, is never read)
  uint4* dst = reinterpret_cast<uint4*>(a.list + tile * kScTile);
  const uint4* src = reinterpret_cast<const uint4*>(s_list);
  for (uint32_t i = tid; i < (s_carry + 7) / 8; i += kScThreads) dst[i] = src[i];
}

// Per region (a block), its instances before each tile, in place of the
// tiles' counts, and its total.
__global__ __launch_bounds__(1024) void k_pr_rscan(ProbeArgs a) {
  __shared__ uint32_t s_carry;
  __shared__ uint32_t s_w[16];
  const uint64_t T = ceil_div(sb_count(a.ref), kScTile);
  uint32_t* row = a.ref.hist + (uint64_t)blockIdx.x * a.ref.tiles_max;
  if (threadIdx.x == 0) s_carry = 0;
  __syncthreads();
  for (uint64_t t0 = 0; t0 < T; t0 += 1024) {
    const uint64_t t = t0 + threadIdx.x;
    const uint32_t v = t < T ? row[t] : 0u;
    const uint32_t ex = block_excl_scan<1024>(v, s_w, &s_carry);
    if (t < T) row[t] = ex;
  }
  if (threadIdx.x == 0) a.rtot[blockIdx.x] = s_carry;
}

struct PrJoinShared {
  uint32_t hist[kPrDigits * kRadixBins];
  uint32_t cnt[kPrJoinThreads / 64][3];
};

// A probe's outputs and sort element (x: the joined instance, or a.none).
// Every lane with a probe of the wave calls it together.
__device__ __forceinline__ void pr_emit(const ProbeArgs& a, PrJoinShared& s, uint32_t nd_code, uint64_t j,
                                        uint64_t x, uint64_t lat_in) {
  const bool hit = x != a.none;
  const uint64_t lat = hit ? lat_in : 0ull;
  uint64_t done = kU64Max;
  if (hit) {
    const uint4 ib = reinterpret_cast<const uint4*>(a.inst)[2 * x];
    done = ((uint64_t)ib.x | ((uint64_t)ib.y << 32)) + lat;
  }
  a.ref_out[j] = hit ? (uint32_t)x : 0xFFFFFFFFu;
  a.completion[j] = done;
  a.r.key[0][j] = lat;
  a.r.ctxw[0][j] = (uint32_t)x;
  for (uint32_t d = 0; d < 8; ++d) hist_digit(s.hist + d * kRadixBins, (uint32_t)(lat >> (8 * d)) & 0xFFu, true);
  for (uint32_t d = 0; d < nd_code; ++d)
    hist_digit(s.hist + (8 + d) * kRadixBins, (uint32_t)(x >> (8 * d)) & 0xFFu, true);
}

// Bytes of the instance codes.
__device__ __forceinline__ uint32_t pr_code_digits(const ProbeArgs& a) { return (bit_width64(a.none | 1ull) + 7) / 8; }

__device__ __forceinline__ void pr_join_begin(PrJoinShared& s) {
  for (uint32_t i = threadIdx.x; i < kPrDigits * kRadixBins; i += kPrJoinThreads) s.hist[i] = 0;
  __syncthreads();
}

// The block's digit counts, and its probe counts (added up by k_pr_groups:
// an atomic per wave on one counter takes 5 ns each, one after another).
__device__ __forceinline__ void pr_join_end(const ProbeArgs& a, PrJoinShared& s, uint32_t bad, uint32_t joined,
                                            uint32_t unjoined) {
  const uint32_t v[3] = {bad, joined, unjoined};
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const uint32_t t = rows_sum32(row_sum32(v[q]));
    if ((threadIdx.x & 63) == 0) s.cnt[threadIdx.x >> 6][q] = t;
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < kPrDigits * kRadixBins; i += kPrJoinThreads)
    if (s.hist[i]) atomicAdd(&a.dig[i], s.hist[i]);
  if (threadIdx.x < 3) {
    uint32_t t = 0;
    for (uint32_t q = 0; q < kPrJoinThreads / 64; ++q) t += s.cnt[q][threadIdx.x];
    a.bcnt[4 * blockIdx.x + threadIdx.x] = t;
  }
}

// The join by the index: the context's first instance (a search over the
// tiles' first contexts, then within a tile), the region's instances before
// it, and from the target's number among the region's instances its tile and
// its place.  One probe per thread: the searches are short and mostly in the
// caches.
__global__ __launch_bounds__(kPrJoinThreads) void k_pr_join_index(ProbeArgs a) {
  __shared__ PrJoinShared s;
  pr_join_begin(s);
  const uint64_t n = sb_count(a.ref);
  const uint32_t T = (uint32_t)ceil_div(n, kScTile);
  const uint32_t* iw = reinterpret_cast<const uint32_t*>(a.inst);  // 8 words per instance; 4: context
  const uint32_t nd_code = pr_code_digits(a);
  uint32_t bad = 0, joined = 0, unjoined = 0;
  for (uint64_t j = (uint64_t)blockIdx.x * kPrJoinThreads + threadIdx.x; j < a.np;
       j += (uint64_t)gridDim.x * kPrJoinThreads) {
    const uint4 g0 = a.probes[2 * j], g1 = a.probes[2 * j + 1];
    const uint64_t ts = (uint64_t)g0.x | ((uint64_t)g0.y << 32), te = (uint64_t)g0.z | ((uint64_t)g0.w << 32);
    const uint32_t ctx = g1.x, it = g1.y, op = g1.z & 0xFFFFu;
    const bool ok = !(te < ts || op >= a.R);
    uint64_t x = a.none;
    if (ok && n) {
      uint32_t lo = 0, hi = T;  // first tile whose first context is not below ctx
      while (lo < hi) {
        const uint32_t m = (lo + hi) >> 1;
        if (a.tctx[m] < ctx) lo = m + 1;
        else hi = m;
      }
      const uint32_t t0 = lo > 0 ? lo - 1 : 0u;
      const uint64_t b0 = (uint64_t)t0 * kScTile;
      // the context's first instance lies in tile t0 or starts the next one
      uint32_t l0 = 0, l1 = lo > 0 ? (n - b0 < (uint64_t)kScTile ? (uint32_t)(n - b0) : kScTile) : 0u;
      while (l0 < l1) {
        const uint32_t m = (l0 + l1) >> 1;
        if (iw[8 * (b0 + m) + 4] < ctx) l0 = m + 1;
        else l1 = m;
      }
      // the region's instances before it
      const uint32_t* row = a.ref.hist + (uint64_t)op * a.ref.tiles_max;
      const uint32_t tot = a.rtot[op], c0 = row[t0], c1 = t0 + 1 < T ? row[t0 + 1] : tot;
      const uint16_t* ll = a.list + b0 + a.lstart[(uint64_t)t0 * a.R + op];
      uint32_t k0 = 0, k1 = c1 - c0;
      while (k0 < k1) {
        const uint32_t m = (k0 + k1) >> 1;
        if (ll[m] < l0) k0 = m + 1;
        else k1 = m;
      }
      const uint64_t target = (uint64_t)c0 + k0 + it;
      if (target < tot) {
        // the last tile with at most `target` before it, galloping from t0
        uint64_t a0 = t0, a1 = (uint64_t)t0 + 1, step = 1;
        while (a1 < T && row[a1] <= target) {
          a0 = a1;
          step *= 2;
          a1 = a0 + step;
        }
        if (a1 > T) a1 = T;
        while (a0 + 1 < a1) {
          const uint64_t m = (a0 + a1) >> 1;
          if (row[m] <= target) a0 = m;
          else a1 = m;
        }
        const uint64_t at = a0 * kScTile + a.lstart[a0 * a.R + op] + (uint32_t)(target - row[a0]);
        const uint64_t y = a0 * kScTile + a.list[at];
        if (iw[8 * y + 4] == ctx) x = y;
      }
    }
    bad += !ok;
    joined += ok && x != a.none;
    unjoined += ok && x == a.none;
    pr_emit(a, s, nd_code, j, x, te - ts);
  }
  pr_join_end(a, s, bad, joined, unjoined);
}

// The join by the sorted reference (more than kPrIndexRegions regions): for
// (operation region, context) a run, found by a binary search, in which the
// iteration-th element is the joined instance.
__global__ __launch_bounds__(kPrJoinThreads) void k_pr_join(ProbeArgs a) {
  __shared__ PrJoinShared s;
  pr_join_begin(s);
  const uint64_t nref = sb_count(a.ref);
  const uint64_t* ra = a.ref.a[a.ref_buf];
  const uint64_t* rb = a.ref.b[a.ref_buf];
  const uint32_t nd_code = pr_code_digits(a);
  uint32_t bad = 0, joined = 0, unjoined = 0;
  // Two probes per thread (j and j + stride), their reference searches in
  // lockstep: each search is a chain of dependent loads, and two chains per
  // lane keep more in flight.
  const uint64_t stride = (uint64_t)gridDim.x * kPrJoinThreads;
  auto finish = [&](uint64_t j, uint64_t lat, uint32_t ctx, uint32_t op, bool ok, uint64_t tgt) {
    uint64_t x = a.none;
    if (ok && nref) {
      // both words of the target loaded together (index clamped)
      const uint64_t tc = tgt < nref ? tgt : nref - 1;
      const uint64_t av = ra[tc], bv = rb[tc];
      if ((tgt < nref) & (av == op) & ((uint32_t)(bv >> 32) == ctx)) x = (uint32_t)bv;
    }
    bad += !ok;
    joined += ok && x != a.none;
    unjoined += ok && x == a.none;
    pr_emit(a, s, nd_code, j, x, lat);
  };
  for (uint64_t j = (uint64_t)blockIdx.x * kPrJoinThreads + threadIdx.x; j < a.np; j += 2 * stride) {
    const uint64_t j1 = j + stride;
    const bool has1 = j1 < a.np;
    const uint4 g0 = a.probes[2 * j], g1 = a.probes[2 * j + 1];
    const uint4 q0 = a.probes[2 * (has1 ? j1 : j)], q1 = a.probes[2 * (has1 ? j1 : j) + 1];
    const uint64_t ts0 = (uint64_t)g0.x | ((uint64_t)g0.y << 32), te0 = (uint64_t)g0.z | ((uint64_t)g0.w << 32);
    const uint64_t ts1 = (uint64_t)q0.x | ((uint64_t)q0.y << 32), te1 = (uint64_t)q0.z | ((uint64_t)q0.w << 32);
    const uint32_t ctx0 = g1.x, it0 = g1.y, op0 = g1.z & 0xFFFFu;
    const uint32_t ctx1 = q1.x, it1 = q1.y, op1 = q1.z & 0xFFFFu;
    const bool ok0 = !(te0 < ts0 || op0 >= a.R), ok1 = has1 && !(te1 < ts1 || op1 >= a.R);
    uint64_t lo0 = 0, hi0 = ok0 ? nref : 0, lo1 = 0, hi1 = ok1 ? nref : 0;
    while ((lo0 < hi0) | (lo1 < hi1)) {
      const bool c0 = lo0 < hi0, c1 = lo1 < hi1;
      const uint64_t m0 = (lo0 + hi0) >> 1, m1 = (lo1 + hi1) >> 1;
      const uint64_t r0 = c0 ? m0 : 0, r1 = c1 ? m1 : 0;  // a finished chain reads element 0
      const uint64_t am0 = ra[r0], am1 = ra[r1];
      const uint32_t cm0 = (uint32_t)(rb[r0] >> 32), cm1 = (uint32_t)(rb[r1] >> 32);
      const bool less0 = (am0 < op0) | ((am0 == op0) & (cm0 < ctx0));
      const bool less1 = (am1 < op1) | ((am1 == op1) & (cm1 < ctx1));
      if (c0) {
        if (less0) lo0 = m0 + 1;
        else hi0 = m0;
      }
      if (c1) {
        if (less1) lo1 = m1 + 1;
        else hi1 = m1;
      }
    }
    finish(j, te0 - ts0, ctx0, op0, ok0, lo0 + it0);
    if (has1) finish(j1, te1 - ts1, ctx1, op1, ok1, lo1 + it1);
  }
  pr_join_end(a, s, bad, joined, unjoined);
}

// The probes in (instance code, latency) order: stable passes over the
// latency's bytes and then the code's, those whose byte is the same for every
// probe left out, as phases of one kernel.  (A launch for each of three
// kernels per possible pass took 0.30 ms over 491,520 probes, most of it for
// passes with nothing to do.)  Which buffer holds the result goes to word 0
// of the flags.
__global__ __launch_bounds__(kSortThreads, 4) void k_pr_sort(ProbeArgs a) {
  __shared__ RadixShared s;
  KeySpace ks{};
  ks.ts_bits = 64;
  ks.wide = 1;
  uint32_t act = digits_varying<8>(a.dig, 8);
  act |= digits_varying<4>(a.dig + 8 * kRadixBins, 4) << 8;
  uint32_t src = 0;
  for (uint32_t d = 0; d < kPrDigits; ++d) {
    if (!((act >> d) & 1u)) continue;
    RadixPass ps;
    ps.src = src;
    ps.dst = src ^ 1u;
    ps.mode = d < 8 ? kDigKey : kDigCtx;
    ps.shift = 8 * (d & 7u);
    ps.tag = 1 + d;
    ps.n_out = (uint32_t)a.np;
    ps.n_elems = a.np;
    radix_offsets(s, a.dig + d * kRadixBins);
    bool fin;
    const uint32_t mine = radix_phase<3>(a.r, s, ks, ps, d, (act >> (d + 1)) == 0, &fin);
    src = ps.dst;
    // (the last pass only: an earlier one's block may come here late)
    if (fin && threadIdx.x == 0 && (act >> (d + 1)) == 0) a.r.counters[0] = src;
    if (!mine) return;
  }
}

// Tiles of 1024 sorted probes in order: the group heads (the number of the
// first from a look-back over the tiles), and for each its group's count,
// sum, issue time, mean and nearest-rank percentiles (its latencies are in
// increasing order).
__global__ __launch_bounds__(kScThreads) void k_pr_groups(ProbeArgs a) {
  __shared__ uint32_t s_slot, s_w[kScThreads / 64], s_ex;
  constexpr uint32_t kPer = kPrTile / kScThreads;
  const uint32_t buf = (uint32_t)a.r.counters[0];
  const uint64_t* la = a.r.key[buf];
  const uint32_t* code = a.r.ctxw[buf];
  const uint32_t tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const uint32_t tiles = (uint32_t)ceil_div(a.np, kPrTile), none = (uint32_t)a.none;
  const uint64_t lt = lanemask_lt();
  for (;;) {
    const uint32_t tile = phase_take(phase_ctr(a.r.ctrs, kPrPhGroups), &s_slot);
    if (tile >= tiles) break;
    const uint64_t k0 = (uint64_t)tile * kPrTile + w * (kPer * 64) + lane;
    uint32_t c[kPer];
    uint64_t hm[kPer];
    uint32_t heads = 0;
#pragma unroll
    for (uint32_t q = 0; q < kPer; ++q) {
      const uint64_t k = k0 + 64 * q;
      c[q] = k < a.np ? code[k] : none;
      const uint32_t before = k > 0 && k < a.np ? code[k - 1] : none;
      hm[q] = __ballot(c[q] != none && (k == 0 || before != c[q]));
      heads += (uint32_t)__popcll(hm[q]);
    }
    if (lane == 0) s_w[w] = heads;
    __syncthreads();
    uint32_t wpre = 0, total = 0;
#pragma unroll
    for (uint32_t q = 0; q < kScThreads / 64; ++q) {
      wpre += q < w ? s_w[q] : 0u;
      total += s_w[q];
    }
    if (w == 0) {
      const uint32_t ex = (uint32_t)scan_lookback(a.scan, tile, total, &a.r.counters[31], 2048);
      if (lane == 0) s_ex = ex;
    }
    __syncthreads();
    uint64_t g = (uint64_t)s_ex + wpre;
    if (tile + 1 == tiles && tid == 0) {
      a.counters[ARGUS_PR_N_PROBES] = a.np;
      a.counters[ARGUS_PR_N_GROUPS] = (uint64_t)s_ex + total;
    }
#pragma unroll
    for (uint32_t q = 0; q < kPer; ++q) {
      const uint64_t k = k0 + 64 * q;
      if ((hm[q] >> lane) & 1u) {
        const uint32_t r = c[q];
        // end of the run: the first position whose code exceeds r, galloping
        uint64_t lo = k + 1, step = 1, hi = k + 2;
        while (hi <= a.np && code[hi - 1] == r) {
          lo = hi;
          step *= 2;
          hi = lo + step;
        }
        if (hi > a.np) hi = a.np + 1;
        while (lo + 1 < hi) {  // code[lo - 1] == r, code[hi - 1] != r (or past the end)
          const uint64_t m = (lo + hi) >> 1;
          if (code[m - 1] == r) lo = m;
          else hi = m;
        }
        const uint64_t cnt = lo - k;
        uint64_t sum = 0;
#pragma unroll 4
        for (uint64_t i = k; i < lo; ++i) sum += la[i];
        const uint64_t at = g + (uint32_t)__popcll(hm[q] & lt);
        uint64_t* row = a.groups + at * ARGUS_PG_WIDTH;
        row[ARGUS_PG_INSTANCE] = r;
        row[ARGUS_PG_COUNT] = cnt;
        row[ARGUS_PG_SUM] = sum;
        const uint4 ib = reinterpret_cast<const uint4*>(a.inst)[2 * (uint64_t)r];
        row[ARGUS_PG_ISSUE] = (uint64_t)ib.x | ((uint64_t)ib.y << 32);
        const uint32_t pq[6] = {0, 20, 40, 60, 80, 100};
#pragma unroll
        for (int t = 0; t < 6; ++t) {
          uint64_t rank = ((uint64_t)pq[t] * cnt + 99) / 100;
          if (rank < 1) rank = 1;
          row[ARGUS_PG_P0 + t] = la[k + rank - 1];
        }
        a.mean[at] = (double)sum / (double)cnt;
      }
      g += (uint32_t)__popcll(hm[q]);
    }
    if (tile == 0 && w < 3) {
      // the join blocks' counts
      uint64_t t = 0;
      for (uint32_t b = lane; b < a.jblocks; b += 64) t += a.bcnt[4 * b + w];
      t = rows_sum64(row_sum64(t));
      if (lane == 0) a.counters[w == 0 ? ARGUS_PR_N_BAD : w == 1 ? ARGUS_PR_N_JOINED : ARGUS_PR_N_UNJOINED] = t;
    }
  }
  // (a wait that gave up, which does not happen, shows in the last counter)
  if (blockIdx.x == 0 && tid == 0) {
    const uint64_t e = ld_agent(&a.r.counters[31]);
    if (e) a.counters[ARGUS_PR_NUM_COUNTERS - 1] = e;
  }
}

// ------------------------------------------------------------ phase handoffs
// Section 4.2: the time between successive cooperative phases of a
// persistent kernel is a quantity of its own.  Phases are the instances of
// one level L; y follows x when it is the next level-L child of the same
// parent (for L = 0, the next top-level instance of the context).  Between
// two such siblings lie only descendants of the first, so after compacting
// the instances of level <= L (in canonical order), a phase's predecessor is
// simply the element before it, when that one has level L, the same context
// and the same parent.

constexpr uint32_t kHoMaxCompact = 4096;  // compaction blocks
constexpr uint32_t kHoThreads = 1024;
// Instances per compaction tile of NT threads, and up to which capacity of the
// instance buffer the compaction has 256 threads: tiles of 1024 threads are
// faster (33 M instances 0.31 -> 0.27 ms), but while they are fewer than 96,
// many compute units have none (whole calls, decode, level 1, buffers half
// full, with tiles of 4096 and of 16384: capacity 2^16 34 and 41 us, 2^20 53 and
// 58, 2^21 67 and 65, 2^22 92 and 81).
constexpr uint32_t ho_tile(uint32_t nt) { return nt * kScRounds; }
constexpr uint64_t kHoSmall = 3ull << 19;

struct HandoffArgs {
  const argus_instance* inst;
  const uint64_t* n_inst;
  uint64_t max_inst;
  uint32_t R, L;
  uint32_t* comp;    // instances of level <= L in canonical order
  uint64_t* status;  // [tiles] look-back words of the compaction (count, flags)
  uint32_t* tctr;    // tile counter of the compaction
  uint32_t* atl;     // [compaction blocks] instances of level L each saw, where pair block 0 later
                     // dumps (it has added them up by then)
  uint32_t cblocks;  // compaction blocks launched
  uint64_t* mtot;    // instances compacted
  uint64_t* pairs;  // [R][R][4]: count, sum, min, max (the output)
  uint32_t* dkey;   // [dumps][kHoSlots]: each pair block's hash table keys (0: empty)
  uint64_t* dval;   // [dumps][kHoSlots][4]: and its count, sum, min, max
  uint32_t dumps;   // pair blocks launched
  uint64_t* hist;   // [65]
  uint64_t* parent_gap;  // [max_inst] or NULL
  uint64_t* counters;
};

__device__ __forceinline__ uint64_t ho_count(const HandoffArgs& a) {
  const uint64_t v = *a.n_inst;
  return v < a.max_inst ? v : a.max_inst;
}

__global__ __launch_bounds__(kScThreads) void k_ho_init(HandoffArgs a) {
  const uint64_t stride = (uint64_t)gridDim.x * kScThreads;
  const uint64_t first = (uint64_t)blockIdx.x * kScThreads + threadIdx.x;
  const uint64_t np = (uint64_t)a.R * a.R * 4;
  for (uint64_t i = first; i < np; i += stride) a.pairs[i] = (i & 3) == 2 ? kU64Max : 0ull;
  if (a.parent_gap)
    for (uint64_t i = first; i < a.max_inst; i += stride) a.parent_gap[i] = 0;
  if (first < 65) a.hist[first] = 0;
  if (first < ARGUS_HO_NUM_COUNTERS) a.counters[first] = 0;
  const uint64_t tiles = ceil_div(a.max_inst, ho_tile(kScThreads));  // (of either size at most)
  for (uint64_t i = first; i < tiles; i += stride) a.status[i] = 0;
  if (first == 0) {
    *a.tctr = 0;
    *a.mtot = 0;
  }
}

// The instances of level <= L compacted in canonical order, in one pass:
// blocks take tiles of 4096 or 16384 instances in order (a counter; a block takes its
// next tile once this one's loads are on their way, so that the counter's
// round trip is hidden: nothing waits for a tile that comes after one still
// in work), count the tile's qualifying instances (a ballot per round of 64,
// the waves' counts through LDS), publish the count, find the count before
// the tile by decoupled look-back, 64 tiles a step, and write the indices.
// The tile holding the last instance records the total.
template <int NT>
__global__ __launch_bounds__(NT) void k_ho_compact(HandoffArgs a) {
  constexpr uint32_t kHoTile = ho_tile(NT);
  __shared__ uint32_t s_tile, s_w[NT / 64];
  __shared__ uint64_t s_base;
  const uint64_t n = ho_count(a);
  const uint64_t T = (n + kHoTile - 1) / kHoTile;
  const uint32_t* iw = reinterpret_cast<const uint32_t*>(a.inst);  // 8 words per instance
  const uint32_t tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const uint64_t lt = lanemask_lt();
  uint32_t at = 0;
  uint32_t nxt = 0;  // (thread 0) the block's next tile
  if (tid == 0) nxt = atomicAdd(a.tctr, 1u);
  for (;;) {
    if (tid == 0) s_tile = nxt;
    __syncthreads();
    const uint64_t tile = s_tile;
    if (tile >= T) break;
    const uint64_t base = tile * kHoTile;
    uint64_t qm[kScRounds];  // ballot of the qualifying lanes of each round
    uint32_t lv[kScRounds];
    // all the tile's loads issued before the first is used (indices clamped
    // to the last instance, n >= 1 here, instead of a branch per load)
#pragma unroll
    for (int r = 0; r < kScRounds; ++r) {
      const uint64_t x = base + w * (kScRounds * 64) + (uint32_t)r * 64 + lane;
      lv[r] = iw[8 * (x < n ? x : n - 1) + 6];
    }
    if (tid == 0) nxt = atomicAdd(a.tctr, 1u);
    uint32_t wc = 0;
#pragma unroll
    for (int r = 0; r < kScRounds; ++r) {
      const uint64_t x = base + w * (kScRounds * 64) + (uint32_t)r * 64 + lane;
      const bool in = x < n;
      const uint32_t lvl = lv[r];
      at += in && lvl == a.L;
      qm[r] = __ballot(in && lvl <= a.L);
      wc += (uint32_t)__popcll(qm[r]);
    }
    if (lane == 0) s_w[w] = wc;
    __syncthreads();
    uint32_t wpre = 0, cnt = 0;
#pragma unroll
    for (int q = 0; q < NT / 64; ++q) {
      wpre += q < (int)w ? s_w[q] : 0u;
      cnt += s_w[q];
    }
    if (w == 0) {
      const uint64_t excl = scan_lookback(a.status, (uint32_t)tile, cnt, &a.counters[ARGUS_HO_INTERNAL], 1);
      if (lane == 0) {
        s_base = excl;
        if (tile == T - 1) *a.mtot = excl + cnt;
      }
    }
    __syncthreads();
    uint64_t o = s_base + wpre;
#pragma unroll
    for (int r = 0; r < kScRounds; ++r) {
      if ((qm[r] >> lane) & 1u)
        a.comp[o + (uint32_t)__popcll(qm[r] & lt)] =
            (uint32_t)(base + w * (kScRounds * 64) + (uint32_t)r * 64 + lane);
      o += (uint32_t)__popcll(qm[r]);
    }
  }
  // the block's instances of level L, added up by k_ho_pairs (an atomic per
  // wave on one counter takes 5 ns each, one after another)
  __syncthreads();
  const uint32_t tot = rows_sum32(row_sum32(at));
  if (lane == 0) s_w[w] = tot;
  __syncthreads();
  if (tid == 0) {
    uint32_t t = 0;
    for (uint32_t q = 0; q < NT / 64; ++q) t += s_w[q];
    a.atl[blockIdx.x] = t;
  }
}

// Successive pairs, aggregated per block in an LDS hash table of (x region,
// y region) keys (linear probing from the key's home slot, keys claimed with a
// compare-and-swap): count, sum, min and max by LDS atomics.  At the end each
// block stores its table, keys and values, into its own dump with plain
// stores; k_ho_merge adds the dumps up.  A pair whose key finds no slot goes
// to the output row directly, by global atomics (such a key is never in the
// table: every insertion of a key probes the same slots from its home).  One
// block of 1024 threads per compute unit holds 4096 keys in 144 KiB of LDS.
// The histogram is in LDS, added once per block.  The loop runs in steps of
// one wave over 64 consecutive pairs, so that the histogram and the
// per-parent sums are combined across the wave first: one LDS add per
// distinct bit width and one global add per run of lanes with the same parent
// (the phases of one parent step are consecutive, so a wave holds one or two
// parents, where an add per lane would queue 64 atomics on one address).
constexpr uint32_t kHoSlots = 4096;
constexpr int kHoProbes = 16;
constexpr uint32_t kHoHashShift = 20;  // 32 - log2(kHoSlots)
constexpr uint32_t kHoMaxDumps = 256;  // pair blocks at most: one per compute unit
static_assert(sizeof(uint32_t) * kHoMaxCompact <= sizeof(uint64_t) * 4 * kHoSlots, "level counts lie in one dump");

__device__ __forceinline__ uint32_t ho_hash(uint32_t key) { return key * 2654435761u; }

__global__ __launch_bounds__(kHoThreads) void k_ho_pairs(HandoffArgs a) {
  __shared__ unsigned long long s_hist[65];
  __shared__ uint32_t s_key[kHoSlots];                // 1 + rx * R + ry; 0: empty
  __shared__ unsigned long long s_v[4][kHoSlots];      // count, sum, min, max
  for (int i = threadIdx.x; i < 65; i += kHoThreads) s_hist[i] = 0;
  for (uint32_t i = threadIdx.x; i < kHoSlots; i += kHoThreads) {
    s_key[i] = 0;
    s_v[0][i] = 0;
    s_v[1][i] = 0;
    s_v[2][i] = ~0ull;
    s_v[3][i] = 0;
  }
  __syncthreads();
  const uint64_t n = ho_count(a);
  const uint4* inst = reinterpret_cast<const uint4*>(a.inst);
  const uint64_t m = *a.mtot;
  const uint32_t lane = threadIdx.x & 63;
  uint64_t gaps = 0, gsum = 0;
  for (uint64_t k0 = (uint64_t)blockIdx.x * kHoThreads + (threadIdx.x & ~63u); k0 + 1 < m;
       k0 += (uint64_t)gridDim.x * kHoThreads) {
    const uint64_t k = k0 + lane;
    bool ok = k + 1 < m;
    uint64_t gap = 0;
    uint32_t par = kNoParent;
    if (ok) {
      const uint64_t x = a.comp[k], y = a.comp[k + 1];
      // both instances loaded together (y is at level L for nearly every
      // pair), not x after y's test
      const uint4 ya = inst[2 * y], yb = inst[2 * y + 1];
      const uint4 xa = inst[2 * x], xb = inst[2 * x + 1];
      asm volatile("" ::"v"(yb.z), "v"(xb.z));
      ok = yb.z == a.L;
      if (ok) {
        const uint32_t rx = xb.w & 0xFFFFu, ry = yb.w & 0xFFFFu;
        ok = xb.z == a.L && xb.x == yb.x && xb.y == yb.y &&  // level, context, parent
             (xb.w >> 16) != kNoEnd && rx < a.R && ry < a.R;
        if (ok) {
          const uint64_t te = (uint64_t)xa.z | ((uint64_t)xa.w << 32);
          const uint64_t tb = (uint64_t)ya.x | ((uint64_t)ya.y << 32);
          gap = tb - te;
          par = yb.y;
          const uint32_t key = 1u + rx * a.R + ry;
          uint32_t h = ho_hash(key) >> kHoHashShift;
          int slot = -1;
          for (int p = 0; p < kHoProbes; ++p) {
            const uint32_t cur = __hip_atomic_load(&s_key[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (cur == key) {
              slot = (int)h;
              break;
            }
            if (cur == 0) {
              const uint32_t prev = atomicCAS(&s_key[h], 0u, key);
              if (prev == 0u || prev == key) {
                slot = (int)h;
                break;
              }
            }
            h = (h + 1) & (kHoSlots - 1);
          }
          if (slot >= 0) {
            atomicAdd(&s_v[0][slot], 1ull);
            atomicAdd(&s_v[1][slot], (unsigned long long)gap);
            atomicMin(&s_v[2][slot], (unsigned long long)gap);
            atomicMax(&s_v[3][slot], (unsigned long long)gap);
          } else {
            unsigned long long* row = (unsigned long long*)(a.pairs + 4 * ((uint64_t)rx * a.R + ry));
            atomicAdd(&row[0], 1ull);
            atomicAdd(&row[1], (unsigned long long)gap);
            if (gap < __hip_atomic_load(&row[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
              atomicMin(&row[2], (unsigned long long)gap);
            if (gap > __hip_atomic_load(&row[3], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
              atomicMax(&row[3], (unsigned long long)gap);
          }
        }
      }
    }
    // histogram: one leader lane per distinct bit width adds the lanes that share it
    const uint32_t bin = ok ? bit_width64(gap) : 65u;
    for (uint64_t pend = __ballot(ok); pend;) {
      const uint32_t l = (uint32_t)__builtin_ctzll(pend);
      const uint32_t b = (uint32_t)__builtin_amdgcn_readlane((int)bin, (int)l);
      const uint64_t same = __ballot(bin == b);
      if (lane == l) atomicAdd(&s_hist[b], (unsigned long long)__popcll(same));
      pend &= ~same;
    }
    if (a.parent_gap) {
      // segmented inclusive scan over runs of equal parents (head flag, sum),
      // then the last lane of each run adds the run's sum
      const bool pc = ok && par != kNoParent && par < n;
      const uint32_t p = pc ? par : kNoParent;
      uint32_t f = lane_prev(p, ~p) != p;
      uint64_t v = pc ? gap : 0;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const uint64_t vu = __shfl_up(v, d);
        const uint32_t fu = __shfl_up(f, d);
        if (lane >= (uint32_t)d) {
          if (!f) v += vu;
          f |= fu;
        }
      }
      const uint32_t pn = __shfl_down(p, 1);
      if (pc && (lane == 63 || pn != p))
        atomicAdd((unsigned long long*)&a.parent_gap[p], (unsigned long long)v);
    }
    gaps += ok ? 1 : 0;
    gsum += gap;
  }
  // the counters once per block, not per wave; block 0 adds up the
  // compaction's counts of level L
  __shared__ uint64_t s_red[3][kHoThreads / 64];
  uint64_t atl = 0;
  if (blockIdx.x == 0)
    for (uint32_t b = threadIdx.x; b < a.cblocks; b += kHoThreads) atl += a.atl[b];
  const uint64_t g1 = rows_sum64(row_sum64(gaps)), g2 = rows_sum64(row_sum64(gsum)), g3 = rows_sum64(row_sum64(atl));
  if ((threadIdx.x & 63) == 0) {
    s_red[0][threadIdx.x >> 6] = g1;
    s_red[1][threadIdx.x >> 6] = g2;
    s_red[2][threadIdx.x >> 6] = g3;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    uint64_t v = 0;
    for (uint32_t q = 0; q < kHoThreads / 64; ++q) v += s_red[threadIdx.x][q];
    constexpr int slot[3] = {ARGUS_HO_N_GAPS, ARGUS_HO_GAP_SUM, ARGUS_HO_N_AT_LEVEL};
    if (v) atomicAdd((unsigned long long*)&a.counters[slot[threadIdx.x]], (unsigned long long)v);
  }
  for (int i = threadIdx.x; i < 65; i += kHoThreads)
    if (s_hist[i]) atomicAdd((unsigned long long*)&a.hist[i], s_hist[i]);
  uint32_t* dk = a.dkey + (uint64_t)blockIdx.x * kHoSlots;
  ulonglong2* dv = reinterpret_cast<ulonglong2*>(a.dval + (uint64_t)blockIdx.x * kHoSlots * 4);
  for (uint32_t i = threadIdx.x; i < kHoSlots; i += kHoThreads) {
    const uint32_t key = s_key[i];
    dk[i] = key;
    if (key) {
      dv[2 * i] = make_ulonglong2(s_v[0][i], s_v[1][i]);
      dv[2 * i + 1] = make_ulonglong2(s_v[2][i], s_v[3][i]);
    }
  }
}

// The dumps merged.  Block j owns the keys whose home slot lies in
// [j kHoSpan, (j + 1) kHoSpan): in every dump such a key sits less than
// kHoProbes slots after its home, so the block reads that window of each dump
// (kHoWin lanes per dump, several dumps at a time), adds the entries it owns
// in an LDS table and then into their output rows, which no other block
// writes (keys that overflowed there are never in a dump; keys that overflow
// the merge table are added with atomics).
constexpr uint32_t kHoSpan = 16;
constexpr uint32_t kHoWin = 32;  // lanes per dump: kHoSpan + kHoProbes - 1 of them read
constexpr uint32_t kMgSlots = 1024;
constexpr int kMgProbes = 16;
static_assert(kHoSpan + kHoProbes - 1 <= kHoWin && kHoSlots % kHoSpan == 0, "merge window");

__global__ __launch_bounds__(kScThreads) void k_ho_merge(HandoffArgs a) {
  __shared__ uint32_t s_key[kMgSlots];
  __shared__ unsigned long long s_v[4][kMgSlots];
  for (uint32_t i = threadIdx.x; i < kMgSlots; i += kScThreads) {
    s_key[i] = 0;
    s_v[0][i] = 0;
    s_v[1][i] = 0;
    s_v[2][i] = ~0ull;
    s_v[3][i] = 0;
  }
  __syncthreads();
  const uint32_t lo = blockIdx.x * kHoSpan;
  const uint32_t o = threadIdx.x % kHoWin;
  const uint32_t slot = (lo + o) & (kHoSlots - 1);
  if (o < kHoSpan + kHoProbes - 1) {
    for (uint32_t d = threadIdx.x / kHoWin; d < a.dumps; d += kScThreads / kHoWin) {
      const uint64_t e = (uint64_t)d * kHoSlots + slot;
      const uint32_t key = a.dkey[e];
      if (!key) continue;
      const uint32_t hk = ho_hash(key), home = hk >> kHoHashShift;
      if (home < lo || home >= lo + kHoSpan) continue;
      const ulonglong2* v = reinterpret_cast<const ulonglong2*>(a.dval + 4 * e);
      const ulonglong2 cs = v[0], mm = v[1];
      uint32_t h = (hk >> 10) & (kMgSlots - 1);  // the bits below the home slot's
      int at = -1;
      for (int p = 0; p < kMgProbes; ++p) {
        const uint32_t cur = __hip_atomic_load(&s_key[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (cur == key) {
          at = (int)h;
          break;
        }
        if (cur == 0) {
          const uint32_t prev = atomicCAS(&s_key[h], 0u, key);
          if (prev == 0u || prev == key) {
            at = (int)h;
            break;
          }
        }
        h = (h + 1) & (kMgSlots - 1);
      }
      if (at >= 0) {
        atomicAdd(&s_v[0][at], cs.x);
        atomicAdd(&s_v[1][at], cs.y);
        atomicMin(&s_v[2][at], mm.x);
        atomicMax(&s_v[3][at], mm.y);
      } else {
        unsigned long long* row = (unsigned long long*)(a.pairs + 4 * (uint64_t)(key - 1u));
        atomicAdd(&row[0], cs.x);
        atomicAdd(&row[1], cs.y);
        atomicMin(&row[2], mm.x);
        atomicMax(&row[3], mm.y);
      }
    }
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < kMgSlots; i += kScThreads) {
    const uint32_t key = s_key[i];
    if (!key) continue;
    uint64_t* row = a.pairs + 4 * (uint64_t)(key - 1u);
    row[0] += s_v[0][i];
    row[1] += s_v[1][i];
    row[2] = s_v[2][i] < row[2] ? s_v[2][i] : row[2];
    row[3] = s_v[3][i] > row[3] ? s_v[3][i] : row[3];
  }
}

}  // namespace argus

using namespace argus;

namespace {

constexpr size_t kScAlign = 256;
size_t sc_align(size_t v) { return (v + kScAlign - 1) & ~(kScAlign - 1); }

struct Carver {
  size_t o = 0;
  size_t take(size_t b) {
    const size_t at = o;
    o = sc_align(o + (b ? b : 1));
    return at;
  }
};

uint64_t tiles_for(uint64_t n) { return ((n ? n : 1) + kScTile - 1) / kScTile; }
uint64_t scan_blocks_for(uint64_t entries) { return (entries + kScScanBlock - 1) / kScScanBlock; }

// Workspace of one 16-byte-element sort of up to m elements (its buffers);
// the digit table and scan sums are shared and sized by the caller.
struct SortLayout {
  size_t a[2], b[2];
};
SortLayout carve_sort(Carver& c, uint64_t m) {
  SortLayout L{};
  const uint64_t mm = m ? m : 1;
  for (int k = 0; k < 2; ++k) {
    L.a[k] = c.take(sizeof(uint64_t) * mm);
    L.b[k] = c.take(sizeof(uint64_t) * mm);
  }
  return L;
}

struct ScLayout {
  SortLayout ref;
  size_t hist, bsum, octr, tail, cflag, segb, segm, total;
};
ScLayout sc_layout(uint64_t max_inst) {
  Carver c;
  ScLayout L{};
  L.ref = carve_sort(c, max_inst);
  L.hist = c.take(sizeof(uint32_t) * 256 * tiles_for(max_inst));
  L.bsum = c.take(sizeof(uint32_t) * scan_blocks_for(256 * tiles_for(max_inst)));
  L.octr = c.take(sizeof(uint32_t) * kOrdMaxBuckets);
  // chunk-local ordinals: per chunk (tile) and region up to kSoMaxRegions
  const uint64_t chunks = tiles_for(max_inst), segs = (chunks + kSoSeg - 1) / kSoSeg;
  L.tail = c.take(sizeof(uint32_t) * chunks * kSoMaxRegions);
  L.cflag = c.take(sizeof(uint32_t) * chunks);
  L.segb = c.take(sizeof(uint32_t) * segs * kSoMaxRegions);
  L.segm = c.take(sizeof(uint32_t) * segs);
  L.total = c.o;
  return L;
}

struct PrLayout {
  SortLayout ref;
  size_t hist, bsum, list, lstart, tctx, rtot, key[2], code[2], dig, lb, scan, ctrs, flag, bcnt, total;
};
PrLayout pr_layout(uint64_t max_inst, uint64_t np) {
  Carver c;
  PrLayout L{};
  const uint64_t tiles = tiles_for(max_inst), n = np ? np : 1;
  // the reference is sorted or indexed, as the regions go: the index lies
  // where the sort's buffers would
  Carver ix = c;
  L.ref = carve_sort(c, max_inst);
  L.list = ix.take(sizeof(uint16_t) * 8 * ceil_div(max_inst ? max_inst : 1, 8));
  L.lstart = ix.take(sizeof(uint16_t) * 256 * tiles);
  L.tctx = ix.take(sizeof(uint32_t) * tiles);
  L.rtot = ix.take(sizeof(uint32_t) * 256);
  c.o = std::max(c.o, ix.o);
  L.hist = c.take(sizeof(uint32_t) * 256 * tiles);
  L.bsum = c.take(sizeof(uint32_t) * scan_blocks_for(256 * tiles));
  for (int k = 0; k < 2; ++k) {
    L.key[k] = c.take(sizeof(uint64_t) * n);
    L.code[k] = c.take(sizeof(uint32_t) * n);
  }
  L.dig = c.take(sizeof(uint32_t) * kPrDigits * kRadixBins);
  L.lb = c.take(sizeof(uint64_t) * kRadixBins * ceil_div(n, kSortTile));
  L.scan = c.take(sizeof(uint64_t) * ceil_div(n, kPrTile));
  L.ctrs = c.take(sizeof(uint32_t) * kPrCtrWords);
  L.flag = c.take(sizeof(uint64_t) * 32);
  L.bcnt = c.take(sizeof(uint32_t) * 4 * kPrJoinBlocks);
  L.total = c.o;
  return L;
}

SortBufs make_bufs(char* base, const SortLayout& L, size_t hist, size_t bsum, uint64_t count_max,
                   const uint64_t* count_ptr, const argus_instance* inst) {
  SortBufs s{};
  for (int k = 0; k < 2; ++k) {
    s.a[k] = (uint64_t*)(base + L.a[k]);
    s.b[k] = (uint64_t*)(base + L.b[k]);
  }
  s.hist = (uint32_t*)(base + hist);
  s.bsum = (uint32_t*)(base + bsum);
  s.tiles_max = tiles_for(count_max);
  s.count_ptr = count_ptr;
  s.count_max = count_max;
  s.inst = inst;
  return s;
}

void scan_u32(uint32_t* data, uint64_t total, uint32_t* bsum, hipStream_t st) {
  if (total <= kScSmallMax) {
    hipLaunchKernelGGL(k_scan_small, dim3(1), dim3(1024), 0, st, data, total);
    return;
  }
  const uint32_t blocks = (uint32_t)scan_blocks_for(total ? total : 1);
  hipLaunchKernelGGL(k_scan_sums, dim3(blocks), dim3(kScThreads), 0, st, data, total, bsum);
  hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(1024), 0, st, bsum, blocks);
  hipLaunchKernelGGL(k_scan_apply, dim3(blocks), dim3(kScThreads), 0, st, data, total, bsum);
}

// One stable pass on digit (word, shift), reading buffer `in` (or the
// instances) and writing buffer `out`.
void sort_pass(const SortBufs& s, bool from_inst, int in, int out, int word, int shift,
               hipStream_t st) {
  const uint32_t tiles = (uint32_t)s.tiles_max;
  if (from_inst)
    hipLaunchKernelGGL(k_sort_hist<kSrcInst>, dim3(tiles), dim3(kScThreads), 0, st, s, in, word,
                       shift);
  else
    hipLaunchKernelGGL(k_sort_hist<kSrcBuf>, dim3(tiles), dim3(kScThreads), 0, st, s, in, word,
                       shift);
  scan_u32(s.hist, 256ull * s.tiles_max, s.bsum, st);
  if (from_inst)
    hipLaunchKernelGGL(k_sort_scatter<kSrcInst>, dim3(tiles), dim3(kScThreads), kScStageBytes, st, s,
                       in, out, word, shift);
  else
    hipLaunchKernelGGL(k_sort_scatter<kSrcBuf>, dim3(tiles), dim3(kScThreads), kScStageBytes, st, s,
                       in, out, word, shift);
}

// The instances sorted by (BEGIN region, context), canonical order kept
// within (more than 256 regions: two digits); returns the buffer holding the
// result.
int sort_reference(const SortBufs& s, hipStream_t st) {
  sort_pass(s, true, 0, 0, 0, 0, st);
  sort_pass(s, false, 0, 1, 0, 8, st);
  return 1;
}

std::mutex g_sc_mu;
int g_sc_dev_ok[64] = {};

int sc_check_device() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return ARGUS_E_HIP;
  if (dev < 0 || dev >= 64) return ARGUS_E_DEVICE;
  std::lock_guard<std::mutex> lock(g_sc_mu);
  if (!g_sc_dev_ok[dev]) {
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, dev) != hipSuccess) return ARGUS_E_HIP;
    if (strncmp(prop.gcnArchName, "gfx950", 6) != 0) return ARGUS_E_DEVICE;
    // the sort scatter stages a whole tile (64 KiB of dynamic LDS)
    for (const void* f : {(const void*)k_sort_scatter<kSrcInst>, (const void*)k_sort_scatter<kSrcBuf>})
      if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kScStageBytes) !=
          hipSuccess)
        return ARGUS_E_HIP;
    g_sc_dev_ok[dev] = 1;
  }
  return ARGUS_OK;
}

uint32_t sc_grid(uint64_t items, uint64_t per_block, uint32_t cap) {
  uint64_t g = (items + per_block - 1) / per_block;
  if (g > cap) g = cap;
  return g < 1 ? 1u : (uint32_t)g;
}

bool misaligned(const void* p, uintptr_t to) { return ((uintptr_t)p & (to - 1)) != 0; }

}  // namespace

extern "C" size_t argus_attr_scope_workspace_bytes(uint64_t max_instances) {
  if (max_instances >= (1ull << 31)) return 0;
  return sc_layout(max_instances).total;
}

extern "C" int argus_attr_scope(const argus_scope_config* cfg, const argus_scope_io* io,
                                void* d_workspace, size_t workspace_bytes, void* stream_v) {
  if (!cfg || !io) return ARGUS_E_INVAL;
  if (cfg->abi_version != ARGUS_ATTR_ABI_VERSION) return ARGUS_E_ABI;
  if (cfg->num_regions < 1 || cfg->num_regions > 65535) return ARGUS_E_INVAL;
  if (io->max_instances >= (1ull << 31)) return ARGUS_E_CAPACITY;
  if (!io->d_n_instances || !io->d_ordinal || !io->d_stats || !io->d_counters)
    return ARGUS_E_INVAL;
  if (io->max_instances > 0 && (!io->d_instances || !io->d_instance_excl)) return ARGUS_E_INVAL;
  if (!d_workspace) return ARGUS_E_INVAL;
  if (misaligned(io->d_instances, 16) || misaligned(io->d_instance_excl, 8) ||
      misaligned(io->d_n_instances, 8) || misaligned(io->d_ordinal, 4) ||
      misaligned(io->d_stats, 8) || misaligned(io->d_counters, 8) ||
      misaligned(d_workspace, kScAlign))
    return ARGUS_E_ALIGN;
  const ScLayout L = sc_layout(io->max_instances);
  if (workspace_bytes < L.total) return ARGUS_E_CAPACITY;
  const int dc = sc_check_device();
  if (dc != ARGUS_OK) return dc;

  char* base = (char*)d_workspace;
  ScopeArgs a{};
  a.inst = io->d_instances;
  a.excl = io->d_instance_excl;
  a.R = cfg->num_regions;
  a.sc = cfg->scope;
  a.region_mask = io->d_region_mask;
  a.ordinal = io->d_ordinal;
  a.stats = io->d_stats;
  a.counters = io->d_counters;
  a.s = make_bufs(base, L.ref, L.hist, L.bsum, io->max_instances, io->d_n_instances,
                  io->d_instances);
  a.octr = (uint32_t*)(base + L.octr);
  a.tail = (uint32_t*)(base + L.tail);
  a.cflag = (uint32_t*)(base + L.cflag);
  a.segb = (uint32_t*)(base + L.segb);
  a.segm = (uint32_t*)(base + L.segm);
  a.fast = a.R <= kSoMaxRegions ? 1u : 0u;
  hipStream_t st = (hipStream_t)stream_v;
  hipLaunchKernelGGL(k_sc_init, dim3(sc_grid((uint64_t)a.R * ARGUS_RS_WIDTH, kScThreads, 1024)),
                     dim3(kScThreads), 0, st, a);
  if (a.fast) {
    // the sort buffers are free
    a.hkey = reinterpret_cast<uint32_t*>(a.s.b[1]);
    a.gcnt = reinterpret_cast<uint16_t*>(a.s.a[1]);
    a.cneed = reinterpret_cast<uint32_t*>(a.s.a[0]);
    const uint64_t chunks = tiles_for(io->max_instances);
    const uint64_t segs = (chunks + kSoSeg - 1) / kSoSeg;
    // four chunks at a time per block (a wave each), each wave with its row
    // of R counters
    const size_t so_lds = (size_t)4 * a.R * sizeof(uint32_t);
    const bool mark = io->max_instances > kSoMarkMin;
    const void* local = mark ? (const void*)k_so_local<true> : (const void*)k_so_local<false>;
    (void)hipFuncSetAttribute(local, hipFuncAttributeMaxDynamicSharedMemorySize, (int)so_lds);
    void* largs[] = {&a};
    if (hipLaunchKernel(local, dim3((uint32_t)std::min<uint64_t>((chunks + 3) / 4, persistent_blocks(local, kScThreads))),
                        dim3(kScThreads), largs, so_lds, st) != hipSuccess)
      return ARGUS_E_HIP;
    const uint64_t cells = segs * a.R;
    hipLaunchKernelGGL(k_so_seg, dim3((uint32_t)((cells + kScThreads - 1) / kScThreads)),
                       dim3(kScThreads), 0, st, a);
    hipLaunchKernelGGL(k_so_top, dim3((a.R + kScThreads - 1) / kScThreads), dim3(kScThreads), 0, st, a);
    hipLaunchKernelGGL(k_so_down, dim3((uint32_t)((cells + kScThreads - 1) / kScThreads)),
                       dim3(kScThreads), 0, st, a);
  } else {
    const int buf = sort_reference(a.s, st);
    a.pairs = a.s.a[buf ^ 1];  // free once the sort is done
    hipLaunchKernelGGL(k_sc_ordinal, dim3(sc_grid(io->max_instances, kScTile, 2048)),
                       dim3(kScThreads), 0, st, a, buf);
    const uint64_t nbk = (io->max_instances + (1ull << kOrdBucketBits) - 1) >> kOrdBucketBits;
    const uint64_t blocks = 8ull * ((nbk + 7) / 8) * kOrdSlices;
    hipLaunchKernelGGL(k_sc_ord_place, dim3((uint32_t)(blocks ? blocks : 1)), dim3(kScThreads), 0, st, a);
    a.hkey = reinterpret_cast<uint32_t*>(a.s.b[buf ^ 1]);  // free once the sort is done
  }
  if (io->max_instances == 0) {
    // (no instance: the counters stand as k_sc_init left them)
    return hipGetLastError() == hipSuccess ? ARGUS_OK : ARGUS_E_HIP;
  }
  if (a.fast) {
    const uint64_t waves = (io->max_instances + kSoGranule - 1) / kSoGranule;
    const bool rows = a.R <= kScLdsRegions;
    const size_t lds = rows ? (size_t)a.R * kScCols * sizeof(uint64_t) : 0;
    const void* kern = rows ? (const void*)k_sc_stats<true> : (const void*)k_sc_stats<false>;
    if (rows) (void)hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    // the blocks that fit at once, a granule per wave: each flushes its rows
    // once.  While granules are few, fewer per block, so that their adds do not
    // queue in one compute unit (4096 instances, 3000 regions: one block 31 us,
    // one per granule 9.5); with rows, which each block flushes, up to four.
    const uint64_t fit = persistent_blocks(kern, kScStatThreads, lds);
    const uint32_t blocks = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(fit, !rows ? waves : std::max<uint64_t>((waves + 15) / 16, std::min<uint64_t>(4, (waves + 3) / 4))));
    if (rows) hipLaunchKernelGGL(k_sc_stats<true>, dim3(blocks), dim3(kScStatThreads), lds, st, a);
    else hipLaunchKernelGGL(k_sc_stats<false>, dim3(blocks), dim3(kScStatThreads), 0, st, a);
    // as few slices of regions as fit, of equal size
    const uint32_t slices = (uint32_t)ceil_div((uint64_t)a.R * 130 * sizeof(uint32_t), kScHistLds);
    a.hslice = (uint32_t)ceil_div(a.R, slices);
    a.hslices = slices;
    const size_t hb = (size_t)a.hslice * 130 * sizeof(uint32_t);
    (void)hipFuncSetAttribute((const void*)k_sc_hist, hipFuncAttributeMaxDynamicSharedMemorySize, (int)hb);
    // as many ranges as fit at once: each block clears and flushes its slice
    // once (256 ranges of 4 slices, four times the blocks that fit, took 141 us
    // where few granules have keys)
    const uint64_t hfit = ceil_div(persistent_blocks((const void*)k_sc_hist, kScStatThreads, hb), 8ull * slices) * 8;
    a.hranges = (uint32_t)std::min<uint64_t>(hfit, ceil_div(ceil_div(waves, 16 * 64), 8) * 8);
    a.hper = (uint32_t)std::min<uint64_t>(64, ceil_div(waves, (uint64_t)a.hranges * (kScStatThreads / 64)));
    hipLaunchKernelGGL(k_sc_hist, dim3(a.hranges * slices), dim3(kScStatThreads), hb, st, a);
  } else {
    hipLaunchKernelGGL(k_sc_stats_sorted, dim3(sc_grid(io->max_instances, kScStatThreads, 1024)),
                       dim3(kScStatThreads), 0, st, a);
    if (launch_hist_keys(a.hkey, io->d_n_instances, io->max_instances, a.stats, a.R, st) != hipSuccess)
      return ARGUS_E_HIP;
  }
  return hipGetLastError() == hipSuccess ? ARGUS_OK : ARGUS_E_HIP;
}

extern "C" size_t argus_attr_probes_workspace_bytes(uint64_t max_instances, uint64_t n_probes) {
  if (max_instances >= (1ull << 31) || n_probes >= (1ull << 31)) return 0;
  return pr_layout(max_instances, n_probes).total;
}

extern "C" int argus_attr_probes(const argus_probes_config* cfg, const argus_probes_io* io,
                                 void* d_workspace, size_t workspace_bytes, void* stream_v) {
  if (!cfg || !io) return ARGUS_E_INVAL;
  if (cfg->abi_version != ARGUS_ATTR_ABI_VERSION) return ARGUS_E_ABI;
  if (cfg->num_regions < 1 || cfg->num_regions > 65535) return ARGUS_E_INVAL;
  if (io->max_instances >= (1ull << 31) || io->n_probes >= (1ull << 31)) return ARGUS_E_CAPACITY;
  if (!io->d_n_instances || !io->d_counters) return ARGUS_E_INVAL;
  if (io->max_instances > 0 && !io->d_instances) return ARGUS_E_INVAL;
  if (io->n_probes > 0 && (!io->d_probes || !io->d_ref || !io->d_completion || !io->d_groups ||
                           !io->d_mean))
    return ARGUS_E_INVAL;
  if (!d_workspace) return ARGUS_E_INVAL;
  if (misaligned(io->d_instances, 16) || misaligned(io->d_probes, 16) ||
      misaligned(io->d_n_instances, 8) || misaligned(io->d_ref, 4) ||
      misaligned(io->d_completion, 8) || misaligned(io->d_groups, 8) ||
      misaligned(io->d_mean, 8) || misaligned(io->d_counters, 8) ||
      misaligned(d_workspace, kScAlign))
    return ARGUS_E_ALIGN;
  const PrLayout L = pr_layout(io->max_instances, io->n_probes);
  if (workspace_bytes < L.total) return ARGUS_E_CAPACITY;
  const int dc = sc_check_device();
  if (dc != ARGUS_OK) return dc;

  char* base = (char*)d_workspace;
  ProbeArgs a{};
  a.inst = io->d_instances;
  a.probes = reinterpret_cast<const uint4*>(io->d_probes);
  a.np = io->n_probes;
  a.R = cfg->num_regions;
  a.none = io->max_instances;
  a.ref = make_bufs(base, L.ref, L.hist, L.bsum, io->max_instances, io->d_n_instances,
                    io->d_instances);
  a.list = (uint16_t*)(base + L.list);
  a.lstart = (uint16_t*)(base + L.lstart);
  a.tctx = (uint32_t*)(base + L.tctx);
  a.rtot = (uint32_t*)(base + L.rtot);
  for (int k = 0; k < 2; ++k) {
    a.r.key[k] = (uint64_t*)(base + L.key[k]);
    a.r.ctxw[k] = (uint32_t*)(base + L.code[k]);
  }
  a.dig = (uint32_t*)(base + L.dig);
  a.r.lb = (uint64_t*)(base + L.lb);
  a.scan = (uint64_t*)(base + L.scan);
  a.r.ctrs = (uint32_t*)(base + L.ctrs);
  a.r.counters = (uint64_t*)(base + L.flag);
  a.bcnt = (uint32_t*)(base + L.bcnt);
  a.ref_out = io->d_ref;
  a.completion = io->d_completion;
  a.groups = io->d_groups;
  a.mean = io->d_mean;
  a.counters = io->d_counters;
  hipStream_t st = (hipStream_t)stream_v;
  const uint64_t clear = std::max<uint64_t>(ceil_div(a.np, kSortTile) * kRadixBins, kPrDigits * kRadixBins);
  hipLaunchKernelGGL(k_pr_init, dim3(sc_grid(clear, kScThreads, 2048)), dim3(kScThreads), 0, st, a);
  if (a.np > 0) {
    if (a.R <= kPrIndexRegions) {
      const uint32_t tiles = (uint32_t)a.ref.tiles_max;
      hipLaunchKernelGGL(k_pr_index, dim3(tiles), dim3(kScThreads), 0, st, a);
      hipLaunchKernelGGL(k_pr_rscan, dim3(a.R), dim3(1024), 0, st, a);
      a.jblocks = sc_grid(a.np, kPrJoinThreads, kPrJoinBlocks);
      hipLaunchKernelGGL(k_pr_join_index, dim3(a.jblocks), dim3(kPrJoinThreads), 0, st, a);
    } else {
      a.ref_buf = sort_reference(a.ref, st);
      a.jblocks = sc_grid(a.np, 2 * kPrJoinThreads, kPrJoinBlocks);  // two probes per thread
      hipLaunchKernelGGL(k_pr_join, dim3(a.jblocks), dim3(kPrJoinThreads), 0, st, a);
    }
    hipLaunchKernelGGL(k_pr_sort, dim3(sort_blocks((const void*)k_pr_sort, a.np)), dim3(kSortThreads), 0, st, a);
    hipLaunchKernelGGL(k_pr_groups, dim3(sc_grid(a.np, kPrTile, 2048)), dim3(kScThreads), 0, st, a);
  }
  return hipGetLastError() == hipSuccess ? ARGUS_OK : ARGUS_E_HIP;
}

namespace {

struct HoLayout {
  size_t comp, status, tctr, mtot, dkey, dval, total;
};
HoLayout ho_layout(uint64_t max_instances, uint32_t R) {
  Carver c;
  HoLayout L{};
  const uint64_t m = max_instances ? max_instances : 1;
  L.comp = c.take(sizeof(uint32_t) * m);
  L.status = c.take(sizeof(uint64_t) * tiles_for(m));
  L.tctr = c.take(sizeof(uint32_t));
  L.mtot = c.take(sizeof(uint64_t));
  L.dkey = c.take(sizeof(uint32_t) * (uint64_t)kHoMaxDumps * kHoSlots);
  L.dval = c.take(sizeof(uint64_t) * 4 * (uint64_t)kHoMaxDumps * kHoSlots);
  L.total = c.o;
  return L;
}

}  // namespace

extern "C" size_t argus_attr_handoffs_workspace_bytes(uint64_t max_instances,
                                                      uint32_t num_regions) {
  if (max_instances >= (1ull << 31) || num_regions < 1 || num_regions > 4096) return 0;
  return ho_layout(max_instances, num_regions).total;
}

extern "C" int argus_attr_handoffs(const argus_handoffs_config* cfg, const argus_handoffs_io* io,
                                   void* d_workspace, size_t workspace_bytes, void* stream_v) {
  if (!cfg || !io) return ARGUS_E_INVAL;
  if (cfg->abi_version != ARGUS_ATTR_ABI_VERSION) return ARGUS_E_ABI;
  if (cfg->num_regions < 1 || cfg->num_regions > 4096) return ARGUS_E_INVAL;
  if (io->max_instances >= (1ull << 31)) return ARGUS_E_CAPACITY;
  if (!io->d_n_instances || !io->d_pairs || !io->d_hist || !io->d_counters) return ARGUS_E_INVAL;
  if (io->max_instances > 0 && !io->d_instances) return ARGUS_E_INVAL;
  if (!d_workspace) return ARGUS_E_INVAL;
  if (misaligned(io->d_instances, 16) || misaligned(io->d_n_instances, 8) ||
      misaligned(io->d_pairs, 8) || misaligned(io->d_hist, 8) ||
      misaligned(io->d_parent_gap, 8) || misaligned(io->d_counters, 8) ||
      misaligned(d_workspace, kScAlign))
    return ARGUS_E_ALIGN;
  const HoLayout HL = ho_layout(io->max_instances, cfg->num_regions);
  if (workspace_bytes < HL.total) return ARGUS_E_CAPACITY;
  const int dc = sc_check_device();
  if (dc != ARGUS_OK) return dc;

  char* base = (char*)d_workspace;
  HandoffArgs a{};
  a.inst = io->d_instances;
  a.n_inst = io->d_n_instances;
  a.max_inst = io->max_instances;
  a.R = cfg->num_regions;
  a.L = cfg->level;
  a.comp = (uint32_t*)(base + HL.comp);
  a.status = (uint64_t*)(base + HL.status);
  a.tctr = (uint32_t*)(base + HL.tctr);
  a.mtot = (uint64_t*)(base + HL.mtot);
  a.dkey = (uint32_t*)(base + HL.dkey);
  a.dval = (uint64_t*)(base + HL.dval);
  a.atl = (uint32_t*)a.dval;
  a.pairs = io->d_pairs;
  a.hist = io->d_hist;
  a.parent_gap = io->d_parent_gap;
  a.counters = io->d_counters;
  hipStream_t st = (hipStream_t)stream_v;
  const uint64_t init_items =
      std::max<uint64_t>((uint64_t)a.R * a.R * 4, io->max_instances);
  hipLaunchKernelGGL(k_ho_init, dim3(sc_grid(std::max<uint64_t>(init_items, 65), kScThreads, 4096)),
                     dim3(kScThreads), 0, st, a);
  if (io->max_instances > 0) {
    const uint32_t g = sc_grid(io->max_instances, kScThreads, 4096);
    // resident blocks only: they take the tiles in order
    const bool small = io->max_instances <= kHoSmall;
    const void* compact = small ? (const void*)k_ho_compact<kScThreads> : (const void*)k_ho_compact<kHoThreads>;
    const uint32_t nt = small ? (uint32_t)kScThreads : kHoThreads;
    a.cblocks = (uint32_t)std::min<uint64_t>(
        std::min<uint64_t>(ceil_div(io->max_instances, ho_tile(nt)), persistent_blocks(compact, (int)nt)), kHoMaxCompact);
    void* cargs[] = {&a};
    if (hipLaunchKernel(compact, dim3(a.cblocks), dim3(nt), cargs, 0, st) != hipSuccess) return ARGUS_E_HIP;
    // resident blocks only (one per compute unit): each stores its table once
    a.dumps = (uint32_t)std::min<uint64_t>(
        std::min<uint64_t>(g, persistent_blocks((const void*)k_ho_pairs, kHoThreads)), kHoMaxDumps);
    hipLaunchKernelGGL(k_ho_pairs, dim3(a.dumps), dim3(kHoThreads), 0, st, a);
    hipLaunchKernelGGL(k_ho_merge, dim3(kHoSlots / kHoSpan), dim3(kScThreads), 0, st, a);
  }
  return hipGetLastError() == hipSuccess ? ARGUS_OK : ARGUS_E_HIP;
}
