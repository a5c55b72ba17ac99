// radix_tile.h -- one tile of one stable LSD radix pass over 8-bit digits.
//
// Stable sorting is how the records of every execution context are put in
// execution order before the per-context stack is replayed (the paper's
// Section 3.2 keeps a stack of open regions for each warp); the same
// pass orders the overlap events by (group, time) where they cannot be merged.
//
// Per tile of 4096 elements (8 waves x 8 rounds x 64 lanes; 16 waves per
// compute unit in two blocks, whose LDS fills it):
//   * rank: each wave finds, with eight ballots, the lanes holding the same
//     digit and counts them in per-wave LDS digit counters (stable order is
//     wave, round, lane = element order);
//   * the tile's 256 digit counts are published for decoupled look-back
//     (Merrill & Garland 2016) with tile ids taken in order from a ticket
//     counter, so every predecessor tile is already running;
//   * elements are staged in LDS in digit order and written out so that a
//     run of equal digits goes to consecutive addresses.
// A pass over a raw source (records or instances) drops invalid elements
// (they are never written) and packs the key.
#pragma once

#include "chain.h"

namespace argus {

// What a pass's digit is taken from.
enum : uint32_t {
  kDigCtx = 0,  // raw context (context offset + ctx_min) >> shift
  kDigKey = 1,  // packed key >> shift
};

struct RadixPass {
  uint32_t src;   // buffer 0/1, or 2: the raw source
  uint32_t dst;   // buffer 0/1
  uint32_t mode;  // kDigCtx / kDigKey
  uint32_t shift;
  uint32_t n_out;    // elements written (the destination's bound)
  uint32_t tag;      // 1..31, distinct for every pass that shares the look-back words
  uint64_t n_elems;  // elements read (a raw source's include the invalid ones)
};

// Look-back words of the radix passes: state in bits 62..63, the pass's tag
// in bits 40..44, the count below.  A word another pass left has another tag
// and reads as not published, so passes share one array without clearing it.
constexpr uint32_t kTagShift = 40;
ARGUS_DEV uint64_t radix_word(uint64_t flag, uint32_t tag, uint64_t v) {
  return flag | ((uint64_t)tag << kTagShift) | v;
}
ARGUS_DEV uint64_t radix_flag(uint64_t w, uint32_t tag) {
  return ((w >> kTagShift) & 31u) == tag ? (w & ~kValMask) : 0ull;
}
constexpr uint64_t kRadixVal = 0xFFFFFFFFull;

struct RadixShared {
  uint32_t ticket;
  uint32_t wave[kSortWaves][kRadixBins];  // per-wave counts, then their places in the staged tile
  uint32_t off[kRadixBins];      // global start of each digit
  uint32_t gbase[kRadixBins];    // global start of this tile's digit run, less its tile-local start
  uint32_t scr[kSortWaves];
  uint32_t total;
  __align__(16) uint64_t key[kSortTile];
  uint32_t pay[kSortTile];
  uint32_t cw[kSortTile];
};

struct RadixArgs {
  DevPlan* plan;
  const uint4* rec;
  const argus_instance* inst;
  const uint8_t* region_class;
  uint32_t R, K, G, shift;
  uint64_t* key[2];
  uint32_t* pay[2];
  uint32_t* ctxw[2];
  uint64_t* lb;         // look-back words, [tiles][256]
  uint32_t clear_lb;    // they are not zero yet
  uint32_t* ctrs;       // phase counters
  uint64_t* counters;
};

// Exclusive prefix sum over the threads of a sort block.
ARGUS_DEV uint32_t sort_excl_scan(uint32_t v, uint32_t* scratch, uint32_t* total) {
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const uint32_t x = (uint32_t)wave_incl_scan32((int32_t)v);
  if (lane == 63) scratch[w] = x;
  __syncthreads();
  uint32_t pre = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < kSortWaves; ++k) {
    const uint32_t c = scratch[k];
    pre += k < w ? c : 0u;
    tot += c;
  }
  __syncthreads();
  *total = tot;
  return pre + x - v;
}

// Adds this wave's digits (lanes in `valid`) to an LDS histogram: one atomic
// when every valid lane holds the same digit, else one per lane.
__device__ __forceinline__ void hist_digit(uint32_t* hist, uint32_t d, bool valid) {
  const uint64_t vm = __ballot(valid);
  if (vm == 0) return;
  const uint32_t first = (uint32_t)__builtin_ctzll(vm);
  const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)d, (int)first);
  if (__ballot(valid && d == d0) == vm) {
    if (lane_id() == first) atomicAdd(&hist[d0], (uint32_t)__popcll(vm));
  } else if (valid) {
    atomicAdd(&hist[d], 1u);
  }
}

// The digits (of N consecutive histograms, the first `nd`) that vary: more
// than one bin in use.  The same in every thread.
template <int N>
ARGUS_DEV uint32_t digits_varying(const uint32_t* hist, uint32_t nd) {
  const uint32_t t = threadIdx.x;
  uint32_t h[N], act = 0;
#pragma unroll
  for (int d = 0; d < N; ++d)
    h[d] = t < (uint32_t)kRadixBins && (uint32_t)d < nd ? ld_agent(&hist[d * kRadixBins + t]) : 0u;
#pragma unroll
  for (int d = 0; d < N; ++d)
    if ((uint32_t)d < nd && __syncthreads_count(h[d] != 0) > 1) act |= 1u << d;
  return act;
}

// The global digit starts of a pass from its histogram, into s.off.
ARGUS_DEV void radix_offsets(RadixShared& s, const uint32_t* hist) {
  const uint32_t t = threadIdx.x;
  uint32_t total;
  const uint32_t ex = sort_excl_scan(t < (uint32_t)kRadixBins ? ld_agent(&hist[t]) : 0u, s.scr, &total);
  if (t < (uint32_t)kRadixBins) s.off[t] = ex;
  __syncthreads();
}

// Clears the look-back words of sort tiles [r0, r1).
ARGUS_DEV void clear_rows(uint64_t* lb, uint64_t r0, uint64_t r1) {
  for (uint64_t i = r0 * kRadixBins + threadIdx.x; i < r1 * kRadixBins; i += kSortThreads) st_agent(&lb[i], 0ull);
}

// Records (RAW 1) or overlap events of instances (RAW 2) as the raw source;
// RAW 3: packed buffers only, without payloads.
template <int RAW>
__device__ __forceinline__ void radix_tile(const RadixArgs& a, RadixShared& s, const KeySpace& ks,
                                           const RadixPass& ps, uint64_t tile) {
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  for (int i = tid; i < kSortWaves * kRadixBins; i += kSortThreads) (&s.wave[0][0])[i] = 0;
  __syncthreads();
  const uint64_t base = tile * kSortTile;
  const uint64_t left = ps.n_elems - base;
  const uint32_t cnt = left < (uint64_t)kSortTile ? (uint32_t)left : (uint32_t)kSortTile;
  const bool wide = ks.wide != 0;

  uint64_t key[kSortItems];
  uint32_t pay[kSortItems], cw[kSortItems], dig[kSortItems], rank[kSortItems];

  // Loads first, all of them unconditional (an index past the tile's end is
  // clamped to its last element, whose digit is then discarded), so that
  // every load of the tile is in flight before the first one is used.
  auto elem = [&](int r) -> uint32_t {
    return (uint32_t)w * (kSortItems * 64) + (uint32_t)r * 64 + lane;
  };
  auto clamp = [&](uint32_t el) -> uint64_t { return base + (el < cnt ? el : cnt - 1); };
  auto digit = [&](uint64_t k, uint32_t c) -> uint32_t {
    if (ps.mode == kDigKey) return (uint32_t)(k >> ps.shift) & 0xFFu;
    const uint64_t rel = wide ? c : (ks.ts_bits >= 64 ? 0ull : (k >> ks.ts_bits));
    return (uint32_t)((ks.ctx_min + rel) >> ps.shift) & 0xFFu;
  };
  if (RAW == 3 || ps.src < 2) {
    const uint64_t* ksrc = ps.src ? a.key[1] : a.key[0];
    const uint32_t* psrc = ps.src ? a.pay[1] : a.pay[0];
    const uint32_t* csrc = ps.src ? a.ctxw[1] : a.ctxw[0];
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
      const uint64_t e = clamp(elem(r));
      key[r] = ld_agent(&ksrc[e]);
      pay[r] = RAW != 3 ? ld_agent(&psrc[e]) : 0u;
      cw[r] = wide ? ld_agent(&csrc[e]) : 0u;
    }
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) dig[r] = elem(r) < cnt ? digit(key[r], cw[r]) : 256u;
  } else if (RAW == 1) {
    uint4 rr[kSortItems];
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) rr[r] = a.rec[clamp(elem(r))];
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
      // branch-free, so that the whole 16-byte record is loaded up front
      const uint64_t ts = (uint64_t)rr[r].x | ((uint64_t)rr[r].y << 32);
      const uint32_t ctx = rr[r].z;
      const uint32_t region = rr[r].w & 0xFFFFu;
      const uint32_t kind = (rr[r].w >> 16) & 0xFFu;
      const bool ok = elem(r) < cnt && (kind == 1 || kind == 2) && region < a.R;
      const uint64_t ts_off = ts - ks.ts_min;
      const uint64_t ctx_rel = (uint64_t)ctx - ks.ctx_min;
      const uint64_t k = wide ? ts_off : ((ks.ts_bits >= 64 ? 0 : (ctx_rel << ks.ts_bits)) | ts_off);
      key[r] = ok ? k : 0;
      cw[r] = ok ? (uint32_t)ctx_rel : 0u;
      const uint32_t cls = ok && swept_ctx(ctx, a.K, a.G, a.shift) ? a.region_class[region] : 0xFFu;
      pay[r] = ok ? pack_payload(region, kind, cls) : 0u;
      dig[r] = ok ? digit(k, (uint32_t)ctx_rel) : 256u;  // 256: invalid (never written)
    }
  } else {
    // Overlap events: element e is the begin (even) or end (odd) of instance
    // e / 2; only matched, classified instances of a group < G.
    uint64_t tv[kSortItems];
    uint32_t cv[kSortItems], rv[kSortItems], cl[kSortItems];
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
      const uint64_t e = clamp(elem(r));
      const argus_instance* ip = a.inst + (e >> 1);
      tv[r] = (e & 1) ? ip->t_end : ip->t_begin;
      cv[r] = ip->ctx_key;
      rv[r] = *(const uint32_t*)&ip->region_id;  // region | end_region << 16
    }
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) cl[r] = a.region_class[rv[r] & 0xFFFFu];
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
      uint32_t d = 256;
      const uint32_t el = elem(r);
      const uint32_t is_end = (uint32_t)((base + el) & 1);
      const uint32_t region = rv[r] & 0xFFFFu, eregion = rv[r] >> 16;
      const uint64_t g = a.shift >= 32 ? 0 : (cv[r] >> a.shift);
      key[r] = 0;
      pay[r] = 0;
      cw[r] = 0;
      if (el < cnt && region == eregion && cl[r] < a.K && g < a.G) {
        const uint64_t ts_off = tv[r] - ks.ts_min;
        key[r] = wide ? ts_off : ((ks.ts_bits >= 64 ? 0 : (g << ks.ts_bits)) | ts_off);
        cw[r] = (uint32_t)g;
        pay[r] = cl[r] | (is_end << 8);
        d = digit(key[r], cw[r]);
      }
      dig[r] = d;
    }
  }
  // Rank among this wave's elements with the same digit (stable order is
  // wave, round, lane).  All loads above are already in flight.
#pragma unroll
  for (int r = 0; r < kSortItems; ++r) {
    const uint32_t d = dig[r];
    const bool part = d < 256;
    const uint64_t vm = __ballot(part);
    uint64_t peers = vm;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const uint32_t bit = (d >> b) & 1u;
      const uint64_t m = __ballot(bit);
      peers &= bit ? m : ~m;
    }
    uint32_t rk = 0;
    if (part) {
      const uint32_t before = (uint32_t)__popcll(peers & lanemask_lt());
      const uint32_t old = s.wave[w][d];
      rk = old + before;
      __builtin_amdgcn_wave_barrier();
      if ((peers >> lane) == 1ull) s.wave[w][d] = old + (uint32_t)__popcll(peers);
    }
    __builtin_amdgcn_wave_barrier();
    rank[r] = rk;
  }
  __syncthreads();

  // Digit totals of the tile (thread d: digit d), per-wave prefixes and
  // tile-local starts.
  const uint32_t dgt = (uint32_t)tid;
  const bool digits = dgt < (uint32_t)kRadixBins;
  uint32_t tot = 0, wc[kSortWaves];
  uint64_t* lb = a.lb + tile * kRadixBins + dgt;
  if (digits) {
#pragma unroll
    for (int q = 0; q < kSortWaves; ++q) {
      wc[q] = s.wave[q][dgt];
      tot += wc[q];
    }
    // published before the tile's own scan: the successors wait for it
    st_agent(lb, radix_word(tile == 0 ? kFlagIncl : kFlagAgg, ps.tag, tot));
  }
  uint32_t all;
  const uint32_t start = sort_excl_scan(tot, s.scr, &all);  // the digit's place in the staged tile
  if (tid == 0) s.total = all;
  if (digits) {
    // each wave's first place of the digit
    uint32_t at = start;
#pragma unroll
    for (int q = 0; q < kSortWaves; ++q) {
      s.wave[q][dgt] = at;
      at += wc[q];
    }
  }
  // Decoupled look-back on the count of this digit in earlier tiles.
  if (digits) {
    uint64_t excl = 0;
    if (tile != 0) {
      // Four predecessors per round trip; consume them nearest first.  (The
      // words come from beyond the L2, so reading more than are used costs:
      // over 2^24 records and two passes 1270 us for the run with 2 to 4 per
      // trip, 1275 with 8, 1395 with 16, 2140 with 32.)
      constexpr int kBack = 4;
      int64_t tt = (int64_t)tile - 1;
      uint32_t spins = 0;
      bool done = false;
      while (!done && tt >= 0) {
        uint64_t v[kBack];
#pragma unroll
        for (int q = 0; q < kBack; ++q)
          v[q] = tt - q >= 0 ? ld_agent(&a.lb[(uint64_t)(tt - q) * kRadixBins + dgt]) : radix_word(kFlagIncl, ps.tag, 0);
        int used = 0;
#pragma unroll
        for (int q = 0; q < kBack; ++q) {
          if (done || used != q) break;
          const uint64_t f = radix_flag(v[q], ps.tag);
          if (f == 0) break;  // not published yet: reload from here
          excl += v[q] & kRadixVal;
          ++used;
          if (f == kFlagIncl) done = true;
        }
        tt -= used;
        if (used == 0) {
          if (++spins > kMaxSpins) {
            flag_internal_error(a.counters, 1);
            break;
          }
          backoff();
        }
      }
      st_agent(lb, radix_word(kFlagIncl, ps.tag, (excl + tot) & kRadixVal));
    }
    s.gbase[dgt] = s.off[dgt] + (uint32_t)excl - start;
  }
  __syncthreads();

  // Stage in LDS in digit order.
#pragma unroll
  for (int r = 0; r < kSortItems; ++r) {
    const uint32_t d = dig[r];
    if (d < 256) {
      const uint32_t lp = s.wave[w][d] + rank[r];
      s.key[lp] = key[r];
      if (RAW != 3) s.pay[lp] = pay[r];
      if (wide) s.cw[lp] = cw[r];
    }
  }
  __syncthreads();

  // Write out: consecutive staged elements of one digit go to consecutive
  // global positions.  (The digit is taken from the staged key again: the
  // tile's LDS accesses conflict, so it stages as little as it can.)
  const uint32_t total = s.total;
  uint64_t* kd = a.key[ps.dst];
  uint32_t* pd = a.pay[ps.dst];
  uint32_t* cd = a.ctxw[ps.dst];
  const uint32_t n_out = ps.n_out;
  for (uint32_t i = tid; i < total; i += kSortThreads) {
    const uint64_t k = s.key[i];
    const uint32_t c = wide ? s.cw[i] : 0u;
    const uint32_t gp = s.gbase[digit(k, c)] + i;
    if (gp >= n_out) {
      flag_internal_error(a.counters, 2);
      continue;
    }
    st_agent(&kd[gp], k);
    if (RAW != 3) st_agent(&pd[gp], s.pay[i]);
    if (wide) st_agent(&cd[gp], c);
  }
  __syncthreads();
}

// One pass as a phase: its tiles, then (last = false) the wait for all of
// them.  Returns how many tiles this block did.  *fin: whether this block did
// the pass's last tile.
template <int RAW>
__device__ __forceinline__ uint32_t radix_phase(const RadixArgs& a, RadixShared& s, const KeySpace& ks,
                                                const RadixPass& ps, uint32_t phase, bool last,
                                                bool* fin) {
  uint32_t* ctr = phase_ctr(a.ctrs, phase);
  const uint32_t tiles = (uint32_t)ceil_div(ps.n_elems, kSortTile);
  uint32_t mine = 0;
  *fin = false;
  for (;;) {
    const uint32_t t = phase_take(ctr, &s.ticket);
    if (t >= tiles) break;
    radix_tile<RAW>(a, s, ks, ps, t);
    ++mine;
    *fin = t + 1 == tiles;
    if (*fin) break;
  }
  if (mine == tiles) {
    // no other block has any (nor will stay)
    drain_stores();
    __syncthreads();
  } else if (mine && !last) {
    phase_done(a.ctrs, phase, mine, tiles, &s.ticket);
    phase_wait(a.ctrs, phase, a.counters);
  }
  return mine;
}

// What a pass did, for the plan read back by measurements.
ARGUS_DEV void note_slot(SlotPlan& sp, uint32_t pos, const RadixPass& ps) {
  sp.active = 1;
  sp.pos = pos;
  sp.src = ps.src;
  sp.dst = ps.dst;
  sp.lb = 0;
  sp.n_out = ps.n_out;
  sp.n_elems = ps.n_elems;
  sp.tiles = ceil_div(ps.n_elems, kSortTile);
}

inline RadixArgs radix_args(const RunArgs& a) {
  RadixArgs ra{};
  ra.plan = a.w.plan;
  ra.rec = (const uint4*)a.rec;
  ra.inst = a.w.inst;
  ra.region_class = a.region_class;
  ra.R = a.R;
  ra.K = a.K;
  ra.G = a.G;
  ra.shift = a.shift;
  for (int b = 0; b < 2; ++b) {
    ra.key[b] = a.w.key[b];
    ra.pay[b] = a.w.pay[b];
    ra.ctxw[b] = a.w.ctxw[b];
  }
  ra.lb = a.w.lb;
  ra.clear_lb = a.n > kInitClearMax ? 1u : 0u;
  ra.ctrs = a.w.tile_ctr;
  ra.counters = a.out.d_counters;
  return ra;
}

// Blocks of a sort over `elems` elements: one per tile, up to those that
// fit at once.
inline uint32_t sort_blocks(const void* kern, uint64_t elems) {
  uint64_t blocks = ceil_div(elems ? elems : 1, kSortTile);
  const uint64_t resident = persistent_blocks(kern, kSortThreads);
  return (uint32_t)(blocks < resident ? blocks : resident);
}

}  // namespace argus
