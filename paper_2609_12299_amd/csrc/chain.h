// chain.h -- several dependent passes in one persistent kernel.
//
// The passes of a sort are planned on the device: which of them run is not
// known when they are enqueued.  A launch per possible pass costs 1.5 to 4.7
// us each even when it finds nothing to do (38 such launches, 180 us, in a
// run over 2^24 interleaved records), so the passes of one sort share a
// kernel.  A pass is a phase: its tiles are taken in order from a ticket
// counter, and the next phase starts when the tiles done add up to the
// phase's total.  A block waits only for tiles that running blocks have
// taken, so the wait ends whatever the number of blocks resident (nothing
// waits for a block that has not started); a block that gets no tile of a
// phase leaves when no later phase has more tiles.
//
// What one block writes and another reads within a kernel goes through
// agent-scope atomics (st_agent / ld_agent: past the L2, of which each XCD
// has its own), and a block reports its tiles after its stores have been
// acknowledged.  Plain stores behind agent-scope fences would need none of
// that, but such a fence writes back or invalidates a whole L2, and with
// hundreds of blocks doing so at each phase the four run passes of a
// 2^28-record trace took 550 instead of 200 us.
#pragma once

#include "internal.h"

namespace argus {

// Counters of one phase: tickets at word 0, tiles done at word 8.
ARGUS_DEV uint32_t* phase_ctr(uint32_t* ctrs, uint32_t phase) { return ctrs + kPhaseBase + phase * kPhaseWords; }

// Every store and atomic of this wave has been acknowledged.
ARGUS_DEV void drain_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// The next tile of the phase, in every thread of the block.
ARGUS_DEV uint32_t phase_take(uint32_t* ctr, uint32_t* s_slot) {
  __syncthreads();  // the previous ticket has been read by every thread
  if (threadIdx.x == 0) *s_slot = atomicAdd(ctr, 1u);
  __syncthreads();
  return *s_slot;
}

// The block's `mine` tiles are done (its agent-scope stores acknowledged);
// the block whose tiles complete the phase's `total` releases the waiting
// blocks.  Returns (in every thread) the tiles done so far, these included.
ARGUS_DEV uint32_t phase_done(uint32_t* ctrs, uint32_t phase, uint32_t mine, uint32_t total, uint32_t* s_slot) {
  drain_stores();
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t done = atomicAdd(phase_ctr(ctrs, phase) + 8, mine) + mine;
    if (done == total) st_agent(&ctrs[phase], 1u);
    *s_slot = done;
  }
  __syncthreads();
  const uint32_t done = *s_slot;
  __syncthreads();
  return done;
}

// Waits until all tiles of the phase are done (bounded, like the look-back
// waits).  The word the blocks poll is written once and lies 256 bytes from
// what others add to: polled by up to 512 blocks, the counter of the tiles
// done kept the blocks still at work from adding to it (and to the tickets, 64
// bytes away): four passes over 2^22 elements took 365 us, this way 178;
// 2^20: 127, 84; 2^24: 907, 718.  (Several such words, or longer sleeps, were
// no faster.)
ARGUS_DEV void phase_wait(const uint32_t* ctrs, uint32_t phase, uint64_t* counters) {
  if (threadIdx.x == 0) {
    uint32_t spins = 0;
    while (ld_agent(&ctrs[phase]) == 0) {
      if (++spins > kMaxSpins) {
        flag_internal_error(counters, 2048);
        break;
      }
      __builtin_amdgcn_s_sleep(2);
    }
  }
  __syncthreads();
  asm volatile("" ::: "memory");
}

// Whether this block is the last of the grid's first `total` blocks to
// arrive: the agent-scope stores and atomics of all the others are then
// visible to its agent-scope loads.  (In every thread.)
ARGUS_DEV bool last_arrival(uint32_t* ctrs, uint32_t which, uint32_t total, uint32_t* s_slot) {
  uint32_t* c = ctrs + kPhaseBase + kPhCount * kPhaseWords + which * kArriveWords;
  drain_stores();
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t g = blockIdx.x % kArriveGroups;
    const uint32_t size = (total - g + kArriveGroups - 1) / kArriveGroups;
    const uint32_t groups = total < kArriveGroups ? total : kArriveGroups;
    uint32_t last = atomicAdd(c + 16 * (g + 1), 1u) + 1 == size;
    if (last) last = atomicAdd(c, 1u) + 1 == groups;
    *s_slot = last;
  }
  __syncthreads();
  const bool last = *s_slot != 0;
  __syncthreads();
  return last;
}

// Exclusive prefix of `tot` (the tile's total) over the tiles of a phase, by
// one wave: the tile's word is published with its own total, then the
// wave reads 64 predecessors per round trip, nearest first, until one holds
// its inclusive prefix.  Totals stay below 2^32.  The words start at zero.
// A wait that gives up sets `code` in *error.
ARGUS_DEV uint64_t scan_lookback(uint64_t* words, uint32_t tile, uint32_t tot, uint64_t* error, uint64_t code) {
  const uint32_t lane = lane_id();
  if (tile == 0) {
    if (lane == 0) st_agent(&words[0], kFlagIncl | tot);
    return 0;
  }
  if (lane == 0) st_agent(&words[tile], kFlagAgg | tot);
  uint64_t excl = 0;
  int64_t top = (int64_t)tile - 1;
  uint32_t spins = 0;
  for (;;) {
    const int64_t q = top - (int64_t)lane;
    const uint64_t v = q >= 0 ? ld_agent(&words[q]) : kFlagIncl;
    const uint64_t f = v & ~kValMask;
    const uint64_t mi = __ballot(f == kFlagIncl), mn = __ballot(f == 0);
    const uint32_t ji = mi ? (uint32_t)__builtin_ctzll(mi) : 64u;  // nearest inclusive
    const uint32_t jn = mn ? (uint32_t)__builtin_ctzll(mn) : 64u;  // nearest not published
    const bool found = ji < jn;
    const uint32_t use = found ? ji + 1 : jn;  // lanes [0, use) are summed
    excl += rows_sum64(row_sum64(lane < use ? (v & kValMask) : 0ull));
    if (found) break;
    top -= jn;
    if (jn == 0) {
      if (++spins > kMaxSpins) {
        if (lane == 0) atomicOr((unsigned long long*)error, (unsigned long long)code);
        break;
      }
      backoff();
    }
  }
  if (lane == 0) st_agent(&words[tile], kFlagIncl | (excl + tot));
  return excl;
}

}  // namespace argus
