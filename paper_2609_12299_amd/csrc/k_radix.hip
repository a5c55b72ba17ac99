// k_radix.hip -- the sorts of the records: by context, and (when some
// context is out of time order in the input) by context and time.  Each
// sort is one persistent kernel whose passes are phases (chain.h).
#include "radix_tile.h"
#include "tile_sums.h"

namespace argus {

// ------------------------------------------------- context sort over runs
//
// When the input holds long runs of one context (trace buffers written per
// warp, interleaved in chunks), a stable sort of the records by context is:
// the runs sorted stably by context (a radix sort over runs, not records),
// each run's first position an exclusive scan of the run lengths in that
// order, and every record written to its run's position plus its rank among
// the run's valid records (k_runs_scatter).  Within a context, runs and the
// records of a run keep input order, so the result equals the record radix
// sort's.

struct CtxSortArgs {
  RadixArgs r;
  const uint32_t* rec_hist;    // raw context digits over records
  // runs
  const uint64_t* runs_raw;
  const uint32_t* chunk_runs;
  uint32_t* run_base;
  uint32_t* run_cnt;
  uint32_t* run_pos;
  uint32_t* run_hist;  // [4][256]
  uint64_t* scan0;     // look-back words over tiles of chunks
  uint64_t* scan1;     // ... over tiles of sorted runs
  ChunkWaves cw;
};

// Tile of 1024 chunks: each chunk's first run index (a scan of the chunks'
// run counts), then the runs of the chunks in input order as sort elements
// (key: context offset << ts_bits, payload: run id), their lengths, and the
// context-digit histograms over runs.  A run without valid records sorts as
// the lowest context.
__device__ __forceinline__ void runs_compact_tile(const CtxSortArgs& a, RadixShared& s, uint32_t* s_hist,
                                                  const KeySpace& ks, uint64_t chunks, uint32_t tile) {
  const uint32_t tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  constexpr int kPer = kChunksPerTile / kSortThreads;
  const uint64_t c0 = (uint64_t)tile * kChunksPerTile + kPer * tid;
  uint32_t word[kPer], cnt[kPer], sum = 0;
#pragma unroll
  for (int q = 0; q < kPer; ++q) word[q] = c0 + q < chunks ? a.chunk_runs[chunk_slot(a.cw, c0 + q)] : 0u;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    cnt[q] = word[q] & ((1u << kChunkCountBits) - 1u);
    sum += cnt[q];
  }
  uint32_t total;
  uint32_t pre = sort_excl_scan(sum, s.scr, &total);
  // per chunk of the tile: first run in the tile, place of its list
  uint32_t* s_first = s.cw;
  uint64_t* s_list = s.key;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    s_first[kPer * tid + q] = pre;
    s_list[kPer * tid + q] = wave_slot0(a.cw, (c0 + q) % a.cw.W) * kChunk + (word[q] >> kChunkCountBits);
    pre += cnt[q];
  }
  if (w == 0) {
    const uint32_t ex = (uint32_t)scan_lookback(a.scan0, tile, total, &a.r.counters[31], 2048);
    if (lane == 0) s.total = ex;
  }
  __syncthreads();
  const uint32_t r0 = s.total;  // runs before the tile
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const uint32_t c = (uint32_t)q * kSortThreads + tid;
    if ((uint64_t)tile * kChunksPerTile + c < chunks) a.run_base[(uint64_t)tile * kChunksPerTile + c] = r0 + s_first[c];
  }
  // consecutive threads take consecutive runs (the chunk of each by a search
  // over the tile's chunks): whole lines are written at once
  for (uint32_t i = tid; i < total; i += kSortThreads) {
    uint32_t lo = 0, hi = kChunksPerTile;  // the last chunk whose first run is <= i
#pragma unroll
    for (int b = 0; b < 10; ++b) {
      const uint32_t mid = (lo + hi) >> 1;
      if (s_first[mid] <= i) lo = mid;
      else hi = mid;
    }
    const uint64_t v = a.runs_raw[s_list[lo] + (i - s_first[lo])];
    const uint32_t n = (uint32_t)(v >> 32);
    const uint64_t rel = n ? (uint64_t)((uint32_t)v - (uint32_t)ks.ctx_min) : 0ull;
    const uint32_t rid = r0 + i;
    st_agent(&a.r.key[0][rid], ks.ts_bits >= 64 ? 0ull : (rel << ks.ts_bits));
    st_agent(&a.r.pay[0][rid], rid);
    st_agent(&a.run_cnt[rid], n);
    const uint32_t ctx = (uint32_t)(ks.ctx_min + rel);
#pragma unroll
    for (int d = 0; d < 4; ++d) atomicAdd(&s_hist[d * kRadixBins + ((ctx >> (8 * d)) & 0xFFu)], 1u);
  }
}

// Tile of 4096 sorted runs: each run's first sorted record position (a scan
// of the run lengths in sorted order), and whether it starts its context: it
// does if it has valid records and the previous run has another context;
// runs without valid records sort as context offset 0, so the runs of
// offset 0 start it only at position 0.
__device__ __forceinline__ void runs_pos_tile(const CtxSortArgs& a, RadixShared& s, const KeySpace& ks,
                                              uint64_t n_runs, uint32_t buf, uint32_t tile) {
  const uint32_t tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const uint32_t* ids = a.r.pay[buf];
  const uint64_t* keys = a.r.key[buf];
  const uint64_t base = (uint64_t)tile * kSortTile;
  constexpr int kPer = kSortItems;
  const uint32_t cnt = n_runs - base < (uint64_t)kSortTile ? (uint32_t)(n_runs - base) : (uint32_t)kSortTile;
  auto ctx_of = [&](uint64_t k) -> uint32_t { return ks.ts_bits >= 64 ? 0u : (uint32_t)(k >> ks.ts_bits); };
  // loaded in rows of 512 consecutive runs; the lengths through LDS, where
  // each thread scans 8 consecutive ones (a pad word after every 8)
  uint32_t* const s_len = (uint32_t*)s.key;
  uint32_t* const s_cx = s.pay;
  auto slot = [](uint32_t i) { return i + (i >> 3); };
  uint32_t id[kPer], len[kPer], cx[kPer];
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const uint32_t i = (uint32_t)q * kSortThreads + tid;
    const uint64_t e = base + (i < cnt ? i : cnt - 1);
    id[q] = ld_agent(&ids[e]);
    cx[q] = ctx_of(ld_agent(&keys[e]));
  }
  const uint32_t prev0 = base > 0 ? ctx_of(ld_agent(&keys[base - 1])) : 0xFFFFFFFFu;
#pragma unroll
  for (int q = 0; q < kPer; ++q) len[q] = ld_agent(&a.run_cnt[id[q]]);
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const uint32_t i = (uint32_t)q * kSortThreads + tid;
    if (i >= cnt) len[q] = 0;
    s_len[slot(i)] = len[q];
    s_cx[i] = cx[q];
  }
  __syncthreads();
  uint32_t v[kPer], sum = 0;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    v[q] = s_len[slot((uint32_t)kPer * tid + q)];
    sum += v[q];
  }
  uint32_t total;
  uint32_t pre = sort_excl_scan(sum, s.scr, &total);
  if (w == 0) {
    const uint32_t ex = (uint32_t)scan_lookback(a.scan1, tile, total, &a.r.counters[31], 2048);
    if (lane == 0) s.total = ex;
  }
  __syncthreads();
  pre += s.total;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    s_len[slot((uint32_t)kPer * tid + q)] = pre;
    pre += v[q];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const uint32_t i = (uint32_t)q * kSortThreads + tid;
    if (i >= cnt) continue;
    const uint32_t pos = s_len[slot(i)], prev = i > 0 ? s_cx[i - 1] : prev0;
    const bool head = len[q] > 0 && (cx[q] == 0 ? pos == 0 : prev != cx[q]);
    a.run_pos[id[q]] = pos | ((head ? 1u : 0u) << 31);
  }
}

// The sort by context.  With long runs of one context in the input: the runs
// compacted, sorted and placed (k_runs_scatter then writes the records);
// else radix passes over the records' varying context digits.  Stable, so
// that contexts already in time order in the input are then sorted.  Nothing
// to do when the ingest has seen a context out of time order: k_full_sort
// starts from the input.
__global__ __launch_bounds__(kSortThreads, 4) void k_ctx_sort(CtxSortArgs a) {
  DevPlan* p = a.r.plan;
  if (p->early) return;
  __shared__ RadixShared s;
  const KeySpace ks = p->rec;
  const bool runs = p->runs != 0;
  const uint64_t n_valid = p->n_valid, n_records = p->n_records, n_runs = p->n_runs;
  const uint32_t tid = threadIdx.x;
  if (runs) {
    uint32_t* s_hist = s.pay;  // [4][256]
    for (uint32_t i = tid; i < 4 * kRadixBins; i += kSortThreads) s_hist[i] = 0;
    const uint64_t chunks = ceil_div(n_records, kChunk);
    const uint32_t tiles = (uint32_t)ceil_div(chunks, kChunksPerTile);
    uint32_t* ctr = phase_ctr(a.r.ctrs, kPhCompact);
    uint32_t mine = 0;
    for (;;) {
      const uint32_t t = phase_take(ctr, &s.ticket);
      if (t >= tiles) break;
      runs_compact_tile(a, s, s_hist, ks, chunks, t);
      if (a.r.clear_lb) {  // this tile's share of the rows that the run passes use
        const uint64_t rows = ceil_div(n_runs, kSortTile);
        clear_rows(a.r.lb, rows * t / tiles, rows * (t + 1) / tiles);
      }
      ++mine;
    }
    for (uint32_t i = tid; mine && i < 4 * kRadixBins; i += kSortThreads) {
      const uint32_t h = s_hist[i];
      if (h) atomicAdd(&a.run_hist[i], h);
    }
    // later phases may have more tiles than this one (up to 32 runs a chunk):
    // a block without a tile here stays
    if (mine) phase_done(a.r.ctrs, kPhCompact, mine, tiles, &s.ticket);
    phase_wait(a.r.ctrs, kPhCompact, a.r.counters);
  } else if (a.r.clear_lb) {
    const uint64_t rows = ceil_div(n_records, kSortTile);
    const uint32_t tiles = (uint32_t)ceil_div(rows, 64);
    uint32_t* ctr = phase_ctr(a.r.ctrs, kPhClear);
    uint32_t mine = 0;
    for (;;) {
      const uint32_t t = phase_take(ctr, &s.ticket);
      if (t >= tiles) break;
      clear_rows(a.r.lb, 64ull * t, 64ull * t + 64 < rows ? 64ull * t + 64 : rows);
      ++mine;
    }
    if (mine) phase_done(a.r.ctrs, kPhClear, mine, tiles, &s.ticket);
    phase_wait(a.r.ctrs, kPhClear, a.r.counters);
  }
  const uint32_t* hist = runs ? a.run_hist : a.rec_hist;
  uint32_t act = digits_varying<4>(hist, 4);
  if (!runs && !act) act = 1;  // one pass packs the records
  uint32_t src = runs ? 0u : 2u;
  for (uint32_t pos = 0; pos < 4; ++pos) {
    if (!((act >> pos) & 1u)) continue;
    RadixPass ps;
    ps.src = src;
    ps.dst = src == 2 ? 0u : src ^ 1u;
    ps.mode = kDigCtx;
    ps.shift = 8 * pos;
    ps.tag = 1 + pos;
    ps.n_out = (uint32_t)(runs ? n_runs : n_valid);
    ps.n_elems = runs ? n_runs : src == 2 ? n_records : n_valid;
    radix_offsets(s, hist + pos * kRadixBins);
    const bool last = !runs && (act >> (pos + 1)) == 0;
    bool fin;
    const uint32_t mine = radix_phase<1>(a.r, s, ks, ps, kPhCtx + pos, last, &fin);
    src = ps.dst;
    if (fin && tid == 0) {
      note_slot(p->rs[pos], pos, ps);
      // the last pass only: the block of an earlier one's last tile may come
      // here after a later pass has ended (over runs: the scatter writes
      // buffer 0)
      if (!runs && (act >> (pos + 1)) == 0) p->rec_final = ps.dst;
    }
    if (!mine) return;
  }
  if (runs) {
    uint32_t* ctr = phase_ctr(a.r.ctrs, kPhRunPos);
    const uint32_t tiles = (uint32_t)ceil_div(n_runs, kSortTile);
    for (;;) {
      const uint32_t t = phase_take(ctr, &s.ticket);
      if (t >= tiles) break;
      runs_pos_tile(a, s, ks, n_runs, src, t);
    }
  }
}

hipError_t launch_ctx_sort(const RunArgs& a, hipStream_t s) {
  CtxSortArgs c{};
  c.r = radix_args(a);
  c.rec_hist = a.w.rec_hist;
  c.runs_raw = a.w.key[1];
  c.chunk_runs = a.w.chunk_runs;
  c.run_base = a.w.run_base;
  c.run_cnt = a.w.run_cnt;
  c.run_pos = a.w.run_pos;
  c.run_hist = a.w.run_hist;
  c.scan0 = a.w.scan_lb;
  c.scan1 = a.w.scan_lb + ceil_div(a.w.chunks, kChunksPerTile);
  c.cw = chunk_waves(a.w.chunks, ingest_blocks(a.n) * 4);
  hipLaunchKernelGGL(k_ctx_sort, dim3(sort_blocks((const void*)k_ctx_sort, a.n)), dim3(kSortThreads), 0, s, c);
  return hipGetLastError();
}

// ------------------------------------------------------------- full sort

struct FullSortArgs {
  RadixArgs r;
  uint32_t* hist;            // [8][256] packed-key digits (zero on entry)
  const uint32_t* ctx_hist;  // [4][256] raw context digits over records
  TsumArgs t;
};

// Some context is out of time order in the input: a stable sort on the
// whole packed key (or, where context and time do not fit 64 bits, on the
// time digits and then the context digits), from the input itself when the
// ingest saw it, else from the context-sorted records; then the tile sums.
// Digits are taken from the key's offsets, so no pass goes over bits that
// ts_min and ctx_min have in common.
__global__ __launch_bounds__(kSortThreads, 4) void k_full_sort(FullSortArgs a) {
  DevPlan* p = a.r.plan;
  if (!p->unsorted) return;
  __shared__ RadixShared s;
  static_assert(sizeof(TsumShared) <= sizeof(s.key), "tile sums share the stage");
  TsumShared& ts = *reinterpret_cast<TsumShared*>(s.key);
  const KeySpace ks = p->rec;
  const bool wide = ks.wide != 0;
  const uint64_t n_valid = p->n_valid, n_records = p->n_records;
  const uint32_t tid = threadIdx.x;
  const uint32_t src0 = p->early ? 2u : p->rec_final;
  const uint32_t key_bits = wide ? ks.ts_bits : ks.ts_bits + ks.ctx_bits;
  const uint32_t nd = (key_bits + 7) / 8;  // key digits (at most 8)
  {  // histograms of the key digits
    uint32_t* s_hist = s.pay;  // [8][256]
    for (uint32_t i = tid; i < nd * kRadixBins; i += kSortThreads) s_hist[i] = 0;
    const uint64_t n = src0 == 2 ? n_records : n_valid;
    const uint32_t tiles = (uint32_t)ceil_div(n, kSortTile);
    const uint64_t* ksrc = a.r.key[src0 & 1u];
    uint32_t* ctr = phase_ctr(a.r.ctrs, kPhHist);
    uint32_t mine = 0;
    for (;;) {
      const uint32_t t = phase_take(ctr, &s.ticket);
      if (t >= tiles) break;
      if (a.r.clear_lb) clear_rows(a.r.lb, t, t + 1);
      const uint64_t base = (uint64_t)t * kSortTile;
      uint64_t k[kSortItems];
      bool ok[kSortItems];
      if (src0 == 2) {
        uint4 v[kSortItems];
#pragma unroll
        for (int r = 0; r < kSortItems; ++r) {
          const uint64_t i = base + (uint32_t)r * kSortThreads + tid;
          v[r] = a.r.rec[i < n ? i : n - 1];
        }
#pragma unroll
        for (int r = 0; r < kSortItems; ++r) {
          const uint32_t kind = (v[r].w >> 16) & 0xFFu;
          ok[r] = base + (uint32_t)r * kSortThreads + tid < n && (kind == 1 || kind == 2) && (v[r].w & 0xFFFFu) < a.r.R;
          const uint64_t t_off = ((uint64_t)v[r].x | ((uint64_t)v[r].y << 32)) - ks.ts_min;
          const uint64_t c_rel = (uint64_t)v[r].z - ks.ctx_min;
          k[r] = wide ? t_off : ((ks.ts_bits >= 64 ? 0 : (c_rel << ks.ts_bits)) | t_off);
        }
      } else {
#pragma unroll
        for (int r = 0; r < kSortItems; ++r) {
          const uint64_t i = base + (uint32_t)r * kSortThreads + tid;
          ok[r] = i < n;
          k[r] = ksrc[i < n ? i : n - 1];
        }
      }
      for (uint32_t d = 0; d < nd; ++d)
#pragma unroll
        for (int r = 0; r < kSortItems; ++r)
          hist_digit(s_hist + d * kRadixBins, (uint32_t)(k[r] >> (8 * d)) & 0xFFu, ok[r]);
      ++mine;
      if (t + 1 == tiles) break;
    }
    // a block without a tile leaves: the passes have no more tiles than this
    // phase (the tile sums have up to two per tile: each block takes several)
    if (!mine) return;
    __syncthreads();
    for (uint32_t i = tid; i < nd * kRadixBins; i += kSortThreads) {
      const uint32_t h = s_hist[i];
      if (h) atomicAdd(&a.hist[i], h);
    }
    phase_done(a.r.ctrs, kPhHist, mine, tiles, &s.ticket);
    if (mine < tiles) phase_wait(a.r.ctrs, kPhHist, a.r.counters);
  }
  // pass k < 8: key digit k; 8 + k: raw context digit k (wide keys only)
  uint32_t act = digits_varying<8>(a.hist, nd);
  if (wide) act |= digits_varying<4>(a.ctx_hist, 4) << 8;
  if (!act && src0 == 2) act = nd ? 1u : 1u << 8;  // one pass packs the records
  uint32_t src = src0;
  for (uint32_t d = 0; d < 12; ++d) {
    if (!((act >> d) & 1u)) continue;
    RadixPass ps;
    ps.src = src;
    ps.dst = src == 2 ? 0u : src ^ 1u;
    ps.mode = d < 8 ? kDigKey : kDigCtx;
    ps.shift = 8 * (d & 7u);
    ps.tag = 5 + d;
    ps.n_out = (uint32_t)n_valid;
    ps.n_elems = src == 2 ? n_records : n_valid;
    radix_offsets(s, d < 8 ? a.hist + d * kRadixBins : a.ctx_hist + (d - 8) * kRadixBins);
    bool fin;
    const uint32_t mine = radix_phase<1>(a.r, s, ks, ps, kPhFull + d, false, &fin);
    src = ps.dst;
    if (fin && tid == 0) note_slot(p->rs[kPhase2Slot + d], d < 8 ? 4 + d : d - 8, ps);
    if (!mine) return;
  }
  // tile sums of the sorted records, and their scan by the last block (plain
  // loads: what this XCD's caches hold of the buffers is dropped first)
  if (tid < 64) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  __syncthreads();
  uint32_t* ctr = phase_ctr(a.r.ctrs, kPhTsum);
  uint32_t mine = 0;
  for (;;) {
    const uint32_t vb = phase_take(ctr, &s.ticket);
    if (vb >= a.t.nblk) break;
    tsum_run<false, kSortThreads>(a.t, ts, ks, n_valid, src, vb);
    ++mine;
    if (vb + 1 == a.t.nblk) break;
  }
  if (!mine || phase_done(a.r.ctrs, kPhTsum, mine, a.t.nblk, &s.ticket) != a.t.nblk) return;
  mscan_top<kSortThreads>(a.t, ts, ceil_div(n_valid, kMatchTile));
  if (tid == 0) p->rec_final = src;
}

hipError_t launch_full_sort(const RunArgs& a, hipStream_t s) {
  FullSortArgs f{};
  f.r = radix_args(a);
  f.hist = a.w.rec_hist + 4 * kRadixBins;
  f.ctx_hist = a.w.rec_hist;
  f.t = tsum_args(a);
  hipLaunchKernelGGL(k_full_sort, dim3(sort_blocks((const void*)k_full_sort, a.n)), dim3(kSortThreads), 0, s, f);
  return hipGetLastError();
}

}  // namespace argus
