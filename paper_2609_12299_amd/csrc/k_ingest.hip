// k_ingest.hip -- run initialisation, record validation and the sort plans.
//
// Validation follows the definition of a marker record: only BEGIN (1) and
// END (2) transitions of known regions (id < R) carry region identity (the
// paper's Section 3.2); anything else is counted and dropped.
#include "tile_sums.h"

namespace argus {

// ---------------------------------------------------------------- helpers

template <typename T>
__device__ __forceinline__ T wave_min(T v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    T u = __shfl_xor(v, o);
    v = u < v ? u : v;
  }
  return v;
}
template <typename T>
__device__ __forceinline__ T wave_max(T v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    T u = __shfl_xor(v, o);
    v = u > v ? u : v;
  }
  return v;
}

// ------------------------------------------------- runs of one context
// A wave holds one input chunk of 256 records as 4 rows of 64 lanes (record
// 64 j + lane of the chunk in row j); masks over the chunk have bit
// p = 64 j + lane in word j.
static_assert(kChunk == 256, "a chunk is 4 rows of a wave");

// Run heads (a record whose predecessor in the chunk has another context,
// or the chunk's first record) and valid records of the chunk.
__device__ __forceinline__ void chunk_masks(const uint32_t (&ctx)[4], const bool (&in)[4],
                                            const bool (&valid)[4], uint64_t (&H)[4],
                                            uint64_t (&V)[4]) {
  const uint32_t lane = lane_id();
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    // previous record: the previous lane, or the last lane of the row before
    const uint32_t prev =
        lane_prev(ctx[j], j > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)ctx[j > 0 ? j - 1 : 0], 63) : ctx[j]);
    const bool head = in[j] && ((j == 0 && lane == 0) || prev != ctx[j]);
    H[j] = __ballot(head);
    V[j] = __ballot(valid[j]);
  }
}

// ------------------------------------------------------------------ init

struct Fill {
  uint64_t* p;
  uint64_t n;
  uint64_t v;
};
constexpr int kMaxFill = 16;
struct FillList {
  Fill f[kMaxFill];
  int count;
  uint64_t n_records;
  uint32_t R;
  uint32_t force_full;
  uint64_t* counters;
  uint64_t* rstats;
  DevPlan* plan;
};

// Initialises every output and the parts of the workspace that a run needs
// zeroed.  A fill kernel rather than hipMemsetAsync keeps the run
// capturable into a HIP graph.
__global__ __launch_bounds__(256) void k_init(FillList fl) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  const uint64_t tid = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (int s = 0; s < fl.count; ++s) {
    const Fill f = fl.f[s];
    for (uint64_t i = tid; i < f.n; i += stride) f.p[i] = f.v;
  }
  // counters
  if (tid < ARGUS_NUM_COUNTERS) {
    uint64_t v = 0;
    if (tid == ARGUS_C_N_RECORDS) v = fl.n_records;
    if (tid == ARGUS_C_TS_MIN || tid == ARGUS_C_CTX_MIN) v = kU64Max;
    fl.counters[tid] = v;
  }
  // region statistics: zero, except the minima
  const uint64_t nrs = (uint64_t)fl.R * ARGUS_RS_WIDTH;
  for (uint64_t i = tid; i < nrs; i += stride) {
    const uint32_t col = (uint32_t)(i % ARGUS_RS_WIDTH);
    fl.rstats[i] = (col == ARGUS_RS_INCL_MIN || col == ARGUS_RS_EXCL_MIN) ? kU64Max : 0;
  }
  if (tid == 0) {
    fl.plan->n_records = fl.n_records;
    fl.plan->force_full = fl.force_full;
  }
}

hipError_t launch_init(const RunArgs& a, hipStream_t s) {
  FillList fl{};
  const Work& w = a.w;
  auto add = [&](void* p, uint64_t bytes, uint64_t v) {
    if (fl.count < kMaxFill && bytes >= 8) fl.f[fl.count++] = Fill{(uint64_t*)p, bytes / 8, v};
  };
  add(w.plan, sizeof(DevPlan), 0);
  add(w.rec_hist, sizeof(uint32_t) * kDigitPositions * kRadixBins, 0);
  add(w.ev_hist, sizeof(uint32_t) * kDigitPositions * kRadixBins, 0);
  add(w.tile_ctr, sizeof(uint32_t) * kCtrWords, 0);
  add(w.run_hist, sizeof(uint32_t) * 4 * kRadixBins, 0);
  // look-back words of the run scans and of the record passes (whose tiles
  // cover every record; the event sort clears its own)
  add(w.scan_lb, sizeof(uint64_t) * w.scan_words, 0);
  if (a.n <= kInitClearMax) add(w.lb, sizeof(uint64_t) * ceil_div(a.n ? a.n : 1, kSortTile) * kRadixBins, 0);
  if (a.K > 0) {
    add(w.ov_mask, sizeof(uint64_t) * kMasks * a.G, 0);
    add(w.ov_q, sizeof(uint64_t) * kQPairs * a.G, 0);
    add(a.out.d_overlap_group, sizeof(uint64_t) * 2ull * a.K * a.K * a.G, 0);
    add(a.out.d_overlap_global, sizeof(uint64_t) * 2ull * a.K * a.K, 0);
  }
  fl.n_records = a.n;
  fl.R = a.R;
  fl.force_full = (a.flags & ARGUS_FORCE_FULL_SORT) ? 1u : 0u;
  fl.counters = a.out.d_counters;
  fl.rstats = a.out.d_region_stats;
  fl.plan = w.plan;
  uint64_t most = (uint64_t)a.R * ARGUS_RS_WIDTH;
  for (int i = 0; i < fl.count; ++i) most = most > fl.f[i].n ? most : fl.f[i].n;
  uint64_t blocks = ceil_div(most, 256 * 4);
  if (blocks < 1) blocks = 1;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_init, dim3((uint32_t)blocks), dim3(256), 0, s, fl);
  return hipGetLastError();
}

// ---------------------------------------------------------------- ingest

struct IngestArgs {
  const uint4* rec;
  uint64_t n;
  uint32_t R;
  uint64_t* counters;
  uint32_t* hist;        // rec_hist: positions 0..3 (raw context digits)
  DevPlan* plan;
  uint64_t* runs_raw;    // [chunk * 256 + j]: context | valid records << 32 of run j
  uint32_t* chunk_runs;  // [chunk slot]: count | place << kChunkCountBits
  uint32_t* ctrs;        // phase counters
  uint32_t force_radix;  // ARGUS_FORCE_RECORD_RADIX
  uint64_t run_cap;      // runs the run path accepts
};

__device__ __forceinline__ uint64_t mask_bits(uint32_t bits) {
  return bits >= 64 ? kU64Max : ((1ull << bits) - 1);
}

// The plan of the sorts, by one thread of the ingest's last block (no launch
// and no host round trip in between).
__device__ __forceinline__ void make_plan(const IngestArgs& a) {
  DevPlan* p = a.plan;
  auto counter = [&](int i) { return ld_agent(&a.counters[i]); };
  const uint64_t n_valid = counter(ARGUS_C_N_VALID);
  p->n_valid = n_valid;
  p->n_begin = counter(ARGUS_C_N_BEGIN);
  KeySpace k{};
  if (n_valid) {
    const uint64_t ts_min = counter(ARGUS_C_TS_MIN), ts_max = counter(ARGUS_C_TS_MAX);
    const uint64_t c_min = counter(ARGUS_C_CTX_MIN), c_max = counter(ARGUS_C_CTX_MAX);
    k.ts_min = ts_min;
    k.ts_bits = bit_width64(ts_max - ts_min);
    k.ctx_min = c_min;
    k.ctx_bits = bit_width64(c_max - c_min);
  }
  k.ts_mask = mask_bits(k.ts_bits);
  k.wide = (k.ts_bits + k.ctx_bits > 64) ? 1u : 0u;
  p->rec = k;
  p->match_tiles = ceil_div(n_valid, kMatchTile);
  // Long runs of one context in the input (per-warp buffers written in
  // chunks): sort the runs, then place the records, instead of radix
  // passes over every record.
  p->runs = (!a.force_radix && !k.wide && n_valid > 0 && ld_agent(&p->n_runs) <= a.run_cap) ? 1u : 0u;
  const uint32_t early = p->force_full | ld_agent(&p->unsorted);
  if (early) p->unsorted = 1;
  p->early = early;  // what the ingest saw: the full sort starts from the input
}

// Staged run lists per wave (entries; chunk table words).
constexpr uint32_t kStageRuns = 512;
constexpr uint32_t kStageChunks = 256;
static_assert(kStageRuns >= kChunk, "a chunk's runs fit the stage");
constexpr int kFewRuns = 4;  // runs of a row that add their digits one by one

// One coalesced 16-byte load per record.  Counts kinds and regions, reduces
// the timestamp and context ranges of valid records, and builds the 256-bin
// histograms of the four raw context digits (used by the context passes of
// the sort).  Each wave step covers one 256-record chunk, whose runs of one
// context (and their valid records) are recorded for the context sort over
// runs; the histograms and the context range are added per run.
__global__ __launch_bounds__(256) void k_ingest(IngestArgs a) {
  __shared__ uint32_t s_hist[4][kRadixBins];
  __shared__ uint64_t s_red[4][8];
  __shared__ unsigned long long s_runs;
  __shared__ uint64_t s_stage[4][kStageRuns];
  __shared__ uint32_t s_ctab[4][kStageChunks];
  __shared__ uint32_t s_slot;
  if (threadIdx.x == 0) s_runs = 0;
  for (int i = threadIdx.x; i < 4 * kRadixBins; i += 256) (&s_hist[0][0])[i] = 0;
  __syncthreads();

  // Counts are wave-uniform (from ballots); extremes are per lane.
  uint64_t n_valid = 0, n_badk = 0, n_badr = 0, n_begin = 0;
  uint64_t ts_min = kU64Max, ts_max = 0;
  uint64_t ctx_min = kU64Max, ctx_max = 0;
  bool bad = false;  // a record earlier than the one before it, both of one context
  // Each wave takes 4 x 64 consecutive records per step (4 loads in flight
  // per lane); every lane of a wave iterates the same number of times.
  constexpr int kPer = 4;
  const uint64_t stride = (uint64_t)gridDim.x * 256 * kPer;
  const uint32_t lane = threadIdx.x & 63;
  const uint64_t first = ((uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * (64 * kPer);
  static_assert(kPer * 64 == kChunk, "a wave step is one chunk");
  uint64_t wave_runs = 0;
  // this wave's run list and chunk table words: staged, then written out
  const uint32_t wv = threadIdx.x >> 6;
  const ChunkWaves cw = chunk_waves((a.n + kChunk - 1) / kChunk, gridDim.x * 4);
  const uint64_t slot0 = wave_slot0(cw, (uint64_t)blockIdx.x * 4 + wv);
  uint64_t* const list = a.runs_raw + slot0 * kChunk;
  uint32_t n_out = 0, n_staged = 0;  // runs written out, runs staged
  uint32_t c_out = 0, c_staged = 0;  // chunk words written out, staged
  auto wave_sync = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  auto flush_runs = [&] {
    wave_sync();
    for (uint32_t i = lane; i < n_staged; i += 64) list[n_out + i] = s_stage[wv][i];
    n_out += n_staged;
    n_staged = 0;
    wave_sync();
  };
  auto flush_chunks = [&] {
    wave_sync();
    for (uint32_t i = lane; i < c_staged; i += 64) a.chunk_runs[slot0 + c_out + i] = s_ctab[wv][i];
    c_out += c_staged;
    c_staged = 0;
    wave_sync();
  };
  uint4 nr_[kPer];  // the next chunk, loaded while this one is processed
  auto issue = [&](uint64_t b) {
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const uint64_t i = b + (uint64_t)j * 64 + lane;
      nr_[j] = a.rec[i < a.n ? i : a.n - 1];
    }
  };
  if (first < a.n) issue(first);
  for (uint64_t base = first; base < a.n; base += stride) {
    uint4 r[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) r[j] = nr_[j];
    if (base + stride < a.n) issue(base + stride);
    uint32_t cx[kPer];
    bool inr[kPer], vl[kPer];
    const uint32_t rem = a.n - base < (uint64_t)kChunk ? (uint32_t)(a.n - base) : (uint32_t)kChunk;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const uint32_t kind = (r[j].w >> 16) & 0xFFu;
      const uint32_t region = r[j].w & 0xFFFFu;
      const bool kind_ok = kind == 1 || kind == 2;
      cx[j] = r[j].z;
      inr[j] = 64u * j + lane < rem;
      vl[j] = inr[j] && kind_ok && region < a.R;
      n_badk += (uint64_t)__popcll(__ballot(inr[j] && !kind_ok));
      n_badr += (uint64_t)__popcll(__ballot(inr[j] && kind_ok && region >= a.R));
      n_begin += (uint64_t)__popcll(__ballot(vl[j] && kind == 1));
      const uint64_t ts = (uint64_t)r[j].x | ((uint64_t)r[j].y << 32);
      ts_min = vl[j] && ts < ts_min ? ts : ts_min;
      ts_max = vl[j] && ts > ts_max ? ts : ts_max;
    }
    // One row of the chunk against the records before them (an invalid one
    // counts as time 0): enough to notice buffers that arrive shuffled;
    // whatever it misses the check after the sort by context finds.
    {
      const uint32_t tx = vl[0] ? r[0].x : 0u, ty = vl[0] ? r[0].y : 0u;
      const uint64_t ts = ((uint64_t)ty << 32) | tx;
      const uint64_t tp = ((uint64_t)lane_prev(ty, ty) << 32) | lane_prev(tx, tx);
      bad |= vl[0] && lane_prev(cx[0], cx[0]) == cx[0] && tp > ts;
    }
    // runs of one context in this chunk
    uint64_t H[4], V[4];
    chunk_masks(cx, inr, vl, H, V);
    uint32_t nr = 0, nvc = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      nr += (uint32_t)__popcll(H[j]);
      nvc += (uint32_t)__popcll(V[j]);
    }
    n_valid += nvc;
    if (n_staged + nr > kStageRuns) flush_runs();
    if (c_staged == kStageChunks) flush_chunks();
    // per row (wave-uniform): heads and valid records before it, and the
    // valid records before the first head of the rows after it (all of the
    // chunk's if none)
    uint32_t hbase[kPer], vbase[kPer], vnext[kPer];
    {
      uint32_t hb = 0, vb = 0;
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        hbase[j] = hb;
        vbase[j] = vb;
        hb += (uint32_t)__popcll(H[j]);
        vb += (uint32_t)__popcll(V[j]);
      }
      uint32_t vn = vb;
#pragma unroll
      for (int j = kPer - 1; j >= 0; --j) {
        vnext[j] = vn;
        if (H[j]) {
          const uint32_t b = (uint32_t)__ffsll((unsigned long long)H[j]) - 1u;
          vn = vbase[j] + (uint32_t)__popcll(V[j] & ((1ull << b) - 1ull));
        }
      }
    }
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      if (!((H[j] >> lane) & 1ull)) continue;
      const uint32_t li = hbase[j] + __builtin_amdgcn_mbcnt_hi((uint32_t)(H[j] >> 32),
                                                                __builtin_amdgcn_mbcnt_lo((uint32_t)H[j], 0u));
      const uint32_t vp = vbase[j] + __builtin_amdgcn_mbcnt_hi((uint32_t)(V[j] >> 32),
                                                                __builtin_amdgcn_mbcnt_lo((uint32_t)V[j], 0u));
      // the next head in this row (two shifts: lane + 1 may be 64)
      const uint64_t later = H[j] & ((~0ull << lane) << 1);
      uint32_t vq = vnext[j];
      if (later) {
        const uint32_t b = (uint32_t)__ffsll((unsigned long long)later) - 1u;
        vq = vbase[j] + (uint32_t)__popcll(V[j] & ((1ull << b) - 1ull));
      }
      const uint32_t cnt = vq - vp;
      s_stage[wv][n_staged + li] = (uint64_t)cx[j] | ((uint64_t)cnt << 32);
      if (cnt) {
        // the context range, and the context digit histograms, per run
        ctx_min = cx[j] < ctx_min ? cx[j] : ctx_min;
        ctx_max = cx[j] > ctx_max ? cx[j] : ctx_max;
        atomicAdd(&s_hist[0][cx[j] & 0xFFu], cnt);
        // The runs of a row with many mostly agree in the higher digits: one
        // lane then adds their records (those after the first run's start, up
        // to the next row's first head).  An add per run on one address takes
        // the lanes one after another: with runs of one record each, as in a
        // trace of 2^24 records drained one by one, the kernel took 196 us,
        // this way 120.
        const uint32_t hi = cx[j] >> 8, hi0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)hi);
        uint32_t add = cnt;
        if (__popcll(H[j]) > kFewRuns && __ballot(hi != hi0) == 0) {
          const uint32_t v0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)vp);
          add = lane == (uint32_t)__builtin_ctzll(__ballot(true)) ? vnext[j] - v0 : 0u;
        }
        if (add) {
#pragma unroll
          for (int d = 0; d < 3; ++d) atomicAdd(&s_hist[d + 1][(hi >> (8 * d)) & 0xFFu], add);
        }
      }
    }
    if (lane == 0) s_ctab[wv][c_staged] = nr | ((n_out + n_staged) << kChunkCountBits);
    ++c_staged;
    n_staged += nr;
    wave_runs += nr;
  }
  if (n_staged) flush_runs();
  if (c_staged) flush_chunks();
  ts_min = wave_min(ts_min);
  ts_max = wave_max(ts_max);
  const uint64_t cmin = wave_min(ctx_min);
  const uint64_t cmax = wave_max(ctx_max);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0 && wave_runs) atomicAdd(&s_runs, (unsigned long long)wave_runs);
  if ((threadIdx.x & 63) == 0) {
    s_red[w][0] = n_valid;
    s_red[w][1] = n_badk;
    s_red[w][2] = n_badr;
    s_red[w][3] = n_begin;
    s_red[w][4] = ts_min;
    s_red[w][5] = ts_max;
    s_red[w][6] = cmin;
    s_red[w][7] = cmax;
  }
  __syncthreads();
  // The block's counters, several lanes of one wave in one request where they
  // do the same to one line: such requests are served one after another, ten
  // from each of a thousand blocks at the end of the kernel.
  if (threadIdx.x < 9) {
    const uint32_t k = threadIdx.x;
    // 0..3: valid, bad kind, bad region, BEGIN; 4: END; 5, 6: ts and context
    // minima, 7, 8: maxima
    constexpr int slot[9] = {ARGUS_C_N_VALID, ARGUS_C_N_BAD_KIND, ARGUS_C_N_BAD_REGION, ARGUS_C_N_BEGIN, ARGUS_C_N_END,
                             ARGUS_C_TS_MIN,  ARGUS_C_CTX_MIN,    ARGUS_C_TS_MAX,       ARGUS_C_CTX_MAX};
    constexpr int col[9] = {0, 1, 2, 3, 0, 4, 6, 5, 7};
    uint64_t v = k == 5 || k == 6 ? kU64Max : 0ull, valid = 0;
    for (int q = 0; q < 4; ++q) {
      const uint64_t x = s_red[q][col[k]];
      if (k < 5) v += x - (k == 4 ? s_red[q][3] : 0ull);
      else if (k < 7) v = x < v ? x : v;
      else v = x > v ? x : v;
      valid += s_red[q][0];
    }
    unsigned long long* c = (unsigned long long*)&a.counters[slot[k]];
    if (k < 5) {
      if (v) atomicAdd(c, v);
    } else if (valid) {
      if (k < 7) atomicMin(c, v);
      else atomicMax(c, v);
    }
    if (k == 0 && s_runs) atomicAdd((unsigned long long*)&a.plan->n_runs, s_runs);
  }
  for (int i = threadIdx.x; i < 4 * kRadixBins; i += 256) {
    const uint32_t h = (&s_hist[0][0])[i];
    if (h) atomicAdd(&a.hist[i], h);
  }
  if (__syncthreads_or(bad) && threadIdx.x == 0) st_agent(&a.plan->unsorted, 1u);
  if (last_arrival(a.ctrs, kArIngest, gridDim.x, &s_slot) && threadIdx.x == 0) make_plan(a);
}

hipError_t launch_ingest(const RunArgs& a, hipStream_t s) {
  IngestArgs ia{(const uint4*)a.rec, a.n, a.R, a.out.d_counters, a.w.rec_hist, a.w.plan,
                a.w.key[1], a.w.chunk_runs, a.w.tile_ctr,
                (a.flags & ARGUS_FORCE_RECORD_RADIX) ? 1u : 0u, a.w.run_cap};
  // up to 1024 blocks: four waves per SIMD, each streaming many chunks
  // (measured faster than more or fewer on the 2^28-record trace)
  hipLaunchKernelGGL(k_ingest, dim3(ingest_blocks(a.n)), dim3(256), 0, s, ia);
  return hipGetLastError();
}

// ------------------------------------------------------- the run scatter

struct RunScatterArgs {
  DevPlan* plan;
  const uint4* rec;
  uint64_t n;
  uint32_t R;
  const uint32_t* run_base;
  const uint32_t* run_pos;
  uint64_t* key;  // key[0]
  uint32_t* pay;  // pay[0]
  uint64_t* counters;
  const uint8_t* region_class;
  uint32_t K, G, shift;
  // for the tile sums: which runs start their context
  const uint32_t* run_cnt;
};

// Every valid record to its run's position plus its rank among the run's
// valid records, packed as in the radix path (key (ctx - ctx_min) << ts_bits
// | (ts - ts_min), payload region | (kind - 1) << 16 | class << 24).  One
// wave per chunk, as in the ingest.  For the tile sums it also marks the
// first record of each context in its payload (kPayStart) and checks that
// the valid records of a context in the chunk are in time order
// (k_tsum checks where runs meet).
__global__ __launch_bounds__(256) void k_runs_scatter(RunScatterArgs a) {
  DevPlan* p = a.plan;
  if (!p->runs || p->early) return;
  __shared__ uint8_t s_cls[kClsLds];
  // per wave and run of the chunk: first position minus its head's rank,
  // first position, valid records | starts its context << 31
  __shared__ uint32_t s_roff[4][kChunk], s_rpos[4][kChunk], s_rcnt[4][kChunk];
  // per wave and chunk position: timestamp and context
  __shared__ uint64_t s_ts[4][kChunk];
  __shared__ uint32_t s_cx[4][kChunk];
  const uint32_t wv = threadIdx.x >> 6;
  bool bad = false;
  const bool cls_lds = a.K && a.R <= kClsLds;
  if (cls_lds)
    for (uint32_t r = threadIdx.x; r < a.R; r += 256) s_cls[r] = a.region_class[r];
  __syncthreads();
  const KeySpace ks = p->rec;
  const uint64_t nv = p->n_valid;
  constexpr int kPer = 4;
  const uint64_t stride = (uint64_t)gridDim.x * 256 * kPer;
  const uint32_t lane = threadIdx.x & 63;
  const uint64_t first = ((uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * (64 * kPer);
  // the next chunk's records and run base are loaded while this one is written
  uint4 nr_[kPer];
  uint32_t nrb = 0;
  auto issue = [&](uint64_t b) {
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const uint64_t i = b + (uint64_t)j * 64 + lane;
      nr_[j] = a.rec[i < a.n ? i : a.n - 1];
    }
    nrb = a.run_base[b / kChunk];
  };
  if (first < a.n) issue(first);
  for (uint64_t base = first; base < a.n; base += stride) {
    uint4 r[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) r[j] = nr_[j];
    const uint32_t rb = nrb;
    if (base + stride < a.n) issue(base + stride);
    uint32_t cx[kPer];
    bool inr[kPer], vl[kPer];
    const uint32_t rem = a.n - base < (uint64_t)kChunk ? (uint32_t)(a.n - base) : (uint32_t)kChunk;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const uint32_t kind = (r[j].w >> 16) & 0xFFu;
      cx[j] = r[j].z;
      inr[j] = 64u * j + lane < rem;
      vl[j] = inr[j] && (kind == 1 || kind == 2) && (r[j].w & 0xFFFFu) < a.R;
    }
    // the positions, context-start flags and sizes of the chunk's first 64
    // runs, one per lane, in flight while the masks are built
    const uint64_t n_runs = p->n_runs;
    const uint32_t prid = rb + lane;
    const bool pin = prid < n_runs;
    const uint32_t pre_word = pin ? a.run_pos[prid] : 0u;
    const uint32_t pre_pos = pre_word & kRunPosMask, pre_head = pre_word >> 31;
    const uint32_t pre_cnt = pin ? a.run_cnt[prid] : 0u;
    uint64_t H[4], V[4];
    chunk_masks(cx, inr, vl, H, V);
    // Run of each record (heads before it, inclusive) and its rank among the
    // chunk's valid records; each run head publishes its run's first
    // position minus its own rank in the wave's LDS slots.  A chunk whose
    // in-range records are all valid (the usual case) needs no more LDS:
    // its order check and run bounds come from neighbouring lanes.
    uint64_t IR[kPer];
    bool all_valid = true;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      IR[j] = __ballot(inr[j]);
      all_valid = all_valid && V[j] == IR[j];
    }
    uint32_t li[kPer], vr[kPer], hflag[kPer];
    int32_t lastv[kPer];  // last valid chunk position in earlier rows (-1: none)
    uint32_t hb = 0, vb = 0;
    int32_t lv = -1;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const uint32_t hr = hb + (uint32_t)__builtin_amdgcn_mbcnt_hi(
                                   (uint32_t)(H[j] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)H[j], 0u));
      vr[j] = vb + (uint32_t)__builtin_amdgcn_mbcnt_hi(
                       (uint32_t)(V[j] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)V[j], 0u));
      const bool head = (H[j] >> lane) & 1ull;
      const uint32_t sp = (uint32_t)__shfl((int)pre_pos, (int)(hr & 63u));
      const uint32_t sh = (uint32_t)__shfl((int)pre_head, (int)(hr & 63u));
      const uint32_t sc = (uint32_t)__shfl((int)pre_cnt, (int)(hr & 63u));
      hflag[j] = 0;
      if (head) {
        const uint32_t rid = rb + hr;
        const bool near = hr < 64u;
        const uint32_t far_word = near ? 0u : a.run_pos[rid];
        const uint32_t rp = near ? sp : (far_word & kRunPosMask);
        s_roff[wv][hr] = rp - vr[j];
        hflag[j] = near ? sh : far_word >> 31;
        if (!all_valid) {
          s_rpos[wv][hr] = rp;
          s_rcnt[wv][hr] = (near ? sc : a.run_cnt[rid]) | (hflag[j] << 31);
        }
      }
      li[j] = hr + (head ? 1u : 0u) - 1u;
      if (!all_valid) {
        s_ts[wv][64 * j + lane] = (uint64_t)r[j].x | ((uint64_t)r[j].y << 32);
        s_cx[wv][64 * j + lane] = cx[j];
        lastv[j] = lv;
        if (V[j]) lv = 64 * j + 63 - (int32_t)__clzll((long long)V[j]);
      }
      hb += (uint32_t)__popcll(H[j]);
      vb += (uint32_t)__popcll(V[j]);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const uint64_t ts = (uint64_t)r[j].x | ((uint64_t)r[j].y << 32);
      bool first_v = false, starts = false;
      if (all_valid) {
        // previous record: the previous lane, or the last lane of the row before
        // (lane 0 of the first row starts a run: its value is not used)
        const int jp = j > 0 ? j - 1 : 0;
        const uint32_t fx = (uint32_t)__builtin_amdgcn_readlane((int)r[jp].x, 63);
        const uint32_t fy = (uint32_t)__builtin_amdgcn_readlane((int)r[jp].y, 63);
        const uint64_t tp = ((uint64_t)lane_prev(r[j].y, fy) << 32) | lane_prev(r[j].x, fx);
        const bool h = (H[j] >> lane) & 1ull;
        if (vl[j] && !h && tp > ts) bad = true;
        first_v = h;
        starts = h && hflag[j];
      }
      if (!vl[j]) continue;
      const uint32_t run = li[j];
      const uint64_t out = (uint64_t)(uint32_t)(s_roff[wv][run] + vr[j]);
      if (out >= nv) {
        flag_internal_error(a.counters, 1024);
        continue;
      }
      if (!all_valid) {
        // the previous valid record of the chunk, if it has the same context
        const uint64_t below = V[j] & ((1ull << lane) - 1ull);
        const int32_t pv = below ? 64 * j + 63 - (int32_t)__clzll((long long)below) : lastv[j];
        if (pv >= 0 && s_cx[wv][pv] == cx[j] && s_ts[wv][pv] > ts) bad = true;
        const uint32_t rpos = s_rpos[wv][run], rc = s_rcnt[wv][run];
        first_v = (uint32_t)out == rpos;
        starts = first_v && (rc >> 31);
      }
      const uint64_t rel = (uint64_t)(cx[j] - (uint32_t)ks.ctx_min);
      a.key[out] = (ks.ts_bits >= 64 ? 0ull : (rel << ks.ts_bits)) | (ts - ks.ts_min);
      const uint32_t region = r[j].w & 0xFFFFu;
      uint32_t cls = 0xFFu;
      if (swept_ctx(cx[j], a.K, a.G, a.shift)) cls = cls_lds ? s_cls[region] : a.region_class[region];
      a.pay[out] = pack_payload(region, (r[j].w >> 16) & 0xFFu, cls) | (starts ? kPayStart : 0u);
    }
  }
  if (__syncthreads_or(bad) && threadIdx.x == 0) p->unsorted = 1;
}

hipError_t launch_runs_scatter(const RunArgs& a, hipStream_t s) {
  RunScatterArgs r{a.w.plan, (const uint4*)a.rec, a.n, a.R, a.w.run_base, a.w.run_pos,
                   a.w.key[0], a.w.pay[0], a.out.d_counters, a.region_class, a.K, a.G, a.shift,
                   a.w.run_cnt};
  // 1280 blocks, five per compute unit (as many as the LDS holds), measured
  // fastest: more loads in flight than with 1024 or fewer
  uint64_t blocks = ceil_div(a.n, 256 * 4 * 4);
  if (blocks > 1280) blocks = 1280;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_runs_scatter, dim3((uint32_t)blocks), dim3(256), 0, s, r);
  return hipGetLastError();
}

// ------------------------------------------------------------- tile sums

static uint32_t tsum_blocks(const RunArgs& a) {
  uint64_t blocks = a.w.match_tiles;
  if (blocks > kMaxScanBlocks) blocks = kMaxScanBlocks;
  return blocks < 1 ? 1u : (uint32_t)blocks;
}

TsumArgs tsum_args(const RunArgs& a) {
  TsumArgs t{};
  t.plan = a.w.plan;
  for (int b = 0; b < 2; ++b) {
    t.key[b] = a.w.key[b];
    t.pay[b] = a.w.pay[b];
    t.ctxw[b] = a.w.ctxw[b];
  }
  t.tsum = a.w.tsum;
  t.bsum = a.w.bsum;
  t.carry = a.w.carry;
  t.nblk = tsum_blocks(a);
  t.direct = a.w.match_tiles <= kMaxScanBlocks ? 1u : 0u;
  t.run_cnt = a.w.run_cnt;
  t.run_pos = a.w.run_pos;
  t.ctrs = a.w.tile_ctr;
  t.counters = a.out.d_counters;
  return t;
}

// The tile sums after the sort by context, with the check that it left
// (ctx, ts) non-decreasing; if not (some context was out of time order in
// the input) k_full_sort does both again.  After the run scatter, which has
// checked the order inside each chunk, the check is where runs meet: the
// first record of each run against the record before it in sorted order,
// when both belong to one context.  Block b takes the b-th contiguous run of
// tiles; the last block to finish scans the runs.
__global__ __launch_bounds__(256, 8) void k_tsum(TsumArgs a) {
  DevPlan* p = a.plan;
  if (p->early) return;
  __shared__ TsumShared s;
  const KeySpace ks = p->rec;
  const uint64_t nv = p->n_valid;
  bool bad = false;
  if (p->runs) {
    const uint64_t n_runs = p->n_runs;
    const uint32_t tb = ks.ts_bits;
    const uint64_t* key = a.key[0];
    const uint64_t stride = (uint64_t)gridDim.x * 256;
    for (uint64_t r = (uint64_t)blockIdx.x * 256 + threadIdx.x; r < n_runs; r += stride) {
      const uint32_t pos = a.run_pos[r] & kRunPosMask;
      if (a.run_cnt[r] == 0 || pos == 0) continue;
      const uint64_t k0 = key[pos - 1], k1 = key[pos];
      // same context (key bits above ts_bits) and time going back
      if ((tb >= 64 || (k0 >> tb) == (k1 >> tb)) && k0 > k1) bad = true;
    }
    tsum_codes_run(a, s, nv, blockIdx.x);
  } else {
    bad = tsum_run<true, 256>(a, s, ks, nv, p->rec_final, blockIdx.x);
  }
  if (__syncthreads_or(bad) && threadIdx.x == 0) p->unsorted = 1;
  if (last_arrival(a.ctrs, kArTsum, gridDim.x, &s.ticket)) mscan_top<256>(a, s, ceil_div(nv, kMatchTile));
}

hipError_t launch_tsum(const RunArgs& a, hipStream_t s) {
  const TsumArgs t = tsum_args(a);
  hipLaunchKernelGGL(k_tsum, dim3(t.nblk), dim3(256), 0, s, t);
  return hipGetLastError();
}

struct MscanArgs {
  const DevPlan* plan;
  const uint64_t* tsum;
  const BlockSum* bsum;  // what comes before each run of tiles
  TileCarry* carry;
};

// Entering values of every matching tile where the runs are longer than one
// tile: block b scans its run of tile sums (256 at a time) after what comes
// before the run.
__global__ __launch_bounds__(256) void k_mscan_tiles(MscanArgs a) {
  __shared__ Fn s_wfn[4];
  __shared__ uint32_t s_wnb[4], s_wnh[4];
  const uint64_t tiles = a.plan->match_tiles;
  const uint64_t per = ceil_div(tiles, gridDim.x);
  const uint64_t t0 = (uint64_t)blockIdx.x * per, t1 = t0 + per < tiles ? t0 + per : tiles;
  const uint32_t t = threadIdx.x, lane = t & 63, w = t >> 6;
  const BlockSum b0 = ld_bsum(&a.bsum[blockIdx.x]);
  Fn run = b0.f;
  uint64_t run_nb = b0.nb, run_nh = b0.nh;
  for (uint64_t c0 = t0; c0 < t1; c0 += 256) {
    const uint64_t k = c0 + t;
    Fn g = fn_id();
    uint32_t nbh = 0;
    if (k < t1) unpack_tile_sum(a.tsum[k], &g, &nbh);
    const uint32_t nb = nbh & 0xFFFFu, nh = nbh >> 16;
    const Fn x = wave_scan_fn(g);
    const uint32_t xb = (uint32_t)wave_incl_scan32((int32_t)nb);
    const uint32_t xh = (uint32_t)wave_incl_scan32((int32_t)nh);
    if (lane == 63) {
      s_wfn[w] = x;
      s_wnb[w] = xb;
      s_wnh[w] = xh;
    }
    Fn ex = Fn{(uint32_t)__shfl_up((int)x.reset, 1), __shfl_up(x.a, 1), __shfl_up(x.c, 1)};
    if (lane == 0) ex = fn_id();
    __syncthreads();
    Fn pre = run, all = run;
    uint64_t pb = run_nb, ph = run_nh, ab = run_nb, ah = run_nh;
    for (uint32_t q = 0; q < 4; ++q) {
      if (q < w) {
        pre = compose(pre, s_wfn[q]);
        pb += s_wnb[q];
        ph += s_wnh[q];
      }
      all = compose(all, s_wfn[q]);
      ab += s_wnb[q];
      ah += s_wnh[q];
    }
    pre = compose(pre, ex);
    pb += xb - nb;
    ph += xh - nh;
    if (k < t1) {
      TileCarry c;
      c.s_in = (uint32_t)apply(pre, 0);
      c.hpre = (uint32_t)ph;
      c.nbpre = pb;
      a.carry[k] = c;
    }
    run = all;
    run_nb = ab;
    run_nh = ah;
    __syncthreads();
  }
}

hipError_t launch_mscan(const RunArgs& a, hipStream_t s) {
  const TsumArgs t = tsum_args(a);
  if (t.direct) return hipSuccess;
  MscanArgs m{a.w.plan, a.w.tsum, a.w.bsum, a.w.carry};
  hipLaunchKernelGGL(k_mscan_tiles, dim3(t.nblk), dim3(256), 0, s, m);
  return hipGetLastError();
}

}  // namespace argus
