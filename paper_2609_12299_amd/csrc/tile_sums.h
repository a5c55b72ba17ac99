// tile_sums.h -- the depth map, BEGINs and context starts of each matching
// tile (2048 consecutive sorted records), from which a scan gives every
// tile's entering values, so that matching needs no look-back.
#pragma once

#include "chain.h"

namespace argus {

struct TsumArgs {
  DevPlan* plan;
  const uint64_t* key[2];
  const uint32_t* pay[2];
  const uint32_t* ctxw[2];
  uint64_t* tsum;     // [match tiles]
  BlockSum* bsum;     // [nblk]: each run of tiles composed, then what comes before it
  TileCarry* carry;   // written here when a run is one tile (direct), else by k_mscan_tiles
  uint32_t nblk;      // runs of tiles
  uint32_t direct;
  const uint32_t* run_cnt;  // after the run scatter: see k_tsum
  const uint32_t* run_pos;
  uint32_t* ctrs;
  uint64_t* counters;
};

// Run sums pass from block to block within a kernel, as two words: c and a
// (c >= 0; the reset flag in its top bit), starts and BEGINs.
ARGUS_DEV void st_bsum(BlockSum* p, const BlockSum& b) {
  uint64_t* w = (uint64_t*)p;
  st_agent(&w[0], ((uint64_t)((uint32_t)b.f.c | (b.f.reset << 31)) << 32) | (uint32_t)b.f.a);
  st_agent(&w[1], ((uint64_t)b.nh << 32) | b.nb);
}
ARGUS_DEV BlockSum unpack_bsum(uint64_t u, uint64_t v) {
  BlockSum b;
  b.f.reset = (uint32_t)(u >> 63);
  b.f.a = (int32_t)(uint32_t)u;
  b.f.c = (int32_t)((uint32_t)(u >> 32) & 0x7FFFFFFFu);
  b.nb = (uint32_t)v;
  b.nh = (uint32_t)(v >> 32);
  return b;
}
ARGUS_DEV BlockSum ld_bsum(const BlockSum* p) {
  const uint64_t* w = (const uint64_t*)p;
  return unpack_bsum(ld_agent(&w[0]), ld_agent(&w[1]));
}

struct TsumShared {
  Fn wfn[8];
  uint32_t wnb[8], wnh[8];
  uint32_t ticket;
  __align__(8) uint8_t code[4][kMatchTile / 4];  // per wave: 4 records per byte
};

// Run vb of the tiles (the vb-th contiguous share of a.nblk): per tile the
// map from the depth before it to the depth after it, its BEGINs and its
// context starts; the run composed.  CHECK also reports (per thread) whether
// two neighbouring records are out of (ctx, ts) order.
template <bool CHECK, int NT>
__device__ __forceinline__ bool tsum_run(const TsumArgs& a, TsumShared& s, const KeySpace& ks, uint64_t nv,
                                         uint32_t buf, uint32_t vb) {
  constexpr int IT = kMatchTile / NT;  // consecutive records per thread
  const uint64_t tiles = ceil_div(nv, kMatchTile);
  const uint64_t* key = a.key[buf];
  const uint32_t* pay = a.pay[buf];
  const uint32_t* cw = a.ctxw[buf];
  const bool wide = ks.wide != 0;
  const uint32_t tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const uint32_t p0 = tid * IT;
  auto ctx_of = [&](uint64_t i, uint64_t k) -> uint32_t {
    return wide ? cw[i] : (ks.ts_bits >= 64 ? 0u : (uint32_t)(k >> ks.ts_bits));
  };
  bool bad = false;
  const uint64_t per = ceil_div(tiles, a.nblk);
  const uint64_t t0 = (uint64_t)vb * per, t1 = t0 + per < tiles ? t0 + per : tiles;
  Fn run = fn_id();
  uint32_t run_nb = 0, run_nh = 0;
  for (uint64_t tile = t0; tile < t1; ++tile) {
    const uint64_t base = tile * kMatchTile;
    const uint32_t cnt = nv - base < (uint64_t)kMatchTile ? (uint32_t)(nv - base) : (uint32_t)kMatchTile;
    uint64_t k[IT];
    uint32_t c[IT], kind = 0, fv = 0;
    if (p0 + IT <= cnt) {
      const uint4* k4 = (const uint4*)(key + base + p0);
#pragma unroll
      for (int q = 0; q < IT / 2; ++q) {
        const uint4 v = k4[q];
        k[2 * q] = (uint64_t)v.x | ((uint64_t)v.y << 32);
        k[2 * q + 1] = (uint64_t)v.z | ((uint64_t)v.w << 32);
      }
      const uint4* p4 = (const uint4*)(pay + base + p0);
#pragma unroll
      for (int q = 0; q < IT / 4; ++q) {
        const uint4 v = p4[q];
        kind |= ((v.x >> 16) & 1u) << (4 * q) | ((v.y >> 16) & 1u) << (4 * q + 1) |
                ((v.z >> 16) & 1u) << (4 * q + 2) | ((v.w >> 16) & 1u) << (4 * q + 3);
      }
      fv = (1u << IT) - 1u;
    } else {
#pragma unroll
      for (int i = 0; i < IT; ++i) {
        const uint32_t q = p0 + i;
        k[i] = q < cnt ? key[base + q] : 0ull;
        if (q < cnt) {
          kind |= ((pay[base + q] >> 16) & 1u) << i;
          fv |= 1u << i;
        }
      }
    }
#pragma unroll
    for (int i = 0; i < IT; ++i) c[i] = ctx_of(base + p0 + i < nv ? base + p0 + i : 0, k[i]);
    // the record before this thread's first one
    uint32_t c_prev = (uint32_t)__shfl_up((int)c[IT - 1], 1);
    uint64_t k_prev = __shfl_up(k[IT - 1], 1);
    bool has_prev = true;
    if (lane == 0) {
      const uint64_t pp = base + p0;
      has_prev = pp > 0 && pp <= nv;
      if (has_prev) {
        k_prev = key[pp - 1];
        c_prev = ctx_of(pp - 1, k_prev);
      }
    }
    Fn f = fn_id();
    uint32_t nb = 0, nh = 0;
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      if (!((fv >> i) & 1u)) continue;
      const bool hp = i > 0 || has_prev;
      const uint32_t cp = i > 0 ? c[i - 1] : c_prev;
      const uint64_t kp = i > 0 ? k[i - 1] : k_prev;
      const bool head = !hp || cp != c[i];
      if (CHECK && hp) bad |= wide ? (cp > c[i] || (cp == c[i] && kp > k[i])) : kp > k[i];
      const bool isb = ((kind >> i) & 1u) == 0;
      const Fn e = head ? Fn{1u, 0, isb ? 1 : 0} : Fn{0u, isb ? 1 : -1, 0};
      f = compose(f, e);
      nb += isb;
      nh += head;
    }
    // tile sums: wave scans, then the waves in order
    const Fn x = wave_scan_fn(f);
    const uint32_t nbx = (uint32_t)wave_incl_scan32((int32_t)(nb | (nh << 16)));
    if (lane == 63) {
      s.wfn[w] = x;
      s.wnb[w] = nbx;
    }
    __syncthreads();
    if (tid == 0) {
      Fn all = fn_id();
      uint32_t nball = 0;
      for (int q = 0; q < NT / 64; ++q) {
        all = compose(all, s.wfn[q]);
        nball += s.wnb[q];
      }
      a.tsum[tile] = pack_tile_sum(all, nball);
      run = compose(run, all);
      run_nb += nball & 0xFFFFu;
      run_nh += nball >> 16;
    }
    __syncthreads();
  }
  if (tid == 0) st_bsum(&a.bsum[vb], BlockSum{run, run_nb, run_nh});
  return bad;
}

// The same sums from the payloads the run scatter wrote (kind and
// context-start bits), without the keys.  One wave per tile, the block's
// four waves on four consecutive tiles: the wave loads the tile's payloads
// contiguously, keeps two bits per record in LDS, and each lane then composes
// 32 consecutive records.
__device__ __forceinline__ void tsum_codes_run(const TsumArgs& a, TsumShared& s, uint64_t nv, uint32_t vb) {
  constexpr uint32_t kPerLane = kMatchTile / 64;  // 32
  const uint32_t* gpay = a.pay[0];
  const uint64_t tiles = ceil_div(nv, kMatchTile);
  const uint32_t tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const uint32_t p0 = lane * kPerLane;
  const uint64_t per = ceil_div(tiles, a.nblk);
  const uint64_t t0 = (uint64_t)vb * per, t1 = t0 + per < tiles ? t0 + per : tiles;
  Fn run = fn_id();
  uint32_t run_nb = 0, run_nh = 0;
  auto code_of = [](uint32_t v) -> uint32_t {
    return (((v >> 16) & 1u) ^ 1u) | ((v & kPayStart) ? 2u : 0u);  // BEGIN | start << 1
  };
  for (uint64_t tq = t0; tq < t1; tq += 4) {
    const uint64_t tile = tq + w;
    Fn f = fn_id();
    uint32_t nb = 0, nh = 0;
    if (tile < t1) {
      const uint64_t base = tile * kMatchTile;
      const uint32_t cnt = nv - base < (uint64_t)kMatchTile ? (uint32_t)(nv - base) : (uint32_t)kMatchTile;
      // a full tile (all but the last) loads its payloads in one batch; a
      // choice per load would make each wait for the one before
      uint4 u[kPerLane / 4];
      if (cnt == kMatchTile) {
#pragma unroll
        for (int q = 0; q < (int)kPerLane / 4; ++q)
          u[q] = *(const uint4*)(gpay + base + (uint32_t)q * 256u + 4u * lane);
      } else {
#pragma unroll
        for (int q = 0; q < (int)kPerLane / 4; ++q) {
          const uint32_t r0 = (uint32_t)q * 256u + 4u * lane;
          u[q].x = r0 < cnt ? gpay[base + r0] : 0u;
          u[q].y = r0 + 1 < cnt ? gpay[base + r0 + 1] : 0u;
          u[q].z = r0 + 2 < cnt ? gpay[base + r0 + 2] : 0u;
          u[q].w = r0 + 3 < cnt ? gpay[base + r0 + 3] : 0u;
        }
      }
#pragma unroll
      for (int q = 0; q < (int)kPerLane / 4; ++q) {
        const uint32_t r0 = (uint32_t)q * 256u + 4u * lane;
        s.code[w][r0 >> 2] = (uint8_t)(code_of(u[q].x) | code_of(u[q].y) << 2 |
                                       code_of(u[q].z) << 4 | code_of(u[q].w) << 6);
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      const uint64_t c = *(const uint64_t*)&s.code[w][p0 >> 2];
#pragma unroll
      for (int i = 0; i < (int)kPerLane; ++i) {
        if (p0 + (uint32_t)i >= cnt) break;
        const uint32_t ci = (uint32_t)(c >> (2 * i)) & 3u;
        const bool isb = ci & 1u, head = (ci >> 1) & 1u;
        const Fn e = head ? Fn{1u, 0, isb ? 1 : 0} : Fn{0u, isb ? 1 : -1, 0};
        f = compose(f, e);
        nb += isb;
        nh += head;
      }
    }
    const Fn x = wave_scan_fn(f);
    const uint32_t nbx = (uint32_t)wave_incl_scan32((int32_t)(nb | (nh << 16)));
    if (lane == 63) {
      if (tile < t1) a.tsum[tile] = pack_tile_sum(x, nbx);
      s.wfn[w] = x;
      s.wnb[w] = nbx;
    }
    __syncthreads();
    if (tid == 0) {
      for (int q = 0; q < 4; ++q) {
        run = compose(run, s.wfn[q]);  // identity for tiles past the run
        run_nb += s.wnb[q] & 0xFFFFu;
        run_nh += s.wnb[q] >> 16;
      }
    }
    __syncthreads();
  }
  if (tid == 0) st_bsum(&a.bsum[vb], BlockSum{run, run_nb, run_nh});
}

// By the last block to finish its run (each thread a contiguous stretch of
// the runs): overwrites each run's sum with the composition of everything
// before it, or, when every run is one tile, writes the tiles' entering
// values at once.
template <int NT>
__device__ __forceinline__ void mscan_top(const TsumArgs& a, TsumShared& s, uint64_t tiles) {
  const uint32_t t = threadIdx.x, lane = t & 63, w = t >> 6;
  constexpr uint32_t kPer = kMaxScanBlocks / NT;
  const uint32_t per = (a.nblk + NT - 1) / NT;
  const uint32_t k0 = t * per;
  // the thread's loads together, kept packed (all zero, which is the
  // identity, past its stretch)
  uint64_t u[kPer], v[kPer];
#pragma unroll
  for (uint32_t q = 0; q < kPer; ++q) {
    const uint64_t* w2 = (const uint64_t*)&a.bsum[q < per && k0 + q < a.nblk ? k0 + q : 0u];
    u[q] = ld_agent(&w2[0]);
    v[q] = ld_agent(&w2[1]);
  }
#pragma unroll
  for (uint32_t q = 0; q < kPer; ++q)
    if (!(q < per && k0 + q < a.nblk)) u[q] = v[q] = 0;
  Fn f = fn_id();
  uint32_t nb = 0, nh = 0;
#pragma unroll
  for (uint32_t q = 0; q < kPer; ++q) {
    const BlockSum b = unpack_bsum(u[q], v[q]);
    f = compose(f, b.f);
    nb += b.nb;
    nh += b.nh;
  }
  const Fn x = wave_scan_fn(f);
  const uint32_t xb = (uint32_t)wave_incl_scan32((int32_t)nb);
  const uint32_t xh = (uint32_t)wave_incl_scan32((int32_t)nh);
  if (lane == 63) {
    s.wfn[w] = x;
    s.wnb[w] = xb;
    s.wnh[w] = xh;
  }
  Fn ex = Fn{(uint32_t)__shfl_up((int)x.reset, 1), __shfl_up(x.a, 1), __shfl_up(x.c, 1)};
  if (lane == 0) ex = fn_id();
  __syncthreads();
  Fn pre = fn_id();
  uint32_t pb = xb - nb, ph = xh - nh;
  for (uint32_t q = 0; q < w; ++q) {
    pre = compose(pre, s.wfn[q]);
    pb += s.wnb[q];
    ph += s.wnh[q];
  }
  f = compose(pre, ex);
#pragma unroll
  for (uint32_t q = 0; q < kPer; ++q) {
    const uint32_t k = k0 + q;
    if (q < per && k < a.nblk) {
      if (!a.direct) st_bsum(&a.bsum[k], BlockSum{f, pb, ph});
      else if (k < tiles) a.carry[k] = TileCarry{(uint32_t)apply(f, 0), ph, pb};
    }
    const BlockSum b = unpack_bsum(u[q], v[q]);
    f = compose(f, b.f);
    pb += b.nb;
    ph += b.nh;
  }
}

TsumArgs tsum_args(const RunArgs& a);

}  // namespace argus
