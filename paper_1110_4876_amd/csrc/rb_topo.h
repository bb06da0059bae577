// rb_topo.h -- the level ranges of the cells that start and end at a slot of
// the sorted keys, and a tile's counts of them (k_topo.hip explains the tree).
#pragma once
#include "rb_internal.h"

struct TopoRange {
  int lo_s, hi_s, lo_e, hi_e;  // start and end level ranges (empty if lo > hi)
};

__device__ __forceinline__ TopoRange rb_topo_range(const uint64_t *__restrict__ key,
                                                   uint32_t st, uint32_t i, uint32_t nl, int L,
                                                   int nvirt) {
  const uint64_t *k = key + st;
  int lf = 0;
  if (nl > (uint32_t)L) {
    int D = 0;
    const uint32_t jlo = (i >= (uint32_t)L) ? i - L : 0u;
    const uint32_t jhi = (i <= nl - 1 - L) ? i : nl - 1 - L;
    for (uint32_t j = jlo; j <= jhi; ++j) {
      const int v = rb_lcp(k[j], k[j + L]);
      D = v > D ? v : D;
    }
    lf = D + 1 < RB_DEPTH ? D + 1 : RB_DEPTH;
  }
  // the cells above the root boxes are never leaves: every occupied one
  // exists down to its root box (the root of that box's own tree)
  if (lf < nvirt) lf = nvirt;
  TopoRange r;
  r.lo_s = (i == 0) ? 0 : rb_lcp(k[i - 1], k[i]) + 1;
  r.hi_s = lf;
  r.lo_e = (i + 1 == nl) ? 0 : rb_lcp(k[i], k[i + 1]) + 1;
  r.hi_e = lf;
  return r;
}

// the levels at which any lane of the wave starts or ends a node
__device__ __forceinline__ void rb_topo_levels(const TopoRange &tr, bool valid, int &lmin,
                                               int &lmax) {
  lmin = valid ? min(tr.lo_s, tr.lo_e) : RB_NLEV;
  lmax = valid ? max(tr.hi_s, tr.hi_e) : -1;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    lmin = min(lmin, __shfl_xor(lmin, d, 64));
    lmax = max(lmax, __shfl_xor(lmax, d, 64));
  }
}

// live keys of a patch's slots [st, en): the dead ones sort last
__device__ __forceinline__ uint32_t rb_live_keys(const uint64_t *__restrict__ key, uint32_t st,
                                                 uint32_t en) {
  if (en == st) return 0u;
  if (key[en - 1] != RB_KEY_DEAD) return en - st;
  uint32_t lo = st, hi = en - 1;  // the first dead one
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if (key[mid] == RB_KEY_DEAD) hi = mid; else lo = mid + 1;
  }
  return lo - st;
}

// What the counts of a tile are read from and written to.
struct TopoCount {
  const uint32_t *tile_start, *tile_end, *tile_patch;
  uint32_t n_tiles;
  int L, nvirt;
  uint32_t *cnt;
};

// Starts and ends of nodes per level in tile b (slots of patch p, whose first
// is st, nl of them live), by one wave.
__device__ __forceinline__ void rb_topo_count_tile(const TopoCount &t, uint32_t b, uint32_t lane,
                                                   const uint64_t *__restrict__ key, uint32_t st,
                                                   uint32_t nl) {
  const uint32_t s0 = t.tile_start[b], s1 = t.tile_end[b];
  uint32_t cs = 0, ce = 0;  // lane l < 22 keeps the counts of level l
  for (uint32_t r0 = s0; r0 < s1; r0 += 64) {
    const uint32_t s = r0 + lane;
    const bool valid = s < s1 && (s - st) < nl;
    TopoRange tr = {1, 0, 1, 0};
    if (valid) tr = rb_topo_range(key, st, s - st, nl, t.L, t.nvirt);
    int lmin, lmax;
    rb_topo_levels(tr, valid, lmin, lmax);
#pragma unroll
    for (int l = 0; l < RB_NLEV; ++l) {
      if (l < lmin || l > lmax) continue;  // uniform: nothing starts or ends here
      const uint32_t ns = (uint32_t)__popcll(__ballot(l >= tr.lo_s && l <= tr.hi_s));
      const uint32_t ne = (uint32_t)__popcll(__ballot(l >= tr.lo_e && l <= tr.hi_e));
      if (lane == (uint32_t)l) { cs += ns; ce += ne; }
    }
  }
  if (lane < RB_NLEV) {
    // by level, or by tile where k_topo_write adds the tiles up itself
    const size_t at = t.n_tiles <= RB_TOPO_FEW ? (size_t)b * 2 * RB_NLEV + lane
                                               : (size_t)lane * t.n_tiles + b;
    const size_t ends = t.n_tiles <= RB_TOPO_FEW ? RB_NLEV : (size_t)RB_NLEV * t.n_tiles;
    t.cnt[at] = cs;
    t.cnt[at + ends] = ce;
  }
}

inline TopoCount rb_topo_tiles(const rb_ctx *c) {
  return {c->d_tile_start, c->d_tile_end, c->d_tile_patch, c->n_tiles, c->p.leaf_size,
          (int)c->h_patch[0].nvirt, c->d_cnt};
}
