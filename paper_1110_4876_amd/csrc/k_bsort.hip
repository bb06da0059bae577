// k_bsort.hip -- sort of (Morton key, slot) pairs for small systems by
// buckets of the top 12 key bits (the cells of octree level 4).
//
// Sorting by (key, slot) gives the stable order of the keys (ties keep the
// order of the slots), so the pieces below need not be stable themselves:
//   counting        -- the kernel that writes the keys counts them per
//                      (patch, bucket) (rb_bucket_add; bucket 4096 holds
//                      removed particles, whose all-ones key sorts last);
//   k_bsort_scan    -- per patch: bucket cursors, and segments: runs of
//                      whole buckets that start in the same window of 64
//                      slots (at most 127 keys), a bucket above 64 keys
//                      being a segment of its own (small segments keep
//                      more CUs busy and networks short);
//   k_bsort_scatter -- every key to its bucket (one atomic per bucket and
//                      wave);
//   k_bsort_local   -- per segment of up to 512 keys: a bitonic sort of
//                      (key, slot) held in registers, by one wave (partners
//                      in the same lane or swizzled across lanes); a larger
//                      bucket is first split by a workgroup, by the ten bits
//                      below its keys' common prefix, as often as it takes.
// Keys and slots arrive in buffer 0, go to their buckets in buffer 1 and
// come back sorted to buffer 0.
#include "rb_internal.h"

#define BS_WIN 64    // segment window (slots)
#define BS_WAVE_MAX 512  // segments up to this size are sorted by one wave
#define BS_SPLIT 1024    // parts that a larger one is split into
#define BS_ONE 2048      // patches up to this size are sorted by one workgroup
#define BS_RUNS 1024     // windows of one split at most
// parts still to be split (each above BS_WAVE_MAX, of the 2^18 slots of the
// largest patch)
#define BS_TODO ((1 << 18) / BS_WAVE_MAX)

// lanes of the wave holding the same value in the low `bits` bits
__device__ __forceinline__ uint64_t bs_match(uint64_t peers, uint32_t v, bool valid, int bits) {
  for (int bit = 0; bit < bits; ++bit) {
    const bool on = (v >> bit) & 1u;
    const uint64_t m = __ballot(valid && on);
    peers &= on ? m : ~m;
  }
  return peers;
}

// One block of 1024 threads per patch (5 buckets per thread).
__global__ __launch_bounds__(1024) void k_bsort_scan(uint32_t *__restrict__ bcnt,
                                                     uint32_t *__restrict__ bcur,
                                                     const uint32_t *__restrict__ starts,
                                                     uint2 *__restrict__ seg,
                                                     uint2 *__restrict__ big,
                                                     uint32_t *__restrict__ ctl) {
  constexpr int PER = (BS_NB + 1023) / 1024;
  __shared__ uint32_t wsum[16];
  __shared__ int wmax[16];
  __shared__ uint32_t s_base;
  const uint32_t p = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const uint32_t st = starts[p];
  uint32_t *cnt = bcnt + (size_t)p * BS_NB;
  uint32_t c[PER], tot = 0;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const uint32_t b = tid * PER + k;
    c[k] = (b < BS_NB) ? cnt[b] : 0u;
    if (b < BS_NB) cnt[b] = 0u;  // ready for the next sort
    tot += c[k];
  }
  // bucket offsets within the patch
  const uint32_t incl = rb_wave_incl_scan(tot);
  if (lane == 63) wsum[w] = incl;
  __syncthreads();
  uint32_t off = incl - tot;
  for (uint32_t q = 0; q < w; ++q) off += wsum[q];
  uint32_t start[PER];
  int win[PER], mx = -1;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    start[k] = off;
    win[k] = c[k] ? (int)(off / BS_WIN) : -1;
    mx = win[k] > mx ? win[k] : mx;
    off += c[k];
    const uint32_t b = tid * PER + k;
    if (b < BS_NB) bcur[(size_t)p * BS_NB + b] = st + start[k];
    if (c[k] > BS_WAVE_MAX)
      big[atomicAdd(&ctl[2], 1u)] = make_uint2(st + start[k], st + start[k] + c[k]);
  }
  // window of the last non-empty bucket before this thread's: an
  // exclusive max-scan (windows never decrease along the buckets)
  int run = mx;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int v = __shfl_up(run, d, 64);
    if (lane >= (uint32_t)d) run = v > run ? v : run;
  }
  if (lane == 63) wmax[w] = run;
  __syncthreads();
  int prev = -1;
  for (uint32_t q = 0; q < w; ++q) prev = wmax[q] > prev ? wmax[q] : prev;
  const int up = __shfl_up(run, 1, 64);
  if (lane > 0) prev = up > prev ? up : prev;
  // a segment starts at a non-empty bucket in a new window, and at a
  // bucket above the window size
  uint32_t flags = 0, nf = 0;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    if (c[k] && (win[k] != prev || c[k] > BS_WIN)) { flags |= 1u << k; ++nf; }
    if (c[k]) prev = win[k];
  }
  const uint32_t fin = rb_wave_incl_scan(nf);
  __syncthreads();  // wsum is reused
  if (lane == 63) wsum[w] = fin;
  __syncthreads();
  uint32_t fo = fin - nf;
  for (uint32_t q = 0; q < w; ++q) fo += wsum[q];
  if (tid == 1023) s_base = atomicAdd(&ctl[0], fo + nf);
  __syncthreads();
  const uint32_t base = s_base;
#pragma unroll
  for (int k = 0; k < PER; ++k)
    if (flags & (1u << k)) seg[base + fo++] = make_uint2(st + start[k], p);
}

__global__ __launch_bounds__(256) void k_bsort_scatter(
    const uint64_t *__restrict__ kin, const uint32_t *__restrict__ vin,
    uint64_t *__restrict__ kout, uint32_t *__restrict__ vout, const uint32_t *__restrict__ starts,
    uint32_t P, uint32_t n, uint32_t *__restrict__ bcur) {
  const uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  const bool valid = s < n;
  const uint64_t k = valid ? kin[s] : 0ull;
  const uint32_t v = valid ? vin[s] : 0u;
  const uint32_t p = (valid && P > 1) ? rb_patch_of(starts, P, s) : 0u;
  const uint32_t b = valid ? bs_bucket(k) : 0u;
  // lanes with the same (patch, bucket) share one atomic
  uint64_t peers = bs_match(__ballot(valid), b, valid, BS_BITS + 1);
  if (P > 1) peers = bs_match(peers, p, valid, 32 - __clz((int)(P - 1)));
  const uint32_t lane = rb_lane();
  const uint32_t leader = peers ? (uint32_t)(__ffsll((long long)peers) - 1) : lane;
  uint32_t pos = 0;
  if (valid && lane == leader)
    pos = atomicAdd(&bcur[(size_t)p * BS_NB + b], (uint32_t)__popcll(peers));
  pos = (uint32_t)__shfl((int)pos, (int)leader, 64) + rb_mbcnt(peers);
  if (valid) {
    kout[pos] = k;
    vout[pos] = v;
  }
}

__device__ __forceinline__ bool bs_less(uint64_t ka, uint32_t va, uint64_t kb, uint32_t vb) {
  return ka < kb || (ka == kb && va < vb);
}

// Bitonic network on (key, slot) pairs of one segment of at most 64 R
// keys by one wave, lane-major: element e = lane R + r sits in register r of
// the lane, so partners closer than R are in the same lane and the others
// R-multiples of lanes apart (ds_swizzle below 32 lanes, a shuffle at 32).
// The pairs are compared as (key, slot), so equal keys come out in slot
// order and the padding (all-ones key, all-ones slot) last.
template <int S>
__device__ __forceinline__ void bs_lane_xor(uint64_t &k, uint32_t &v) {
  if (S < 32) {
    constexpr int pat = 0x1F | (S << 10);  // bit-mask mode: lane ^ S in each half
    const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_swizzle((int)(uint32_t)k, pat);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_swizzle((int)(uint32_t)(k >> 32), pat);
    k = ((uint64_t)hi << 32) | lo;
    v = (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, pat);
  } else {
    k = __shfl_xor(k, S, 64);
    v = (uint32_t)__shfl_xor((int)v, S, 64);
  }
}

template <int R, int S>
__device__ __forceinline__ void bs_wave_lanes(uint64_t (&k)[R], uint32_t (&v)[R], uint32_t lane,
                                              uint32_t size) {
  // partners S lanes apart: element stride S * R
#pragma unroll
  for (int r = 0; r < R; ++r) {
    uint64_t pk = k[r];
    uint32_t pv = v[r];
    bs_lane_xor<S>(pk, pv);
    const uint32_t e = lane * R + (uint32_t)r;
    const bool asc = (e & size) == 0;
    const bool lower = (e & (uint32_t)(S * R)) == 0;
    if ((lower == asc) == bs_less(pk, pv, k[r], v[r])) { k[r] = pk; v[r] = pv; }
  }
}

template <int R>
__device__ __forceinline__ void bs_wave_sort(const uint64_t *k1, const uint32_t *v1, uint32_t b,
                                             uint64_t *k0, uint32_t *v0, uint32_t a, uint32_t m,
                                             uint32_t lane) {
  uint64_t k[R];
  uint32_t v[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t e = lane * R + (uint32_t)r;
    k[r] = e < m ? k1[b + e] : ~0ull;
    v[r] = e < m ? v1[b + e] : ~0u;
  }
#pragma unroll
  for (uint32_t size = 2; size <= 64u * R; size <<= 1) {
#pragma unroll
    for (uint32_t stride = size >> 1; stride > 0; stride >>= 1) {
      if (stride >= (uint32_t)R) {
        switch (stride / R) {
          case 1: bs_wave_lanes<R, 1>(k, v, lane, size); break;
          case 2: bs_wave_lanes<R, 2>(k, v, lane, size); break;
          case 4: bs_wave_lanes<R, 4>(k, v, lane, size); break;
          case 8: bs_wave_lanes<R, 8>(k, v, lane, size); break;
          case 16: bs_wave_lanes<R, 16>(k, v, lane, size); break;
          default: bs_wave_lanes<R, 32>(k, v, lane, size); break;
        }
      } else {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int r2 = r | (int)stride;
          if ((r & (int)stride) == 0 && r2 < R) {
            const bool asc = ((lane * R + (uint32_t)r) & size) == 0;
            if (bs_less(k[r2], v[r2], k[r], v[r]) == asc) {
              const uint64_t tk = k[r]; k[r] = k[r2]; k[r2] = tk;
              const uint32_t tv = v[r]; v[r] = v[r2]; v[r2] = tv;
            }
          }
        }
      }
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t e = lane * R + (uint32_t)r;
    if (e < m) { k0[a + e] = k[r]; v0[a + e] = v[r]; }
  }
}

// slot range [a, e) of segment i
__device__ __forceinline__ void bs_segment(const uint2 *__restrict__ seg,
                                           const uint32_t *__restrict__ starts, uint32_t nseg,
                                           uint32_t i, uint32_t &a, uint32_t &e) {
  const uint2 me = seg[i];
  a = me.x;
  e = starts[me.y + 1];
  if (i + 1 < nseg) {
    const uint2 nx = seg[i + 1];
    if (nx.y == me.y) e = nx.x;
  }
}

// m <= BS_WAVE_MAX pairs from place b of (k1, v1), sorted to place a of (k0,
// v0) by one wave (which may be the same: all are read before any is written).
__device__ __forceinline__ void bs_wave(const uint64_t *k1, const uint32_t *v1, uint32_t b,
                                        uint64_t *k0, uint32_t *v0, uint32_t a, uint32_t m,
                                        uint32_t lane) {
  if (m == 1) {
    if (lane == 0) { k0[a] = k1[b]; v0[a] = v1[b]; }
  } else if (m <= 64) {
    bs_wave_sort<1>(k1, v1, b, k0, v0, a, m, lane);
  } else if (m <= 128) {
    bs_wave_sort<2>(k1, v1, b, k0, v0, a, m, lane);
  } else if (m <= 256) {
    bs_wave_sort<4>(k1, v1, b, k0, v0, a, m, lane);
  } else {
    bs_wave_sort<8>(k1, v1, b, k0, v0, a, m, lane);
  }
}

template <int NT>
struct BsSplit {
  uint64_t k[BS_SPLIT];  // the pairs of a bucket of up to BS_SPLIT keys
  uint32_t v[BS_SPLIT];
  uint32_t cnt[BS_SPLIT];  // counts, then cursors
  uint32_t run[2 * BS_RUNS + 3];  // (two start in a window at most)
  uint2 todo[BS_TODO];  // slots [x, y), the top bit of y: in buffer 1
  unsigned long long any, all;
  uint32_t vany, vall, n_todo, wsum[NT / 64];
  int wmax[NT / 64];
};

// A bucket of more than BS_WAVE_MAX keys by one workgroup: its keys are dealt
// to BS_SPLIT parts by the ten bits from the first in which they differ on
// (equal keys by their slots' bits) and put in the other buffer, or in LDS if
// they fit; runs of whole parts are sorted by a wave each, larger parts split
// again.  A split
// tells at least two keys apart and its parts share ten more bits, so they
// end.  Bound by the waves' networks, one after another.  Concentrated systems
// have most of their particles in a few buckets: forces of spheres at theta 0.9
// (nine radix passes over global memory by one workgroup before, and four
// large buckets in turn), 30,000 particles 579 -> 315 us, 260,000 2314 -> 1195.
template <int NT>
__device__ void bs_split(uint64_t *k1, uint32_t *v1, uint64_t *k0, uint32_t *v0, uint32_t a,
                         uint32_t e, BsSplit<NT> &sh) {
  constexpr int PER = BS_SPLIT / NT, NW = NT / 64;
  const uint32_t tid = threadIdx.x, lane = tid & 63;
  const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  uint32_t one = 1u;  // the keys are in buffer 1
  if (tid == 0) sh.n_todo = 0;
  for (;;) {
    const uint64_t *ki = one ? k1 : k0;
    const uint32_t *vi = one ? v1 : v0;
    uint64_t *ko = one ? k0 : k1;
    uint32_t *vo = one ? v0 : v1;
    // the pairs from s0 on, four per thread, read once if they are few
    const bool few = e - a <= BS_SPLIT;
    uint64_t k[4];
    uint32_t v[4], at = RB_NONE;
    auto load = [&](uint32_t s0) {
      if (at == s0) return;
      at = s0;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const uint32_t s = s0 + (uint32_t)(NT * r) + tid;
        if (s < e) { k[r] = ki[s]; v[r] = vi[s]; }
      }
    };
    auto each = [&](auto &&f) {
      for (uint32_t s0 = a; s0 < e; s0 += 4 * NT) {
        load(s0);
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (s0 + (uint32_t)(NT * r) + tid < e) f(k[r], v[r]);
      }
    };
    // the bits that differ
    if (tid == 0) { sh.any = 0; sh.all = ~0ull; sh.vany = 0; sh.vall = ~0u; }
    for (uint32_t i = tid; i < BS_SPLIT; i += NT) sh.cnt[i] = 0;
    __syncthreads();
    {
      uint64_t any = 0, all = ~0ull;
      uint32_t vany = 0, vall = ~0u;
      each([&](uint64_t kk, uint32_t vv) { any |= kk; all &= kk; vany |= vv; vall &= vv; });
      atomicOr(&sh.any, (unsigned long long)any);
      atomicAnd(&sh.all, (unsigned long long)all);
      atomicOr(&sh.vany, vany);
      atomicAnd(&sh.vall, vall);
    }
    __syncthreads();
    const uint64_t diff = sh.any & ~sh.all;
    const uint32_t vdiff = sh.vany & ~sh.vall;
    const bool by_key = diff != 0;  // (slots differ)
    const int top = by_key ? 63 - __clzll((long long)diff) : 31 - __clz((int)vdiff);
    const int shift = top > 9 ? top - 9 : 0;
    auto part = [&](uint64_t kk, uint32_t vv) {
      return (uint32_t)((by_key ? kk : (uint64_t)vv) >> shift) & (BS_SPLIT - 1u);
    };
    each([&](uint64_t kk, uint32_t vv) { atomicAdd(&sh.cnt[part(kk, vv)], 1u); });
    __syncthreads();
    // cursors, and runs of whole parts that start in the same window (a part
    // as large as a window by itself): as the segments of k_bsort_scan
    uint32_t c[PER], tot = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) { c[q] = sh.cnt[PER * tid + q]; tot += c[q]; }
    const uint32_t incl = rb_wave_incl_scan(tot);
    if (lane == 63) sh.wsum[w] = incl;
    __syncthreads();
    uint32_t off = incl - tot;
    for (uint32_t q = 0; q < w; ++q) off += sh.wsum[q];
    // the smallest windows of at least 64 pairs that are few enough
    int wl = 6;
    while (((e - a - 1) >> wl) >= BS_RUNS) ++wl;
    uint32_t start[PER];
    int mx = -1;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      start[q] = off;
      if (c[q]) mx = (int)(off >> wl);
      sh.cnt[PER * tid + q] = a + off;
      off += c[q];
    }
    int run = mx;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int o = __shfl_up(run, d, 64);
      if (lane >= (uint32_t)d) run = o > run ? o : run;
    }
    if (lane == 63) sh.wmax[w] = run;
    const int up = __shfl_up(run, 1, 64);
    __syncthreads();
    int prev = -1;
    for (uint32_t q = 0; q < w; ++q) prev = sh.wmax[q] > prev ? sh.wmax[q] : prev;
    if (lane > 0 && up > prev) prev = up;
    uint32_t flags = 0, nf = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int win = (int)(start[q] >> wl);
      if (c[q] && (win != prev || (c[q] >> wl) != 0)) { flags |= 1u << q; ++nf; }
      if (c[q]) prev = win;
    }
    const uint32_t fin = rb_wave_incl_scan(nf);
    if (lane == 63) sh.wsum[w] = fin;
    __syncthreads();
    uint32_t fo = fin - nf, n_run = 0;
    for (uint32_t q = 0; q < NW; ++q) {
      if (q < w) fo += sh.wsum[q];
      n_run += sh.wsum[q];
    }
#pragma unroll
    for (int q = 0; q < PER; ++q)
      if (flags & (1u << q)) sh.run[fo++] = a + start[q];
    if (tid == 0) sh.run[n_run] = e;
    uint64_t *const tk = few ? sh.k : ko;
    uint32_t *const tv = few ? sh.v : vo;
    const uint32_t base = few ? a : 0u;
    each([&](uint64_t kk, uint32_t vv) {
      const uint32_t to = atomicAdd(&sh.cnt[part(kk, vv)], 1u) - base;
      tk[to] = kk;
      tv[to] = vv;
    });
    __syncthreads();
    for (uint32_t i = w; i < n_run; i += NW) {
      const uint32_t x = sh.run[i], y = sh.run[i + 1];
      if (y - x <= BS_WAVE_MAX) {
        bs_wave(tk, tv, x - base, k0, v0, x, y - x, lane);
        continue;
      }
      if (few)
        for (uint32_t j = x + lane; j < y; j += 64) { ko[j] = tk[j - a]; vo[j] = tv[j - a]; }
      if (lane == 0)
        sh.todo[atomicAdd(&sh.n_todo, 1u)] = make_uint2(x, y | (one ? 0u : 0x80000000u));
    }
    __syncthreads();
    const uint32_t left = sh.n_todo;
    if (left == 0) break;  // uniform
    const uint2 next = sh.todo[left - 1];
    __syncthreads();
    if (tid == 0) sh.n_todo = left - 1;
    a = next.x;
    e = next.y & 0x7FFFFFFFu;
    one = next.y >> 31;
  }
  __syncthreads();  // LDS is used again by the next segment
}

// Workgroups split the large buckets, one each in turn, and then every wave
// sorts segments of up to BS_WAVE_MAX keys, one in the grid's number of waves
// (with a counter and barriers between them, a step of 64 patches took 4 %
// longer).
template <int NT>
__global__ __launch_bounds__(NT) void k_bsort_local(
    uint64_t *k1, uint32_t *v1, uint64_t *k0, uint32_t *v0, const uint2 *__restrict__ seg,
    const uint2 *__restrict__ big, const uint32_t *__restrict__ ctl,
    const uint32_t *__restrict__ starts) {
  __shared__ BsSplit<NT> sh;
  const uint32_t tid = threadIdx.x, lane = tid & 63;
  const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  const uint32_t nseg = ctl[0], nbig = ctl[2];
  for (uint32_t i = blockIdx.x; i < nbig; i += gridDim.x)
    bs_split<NT>(k1, v1, k0, v0, big[i].x, big[i].y, sh);
  for (uint32_t i = NT / 64 * blockIdx.x + w; i < nseg; i += NT / 64 * gridDim.x) {
    uint32_t a, e;
    bs_segment(seg, starts, nseg, i, a, e);
    if (e - a <= BS_WAVE_MAX) bs_wave(k1, v1, a, k0, v0, a, e - a, lane);
  }
}

// Patches of up to BS_ONE slots: all of it by one workgroup, the buckets in
// LDS, where three launches are bound by their latency (four steps of sheets:
// 300 particles 355 -> 335 us, 1,024 396 -> 379, 2,048 423 -> 417; 4,000
// 444 -> 466, sixteen waves taking longer than many workgroups).
__global__ __launch_bounds__(1024) void k_bsort_one(uint64_t *k1, uint32_t *v1, uint64_t *k0,
                                                    uint32_t *v0,
                                                    const uint32_t *__restrict__ starts,
                                                    uint32_t *__restrict__ bcnt) {
  constexpr int PER = (BS_NB + 1023) / 1024, ROWS = BS_ONE / 1024;
  struct One {
    uint64_t k[BS_ONE];
    uint32_t v[BS_ONE], cur[BS_NB];
  };
  // (the pairs have left LDS when a large bucket is split)
  __shared__ union { One o; BsSplit<1024> split; } sh;
  __shared__ uint32_t seg[2 * (BS_ONE / BS_WIN) + 2], wsum[16], s_big[BS_ONE / BS_WAVE_MAX][2], n_big;
  __shared__ int wmax[16];
  const uint32_t p = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  const uint32_t st = starts[p], n = starts[p + 1] - st;
  if (n == 0 || n > BS_ONE) return;  // (larger: never launched)
  uint64_t k[ROWS];
  uint32_t v[ROWS];
#pragma unroll
  for (int r = 0; r < ROWS; ++r) {
    const uint32_t i = 1024u * (uint32_t)r + tid;
    k[r] = i < n ? k0[st + i] : 0ull;
    v[r] = i < n ? v0[st + i] : 0u;
  }
  // bucket offsets and segments, as k_bsort_scan finds them
  uint32_t *cnt = bcnt + (size_t)p * BS_NB;
  uint32_t c[PER], tot = 0;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const uint32_t b = tid * PER + q;
    c[q] = (b < BS_NB) ? cnt[b] : 0u;
    if (b < BS_NB) cnt[b] = 0u;  // ready for the next sort
    tot += c[q];
  }
  if (tid == 0) n_big = 0;
  const uint32_t incl = rb_wave_incl_scan(tot);
  if (lane == 63) wsum[w] = incl;
  __syncthreads();
  uint32_t off = incl - tot;
  for (uint32_t q = 0; q < w; ++q) off += wsum[q];
  uint32_t start[PER];
  int mx = -1;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const uint32_t b = tid * PER + q;
    start[q] = off;
    if (c[q]) mx = (int)(off / BS_WIN);
    if (b < BS_NB) sh.o.cur[b] = off;
    if (c[q] > BS_WAVE_MAX) {
      const uint32_t i = atomicAdd(&n_big, 1u);
      s_big[i][0] = off;
      s_big[i][1] = off + c[q];
    }
    off += c[q];
  }
  int run = mx;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int o = __shfl_up(run, d, 64);
    if (lane >= (uint32_t)d) run = o > run ? o : run;
  }
  if (lane == 63) wmax[w] = run;
  const int up = __shfl_up(run, 1, 64);
  __syncthreads();
  int prev = -1;
  for (uint32_t q = 0; q < w; ++q) prev = wmax[q] > prev ? wmax[q] : prev;
  if (lane > 0 && up > prev) prev = up;
  uint32_t flags = 0, nf = 0;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int win = (int)(start[q] / BS_WIN);
    if (c[q] && (win != prev || c[q] > BS_WIN)) { flags |= 1u << q; ++nf; }
    if (c[q]) prev = win;
  }
  const uint32_t fin = rb_wave_incl_scan(nf);
  if (lane == 63) wsum[w] = fin;
  __syncthreads();
  uint32_t fo = fin - nf, nseg = 0;
  for (uint32_t q = 0; q < 16; ++q) {
    if (q < w) fo += wsum[q];
    nseg += wsum[q];
  }
#pragma unroll
  for (int q = 0; q < PER; ++q)
    if (flags & (1u << q)) seg[fo++] = start[q];
  if (tid == 0) seg[nseg] = n;
  // keys to their buckets
#pragma unroll
  for (int r = 0; r < ROWS; ++r) {
    if (1024u * (uint32_t)r + tid < n) {
      const uint32_t to = atomicAdd(&sh.o.cur[bs_bucket(k[r])], 1u);
      if (to < BS_ONE) { sh.o.k[to] = k[r]; sh.o.v[to] = v[r]; }
    }
  }
  __syncthreads();
  for (uint32_t i = w; i < nseg; i += 16) {
    const uint32_t x = seg[i], y = seg[i + 1];
    if (y - x <= BS_WAVE_MAX) bs_wave(sh.o.k, sh.o.v, x, k0, v0, st + x, y - x, lane);
  }
  const uint32_t big = n_big;
  if (big == 0) return;  // uniform
  for (uint32_t i = 0; i < big; ++i)
    for (uint32_t j = s_big[i][0] + tid; j < s_big[i][1]; j += 1024) {
      k1[st + j] = sh.o.k[j];
      v1[st + j] = sh.o.v[j];
    }
  __syncthreads();
  for (uint32_t i = 0; i < big; ++i)
    bs_split<1024>(k1, v1, k0, v0, st + s_big[i][0], st + s_big[i][1], sh.split);
}

hipError_t launch_bsort(rb_ctx *c) {
  const uint32_t n = (uint32_t)c->h_starts[c->P];
  if (n == 0) return hipSuccess;
  if (c->sort_largest <= BS_ONE) {
    hipLaunchKernelGGL(k_bsort_one, dim3(c->P), dim3(1024), 0, c->stream, c->d_key[1], c->d_idx[1],
                       c->d_key[0], c->d_idx[0], c->d_starts, c->d_bcnt);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_bsort_scan, dim3(c->P), dim3(1024), 0, c->stream, c->d_bcnt, c->d_bcur,
                     c->d_starts, c->d_bseg, c->d_bbig, c->d_bctl);
  hipLaunchKernelGGL(k_bsort_scatter, dim3(rb_div_up(n, 256)), dim3(256), 0, c->stream,
                     c->d_key[0], c->d_idx[0], c->d_key[1], c->d_idx[1], c->d_starts, c->P, n,
                     c->d_bcur);
  const int nt = c->sort_threads;
  const unsigned grid = (unsigned)std::min<uint64_t>(262144 / nt, rb_div_up(n, nt) + c->P);
#define RB_BS_LOCAL(NT)                                                                       \
  hipLaunchKernelGGL(k_bsort_local<NT>, dim3(grid), dim3(NT), 0, c->stream, c->d_key[1],       \
                     c->d_idx[1], c->d_key[0], c->d_idx[0], c->d_bseg, c->d_bbig, c->d_bctl,  \
                     c->d_starts)
  if (nt == 256) RB_BS_LOCAL(256);
  else RB_BS_LOCAL(1024);
#undef RB_BS_LOCAL
  return hipGetLastError();
}
