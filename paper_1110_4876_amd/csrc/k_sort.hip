// k_sort.hip -- stable LSD radix sort of (Morton key, slot) pairs inside every
// patch, for large systems: 8 passes of 8-bit digits over the 64-bit keys,
// three launches per pass.  (Small systems use the bucket sort of k_bsort.hip.)
//
// Each pass works on tiles of 256 * R consecutive slots of one patch, by
// workgroups of 256 threads:
//   k_sort_count -- every tile's count of every digit;
//   k_sort_scan  -- per patch and digit, the keys of the digit in earlier
//                   tiles, and in the patch;
//   k_sort_pass  -- every wave ranks its R rows of 64 keys in order: the lanes
//                   holding the same digit find each other with 8 ballots, a
//                   lane's rank is the count of equal-digit lanes below it
//                   plus the digit's running count of the wave (LDS), so
//                   equal keys keep their order.  The tile is put in digit
//                   order in LDS and written out in runs, after the patch's
//                   keys of smaller digits and of this digit in earlier tiles.
// Sentinel keys of removed particles (all ones) sort last.
//
// Bound by the launches and their round trips at 10^6 keys, by HBM above: a
// pass takes 22 us (count 5.4, scan 4.6, ranks and writes 12.4) at 1,000,003
// keys and 87 us (20, 7, 60; 1.9 times its 24 bytes a key at the copy rate) at
// 2^23.  One launch per pass with a decoupled look-back -- each tile waiting
// for its predecessors' published counts and adding them up, 32 words a round
// trip over 500 to 4,000 tiles -- took 56 and 184 us, and a counting launch
// for all passes 22 and 119 us.
#include "rb_internal.h"

#define SORT_BITS 8
#define SORT_BINS 256
#define SORT_PASSES 8

// lanes of the wave holding the same 8-bit digit
__device__ __forceinline__ uint64_t wave_match8(uint32_t d, bool valid) {
  uint64_t peers = __ballot(valid);
#pragma unroll
  for (int bit = 0; bit < SORT_BITS; ++bit) {
    const bool on = (d >> bit) & 1u;
    const uint64_t m = __ballot(valid && on);
    peers &= on ? m : ~m;
  }
  return peers;
}

// Every tile's count of every digit of this pass, digit-major (the scan below
// reads a digit's counts in a row).
template <int R>
__global__ __launch_bounds__(256) void k_sort_count(int pass, const uint64_t *__restrict__ kin,
                                                    const uint32_t *__restrict__ tile_start,
                                                    const uint32_t *__restrict__ tile_end,
                                                    uint32_t n_tiles,
                                                    uint32_t *__restrict__ cnt) {
  __shared__ uint32_t h[4][SORT_BINS];
  const uint32_t tid = threadIdx.x, w = tid >> 6, t = blockIdx.x;
  const uint32_t s0 = tile_start[t], s1 = tile_end[t];
  const int shift = SORT_BITS * pass;
  uint64_t kk[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t s = s0 + r * 256 + tid;
    kk[r] = s < s1 ? kin[s] : 0ull;
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) h[q][tid] = 0;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const bool valid = s0 + r * 256 + tid < s1;
    const uint64_t vm = __ballot(valid);
    if (vm == 0) break;  // uniform over the wave
    const uint32_t d = (uint32_t)(kk[r] >> shift) & (SORT_BINS - 1);
    // a digit that the whole wave shares: one LDS atomic
    const uint32_t d0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)d);
    if (__ballot(valid && d == d0) == vm) {
      if (rb_lane() == 0) atomicAdd(&h[w][d0], (uint32_t)__popcll(vm));
    } else if (valid) {
      atomicAdd(&h[w][d], 1u);
    }
  }
  __syncthreads();
  cnt[(size_t)tid * n_tiles + t] = h[0][tid] + h[1][tid] + h[2][tid] + h[3][tid];
}

// Block (d, p): the counts of digit d in patch p's tiles become the counts in
// the tiles before each; their sum goes to tot.
__global__ __launch_bounds__(256) void k_sort_scan(uint32_t *__restrict__ cnt,
                                                   const uint32_t *__restrict__ patch_tile0,
                                                   uint32_t P, uint32_t n_tiles,
                                                   uint32_t *__restrict__ tot) {
  __shared__ uint32_t wsum[4];
  const uint32_t tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const uint32_t d = blockIdx.x;
  for (uint32_t p = blockIdx.y; p < P; p += gridDim.y) {
    uint32_t carry = 0;
    const uint32_t t0 = patch_tile0[p], t1 = patch_tile0[p + 1];
    uint32_t *row = cnt + (size_t)d * n_tiles;
    // 1024 tiles per round, four consecutive ones per thread
    for (uint32_t off = t0; off < t1; off += 1024) {
      const uint32_t i0 = off + 4 * tid;
      uint32_t v[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = (i0 + k < t1) ? row[i0 + k] : 0u;
      const uint32_t sum = v[0] + v[1] + v[2] + v[3];
      const uint32_t incl = rb_wave_incl_scan(sum);
      if (lane == 63) wsum[w] = incl;
      __syncthreads();
      uint32_t ex = carry + incl - sum;
      for (uint32_t q = 0; q < w; ++q) ex += wsum[q];
      carry += wsum[0] + wsum[1] + wsum[2] + wsum[3];
      __syncthreads();  // (wsum is rewritten)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (i0 + k < t1) row[i0 + k] = ex;
        ex += v[k];
      }
    }
    if (tid == 0) tot[(size_t)p * SORT_BINS + d] = carry;
  }
}

template <int R>
__global__ __launch_bounds__(256) void k_sort_pass(
    int pass, const uint64_t *__restrict__ kin, const uint32_t *__restrict__ vin,
    uint64_t *__restrict__ kout, uint32_t *__restrict__ vout,
    const uint32_t *__restrict__ tile_start, const uint32_t *__restrict__ tile_end,
    const uint32_t *__restrict__ tile_patch, const uint32_t *__restrict__ starts,
    uint32_t n_tiles, const uint32_t *__restrict__ earlier, const uint32_t *__restrict__ tot) {
  __shared__ uint32_t cnt[4][SORT_BINS];  // per-wave digit counts, then places in the tile
  __shared__ uint32_t base[SORT_BINS];    // first slot of a digit less its place in the tile
  __shared__ uint32_t wsum[4], psum[4];
  __shared__ uint64_t sk[256 * R];
  __shared__ uint32_t sv[256 * R];
  const uint32_t tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int shift = SORT_BITS * pass;
  const uint32_t t = blockIdx.x;
  const uint32_t s0 = tile_start[t], s1 = tile_end[t];
  const uint32_t p = tile_patch[t];
  const uint32_t before = earlier[(size_t)tid * n_tiles + t];
  const uint32_t in_patch = tot[(size_t)p * SORT_BINS + tid];
#pragma unroll
  for (int q = 0; q < 4; ++q) cnt[q][tid] = 0;
  // rank: wave w owns rows [w R, (w + 1) R) of the tile
  uint64_t kk[R];
  uint32_t vv[R], lr[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t s = s0 + (w * R + r) * 64 + lane;
    const bool valid = s < s1;
    kk[r] = valid ? kin[s] : 0ull;
    vv[r] = valid ? vin[s] : 0u;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t s = s0 + (w * R + r) * 64 + lane;
    const bool valid = s < s1;
    const uint32_t d = (uint32_t)(kk[r] >> shift) & (SORT_BINS - 1);
    const uint64_t peers = wave_match8(d, valid);
    const uint32_t rank = rb_mbcnt(peers);
    // one LDS read for all lanes, then the lowest lane of each digit group
    // advances the count with the value it read (data-dependent: the read
    // of every lane precedes the write)
    const uint32_t b0 = valid ? cnt[w][d] : 0u;
    lr[r] = b0 + rank;
    if (valid && rank == 0) cnt[w][d] = b0 + (uint32_t)__popcll(peers);
  }
  __syncthreads();
  // per digit (thread tid): its place in the tile, and each wave's in it
  const uint32_t c0 = cnt[0][tid], c1 = cnt[1][tid], c2 = cnt[2][tid], c3 = cnt[3][tid];
  const uint32_t all = c0 + c1 + c2 + c3;
  const uint32_t incl = rb_wave_incl_scan(all), pincl = rb_wave_incl_scan(in_patch);
  if (lane == 63) {
    wsum[w] = incl;
    psum[w] = pincl;
  }
  __syncthreads();
  uint32_t at = incl - all, slot0 = starts[p] + pincl - in_patch + before;
  for (uint32_t q = 0; q < w; ++q) {
    at += wsum[q];
    slot0 += psum[q];
  }
  cnt[0][tid] = at;
  cnt[1][tid] = at + c0;
  cnt[2][tid] = at + c0 + c1;
  cnt[3][tid] = at + c0 + c1 + c2;
  base[tid] = slot0 - at;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t s = s0 + (w * R + r) * 64 + lane;
    if (s < s1) {
      const uint32_t d = (uint32_t)(kk[r] >> shift) & (SORT_BINS - 1);
      const uint32_t q = cnt[w][d] + lr[r];
      sk[q] = kk[r];
      sv[q] = vv[r];
    }
  }
  __syncthreads();
  // out in digit order: neighbouring threads write neighbouring slots
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t q = r * 256 + tid;
    if (s0 + q < s1) {
      const uint64_t k = sk[q];
      const uint32_t pos = base[(uint32_t)(k >> shift) & (SORT_BINS - 1)] + q;
      kout[pos] = k;
      vout[pos] = sv[q];
    }
  }
}

hipError_t launch_sort(rb_ctx *c) {
  if (c->sort_small) return launch_bsort(c);
  if (c->n_stiles == 0) return hipSuccess;
  const dim3 grid(c->n_stiles), block(256);
  const dim3 sgrid(SORT_BINS, std::min<uint32_t>(c->P, 64u));
  int src = 0;
  for (int pass = 0; pass < SORT_PASSES; ++pass) {
#define RB_SORT_R(R)                                                                         \
  do {                                                                                       \
    hipLaunchKernelGGL(k_sort_count<R>, grid, block, 0, c->stream, pass, c->d_key[src],       \
                       c->d_stile_start, c->d_stile_end, c->n_stiles, c->d_scnt);             \
    hipLaunchKernelGGL(k_sort_scan, sgrid, block, 0, c->stream, c->d_scnt, c->d_spatch_tile0, \
                       c->P, c->n_stiles, c->d_stot);                                         \
    hipLaunchKernelGGL(k_sort_pass<R>, grid, block, 0, c->stream, pass, c->d_key[src],        \
                       c->d_idx[src], c->d_key[1 - src], c->d_idx[1 - src], c->d_stile_start, \
                       c->d_stile_end, c->d_stile_patch, c->d_starts, c->n_stiles, c->d_scnt, \
                       c->d_stot);                                                            \
  } while (0)
    if (c->sort_rows == 4) RB_SORT_R(4);
    else RB_SORT_R(8);
#undef RB_SORT_R
    src = 1 - src;
  }
  return hipGetLastError();  // an even number of passes: the result is in buffer 0
}

// ---------------------------------------------------------------------------
// exclusive scan of the topology's per-tile level counts: one 256-thread
// block per (kind, level) row of n_tiles entries; row totals to row_tot.
__global__ __launch_bounds__(256) void k_rowscan(uint32_t *__restrict__ data, uint32_t n_tiles,
                                                 uint32_t *__restrict__ row_tot,
                                                 const uint32_t *__restrict__ reuse) {
  __shared__ uint32_t wsum[4];
  if (reuse && *reuse == 0u) return;  // the step keeps the last tree
  const uint32_t r = blockIdx.x, tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const size_t base = (size_t)r * n_tiles;
  uint32_t carry = 0;
  // 1024 entries per round: four consecutive ones per thread, summed in the
  // thread, then the threads' totals scanned across the block
  for (uint32_t off = 0; off < n_tiles; off += 1024) {
    const uint32_t i0 = off + 4 * tid;
    uint32_t v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = (i0 + k < n_tiles) ? data[base + i0 + k] : 0u;
    const uint32_t s1 = v[0], s2 = s1 + v[1], s3 = s2 + v[2], s4 = s3 + v[3];
    const uint32_t incl = rb_wave_incl_scan(s4);
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    uint32_t add = 0;
    for (uint32_t q = 0; q < w; ++q) add += wsum[q];
    const uint32_t tot = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    __syncthreads();
    const uint32_t ex = carry + add + incl - s4;  // before the thread's first entry
    const uint32_t out[4] = {ex, ex + s1, ex + s2, ex + s3};
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (i0 + k < n_tiles) data[base + i0 + k] = out[k];
    carry += tot;
  }
  if (tid == 0) row_tot[r] = carry;
}

hipError_t launch_rowscan_levels(rb_ctx *c, const uint32_t *reuse) {
  hipLaunchKernelGGL(k_rowscan, dim3(2 * RB_NLEV), dim3(256), 0, c->stream, c->d_cnt,
                     c->n_tiles, c->d_lev_tot, reuse);
  return hipGetLastError();
}
