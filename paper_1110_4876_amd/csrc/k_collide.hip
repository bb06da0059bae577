// k_collide.hip -- collisions at the end of a step (Sect. 5 of the paper):
// overlapping pairs found by the octree search of Eq. (3) over the ghost
// boxes, a collision queue in a random order, and hard-sphere resolution
// with a normal coefficient of restitution, one collision after the other in
// queue order.
//
// Detection: the criterion of Eq. (3) opens a cell for particle i while the
// distance from x_i to the image-shifted cell centre is below R_i + R_max +
// (sqrt 3 / 2) w; every particle of the cell that could overlap i passes it,
// so the search finds every overlap.  One wave searches for the (up to 64)
// Morton-consecutive particles of a work item at once: a cell is opened when
// it is within R_g + R_max + (sqrt 3 / 2) w of the item's bounding box (R_g
// the item's largest radius), which holds whenever it holds for any member.
// Opened leaves go to an LDS list that every lane then tests against its own
// particle: j overlaps i when |x_j + o_k - x_i| < R_i + R_j; the pair is
// queued once, from its lower caller index i, as the code i 2^35 + j 2^7 + k.
//
// Order and resolution: the queue's order is ascending h = splitmix64(seed +
// code) (a bijection, so the order is total).  Resolving the collisions one
// after the other in that order gives each of them the velocities left by the
// earlier collisions of its own two particles, and collisions without a
// common particle commute: so a collision may be resolved as soon as its
// predecessors, the last earlier one of each particle, have been (k_coll_run).
// Resolution applies v_n' = -eps v_n, v_t' = v_t with momentum conservation
// when the pair approaches (d . u < 0, u = v_j + w_k - v_i with w_k the
// image's shear velocity).
//
// Compiled without FP contraction so that the pair tests and the velocity
// updates round exactly as a plain evaluation of the same expressions.
#include "rb_internal.h"


__device__ __forceinline__ uint64_t rb_splitmix64(uint64_t x) {
  uint64_t z = x + 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// largest radius of the live particles (as ordered bits of a non-negative
// double): slots strided over the grid, one atomic per workgroup
__global__ __launch_bounds__(256) void k_coll_rmax(const double *__restrict__ R,
                                                   const uint32_t *__restrict__ orig,
                                                   const uint32_t *__restrict__ starts,
                                                   const uint32_t *__restrict__ nlive,
                                                   uint32_t P, uint32_t n,
                                                   unsigned long long *__restrict__ rmax,
                                                   uint32_t *__restrict__ head) {
  __shared__ double part[4];
  double r = 0.0;
  for (uint32_t s = blockIdx.x * blockDim.x + threadIdx.x; s < n; s += gridDim.x * blockDim.x) {
    head[s] = RB_NONE;  // the particles' lists of pairs start empty
    const uint32_t p = (P == 1) ? 0u : rb_patch_of(starts, P, s);
    if (s - starts[p] < nlive[p]) {
      const double v = R[orig[s]];
      r = v > r ? v : r;  // (a NaN radius is never larger)
    }
  }
  for (int d = 32; d >= 1; d >>= 1) r = fmax(r, __shfl_xor(r, d, 64));
  if (rb_lane() == 0) part[threadIdx.x >> 6] = r;
  __syncthreads();
  if (threadIdx.x == 0) {
    r = fmax(fmax(part[0], part[1]), fmax(part[2], part[3]));
    if (r > 0.0) atomicMax(rmax, (unsigned long long)__double_as_longlong(r));
  }
}

// order a wave's LDS writes before its later reads (a wave runs in lockstep)
__device__ __forceinline__ void coll_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

#define CG_SCAP 768   // traversal stack entries per wave (node << 5 | image)
#define CG_RESERVE (7 * RB_DEPTH + 8)
#define CG_LL 128     // opened-leaf list capacity per wave (tested at >= 64)

__device__ __forceinline__ double rb_wave_min_d(double v) {
  for (int d = 32; d >= 1; d >>= 1) v = fmin(v, __shfl_xor(v, d, 64));
  return v;
}
__device__ __forceinline__ double rb_wave_max_d(double v) {
  for (int d = 32; d >= 1; d >>= 1) v = fmax(v, __shfl_xor(v, d, 64));
  return v;
}

// The cell as the search reads it (one 32-byte record): the centre of the
// cell in its own root box, a = first child (internal) or first slot (leaf),
// b = leaf << 31 | level << 26 | (children - 1, or last slot - first slot).
struct __align__(32) CollNode {
  double cx, cy, cz;
  uint32_t a, b;
};

// the cells' records, from the topology of the sorted particles
__global__ __launch_bounds__(256) void k_coll_geom(
    const double *__restrict__ sx, const double *__restrict__ sy, const double *__restrict__ sz,
    const PatchInfo *__restrict__ patch, const uint32_t *__restrict__ starts, uint32_t P,
    const uint32_t *__restrict__ lev_off, uint64_t node_cap,
    const uint32_t *__restrict__ nfirst, const uint32_t *__restrict__ nlast,
    const uint32_t *__restrict__ nchild, const uint32_t *__restrict__ nlastchild,
    const uint8_t *__restrict__ nlevel, const uint8_t *__restrict__ nleaf,
    CollNode *__restrict__ out, uint32_t *__restrict__ err, uint32_t *__restrict__ clear) {
  const uint32_t node = blockIdx.x * blockDim.x + threadIdx.x;
  // (collisions inside a step: the counters of this step start at zero)
  if (clear && node < 10) clear[node] = 0u;
  const uint64_t total = lev_off[RB_NLEV];
  if (node >= total || node >= node_cap) return;
  const uint32_t f = nfirst[node];
  const uint32_t p = (P == 1) ? 0u : rb_patch_of(starts, P, f);
  const PatchInfo pi = patch[p];
  const int l = nlevel[node];
  const double w = ldexp(pi.W, -l);
  uint32_t qx = 0, qy = 0, qz = 0;
  (void)rb_quantise(sx[f], pi.x0[0], pi.L[0], pi.S, pi.qtop[0], qx);
  (void)rb_quantise(sy[f], pi.x0[1], pi.L[1], pi.S, pi.qtop[1], qy);
  (void)rb_quantise(sz[f], pi.x0[2], pi.L[2], pi.S, pi.qtop[2], qz);
  const int sft = RB_DEPTH - l;
  CollNode r;
  r.cx = pi.x0[0] + ((double)(qx >> sft) + 0.5) * w;
  r.cy = pi.x0[1] + ((double)(qy >> sft) + 0.5) * w;
  r.cz = pi.x0[2] + ((double)(qz >> sft) + 0.5) * w;
  if (nleaf[node]) {
    const uint32_t span = nlast[node] - f;
    if (nlast[node] < f || span >= (1u << 26)) atomicOr(err, RB_ERR_TREE);
    r.a = f;
    r.b = 0x80000000u | ((uint32_t)l << 26) | (span & ((1u << 26) - 1u));
  } else {
    const uint32_t c0 = nchild[node], c1 = nlastchild[node];
    const bool ok = c1 >= c0 && c1 - c0 < 8;
    if (!ok) atomicOr(err, RB_ERR_TREE);
    r.a = c0;
    // a broken range is treated as a childless cell (flagged above)
    r.b = ((uint32_t)l << 26) | (ok ? c1 - c0 : 0u) | (ok ? 0u : 0x8u);
  }
  out[node] = r;
}

// One wave searches for SUB particles of a work item (consecutive sibling
// subtrees of at most group_size particles; an item is split into parts of
// SUB slots, one part per wave), 64 / SUB lanes per particle.  Four
// waves per workgroup, parts strided over the grid.
//
// STEP: the search at the end of a step, on the tree built mid-step.  The
// particles have moved by at most D (the largest displacement) since, and
// some have been wrapped into the box: the search runs on their unwrapped
// positions x^u = x + o(w) (w the image the wrap moved them out of) with
// every cell's reach widened by D, and a pair found through image k' of the
// unwrapped positions is the pair through image k' + w_j - w_i of the
// wrapped ones, where the contact test is evaluated.
template <bool STEP, uint32_t SUB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5, 8))) void k_coll_detect(
    const WalkItem *__restrict__ items, const WalkItem *__restrict__ items_mid,
    const uint32_t *__restrict__ gctr, uint64_t cap, const double *__restrict__ sx,
    const double *__restrict__ sy, const double *__restrict__ sz,
    const uint32_t *__restrict__ orig, const double *__restrict__ R,
    const PatchInfo *__restrict__ patch, const uint32_t *__restrict__ starts,
    const uint32_t *__restrict__ nlive, const uint32_t *__restrict__ root,
    const CollNode *__restrict__ cells, int ngx, int ngy, int boundary, double omega, double t,
    const unsigned long long *__restrict__ rmax_bits, CollQueue Q, uint32_t *__restrict__ err,
    const uint16_t *__restrict__ wrap, const unsigned long long *__restrict__ disp_bits,
    const double *__restrict__ sched, const uint32_t *__restrict__ ctr, int slot,
    uint32_t P) {
  constexpr uint32_t NS = 64 / SUB;  // parts per item (items hold <= 64 slots)
  __shared__ uint32_t stk_all[4][CG_SCAP];
  __shared__ uint32_t lfa_all[4][CG_LL], lfb_all[4][CG_LL], lsc_all[4][64];
  // staged candidates: position, radius, caller index, image (ix + 8) |
  // (iy + 8) << 4 of the unwrapped search plus the candidate's own wrap
  __shared__ double cx_all[4][64], cy_all[4][64], cz_all[4][64], cr_all[4][64];
  __shared__ uint32_t co_all[4][64];
  __shared__ uint8_t ck_all[4][64];
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t wv = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  uint32_t *stk = stk_all[wv];
  uint32_t *lfa = lfa_all[wv], *lfb = lfb_all[wv], *lsc = lsc_all[wv];
  double *cx_ = cx_all[wv], *cy_ = cy_all[wv], *cz_ = cz_all[wv], *cr_ = cr_all[wv];
  uint32_t *co_ = co_all[wv];
  uint8_t *ck_ = ck_all[wv];
  const uint32_t pidx = lane % SUB, sub = lane / SUB;
  const uint32_t n_big = gctr[2], n_mid = gctr[3], n_items = n_big + n_mid + gctr[4];
  const double rmax = __longlong_as_double((long long)rmax_bits[0]);
  const double slack = STEP ? __longlong_as_double((long long)disp_bits[0]) : 0.0;
  const double hd = 0.8660254037844386;  // half the diagonal of a unit cube
  const int n_img = (boundary == RB_OPEN) ? 1 : (2 * ngx + 1) * (2 * ngy + 1);
  const int ny = 2 * ngy + 1;
  const double *s_end = STEP ? sched + (size_t)ctr[slot] * 2 * P + P : nullptr;
  for (uint32_t u = 4u * blockIdx.x + wv; u < n_items * NS; u += 4u * gridDim.x) {
    const WalkItem it = rb_walk_item(items, items_mid, u / NS, n_big, n_mid, cap);
    const uint32_t s0 = it.start + (u % NS) * SUB;
    if (s0 >= it.end || it.end - it.start > 64u) continue;  // uniform
    const uint32_t p = it.patch, st = starts[p];
    const uint32_t s = s0 + pidx;
    bool act = s < it.end && s - st < nlive[p];
    if (STEP && act) act = !isnan(sx[s]);  // (left an open box this step)
    if (!__ballot(act)) continue;
    const PatchInfo pi = patch[p];
    const double W = pi.W;
    const double sh = (boundary != RB_SHEAR) ? 0.0
                      : STEP ? s_end[p] : remainder(1.5 * omega * W * t, W);
    const double xi = act ? sx[s] : 0.0, yi = act ? sy[s] : 0.0, zi = act ? sz[s] : 0.0;
    const uint32_t oi = act ? orig[s] : 0u;
    const double Ri = act ? R[oi] : 0.0;
    int wxi = 0, wyi = 0;  // the lane's own wrap
    double qx = xi, qy = yi;
    if (STEP && act) {
      const uint32_t wb = wrap[s];
      wxi = (int)(wb & 15u) - 2;
      wyi = (int)(wb >> 4) - 2;
      double ox, oy, wy;
      rb_coll_image_xy(wxi, wyi, boundary, W, sh, omega, ox, oy, wy);
      qx = xi + ox;
      qy = yi + oy;
    }
    const double lx = rb_wave_min_d(act ? qx : INFINITY);
    const double hx = rb_wave_max_d(act ? qx : -INFINITY);
    const double ly = rb_wave_min_d(act ? qy : INFINITY);
    const double hy = rb_wave_max_d(act ? qy : -INFINITY);
    const double lz = rb_wave_min_d(act ? zi : INFINITY);
    const double hz = rb_wave_max_d(act ? zi : -INFINITY);
    const double reach = rb_wave_max_d(act ? Ri : 0.0) + rmax + slack;
    uint64_t mine[RB_COLL_LOCAL];
    uint32_t nm = 0;
    for (int k = lane; k < n_img; k += 64) stk[k] = (root[p] << 5) | (uint32_t)k;
    int sp = n_img;
    int nl = 0;
    coll_wave_sync();
    for (;;) {
      int T = sp < 64 ? sp : 64;
      if (sp + 7 * T > CG_SCAP - CG_RESERVE) {
        T = (CG_SCAP - CG_RESERVE - sp) / 7;
        if (T < 1) T = (sp > 0) ? 1 : 0;
      }
      // test the opened leaves' particles against the lanes' particles: up
      // to 64 leaves at a time, their particles staged in LDS 64 at a time
      // (image-shifted, one load per lane), candidate q then tested by the
      // lanes with sub = q mod (64 / SUB)
      if (nl >= 64 || (T == 0 && nl > 0)) {
        for (int lb = 0; lb < nl; lb += 64) {
          const int L = min(64, nl - lb);
          const uint32_t cntq = (int)lane < L ? (lfb[lb + (int)lane] >> 5) + 1u : 0u;
          const uint32_t incl = rb_wave_incl_scan(cntq);
          const uint32_t M =
              (uint32_t)__builtin_amdgcn_readfirstlane((int)__shfl(incl, 63, 64));
          lsc[lane] = incl;
          coll_wave_sync();
          for (uint32_t e0 = 0; e0 < M; e0 += 64) {
            const uint32_t e = e0 + lane;
            if (e < M) {
              int lo = 0, hi = L - 1;  // first leaf whose inclusive count exceeds e
              while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (lsc[mid] > e) hi = mid; else lo = mid + 1;
              }
              const uint32_t eb = lfb[lb + lo];
              const uint32_t j = lfa[lb + lo] + (e - (lsc[lo] - ((eb >> 5) + 1u)));
              const int k = (int)(eb & 31u);
              const uint32_t oj = orig[j];
              if (STEP) {
                // raw position and the image relative to the box both wraps
                // are counted from (the lane's own wrap is taken off later)
                const uint32_t wb = wrap[j];
                const int kx = ((boundary == RB_OPEN) ? 0 : k / ny - ngx) + (int)(wb & 15u) - 2;
                const int ky = ((boundary == RB_OPEN) ? 0 : k % ny - ngy) + (int)(wb >> 4) - 2;
                cx_[lane] = sx[j];
                cy_[lane] = sy[j];
                ck_[lane] = (uint8_t)((kx + 8) | ((ky + 8) << 4));
              } else {
                // the image-shifted position (the lanes' particles are in the box)
                double ox, oy, wy;
                rb_coll_image(k, ngx, ngy, boundary, W, sh, omega, ox, oy, wy);
                cx_[lane] = sx[j] + ox;
                cy_[lane] = sy[j] + oy;
                ck_[lane] = (uint8_t)k;
              }
              cz_[lane] = sz[j];
              cr_[lane] = R[oj];
              co_[lane] = oj;
            }
            coll_wave_sync();
            const int C = (int)min(64u, M - e0);
            if (act) {
              for (int q = (int)sub; q < C; q += (int)NS) {
                const uint32_t oj = co_[q];
                if (oi >= oj) continue;  // each pair once, from its lower caller index
                const uint32_t kb = ck_[q];
                double d0, d1;
                uint32_t kc;
                if (STEP) {
                  // the image of j relative to i in the (wrapped) box
                  const int ix = (int)(kb & 15u) - 8 - wxi, iy = (int)(kb >> 4) - 8 - wyi;
                  if (ix < -ngx || ix > ngx || iy < -ngy || iy > ngy) continue;
                  double ox, oy, wy;
                  rb_coll_image_xy(ix, iy, boundary, W, sh, omega, ox, oy, wy);
                  d0 = (cx_[q] + ox) - xi;
                  d1 = (cy_[q] + oy) - yi;
                  kc = (boundary == RB_OPEN) ? 0u : (uint32_t)((ix + ngx) * ny + (iy + ngy));
                } else {
                  d0 = cx_[q] - xi;
                  d1 = cy_[q] - yi;
                  kc = (boundary == RB_OPEN) ? 0u : kb;
                }
                const double d2 = cz_[q] - zi;
                const double sum = Ri + cr_[q];
                if (d0 * d0 + d1 * d1 + d2 * d2 < sum * sum)
                  rb_coll_keep(((uint64_t)oi << 35) | ((uint64_t)oj << 7) | (uint64_t)kc,
                               mine, nm, Q);
              }
            }
            coll_wave_sync();
          }
        }
        nl = 0;
      }
      if (T == 0) break;  // uniform
      const int base = sp - T;
      const bool has = (int)lane < T;
      const uint32_t e = has ? stk[base + (int)lane] : 0u;
      coll_wave_sync();
      sp = base;
      bool open = false, leaf = false;
      uint32_t c0 = 0, nc = 0, span = 0;
      if (has) {
        const CollNode cn = cells[e >> 5];
        const int k = (int)(e & 31u);
        double ox, oy, wy;
        rb_coll_image(k, ngx, ngy, boundary, W, sh, omega, ox, oy, wy);
        const int l = (int)((cn.b >> 26) & 31u);
        const double w = ldexp(W, -l);
        const double cx = cn.cx + ox, cy = cn.cy + oy, cz = cn.cz;
        const double dx = fmax(fmax(lx - cx, cx - hx), 0.0);
        const double dy = fmax(fmax(ly - cy, cy - hy), 0.0);
        const double dz = fmax(fmax(lz - cz, cz - hz), 0.0);
        const double lim = (reach + hd * w) * (1.0 + 1e-9);
        open = dx * dx + dy * dy + dz * dz < lim * lim;
        leaf = (cn.b >> 31) != 0;
        c0 = cn.a;
        span = cn.b & ((1u << 26) - 1u);
        // (a flagged broken child range has bit 3 set and opens nothing)
        if (open && !leaf && span < 8u) nc = span + 1u;
      }
      // opened internal nodes push their children, opened leaves join the list
      const uint32_t incl = rb_wave_incl_scan(nc);
      const uint32_t tot = (uint32_t)__builtin_amdgcn_readfirstlane((int)__shfl(incl, 63, 64));
      if (sp + (int)tot > CG_SCAP) {  // cannot happen with the reserve above
        if (lane == 0) atomicOr(err, RB_ERR_STACK);
        break;
      }
      for (uint32_t q = 0; q < nc; ++q)
        stk[sp + (int)(incl - nc + q)] = ((c0 + q) << 5) | (e & 31u);
      sp += (int)tot;
      const uint64_t lm = __ballot(open && leaf);
      if (open && leaf) {
        const int at = nl + (int)rb_mbcnt(lm);
        lfa[at] = c0;
        lfb[at] = (span << 5) | (e & 31u);
      }
      nl += __popcll(lm);
      coll_wave_sync();
    }
    rb_coll_rest(mine, nm, Q);
  }
}

// Words that another thread of the same launch may just have written, or may
// read next, are loaded and exchanged at the device's coherent point.  An
// exchange that has returned has been performed there: coll_performed waits
// for the returned words, so whatever this thread sends out afterwards is
// seen only after them.
__device__ __forceinline__ double coll_ld(const double *p) {
  return __longlong_as_double((long long)__hip_atomic_load(
      reinterpret_cast<unsigned long long *>(const_cast<double *>(p)), __ATOMIC_RELAXED,
      __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ uint32_t coll_xchg(double *p, double v) {
  return (uint32_t)__hip_atomic_exchange(reinterpret_cast<unsigned long long *>(p),
                                         (unsigned long long)__double_as_longlong(v),
                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t coll_xchg(uint32_t *p, uint32_t v) {
  return __hip_atomic_exchange(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void coll_performed(uint32_t returned) {
  asm volatile("" ::"v"(returned) : "memory");
}

// Resolve the collision of code c if its particles approach (d . u < 0);
// returns whether it did.  Its predecessors are done and its successors wait
// for it, so no other thread uses the two velocities meanwhile.
// The arrays are in caller order, or (inv given: collisions inside a step)
// in the step's sorted order, inv mapping caller indices to slots; the
// shear offset is taken from the step's schedule row when s_end is given.
__device__ __forceinline__ bool rb_coll_apply(
    uint64_t c, const double *__restrict__ x, const double *__restrict__ y,
    const double *__restrict__ z, double *__restrict__ vx, double *__restrict__ vy,
    double *__restrict__ vz,
    const double *__restrict__ m, const PatchInfo *__restrict__ patch,
    const uint32_t *__restrict__ starts, uint32_t P, int ngx, int ngy, int boundary,
    double omega, double t, double eps, const uint32_t *__restrict__ inv = nullptr,
    const double *__restrict__ s_end = nullptr) {
  const uint32_t ci = (uint32_t)(c >> 35), cj = (uint32_t)((c >> 7) & ((1ull << 28) - 1ull));
  const int k = (int)(c & 127ull);
  // (patches hold the same ranges in caller and sorted order)
  const uint32_t p = (P == 1) ? 0u : rb_patch_of(starts, P, ci);
  const uint32_t i = inv ? inv[ci] : ci, j = inv ? inv[cj] : cj;
  const double W = patch[p].W;
  const double sh = (boundary != RB_SHEAR) ? 0.0
                    : s_end ? s_end[p] : remainder(1.5 * omega * W * t, W);
  double ox, oy, wy;
  rb_coll_image(k, ngx, ngy, boundary, W, sh, omega, ox, oy, wy);
  const double vi0 = coll_ld(vx + i), vi1 = coll_ld(vy + i), vi2 = coll_ld(vz + i);
  const double vj0 = coll_ld(vx + j), vj1 = coll_ld(vy + j), vj2 = coll_ld(vz + j);
  const double d0 = (x[j] + ox) - x[i];
  const double d1 = (y[j] + oy) - y[i];
  const double d2 = (z[j] + 0.0) - z[i];
  const double u0 = vj0 - vi0;
  const double u1 = (vj1 + wy) - vi1;
  const double u2 = vj2 - vi2;
  const double M = m[i] + m[j];
  if (!(d0 * u0 + d1 * u1 + d2 * u2 < 0.0 && M > 0.0)) return false;
  const double dist = sqrt(d0 * d0 + d1 * d1 + d2 * d2);
  const double n0 = d0 / dist, n1 = d1 / dist, n2 = d2 / dist;
  const double vn = n0 * u0 + n1 * u1 + n2 * u2;
  const double f = (1.0 + eps) * vn;
  const double fi = (m[j] / M) * f, fj = (m[i] / M) * f;
  coll_performed(coll_xchg(vx + i, vi0 + fi * n0) ^ coll_xchg(vy + i, vi1 + fi * n1) ^
                 coll_xchg(vz + i, vi2 + fi * n2) ^ coll_xchg(vx + j, vj0 - fj * n0) ^
                 coll_xchg(vy + j, vj1 - fj * n1) ^ coll_xchg(vz + j, vj2 - fj * n2));
  return true;
}

// Arrivals at a pair: three start it.  The owner thread brings one for
// itself and one for each side without a predecessor, once the pair's
// successors are written; every predecessor brings one.  The arrival that
// completes them runs the pair (nobody waits for anybody).  An arrival is
// sent only once the velocities and successors before it have been performed
// (coll_performed), so the thread that completes the pair loads them as they
// were left.  (Release and acquire fences instead write back and invalidate
// an XCD's whole L2 each time: 220,617 pairs took 2.10 ms per call with them,
// 1.03 ms this way.)
__device__ __forceinline__ uint32_t coll_arrive(uint32_t *arr, uint32_t q, uint32_t v) {
  return __hip_atomic_fetch_add(&arr[q], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + v;
}

// the queue's launch: one pair per thread up to 65,536 pairs
#define CR_BLOCKS 256
#define CR_THREADS 256u
#define CR_READY 256  // pairs ready to run that a wave's lanes share

// The whole queue in one launch, in the order of the keys h at every
// particle.  Thread by thread over the pairs: the pair's place among its
// particles' other pairs (the smallest later key of each side is its
// successor, an earlier key means it has a predecessor), then its arrival; a
// thread whose arrival completes a pair resolves it and follows its
// successors from there.  A thread that completes both keeps one and puts the
// other on its wave's stack, from which the lanes without a pair take theirs:
// threads whose arrival completes nothing have no work left, so where many
// particles overlap one another few threads complete all the rest (left to
// each thread by itself, a call on 80 particles in one place, 3,160 pairs, took
// 4.0 ms instead of 0.68, on 300, 44,850 pairs, 55.5 instead of 2.7; on the
// sheet of 50,000 with 28,553 pairs 279 instead of 252 us).
//
// Inside a step (inv given) the arrays are in the step's sorted order, inv
// maps caller indices to slots, the seed is the step's (seedp[0] + the step
// index), the shear offset the step's end-time offset, and the pairs and
// resolutions are added to the running totals in cum.  Being the last kernel
// before the host reads the counts, it copies the error word next to them
// (cnt[3]).
//
// Bound by latency: the links of the longest chain of dependent collisions,
// each a round trip for the pair's words, one for the velocities and one for
// the exchanges and arrivals.  A round at a time in one workgroup (three
// barriers and three passes over the list each), or, between calls, in three
// launches and the counts read back by the host every four rounds, against
// one launch: 50,000-particle settled sheet inside a step 282 -> 34 us; as a
// call 80 -> 41 us (9,938 pairs); ring with 27,939 pairs 234 -> 82 us.  With
// no pair at all the launch costs 1 us more than the one workgroup did.
__global__ __launch_bounds__(CR_THREADS) void k_coll_run(
    CollQueue Q, uint32_t *__restrict__ succ, uint64_t seed, const double *__restrict__ x,
    const double *__restrict__ y, const double *__restrict__ z, double *__restrict__ vx,
    double *__restrict__ vy, double *__restrict__ vz, const double *__restrict__ m,
    const PatchInfo *__restrict__ patch, const uint32_t *__restrict__ starts, uint32_t P,
    int ngx, int ngy, int boundary, double omega, double t, double eps,
    unsigned long long *__restrict__ n_res, const uint32_t *__restrict__ inv,
    const uint64_t *__restrict__ seedp, const double *__restrict__ sched,
    const uint32_t *__restrict__ ctr, int slot, unsigned long long *__restrict__ cum) {
  __shared__ uint32_t ready_all[CR_THREADS / 64][CR_READY];
  // a call that ends with an error (a full queue, whose pairs are no particular
  // ones, or any other) leaves the velocities as they were; nothing in this
  // launch writes the error word
  const uint32_t failed = inv ? 0u : Q.err[0];
  if (failed) {
    if (blockIdx.x == 0 && threadIdx.x == 0) Q.cnt[3] = failed;
    return;
  }
  const uint32_t n = min(Q.cnt[0], Q.cap);
  const double *s_end = inv ? sched + (size_t)ctr[slot] * 2 * P + P : nullptr;
  if (inv) seed = seedp[0] + ctr[slot];
  const uint32_t lane = rb_lane();
  uint32_t *ready = ready_all[__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6))];
  uint32_t done = 0;
  for (uint32_t own0 = blockIdx.x * CR_THREADS + (threadIdx.x & ~63u); own0 < n;
       own0 += gridDim.x * CR_THREADS) {  // uniform over the wave
    const uint32_t own = own0 + lane;
    // the pair to run, and a list of pairs ready to run after it (linked
    // through their arrival words, which nobody adds to any more)
    uint32_t run = RB_NONE, more = RB_NONE;
    if (own < n) {
      const uint64_t code = Q.code[own];
      const uint64_t h = rb_splitmix64(seed + code);
      uint32_t node[2] = {Q.head[rb_coll_i(code)], Q.head[rb_coll_j(code)]};
      uint64_t best[2] = {~0ull, ~0ull};
      uint32_t next[2] = {RB_NONE, RB_NONE};
      bool pred[2] = {false, false};
      while ((node[0] & node[1]) != RB_NONE) {  // both lists side by side
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          if (node[e] == RB_NONE) continue;
          const uint32_t q = node[e] >> 1;
          const uint64_t hq = rb_splitmix64(seed + Q.code[q]);
          node[e] = Q.link[node[e]];
          if (hq < h) pred[e] = true;
          if (hq > h && hq <= best[e]) {  // (the largest key there is counts too)
            best[e] = hq;
            next[e] = q;
          }
        }
      }
      coll_performed(coll_xchg(&succ[2 * (size_t)own], next[0]) ^
                     coll_xchg(&succ[2 * (size_t)own + 1], next[1]));
      if (coll_arrive(Q.arr, own, 3u - (pred[0] ? 1u : 0u) - (pred[1] ? 1u : 0u)) == 3u) run = own;
    }
    int n_ready = 0;  // on the wave's stack
    for (;;) {
      if (n_ready > 0) {  // idle lanes take ready pairs
        const bool idle = run == RB_NONE;
        const uint64_t im = __ballot(idle);
        const int k = (int)rb_mbcnt(im), take = min(n_ready, (int)__popcll(im));
        if (idle && k < take) run = ready[n_ready - 1 - k];
        n_ready -= take;
      }
      if (__ballot(run != RB_NONE) == 0) break;
      uint32_t also = RB_NONE;
      if (run != RB_NONE) {
        asm volatile("" ::: "memory");  // no load of the pair's words before its last arrival
        const uint32_t s0 = __hip_atomic_load(&succ[2 * (size_t)run], __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t s1 = __hip_atomic_load(&succ[2 * (size_t)run + 1], __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT);
        if (rb_coll_apply(Q.code[run], x, y, z, vx, vy, vz, m, patch, starts, P, ngx, ngy, boundary,
                          omega, t, eps, inv, s_end))
          ++done;
        run = RB_NONE;
        const uint32_t a0 = s0 != RB_NONE ? coll_arrive(Q.arr, s0, 1u) : 0u;
        const uint32_t a1 = s1 != RB_NONE ? coll_arrive(Q.arr, s1, 1u) : 0u;
        if (a0 == 3u) run = s0;
        if (a1 == 3u) {
          if (run == RB_NONE) run = s1;
          else also = s1;
        }
      }
      const uint64_t am = __ballot(also != RB_NONE);
      if (am) {  // a lane's second one goes on the stack, or on its own list when that is full
        const int at = n_ready + (int)rb_mbcnt(am);
        if (also != RB_NONE) {
          if (at < CR_READY) {
            ready[at] = also;
          } else {
            Q.arr[also] = more;
            more = also;
          }
        }
        n_ready = min(n_ready + (int)__popcll(am), CR_READY);
        coll_wave_sync();
      }
      if (run == RB_NONE && more != RB_NONE) {
        run = more;
        more = Q.arr[run];
      }
    }
  }
  for (int d = 32; d >= 1; d >>= 1) done += (uint32_t)__shfl_xor((int)done, d, 64);
  if (rb_lane() == 0 && done) {
    atomicAdd(n_res, (unsigned long long)done);
    if (cum) atomicAdd(&cum[1], (unsigned long long)done);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    Q.cnt[3] = Q.err[0];
    if (cum) cum[0] += (unsigned long long)n;
  }
}

// R_max, the cells' records and the work items of the search
hipError_t launch_coll_prep(rb_ctx *c, const double *radius) {
  const uint32_t n = (uint32_t)c->h_starts[c->P];
  if (n == 0) return hipSuccess;
  const unsigned grid = std::min(rb_div_up(n, 1024), 128u);
  hipLaunchKernelGGL(k_coll_rmax, dim3(grid), dim3(256), 0, c->stream, radius, c->d_orig[0],
                     c->d_starts, c->d_nlive, c->P, n, c->d_cmax, c->d_chead);
  CollNode *cells = reinterpret_cast<CollNode *>(c->d_cgeo);
  hipLaunchKernelGGL(k_coll_geom, dim3(rb_div_up(c->node_cap, 256)), dim3(256), 0, c->stream,
                     c->d_px[0][0], c->d_px[0][1], c->d_px[0][2], c->d_patch, c->d_starts, c->P,
                     c->d_lev_off, c->node_cap, c->d_nfirst, c->d_nlast, c->d_nchild,
                     c->d_nlastchild, c->d_nlevel, c->d_nleaf, cells, c->d_err, nullptr);
  return launch_groups(c);
}

// Particles per wave of the search: few where the waves are too few for the
// chip, many where they are plenty and share more of the descent (search, us,
// with 8 / 16 / 32: sheets of 5,000 particles 25 / 35 / 45, 20,000 45 / 43 / 62,
// 50,000 79 / 65 / 67, in a step 87 / 72 / 91, 200,000 264 / 179 / 144).
static int coll_sub(uint32_t n) { return n <= 15000 ? 8 : n <= 100000 ? 16 : 32; }

// about one wave per non-empty item part (parts average over half their
// particles); the loop strides over any others
static unsigned coll_grid(uint32_t n, int sub) {
  return std::min(4096u, rb_div_up(n, 4 * (uint64_t)sub / 2));
}

#define RB_COLL_DETECT(STEP, SUB, ...)                                                      \
  do {                                                                                      \
    const dim3 g(coll_grid(n, SUB)), b(256);                                                \
    if (SUB == 8) hipLaunchKernelGGL((k_coll_detect<STEP, 8>), g, b, 0, c->stream, __VA_ARGS__);        \
    else if (SUB == 16) hipLaunchKernelGGL((k_coll_detect<STEP, 16>), g, b, 0, c->stream, __VA_ARGS__); \
    else hipLaunchKernelGGL((k_coll_detect<STEP, 32>), g, b, 0, c->stream, __VA_ARGS__);                \
  } while (0)

hipError_t launch_coll_detect(rb_ctx *c, const double *radius, double t) {
  const uint32_t n = (uint32_t)c->h_starts[c->P];
  if (n == 0) return hipSuccess;
  CollNode *cells = reinterpret_cast<CollNode *>(c->d_cgeo);
  const int sub = coll_sub(n);
  RB_COLL_DETECT(false, sub, c->d_witems,
                     c->d_witems_mid, c->d_gctr, c->cap, c->d_px[0][0], c->d_px[0][1],
                     c->d_px[0][2], c->d_orig[0], radius, c->d_patch, c->d_starts, c->d_nlive,
                     c->d_root, cells, c->p.n_ghost[0], c->p.n_ghost[1], c->p.boundary,
                     c->p.omega, t, c->d_cmax, rb_coll_queue(c), c->d_err,
                     nullptr, nullptr, nullptr, nullptr, 0, c->P);
  return hipGetLastError();
}

// the queue that the search left, on the caller's arrays
hipError_t launch_coll_run(rb_ctx *c, const rb_particles *pp, double t, double eps,
                           uint64_t seed) {
  hipLaunchKernelGGL(k_coll_run, dim3(CR_BLOCKS), dim3(CR_THREADS), 0, c->stream, rb_coll_queue(c),
                     c->d_csucc, seed, pp->x, pp->y, pp->z, pp->vx, pp->vy, pp->vz, pp->m,
                     c->d_patch, c->d_starts, c->P, c->p.n_ghost[0], c->p.n_ghost[1],
                     c->p.boundary, c->p.omega, t, eps, c->d_cres, nullptr, nullptr, nullptr,
                     nullptr, 0, nullptr);
  return hipGetLastError();
}

// ---- collisions inside a step (the tree of the step, in its sorted order)

// before the kick: the cells' records from the build's (mid-step)
// positions in buffer buf and the step's counters cleared (R_max and the
// caller-to-slot map come from the first post kernel, k_post<1>)
hipError_t launch_coll_step_prep(rb_ctx *c, int buf) {
  const uint32_t n = (uint32_t)c->h_starts[c->P];
  if (n == 0) return hipSuccess;
  CollNode *cells = reinterpret_cast<CollNode *>(c->d_cgeo);
  hipLaunchKernelGGL(k_coll_geom, dim3(rb_div_up(c->node_cap, 256)), dim3(256), 0, c->stream,
                     c->d_px[buf][0], c->d_px[buf][1], c->d_px[buf][2], c->d_patch,
                     c->d_starts, c->P, c->d_lev_off, c->node_cap, c->d_nfirst, c->d_nlast,
                     c->d_nchild, c->d_nlastchild, c->d_nlevel, c->d_nleaf, cells, c->d_err,
                     c->d_ccnt);
  return hipGetLastError();
}

// after the second drift (the end-of-step state in buffer buf): the search
hipError_t launch_coll_step_search(rb_ctx *c, int buf, int slot) {
  const uint32_t n = (uint32_t)c->h_starts[c->P];
  if (n == 0) return hipSuccess;
  CollNode *cells = reinterpret_cast<CollNode *>(c->d_cgeo);
  const int sub = coll_sub(n);
  RB_COLL_DETECT(true, sub, c->d_witems,
                     c->d_witems_mid, c->d_gctr, c->cap, c->d_px[buf][0], c->d_px[buf][1],
                     c->d_px[buf][2], c->d_orig[buf], c->coll_R, c->d_patch, c->d_starts,
                     c->d_nlive, c->d_root, cells, c->p.n_ghost[0], c->p.n_ghost[1],
                     c->p.boundary, c->p.omega, 0.0, c->d_cmax, rb_coll_queue(c), c->d_err,
                     c->d_cwrap,
                     reinterpret_cast<const unsigned long long *>(c->d_ccnt + 8), c->d_sched,
                     c->d_ctr, slot, c->P);
  return hipGetLastError();
}

// then the queue, on the sorted state (without particles no search has
// cleared and filled the queue: it may still hold an earlier call's pairs)
hipError_t launch_coll_step_run(rb_ctx *c, int buf, int slot) {
  if (c->h_starts[c->P] == 0) return hipSuccess;
  double *const *b = c->d_px[buf];
  hipLaunchKernelGGL(k_coll_run, dim3(CR_BLOCKS), dim3(CR_THREADS), 0, c->stream, rb_coll_queue(c),
                     c->d_csucc, 0ull, b[0], b[1], b[2], b[3], b[4], b[5], b[6], c->d_patch,
                     c->d_starts, c->P, c->p.n_ghost[0], c->p.n_ghost[1], c->p.boundary,
                     c->p.omega, 0.0, c->coll_eps, c->d_cres, c->d_cinv,
                     reinterpret_cast<const uint64_t *>(c->d_ctr + 4), c->d_sched, c->d_ctr,
                     slot, reinterpret_cast<unsigned long long *>(c->d_ccnt + 10));
  return hipGetLastError();
}
