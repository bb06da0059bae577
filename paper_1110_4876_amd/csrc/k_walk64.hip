// k_walk64.hip -- per-particle FP64 tree walk (Sect. 4.2 of the paper).
//
// The result is the plain per-particle Barnes-Hut sum: every particle makes
// its own opening decisions, w^2 < theta^2 R^2 with R measured from its own
// position to the cell's centre of mass, and adds the terms of exactly the
// nodes that its own stackless walk (child link when opening, skip link
// otherwise) would visit.  The opening test, the image shifts and the term
// arithmetic round exactly as a plain sequential FP64 walk does, so the
// decisions are reproducible bit for bit; only the order of the sums differs
// between the schedules.
//
// k_walk64, the walk unless another schedule is asked for: rounds over a
// stack of opened nodes, four to sixteen waves per 64 Morton-consecutive
// particles (described there).
//
// k_walk64_parts (schedules 2 and 3): one wave takes 64 Morton-consecutive
// particles (one per lane) and walks the tree once for all of them.  The
// node in hand is the same for the whole wave, so its record is read with
// scalar loads; each lane tests it against its own particle.  A lane takes
// part in a node only if it opened every ancestor of that node; each lane
// keeps the deepest level down to which it did so along the current path,
// and a node of level l is its when that level is at least l.  Lanes that
// accept a cell add its monopole (and quadrupole) term; the wave descends to
// the children when any lane opened it and moves on to the next node after
// the subtree otherwise.
//
// k_walk64_lane (schedule 1): every lane follows its stackless walk on its
// own, with its own loads.
#include "rb_internal.h"

// 1 / sqrt(x): hardware estimate y (relative error ~2^-23) refined by one
// third-order step.  With e = 1 - x y^2, 1/sqrt(x) = y (1 - e)^(-1/2) =
// y (1 + e/2 + 3e^2/8 + O(e^3)), so one step takes the error from 2^-23 to
// ~2^-70, below the rounding of the last operations (about one ulp; two
// Newton steps give about two).
__device__ __forceinline__ double rb_rsqrt64(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = __builtin_fma(-(x * y), y, 1.0);
  return __builtin_fma(y * e, __builtin_fma(0.375, e, 0.5), y);
}

// The terms a particle adds (d = source - particle, rho^2 = |d|^2 + b^2):
//   monopole   G M d / rho^3
//   quadrupole (5/2) G (d.Q.d) d / rho^7 - G (Q d) / rho^5
// The monopole and the radial part of the quadrupole share the factor
// (G M + (5/2) G (d.Q.d) / rho^4) / rho^3, so a cell costs two fused
// multiply-adds per axis.
__device__ __forceinline__ void w64_mono(double Gm, double d0, double d1, double d2,
                                         double r2, double &ax, double &ay, double &az) {
  const double ri = rb_rsqrt64(r2);
  const double f = Gm * (ri * (ri * ri));
  ax = __builtin_fma(f, d0, ax);
  ay = __builtin_fma(f, d1, ay);
  az = __builtin_fma(f, d2, az);
}

template <bool QUAD>
__device__ __forceinline__ void w64_cell(double G, double Gm, const double *q, double d0,
                                         double d1, double d2, double rho2, double &ax,
                                         double &ay, double &az) {
  const double ri = rb_rsqrt64(rho2);
  const double u = ri * ri, g = ri * u;  // rho^-2, rho^-3
  if (QUAD) {
    const double e0 = __builtin_fma(q[0], d0, __builtin_fma(q[1], d1, q[2] * d2));
    const double e1 = __builtin_fma(q[1], d0, __builtin_fma(q[3], d1, q[4] * d2));
    const double e2 = __builtin_fma(q[2], d0, __builtin_fma(q[4], d1, q[5] * d2));
    const double dqd = __builtin_fma(d0, e0, __builtin_fma(d1, e1, d2 * e2));
    const double gs = g * __builtin_fma((2.5 * G) * dqd, u * u, Gm);
    const double gu = (G * g) * u;
    ax = __builtin_fma(-gu, e0, __builtin_fma(gs, d0, ax));
    ay = __builtin_fma(-gu, e1, __builtin_fma(gs, d1, ay));
    az = __builtin_fma(-gu, e2, __builtin_fma(gs, d2, az));
  } else {
    const double f = Gm * g;
    ax = __builtin_fma(f, d0, ax);
    ay = __builtin_fma(f, d1, ay);
    az = __builtin_fma(f, d2, az);
  }
}

// |d|^2 + b^2
__device__ __forceinline__ double w64_r2(double d0, double d1, double d2, double b2) {
  return __builtin_fma(d0, d0, __builtin_fma(d1, d1, __builtin_fma(d2, d2, b2)));
}

// image ordinal -> offset (ix Lx, iy Ly - ix s, 0), ix outer, iy inner; Lx, Ly
// the domain's extents
__device__ __forceinline__ void rb_image(int im, int ngx, int ngy, int boundary, double Lx,
                                         double Ly, double s, double &ox, double &oy,
                                         bool &self) {
  if (boundary == RB_OPEN) {
    ox = 0.0; oy = 0.0; self = true;
    return;
  }
  const int ny = 2 * ngy + 1;
  const int ix = im / ny - ngx, iy = im % ny - ngy;
  const double fx = (double)ix, fy = (double)iy;
  const double sh = (boundary == RB_SHEAR) ? s : 0.0;
  ox = fx * Lx;
  oy = fy * Ly - fx * sh;
  self = (ix == 0 && iy == 0);
}

// Node records read through the constant address space: the node index is
// uniform over the wave, so these become scalar loads.
typedef __attribute__((address_space(4))) const uint32_t *w64_u32_p;
typedef __attribute__((address_space(4))) const double *w64_dbl_p;

// a node's walk record, in scalar registers
struct W64Rec {
  uint32_t child, skip, count, lvl;
  double cx, cy, cz, m;
};

// A node's record.  With OFF32 the byte offsets of the node's records
// (16 v, 32 v and 48 v for its quadrupole) fit 32 bits, and the scalar
// loads take them as a register offset to the arrays' base, sparing the
// 64-bit address arithmetic of every visit.
template <bool OFF32>
__device__ __forceinline__ const void *w64_at(const void *base, uint32_t v, uint32_t bytes) {
  typedef __attribute__((address_space(4))) const char *cbyte;
  if (OFF32) return (const void *)((cbyte)base + v * bytes);
  return (const void *)((cbyte)base + (size_t)v * bytes);
}

template <bool OFF32>
__device__ __forceinline__ void w64_fetch(w64_u32_p link, w64_dbl_p mcom, uint32_t v,
                                          W64Rec &r) {
  const w64_u32_p lp = (w64_u32_p)w64_at<OFF32>((const void *)link, v, 16u);
  r.child = lp[0]; r.skip = lp[1]; r.count = lp[2]; r.lvl = lp[3];
  const w64_dbl_p mp = (w64_dbl_p)w64_at<OFF32>((const void *)mcom, v, 32u);
  r.cx = mp[0]; r.cy = mp[1]; r.cz = mp[2]; r.m = mp[3];
}

__device__ __forceinline__ uint32_t w64_uniform(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

// One wave per workgroup: a wave's slot on the CU is refilled as soon as it
// ends (with four waves per workgroup the slot waits for the slowest of the
// four; measured 2.6-5% slower).  Eight waves per SIMD: the register budget
// that allows them (78 scalar registers, against 106 unbounded) moves only
// set-up values out to vector lanes, none of the node loop's, and the extra
// waves cover more of the node loads' latency (measured 10% faster on the
// 256-patch ensemble).
template <bool QUAD, bool STATS, int PD, bool OFF32>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_walk64_parts(
    const WalkItem *__restrict__ items, uint32_t n_items, int img_split, int n_img, int parts,
    int ngx, int ngy, int boundary, const PatchInfo *__restrict__ patch,
    const uint32_t *__restrict__ nlive, const uint32_t *__restrict__ root,
    const NodeLink *__restrict__ link_g, const double4 *__restrict__ mcom_g,
    const double *__restrict__ Q_g, const double *__restrict__ sx_g,
    const double *__restrict__ sy_g, const double *__restrict__ sz_g,
    const double *__restrict__ msrc_g, const double *__restrict__ sched,
    const uint32_t *__restrict__ ctr, uint32_t P, double G, double b2, double theta2,
    double *__restrict__ acc, uint64_t cap, unsigned long long *__restrict__ stats,
    const uint32_t *__restrict__ lev_off, uint32_t *__restrict__ err, int slot,
    uint32_t *__restrict__ ord) {
  const w64_u32_p link = (w64_u32_p)link_g;
  const w64_dbl_p mcom = (w64_dbl_p)mcom_g;
  const w64_dbl_p Qarr = (w64_dbl_p)Q_g;
  const w64_dbl_p msrc = (w64_dbl_p)msrc_g;
  const w64_dbl_p sxc = (w64_dbl_p)sx_g, syc = (w64_dbl_p)sy_g, szc = (w64_dbl_p)sz_g;
  const uint32_t lane = threadIdx.x & 63u;
  // a unit: a part, an item and its image (when split).  With parts, each
  // part walks one subtree one or two levels below the root (PD levels:
  // 8^PD parts), so a system of few items still gives many units, each with
  // a short chain of node loads; every particle still sees each node once,
  // and the parts' sums are added in order afterwards.  Units are
  // part-major: neighbouring waves (and an XCD's range) walk the same
  // subtree for neighbouring particles and share its node records in the
  // caches.
  const uint32_t np = PD ? (uint32_t)parts : 1u;
  const uint32_t per_part = n_items * (img_split ? (uint32_t)n_img : 1u);
  const uint32_t n_units = per_part * np;
  // One unit per wave.  Workgroups are dealt to the eight XCDs in turn;
  // block b takes its unit from the (b mod 8)-th eighth of the units, so
  // each XCD's L2 holds the nodes of one contiguous eighth of them.  An
  // ordered launch (ctl) first runs the units listed as costly (the first
  // RB_WALK64_HEAVY_MAX blocks, spread over all XCDs), then the rest in
  // that order; a listed unit's own block there has nothing left to do.
  // (only the 64-part instance is ever launched ordered)
  constexpr bool ORD = PD == 2;
  W64Ctl *const ctl = ORD ? (W64Ctl *)ord : nullptr;
  uint32_t unit = 0;
  bool run;
  if (ORD && ctl && blockIdx.x < RB_WALK64_HEAVY_MAX) {  // a listed unit
    // XCD x = b mod 8 runs the list of its own share
    const uint32_t x = blockIdx.x & 7u, j = blockIdx.x >> 3;
    run = j < min(ctl->cnt[ctl->cur & 1u][x], RB_WALK64_HEAVY_MAX / 8u);
    if (run) unit = w64_uniform(ord[RB_W64_HEAVY_OFF + x * (RB_WALK64_HEAVY_MAX / 8u) + j]);
    run = run && unit < n_units;
  } else {  // the units in order (XCD x = b mod 8 either way)
    const uint32_t off = (ORD && ctl) ? RB_WALK64_HEAVY_MAX : 0u;
    const uint32_t b = blockIdx.x - off, nb = gridDim.x - off;
    const uint32_t q = nb >> 3, r = nb & 7u, x = b & 7u;
    unit = x * q + (x < r ? x : r) + (b >> 3);
    run = unit < n_units;  // whole waves
    if (ORD && ctl && run) run = w64_uniform(ord[RB_W64_TAG_OFF + unit]) != ctl->cur;
  }
  if (!run) return;
  // a depth-first walk visits every node at most once per image: more
  // visits, or an index past the node count, mean inconsistent links
  const uint32_t n_nodes = lev_off[RB_NLEV];
  const int part = (int)(unit / per_part);
  const uint32_t sub = unit % per_part;
  const uint32_t item = img_split ? sub / (uint32_t)n_img : sub;
  const int im0 = img_split ? (int)(sub % (uint32_t)n_img) : 0;
  const int im1 = img_split ? im0 + 1 : n_img;
  const WalkItem it = items[item];
  const uint32_t p = it.patch;
  const double W = patch[p].W;
  // (W 2^-l)^2 = fl(W W) 2^-2l exactly: scaling by a power of two is exact
  const double W2 = W * W;
  const int nvirt = (int)patch[p].nvirt;
  const uint32_t st = patch[p].start, nl = nlive[p];
  const uint32_t s = it.start + lane;
  const bool valid = s < it.end && (s - st) < nl;
  const double shear = sched[(size_t)ctr[slot] * 2 * P + p];
  double px = 0.0, py = 0.0, pz = 0.0;
  if (valid) { px = sx_g[s]; py = sy_g[s]; pz = sz_g[s]; }
  const uint64_t live = __ballot(valid);
  const uint32_t r0 = live ? w64_uniform(root[p]) : RB_NONE;
  uint32_t n_open = 0, n_cell = 0, n_pp = 0, n_visits = 0;
  double tx = 0.0, ty = 0.0, tz = 0.0;
  for (int im = im0; im < im1; ++im) {
    double ox, oy;
    bool self;
    rb_image(im, ngx, ngy, boundary, patch[p].L[0], patch[p].L[1], shear, ox, oy, self);
    const double y0 = px - ox, y1 = py - oy, y2 = pz;
    double ax = 0.0, ay = 0.0, az = 0.0;
    uint32_t cur = r0, visits = 0;
    // With parts, the octal digits of part k name a path below the root:
    // k = c (PD = 1) walks the subtree of the root's child c, k = 8 c + g
    // (PD = 2) that of grandchild g of child c.  Before that the part tests
    // the nodes on the path for its lanes (only the lanes that opened them
    // go on); a node's own terms belong to the first part below it (part 0
    // for the root, 8 c for child c), as does a leaf on the path (walked
    // below).  A part stops where its subtree ends: at the next sibling
    // (children are numbered consecutively, and in depth-first order a
    // subtree ends where the next sibling starts), or after the parent's
    // subtree for the last child.
    uint32_t stop = RB_NONE;
    uint64_t act0 = live;  // lanes active at the start node, and its level
    int l0 = 0;
    if (PD > 0 && cur != RB_NONE) {
      const uint32_t digit[2] = {PD == 2 ? (uint32_t)part >> 3 : (uint32_t)part,
                                 (uint32_t)part & 7u};
      uint32_t v = cur, after = RB_NONE;
      uint64_t act = live;
      cur = RB_NONE;
#pragma unroll
      for (int depth = 0; depth < PD; ++depth) {
        if (v >= n_nodes) {
          if (lane == 0) atomicOr(err, RB_ERR_TREE);
          break;
        }
        W64Rec rc;
        w64_fetch<OFF32>(link, mcom, v, rc);
        const int l = (int)(rc.lvl & 255u);
        const uint32_t n_child = rc.lvl >> 9;
        const bool owner = depth == 0 ? part == 0 : digit[1] == 0u;
        if (rc.m == 0.0 || l > RB_DEPTH) break;
        if ((rc.lvl & 256u) != 0u) {  // a leaf: its owner walks it
          if (owner) { cur = v; stop = after; act0 = act; l0 = l; }
          break;
        }
        const bool me = ((act >> lane) & 1ull) != 0;
        const double d0 = rc.cx - y0, d1 = rc.cy - y1, d2 = rc.cz - y2;
        const double R2 = __builtin_fma(d2, d2, __builtin_fma(d1, d1, d0 * d0));
        const bool root_or_below = l >= nvirt;
        const bool take = me && root_or_below && (ldexp(W2, -2 * l) < theta2 * R2);
        const uint64_t opened = act & ~__ballot(take);
        if (owner) {
          if (STATS && me && root_or_below) ++n_open;
          if (take) {
            const w64_dbl_p qn = (w64_dbl_p)w64_at<OFF32>((const void *)Qarr, v, 48u);
            const double q[6] = {qn[0], qn[1], qn[2], qn[3], qn[4], qn[5]};
            w64_cell<QUAD>(G, G * rc.m, q, d0, d1, d2, R2 + b2, ax, ay, az);
            if (STATS) ++n_cell;
          }
        }
        const uint32_t dg = digit[depth];
        if (opened == 0ull || dg >= n_child || l >= RB_DEPTH) break;
        const uint32_t w = rc.child + dg;
        after = (dg + 1u < n_child) ? w + 1u : rc.skip;
        act = opened;
        v = w;
        if (depth == PD - 1) { cur = w; stop = after; act0 = opened; l0 = l + 1; }
      }
    }
    // A lane works on a node of level l when it opened every ancestor of
    // the node.  Along the path from the root to the node in hand those are
    // the levels 0..a of a prefix, and alev holds a (below the start node's
    // level when the lane takes no part): a node of level l is the lane's
    // when alev >= l.  When the wave descends from a node of level l, the
    // lanes working on it set alev to l + 1 if they opened it and to l if
    // they did not; nothing else changes alev.  A lane that opened the
    // parent of a node keeps alev >= its level through the earlier
    // siblings' subtrees (every change there sets alev to a deeper level),
    // and one that did not never works below the parent, so alev >= l
    // is exactly the rule.
    int alev = ((act0 >> lane) & 1ull) ? l0 : -1;
    // the node in hand: NodeLink {child_or_first, skip, count, lvl} and
    // double4 {com, M}, read with scalar loads; the other waves on the SIMD
    // cover their latency.  A walk ends at its stop node (RB_NONE for the
    // whole tree); an index past the node count before that, or more
    // visits than nodes, mean inconsistent links.
    while (cur != stop && max(cur, visits) < n_nodes) {
      ++visits;
      W64Rec rc;
      w64_fetch<OFF32>(link, mcom, cur, rc);
      const uint32_t lv = rc.lvl;
      const int l = (int)(lv & 255u);
      const bool leaf = (lv & 256u) != 0;
      const double d0 = rc.cx - y0, d1 = rc.cy - y1, d2 = rc.cz - y2;
      uint32_t next = rc.skip;
      if (rc.m != 0.0) {
        const bool me = alev >= l;
        const bool single = leaf && rc.count == 1;
        // a single-particle leaf is taken by every lane but its own
        // particle's; a cell below the root boxes by the lanes it passes
        bool take;
        double rho2;
        uint64_t opened = 0ull;
        if (single) {
          take = me && !(self && rc.child == s);
          rho2 = w64_r2(d0, d1, d2, b2);
        } else {
          const double R2 = __builtin_fma(d2, d2, __builtin_fma(d1, d1, d0 * d0));
          // cells above the root boxes are always opened
          const bool root_or_below = l >= nvirt;
          take = me && root_or_below && (ldexp(W2, -2 * l) < theta2 * R2);
          opened = __ballot(me && !take);
          rho2 = R2 + b2;
          if (STATS && me && root_or_below) ++n_open;
        }
        if (take) {
          // one body for both: a single-particle leaf's quadrupole is
          // exactly zero (the build adds none for one particle), and with
          // Q d = 0 and d.Q.d = 0 the cell's terms reduce exactly to the
          // point mass's G M d / rho^3
          const double ri = rb_rsqrt64(rho2);
          const double u = ri * ri, g = ri * u;
          double e0 = 0.0, e1 = 0.0, e2 = 0.0, dqd = 0.0;
          if (QUAD) {
            const w64_dbl_p qn = (w64_dbl_p)w64_at<OFF32>((const void *)Qarr, cur, 48u);
            const double q0 = qn[0], q1 = qn[1], q2 = qn[2], q3 = qn[3], q4 = qn[4], q5 = qn[5];
            e0 = __builtin_fma(q0, d0, __builtin_fma(q1, d1, q2 * d2));
            e1 = __builtin_fma(q1, d0, __builtin_fma(q3, d1, q4 * d2));
            e2 = __builtin_fma(q2, d0, __builtin_fma(q4, d1, q5 * d2));
            dqd = __builtin_fma(d0, e0, __builtin_fma(d1, e1, d2 * e2));
          }
          const double gs = g * __builtin_fma((2.5 * G) * dqd, u * u, G * rc.m);
          const double gu = (G * g) * u;
          ax = __builtin_fma(-gu, e0, __builtin_fma(gs, d0, ax));
          ay = __builtin_fma(-gu, e1, __builtin_fma(gs, d1, ay));
          az = __builtin_fma(-gu, e2, __builtin_fma(gs, d2, az));
          if (STATS) { if (single) ++n_pp; else ++n_cell; }
        }
        if (opened != 0ull) {
          if (leaf) {
            // a bucket leaf that failed the test: its members one by one
            const bool mine = ((opened >> lane) & 1ull) != 0;
            const uint32_t j0 = rc.child, j1 = j0 + rc.count;
            for (uint32_t j = j0; j < j1; ++j) {
              const double mj = msrc[j];
              if (mj == 0.0) continue;
              if (mine && !(self && j == s)) {
                const double f0 = sxc[j] - y0, f1 = syc[j] - y1, f2 = szc[j] - y2;
                w64_mono(G * mj, f0, f1, f2, w64_r2(f0, f1, f2, b2), ax, ay, az);
                if (STATS) ++n_pp;
              }
            }
          } else {
            if (me) alev = take ? l : l + 1;
            next = rc.child;
          }
        }
      }
      cur = w64_uniform(next);
    }
    if (cur != stop && lane == 0) atomicOr(err, RB_ERR_TREE);
    n_visits += visits;
    if (img_split) {
      if (s < it.end) {
        double *a = acc + ((size_t)im * np + part) * 3 * cap;
        a[s] = ax; a[cap + s] = ay; a[2 * cap + s] = az;
      }
    } else {
      tx += ax; ty += ay; tz += az;
    }
  }
  if (!img_split && s < it.end) {
    double *a = acc + (size_t)part * 3 * cap;
    a[s] = tx; a[cap + s] = ty; a[2 * cap + s] = tz;
  }
  if (ORD && ctl && lane == 0) ord[RB_W64_COST_OFF + unit] = n_visits;
  if (STATS) {
    unsigned long long o = n_open, c = n_cell, q2 = n_pp;
    for (int d = 32; d >= 1; d >>= 1) {
      o += __shfl_xor(o, d, 64);
      c += __shfl_xor(c, d, 64);
      q2 += __shfl_xor(q2, d, 64);
    }
    if (lane == 0) {
      atomicAdd(&stats[0], o);
      atomicAdd(&stats[1], c);
      atomicAdd(&stats[2], q2);
    }
  }
}

// ---------------------------------------------------------------------------
// The walk of 64 Morton-consecutive particles (one per lane) as rounds over a
// stack of opened nodes, NW waves per item.
//
// An entry of the stack names the children of an opened node, the ghost
// image, and the lanes (a 64-bit mask) that opened the node and all its
// ancestors: the particles that work on the children.  A round takes up to
// eight entries per wave, one child per lane, and sorts the children by the
// opening test over the item's whole bounding box:
//   accepted by every lane   -- the cell's terms are added for the lanes of
//                               the mask, without a test per lane;
//   opened by every lane     -- the children are pushed with the same mask;
//   neither                  -- every lane tests the cell on its own: those
//                               that accept it add its terms, the others are
//                               the mask its children are pushed with.
// The box tests decide exactly as the lanes' own tests would.  A lane's test
// compares fl(theta^2 R^2) with R^2 = fma(dz, dz, fma(dy, dy, dx dx)) and
// d = fl(c - fl(x - o)); rounding is monotone, so the same expression over
// the smallest (largest) |d| per axis that fl(c - y) takes on the box's
// corners y bounds every lane's value from below (above), rounding included.
// So every particle sees exactly the nodes its own stackless walk sees.
//
// Bound by FP64 issue: on 256 sheets of 2,000 to 64,000 particles (four
// waves) the vector units are busy 91% of the time and issue 0.85 of a vector
// instruction per SIMD and quad-cycle, with 53% of their lanes at work (the
// lanes of a mask; 64 particles of a thin sheet need 1.9 times the nodes that
// one needs); on 1,048,583 particles of a sphere 93%, 0.87 and 64%; on one
// sheet of 50,000 (eight waves, 782 items) 58%, 0.55 and 53%.  A cell costs 36
// FP64 operations and one FP32 reciprocal root, its record arriving by scalar
// loads; with the opening tests and the particles' pairs, 60 vector and 26
// scalar instructions are issued for a wave's cell.  Against the node-by-node
// walk of k_walk64_parts, opened nodes cost one lane of a round instead of a
// visit of the whole wave, accepted cells need no test, and the scalar
// instructions of the launch are half (256 sheets 9.2e9; the parts' rate of
// 0.60 per CU and cycle over their 50 ms is 1.8e10).  Whole calls, parts -> rounds:
// 1,024-particle sphere 155 -> 143 us; four steps of the 50,000-particle
// sheet 2.57 -> 2.15 ms (64 accumulator sets per particle become one; 1.84 with
// shared ends, below); a step
// of 64 patches (2.1e6 particles) 13.4 -> 11.1 ms; 1,048,583-particle sphere
// 13.6 -> 10.6 ms (of these, FP32's start of the cells' reciprocal roots:
// 88 instead of 95 ns per cell and SIMD).
//
// NW: sixteen waves share an item below RB_WALK64_WAVES16 items, eight below
// RB_WALK64_WAVES8, four above (FP64 steps, us, at NW = 4 / 8 / 16, with whole
// items only: sheets of 50,000 743 / 611 / 579, 100,000 1074 / 934 / 947, 250,000 2008 / 1922 /
// 2087, 700,000 5090 / 5145 / 5756; one wave is slower than four throughout,
// 11.6 against 11.4 ms on 64 patches: four waves read a common part of the
// tree).  The items of small patches, and the last ones of larger patches that
// an XCD is dealt, are shared by several workgroups (rb_internal.h): all
// walk the item from the root until the stack holds W64G_SHARE entries for
// each, the first alone adding what is accepted on the way; then each keeps
// its own, and writes an accumulator set of its own.  (Shares of 4 entries are
// uneven -- the item's own subtree is one entry -- and of 32 walk too much of
// the tree together: two per item, 6,000 particles, 357 / 307 / 312 us.)
#define W64G_ENTRY 16  // bytes per stack entry
#define W64G_SHARE 8   // stack entries per part when the parts take their shares
// entries that depth-first descent may need on top of a full stack: one
// entry popped and at most eight pushed per level
#define W64G_RESERVE (7 * RB_DEPTH + 8)

// stack entries per item: the rounds' full width while it holds less than
// CAP - RESERVE - 56 NW
template <int NW>
constexpr int w64g_cap() {
  return 512 + 64 * NW;
}

__device__ __forceinline__ double w64_readlane_d(double v, int j) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, j);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), j);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

__device__ __forceinline__ uint64_t w64_readlane_u64(uint32_t lo, uint32_t hi, int j) {
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)hi, j) << 32) |
         (uint32_t)__builtin_amdgcn_readlane((int)lo, j);
}

__device__ __forceinline__ double w64_wave_min(double v) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) v = fmin(v, __shfl_xor(v, d, 64));
  return w64_readlane_d(v, 0);
}

__device__ __forceinline__ double w64_wave_max(double v) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) v = fmax(v, __shfl_xor(v, d, 64));
  return w64_readlane_d(v, 0);
}

// 1 / sqrt(x) as rb_rsqrt64, from FP32's estimate of the rounded x (as good a
// start, about 2^-23 with the rounding of x, in less than half the time of
// the FP64 instruction); for x whose FP32 value is normal and finite.
__device__ __forceinline__ double w64_rsqrt_f32(double x) {
  const double y = (double)__builtin_amdgcn_rsqf((float)x);
  const double e = __builtin_fma(-(x * y), y, 1.0);
  return __builtin_fma(y * e, __builtin_fma(0.375, e, 0.5), y);
}

// A node as the rounds' evaluation reads it, in scalar registers: centre of
// mass, mass, quadrupole (not read for point masses).
struct W64Node {
  double cx, cy, cz, m, q0, q1, q2, q3, q4, q5;
};

template <bool Q, bool OFF32>
__device__ __forceinline__ void w64g_load(w64_dbl_p mcom, w64_dbl_p Qarr, uint32_t v, W64Node &r) {
  const w64_dbl_p mp = (w64_dbl_p)w64_at<OFF32>((const void *)mcom, v, 32u);
  r.cx = mp[0]; r.cy = mp[1]; r.cz = mp[2]; r.m = mp[3];
  if (Q) {
    const w64_dbl_p qp = (w64_dbl_p)w64_at<OFF32>((const void *)Qarr, v, 48u);
    r.q0 = qp[0]; r.q1 = qp[1]; r.q2 = qp[2]; r.q3 = qp[3]; r.q4 = qp[4]; r.q5 = qp[5];
  }
}

// The terms of a cell (per unit G) for the lanes that call it.
template <bool QUAD, bool RS32>
__device__ __forceinline__ void w64g_cell(const W64Node &n, double d0, double d1, double d2,
                                          double rho2, double &ax, double &ay, double &az) {
  const double ri = RS32 ? w64_rsqrt_f32(rho2) : rb_rsqrt64(rho2);
  const double u = ri * ri, g = ri * u;  // rho^-2, rho^-3
  if (QUAD) {
    const double e0 = __builtin_fma(n.q0, d0, __builtin_fma(n.q1, d1, n.q2 * d2));
    const double e1 = __builtin_fma(n.q1, d0, __builtin_fma(n.q3, d1, n.q4 * d2));
    const double e2 = __builtin_fma(n.q2, d0, __builtin_fma(n.q4, d1, n.q5 * d2));
    const double dqd = __builtin_fma(d0, e0, __builtin_fma(d1, e1, d2 * e2));
    const double gs = g * __builtin_fma(2.5 * dqd, u * u, n.m);
    const double gu = g * u;
    ax = __builtin_fma(-gu, e0, __builtin_fma(gs, d0, ax));
    ay = __builtin_fma(-gu, e1, __builtin_fma(gs, d1, ay));
    az = __builtin_fma(-gu, e2, __builtin_fma(gs, d2, az));
  } else {
    const double f = g * n.m;
    ax = __builtin_fma(f, d0, ax);
    ay = __builtin_fma(f, d1, ay);
    az = __builtin_fma(f, d2, az);
  }
}

template <bool QUAD, bool STATS, int NW, bool RS32, bool OFF32>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_walk64(
    const WalkItem *__restrict__ items, uint32_t n_units, int img_split, int n_sets, int n_img,
    int ngx, int ngy, int boundary, const PatchInfo *__restrict__ patch,
    const uint32_t *__restrict__ nlive, const uint32_t *__restrict__ root,
    const NodeLink *__restrict__ link, const double4 *__restrict__ mcom_g,
    const double *__restrict__ Q_g, const double *__restrict__ sx_g,
    const double *__restrict__ sy_g, const double *__restrict__ sz_g,
    const double *__restrict__ msrc_g, const double *__restrict__ sched,
    const uint32_t *__restrict__ ctr, uint32_t P, double G, double b2, double theta2,
    double *__restrict__ acc, uint64_t cap, unsigned long long *__restrict__ stats,
    const uint32_t *__restrict__ lev_off, uint32_t *__restrict__ err, int slot) {
  constexpr int CAP = w64g_cap<NW>();
  // the stack's memory also takes the waves' partial sums at the end
  static_assert(CAP * W64G_ENTRY >= NW * 3 * 64 * 8, "reduction space");
  static_assert(sizeof(uint4) == W64G_ENTRY, "stack entry");
  __shared__ uint4 stk[CAP];
  __shared__ uint32_t s_push[NW];
  __shared__ double2 img[RB_MAX_IMAGES];
  const w64_dbl_p mcom = (w64_dbl_p)mcom_g;
  const w64_dbl_p Qarr = (w64_dbl_p)Q_g;
  const w64_dbl_p msrc = (w64_dbl_p)msrc_g;
  const w64_dbl_p sxc = (w64_dbl_p)sx_g, syc = (w64_dbl_p)sy_g, szc = (w64_dbl_p)sz_g;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t w = w64_uniform(threadIdx.x >> 6);
  // workgroups are dealt to the eight XCDs in turn; workgroup b takes its
  // unit from the (b mod 8)-th eighth, so that each XCD's L2 holds the nodes
  // of one contiguous eighth of them
  const uint32_t nb = gridDim.x, xq = nb >> 3, xr = nb & 7u, xcd = blockIdx.x & 7u;
  const uint32_t unit = xcd * xq + (xcd < xr ? xcd : xr) + (blockIdx.x >> 3);
  if (unit >= n_units) return;  // whole workgroups
  const uint32_t n_nodes = lev_off[RB_NLEV];
  const uint32_t item = img_split ? unit / (uint32_t)n_img : unit;
  const int im0 = img_split ? (int)(unit % (uint32_t)n_img) : 0;
  const int nim = img_split ? 1 : n_img;
  const WalkItem it = items[item];
  // the item's workgroups, and which of them this is (a split walk has one);
  // before they take their shares of the stack, the first one alone adds
  const int parts = (int)(it.node >> 8), part = (int)(it.node & 255u);
  // (eight and sixteen waves only: what four's compiler sees is constant)
  bool whole = NW >= 8 && parts > 1, adds = !whole || part == 0;
  const uint32_t p = it.patch;
  const double W = patch[p].W;
  // (W 2^-l)^2 = fl(W W) 2^-2l exactly: scaling by a power of two is exact
  const double W2 = W * W;
  const int nvirt = (int)patch[p].nvirt;
  const uint32_t st = patch[p].start, nl = nlive[p];
  const uint32_t s = it.start + lane;
  const bool valid = s < it.end && (s - st) < nl;
  double px = 0.0, py = 0.0, pz = 0.0;
  if (valid) { px = sx_g[s]; py = sy_g[s]; pz = sz_g[s]; }
  const uint64_t live = __ballot(valid);
  const uint32_t r0 = live ? w64_uniform(root[p]) : RB_NONE;
  // the item's box
  const double lx = w64_wave_min(valid ? px : INFINITY), hx = w64_wave_max(valid ? px : -INFINITY);
  const double ly = w64_wave_min(valid ? py : INFINITY), hy = w64_wave_max(valid ? py : -INFINITY);
  const double lz = w64_wave_min(valid ? pz : INFINITY), hz = w64_wave_max(valid ? pz : -INFINITY);
  if (threadIdx.x < (uint32_t)n_img) {
    double ox, oy;
    bool self;
    rb_image((int)threadIdx.x, ngx, ngy, boundary, patch[p].L[0], patch[p].L[1],
             sched[(size_t)ctr[slot] * 2 * P + p], ox, oy, self);
    img[threadIdx.x] = make_double2(ox, oy);
  }
  int sp = 0;
  if (r0 != RB_NONE) {
    if (r0 < n_nodes) {
      sp = nim;
      if (threadIdx.x < (uint32_t)nim)
        stk[threadIdx.x] = make_uint4(r0, 1u | ((uint32_t)(im0 + (int)threadIdx.x) << 8),
                                      (uint32_t)live, (uint32_t)(live >> 32));
    } else if (threadIdx.x == 0) {
      atomicOr(err, RB_ERR_TREE);
    }
  }
  const uint32_t self_img = (uint32_t)(n_img / 2);  // the ghost rings' centre
  uint32_t n_open = 0, n_cell = 0, n_pp = 0;
  double ax = 0.0, ay = 0.0, az = 0.0;
  // the image in hand and the particle as it sees it
  uint32_t cur_img = RB_NONE;
  double y0 = 0.0, y1 = 0.0;
  auto to_image = [&](uint32_t im) {
    if (im != cur_img) {  // uniform
      cur_img = im;
      const double2 o = img[im];
      y0 = px - o.x;
      y1 = py - o.y;
    }
  };
  __syncthreads();
  for (;;) {
    if (NW >= 8 && whole && sp >= W64G_SHARE * parts && sp <= 64 * NW) {
      // every part keeps each parts-th entry (neighbours on the stack are
      // siblings) and adds from here on
      const int keep = (sp - part + parts - 1) / parts;
      uint4 en = make_uint4(0u, 0u, 0u, 0u);
      if ((int)threadIdx.x < keep) en = stk[(int)threadIdx.x * parts + part];
      __syncthreads();
      if ((int)threadIdx.x < keep) stk[threadIdx.x] = en;
      __syncthreads();
      sp = keep;
      whole = false;
      adds = true;
    }
    // entries of this round: eight per wave, dealt to the waves in turn
    int k = sp < 8 * NW ? sp : 8 * NW;
    if (sp + 7 * k > CAP - W64G_RESERVE) {
      k = (CAP - W64G_RESERVE - sp) / 7;
      if (k < 1) k = sp > 0 ? 1 : 0;
    }
    if (k == 0) break;  // the same in every wave
    const int pi = (int)(lane >> 3) * NW + (int)w;
    uint4 en = make_uint4(0u, 0u, 0u, 0u);
    if (pi < k) en = stk[sp - 1 - pi];
    const uint32_t c8 = lane & 7u, node = en.x + c8, im = en.y >> 8;
    const bool has = c8 < (en.y & 255u);
    NodeLink lk = {0u, 0u, 0u, 0u};
    double4 mc = make_double4(0.0, 0.0, 0.0, 0.0);
    if (has) {
      lk = link[node];
      mc = mcom_g[node];
    }
    const double2 io = img[has ? im : 0u];
    const int l = (int)(lk.lvl & 255u);
    const bool leaf = (lk.lvl & 256u) != 0;
    const uint32_t nch = lk.lvl >> 9;
    const bool alive = has && mc.w != 0.0;
    const bool single = alive && leaf && lk.count == 1u;
    uint32_t mlo = en.z, mhi = en.w;
    // smallest and largest distance per axis, as the lanes' tests round them
    const double xa = mc.x - (lx - io.x), xb = mc.x - (hx - io.x);
    const double ya = mc.y - (ly - io.y), yb = mc.y - (hy - io.y);
    const double za = mc.z - lz, zb = mc.z - hz;
    const double nx = fmax(fmax(xb, -xa), 0.0), fx = fmax(fabs(xa), fabs(xb));
    const double ny = fmax(fmax(yb, -ya), 0.0), fy = fmax(fabs(ya), fabs(yb));
    const double nz = fmax(fmax(zb, -za), 0.0), fz = fmax(fabs(za), fabs(zb));
    const double near2 = __builtin_fma(nz, nz, __builtin_fma(ny, ny, nx * nx));
    const double far2 = __builtin_fma(fz, fz, __builtin_fma(fy, fy, fx * fx));
    const double w2 = ldexp(W2, -2 * l);
    const bool cell = alive && !single;
    // cells above the root boxes are always opened; a centre that is no
    // number is opened, as by the lanes (their comparison fails)
    const bool below = l >= nvirt;
    const bool ordered = mc.x == mc.x && mc.y == mc.y && mc.z == mc.z;
    const bool all_in = cell && below && ordered && w2 < theta2 * near2;
    const bool all_out = cell && !(below && ordered && w2 < theta2 * far2);
    const bool mixed = cell && !all_in && !all_out;
    if (single && im == self_img) {
      // every lane but the particle itself
      const uint32_t own = lk.child_or_first - it.start;
      if (own < 32u) mlo &= ~(1u << own);
      else if (own < 64u) mhi &= ~(1u << (own - 32u));
    }
    if (STATS && adds) {
      const uint32_t cnt = (uint32_t)(__popc(mlo) + __popc(mhi));
      if (cell && below) n_open += cnt;
      if (all_in) n_cell += cnt;
      if (single) n_pp += cnt;
    }
    // The children of one entry share its image, its mask and their level, and
    // are numbered consecutively: everything but the child's number is read
    // from lane 8 q once per entry.
    const uint64_t b_mixed = __ballot(mixed);
    const int n_mine = k > (int)w ? (k - (int)w + NW - 1) / NW : 0;
    // the lanes that open the cell: all of the mask, or as they find
    uint32_t plo = all_out ? mlo : 0u, phi = all_out ? mhi : 0u;
    for (int q8 = 0; q8 < 8 * n_mine; q8 += 8) {
      uint32_t m = (uint32_t)(b_mixed >> q8) & 255u;
      if (m == 0u) continue;
      const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)node, q8);
      const uint64_t mask = w64_readlane_u64(en.z, en.w, q8);
      const double w2q = w64_readlane_d(w2, q8 + __builtin_ctz(m));
      to_image((uint32_t)__builtin_amdgcn_readlane((int)im, q8));
      do {
        const uint32_t c = (uint32_t)__builtin_ctz(m);
        m &= m - 1u;
        W64Node nd;
        w64g_load<QUAD, OFF32>(mcom, Qarr, first + c, nd);
        const double d0 = nd.cx - y0, d1 = nd.cy - y1, d2 = nd.cz - pz;
        const double R2 = __builtin_fma(d2, d2, __builtin_fma(d1, d1, d0 * d0));
        const bool take = __builtin_amdgcn_inverse_ballot_w64(mask) && w2q < theta2 * R2;
        const uint64_t opened = mask & ~__ballot(take);
        if (take && adds) {
          w64g_cell<QUAD, RS32>(nd, d0, d1, d2, R2 + b2, ax, ay, az);
          if (STATS) ++n_cell;
        }
        if (lane == (uint32_t)q8 + c) { plo = (uint32_t)opened; phi = (uint32_t)(opened >> 32); }
      } while (m);
    }
    // opened nodes onto the stack (children are numbered after their parent,
    // so the descent ends), opened bucket leaves to be summed below
    const bool opens = (plo | phi) != 0u;
    bool push = opens && !leaf;
    if (push && !(lk.child_or_first > node && nch >= 1u && nch <= 8u && lk.child_or_first < n_nodes &&
                  nch <= n_nodes - lk.child_or_first)) {
      atomicOr(err, RB_ERR_TREE);
      push = false;
    }
    const uint64_t pm = __ballot(push);
    if (lane == 0) s_push[w] = (uint32_t)__popcll(pm);
    __syncthreads();  // every wave has read its entries; counts known
    int at = sp - k, all = 0;
#pragma unroll
    for (int q = 0; q < NW; ++q) {
      const int t = (int)s_push[q];
      if (q < (int)w) at += t;
      all += t;
    }
    sp = sp - k + all;
    if (sp > CAP) {  // cannot happen with the reserve above
      if (threadIdx.x == 0) atomicOr(err, RB_ERR_STACK);
      sp = 0;
    } else if (push) {
      stk[at + (int)rb_mbcnt(pm)] = make_uint4(lk.child_or_first, nch | (im << 8), plo, phi);
    }
    // accepted cells, then single-particle leaves
    const uint64_t b_in = adds ? __ballot(all_in) : 0ull;
    const uint64_t b_single = adds ? __ballot(single) : 0ull;
    for (int q8 = 0; q8 < 8 * n_mine; q8 += 8) {
      uint32_t m = (uint32_t)(b_in >> q8) & 255u;
      uint32_t ms = (uint32_t)(b_single >> q8) & 255u;
      if ((m | ms) == 0u) continue;
      const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)node, q8);
      const uint64_t mask = w64_readlane_u64(en.z, en.w, q8);
      const uint32_t imq = (uint32_t)__builtin_amdgcn_readlane((int)im, q8);
      to_image(imq);
      if (m && __builtin_amdgcn_inverse_ballot_w64(mask)) {
        do {
          W64Node nd;
          w64g_load<QUAD, OFF32>(mcom, Qarr, first + (uint32_t)__builtin_ctz(m), nd);
          m &= m - 1u;
          const double d0 = nd.cx - y0, d1 = nd.cy - y1, d2 = nd.cz - pz;
          w64g_cell<QUAD, RS32>(nd, d0, d1, d2, w64_r2(d0, d1, d2, b2), ax, ay, az);
        } while (m);
      }
      while (ms) {
        const uint32_t c = (uint32_t)__builtin_ctz(ms);
        ms &= ms - 1u;
        W64Node nd;
        w64g_load<false, OFF32>(mcom, Qarr, first + c, nd);
        // the mask without the particle itself
        const uint64_t others = imq == self_img ? w64_readlane_u64(mlo, mhi, q8 + (int)c) : mask;
        if (__builtin_amdgcn_inverse_ballot_w64(others)) {
          const double d0 = nd.cx - y0, d1 = nd.cy - y1, d2 = nd.cz - pz;
          w64_mono(nd.m, d0, d1, d2, w64_r2(d0, d1, d2, b2), ax, ay, az);
        }
      }
    }
    // opened bucket leaves: their members one by one, all four words requested
    // before the first is looked at (forces of spheres of 3,000 with leaves of
    // 32 256 -> 227 us, 40 patches of 500 to 6,000 with leaves of 16 483 -> 453;
    // from lanes that hold a member each, 64 of a leaf or of all leaves at a
    // time, 236 and 509: what is read back lane by lane is issued by the VALU)
    for (uint64_t m = adds ? __ballot(opens && leaf) : 0ull; m; m &= m - 1) {
      const int j = __ffsll((long long)m) - 1;
      const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)lk.child_or_first, j);
      const uint32_t e = a + (uint32_t)__builtin_amdgcn_readlane((int)lk.count, j);
      const uint64_t mine = w64_readlane_u64(plo, phi, j);
      const uint32_t imj = (uint32_t)__builtin_amdgcn_readlane((int)im, j);
      to_image(imj);
      if (e < a || e > cap) {
        if (lane == 0) atomicOr(err, RB_ERR_TREE);
        continue;
      }
      for (uint32_t q = a; q < e; ++q) {
        const double mj = msrc[q], xj = sxc[q], yj = syc[q], zj = szc[q];
        const uint64_t on = mj != 0.0 ? mine : 0ull;
        if (__builtin_amdgcn_inverse_ballot_w64(on) && !(imj == self_img && q == s)) {
          const double f0 = xj - y0, f1 = yj - y1, f2 = zj - pz;
          w64_mono(mj, f0, f1, f2, w64_r2(f0, f1, f2, b2), ax, ay, az);
          if (STATS) ++n_pp;
        }
      }
    }
    __syncthreads();  // entries written before the next round reads them
  }
  double *a = acc + (size_t)(im0 + part) * 3 * cap;
  // the waves' sums, added in wave order
  double(*red)[3][64] = reinterpret_cast<double(*)[3][64]>(&stk[0]);
  red[w][0][lane] = ax; red[w][1][lane] = ay; red[w][2][lane] = az;
  __syncthreads();
  ax = ay = az = 0.0;
  if (w == 0) {
#pragma unroll
    for (int q = 0; q < NW; ++q) {
      ax += red[q][0][lane]; ay += red[q][1][lane]; az += red[q][2][lane];
    }
  }
  if (w == 0 && s < it.end) {
    a[s] = G * ax; a[cap + s] = G * ay; a[2 * cap + s] = G * az;
    // the sets that only other items' shares fill, after the last share's
    for (int q = parts; part == parts - 1 && q < n_sets; ++q) {
      a += 3 * cap;
      a[s] = 0.0; a[cap + s] = 0.0; a[2 * cap + s] = 0.0;
    }
  }
  if (STATS) {
    unsigned long long o = n_open, c = n_cell, q2 = n_pp;
    for (int d = 32; d >= 1; d >>= 1) {
      o += __shfl_xor(o, d, 64);
      c += __shfl_xor(c, d, 64);
      q2 += __shfl_xor(q2, d, 64);
    }
    if (lane == 0) {
      atomicAdd(&stats[0], o);
      atomicAdd(&stats[1], c);
      atomicAdd(&stats[2], q2);
    }
  }
}

template <bool QUAD, bool STATS>
__global__ __launch_bounds__(64) void k_walk64_lane(
    const WalkItem *__restrict__ items, int img_split, int n_img, int ngx, int ngy,
    int boundary, const PatchInfo *__restrict__ patch, const uint32_t *__restrict__ nlive,
    const uint32_t *__restrict__ root, const NodeLink *__restrict__ link,
    const double4 *__restrict__ mcom, const double *__restrict__ Qarr,
    const double *__restrict__ sx, const double *__restrict__ sy,
    const double *__restrict__ sz, const double *__restrict__ msrc,
    const double *__restrict__ sched, const uint32_t *__restrict__ ctr, uint32_t P,
    double G, double b2, double theta2, double *__restrict__ acc, uint64_t cap,
    unsigned long long *__restrict__ stats, const uint32_t *__restrict__ lev_off,
    uint32_t *__restrict__ err, int slot) {
  // a depth-first walk visits every node at most once per image: more
  // visits, or an index past the node count, mean inconsistent links
  const uint32_t n_nodes = lev_off[RB_NLEV];
  const uint32_t item = img_split ? blockIdx.x / n_img : blockIdx.x;
  const int im0 = img_split ? (int)(blockIdx.x % n_img) : 0;
  const int im1 = img_split ? im0 + 1 : n_img;
  const WalkItem it = items[item];
  const uint32_t p = it.patch;
  const double W = patch[p].W;
  const uint32_t st = patch[p].start, nl = nlive[p];
  const uint32_t s = it.start + threadIdx.x;
  const bool valid = s < it.end && (s - st) < nl;
  const double shear = sched[(size_t)ctr[slot] * 2 * P + p];
  double px = 0.0, py = 0.0, pz = 0.0;
  if (valid) { px = sx[s]; py = sy[s]; pz = sz[s]; }
  const uint32_t r0 = valid ? root[p] : RB_NONE;
  uint32_t n_open = 0, n_cell = 0, n_pp = 0;
  double tx = 0.0, ty = 0.0, tz = 0.0;
  for (int im = im0; im < im1; ++im) {
    double ox, oy;
    bool self;
    rb_image(im, ngx, ngy, boundary, patch[p].L[0], patch[p].L[1], shear, ox, oy, self);
    const double y0 = px - ox, y1 = py - oy, y2 = pz;
    double ax = 0.0, ay = 0.0, az = 0.0;
    uint32_t cur = r0, visits = 0;
    while (cur != RB_NONE) {
      if (cur >= n_nodes || ++visits > n_nodes) {
        atomicOr(err, RB_ERR_TREE);
        break;
      }
      const NodeLink lk = link[cur];
      const double4 mc = mcom[cur];
      uint32_t next = lk.skip;
      if (mc.w != 0.0) {
        const bool leaf = (lk.lvl & 256u) != 0;
        if (leaf && lk.count == 1) {
          if (!(self && lk.child_or_first == s)) {
            const double d0 = mc.x - y0, d1 = mc.y - y1, d2 = mc.z - y2;
            w64_mono(G * mc.w, d0, d1, d2, w64_r2(d0, d1, d2, b2), ax, ay, az);
            if (STATS) ++n_pp;
          }
        } else {
          const double d0 = mc.x - y0, d1 = mc.y - y1, d2 = mc.z - y2;
          const double R2 = __builtin_fma(d2, d2, __builtin_fma(d1, d1, d0 * d0));
          const int lv = (int)(lk.lvl & 255u);
          const double w = ldexp(W, -lv);
          // cells above the root boxes are always opened
          const bool root_or_below = lv >= (int)patch[p].nvirt;
          if (STATS && root_or_below) ++n_open;
          if (root_or_below && w * w < theta2 * R2) {
            w64_cell<QUAD>(G, G * mc.w, Qarr + 6 * (size_t)cur, d0, d1, d2, R2 + b2, ax, ay,
                           az);
            if (STATS) ++n_cell;
          } else if (leaf) {
            const uint32_t j0 = lk.child_or_first, j1 = j0 + lk.count;
            for (uint32_t j = j0; j < j1; ++j) {
              const double mj = msrc[j];
              if (mj == 0.0 || (self && j == s)) continue;
              const double e0 = sx[j] - y0, e1 = sy[j] - y1, e2 = sz[j] - y2;
              w64_mono(G * mj, e0, e1, e2, w64_r2(e0, e1, e2, b2), ax, ay, az);
              if (STATS) ++n_pp;
            }
          } else {
            next = lk.child_or_first;
          }
        }
      }
      cur = next;
    }
    if (img_split) {
      if (s < it.end) {
        double *a = acc + (size_t)im * 3 * cap;
        a[s] = ax; a[cap + s] = ay; a[2 * cap + s] = az;
      }
    } else {
      tx += ax; ty += ay; tz += az;
    }
  }
  if (!img_split && s < it.end) {
    acc[s] = tx; acc[cap + s] = ty; acc[2 * cap + s] = tz;
  }
  if (STATS) {
    unsigned long long o = n_open, c = n_cell, q = n_pp;
    for (int d = 32; d >= 1; d >>= 1) {
      o += __shfl_xor(o, d, 64);
      c += __shfl_xor(c, d, 64);
      q += __shfl_xor(q, d, 64);
    }
    if (threadIdx.x == 0) {
      atomicAdd(&stats[0], o);
      atomicAdd(&stats[1], c);
      atomicAdd(&stats[2], q);
    }
  }
}

// Dispatch order of the 64-part walk's units.  Near-field units take
// several times longer than the median one, and in part-major order some
// start late and leave the chip with a tail of a few waves.  The walk
// records each unit's node visits; before the next launch the units that
// cost at least the threshold (about the top 1/32, from the costs one
// launch earlier) are listed to run first, the rest keeping their
// part-major order.  The order decides only which wave starts first: every
// unit writes its own accumulator set, so the sums do not depend on it.
// Launched for at least RB_WALK64_ORDER_MIN units (so a share holds at
// least 512).
__global__ __launch_bounds__(1024) void k_w64_list(uint32_t *__restrict__ ord,
                                                   uint32_t n_units) {
  __shared__ uint32_t lh[33];
  __shared__ uint32_t lcnt[8], lbase[8];
  __shared__ uint32_t last;
  W64Ctl *const ctl = (W64Ctl *)ord;
  const uint32_t t = threadIdx.x, lane = t & 63u, u = blockIdx.x * 1024u + t;
  const bool in = u < n_units;
  const uint32_t v = in ? ord[RB_W64_COST_OFF + u] : 0u;
  const uint32_t e = ctl->epoch;
  const bool heavy = in && v >= ctl->thr;
  if (t < 33u) lh[t] = 0u;
  if (t < 8u) lcnt[t] = 0u;
  __syncthreads();
  // the XCD share of the walk's grid the unit belongs to (share x starts at
  // unit x q + min(x, r)); a wave's 64 units span at most two shares.  Each
  // wave takes its listed units' places in the block's count of each share
  // (one LDS atomic per wave and share), and the block then reserves its
  // places in the share's list with one atomic per share.
  const uint32_t q = n_units >> 3, r = n_units & 7u;
  const uint32_t x = u < r * (q + 1u) ? u / (q + 1u) : q ? r + (u - r * (q + 1u)) / q : 7u;
  uint32_t k = 0;
  uint64_t todo = __ballot(heavy);
  while (todo) {
    const uint32_t xl = (uint32_t)__shfl((int)x, __ffsll((long long)todo) - 1, 64);
    const uint64_t mine = __ballot(heavy && x == xl);
    uint32_t base = 0;
    if (lane == (uint32_t)(__ffsll((long long)mine) - 1))
      base = atomicAdd(&lcnt[xl], (uint32_t)__popcll(mine));
    base = (uint32_t)__shfl((int)base, __ffsll((long long)mine) - 1, 64);
    if (heavy && x == xl) k = base + (uint32_t)__popcll(mine & ((1ull << lane) - 1ull));
    todo &= ~mine;
  }
  __syncthreads();
  if (t < 8u && lcnt[t] != 0u) lbase[t] = atomicAdd(&ctl->cnt[e & 1u][t], lcnt[t]);
  __syncthreads();
  if (heavy) {
    k += lbase[x];
    if (k < RB_WALK64_HEAVY_MAX / 8u) {
      ord[RB_W64_HEAVY_OFF + x * (RB_WALK64_HEAVY_MAX / 8u) + k] = u;
      ord[RB_W64_TAG_OFF + u] = e;
    }
  }
  // the costs by bit length, block by block into the launch's histogram
  // (one LDS atomic per wave and bit length present)
  const uint32_t bl = v ? 32u - (uint32_t)__clz(v) : 0u;
  uint64_t hm = __ballot(in);
  while (hm) {
    const uint32_t bb = (uint32_t)__shfl((int)bl, __ffsll((long long)hm) - 1, 64);
    const uint64_t m = __ballot(in && bl == bb);
    if (lane == (uint32_t)(__ffsll((long long)m) - 1)) atomicAdd(&lh[bb], (uint32_t)__popcll(m));
    hm &= ~m;
  }
  __syncthreads();
  if (t < 33u && lh[t] != 0u) atomicAdd(&ctl->hist[t], lh[t]);
  __threadfence();
  __syncthreads();
  if (t == 0) last = atomicAdd(&ctl->done, 1u) == gridDim.x - 1u ? 1u : 0u;
  __syncthreads();
  if (last == 0u || t >= 64u) return;
  // the last block: the next threshold is the largest power of two such
  // that at least n_units / 32 units cost that much or more (none while no
  // unit reached it)
  __threadfence();
  const uint32_t h = t < 33u ? atomicExch(&ctl->hist[t], 0u) : 0u;
  uint32_t acc = 0, thr = 0xFFFFFFFFu;
  for (int bl = 32; bl >= 1; --bl) {
    acc += (uint32_t)__builtin_amdgcn_readlane((int)h, bl);
    if (acc > 0 && acc >= n_units / 32u) {
      thr = 1u << (bl - 1);
      break;
    }
  }
  if (t == 0) {
    ctl->thr = thr;
    ctl->cur = e;
    ctl->epoch = e + 1u;
    for (int j = 0; j < 8; ++j) ctl->cnt[(e + 1u) & 1u][j] = 0u;
    ctl->done = 0u;
  }
}

// Whether every accepted cell's rho^2 is a normal, finite FP32 value, so that
// its reciprocal root may start from FP32's estimate: an accepted cell has
// R^2 > (W 2^-21)^2 / theta^2, and no distance in the box or to an image is
// above 8 times its longest side.  (Particle pairs may be closer than any
// such bound; they always start from the FP64 instruction.)
static bool w64_fp32_seed(const rb_ctx *c, double theta2, double b2) {
  const double lo = 0x1p-120, hi = 0x1p+120;
  if (!(b2 < hi)) return false;
  for (const PatchInfo &p : c->h_patch) {
    const double L = fmax(fmax(p.L[0], p.L[1]), p.L[2]);
    if (!(p.W * p.W * 0x1p-42 > lo * theta2) || !(64.0 * L * L < hi)) return false;
  }
  return true;
}

hipError_t launch_walk64(rb_ctx *c, const double *sx, const double *sy, const double *sz,
                         int slot) {
  const uint32_t n_items = (uint32_t)c->h_items64.size();
  if (n_items == 0) return hipSuccess;
  const int split = c->img_split;
  const uint32_t units = split ? n_items * (uint32_t)c->n_img : n_items;
  const double b2 = c->p.softening * c->p.softening;
  const double th2 = c->p.theta * c->p.theta;
  const bool quad = c->p.quadrupole != 0, stats = (c->p.profile & 2) != 0;
  if (c->walk64_mode == 0) {
    const dim3 g(units);
    const bool rs32 = w64_fp32_seed(c, th2, b2);
#define RB_W64G_ARGS                                                                        \
  c->d_items64, units, split, c->walk_parts, c->n_img, c->p.n_ghost[0], c->p.n_ghost[1],     \
      c->p.boundary,                                                                         \
      c->d_patch, c->d_nlive, c->d_root, c->d_link, c->d_mcom, c->d_Q, sx, sy, sz, c->d_msrc, \
      c->d_sched, c->d_ctr, c->P, c->p.G, b2, th2, c->d_acc, c->cap, c->d_stats,             \
      c->d_lev_off, c->d_err, slot
#define RB_W64G_NW(Q, S, R, O)                                                               \
  do {                                                                                       \
    if (nw == 4) hipLaunchKernelGGL((k_walk64<Q, S, 4, R, O>), g, dim3(256), 0, c->stream, RB_W64G_ARGS); \
    else if (nw == 8) hipLaunchKernelGGL((k_walk64<Q, S, 8, R, O>), g, dim3(512), 0, c->stream, RB_W64G_ARGS); \
    else hipLaunchKernelGGL((k_walk64<Q, S, 16, R, O>), g, dim3(1024), 0, c->stream, RB_W64G_ARGS); \
  } while (0)
#define RB_W64G_S(Q, S)                             \
  do {                                              \
    if (rs32 && off32) RB_W64G_NW(Q, S, true, true); \
    else if (rs32) RB_W64G_NW(Q, S, true, false);    \
    else RB_W64G_NW(Q, S, false, false);             \
  } while (0)
    const int nw = c->walk64_waves;
    const bool off32 = c->node_cap * 48ull < (1ull << 32);
    if (quad && stats) RB_W64G_S(true, true);
    else if (quad) RB_W64G_S(true, false);
    else if (stats) RB_W64G_S(false, true);
    else RB_W64G_S(false, false);
#undef RB_W64G_S
#undef RB_W64G_NW
#undef RB_W64G_ARGS
    return hipGetLastError();
  }
  if (c->walk64_mode != 1) {
    const int parts = c->walk_parts;
    unsigned grid = units * (uint32_t)parts;  // one unit per wave and workgroup
    // the 64-part walk runs its costliest units first (by the last launch;
    // measured: the top 1/32 first beats 1/16 and 1/64, and below
    // RB_WALK64_ORDER_MIN units the listing costs more than it saves)
    const bool ordered = parts == RB_WALK64_PARTS2 && grid >= RB_WALK64_ORDER_MIN &&
                         grid <= RB_WALK64_ORDER_CAP;
    uint32_t *ord = ordered ? c->d_w64_ord : nullptr;
    if (ordered) {
      hipLaunchKernelGGL(k_w64_list, dim3(rb_div_up(grid, 1024)), dim3(1024), 0, c->stream, ord,
                         grid);
      grid += RB_WALK64_HEAVY_MAX;
    }
#define RB_WALK64_ARGS                                                                     \
  c->d_items64, n_items, split, c->n_img, parts, c->p.n_ghost[0], c->p.n_ghost[1],          \
      c->p.boundary,                                                                       \
      c->d_patch, c->d_nlive, c->d_root, c->d_link, c->d_mcom, c->d_Q, sx, sy, sz,         \
      c->d_msrc, c->d_sched, c->d_ctr, c->P, c->p.G, b2, th2, c->d_acc, c->cap,           \
      c->d_stats, c->d_lev_off, c->d_err, slot, ord
    const dim3 g(grid), bl(64);
    // 32-bit byte offsets of the node records (48 bytes for a quadrupole)
    const bool off32 = c->node_cap * 48ull < (1ull << 32);
#define RB_W64_LAUNCH(PD)                                                                          \
  do {                                                                                             \
    if (quad && stats) hipLaunchKernelGGL((k_walk64_parts<true, true, PD, false>), g, bl, 0, c->stream, RB_WALK64_ARGS); \
    else if (quad && off32) hipLaunchKernelGGL((k_walk64_parts<true, false, PD, true>), g, bl, 0, c->stream, RB_WALK64_ARGS); \
    else if (quad) hipLaunchKernelGGL((k_walk64_parts<true, false, PD, false>), g, bl, 0, c->stream, RB_WALK64_ARGS); \
    else if (stats) hipLaunchKernelGGL((k_walk64_parts<false, true, PD, false>), g, bl, 0, c->stream, RB_WALK64_ARGS); \
    else if (off32) hipLaunchKernelGGL((k_walk64_parts<false, false, PD, true>), g, bl, 0, c->stream, RB_WALK64_ARGS); \
    else hipLaunchKernelGGL((k_walk64_parts<false, false, PD, false>), g, bl, 0, c->stream, RB_WALK64_ARGS); \
  } while (0)
    if (parts == 64) RB_W64_LAUNCH(2);
    else if (parts == 8) RB_W64_LAUNCH(1);
    else RB_W64_LAUNCH(0);
#undef RB_W64_LAUNCH
#undef RB_WALK64_ARGS
    return hipGetLastError();
  }
  const unsigned grid = units;
#define RB_WALK64_LANE_ARGS                                                              \
  c->d_items64, split, c->n_img, c->p.n_ghost[0], c->p.n_ghost[1], c->p.boundary,        \
      c->d_patch, c->d_nlive, c->d_root, c->d_link, c->d_mcom, c->d_Q, sx, sy, sz,       \
      c->d_msrc, c->d_sched, c->d_ctr, c->P, c->p.G, b2, th2, c->d_acc, c->cap, c->d_stats, \
      c->d_lev_off, c->d_err, slot
  if (quad && stats)
    hipLaunchKernelGGL((k_walk64_lane<true, true>), dim3(grid), dim3(64), 0, c->stream, RB_WALK64_LANE_ARGS);
  else if (quad)
    hipLaunchKernelGGL((k_walk64_lane<true, false>), dim3(grid), dim3(64), 0, c->stream, RB_WALK64_LANE_ARGS);
  else if (stats)
    hipLaunchKernelGGL((k_walk64_lane<false, true>), dim3(grid), dim3(64), 0, c->stream, RB_WALK64_LANE_ARGS);
  else
    hipLaunchKernelGGL((k_walk64_lane<false, false>), dim3(grid), dim3(64), 0, c->stream, RB_WALK64_LANE_ARGS);
#undef RB_WALK64_LANE_ARGS
  return hipGetLastError();
}
