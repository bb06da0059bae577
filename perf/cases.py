"""Cases that a performance measurement of this package runs, each through the
public entry points a program calls (``paper_1110_4876_amd.rb``).

A case is a dict of plain values; ``kind`` names the entry point:

* ``gravity``  -- ``rb_gravity``: tree accelerations of one system;
* ``step``     -- ``rb_step``: drift-kick-drift steps of one system, with
                  collisions at the end of every step when ``collisions``;
* ``batch``    -- ``rb_batch_step``: the same for many independent patches;
* ``collide``  -- ``rb_collide``: tree search and resolution as a call;
* ``sweep``    -- ``rb_sweep``: plane sweep and resolution as a call.

Sizes, opening angles and launch options are those of the package's
operating points, benchmark and tests.  ``prepare`` makes what a program has
in hand: particles on the GPU and a context.  ``run`` starts every pass from
the prepared particles (a step and a collision change them in place), so that
a pass does the same work however often it is repeated.  ``exact`` is plain
torch and numpy in 64 bits: direct summation of Eq. (1) over all pairs and
ghost images, the drifts and boundaries of Sect. 2.3 and 3, and pair searches
over all pairs.
"""
import math
import random

import numpy as np
import torch

from paper_1110_4876_amd import inputs, rb

FIELDS = ("x", "y", "z", "vx", "vy", "vz")
EPSILON = 0.5      # coefficient of restitution of the benchmark's collisions
EXACT_PAIRS = 2e11  # pairs that the 64-bit reference sums in about 15 s


def _case(name, kind, system, n, **kw):
    c = dict(name=name, kind=kind, system=system, n=n, precision="fp64", theta=0.5,
             quadrupole=True, leaf_size=1, group_size=64, walk_waves=1, use_graph=False,
             steps=1, collisions=False, tau=0.5, ng=1, patches=1, n_min=0, axis="x")
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: forces of a small cluster, monopoles, where the
        # chain of launches and their latency count
        _case("plummer1k_gravity_fp64", "gravity", "plummer", 1024, theta=0.5,
              quadrupole=False),
        # a small shearing-sheet patch of odd size, a few steps at a time
        _case("sheet3k_step_fp32", "step", "sheet", 3001, precision="fp32", theta=0.32,
              walk_waves=4, steps=4),
        # the 50,000-particle shearing sheet at its operating points: plain
        # FP64, FP32-mixed, and FP32-mixed with collisions at the end of
        # every step
        _case("sheet50k_step_fp64", "step", "sheet", 50000, theta=0.26, steps=4),
        _case("sheet50k_step_fp32", "step", "sheet", 50000, precision="fp32", theta=0.32,
              walk_waves=4, steps=4),
        _case("sheet50k_collisions_fp32", "step", "sheet", 50000, precision="fp32", theta=0.42,
              walk_waves=4, steps=4, collisions=True),
        # a million-particle sheet of odd size: the large-system sort
        _case("sheet1m_step_fp32", "step", "sheet", 1000003, precision="fp32", theta=0.4),
        # the ensemble of uneven sheet patches (2,000 to 64,000 particles
        # each), steps replayed from a captured graph: all 256 patches
        # FP32-mixed, a quarter of them in plain FP64
        _case("batch256_step_fp32", "batch", "sheet", 64000, precision="fp32", theta=0.32,
              use_graph=True, patches=256, n_min=2000),
        _case("batch64_step_fp64", "batch", "sheet", 64000, theta=0.26, use_graph=True,
              patches=64, n_min=2000),
        # the largest single system: 2^23-particle Plummer sphere, one step
        _case("plummer8m_step_fp32", "step", "plummer", 1 << 23, precision="fp32", theta=0.42,
              use_graph=True),
        # forces of a million-particle cluster in plain FP64, odd size
        _case("plummer1m_gravity_fp64", "gravity", "plummer", 1048583, theta=0.38),
        # collision search and resolution as calls of their own: the octree
        # search on the sheet, the azimuthal plane sweep on a narrow ring
        _case("sheet50k_collide", "collide", "sheet", 50000),
        _case("ring50k_sweep_phi", "sweep", "ring", 50000, axis="phi"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("gravity", "step", "step", "batch", "collide", "sweep"))
    prec = rng.choice(("fp32", "fp64"))
    if kind == "gravity":
        c = _case("", kind, rng.choice(("plummer", "sheet")), _log_int(rng, 700, 1000000),
                  theta=round(rng.uniform(0.35, 0.7), 3), quadrupole=rng.random() < 0.75,
                  leaf_size=rng.choice((1, 1, 1, 4, 8)), tau=round(rng.uniform(0.2, 1.0), 3))
    elif kind == "step":
        coll = rng.random() < 0.3
        system = "sheet" if coll else rng.choice(("sheet", "sheet", "plummer"))
        c = _case("", kind, system, _log_int(rng, 1000, 200000 if coll else 1000000),
                  precision=prec, theta=round(rng.uniform(0.3, 0.5), 3), collisions=coll,
                  group_size=rng.choice((32, 64, 64)), walk_waves=rng.choice((1, 2, 4)),
                  use_graph=rng.random() < 0.5, tau=round(rng.uniform(0.2, 1.0), 3))
        c["steps"] = rng.choice((2, 3, 4)) if c["n"] < 100000 else 1
    elif kind == "batch":
        c = _case("", kind, "sheet", _log_int(rng, 8000, 64000), precision=prec,
                  theta=round(rng.uniform(0.28, 0.45), 3), use_graph=rng.random() < 0.7,
                  patches=_log_int(rng, 4, 128 if prec == "fp32" else 40), n_min=2000)
    elif kind == "collide":
        c = _case("", kind, "sheet", _log_int(rng, 2000, 300000),
                  tau=round(rng.uniform(0.2, 1.0), 3))
    else:
        axis = rng.choice(("x", "phi"))
        c = _case("", kind, "ring" if axis == "phi" else "sheet", _log_int(rng, 2000, 120000),
                  axis=axis)
    del c["name"]
    return c


# ---- inputs -----------------------------------------------------------------

def _rand(gen, *shape):
    return torch.rand(*shape, generator=gen, device="cuda", dtype=torch.float64)


def _randn(gen, *shape):
    return torch.randn(*shape, generator=gen, device="cuda", dtype=torch.float64)


def _isotropic(gen, n):
    c, phi = 2.0 * _rand(gen, n) - 1.0, 2.0 * math.pi * _rand(gen, n)
    s = torch.sqrt(1.0 - c * c)
    return torch.stack([s * torch.cos(phi), s * torch.sin(phi), c])


def _plummer(c, gen):
    """Plummer sphere as in ``inputs.plummer`` (total mass 1, scale radius 1)."""
    n = c["n"]
    r = 1.0 / torch.sqrt((0.999 * _rand(gen, n)) ** (-2.0 / 3.0) - 1.0)
    pos = r * _isotropic(gen, n)
    q, got = [], 0
    while got < n:
        a, g = _rand(gen, 2 * n + 64), 0.1 * _rand(gen, 2 * n + 64)
        q.append(a[g < a * a * (1.0 - a * a) ** 3.5])
        got += len(q[-1])
    v = torch.cat(q)[:n] * math.sqrt(2.0) * (1.0 + r * r) ** -0.25
    vel = v * _isotropic(gen, n)
    pos, vel = pos - pos.mean(1, keepdim=True), vel - vel.mean(1, keepdim=True)
    params = inputs.base_params(G=1.0, b=0.01 if n < 100000 else 0.001, theta=c["theta"],
                                quadrupole=c["quadrupole"], n_leaf=c["leaf_size"], W=128.0,
                                x0=(-64.0,) * 3, group_size=c["group_size"])
    return dict(X=torch.cat([pos, vel, torch.full((1, n), 1.0 / n, device="cuda",
                                                  dtype=torch.float64)]),
                params=params, dt=1e-4, radius=None)


def _sheet(c, gen, n=None, tau=None):
    """Shearing-sheet patch with the sizes, masses and speeds of
    ``inputs.sheet``, settled: the particles stand on a jittered grid with
    some empty places, since those of a real ring do not sit inside one
    another (a few per cent still touch)."""
    n = c["n"] if n is None else n
    tau = c["tau"] if tau is None else tau
    omega = 1.95e-4
    R = (1.0 - _rand(gen, n) * (1.0 - 4.0 ** -2)) ** -0.5
    W = math.sqrt(float(torch.sum(math.pi * R * R)) / tau)
    g = math.ceil(math.sqrt(1.1 * n))
    cell = torch.randperm(g * g, generator=gen, device="cuda")[:n]
    x = (((cell % g).double() + 0.25 + 0.5 * _rand(gen, n)) / g - 0.5) * W
    y = ((torch.div(cell, g, rounding_mode="floor").double() + 0.25 + 0.5 * _rand(gen, n)) / g
         - 0.5) * W
    vel = 0.01 * _randn(gen, 3, n)
    vel[1] -= 1.5 * omega * x
    m = 4.0 / 3.0 * math.pi * 400.0 * R ** 3
    params = inputs.base_params(G=inputs.G_SI, theta=c["theta"], quadrupole=c["quadrupole"],
                                W=W, x0=(-W / 2,) * 3, boundary=inputs.SHEAR,
                                ng=(c["ng"], c["ng"]), drift=inputs.EPICYCLE, omega=omega,
                                n_leaf=c["leaf_size"], group_size=c["group_size"])
    return dict(X=torch.cat([torch.stack([x, y, _randn(gen, n) * R]), vel, m[None]]),
                params=params, dt=1e-3 * 2.0 * math.pi / omega, radius=R)


def _ring(c, gen):
    """Narrow ring around a central mass, as in ``inputs.ring``."""
    n, width = c["n"], 0.01
    Rt = (1.0 - _rand(gen, n) * (1.0 - 4.0 ** -2)) ** -0.5
    scale = math.sqrt(c["tau"] * 2.0 * math.pi * width / float(torch.sum(math.pi * Rt * Rt)))
    R = Rt * scale
    r = 1.0 + width * (_rand(gen, n) - 0.5)
    ph = math.pi * (2.0 * _rand(gen, n) - 1.0)
    dv = 2.0 * float(R.mean()) * _randn(gen, 3, n)
    vk = 1.0 / torch.sqrt(r)
    X = torch.stack([r * torch.cos(ph), r * torch.sin(ph), _randn(gen, n) * R,
                     dv[0] - vk * torch.sin(ph), dv[1] + vk * torch.cos(ph), dv[2],
                     4.0 / 3.0 * math.pi * R ** 3])
    W = 2.2 * (1.0 + width)
    return dict(X=X, params=inputs.base_params(G=1.0, W=W, x0=(-W / 2,) * 3),
                dt=1e-3 * 2.0 * math.pi, radius=R)


def _patches(c):
    """Sizes and optical depths of a batch's patches: the case's own, the same
    for every seed."""
    r = random.Random(c["patches"] * 100003 + c["n"])
    return [(r.randint(c["n_min"], c["n"]), r.uniform(0.2, 1.0)) for _ in range(c["patches"])]


def _inputs(c, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    return {"plummer": _plummer, "sheet": _sheet, "ring": _ring}[c["system"]](c, gen)


class _State:
    """A context with its particles; the context ends with the state."""

    def __init__(self, case, seed):
        self.case = case
        opts = dict(precision=rb.RB_FP32_MIXED if case["precision"] == "fp32" else rb.RB_FP64,
                    use_graph=int(case["use_graph"]), walk_waves=case["walk_waves"],
                    split_images=0)
        if case["kind"] == "batch":
            gen = torch.Generator(device="cuda")
            gen.manual_seed(int(seed))
            every = [_sheet(case, gen, n, tau) for n, tau in _patches(case)]
            inp = every[0]
            X = torch.cat([p["X"] for p in every], 1)
            offsets = np.concatenate([[0], np.cumsum([p["X"].shape[1] for p in every])])
            self.ctx = rb.rb_batch_create(rb.params_from_problem(inp["params"], **opts), offsets,
                                          [p["params"]["W"] for p in every],
                                          [p["params"]["x0"] for p in every])
        else:
            inp = _inputs(case, seed)
            X = inp["X"]
            self.ctx = rb.rb_create(rb.params_from_problem(inp["params"], **opts), X.shape[1])
        self.start = X.contiguous()
        self.X = self.start.clone()
        self.n = X.shape[1]
        self.dt = inp["dt"]
        self.radius = inp["radius"]
        self.parts = rb.particles(self.X[0], self.X[1], self.X[2], self.X[6], self.X[3],
                                  self.X[4], self.X[5])
        self.acc = None
        if case["kind"] == "gravity":
            self.acc = torch.empty((3, self.n), dtype=torch.float64, device="cuda")
        if case["collisions"]:
            rb.rb_set_collisions(self.ctx, self.radius, EPSILON, 1000, True)

    def __del__(self):
        ctx, self.ctx = getattr(self, "ctx", None), None
        if ctx is not None:
            rb.rb_destroy(ctx)


def prepare(case, seed):
    return _State(case, seed)


def run(st):
    kind = st.case["kind"]
    if kind == "gravity":
        rb.rb_gravity(st.ctx, st.parts, st.n, st.n, 0.0, st.acc[0], st.acc[1], st.acc[2])
        return dict(zip(("ax", "ay", "az"), st.acc))
    st.X[:6].copy_(st.start[:6])
    if kind == "step":
        rb.rb_step(st.ctx, st.parts, st.n, st.n, 0.0, st.dt, st.case["steps"])
    elif kind == "batch":
        rb.rb_batch_step(st.ctx, st.parts, 0.0, st.dt, st.case["steps"])
    elif kind == "collide":
        pairs, resolved = rb.rb_collide(st.ctx, st.parts, st.radius, st.n, 0.0, EPSILON, 7)
    else:
        axis = rb.RB_SWEEP_PHI if st.case["axis"] == "phi" else rb.RB_SWEEP_X
        pairs, resolved = rb.rb_sweep(st.ctx, st.parts, st.radius, st.n, 0.0, st.dt, EPSILON, 7,
                                      axis=axis)
    if kind in ("collide", "sweep"):
        return dict(vx=st.X[3], vy=st.X[4], vz=st.X[5], pairs=pairs, resolved=resolved)
    return dict(zip(FIELDS, st.X))


# ---- work -------------------------------------------------------------------

def _walk_flops(system, n, theta, ng):
    """Flops per particle of the per-particle walk (9 per opening test, 20 per
    point mass, 56 per quadrupole cell), fitted to the counts the library
    reports: sheets with one ghost ring 85.6e3 at (50,000, 0.32) and 65.7e3
    at (10^6, 0.40); Plummer spheres 263e3 at (2^23, 0.42) and 340e3 at
    (2^23, 0.38); never more than the direct sum."""
    if system == "sheet":
        f = (39e3 + 4.3e3 * math.log(n)) * (0.32 / theta) ** 1.8
        return min(f, 20.0 * n * (2 * ng + 1) ** 2)
    return min(16.5e3 * math.log(n) * (0.42 / theta) ** 2.6, 20.0 * n)


def work(c):
    sizes = [n for n, _ in _patches(c)] if c["kind"] == "batch" else [c["n"]]
    n = float(sum(sizes))
    walk = sum(k * _walk_flops(c["system"], k, c["theta"], c["ng"]) for k in sizes)
    if not c["quadrupole"]:
        walk *= 0.5
    if c["kind"] == "gravity":
        return dict(bytes=56.0 * n, flops=walk)
    if c["kind"] in ("step", "batch"):
        return dict(bytes=(104.0 + (8.0 if c["collisions"] else 0.0)) * n,
                    flops=walk * c["steps"])
    # positions, velocities, masses and radii in, velocities out; the search
    # tests a few tens of candidates per particle at 9 flops
    return dict(bytes=88.0 * n, flops=500.0 * n)


# ---- 64-bit reference -------------------------------------------------------

def _images(p, t):
    """Ghost-box offsets (ix Lx, iy Ly - ix s) and shear velocities, ix outer."""
    if p["boundary"] == inputs.OPEN:
        return [(0.0, 0.0, 0.0)]
    W, s = p["W"], math.remainder(1.5 * p["omega"] * p["W"] * t, p["W"])
    return [(ix * W, iy * W - ix * s, -1.5 * p["omega"] * W * ix)
            for ix in range(-p["ng"][0], p["ng"][0] + 1)
            for iy in range(-p["ng"][1], p["ng"][1] + 1)]


def _direct(X, p, t):
    """Eq. (1) over all pairs and ghost images."""
    n, out = X.shape[1], torch.zeros_like(X[:3])
    rows = max(1, int(6e7) // n)
    for a in range(0, n, rows):
        tgt = X[:3, a:a + rows]
        k = torch.arange(tgt.shape[1], device=X.device)
        for ox, oy, _ in _images(p, t):
            d = [(X[0] + ox)[None] - tgt[0][:, None], (X[1] + oy)[None] - tgt[1][:, None],
                 X[2][None] - tgt[2][:, None]]
            f = d[0] * d[0]
            f.addcmul_(d[1], d[1]).addcmul_(d[2], d[2]).add_(p["b"] ** 2)
            if ox == 0.0 and oy == 0.0:
                f[k, a + k] = math.inf
            f = f.pow_(-1.5).mul_(p["G"] * X[6])
            for j in range(3):
                out[j, a:a + rows] += d[j].mul_(f).sum(1)
    return out


def _drift(X, p, h):
    """Leap-frog (Sect. 3.1) or epicycle (Sect. 3.3) drift over h."""
    if p["drift"] == inputs.LEAPFROG:
        X[:3] += h * X[3:6]
        return
    w = p["omega"]
    c, s = math.cos(w * h), math.sin(w * h)
    x, y, z, vx, vy, vz = X[:6].clone()
    C = vy + 2.0 * w * x
    xg = 2.0 * C / w
    dx, u = x - xg, vx / w
    X[0] = xg + dx * c + u * s
    X[1] = y - 3.0 * C * h - 2.0 * dx * s - 2.0 * u * (1.0 - c)
    X[2] = z * c + vz / w * s
    X[3] = -w * dx * s + vx * c
    X[4] = C - 2.0 * w * X[0]
    X[5] = -w * z * s + vz * c


def _boundary(X, p, t):
    """Shear-periodic x, periodic y (Sect. 2.3); open boxes are large enough."""
    if p["boundary"] == inputs.OPEN:
        return
    W, jump = p["W"], 1.5 * p["omega"] * p["W"]
    s = math.remainder(jump * t, W)
    up, down = X[0] >= W / 2, X[0] < -W / 2
    side = up.double() - down.double()
    X[0] -= side * W
    X[1] += side * s
    X[4] += side * jump
    X[1] += ((X[1] < -W / 2).double() - (X[1] >= W / 2).double()) * W


def _splitmix64(z):
    with np.errstate(over="ignore"):
        z = z + np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        return z ^ (z >> np.uint64(31))


def _pairs(X, R, p, t, dt):
    """Pairs i < j (image k of j) in contact at t, or at their closest
    approach on straight lines over the past dt."""
    n, found = X.shape[1], []
    rows = max(1, int(4e7) // n)
    j = torch.arange(n, device=X.device)
    for k, (ox, oy, wy) in enumerate(_images(p, t)):
        off = (ox, oy, 0.0, 0.0, wy, 0.0)
        for a in range(0, n, rows):
            d = [(X[q] + off[q])[None] - X[q, a:a + rows, None] for q in range(6)]
            r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2]
            hit = (R[None] + R[a:a + rows, None]) ** 2
            near = r2 < hit
            if dt > 0.0:
                du = d[0] * d[3] + d[1] * d[4] + d[2] * d[5]
                uu = d[3] * d[3] + d[4] * d[4] + d[5] * d[5]
                s = torch.clamp(-du / uu, min=-dt)
                e = [d[q] + s * d[q + 3] for q in range(3)]
                near |= (du > 0.0) & (e[0] * e[0] + e[1] * e[1] + e[2] * e[2] < hit)
            near &= j[None] > j[a:a + rows, None]
            i, jj = torch.nonzero(near, as_tuple=True)
            found.append(torch.stack([i + a, jj, torch.full_like(i, k)], 1))
    return torch.cat(found).cpu().numpy()


def _collide(X, R, p, t, dt, seed):
    """The collision queue of Sect. 5, one collision after the other."""
    pairs = _pairs(X, R, p, t, dt)
    img = _images(p, t)
    u = pairs.astype(np.uint64)
    code = (u[:, 0] << np.uint64(35)) | (u[:, 1] << np.uint64(7)) | u[:, 2]
    order = np.argsort(_splitmix64(code + np.uint64(seed)))
    H = X.cpu().numpy()
    x, v, m, resolved = H[:3].T.copy(), H[3:6].T.copy(), H[6], 0
    for i, j, k in pairs[order]:
        ox, oy, wy = img[k]
        d = x[j] - x[i] + (ox, oy, 0.0)
        w = v[j] - v[i] + (0.0, wy, 0.0)
        du, M = d @ w, m[i] + m[j]
        if du < 0.0 and M > 0.0:
            kick = (1.0 + EPSILON) * du / (d @ d) * d
            v[i] += m[j] / M * kick
            v[j] -= m[i] / M * kick
            resolved += 1
    X[3:6] = torch.as_tensor(v.T.copy(), device=X.device)
    return len(pairs), resolved


def exact(case, seed):
    c = case
    if c["kind"] == "batch":
        return None
    n_img = (2 * c["ng"] + 1) ** 2 if c["system"] == "sheet" else 1
    passes = c["steps"] * (2 if c["collisions"] else 1)
    if float(c["n"]) ** 2 * n_img * passes > EXACT_PAIRS:
        return None
    inp = _inputs(c, seed)
    X, p, dt, R = inp["X"].clone(), inp["params"], inp["dt"], inp["radius"]
    if c["kind"] == "gravity":
        return dict(zip(("ax", "ay", "az"), _direct(X, p, 0.0)))
    if c["kind"] in ("collide", "sweep"):
        pairs, resolved = _collide(X, R, p, 0.0, dt if c["kind"] == "sweep" else 0.0, 7)
        return dict(vx=X[3], vy=X[4], vz=X[5], pairs=pairs, resolved=resolved)
    for k in range(c["steps"]):
        t = k * dt
        _drift(X, p, 0.5 * dt)
        _boundary(X, p, t + 0.5 * dt)
        X[3:6] += dt * _direct(X, p, t + 0.5 * dt)
        _drift(X, p, 0.5 * dt)
        _boundary(X, p, (k + 1) * dt)
        if c["collisions"]:
            _collide(X, R, p, (k + 1) * dt, 0.0, 1000 + k)
    return dict(zip(FIELDS, X))
