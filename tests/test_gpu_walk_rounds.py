"""The FP64 walk in rounds over a stack of opened nodes, at the edges of its
dispatch: each number of waves per 64 particles (by system size), ragged last
items, bucket leaves, the depth-first descent on a nearly full stack, boxes so
small or so large that the reciprocal roots cannot start from FP32, against
the oracle's walk (same decisions, so the counts are equal and the sums agree
to rounding)."""
import numpy as np
import pytest

from paper_1110_4876_amd import inputs

pytestmark = pytest.mark.gpu

# identical decisions, FP64 sums in another order: as the walk's other
# schedules
TOL = 1e-12


def _scaled(pr, f):
    """The problem with lengths times f (masses as they are)."""
    p = dict(pr.params, W=pr.params["W"] * f, b=pr.params["b"] * f,
             x0=tuple(v * f for v in pr.params["x0"]))
    return inputs.Problem(pr.x * f, pr.y * f, pr.z * f, pr.vx, pr.vy, pr.vz, pr.m, p,
                          pr.n_active, pr.dt)


def _clustered(n):
    """Half the particles in a ball of 2^-20 of the box, some exactly alike."""
    pr = inputs.plummer(n, seed=5, quadrupole=True)
    k = n // 2
    for a in (pr.x, pr.y, pr.z):
        a[:k] = 0.3 + a[:k] * 1e-6
        a[:40] = a[0]
    return pr


CASES = [
    ("one", lambda: inputs.plummer(1, seed=1), 1, 0.0),
    ("item_65", lambda: inputs.plummer(65, seed=1, quadrupole=True), 1, 0.0),
    ("waves16_1023_items", lambda: inputs.plummer(1023 * 64, seed=2, theta=0.8), 1, 0.0),
    ("waves8_1024_items", lambda: inputs.plummer(1023 * 64 + 1, seed=2, theta=0.8), 1, 0.0),
    ("waves8_sheet", lambda: inputs.sheet(70001, seed=3, theta=0.6), 4, 1234.5),
    ("waves4", lambda: inputs.plummer(8191 * 64 + 7, seed=4, quadrupole=True, theta=1.0), 8, 0.0),
    ("theta0_rings2", lambda: inputs.sheet(700, seed=7, ng=(2, 2), theta=0.0), 1, 300.0),
    ("theta0_leaf8", lambda: inputs.sheet(900, seed=8, theta=0.0), 8, 300.0),
    ("deep_cluster", lambda: _clustered(3000), 1, 0.0),
    ("deep_cluster_leaf4", lambda: _clustered(3000), 4, 0.0),
    ("tiny_box", lambda: _scaled(inputs.plummer(2000, seed=6, quadrupole=True), 1e-18), 1, 0.0),
    ("huge_box", lambda: _scaled(inputs.plummer(2000, seed=6, quadrupole=True), 1e18), 1, 0.0),
]


@pytest.mark.parametrize("name,maker,leaf,t", CASES, ids=[c[0] for c in CASES])
@pytest.mark.parametrize("split", [0, 1])
def test_rounds_match_oracle(orc, name, maker, leaf, t, split):
    import torch
    from gpu_util import Dev, make_ctx, rms_rel
    from paper_1110_4876_amd import rb
    pr = maker()
    if split and pr.params["boundary"] == inputs.OPEN:
        pytest.skip("one image")
    p = orc.make_params(**dict(pr.params, n_leaf=leaf))
    s = orc.shear_offset(p, t)
    tg = inputs.sample_targets(pr.n, 2048, seed=9)
    ref = orc.bh(p, pr.x, pr.y, pr.z, pr.m, s=s, targets=tg)
    ctx = make_ctx(pr, leaf_size=leaf, split_images=split, profile=2)
    try:
        d = Dev(pr, with_v=False)
        a = torch.empty((3, pr.n), dtype=torch.float64, device="cuda")
        rb.rb_gravity(ctx, d.parts, pr.n, pr.n, t, a[0], a[1], a[2])
        st = rb.rb_stats(ctx)
    finally:
        rb.rb_destroy(ctx)
    assert rms_rel(a.cpu().numpy().T[tg], ref) <= TOL
    if pr.n <= 70000:
        T = orc.Tree(p, pr.x, pr.y, pr.z, pr.m)
        T.walk(s=s)
        for k in ("open_tests", "cells", "pp"):
            assert st[k] == T.stats[k], (k, st[k], T.stats[k])
