"""Walks: how the lanes share a list among an item's members, the waves per item
by the number of items, and items shared by several workgroups."""
import numpy as np
import pytest

from paper_1110_4876_amd import inputs

pytestmark = pytest.mark.gpu


def _gravity(pr, **kw):
    from gpu_util import Dev, gravity, make_ctx
    from paper_1110_4876_amd import rb
    d = Dev(pr, with_v=False)
    c = make_ctx(pr, **kw)
    try:
        a = gravity(c, d, pr.n, 100.0)
        np.testing.assert_array_equal(gravity(c, d, pr.n, 100.0), a)
    finally:
        rb.rb_destroy(c)
    assert np.all(np.isfinite(a))
    return a


def _close(a, b, tol):
    assert np.sqrt(np.sum((a - b) ** 2)) <= tol * np.sqrt(np.sum(b ** 2))


@pytest.mark.parametrize("G", [16, 32, 64])
@pytest.mark.parametrize("n,leaf", [(5, 1), (16, 1), (33, 1), (64, 1), (65, 1), (6000, 1), (6000, 8)])
def test_one_wave_matches_two(n, G, leaf):
    # Items of 1 to G members: a group of four lanes serves one block of
    # members or two, and the last block may be partial.  One wave and two per
    # item accept the same entries and differ in the FP32 summation order
    # only: both sum at most 64 terms in FP32 (unit roundoff 6e-8) and the rest
    # in FP64, so 1e-6 of the rms covers the cancellation of in-plane terms.
    from paper_1110_4876_amd import rb
    pr = inputs.sheet(n, seed=G).with_params(theta=0.45)
    kw = dict(precision=rb.RB_FP32_MIXED, group_size=G, leaf_size=leaf)
    _close(_gravity(pr, walk_waves=1, **kw), _gravity(pr, walk_waves=2, **kw), 1e-6)


@pytest.mark.parametrize("n", [63, 64, 65, 896, 897, 1760, 1761, 5120, 5121])
@pytest.mark.parametrize("leaf", [1, 8])
def test_eight_waves_match_one(n, leaf):
    # walk_waves = 4 runs eight waves per item up to 320 G particles, four
    # above, and four workgroups per item up to 56 G, two up to 110 G
    from paper_1110_4876_amd import rb
    pr = inputs.sheet(n, seed=3).with_params(theta=0.4)
    kw = dict(precision=rb.RB_FP32_MIXED, group_size=16, leaf_size=leaf)
    _close(_gravity(pr, walk_waves=4, **kw), _gravity(pr, walk_waves=1, **kw), 1e-6)


@pytest.mark.parametrize("n", [40, 64, 65, 700, 2048, 2049, 8192, 8193])
@pytest.mark.parametrize("leaf", [1, 4])
def test_fp64_items_shared_by_workgroups(n, leaf):
    # up to 32 items of 64 particles four workgroups an item, up to 128 two,
    # against each lane's own walk.  The sums differ in their order only: at most a few
    # thousand FP64 terms (1.1e-16 each), and the in-plane cancellation of a
    # sheet (under 100)
    for pr in (inputs.sheet(n, seed=n).with_params(theta=0.5),
               inputs.plummer(n, seed=n, b=0.01).with_params(theta=0.6)):
        _close(_gravity(pr, leaf_size=leaf), _gravity(pr, leaf_size=leaf, walk64_schedule=1), 1e-11)


@pytest.mark.parametrize("n", [16384, 16385, 32769, 34752, 34753, 65537, 70001])
def test_fp64_last_items_shared(n):
    # more than 256 items: the last four of every eighth by two workgroups, from
    # 544 items on (eight waves) the last eight; the bound as above
    for pr in (inputs.sheet(n, seed=n).with_params(theta=0.5),
               inputs.plummer(n, seed=n, b=0.01).with_params(theta=0.6)):
        _close(_gravity(pr), _gravity(pr, walk64_schedule=1), 1e-11)


def test_shared_items_beside_whole_ones():
    # a batch of patches under and over 32 and 128 items, and one so large that
    # none is shared: every patch has the lanes' own walks' forces
    import torch
    from gpu_util import Dev
    from paper_1110_4876_amd import rb
    from test_gpu_batch import _batch_ctx, _concat
    # (and on both sides of 4,096 items and of a third of them: eight waves with
    # the largest patch's last items shared, and four)
    for sizes in ((100, 2048, 2049, 9000, 64), (100, 2048, 33000), (20000, 40000, 9000),
                  (100000, 90000, 80000), (90000, 90000, 90000)):
        ps = [inputs.sheet(n, seed=n).with_params(theta=0.5) for n in sizes]
        big, off = _concat(ps)
        out = []
        for kw in ({}, {"walk64_schedule": 1}):
            ctx = _batch_ctx(ps, off, rb.RB_FP64, **kw)
            try:
                d = Dev(big)
                a = [torch.empty(big.n, dtype=torch.float64, device="cuda") for _ in range(3)]
                for _ in range(2):
                    rb.rb_batch_gravity(ctx, d.parts, 50.0, *a)
                rb.rb_sync(ctx)
                out.append(torch.stack(a, 1).cpu().numpy())
            finally:
                rb.rb_destroy(ctx)
        for k in range(len(ps)):
            sl = slice(off[k], off[k + 1])
            _close(out[0][sl], out[1][sl], 1e-11)


@pytest.mark.parametrize("n", [3000, 20000])
def test_items_follow_changed_parameters(n):
    # shared items (four workgroups each, or a patch's last ones) and another
    # schedule, image split or precision set on the same context and back; the
    # bounds as above (FP32-mixed opens other cells: both are within 10% at
    # theta = 0.5)
    from gpu_util import Dev, gravity, make_ctx
    from paper_1110_4876_amd import rb
    pr = inputs.sheet(n, seed=n).with_params(theta=0.5)
    d = Dev(pr, with_v=False)
    ref = _gravity(pr, walk64_schedule=1)
    c = make_ctx(pr)
    try:
        for kw, tol in (({}, 1e-11), ({"split_images": 1}, 1e-11), ({}, 1e-11),
                        ({"walk64_schedule": 2}, 1e-11), ({"walk64_schedule": 3}, 1e-11),
                        ({"precision": rb.RB_FP32_MIXED}, 0.1), ({}, 1e-11),
                        ({"split_images": 0}, 1e-11)):
            rb.rb_set_params(c, rb.params_from_problem(pr.params, **kw))
            _close(gravity(c, d, n, 100.0), ref, tol)
    finally:
        rb.rb_destroy(c)


@pytest.mark.parametrize("G,leaf", [(16, 1), (16, 8), (64, 1)])
def test_sparse_children_of_populous_nodes(orc, G, leaf):
    # A sphere's sparse octants beside its core are items of their own.  A
    # group accepts a cell only where each member would, so the grouped walk
    # errs no more than the FP64 walk, but for FP32 rounding (1e-5 of the rms
    # covers it, as at theta = 0).
    from gpu_util import Dev, export, make_ctx
    from paper_1110_4876_amd import rb
    pr = inputs.plummer(30000, seed=8, b=0.01, quadrupole=True).with_params(theta=0.6)
    tg = inputs.sample_targets(pr.n, 1000, seed=1)
    p = orc.make_params(**pr.params)
    ref = orc.direct(p, pr.x, pr.y, pr.z, pr.m, n_active=pr.n, targets=tg)
    a64 = _gravity(pr, leaf_size=leaf)[tg]
    a32 = _gravity(pr, precision=rb.RB_FP32_MIXED, group_size=G, leaf_size=leaf)[tg]
    den = np.sqrt(np.sum(ref ** 2))
    e64, e32 = (np.sqrt(np.sum((a - ref) ** 2)) / den for a in (a64, a32))
    assert e32 <= e64 + 1e-5, (e32, e64)
    # and the FP64 moments of an FP32-mixed tree, which the items also carry
    c = make_ctx(pr, precision=rb.RB_FP32_MIXED, group_size=G, leaf_size=leaf)
    try:
        rb.rb_tree_build(c, Dev(pr, with_v=False).parts, pr.n, pr.n)
        t = export(c)
    finally:
        rb.rb_destroy(c)
    i = int(np.argmin(t["level"]))
    assert t["count"][i] == pr.n
    assert abs(t["M"][i] - pr.m.sum()) <= 1e-12 * pr.m.sum()
