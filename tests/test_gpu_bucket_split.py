"""The bucket sort where a few buckets hold most of the keys: they are split
again and again, by key bits and among equal keys by slot.  Keys and order
against the oracle's insertion tree, exactly."""
import numpy as np
import pytest

from paper_1110_4876_amd import inputs

pytestmark = pytest.mark.gpu


def _place(n, f, seed=0):
    pr = inputs.plummer(n, seed=seed)
    rng = np.random.default_rng(seed + 1)
    pr.x[:], pr.y[:], pr.z[:] = f(rng, n)
    return pr


def _cell(k):
    # k particles in one cell of level 4 (8 wide in the box of 128), the rest
    # spread over the box
    def f(rng, n):
        p = rng.uniform(-63.0, 63.0, (3, n))
        p[:, :k] = rng.uniform(8.5, 15.5, (3, k))
        return p
    return f


def _equal(k):
    # all particles at k places
    def f(rng, n):
        p = rng.uniform(1.0, 2.0, (3, k))
        return p[:, np.arange(n) % k]
    return f


def _geometric(rng, n):
    # ever closer to a corner: a split tells only a few particles apart
    s = 60.0 * 2.0 ** -(np.arange(n) % 18)
    return np.stack([s, s, s]) * rng.uniform(0.9, 1.0, (3, n))


def _removed(rng, n):
    p = rng.uniform(-1.0, 1.0, (3, n))
    p[0, : n // 2] = np.nan
    return p


CASES = [("plummer", 20000, None), ("plummer70000", 70000, None)] + \
    [(f"cell{k}", 3000, _cell(k)) for k in (511, 512, 513, 1024, 1025, 2900)] + \
    [(f"equal{k}", 3000, _equal(k)) for k in (1, 2, 5, 600)] + \
    [("geometric", 6000, _geometric), ("removed", 3000, _removed)] + \
    [(f"one{n}", n, None) for n in (1, 2, 64, 65, 1023, 1025, 2047, 2048, 2049, 4096, 4097)] + \
    [("one_equal", 2048, _equal(1)), ("one_cells", 2048, _cell(1500)),
     ("one_removed", 1700, _removed)]


@pytest.mark.parametrize("name,n,f", CASES, ids=[c[0] for c in CASES])
def test_concentrated_keys_match_oracle(orc, name, n, f):
    from gpu_util import Dev, export, make_ctx
    from paper_1110_4876_amd import rb
    pr = inputs.plummer(n, seed=3) if f is None else _place(n, f)
    ref = orc.Tree(orc.make_params(**pr.params), pr.x, pr.y, pr.z, pr.m).export()
    ctx = make_ctx(pr)
    try:
        for _ in range(2):  # the counters are ready for a second sort
            rb.rb_tree_build(ctx, Dev(pr, with_v=False).parts, pr.n, pr.n)
            g = export(ctx)
            for k in ("keys", "perm", "level", "first", "count"):
                m = len(ref[k])
                np.testing.assert_array_equal(g[k][:m], ref[k], err_msg=k)
    finally:
        rb.rb_destroy(ctx)


def test_concentrated_patch_behind_many_slots():
    # slots above 2^18 in a bucket that is split: the same order as alone
    from gpu_util import Dev, export, make_ctx
    from paper_1110_4876_amd import rb
    from test_gpu_batch import _batch_ctx, _concat
    ps = [inputs.plummer(n, seed=n) for n in (150000, 130000)]
    big, off = _concat(ps)
    ctx = _batch_ctx(ps, off, rb.RB_FP64)
    try:
        rb.rb_tree_build(ctx, Dev(big, with_v=False).parts, big.n, big.n)
        got = export(ctx, 1)
    finally:
        rb.rb_destroy(ctx)
    c1 = make_ctx(ps[1])
    try:
        rb.rb_tree_build(c1, Dev(ps[1], with_v=False).parts, ps[1].n, ps[1].n)
        ref = export(c1)
    finally:
        rb.rb_destroy(c1)
    assert np.all(ref["keys"][1:ps[1].n] >= ref["keys"][:ps[1].n - 1])
    for k in ("keys", "perm"):
        np.testing.assert_array_equal(got[k][:ps[1].n], ref[k][:ps[1].n], err_msg=k)
