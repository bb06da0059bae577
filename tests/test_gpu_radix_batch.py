"""The radix sort on a batch: one large patch among more than 64 small ones
(empty ones, of 1 to 3 particles, of whole tiles and one more or less, with
removed particles), each in the stable order of its own keys."""
import numpy as np
import pytest

from paper_1110_4876_amd import inputs

pytestmark = pytest.mark.gpu

DEAD = np.uint64(0xFFFFFFFFFFFFFFFF)


def _sizes(large):
    # tiles hold 1,024 or 2,048 slots; the large patch is neither the first nor
    # the last, and the list begins and ends with empty patches
    small = [0, 1, 2, 3, 0, 0, 255, 256, 257, 1023, 1024, 1025, 2047, 2048, 2049, 4096, 5000]
    return (small * 3)[:40] + [large] + (small[::-1] * 3)[:39] + [3, 0]


# (four rows a wave below 2^19 slots in all, eight above)
@pytest.mark.parametrize("large", [(1 << 18) + 1, 600000])
def test_patches_in_stable_key_order(orc, large):
    from gpu_util import Dev, export
    from paper_1110_4876_amd import rb
    from test_gpu_batch import _batch_ctx, _concat
    rng = np.random.default_rng(large)
    ps = []
    for k, n in enumerate(_sizes(large)):
        pr = inputs.plummer(max(n, 1), seed=k)
        pr = inputs.Problem(*(a[:n].copy() for a in (pr.x, pr.y, pr.z, pr.vx, pr.vy, pr.vz, pr.m)),
                            pr.params, n, pr.dt)
        if n > 3:
            pr.x[:n // 5] = pr.x[0]  # alike in x, some of them in all
            pr.y[:n // 7], pr.z[:n // 7] = pr.y[0], pr.z[0]
            if k % 2:
                pr.z[rng.integers(0, n, n // 3)] = np.nan
        elif n > 1 and k % 2:
            pr.x[0] = np.nan
        ps.append(pr)
    assert len(ps) > 64
    big, off = _concat(ps)
    ctx = _batch_ctx(ps, off, rb.RB_FP64)
    try:
        d = Dev(big, with_v=False)
        for _ in range(2):
            rb.rb_tree_build(ctx, d.parts, big.n, big.n)
        live_all = rb.rb_tree_info(ctx)[1]
        # (every patch, or with the largest the ones around it and at the ends)
        some = range(len(ps)) if large < 500000 else [0, 1, 2, 38, 39, 40, 41, 42, 79, 80, 81]
        got = {k: export(ctx, k) for k in some}
    finally:
        rb.rb_destroy(ctx)
    total = 0
    for k, pr in enumerate(ps):
        key = orc.keys(orc.make_params(**pr.params), pr.x, pr.y, pr.z)
        order = np.argsort(key, kind="stable")
        live = int(np.sum(key != DEAD))
        total += live
        if k in got:
            np.testing.assert_array_equal(got[k]["keys"][:live], key[order][:live], err_msg=str(k))
            np.testing.assert_array_equal(got[k]["perm"][:live], order[:live], err_msg=str(k))
    assert total == live_all
