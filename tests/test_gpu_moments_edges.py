"""Moments on both sides of the size up to which one workgroup does the bottom
large nodes too (256 group_size particles): the same bits as level by level."""
import numpy as np
import pytest

from paper_1110_4876_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G,n", [(16, 4096), (16, 4097), (32, 8192), (32, 8193), (64, 16384),
                                 (64, 16385)])
@pytest.mark.parametrize("leaf", [1, 32])
def test_bottom_nodes(G, n, leaf):
    from gpu_util import Dev, export, make_ctx
    from paper_1110_4876_amd import rb
    pr = inputs.plummer(n, seed=n, quadrupole=True)
    out = []
    for k in (0, 6):
        ctx = make_ctx(pr, group_size=G, leaf_size=leaf, moments_level_log2=k)
        try:
            rb.rb_tree_build(ctx, Dev(pr, with_v=False).parts, n, n)
            out.append(export(ctx))
        finally:
            rb.rb_destroy(ctx)
    for f in out[0]:
        np.testing.assert_array_equal(out[0][f], out[1][f], err_msg=f)
    assert abs(out[0]["M"][0] - pr.m.sum()) <= 1e-12 * pr.m.sum()
