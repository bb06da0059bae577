"""FP32-mixed walk, several waves per item: an item's n members have floor(64 / n)
lanes each in every wave, whose sums are added across the waves and then
pairwise, for every number of lanes per member."""
import numpy as np
import pytest

from paper_1110_4876_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 12, 13, 16, 21, 22, 32, 33, 64])
@pytest.mark.parametrize("waves", [2, 4])
def test_members_sums(orc, n, waves):
    # theta = 0: every pair is summed, in FP32 with at most 64 terms to a sum
    # (unit roundoff 6e-8) and FP64 above, positions relative to the item's
    # centre rounded to FP32 (each pair's term to a few 6e-8 at separations
    # comparable to the sphere's): 1e-5 of the rms
    from gpu_util import Dev, gravity, make_ctx, rms_rel
    from paper_1110_4876_amd import rb
    pr = inputs.plummer(n, seed=n, b=0.3).with_params(theta=0.0, W=16.0, x0=(-8.0,) * 3)
    for a in (pr.x, pr.y, pr.z):
        np.clip(a, -7.0, 7.0, out=a)
    c = make_ctx(pr, precision=rb.RB_FP32_MIXED, walk_waves=waves)
    try:
        a = gravity(c, Dev(pr, with_v=False), n)
    finally:
        rb.rb_destroy(c)
    ref = orc.direct(orc.make_params(**pr.params), pr.x, pr.y, pr.z, pr.m)
    if n == 1:
        assert np.all(a == 0.0)
    else:
        assert rms_rel(a, ref) <= 1e-5
