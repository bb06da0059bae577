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


@pytest.mark.parametrize("n", [63, 64, 65, 1000, 5120, 5121])
def test_eight_waves_match_one(n):
    # walk_waves = 4 runs eight waves per item up to 320 G particles, four above
    from paper_1110_4876_amd import rb
    pr = inputs.sheet(n, seed=3).with_params(theta=0.4)
    kw = dict(precision=rb.RB_FP32_MIXED, group_size=16)
    _close(_gravity(pr, walk_waves=4, **kw), _gravity(pr, walk_waves=1, **kw), 1e-6)
