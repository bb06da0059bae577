"""The collision search with 8, 16 and 32 particles per wave, on both sides of
the sizes where it changes: the oracle's pairs and resolutions, and inside a
step those of a search of its own."""
import numpy as np
import pytest

from paper_1110_4876_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 9, 33, 15000, 15001, 100000, 100001])
def test_search_matches_oracle(orc, n):
    from test_gpu_collide import _compare
    pr = inputs.sheet(n, seed=n)
    _compare(orc, pr, pr.extra["radius"], 0.37 * pr.dt, 0.5, 9)


@pytest.mark.parametrize("n", [15000, 15001, 100001])
def test_search_in_step_matches_call(n):
    from test_gpu_collide_step import _steps_then_collide, _steps_with_collisions
    pr = inputs.sheet(n, seed=n).with_params(theta=0.8)
    R = pr.extra["radius"]
    a, pa, ra = _steps_with_collisions(pr, R, 1, 77)
    b, pb, rb_ = _steps_then_collide(pr, R, 1, 77)
    assert pa == pb and ra == rb_ and ra > 0
    for k in a:
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)
