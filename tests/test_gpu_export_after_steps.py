"""The exported tree after any number of steps: each single-particle leaf holds
the mass of the caller's particle that the permutation names."""
import numpy as np
import pytest

from paper_1110_4876_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps", [1, 2, 3, 1025])
@pytest.mark.parametrize("graph", [0, 1])
def test_permutation_after_steps(steps, graph):
    # (schedules are uploaded 1,024 steps at a time)
    from gpu_util import Dev, export, make_ctx
    from paper_1110_4876_amd import rb
    pr = inputs.sheet(400, seed=1).with_params(theta=1.0)
    ctx = make_ctx(pr, use_graph=graph)
    try:
        d = Dev(pr)
        rb.rb_step(ctx, d.parts, pr.n, pr.n, 0.0, 1e-3 * pr.dt, steps)
        for k in (steps, 0):  # and after a build of the same context
            if k == 0:
                rb.rb_tree_build(ctx, d.parts, pr.n, pr.n)
            t = export(ctx)
            one = (t["is_leaf"] == 1) & (t["count"] == 1)
            assert one.sum() > 300
            np.testing.assert_array_equal(np.sort(t["perm"]), np.arange(pr.n))
            np.testing.assert_array_equal(t["M"][one], pr.m[t["perm"][t["first"][one]]])
    finally:
        rb.rb_destroy(ctx)
