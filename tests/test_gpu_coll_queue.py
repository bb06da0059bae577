"""The collision queue between calls: nothing of an earlier call's pairs is
left for the next one."""
import numpy as np
import pytest

from paper_1110_4876_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("graph", [0, 1])
def test_steps_without_particles_leave_the_queue(graph):
    # a step and a call of their own leave their pairs in the queue; steps of no
    # particles then find none, resolve none and change nothing
    from gpu_util import Dev, dev, make_ctx
    from paper_1110_4876_amd import rb
    pr = inputs.sheet(2000, seed=4)
    r = dev(pr.extra["radius"])
    ctx = make_ctx(pr, use_graph=graph)
    try:
        d = Dev(pr)
        rb.rb_set_collisions(ctx, r, 0.5, 7)
        rb.rb_step(ctx, d.parts, pr.n, pr.n, 0.0, pr.dt, 1)
        pairs, resolved = rb.rb_collision_counts(ctx)
        assert pairs > 0 and resolved > 0
        for call in (False, True):
            if call:
                assert rb.rb_collide(ctx, d.parts, r, pr.n, pr.dt, 0.5, 9)[0] > 0
            before = d.state()
            rb.rb_step(ctx, d.parts, 0, 0, pr.dt, pr.dt, 2)
            assert rb.rb_collision_counts(ctx) == (0, 0)
            for k, v in d.state().items():
                np.testing.assert_array_equal(v, before[k], err_msg=k)
        # and the context goes on with particles
        rb.rb_step(ctx, d.parts, pr.n, pr.n, pr.dt, pr.dt, 1)
        assert rb.rb_collision_counts(ctx)[0] > 0
    finally:
        rb.rb_destroy(ctx)
