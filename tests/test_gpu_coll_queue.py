"""The collision queue: nothing of an earlier call's pairs is left for the next
one, and the pair with the largest key that there is has its turn."""
import numpy as np
import pytest

from paper_1110_4876_amd import inputs

pytestmark = pytest.mark.gpu

M64 = (1 << 64) - 1


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


def _unxor(z, s):
    x = z
    for _ in range(64 // s + 1):
        x = z ^ (x >> s)
    return x


def _splitmix64_inverse(h):
    z = _unxor(h, 31)
    z = _unxor(z * pow(0x94D049BB133111EB, -1, 1 << 64) & M64, 27)
    z = _unxor(z * pow(0xBF58476D1CE4E5B9, -1, 1 << 64) & M64, 30)
    return (z - 0x9E3779B97F4A7C15) & M64


@pytest.mark.parametrize("pair", [(0, 1), (1, 2)])
def test_largest_key_is_resolved(orc, pair):
    # three particles in a row, the outer ones moving in; the seed gives one of
    # the two pairs the key 2^64 - 1, so that it follows the other
    from test_gpu_collide import _compare
    seed = (_splitmix64_inverse(M64) - ((pair[0] << 35) | (pair[1] << 7))) & M64
    assert orc.splitmix64(seed + ((pair[0] << 35) | (pair[1] << 7))) == M64
    zero = np.zeros(3)
    params = inputs.base_params(G=1.0, b=0.0, W=16.0, x0=(-8.0,) * 3)
    pr = inputs.Problem(np.array([-0.9, 0.0, 0.9]), zero, zero.copy(), np.array([1.0, 0.0, -1.0]),
                        zero.copy(), zero.copy(), np.ones(3), params, 3, 0.1)
    npair, nres = _compare(orc, pr, np.full(3, 0.5), 0.0, 0.5, seed)
    assert npair == 2 and nres == 2


def test_pile_up_time():
    # 300 particles in one place, 44,850 pairs, chains of about 800: resolved
    # side by side by the lanes of a few waves (2.6 ms), not one after the other
    # (55 ms)
    from gpu_util import Dev, dev, make_ctx
    from paper_1110_4876_amd import rb
    n, pile = 20000, 300
    rng = np.random.default_rng(5)
    x, v = rng.uniform(-30.0, 30.0, (3, n)), rng.normal(size=(3, n))
    x[:, :pile] = 7.0 + rng.uniform(0.0, 0.01, (3, pile))
    params = inputs.base_params(G=1.0, b=0.0, W=64.0, x0=(-32.0,) * 3)
    pr = inputs.Problem(*x, *v, rng.uniform(0.5, 2.0, n), params, n, 0.1)
    r = dev(np.where(np.arange(n) < pile, 0.02, 1e-6))
    ctx = make_ctx(pr, profile=1)
    try:
        ms = []
        for _ in range(3):
            npair, _ = rb.rb_collide(ctx, Dev(pr).parts, r, n, 0.0, 0.5, 3)
            assert npair == pile * (pile - 1) // 2
            ms.append(rb.rb_stats(ctx)["ms"]["collide"])
    finally:
        rb.rb_destroy(ctx)
    assert min(ms) < 15.0, ms
