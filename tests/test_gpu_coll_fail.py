"""Collision calls that end with an error: the caller's velocities are as they
were, with and without the codes asked for, and the context works on."""
import numpy as np
import pytest

from paper_1110_4876_amd import inputs

pytestmark = pytest.mark.gpu


def _problem(n, boundary=inputs.OPEN):
    # all particles overlap one another: n (n - 1) / 2 pairs in contact
    rng = np.random.default_rng(n)
    x, v = rng.uniform(-0.01, 0.01, (3, n)), rng.normal(size=(3, n))
    params = inputs.base_params(G=1.0, b=0.0, W=16.0, x0=(-8.0,) * 3, boundary=boundary)
    return inputs.Problem(*x, *v, rng.uniform(0.5, 2.0, n), params, n, 0.1)


def _call(name, ctx, d, radius, n, codes):
    from paper_1110_4876_amd import rb
    if name == "collide":
        return rb.rb_collide(ctx, d.parts, radius, n, 0.0, 0.5, 3, codes)
    return rb.rb_sweep(ctx, d.parts, radius, n, 0.0, 0.0, 0.5, 3, codes)


@pytest.mark.parametrize("name", ["collide", "sweep"])
@pytest.mark.parametrize("fault", ["full", "outside"])
@pytest.mark.parametrize("n", [150, 600])
def test_failed_call_leaves_velocities(orc, name, fault, n):
    # a queue of 8 n + 1024 places for n (n - 1) / 2 pairs, or a particle past
    # the periodic faces beside few and many pairs
    from gpu_util import Dev, dev, make_ctx
    from paper_1110_4876_amd import rb
    pr = _problem(n, inputs.OPEN if fault == "full" else inputs.PERIODIC)
    R = np.full(n, 0.1)
    k = n if fault == "full" else n // 6  # the others touch nothing
    R[k:] = 0.0
    pr.x[k:], pr.y[k:] = np.linspace(1.0, 7.0, n - k), np.linspace(-7.0, 7.0, n - k)
    good = pr.x.copy()
    if fault == "outside":
        pr.x[n - 1] = 9.0
    ctx = make_ctx(pr)
    try:
        for codes in (None, np.zeros(16, dtype=np.uint64)):
            d = Dev(pr)
            with pytest.raises(rb.RBError) as ex:
                _call(name, ctx, d, dev(R), n, codes)
            assert ex.value.code == (rb.RB_ECAPACITY if fault == "full" else rb.RB_EOUTSIDE)
            for f, v in d.state().items():
                np.testing.assert_array_equal(v, getattr(pr, f), err_msg=f)
        # the same context on a queue that fits (40 particles overlap)
        pr.x[:], R[40:] = good, 0.0
        if fault == "full":
            pr.x[40:] += 1.0
        d = Dev(pr)
        npair, nres = _call(name, ctx, d, dev(R), n, None)
        st = pr.state()
        _, want, wres, ost = orc.collide(orc.make_params(**pr.params), st, pr.m, R, 0.0, 0.5, 3)
        assert (npair, nres) == (want, wres) and npair > 100
        for f in ("vx", "vy", "vz"):
            assert np.abs(getattr(d, f).cpu().numpy() - ost[f]).max() <= 1e-13 * np.abs(ost[f]).max()
    finally:
        rb.rb_destroy(ctx)
