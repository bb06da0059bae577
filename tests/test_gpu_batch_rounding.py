"""A patch in a batch so large that its items have other waves and workgroups
than alone: the same tree and opening decisions, and forces that differ by the
rounding of the sums' order only."""
import numpy as np
import pytest

from paper_1110_4876_amd import inputs

pytestmark = pytest.mark.gpu


# FP64 sums of a few thousand terms (1.1e-16 each) in another order and a
# sheet's in-plane cancellation (under 100); FP32 sums of at most 64 terms (6e-8)
# and FP64 above, the same cancellation.  FP64: 2, 12, 47 and 563 items alone (16
# waves and four, four and two workgroups, 8 waves with shared ends), 624 and
# 5,000 together (8 waves and 4).  FP32-mixed with walk_waves = 4: eight waves and
# four, two and one workgroups alone, four waves together.
@pytest.mark.parametrize("precision,tol", [(0, 1e-11), (1, 1e-6)])
@pytest.mark.parametrize("more", [0, 280000])
def test_patch_in_large_batch(precision, tol, more):
    import torch
    from gpu_util import Dev, gravity, make_ctx
    from paper_1110_4876_amd import rb
    from test_gpu_batch import _batch_ctx, _concat
    ps = [inputs.sheet(n, seed=n).with_params(theta=0.6)
          for n in (100, 750, 3000, 36000) + ((more // 2, more // 2) if more else ())]
    big, off = _concat(ps)
    kw = dict(walk_waves=4) if precision else {}
    ctx = _batch_ctx(ps, off, precision, **kw)
    try:
        d = Dev(big, with_v=False)
        a = torch.empty((3, big.n), dtype=torch.float64, device="cuda")
        rb.rb_batch_gravity(ctx, d.parts, 300.0, a[0], a[1], a[2])
        rb.rb_sync(ctx)
        got = a.cpu().numpy().T
    finally:
        rb.rb_destroy(ctx)
    for k, pr in enumerate(ps[:4]):
        c1 = make_ctx(pr, precision=precision, **kw)
        try:
            ref = gravity(c1, Dev(pr, with_v=False), pr.n, 300.0)
        finally:
            rb.rb_destroy(c1)
        d2 = np.sum((got[off[k]:off[k + 1]] - ref) ** 2)
        assert np.sqrt(d2) <= tol * np.sqrt(np.sum(ref ** 2)), k
