"""The FMM solver on problems scaled by 2^+-400, where t^2 of a source times its weight leaves the
exponent range: f and its derivative scale, so the iteration takes as many steps as on the
unscaled problem but for rounding (2 % of the mean), converges everywhere, and ends within the
stopping test's bound, 2 c n eps (lambda - d_0) each.  300 roots: local expansions of poles alone;
2048: of boxes as well."""
import numpy as np
import pytest

from paper_2108_04209_amd import gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("e", [-400, 400])
@pytest.mark.parametrize("n", [300, 2048])
def test_solver_far_from_one(n, e):
    from paper_2108_04209_amd import native
    from tests import gpu_pipeline as gp
    batch = gen.small_batch([n, n - 17], seed=127)
    s = 2.0 ** e
    sb = gen.Batch(off=batch.off, d=batch.d * s, z=batch.z, rho=batch.rho * s)
    r0, r1 = (gp.run(b, opts=native.default_opts(method=2), vectors=False) for b in (batch, sb))
    assert not r0["status"].any() and not r1["status"].any()
    i0, i1 = (np.mean(r["iters"] & native.ITER_COUNT_MASK) for r in (r0, r1))
    assert abs(i1 - i0) <= 0.02 * i0
    span = batch.d.max() + batch.rho.max() * n
    assert np.all(np.abs(r1["lam"] / s - r0["lam"]) <= 4 * n * 2.0 ** -52 * span)
