"""Work items of the direct solver in LDS whose roots do not fill the workgroup's wavefronts, in
launches whose largest problem is the one they belong to: a wavefront without roots has no pole
of its own among those staged.  One root, and one more than whole items hold, for workgroups of
two, four and eight wavefronts.

Roots against the solver by scalar fetches (persistent = 0).  The stopping test
|f| <= c n eps (1 + |psi| + |phi|) bounds each solution's error by 2 c n eps (lambda - d_0), as
|psi| <= psi' (lambda - d_0)."""
import numpy as np
import pytest

from paper_2108_04209_amd import gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("sizes", [[1], [3, 1], [1023], [1025], [1535, 1], [2049], [4095]])
def test_last_items(sizes):
    from paper_2108_04209_amd import native
    from tests import gpu_pipeline as gp
    batch = gen.small_batch(sizes, seed=111)
    lds, ref = (gp.run(batch, opts=native.default_opts(method=1, persistent=p), vectors=False)
                for p in (1, 0))
    assert not lds["status"].any() and not ref["status"].any()
    np.testing.assert_array_equal(lds["origin"], ref["origin"])
    for p in range(batch.nprob):
        s, e = int(batch.off[p]), int(batch.off[p + 1])
        span = batch.d[e - 1] - batch.d[s] + batch.rho[p] * np.sum(batch.z[s:e] ** 2)
        tol = 4.0 * (e - s) * 2.0 ** -52 * span
        assert np.max(np.abs(lds["lam"][s:e] - ref["lam"][s:e])) <= tol
