"""Which batches the adjoint sums directly, whatever the solver's method: those of few pole-root pairs
and no problem above 64 leaves, bit for bit method 1; and the FMM's tree edges (two leaves and one
pole, leaves of 128, refused problems) in batches that a large problem takes there, to the bar of
the adjoint's other FMM tests."""
import numpy as np
import pytest

from paper_2108_04209_amd import gen
from tests.test_gpu_grad_fmm import gradients, regular

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("sizes,kw", [([600], dict(method=2)), ([1500], dict(method=2, fmm_leaf=256)),
                                      ([4097], dict(method=2, fmm_leaf=256)), ([1024, 300], dict(unshifted=1)),
                                      ([1100] * 20, dict(fmm_crossover=512))])
def test_direct(sizes, kw):
    batch = regular(sizes, 151)
    for a, b in zip(gradients(batch, True, **kw), gradients(batch, True, method=1)):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("proj", [False, True])
@pytest.mark.parametrize("sizes,leaf", [([129, 1025, 20, 4097], 64), ([3000, 200, 5001], 64),
                                        ([2600, 1300, 8193], 128)])
def test_trees(sizes, leaf, proj):
    batch = regular(sizes, 153)
    if sizes[0] == 3000:
        batch.rho[1] = -1.0
    want = gradients(batch, proj, method=1)
    got = gradients(batch, proj, method=2, fmm_leaf=leaf)
    assert not np.array_equal(want[0], got[0], equal_nan=True)
    for w, g in zip(want, got):
        off = batch.off if w.size == batch.total_n else np.arange(batch.nprob + 1)
        for p in range(batch.nprob):
            a, e = int(off[p]), int(off[p + 1])
            if batch.rho[p] <= 0.0:
                assert np.isnan(w[a:e]).all() and np.isnan(g[a:e]).all()
            else:
                assert np.abs(g[a:e] - w[a:e]).max() <= 1e-9 * np.abs(w[a:e]).max(), p
