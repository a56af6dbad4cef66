"""Branches of large launches that other tests do not reach: the adjoint with the far field through
the targets' interval (two items per CU and more), with and without projections, last item of one
target; and evaluation items of two blocks of 16 columns where three are asked for (32 items per
CU and more), the last item half padding.

Tolerances: the adjoint 1e-9 of the largest gradient against direct sums on poles at least a
quarter of their mean distance apart (as for smaller launches: terms exceed the gradients by less
than 1e4, and 40001 of them in another order differ by sqrt(n) eps of their sum); products
1e-12 sum |Qhat_ij X_j| per entry, as for the narrower items."""
import numpy as np
import pytest

from paper_2108_04209_amd import gen
from tests.test_gpu_grad_fmm import gradients, regular

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("proj", [False, True])
def test_adjoint(proj):
    batch = regular([40001], 141)
    want = gradients(batch, proj, method=1)
    got = gradients(batch, proj, method=2)
    for w, g in zip(want, got):
        assert np.abs(g - w).max() <= 1e-9 * np.abs(w).max()


def test_three_blocks():
    from paper_2108_04209_amd import native
    from tests import gpu_pipeline as gp
    n, m = 4097, 48
    batch = gen.small_batch([n] * 64, seed=143)
    ref = gp.run(batch, opts=native.default_opts(method=1))
    X = np.random.default_rng(143).standard_normal((batch.total_n, m))
    rows = np.unique(np.r_[0, 63, 64, n - 2, n - 1, np.random.default_rng(7).choice(n, 24, replace=False)])
    for trans in (0, 1):
        Y = gp.apply_from(batch, ref["zhat"], ref["b"], ref["eta"], ref["origin"], X, trans,
                          opts=native.default_opts(method=2))
        for p in (0, 63):
            s = slice(p * n, p * n + n)
            d, zh, b, eta, org = batch.d[s], *(ref[k][s] for k in ("zhat", "b", "eta", "origin"))
            if trans:
                Q = zh[None, :] * b[rows][:, None] / ((d[None, :] - d[org[rows]][:, None]) - eta[rows][:, None])
            else:
                Q = zh[rows][:, None] * b[None, :] / ((d[rows][:, None] - d[org][None, :]) - eta[None, :])
            assert np.all(np.abs(Y[s][rows] - Q @ X[s]) <= 1e-12 * (np.abs(Q) @ np.abs(X[s])))
