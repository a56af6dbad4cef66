"""Items of two blocks of 16 columns in the FMM evaluation (launches of two such items per CU and
more): column counts around the blocks, a last item of one target, clustered poles, both
products, on sampled rows against the Cauchy matrix of the solver's own factors.

Tolerance: 1e-12 sum |Qhat_ij X_j| per entry, the bound of the narrower items (a column's sums
are the same, in the same order)."""
import numpy as np
import pytest

from paper_2108_04209_amd import gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N, M = 40001, 80


def test_wide_items():
    from paper_2108_04209_amd import native
    from tests import gpu_pipeline as gp
    batch, X = gen.small_batch([N], seed=69, kind="clustered", m=M)
    opts = native.default_opts(method=2)
    res = gp.run(batch, opts=opts)
    pr = batch.problem(0)
    zo, bo, eta, org = (res[k] for k in ("zhat", "b", "eta", "origin"))
    rng = np.random.default_rng(6)
    rows = np.unique(np.r_[0, 63, 64, N - 2, N - 1, rng.choice(N, 32, replace=False)])
    for trans in (0, 1):
        if trans:
            t = (pr.d[None, :] - pr.d[org[rows]][:, None]) - eta[rows][:, None]
            Q = zo[None, :] * bo[rows][:, None] / t
        else:
            t = (pr.d[rows][:, None] - pr.d[org][None, :]) - eta[None, :]
            Q = zo[rows][:, None] * bo[None, :] / t
        for m in (17, 32, 63, 64, 65, 80):
            Y = gp.apply_from(batch, zo, bo, eta, org, X[:, :m], trans, opts=opts)
            want, tol = Q @ X[:, :m], 1e-12 * (np.abs(Q) @ np.abs(X[:, :m]))
            assert np.all(np.abs(Y[rows] - want) <= tol), (m, trans)
