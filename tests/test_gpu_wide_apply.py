"""Blocks of right-hand sides around the column groups (16) and passes (64) of the apply
kernels, in problems around their 64-row tiles and leaves, both products, through the FMM and
by direct sums, against the oracle's product on the oracle's own factors.

Tolerance: 1e-12 sum |Qhat_ij X_j| per entry, the bound of the narrower blocks (the kernels'
sums differ in order only, and the far field's interpolation is the same)."""
import numpy as np
import pytest

from paper_2108_04209_amd import gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("method", [1, 2])
@pytest.mark.parametrize("m", [3, 4, 15, 16, 17, 33, 63, 64, 65, 81])
def test_wide_apply(orc, m, method):
    from paper_2108_04209_amd import native
    from tests import gpu_pipeline as gp
    batch, X = gen.small_batch([1, 63, 65, 128, 129, 1000, 2049], seed=67, kind="clustered", m=m)
    ref = orc.solve_batch(batch)
    for trans in (0, 1):
        Y = gp.apply_from(batch, ref["zhat"], ref["b"], ref["eta"], ref["origin"], X, trans,
                          opts=native.default_opts(method=method))
        for p in range(batch.nprob):
            a, e = int(batch.off[p]), int(batch.off[p + 1])
            pr = batch.problem(p)
            zo, bo, eta, org = (ref[k][a:e] for k in ("zhat", "b", "eta", "origin"))
            Yo = orc.cauchy_apply(pr.d, zo, bo, eta, org, X[a:e], trans=trans)
            Q = zo[:, None] * bo[None, :] / ((pr.d[:, None] - pr.d[org][None, :]) - eta[None, :])
            Qa = np.abs(Q.T if trans else Q)
            tol = 1e-12 * (Qa @ np.abs(X[a:e]))
            assert np.all(np.abs(Y[a:e] - Yo) <= tol), (p, trans)


@pytest.mark.parametrize("n", [40000, 40001])
def test_interval_expansion(orc, n):
    """Far boxes through the targets' interval (launches with two items per CU and more): b, and
    3 and 16 columns of both products, in problems whose last item holds 64 targets or one
    (no interval), clustered poles, on sampled rows."""
    from paper_2108_04209_amd import native
    from tests import gpu_pipeline as gp
    batch, X = gen.small_batch([n], seed=68, kind="clustered", m=16)
    res = gp.run(batch, opts=native.default_opts(method=2))
    pr = batch.problem(0)
    zo, bo, eta, org = (res[k] for k in ("zhat", "b", "eta", "origin"))
    rng = np.random.default_rng(5)
    rows = np.unique(np.r_[0, 63, 64, n - 2, n - 1, rng.choice(n, 48, replace=False)])
    ob = orc.bnorm(pr.d, zo, eta, org, roots=rows)
    assert np.all(np.abs(bo[rows] - ob) <= 1e-12 * ob)
    for trans in (0, 1):
        if trans:
            t = (pr.d[None, :] - pr.d[org[rows]][:, None]) - eta[rows][:, None]
            Q = zo[None, :] * bo[rows][:, None] / t
        else:
            t = (pr.d[rows][:, None] - pr.d[org][None, :]) - eta[None, :]
            Q = zo[rows][:, None] * bo[None, :] / t
        for m in (3, 16):
            Y = gp.apply_from(batch, zo, bo, eta, org, X[:, :m], trans,
                              opts=native.default_opts(method=2))
            Yo = orc.cauchy_apply(pr.d, zo, bo, eta, org, X[:, :m], trans=trans, rows=rows)
            tol = 1e-12 * (np.abs(Q) @ np.abs(X[:, :m]))
            assert np.all(np.abs(Y[rows] - Yo) <= tol), (trans, m)
