"""Deflation's scan in one launch (problems of up to 4096 poles) and in three, at the edges of
its segments, bit for bit against the oracle; and the kernels that take a row through several
columns (the orthogonal factor, row copies): column counts around their groups, leading
dimensions above the rows, overlapping blocks.  A chain of n rotations adds at most 4 eps n
max|X| of rounding against the same rotations in numpy; copies are exact."""
import numpy as np
import pytest

from paper_2108_04209_amd import gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def batch_of(sizes, seed):
    g = gen.rng_for(seed, 0)
    probs = [gen.RankOne(np.full(n, 0.5), np.abs(g.standard_normal(n)) + 0.1, 1.0) if n % 512 == 1
             else gen.deflation_problem(n, g, rho=float(g.uniform(0.2, 2.0))) for n in sizes]
    return gen.concat(probs), probs


def deflated(batch, tau):
    from paper_2108_04209_amd import native
    from tests import gpu_pipeline as gp
    b = native.Batch(gp.context(), batch.off)
    return b, native.deflate(gp.context(), b, gp.to_dev(batch.d), gp.to_dev(batch.z),
                             gp.to_dev(batch.rho), tau)


@pytest.mark.parametrize("sizes", [[512, 64], [511, 513, 1, 1024, 1025, 4096], [4097, 513, 12]])
def test_segments(orc, sizes):
    batch, probs = batch_of(sizes, 911)
    for tau in (1e-10, 1e-6):
        _, df = deflated(batch, tau)
        g = {k: v.cpu().numpy() for k, v in df.items()}
        for p, pr in enumerate(probs):
            a, e = int(batch.off[p]), int(batch.off[p + 1])
            ref = orc.deflate(pr.d, pr.z, pr.rho, tau)
            assert g["status"][p] == 0 and g["kept"][p] == ref["kept"], (p, tau)
            for k, r in (("perm", "perm"), ("rot_right", "rright"), ("rot_left", "rleft"),
                         ("d", "d"), ("z", "z"), ("rot_c", "c"), ("rot_s", "s")):
                assert np.array_equal(g[k][a:e], ref[r]), (p, k, tau)


def expand_reference(batch, g, X, trans):
    Y = np.empty_like(X)
    for p in range(batch.nprob):
        a, e = int(batch.off[p]), int(batch.off[p + 1])
        rr, rc, rs, perm = (g[k][a:e] for k in ("rot_right", "rot_c", "rot_s", "perm"))
        left = [i for i in range(e - a) if rr[i] >= 0]
        if trans == 0:
            V = np.empty((e - a, X.shape[1]))
            V[perm] = X[a:e]
            for i in reversed(left):
                x, y = V[i].copy(), V[rr[i]].copy()
                V[i], V[rr[i]] = rc[i] * x + rs[i] * y, -rs[i] * x + rc[i] * y
            Y[a:e] = V
        else:
            V = X[a:e].copy()
            for i in left:
                x, y = V[i].copy(), V[rr[i]].copy()
                V[i], V[rr[i]] = rc[i] * x - rs[i] * y, rs[i] * x + rc[i] * y
            Y[a:e] = V[perm]
    return Y


@pytest.mark.parametrize("m", [1, 3, 8, 17])
@pytest.mark.parametrize("trans", [0, 1])
def test_expand_columns(m, trans):
    from paper_2108_04209_amd import native
    from tests import gpu_pipeline as gp
    batch, _ = batch_of([1, 513, 300, 2, 1200], 912)
    b, df = deflated(batch, 1e-10)
    n = batch.total_n
    X = np.random.default_rng(m).standard_normal((n, m))
    want = expand_reference(batch, {k: v.cpu().numpy() for k, v in df.items()}, X, trans)
    tol = 4.0 * 2.0 ** -52 * 1200 * np.abs(X).max()
    Xd = torch.zeros((m, n + 5), dtype=torch.float64, device="cuda")
    Xd[:, :n] = gp.to_dev(X.T)
    Y = torch.full((m, n + 3), 7.0, dtype=torch.float64, device="cuda")
    native.deflate_expand(gp.context(), b, df, Xd, trans=trans, Y=Y)
    assert np.abs(Y[:, :n].cpu().numpy().T - want).max() <= tol
    assert (Y[:, n:] == 7.0).all()
    if trans == 1:  # blocks that overlap by all but one column
        both = torch.zeros((m + 1, n), dtype=torch.float64, device="cuda")
        both[:m] = gp.to_dev(X.T)
        native.deflate_expand(gp.context(), b, df, both[:m], trans=1, Y=both[1:])
        assert np.abs(both[1:].cpu().numpy().T - want).max() <= tol


@pytest.mark.parametrize("m", [1, 7, 16, 33])
def test_copy_rows_columns(m):
    from paper_2108_04209_amd import native
    from tests import gpu_pipeline as gp
    ctx = gp.context()
    g = np.random.default_rng(m)
    ns, nd = g.integers(1, 9, 300), g.integers(1, 9, 300)
    ns[7], nd[11] = 700, 900
    soff, doff = (np.concatenate([[0], np.cumsum(v)]).astype(np.int64) for v in (ns, nd))
    rows = g.integers(0, 9, 300).astype(np.int32)
    src = g.standard_normal((m, int(soff[-1])))
    want = np.full((m, int(doff[-1])), -2.0)
    for p in range(300):
        k = min(ns[p], nd[p], rows[p])
        want[:, doff[p]:doff[p] + k] = src[:, soff[p]:soff[p] + k]
    got = native.batch_copy_rows(ctx, native.Batch(ctx, soff), native.Batch(ctx, doff), gp.to_dev(src),
                                 rows=gp.to_dev(rows, torch.int32), fill=-2.0)
    assert np.array_equal(got.cpu().numpy(), want)


@pytest.mark.parametrize("n,leaf", [(60, 30), (2048, 64), (2240, 70), (3200, 100), (4224, 66),
                                    (6144, 96)])
def test_sort_runs(n, leaf):
    """Node sizes around the runs sorted in LDS (2048 keys; ragged last runs), through the
    deflated HSS pass: eigenvalues within 5e-9 of the closed form and whole eigenvectors'
    residual, as for the larger trees (tau = 1e-10)."""
    from tests.test_gpu_hss_deflate import columns, run, tmatvec
    plan, lam, st = run(gen.tridiag_hss(n, leaf), 1e-10)
    assert st == 0 and (np.diff(lam) >= 0).all()
    exact = np.sort(3.0 - 2.0 * np.cos(np.arange(1, n + 1) * np.pi / (n + 1)))
    assert np.abs(lam - exact).max() <= 5e-9
    ks = np.unique(np.linspace(0, n - 1, 25).astype(int))
    Qs = columns(plan, ks, n)
    res = np.linalg.norm(tmatvec(np.full(n, 3.0), np.full(n - 1, -1.0), Qs) - Qs * lam[ks], axis=0)
    assert res.max() <= 5e-9
