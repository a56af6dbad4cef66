"""Structured products with the eigenmatrix of an HSS pass at the column counts around the
leaf kernel's groups of 8, with leading dimensions above n and leaves that end inside a
wavefront, plain and deflated, against the dense eigenmatrix (the product with the identity,
which other tests hold to the dense matrix).  An entry of Q X is a chain of depth r
orthogonal steps and one leaf product, each with at most n terms and a relative error of n eps
in the norm: (depth r + 1) n eps sqrt(n) max|X| on each side."""
import numpy as np
import pytest

from paper_2108_04209_amd import gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

PAD = 3


@pytest.mark.parametrize("tau", [0.0, 1e-10])
@pytest.mark.parametrize("leaf,depth,r", [(66, 1, 2), (2, 3, 1), (64, 2, 3)])
def test_columns(leaf, depth, r, tau):
    from paper_2108_04209_amd import native
    from tests import gpu_pipeline as gp
    ctx, n = gp.context(), leaf << depth
    tree = gen.hss_tree(n=n, leaf=leaf, r=r, cfg=470 + leaf)
    plan = native.HSSPlan(ctx, leaf, depth, r)
    g = {k: gp.to_dev(v) for k, v in native.pack_hss(tree).items()}
    out = native.hss_conquer(ctx, plan, g, opts=native.default_opts(hss_tau=tau))
    assert int(out["status"].cpu()[0]) == 0
    Q = native.hss_apply(ctx, plan, gp.to_dev(np.eye(n)), trans=0).cpu().numpy().T
    rng = gen.rng_for(471, leaf)
    for m in (1, 7, 8, 9, 33):
        X = rng.standard_normal((m, n))
        Xd = torch.full((m, n + PAD), float("nan"), dtype=torch.float64, device="cuda")
        Xd[:, :n] = gp.to_dev(X)
        tol = 2 * (depth * r + 1) * n ** 1.5 * 2.3e-16 * np.abs(X).max()
        for trans in (0, 1):
            Y = torch.full((m, n + PAD), -7.0, dtype=torch.float64, device="cuda")
            native.hss_apply(ctx, plan, Xd, trans=trans, Y=Y)
            Y = Y.cpu().numpy()
            want = X @ (Q if trans else Q.T)
            assert np.abs(Y[:, :n] - want).max() <= tol, (m, trans)
            assert (Y[:, n:] == -7.0).all(), (m, trans)
