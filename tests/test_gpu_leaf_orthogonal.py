"""Orthogonality of the leaves' eigenvectors.  With a tolerance that deflates every rank-one problem
the eigenmatrix of a tree is its leaves' (and permutations), so products with the identity give
them as they are.

Tolerance 1.5 eps sqrt(10 L): a rotation keeps a row's norm and the angle of two rows to about an
eps of rounding, a row goes through one a round, and ten sweeps of L rounds add up at random.  A
rotation whose c^2 + s^2 is off by an ulp to one side adds up in proportion instead."""
import numpy as np
import pytest

from paper_2108_04209_amd import gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("leaf", [30, 64, 126, 128])
def test_leaf_eigenvectors(leaf):
    from paper_2108_04209_amd import native
    from tests import gpu_pipeline as gp
    ctx = gp.context()
    tree = gen.hss_tree(n=leaf * 4, leaf=leaf, r=1, cfg=3)
    plan = native.HSSPlan(ctx, leaf, tree.depth, 1)
    gens = {k: gp.to_dev(v) for k, v in native.pack_hss(tree).items()}
    D = np.random.default_rng(leaf).standard_normal((4, leaf, leaf))
    gens["leaf_D"] = gp.to_dev((D + D.transpose(0, 2, 1)).reshape(gens["leaf_D"].shape))
    native.hss_conquer(ctx, plan, gens, opts=native.default_opts(hss_tau=1e6))
    E = torch.eye(tree.n, dtype=torch.float64, device=gp.dev())
    Q = native.hss_apply(ctx, plan, E, trans=0).cpu().numpy()
    tol = 1.5 * 2.0 ** -52 * np.sqrt(10.0 * leaf)
    for q in range(4):
        V = Q[:, q * leaf:(q + 1) * leaf]
        V = V[np.abs(V).max(1) > 0].astype(np.longdouble)
        assert V.shape == (leaf, leaf)
        assert np.abs(V @ V.T - np.eye(leaf)).max() <= tol
