"""Upper boxes of every class (2, 4, .. 64 leaves to a wavefront, larger ones to a workgroup;
boxes of one leaf and partial boxes at a tree's end) in one batch: zhat, b and the products
through the FMM against the direct kernels on the same roots, to the FMM's 1e-11 of the
largest value."""
import numpy as np
import pytest

from paper_2108_04209_amd import gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("sizes", [[129, 150, 257, 513, 1025, 2049], [4097, 130], [8300, 260, 12345],
                                   [33000, 700]])
@pytest.mark.parametrize("m", [1, 5])
def test_box_classes(sizes, m):
    from paper_2108_04209_amd import native
    from tests import gpu_pipeline as gp
    batch, X = gen.small_batch(sizes, seed=101, m=m)
    ctx = gp.context()
    b = native.Batch(ctx, batch.off)
    d, z, rho = gp.to_dev(batch.d), gp.to_dev(batch.z), gp.to_dev(batch.rho)
    Xd = gp.to_dev(X.T)
    fmm, direct = native.default_opts(method=2), native.default_opts(method=1)
    s = native.secular_solve(ctx, b, d, z, rho, opts=fmm)
    res = []
    for o in (fmm, direct):
        zh, bn = native.loewner(ctx, b, d, z, rho, s["eta"], s["origin"], s["status"], opts=o)
        Y = [native.cauchy_apply(ctx, b, d, zh, bn, s["eta"], s["origin"], s["status"], Xd, trans=t,
                                 opts=o) for t in (0, 1)]
        res.append([x.cpu().numpy() for x in (zh, bn, *Y)])
    assert not s["status"].cpu().numpy().any()
    for p in range(len(sizes)):
        a, e = int(batch.off[p]), int(batch.off[p + 1])
        for f, g in zip(*res):
            assert np.abs(f[..., a:e] - g[..., a:e]).max() <= 1e-11 * np.abs(g[..., a:e]).max(), p


@pytest.mark.parametrize("rho", [1e-6, 1.0, 1e6])
@pytest.mark.parametrize("sizes", [[129, 193, 1025], [4097, 2050]])
def test_last_root_far_out(sizes, rho):
    """zhat where the last root lies just above its pole, a spectrum's width and a million widths
    away (it is kept out of the boxes' moments), and where the last leaf is a single pole:
    through the FMM against the direct products, 1e-12 relative per entry."""
    from paper_2108_04209_amd import native
    from tests import gpu_pipeline as gp
    batch = gen.small_batch(sizes, seed=103)
    batch.rho[:] = rho
    ctx = gp.context()
    b = native.Batch(ctx, batch.off)
    d, z, r = gp.to_dev(batch.d), gp.to_dev(batch.z), gp.to_dev(batch.rho)
    s = native.secular_solve(ctx, b, d, z, r, opts=native.default_opts(method=1))
    zh = [native.loewner(ctx, b, d, z, r, s["eta"], s["origin"], s["status"],
                         opts=native.default_opts(method=mt))[0].cpu().numpy() for mt in (2, 1)]
    assert not s["status"].cpu().numpy().any()
    assert np.max(np.abs(zh[0] - zh[1]) / np.abs(zh[1])) <= 1e-12
