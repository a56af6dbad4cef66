"""The adjoint's sums through the FMM against its direct sums (method 1) on the same roots.

The far field of every sum is interpolated to about 1e-13 of the sum of its absolute terms; on
poles at least a quarter of their mean distance apart the terms exceed the gradients by less
than 1e4, so the two agree to 1e-9 of the largest gradient.  Batches the automatic method
takes directly agree bit for bit."""
import numpy as np
import pytest

from paper_2108_04209_amd import gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def regular(sizes, seed):
    batch = gen.small_batch(sizes, seed=seed)
    g = np.random.default_rng(seed)
    for p in range(batch.nprob):
        a, e = int(batch.off[p]), int(batch.off[p + 1])
        n = e - a
        batch.d[a:e] = (np.arange(n) + 0.75 * g.random(n)) / n
        batch.z[a:e] = g.choice([-1.0, 1.0], n) * (0.25 + 1.5 * g.random(n)) / np.sqrt(n)
    return batch


def gradients(batch, proj, **kw):
    from paper_2108_04209_amd import native
    from tests import gpu_pipeline as gp
    ctx = gp.context()
    b = native.Batch(ctx, batch.off)
    d, z, rho = gp.to_dev(batch.d), gp.to_dev(batch.z), gp.to_dev(batch.rho)
    s = native.secular_solve(ctx, b, d, z, rho, opts=native.default_opts(method=1))
    g = np.random.default_rng(5)
    gl, gp_, u = (gp.to_dev(g.standard_normal(batch.total_n)) for _ in range(3))
    out = native.secular_backward(ctx, b, d, z, rho, s["eta"], s["origin"], s["status"], g_lam=gl,
                                  g_proj=gp_ if proj else None, u=u if proj else None,
                                  opts=native.default_opts(**kw))
    torch.cuda.synchronize()
    return [x.cpu().numpy() for x in out]


@pytest.mark.parametrize("proj", [False, True])
@pytest.mark.parametrize("sizes,leaf", [([129, 1025, 20], 64), ([3000, 200, 5001], 64),
                                        ([2600, 1300], 128)])
def test_fmm_adjoint(sizes, leaf, proj):
    batch = regular(sizes, 97)
    batch.rho[-1] = -1.0 if len(sizes) == 3 and leaf == 64 and sizes[0] == 3000 else batch.rho[-1]
    want = gradients(batch, proj, method=1)
    got = gradients(batch, proj, method=2, fmm_leaf=leaf)
    for w, g in zip(want, got):
        off = batch.off if w.size == batch.total_n else np.arange(batch.nprob + 1)
        for p in range(batch.nprob):
            a, e = int(off[p]), int(off[p + 1])
            if batch.rho[p] <= 0.0:  # refused: NaN on both paths
                assert np.isnan(w[a:e]).all() and np.isnan(g[a:e]).all()
            else:
                assert np.abs(g[a:e] - w[a:e]).max() <= 1e-9 * np.abs(w[a:e]).max(), p


@pytest.mark.parametrize("sizes,direct", [([4096] * 4, True), ([1024] * 66, True),
                                          ([1024] * 67, False), ([4097], False)])
def test_small_batches_directly(sizes, direct):
    batch = regular(sizes, 98)
    auto = gradients(batch, True)
    same = gradients(batch, True, **(dict(method=1) if direct else dict(fmm_crossover=1024)))
    for a, s in zip(auto, same):
        assert np.array_equal(a, s)
