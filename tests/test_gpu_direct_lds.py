"""The direct solver with the poles in LDS against the oracle at the shapes where it can go
wrong: one to three roots, wavefronts whose teams hold a root each (single problems), pairs and
odd numbers of roots and poles per lane, the largest problem that fits and the first that does
not, and batches large enough that a lane holds a root alone.

Bars: eigenvalues within 1e-12 ||A||_2 and equal origins, as for every other solver test; no
root may end its iteration before the stopping test holds or at the cap."""
import numpy as np
import pytest

from paper_2108_04209_amd import gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = {
    "one": [1], "two": [2], "three": [3], "tiny": [1, 2, 3, 4, 5, 7, 8, 9], "65": [65],
    "127": [127, 128, 129], "1023": [1023, 1025], "2049": [2048, 2049], "4096": [4096],
    "4097": [4097, 100], "wave": [33] * 40, "teams": [150, 301] * 60, "lanes": [64] * 3000,
}


@pytest.mark.parametrize("kind", ["uniform", "clustered"])
@pytest.mark.parametrize("shape", list(SHAPES))
def test_direct_solver(orc, shape, kind):
    from paper_2108_04209_amd import native
    from tests import gpu_pipeline as gp
    sizes = SHAPES[shape]
    batch = gen.small_batch(sizes, seed=81, kind=kind)
    res = gp.run(batch, opts=native.default_opts(method=1), vectors=False)
    assert np.all(res["status"] == 0)
    assert np.all(res["iters"] & (native.ITER_UNMET | native.ITER_CAP | native.ITER_SKIPPED) == 0)
    for p in list(range(min(8, batch.nprob))) + [batch.nprob - 1]:
        a, e = int(batch.off[p]), int(batch.off[p + 1])
        pr = batch.problem(p)
        roots = None if e - a <= 1500 else np.unique(np.r_[0, 1, e - a - 1, np.arange(5, e - a, 37)])
        lam, eta, org, its, st = orc.secular(pr.d, pr.z, pr.rho, roots=roots)
        got = slice(a, e) if roots is None else a + roots
        nA = np.abs(lam).max()
        assert np.abs(res["lam"][got] - lam).max() <= 1e-12 * nA
        np.testing.assert_array_equal(res["origin"][got], org)


def test_direct_solver_cap_and_invalid(orc):
    """A cap of one iteration flags the problem and keeps bracketed iterates; an invalid problem
    between valid ones gives NaN and its bits, and leaves the others alone."""
    from paper_2108_04209_amd import native
    from tests import gpu_pipeline as gp
    batch = gen.small_batch([200, 90, 300], seed=82)
    res = gp.run(batch, opts=native.default_opts(method=1, max_iter=1), vectors=False)
    assert np.all(res["status"] == native.ST_NOCONV)
    for p in range(3):
        a, e = int(batch.off[p]), int(batch.off[p + 1])
        d = batch.d[a:e]
        assert np.all(res["lam"][a:e - 1] <= d[1:]) and np.all(res["lam"][a:e] >= d)
    ref = gp.run(batch, opts=native.default_opts(method=1), vectors=False)
    batch.z[int(batch.off[1]) + 7] = 0.0
    bad = gp.run(batch, opts=native.default_opts(method=1), vectors=False)
    a, e = int(batch.off[1]), int(batch.off[2])
    assert list(bad["status"]) == [0, native.ST_ZERO, 0]
    assert np.all(np.isnan(bad["lam"][a:e])) and np.all(bad["iters"][a:e] == native.ITER_SKIPPED)
    keep = np.r_[0:a, e:batch.total_n]
    np.testing.assert_array_equal(bad["lam"][keep], ref["lam"][keep])


@pytest.mark.parametrize("sizes,direct", [([1024], True), ([4096, 300], True), ([1024] * 38, True),
                                          ([1024] * 39, False), ([4097], False),
                                          ([2048] * 10, False)])
def test_small_batches_by_direct_sums(sizes, direct):
    """The automatic method takes direct sums for a batch of few pole-root pairs (4e7 over the
    problems of 1024 roots and more, none above 4096) and the FMM from there: bit for bit
    what method 1, or a crossover of 1024 given, computes."""
    from paper_2108_04209_amd import native
    from tests import gpu_pipeline as gp
    batch = gen.small_batch(sizes, seed=83)
    auto = gp.run(batch)
    same = gp.run(batch, opts=native.default_opts(method=1) if direct
                  else native.default_opts(fmm_crossover=1024))
    for k in ("lam", "eta", "origin", "zhat", "b"):
        assert np.array_equal(auto[k], same[k]), k


@pytest.mark.parametrize("leaf", [64, 256, 1024])
@pytest.mark.parametrize("kind,n", [("uniform", 2049), ("uniform", 20000), ("graded", 5000),
                                    ("stairs", 9000)])
def test_fmm_solver_in_lds(kind, n, leaf):
    """FMM roots against direct sums: items staged in LDS, and leaves that do not fit (large
    leaves, graded poles whose lists are long or overflow) by the same iteration over loads.
    The stopping test |f| <= c n eps (1 + |psi| + |phi|) bounds each solution's error by
    2 c n eps (lambda - d_0), as |psi| <= psi' (lambda - d_0)."""
    from paper_2108_04209_amd import native
    from tests import gpu_pipeline as gp
    batch = gen.small_batch([n, n // 2 + 7], seed=89)
    g = np.random.default_rng(89)
    for p in range(2):
        s, e = int(batch.off[p]), int(batch.off[p + 1])
        m = e - s
        if kind == "graded":
            batch.d[s:e] = np.sort(np.exp(g.uniform(-20.0, 0.0, m))) + 1e-9 * np.arange(m)
        elif kind == "stairs":
            batch.d[s:e] = np.arange(m) // 64 + 1e-7 * (1.0 + np.arange(m) % 64)
    fmm = gp.run(batch, opts=native.default_opts(method=2, fmm_leaf=leaf))
    direct = gp.run(batch, opts=native.default_opts(method=1))
    assert not fmm["status"].any() and not direct["status"].any()
    for p in range(2):
        s, e = int(batch.off[p]), int(batch.off[p + 1])
        span = batch.d[e - 1] - batch.d[s] + batch.rho[p] * np.sum(batch.z[s:e] ** 2)
        tol = 4.0 * native.default_opts().stop_c * (e - s) * 2.0 ** -52 * span
        assert np.max(np.abs(fmm["lam"][s:e] - direct["lam"][s:e])) <= tol


@pytest.mark.parametrize("sizes", [[1], [2, 1, 63, 64, 65], [128, 127, 17], [192, 129, 191, 15], [192] * 5])
@pytest.mark.parametrize("scale", [1.0, 1e-200, 1e150])
def test_small_vectors_in_one_launch(sizes, scale):
    """zhat and b of batches of at most 192 poles (one launch) against the separate kernels
    (persistent = 0) on the same roots: products of up to 192 factors and sums of as many
    positive terms in another order, 4 n eps relative.  A refused problem stays NaN."""
    from paper_2108_04209_amd import native
    from tests import gpu_pipeline as gp
    batch = gen.small_batch(sizes, seed=107)
    batch.d *= scale
    batch.rho *= scale
    if len(sizes) > 2:
        batch.rho[1] = -1.0
    ctx = gp.context()
    b = native.Batch(ctx, batch.off)
    d, z, rho = gp.to_dev(batch.d), gp.to_dev(batch.z), gp.to_dev(batch.rho)
    s = native.secular_solve(ctx, b, d, z, rho)
    res = [[x.cpu().numpy() for x in native.loewner(ctx, b, d, z, rho, s["eta"], s["origin"], s["status"],
                                                    opts=native.default_opts(persistent=p))]
           for p in (1, 0)]
    for got, want in zip(*res):
        assert np.array_equal(np.isnan(got), np.isnan(want))
        ok = ~np.isnan(want)
        assert np.all(np.abs(got[ok] - want[ok]) <= 4 * 192 * 2.0 ** -52 * np.abs(want[ok]))
