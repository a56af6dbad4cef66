"""Gradients of single eigenvalues, entry by entry: dlambda_k/dd_i = alpha_k z_i^2 r_ik^2 and
dlambda_k/dz_i = -2 alpha_k z_i r_ik have one term each, so nothing hides an error of the far field
behind a sum.  From given roots, against long double.

Tolerance 64 eps of each entry: through the FMM a term passes two compressions (pole or root to
leaf, leaf to upper box) and, in large launches, one interpolation on the targets' interval, each a
sum of 16 values whose magnitudes add to less than three times the term, and is then a quotient
squared; alpha_k is the reciprocal of a sum of positive terms formed the same way."""
import numpy as np
import pytest

from paper_2108_04209_amd import gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("kind", ["uniform", "clustered"])
@pytest.mark.parametrize("sizes", [[4097] * 2, [4097] * 8])
def test_single_eigenvalues(sizes, kind):
    from paper_2108_04209_amd import native
    from tests import gpu_pipeline as gp
    batch = gen.small_batch(sizes, seed=117, kind=kind)
    n = sizes[0]
    s = gp.run(batch, opts=native.default_opts(method=1), vectors=False)
    for k in (0, n // 2 + 5, n - 1):
        gl = np.zeros(batch.total_n)
        gl[batch.off[:-1] + k] = 1.0
        gd, gz, gr = gp.backward_from(batch, s["eta"], s["origin"], g_lam=gl,
                                      opts=native.default_opts(method=2))
        for p in (0, batch.nprob - 1):
            a, e = int(batch.off[p]), int(batch.off[p + 1])
            d, z = (v[a:e].astype(np.longdouble) for v in (batch.d, batch.z))
            r = 1 / ((d - d[s["origin"][a + k]]) - np.longdouble(s["eta"][a + k]))
            alpha = 1 / ((z * r) ** 2).sum()
            tol = 64 * 2.0 ** -52
            for got, want in ((gd[a:e], alpha * (z * r) ** 2), (gz[a:e], -2 * alpha * z * r),
                              (gr[p:p + 1], alpha / np.longdouble(batch.rho[p]) ** 2)):
                assert np.all(np.abs(got - want) <= tol * np.abs(want)), (k, p)
