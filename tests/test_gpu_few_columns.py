"""One to three columns, alone or left over beside blocks of 16, are as exact on the matrix cores as
on the VALU: columns with a single entry give single entries of Qhat, compared with long double.

Tolerance 4 eps of each entry: 1.5 eps for the difference (d_i - d_K) - eta (|d_i - d_K| is at
most twice it), 1 for its reciprocal (two Newton steps), 0.5 for each of the two products; through
the FMM, entries at most 63 indices away, which no box holds."""
import numpy as np
import pytest

from paper_2108_04209_amd import gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("sizes,method,m", [([300], 1, 1), ([300, 77], 1, 3), ([2049], 2, 17),
                                            ([4097] * 8, 2, 19), ([2049], 2, 35), ([2049], 2, 2)])
def test_few_columns(orc, sizes, method, m):
    from paper_2108_04209_amd import native
    from tests import gpu_pipeline as gp
    batch = gen.small_batch(sizes, seed=119)
    ref = gp.run(batch, opts=native.default_opts(method=1))
    n = sizes[0]
    zh, b, eta = (ref[k].astype(np.longdouble) for k in ("zhat", "b", "eta"))
    d, org = batch.d.astype(np.longdouble), ref["origin"]
    for k in range(0, n, 37):
        X = np.zeros((batch.total_n, m))
        X[batch.off[:-1] + k % np.diff(batch.off), -1] = 1.0
        for trans in ((0, 1) if method == 1 else (1,)):
            Y = gp.apply_from(batch, ref["zhat"], ref["b"], ref["eta"], org, X, trans,
                              opts=native.default_opts(method=method))[:, -1]
            for p in (0, batch.nprob - 1):
                a, e = int(batch.off[p]), int(batch.off[p + 1])
                j = a + k % (e - a)
                rows = np.arange(a, e) if method == 1 else np.arange(max(a, j - 63), min(e, j + 64))
                i, r = (j, rows) if trans else (rows, j)
                want = zh[i] * b[r] / ((d[i] - d[a + org[r]]) - eta[r])
                assert np.all(np.abs(Y[rows] - want) <= 4 * 2.0 ** -52 * np.abs(want)), (k, trans)
