"""Matrix passes over matrices larger than the memory-side cache, where part of the loads go past the
caches, against float64 sums. Needs an MI355X.

In any order of additions a sum of k rounded products is off by at most (k + 1)·u·(|A||x|), u = 2⁻⁵³ in FP64
and 2⁻²⁴ in FP32, where rounding the values and x to FP32 adds 2 more u. The float64 sums that are compared
with are off by at most (k + 1)·2⁻⁵³ of the same, so (2k + 4)·u covers both.
"""
import sys

import numpy as np
import pytest
import scipy.sparse as sp

from paper_1912_04263_amd import qpg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("entries,precision", [(14_000_000, qpg.QPG_FP64), (23_000_000, qpg.QPG_MIXED)])
def test_passes_over_matrices_beyond_the_cache(entries, precision):
    print("[case] streaming", entries, precision, file=sys.stderr, flush=True)
    m, n = 220_001, 20_003  # windows of several tiles, with remainders
    rng = np.random.default_rng(5)
    per_row = -(-entries // m)
    col = rng.integers(0, n, (m, per_row))
    ptr = np.arange(0, m * per_row + 1, per_row)
    A = sp.csr_matrix((rng.standard_normal(m * per_row), col.ravel(), ptr), shape=(m, n))
    A.sum_duplicates()
    P = sp.diags(rng.random(n) + 0.5).tocsc()
    x, y = rng.standard_normal(n), rng.standard_normal(m)
    u = 2.0**-53 if precision == qpg.QPG_FP64 else 2.0**-24
    aA = abs(A)
    with qpg.Solver(sp.triu(P).tocsc(), np.zeros(n), A.tocsc(), -np.ones(m), np.ones(m), scaling_iters=0,
                    precision="fp64" if precision == qpg.QPG_FP64 else "mixed") as s:
        ax, aty = s.apply(qpg.QPG_OP_A, x, precision), s.apply(qpg.QPG_OP_AT, y, precision)
        again = s.apply(qpg.QPG_OP_A, x, precision)
    assert np.array_equal(ax, again)
    assert np.all(np.abs(ax - A @ x) <= (2 * np.diff(A.indptr) + 4) * u * (aA @ np.abs(x)))
    deg = np.bincount(A.indices, minlength=n)
    assert np.all(np.abs(aty - A.T @ y) <= (2 * deg + 4) * u * (aA.T @ np.abs(y)))
