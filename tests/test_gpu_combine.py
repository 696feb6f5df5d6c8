"""Rows whose sums come from few and from many windows, at the edges of the combine's batches, against
float64 sums. Needs an MI355X.

Both sides add k rounded products, each off by at most (k + 1)·u·(|A||x|) in any order, u = 2⁻⁵³: (2k + 4)·u
covers both. Passes in FP32 round with u = 2⁻²⁴, also the values and x.
"""
import sys

import numpy as np
import pytest
import scipy.sparse as sp

from paper_1912_04263_amd import qpg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [qpg.QPG_FP64, qpg.QPG_MIXED])
@pytest.mark.parametrize("windows", [1, 2, 3, 4, 5, 8, 9, 16, 17, 19, 25, 33, 70])
def test_rows_over_windows(windows, precision):
    print("[case] combine", windows, precision, file=sys.stderr, flush=True)
    m, n = 700, 1024 * windows - 5
    rng = np.random.default_rng(windows)
    A = sp.random(m, n, 0.04, format="csr", random_state=rng, data_rvs=rng.standard_normal)
    x, y = rng.standard_normal(n), rng.standard_normal(m)
    u = 2.0**-53 if precision == qpg.QPG_FP64 else 2.0**-24
    aA = abs(A)
    with qpg.Solver(sp.identity(n, format="csc"), np.zeros(n), A.tocsc(), -np.ones(m), np.ones(m), scaling_iters=0,
                    spmv_window_cols=1024, precision="fp64" if precision == qpg.QPG_FP64 else "mixed") as s:
        ax, aty = s.apply(qpg.QPG_OP_A, x, precision), s.apply(qpg.QPG_OP_AT, y, precision)
    assert np.all(np.abs(ax - A @ x) <= (2 * np.diff(A.indptr) + 4) * u * (aA @ np.abs(x)))
    deg = np.bincount(A.indices, minlength=n)
    assert np.all(np.abs(aty - A.T @ y) <= (2 * deg + 4) * u * (aA.T @ np.abs(y)))
