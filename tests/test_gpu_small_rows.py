"""The one-workgroup kernels of small problems on matrices with empty rows beside rows of several segments,
against the general path (speculate = 0): bitwise the same, and the linear solve right. Needs an MI355X.

The numbers of segments and of rows agree on these matrices although a segment is not a row. The linear
solve stops at ‖r‖∞ ≤ 1e-9·‖b‖∞ with r the recursive residual; its true one, from a float64 product, may differ
by the rounding of a hundred steps: 1e-7 leaves two digits, and products that mix up rows miss by O(1).
"""
import sys

import numpy as np
import pytest
import scipy.sparse as sp

from paper_1912_04263_amd import qpg

pytestmark = pytest.mark.gpu


def problem(empty, long, seed, m=100, n=60):
    rng = np.random.default_rng(seed)
    k = np.full(m, 4)
    k[empty] = 0
    k[long] = 30
    cols = [np.sort(rng.choice(n, c, replace=False)) for c in k]
    ptr = np.concatenate([[0], np.cumsum(k)])
    A = sp.csr_matrix((rng.standard_normal(ptr[-1]), np.concatenate(cols), ptr), shape=(m, n))
    M = sp.random(n, n, 0.1, random_state=rng)
    P = sp.csc_matrix(M @ M.T + 0.1 * sp.identity(n))
    return P, rng.standard_normal(n), A, -rng.random(m), rng.random(m)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("empty,long", [([10], [60]), ([60], [10]), ([0], [99]), ([99], [0]), ([3, 40], [41, 90])])
def test_empty_rows_beside_rows_of_several_segments(empty, long, precision):
    P, q, A, lo, up = problem(empty, long, 7)
    n, m = A.shape[1], A.shape[0]
    b = np.random.default_rng(1).standard_normal(n)
    z = np.random.default_rng(2).choice(np.array([-1, 1], dtype=np.int8), size=(3, n))
    kind = qpg.QPG_FP64 if precision == "fp64" else qpg.QPG_MIXED
    out = {}
    for spec in (1, 0):
        print("[case] empty rows", empty, long, precision, "speculate", spec, file=sys.stderr, flush=True)
        with qpg.Solver(sp.triu(P).tocsc(), q, A, lo, up, precision=precision, speculate=spec, scaling_iters=0) as s:
            assert s.spmv_layout(0)["slots"] == m
            i = s.solve()
            pcg = s.pcg(b, eps=1e-9, max_iter=500, precision=qpg.QPG_FP64)
            low = s.pcg(b, eps=1e-4, max_iter=500, precision=kind)
            out[spec] = (i, s.x(), s.y(), s.z(), pcg, low, s.hutchinson(z, 0.3, eps=1e-9, max_iter=500),
                         s.hutchinson_noalloc(z, 0.3, eps=1e-9, max_iter=500), s.settings.rho, s.settings.sigma)
    (i1, x1, y1, z1, p1, l1, h1, hn1, rho, sigma), (i0, x0, y0, z0, p0, l0, h0, hn0, _, _) = out[1], out[0]
    assert i1.status == "solved"
    same = ("status", "iter", "pcg_iter_total", "pcg_iter_max", "rho_updates", "obj_val", "prim_res", "dual_res")
    assert {f: getattr(i1, f) for f in same} == {f: getattr(i0, f) for f in same}
    assert np.array_equal(x1, x0) and np.array_equal(y1, y0) and np.array_equal(z1, z0)
    assert np.array_equal(p1[0], p0[0]) and p1[1:] == p0[1:]
    assert np.array_equal(l1[0], l0[0]) and l1[1:] == l0[1:]
    assert np.array_equal(h1, h0) and np.array_equal(hn1, hn0)
    K = P + sigma * sp.identity(n) + rho * (A.T @ A)
    assert np.max(np.abs(K @ p1[0] - b)) <= 1e-7 * np.max(np.abs(b))
