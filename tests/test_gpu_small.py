"""The one-workgroup kernels of small problems against the general path. Needs an MI355X.

With speculate = 1 a problem whose vectors, slots and work lists fit in one workgroup's LDS is solved
by kernels that run the ADMM iterations between two host reads in one launch; with speculate = 0 every
pass is a kernel of its own. Both add the same numbers in the same order, so the iterates, the counts
and the residuals must agree bitwise. The sizes lie at the edges of the 64-lane and 256-thread groups,
on both sides of where the ADMM vectors and the matrices fit in LDS, and beyond where the kernels are
used; the settings end solves in each of the ways that hand an iteration back to the host.
"""
import dataclasses
import sys

import numpy as np
import pytest

from paper_1912_04263_amd import problems as pr
from paper_1912_04263_amd import qpg

pytestmark = pytest.mark.gpu


def no_rows(p):
    return dataclasses.replace(p, A=p.A[:0], l=p.l[:0], u=p.u[:0])


CASES = {
    "one variable": (lambda: pr.random_qp(1, 1, 1.0, 1.0, 1), {}),
    "no constraints": (lambda: no_rows(pr.random_qp(30, 4, 0.3, 0.3, 2)), {}),
    "64 x 255": (lambda: pr.random_qp(64, 255, 0.2, 0.2, 3), {}),
    "65 x 257": (lambda: pr.random_qp(65, 257, 0.2, 0.2, 4), {}),
    "256 x 512": (lambda: pr.random_qp(256, 512, 0.03, 0.03, 5), {}),
    "rows of several segments": (lambda: pr.make("random_c0"), {}),
    "control": (lambda: pr.control_qp(8, 3, 20, 0.3, 1), {}),
    "vectors in memory": (lambda: pr.make("portfolio_small"), {}),
    "mixed small, fp64 general": (lambda: pr.make("lasso_small"), {}),
    "beyond": (lambda: pr.make("svm_small"), {}),
    "primal infeasible": (lambda: pr.primal_infeasible_qp(60, 40, 0.3, 3), {}),
    "dual infeasible": (lambda: pr.dual_infeasible_qp(60, 80, 0.3, 3), {}),
    "capped PCG": (lambda: pr.random_qp(200, 400, 0.15, 0.15, 2),
                   dict(pcg_max_iter=3, pcg_eps_fixed=1e-9, max_iter=300)),
    "checks every 7": (lambda: pr.random_qp(100, 200, 0.15, 0.15, 2), dict(check_every=7)),
    "checks every 300": (lambda: pr.random_qp(100, 200, 0.15, 0.15, 2), dict(check_every=300)),
    "ends between checks": (lambda: pr.random_qp(100, 200, 0.15, 0.15, 2), dict(max_iter=13)),
    "tight": (lambda: pr.make("equality_small"), dict(eps_abs=1e-7, eps_rel=1e-7, max_iter=2000)),
    "absolute PCG test": (lambda: pr.random_qp(100, 200, 0.15, 0.15, 2), dict(pcg_rel_test=0)),
    "fixed rho": (lambda: pr.random_qp(100, 200, 0.15, 0.15, 6), dict(rho_update_every=0)),
}


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("name", sorted(CASES))
def test_one_workgroup_kernels_equal_the_general_path(name, precision):
    make, settings = CASES[name]
    p = make()
    out = {}
    for spec in (1, 0):
        print("[case]", name, precision, "speculate", spec, "n", p.n, "m", p.m, file=sys.stderr, flush=True)
        with qpg.Solver.from_qp(p, precision=precision, speculate=spec, **settings) as s:
            i = s.solve()
            b = np.random.default_rng(0).standard_normal(p.n)
            k = qpg.QPG_MIXED if precision == "mixed" else qpg.QPG_FP64
            pcg = s.pcg(b, eps=1e-5 if precision == "mixed" else 1e-9, max_iter=300, precision=k)
            out[spec] = (i, s.x(), s.y(), s.z(), pcg)
    (i1, x1, y1, z1, p1), (i0, x0, y0, z0, p0) = out[1], out[0]
    same = ("status", "iter", "pcg_iter_total", "pcg_iter_max", "rho_updates", "obj_val", "prim_res", "dual_res",
            "rho_final", "fallback_events", "infeas_checks")
    assert {f: getattr(i1, f) for f in same} == {f: getattr(i0, f) for f in same}
    assert np.array_equal(x1, x0) and np.array_equal(y1, y0) and np.array_equal(z1, z0)
    assert np.array_equal(p1[0], p0[0]) and p1[1:] == p0[1:]
