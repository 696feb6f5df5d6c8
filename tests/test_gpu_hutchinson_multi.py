"""Hutchinson estimates with several probes solved together, against one after another. Needs an MI355X.

qpg_hutchinson solves the probes in groups of four that share each read of the matrices;
qpg_hutchinson_noalloc solves them one by one. Every solve adds the same numbers in the same order, so
the estimates agree bitwise: with whole and partial groups, solves of one group that end at different
steps, at the cap, and at once.
"""
import sys

import numpy as np
import pytest

from paper_1912_04263_amd import problems as pr
from paper_1912_04263_amd import qpg

pytestmark = pytest.mark.gpu

PROBLEMS = {
    "svm": lambda: pr.make("svm_small"),
    "portfolio": lambda: pr.portfolio_qp(3_000, 30, 0.5, 5),
    "rows over many windows": lambda: pr.make("random2_small"),
    "wide windows": lambda: pr.random_qp(40_000, 20_000, 1e-4, 2e-3, 6),
}


@pytest.mark.parametrize("nprobes", [1, 2, 4, 5, 9])
@pytest.mark.parametrize("name", sorted(PROBLEMS))
def test_probes_together_equal_probes_one_by_one(name, nprobes):
    print("[case] hutchinson", name, nprobes, file=sys.stderr, flush=True)
    p = PROBLEMS[name]()
    z = np.random.default_rng(nprobes).choice(np.array([-1, 1], dtype=np.int8), size=(nprobes, p.n))
    with qpg.Solver.from_qp(p) as s:
        for rho, eps, cap in ((0.3, 1e-9, 2000), (5.0, 1e-9, 7), (0.3, 2.0, 2000)):
            got = s.hutchinson(z, rho, eps=eps, max_iter=cap)
            assert np.array_equal(got, s.hutchinson_noalloc(z, rho, eps=eps, max_iter=cap)), (rho, eps, cap)
