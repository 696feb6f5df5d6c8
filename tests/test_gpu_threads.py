"""Handles used from several host threads at once give the bits that they give one after another. Needs an MI355X.

One-workgroup kernels of every level, the general path, probes together and the network, whose kernels share their
LDS limits between threads; each thread has a handle of its own, on the default stream.
"""
import sys
import threading

import numpy as np
import pytest

from paper_1912_04263_amd import problems as pr
from paper_1912_04263_amd import qpg

pytestmark = pytest.mark.gpu

PROBLEMS = [
    ("control", lambda: pr.control_qp(8, 3, 20, 0.3, 1), "fp64"),
    ("random", lambda: pr.make("random_c0"), "mixed"),
    ("portfolio", lambda: pr.make("portfolio_small"), "mixed"),
    ("svm", lambda: pr.make("svm_small"), "fp64"),
    ("wide", lambda: pr.lasso_qp(2_000, 20_000, 0.06, 3), "mixed"),
    ("windows", lambda: pr.make("random2_small"), "fp64"),
]


def work(p, precision):
    z = np.random.default_rng(2).choice(np.array([-1, 1], dtype=np.int8), size=(5, p.n))
    with qpg.Solver.from_qp(p, precision=precision) as s:
        i = s.solve()
        net = qpg.Net(qpg.load_weights())
        out = [s.x(), s.y(), s.z(), s.hutchinson(z, 0.3, eps=1e-7, max_iter=50), net.forward(s, 0.3)]
        net.close()
    return (i.status, i.iter, i.pcg_iter_total), out


def test_threads():
    problems = [(name, make(), precision) for name, make, precision in PROBLEMS]
    print("[case] threads", file=sys.stderr, flush=True)
    got, errors = {}, []

    def run(name, p, precision, k):
        try:
            got[name, k] = work(p, precision)
        except Exception as e:  # reported by the main thread
            errors.append((name, e))

    for k in range(3):
        th = [threading.Thread(target=run, args=(*x, k)) for x in problems]
        for t in th:
            t.start()
        for t in th:
            t.join()
    assert not errors
    for name, p, precision in problems:
        ref = work(p, precision)
        for k in range(3):
            assert got[name, k][0] == ref[0], name
            for a, b in zip(got[name, k][1], ref[1]):
                assert np.array_equal(a, b), name
