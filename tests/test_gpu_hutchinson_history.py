"""A Hutchinson estimate of a few PCG steps costs the same after one of thousands as before it. Needs an MI355X.

Launching as many steps before the first host read as an earlier call took would queue 5000 steps of six kernels,
about 0.1 s at 3 µs per launch, where the easy estimate takes about a millisecond: between the two lies the bound of
five times the time before and 10 ms more.
"""
import statistics
import sys
import time

import numpy as np
import pytest

from paper_1912_04263_amd import problems as pr
from paper_1912_04263_amd import qpg

pytestmark = pytest.mark.gpu


def test_an_easy_estimate_after_a_hard_one():
    p = pr.portfolio_qp(3_000, 30, 0.5, 5)
    z = np.random.default_rng(1).choice(np.array([-1, 1], dtype=np.int8), size=(4, p.n))
    with qpg.Solver.from_qp(p) as s:
        def easy():
            t = time.perf_counter()
            d = s.hutchinson(z, 0.3, eps=0.5)
            return time.perf_counter() - t, d

        easy()
        before = statistics.median(easy()[0] for _ in range(5))
        ref = easy()[1]
        print("[case] hutchinson of 5000 steps", file=sys.stderr, flush=True)
        after = []
        for _ in range(3):
            s.hutchinson(z, 0.3, eps=1e-300, max_iter=5000)
            t, got = easy()
            after.append(t)
        after = min(after)
    print("[case] before %.2f ms, after %.2f ms" % (1e3 * before, 1e3 * after), file=sys.stderr, flush=True)
    assert np.array_equal(got, ref)
    assert after <= 5 * before + 0.01
