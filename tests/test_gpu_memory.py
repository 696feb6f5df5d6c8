"""Device memory of a handle. Needs an MI355X."""
import sys

import numpy as np
import pytest
import scipy.sparse as sp

from paper_1912_04263_amd import qpg

pytestmark = pytest.mark.gpu


def handle(m, n, per_row, **settings):
    rng = np.random.default_rng(3)
    col = np.sort(rng.permuted(np.broadcast_to(np.arange(n), (m, n)), axis=1)[:, :per_row], axis=1)
    A = sp.csr_matrix((rng.standard_normal(m * per_row), col.ravel(), np.arange(0, m * per_row + 1, per_row)),
                      shape=(m, n))
    return qpg.Solver(sp.identity(n, format="csc"), np.zeros(n), A.tocsc(), -np.ones(m), np.ones(m), **settings)


@pytest.mark.parametrize("precision,each", [("fp64", 44), ("mixed", 60)])
def test_what_setup_needs_only_for_itself_is_given_back(precision, each):
    """Two problems of the same rows and columns: the difference is what an entry of A keeps: column (4 bytes) and
    value (8), value (8) and 16-bit column (2) as streamed, all for A and for [P | A'] (FP32 copies: 4 + 4 more
    each). Padding, slots and chunks of the segments (over 30 entries on average) may add 5 bytes; the indices that
    place the values, needed during setup only, would add 8."""
    m, n = 20_000, 200
    used = {}
    for per_row in (50, 150):
        print("[case] memory", precision, per_row, file=sys.stderr, flush=True)
        with handle(m, n, per_row, precision=precision) as s:
            held, used[per_row] = s.device_bytes()
            assert s.spmv_layout(0)["plain_positions"] == s.spmv_layout(1)["plain_positions"] == 0
            # the rest of the last block, and of the blocks before it
            assert used[per_row] <= held <= used[per_row] + (64 + 16 + 4 + 1) * 2**20
            print("[case] held", held, "used", used[per_row], file=sys.stderr, flush=True)
    slope = (used[150] - used[50]) / (100 * m)
    print("[case] bytes per entry", slope, file=sys.stderr, flush=True)
    assert each <= slope <= each + 5
