"""Device memory of a handle. Needs an MI355X."""
import ctypes as C
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


def free_bytes():
    L = qpg.lib()  # the HIP runtime that it is linked to
    free, total = C.c_size_t(), C.c_size_t()
    assert L.hipDeviceSynchronize() == 0 and L.hipMemGetInfo(C.byref(free), C.byref(total)) == 0
    return free.value


def test_large_vectors_of_several_probes_are_freed():
    """Four solves at once take 32·(4n + m + 2·(segments of B)) = 112 MB here. One probe alone builds the graph and
    needs none of them; after two, as much memory is free as before them (16 MB allowed to the runtime itself)."""
    n = 500_000
    d = np.linspace(1.0, 2.0, n)
    z = np.random.default_rng(4).choice(np.array([-1, 1], dtype=np.int8), size=(3, n))
    print("[case] memory of several probes, large", file=sys.stderr, flush=True)
    with qpg.Solver(sp.diags(d).tocsc(), np.zeros(n), sp.diags(d[::-1]).tocsc(), -np.ones(n), np.ones(n)) as s:
        assert s.small_level() == 0 and 32 * (5 * n + 2 * s.spmv_layout(1)["slots"]) >= 112 * 10**6
        s.hutchinson(z[:1], 0.3)
        before = free_bytes()
        got = [s.hutchinson(z, 0.3) for _ in range(2)]
        after = free_bytes()
        ref = s.hutchinson_noalloc(z, 0.3)
    assert abs(before - after) <= 16 * 2**20
    assert np.array_equal(got[0], ref) and np.array_equal(got[1], ref)


def test_small_vectors_of_several_probes_stay():
    z = np.random.default_rng(5).choice(np.array([-1, 1], dtype=np.int8), size=(2, 200))
    print("[case] memory of several probes, small", file=sys.stderr, flush=True)
    with handle(20_000, 200, 50) as s:
        assert s.small_level() == 0
        s.hutchinson(z[:1], 0.3)
        used = s.device_bytes()[1]
        s.hutchinson(z, 0.3)
        more = s.device_bytes()[1] - used
        assert 32 * (4 * 200 + 20_000) < more <= 64 * 2**20
        s.hutchinson(z, 0.3)
        assert s.device_bytes()[1] == used + more
