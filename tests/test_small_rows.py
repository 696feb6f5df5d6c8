"""When the one-workgroup kernels may take a segment of Ā for a row (segments_are_rows), on the CPU.

An empty row has no segment and a row of more entries than a segment holds has several, so the counts of
segments and rows also agree where these cancel; then a segment's number is not its row's.
"""
import os
import subprocess

import numpy as np
import pytest
import scipy.sparse as sp

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1912_04263_amd", "csrc")


def matrix(lengths, n, seed):
    rng = np.random.default_rng(seed)
    cols = [np.sort(rng.choice(n, k, replace=False)) for k in lengths]
    indptr = np.concatenate([[0], np.cumsum(lengths)])
    return sp.csr_matrix((rng.standard_normal(indptr[-1]), np.concatenate(cols).astype(np.int32), indptr),
                         shape=(len(lengths), n))


def cancelling(m, empty, long):
    """m rows of 4 entries, but none in the rows `empty` and 30 in the rows `long`."""
    k = np.full(m, 4)
    k[list(empty)] = 0
    k[list(long)] = 30
    return k


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    d = tmp_path_factory.mktemp("rows")
    exe = str(d / "rows_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, os.path.join(ROOT, "tests", "native", "rows_check.cpp"),
                    os.path.join(CSRC, "tiles.cpp"), os.path.join(CSRC, "host_parallel.cpp"), "-lpthread", "-o", exe],
                   check=True)

    def run(M):
        pre = str(d / "m")
        M.indptr.astype(np.int32).tofile(pre + "_ptr.bin")
        M.indices.astype(np.int32).tofile(pre + "_col.bin")
        f = subprocess.run([exe, pre, str(M.shape[1])], check=True, capture_output=True, text=True).stdout.split()
        return {f[i]: int(f[i + 1]) for i in range(0, len(f), 2)}

    return run


@pytest.mark.parametrize("empty,long", [([10], [60]), ([60], [10]), ([0], [99]), ([99], [0]), ([10], [11]),
                                        ([3, 40], [41, 90]), ([0, 1, 2], [97, 98, 99])])
def test_empty_rows_beside_rows_of_several_segments(check, empty, long):
    out = check(matrix(cancelling(100, empty, long), 60, 1))
    assert out["segments"] == out["rows"] == 100
    assert out["flag"] == out["entries"] == 0


@pytest.mark.parametrize("lengths,flag", [([4] * 100, 1), ([16] * 100, 1), ([1], 1), ([30] * 100, 0),
                                          ([4] * 99 + [0], 0), ([0], 0)])
def test_rows_of_one_segment_and_others(check, lengths, flag):
    out = check(matrix(lengths, 60, 2))
    assert out["flag"] == out["entries"] == flag


def test_random_rows(check):
    cancel = 0
    for seed in range(60):
        M = matrix(np.random.default_rng(seed).poisson(7.0, 400), 200, seed)
        out = check(M)
        assert out["flag"] == out["entries"], seed
        cancel += out["segments"] == out["rows"] and not out["flag"]
    assert cancel > 0


def test_level_of_no_handle():
    from paper_1912_04263_amd import qpg
    assert qpg.lib().qpg_small_level(None, qpg.QPG_FP64, None) == qpg.QPG_ERR_ARG
