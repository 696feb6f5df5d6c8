"""Which problems the one-workgroup kernels take, and their ways that other tests leave out, bitwise against the
general path (speculate = 0). Needs an MI355X.

The levels say what is held in LDS: 1 work lists and PCG vectors, 2 the ADMM vectors too, 3 the matrices too, 0
none: the general path. Expected ones follow from 160 KB of LDS and matrices of at most 1.5 MB.
"""
import sys

import numpy as np
import pytest
import scipy.sparse as sp

from paper_1912_04263_amd import problems as pr
from paper_1912_04263_amd import qpg
from test_gpu_hutchinson_multi import PROBLEMS
from test_gpu_small import CASES

pytestmark = pytest.mark.gpu

# levels in FP64 and in FP32, where not (3, 3)
LEVELS = {"256 x 512": (2, 2), "64 x 255": (2, 3), "65 x 257": (2, 3), "absolute PCG test": (2, 3), "beyond": (0, 0),
          "capped PCG": (2, 2), "checks every 300": (2, 3), "checks every 7": (2, 3), "ends between checks": (2, 3),
          "fixed rho": (2, 3), "mixed small, fp64 general": (0, 1), "rows of several segments": (2, 2),
          "tight": (2, 2), "vectors in memory": (0, 1)}


@pytest.mark.parametrize("name", sorted(CASES))
def test_levels(name):
    make, settings = CASES[name]
    with qpg.Solver.from_qp(make(), precision="mixed", **settings) as s:
        print("[case] level", name, s.small_level(qpg.QPG_FP64), s.small_level(qpg.QPG_MIXED), file=sys.stderr, flush=True)
        assert (s.small_level(qpg.QPG_FP64), s.small_level(qpg.QPG_MIXED)) == LEVELS.get(name, (3, 3))


def test_levels_of_other_handles():
    p = pr.make("random_c0")
    with qpg.Solver.from_qp(p, precision="mixed", speculate=0) as s:
        assert s.small_level(qpg.QPG_FP64) == s.small_level(qpg.QPG_MIXED) == 0
    with qpg.Solver.from_qp(p, rho_vector=1) as s:
        assert s.small_level() == 0
        with pytest.raises(qpg.QpgError) as e:
            s.small_level(qpg.QPG_MIXED)
        assert e.value.code == qpg.QPG_ERR_STATE


@pytest.mark.parametrize("name", sorted(PROBLEMS))
def test_problems_of_several_probes_are_beyond_one_workgroup(name):
    with qpg.Solver.from_qp(PROBLEMS[name]()) as s:
        assert s.small_level() == 0


def both(p, precision, level, pcg_eps, pcg_iter, **settings):
    out = {}
    kind = qpg.QPG_MIXED if precision == "mixed" else qpg.QPG_FP64
    for spec in (1, 0):
        print("[case]", p.n, p.m, precision, settings.get("precond"), "speculate", spec, file=sys.stderr, flush=True)
        with qpg.Solver.from_qp(p, precision=precision, speculate=spec, **settings) as s:
            assert s.small_level(kind) == (level if spec else 0)
            i = s.solve()
            b = np.random.default_rng(0).standard_normal(p.n)
            out[spec] = (i, s.x(), s.y(), s.z(), s.pcg(b, eps=pcg_eps, max_iter=pcg_iter, precision=kind))
    (i1, x1, y1, z1, p1), (i0, x0, y0, z0, p0) = out[1], out[0]
    same = ("status", "iter", "pcg_iter_total", "pcg_iter_max", "rho_updates", "obj_val", "prim_res", "dual_res",
            "rho_final", "fallback_events", "infeas_checks", "precond_used", "precond_trials",
            "precond_learned_chosen", "precond_switches")
    assert {f: getattr(i1, f) for f in same} == {f: getattr(i0, f) for f in same}
    for a, b in ((x1, x0), (y1, y0), (z1, z0), (p1[0], p0[0])):
        assert np.array_equal(a, b)
    assert p1[1:] == p0[1:]
    return i1, p1


def tall():
    return pr.random_qp(500, 2000, 0.008, 0.008, 7)


# problem, weights, level, in the precisions where it is that level
WAYS = {
    "matrices in LDS": (lambda: pr.random_qp(40, 80, 0.15, 0.15, 2), "random_h32", 3, ["fp64", "mixed"]),
    "matrices in memory": (lambda: pr.make("random_c0"), "random_h32", 2, ["fp64", "mixed"]),
    "vectors in memory, FP64": (tall, "random_h32", 1, ["fp64"]),
    "vectors in memory, FP32": (lambda: pr.make("portfolio_small"), "portfolio_h32", 1, ["mixed"]),
}
ALL = [(name, precision) for name in sorted(WAYS) for precision in WAYS[name][3]]


@pytest.mark.parametrize("name,precision", ALL)
def test_every_level(name, precision):
    make, _, level, _ = WAYS[name]
    i, _ = both(make(), precision, level, 1e-5 if precision == "mixed" else 1e-9, 300)
    assert i.status == "solved"


@pytest.mark.parametrize("trial", [0, 1])
@pytest.mark.parametrize("name,precision", ALL)
def test_learned_preconditioner(name, precision, trial):
    make, weights, level, _ = WAYS[name]
    i, _ = both(make(), precision, level, 1e-5 if precision == "mixed" else 1e-9, 300, precond="learned",
                precond_weights=qpg.load_weights(weights), precond_trial=trial)
    assert i.rho_updates > 0
    assert i.precond_trials > 0 if trial else i.precond_used == "learned"


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_solves_of_more_steps_than_one_launch_takes(precision):
    """A launch ends after 4096 PCG steps; pcg goes on in a second one, an ADMM iteration in the general path's
    loop. P is a squared second difference of condition ≈ 1e10, whose solves don't end within 6000 steps."""
    n = 400
    D = sp.diags([np.ones(n - 1), -2 * np.ones(n), np.ones(n - 1)], [-1, 0, 1])
    A = sp.csc_matrix((np.full(10, 1e-3), (np.arange(10), np.arange(0, n, n // 10))), shape=(10, n))
    p = pr.QP("difference", sp.triu(sp.csc_matrix(D @ D)).tocsc(), np.ones(n), A, -np.ones(10), np.ones(10), {})
    i, (x, it, rn, broke) = both(p, precision, 3, 1e-300, 5000, pcg_eps_fixed=1e-300, pcg_max_iter=6000, max_iter=2,
                                 scaling_iters=0)
    assert it == 5000 and i.pcg_iter_max == 6000
