"""The network's graph kernels on rows at the edges of their work split. Needs an MI355X.

A wavefront takes a pack of at most 16 rows of at most 16 entries or of 8 rows of at most 256; longer rows
have workgroups of their own, which add them in one chain up to 2048 entries and in 8 chains above, in
batches of 256 and 512 entries; edge weights go by pieces of 512. The rows of Ā (and, transposed, of Āᵀ)
have lengths on both sides of each of these limits. Float32 layers, against the float64 oracle; tolerance as
for the other float32 comparisons of the network (1e-4 of the largest value): the weights of a row sum
to 1, so a sum of up to 9000 float32 products is within 9000·2⁻²⁴ ≈ 5.4e-4 of its largest term in the
worst case and within √9000·2⁻²⁴ ≈ 6e-6 typically.
"""
import sys

import numpy as np
import pytest
import scipy.sparse as sp

from oracle import mpnn
from oracle import ruiz as o_ruiz
from paper_1912_04263_amd import qpg

pytestmark = pytest.mark.gpu

LENGTHS = [1, 2, 15, 16, 17, 3, 1, 63, 64, 65, 511, 512, 513, 1, 1024, 1025, 2000] + [1] * 33 + [16] * 20 + [0, 5, 0]

LONG = [255, 256, 257, 1, 2047, 2048, 2049, 4096, 9000, 1, 0, 3000] + [100] * 50 + [17] * 9 + [1] * 30 + [5000]


def matrix(lengths, n, seed):
    rng = np.random.default_rng(seed)
    rows = [np.sort(rng.choice(n, k, replace=False)) for k in lengths]
    indptr = np.concatenate([[0], np.cumsum(lengths)])
    vals = rng.standard_normal(indptr[-1])
    return sp.csr_matrix((vals, np.concatenate(rows).astype(np.int32), indptr), shape=(len(lengths), n))


@pytest.mark.parametrize("lengths", ["short", "long"])
@pytest.mark.parametrize("transposed", [False, True])
def test_forward_and_gradient_on_rows_of_every_length(transposed, lengths):
    print("[case] pieces", lengths, "transposed" if transposed else "as is", file=sys.stderr, flush=True)
    A = matrix(LENGTHS, 2000, 11) if lengths == "short" else matrix(LONG, 10_000, 3)
    if transposed:
        A = sp.csr_matrix(A.T)
    m, n = A.shape
    rng = np.random.default_rng(12)
    P = sp.identity(n, format="csc")
    q = rng.standard_normal(n)
    lo, up = -rng.random(m), rng.random(m)
    rho, sigma = 0.7, 1e-6
    D, E, c, Pb, qb, Ab, _ = o_ruiz.ruiz(sp.csr_matrix(P), q, A, 10)
    fv, fc, dP, colsq = mpnn.features(Pb, Ab, sigma, E * lo, E * up)
    Ahat, Acheck = mpnn.graph(Ab)
    phi, _ = mpnn.head_inputs(dP, colsq, sigma, rho)
    theta = (mpnn.init_params(3) + 0.3 * rng.standard_normal(mpnn.nparams())).astype(np.float32)
    target = np.log(1.0 + rng.random(n)).astype(np.float32)
    L_o, G_o, g_o = mpnn.loss_grad(theta.astype(np.float64), fv, fc, Ahat, Acheck, phi, target.astype(np.float64))
    with qpg.Solver(P, q, A, lo, up) as s:
        net = qpg.Net(theta, bf16=False)
        g = net.forward(s, rho)
        L, G = net.loss_grad(s, rho, target)
        net.close()
    assert np.max(np.abs(g - g_o)) <= 1e-4 * np.max(np.abs(g_o))
    assert abs(L - L_o) <= 1e-4 * abs(L_o)
    assert np.max(np.abs(G - G_o)) <= 1e-4 * np.max(np.abs(G_o))
