"""The network's graph kernels on rows at the edges of the batches that their workgroups stage: 256 entries of rows in
one chain, 512 of those in eight (more than 2048 entries). Needs an MI355X. Float32, against the float64 oracle,
tolerance as in test_gpu_graph_pieces.py.
"""
import sys

import numpy as np
import pytest
import scipy.sparse as sp

from oracle import mpnn
from oracle import ruiz as o_ruiz
from paper_1912_04263_amd import qpg
from test_gpu_graph_pieces import matrix

pytestmark = pytest.mark.gpu

LENGTHS = [257, 511, 512, 513, 767, 768, 769, 2048, 2049, 2055, 2056, 2057, 2559, 2560, 2561, 3071, 3072, 3073, 4608, 4609]


@pytest.mark.parametrize("transposed", [False, True])
def test_forward_on_rows_at_batch_edges(transposed):
    print("[case] batches", transposed, file=sys.stderr, flush=True)
    A = matrix(LENGTHS, 5000, 8)
    if transposed:
        A = sp.csr_matrix(A.T)
    m, n = A.shape
    rng = np.random.default_rng(13)
    q, lo, up = rng.standard_normal(n), -rng.random(m), rng.random(m)
    P = sp.identity(n, format="csc")
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
