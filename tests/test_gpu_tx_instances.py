"""T.X of c64 blocks: every instance of the restaged kernel on both sides of the lines between them, with equal bits to the
kernel it replaces (BSE_TX2=0), and against the oracle."""
import numpy as np
import pytest
import torch

import oracle as O
from synth import dense_kmesh, make_problem, random_block
from tolerances import KERNEL_TOL, diag_times, kernel_err

pytestmark = pytest.mark.gpu


def T(a, dt=torch.complex128):
    return torch.as_tensor(np.ascontiguousarray(a)).to(torch.device("cuda:0"), dt)


# n_v, n_c, vectors: 510, 525, 1020 and 1035 elements of X (up to 8 tiles); 9, 16 and 18 tiles at up to 64 transitions; 65
# and more with up to 1024 elements and 16 tiles, and beyond; 88 (two blocks per CU) and 90 transitions (one)
CASES = [(3, 5, 34), (3, 5, 35), (3, 17, 20), (5, 9, 23), (3, 15, 17), (7, 9, 25), (5, 9, 41), (5, 13, 15), (5, 13, 16),
         (5, 14, 14), (5, 14, 15), (7, 11, 13), (8, 11, 4), (9, 10, 8), (9, 10, 9)]


@pytest.mark.parametrize("prec", ["f32", "bf16x3"])
@pytest.mark.parametrize("nv,nc,nb", CASES)
def test_tx_instances(monkeypatch, prec, nv, nc, nb):
    from paper_2607_05853_amd import bse as B
    p = make_problem(dict(cfg_id=79, coarse=(2, 2, 1), dense=(3, 2, 1), n_ao=2 * nc, nv=nv, nc=nc, n_aux=16), 0, "G2")
    W = O.interpolate_W_matmul(p.W_R, p.R, p.w_R, dense_kmesh(p.nk))
    plan = B.plan_from_problem(p, T(W), prec=prec, max_nb=nb)
    X = random_block(p.N, nb, seed=5)
    Y = plan.apply(T(X)).cpu().numpy()
    monkeypatch.setenv("BSE_TX2", "0")
    Z = plan.apply(T(X)).cpu().numpy()
    plan.close()
    e = kernel_err(Y, O.build_H(p, W) @ X, diag_times(p, X))
    print("[tx %s %d x %d, %d vectors] %.1e" % (prec, nv, nc, nb, e), flush=True)
    assert e < KERNEL_TOL[prec]
    assert np.array_equal(Y, Z)
