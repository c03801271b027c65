"""T.X for band counts whose product is not a multiple of 16, at the edges of the kernel's instances: equal bits to the
kernel it replaces (BSE_TX2=0) up to the FP64 sums over q chunks both share, and the oracle."""
import os

import numpy as np
import pytest
import torch

import oracle as O
from synth import dense_kmesh, make_problem, random_block
from tolerances import KERNEL_TOL, diag_times, kernel_err

pytestmark = pytest.mark.gpu


def T(a, dt=torch.complex128):
    return torch.as_tensor(np.ascontiguousarray(a)).to(torch.device("cuda:0"), dt)


# n_v, n_c, vectors: 1 transition; 15, 17, 31 and 33 around tiles and instances; 63, 65; 90, 95 and 96, the largest
CASES = [(1, 1, 1), (1, 1, 16), (3, 5, 17), (1, 17, 3), (1, 31, 16), (3, 11, 15), (7, 9, 16), (5, 13, 9), (9, 10, 2),
         (8, 12, 1), (5, 19, 6)]


@pytest.mark.parametrize("prec", ["f32", "bf16x3"])
@pytest.mark.parametrize("nv,nc,nb", CASES)
def test_tx_restaged(prec, nv, nc, nb):
    from paper_2607_05853_amd import bse as B
    p = make_problem(dict(cfg_id=79, coarse=(2, 2, 1), dense=(3, 2, 1), n_ao=2 * nc, nv=nv, nc=nc, n_aux=16), 0, "G2")
    W = O.interpolate_W_matmul(p.W_R, p.R, p.w_R, dense_kmesh(p.nk))
    plan = B.plan_from_problem(p, T(W), prec=prec, max_nb=nb)
    X = random_block(p.N, nb, seed=5)
    Y = plan.apply(T(X)).cpu().numpy()
    old = os.environ.get("BSE_TX2")
    os.environ["BSE_TX2"] = "0"
    try:
        Z = plan.apply(T(X)).cpu().numpy()
    finally:
        if old is None:
            del os.environ["BSE_TX2"]
        else:
            os.environ["BSE_TX2"] = old
    plan.close()
    H = O.build_H(p, W)
    e = kernel_err(Y, H @ X, diag_times(p, X))
    print("[tx %s %d x %d, %d vectors] %.1e, equal %s" % (prec, nv, nc, nb, e, np.array_equal(Y, Z)), flush=True)
    assert e < KERNEL_TOL[prec]
    if (nv * nc) % 16 and ((nv * nc + 15) // 16) * ((2 * nb + 15) // 16) <= 32:
        assert np.array_equal(Y, Z)
