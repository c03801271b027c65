"""The FP32 direct block at n_v <= 4 on direct-to-LDS 64 x 16 tiles, at the edges of its rule: N_aux at and past the least
number of stages, n_c^2 rows around one and two tiles, n_v^2 columns up to 16, an odd number of k.  Oracle's rows of A X;
bound: the FP32 bound of the kernel part."""
import numpy as np
import pytest
import torch

import oracle as O
from synth import dense_kmesh, make_problem, random_block
from tolerances import KERNEL_TOL, diag_times, kernel_err

pytestmark = pytest.mark.gpu


def T(a, dt=torch.complex128):
    return torch.as_tensor(np.ascontiguousarray(a)).to(torch.device("cuda:0"), dt)


# nv, nc, n_aux: K = 64 is the least, 48 and 72 keep the other tile; 5 stages and more than the four slots at 80, 112
CASES = [(4, 8, 64), (4, 9, 80), (3, 8, 112), (2, 5, 256), (4, 5, 48), (4, 10, 72), (1, 5, 64)]


@pytest.mark.parametrize("nv,nc,na", CASES)
def test_narrow_direct_block(nv, nc, na):
    from paper_2607_05853_amd import bse as B
    p = make_problem(dict(cfg_id=83, coarse=(2, 2, 2), dense=(3, 3, 1), n_ao=2 * nc, nv=nv, nc=nc, n_aux=na), 0, "G2")
    W = O.interpolate_W_matmul(p.W_R, p.R, p.w_R, dense_kmesh(p.nk))
    plan = B.plan_from_problem(p, T(W), prec="f32", max_nb=3)
    X = random_block(p.N, 3, seed=6)
    Y = plan.apply(T(X)).cpu().numpy()
    plan.close()
    rows = [0, 4, p.Nk - 1]
    nt = nv * nc
    ref = O.apply_H_rows_allpairs(p, W, X, rows)
    err = kernel_err(np.concatenate([Y[k * nt:(k + 1) * nt] for k in rows]), ref, diag_times(p, X, rows))
    print("[narrow direct block nv %d nc %d na %d] %.1e" % (nv, nc, na, err), flush=True)
    assert err < KERNEL_TOL["f32"]
