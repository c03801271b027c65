"""The 256 x 128 W-step tile and the 128 x 64 direct-block tile at the edges of their rules, against the tiles they
replace (same accumulation order: equal bits) and the oracle."""
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


# n_aux 272, 384: half-empty last 256 columns (tall tile); 400: more than half (wide tile).  n_c^2 = 81, 100, 144,
# 289 rows against n_v^2 = 4, 25, 36, 49, 64 columns of the direct block; an odd number of k (row tiles cut by M)
CASES = [((3, 3, 3), 6, 10, 272), ((3, 2, 2), 2, 12, 384), ((3, 3, 1), 7, 9, 400), ((2, 2, 2), 5, 17, 32), ((2, 2, 1), 8, 12, 32)]


@pytest.mark.parametrize("dense,nv,nc,na", CASES)
def test_tall_tiles(dense, nv, nc, na):
    from paper_2607_05853_amd import bse as B
    no = 2 * max(nv, nc) + (2 * max(nv, nc)) % 16
    p = make_problem(dict(cfg_id=77, coarse=(2, 2, 2), dense=dense, n_ao=no, nv=nv, nc=nc, n_aux=na), 0, "G2")
    kq = dense_kmesh(p.nk)
    W = O.interpolate_W_matmul(p.W_R, p.R, p.w_R, kq)
    plan = B.plan_from_problem(p, T(W), prec="bf16x3", max_nb=2, conduction="mc")
    X = random_block(p.N, 2, seed=5)
    Y = plan.apply(T(X)).cpu().numpy()
    old = os.environ.get("BSE_WIDE_TILES")
    os.environ["BSE_WIDE_TILES"] = "0"
    try:
        Z = plan.apply(T(X)).cpu().numpy()
    finally:
        if old is None:
            del os.environ["BSE_WIDE_TILES"]
        else:
            os.environ["BSE_WIDE_TILES"] = old
    plan.close()
    rows = [0, p.Nk - 1]
    nt = nv * nc
    ref = O.apply_H_rows_allpairs(p, W, X, rows)
    got = np.concatenate([Y[k * nt:(k + 1) * nt] for k in rows])
    err = kernel_err(got, ref, diag_times(p, X, rows))
    print("[tall tiles %s nv %d nc %d na %d] %.1e, W step identical to the 64 x 128 tile: %s" %
          (dense, nv, nc, na, err, np.array_equal(Y, Z)), flush=True)
    assert err < KERNEL_TOL["bf16x3"]
    assert np.array_equal(Y, Z)
