"""The streaming pair-density kernel at K = 96 and with a c64 result (the gradient's M_c where n_v^2 is not a multiple of
8), on halves in fragment order and in row order, at row counts around its 32-row sub-tiles and 128-row blocks: equal
bits between the layouts and the tiled kernels, and the oracle's rows and gradient."""
import os

import numpy as np
import pytest
import torch

import oracle as O
from synth import dense_kmesh, make_problem, random_block
from tolerances import GRAD_TOL, KERNEL_TOL, diag_times, kernel_err

pytestmark = pytest.mark.gpu


def T(a, dt=torch.complex128):
    return torch.as_tensor(np.ascontiguousarray(a)).to(torch.device("cuda:0"), dt)


class env:
    def __init__(self, **kw):
        self.kw = kw

    def __enter__(self):
        self.old = {k: os.environ.get(k) for k in self.kw}
        os.environ.update(self.kw)

    def __exit__(self, *a):
        for k, v in self.old.items():
            if v is None:
                del os.environ[k]
            else:
                os.environ[k] = v


# dense mesh, n_ao, nv, nc, n_aux, q per batch: rows (q, band) 1 x nc, 31..33, 127..129 and above 256
CASES = [((3, 2, 2), 96, 3, 5, 352, 1), ((4, 3, 2), 96, 3, 11, 352, 3), ((5, 5, 2), 96, 2, 3, 384, 43),
         ((5, 5, 2), 64, 3, 7, 160, 50), ((3, 3, 2), 128, 5, 6, 288, 18), ((5, 3, 2), 96, 4, 9, 1056, 30)]


@pytest.mark.parametrize("dense,no,nv,nc,na,q", CASES)
def test_stream_depths(dense, no, nv, nc, na, q):
    from paper_2607_05853_amd import bse as B
    p = make_problem(dict(cfg_id=78, coarse=(2, 2, 2), dense=dense, n_ao=no, nv=nv, nc=nc, n_aux=na), 0, "G2")
    W = O.interpolate_W_matmul(p.W_R, p.R, p.w_R, dense_kmesh(p.nk))
    X, Yb = random_block(p.N, 2, seed=5), random_block(p.N, 2, seed=6)
    out = []
    for frag in ("1", "0"):
        for stream in ("1", "0"):
            with env(BSE_FRAG_HALVES=frag, BSE_STREAM_PD=stream, BSE_QBATCH=str(q)):
                plan = B.plan_from_problem(p, T(W), prec="bf16x3", max_nb=2, conduction="mc")
                assert plan.frag == (frag == "1")
                Y = plan.apply(T(X)).cpu().numpy()
                g = plan.apply_adjoint(T(Yb), T(X), want_WR=False, want_Wq=True)["W_q"].cpu().numpy()
                plan.close()
                out.append((Y, g))
    assert all(np.array_equal(out[0][0], o[0]) and np.array_equal(out[0][1], o[1]) for o in out[1:])
    Y, g = out[0]
    rows, nt = [0, p.Nk - 1], nv * nc
    ref = O.apply_H_rows_allpairs(p, W, X, rows)
    e = kernel_err(np.concatenate([Y[k * nt:(k + 1) * nt] for k in rows]), ref, diag_times(p, X, rows))
    r = O.grad_Wq_at(p, Yb, X, [1])[0]
    d = np.abs(g[1] - r).max() / np.abs(r).max()
    print("[stream K %d, %d and %d rows] apply %.1e gradient %.1e" % (no, q * nv, q * nc, e, d), flush=True)
    assert e < KERNEL_TOL["bf16x3"] and d < GRAD_TOL["bf16x3"]
