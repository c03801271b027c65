"""BF16x3 plans whose N_ao or N_aux are not multiples of 16 store a zero-padded problem: apply, gradient, spectrum
VJP, coupling block and start vectors come back in the sizes given.  Against the oracle, with the BF16x3 bounds."""
import numpy as np
import pytest
import torch

import oracle as O
from synth import dense_kmesh, make_problem, polarisations, random_block
from tolerances import GRAD_TOL, KERNEL_TOL, diag_times, kernel_err

pytestmark = pytest.mark.gpu


def T(a, dt=torch.complex128):
    return torch.as_tensor(np.ascontiguousarray(a)).to(torch.device("cuda:0"), dt)


def rel(a, b):
    return np.abs(a - b).max() / np.abs(b).max()


SIZES = [(15, 17), (16, 33), (33, 48), (17, 31), (97, 40), (20, 241)]


@pytest.mark.parametrize("no,na", SIZES)
@pytest.mark.parametrize("conduction", ["mc", "u"])
def test_apply_and_gradient(no, na, conduction):
    from paper_2607_05853_amd import bse as B
    p = make_problem(dict(cfg_id=72, coarse=(3, 2, 2), dense=(3, 2, 2), n_ao=no, nv=2, nc=3, n_aux=na), 1, "G2")
    W = O.interpolate_W_matmul(p.W_R, p.R, p.w_R, dense_kmesh(p.nk))
    X, Yb = random_block(p.N, 3, seed=2), random_block(p.N, 3, seed=4)
    plan = B.plan_from_problem(p, T(W), prec="bf16x3", max_nb=3, conduction=conduction)
    plan.set_R(p.R, p.w_R)
    H = O.build_H(p, W)
    err = kernel_err(plan.apply(T(X)).cpu().numpy(), H @ X, diag_times(p, X))
    g = plan.apply_adjoint(T(Yb), T(X), want_Wq=True)
    only = plan.apply_adjoint(T(Yb), T(X))
    plan.close()
    ge, gq = O.grad_apply(p, W, Yb, X)
    gR = O.grad_WR_from_Wq(gq, p.R, p.w_R, dense_kmesh(p.nk))
    e = [err / KERNEL_TOL["bf16x3"], rel(g["W_q"].cpu().numpy(), gq) / GRAD_TOL["bf16x3"],
         rel(g["W_R"].cpu().numpy(), gR) / GRAD_TOL["bf16x3"], rel(g["eps"].cpu().numpy(), ge) / 1e-12]
    print("[rounded %d %d %s] of the bounds: %s" % (no, na, conduction, ["%.2f" % x for x in e]), flush=True)
    assert max(e) < 1
    assert torch.equal(only["W_R"], g["W_R"])


def test_two_centre_and_coupling():
    from paper_2607_05853_amd import bse as B
    p = make_problem(dict(cfg_id=73, coarse=(2, 2, 2), dense=(2, 2, 3), n_ao=10, nv=2, nc=3, n_aux=22), 0, "G2",
                     two_centre=True)
    W = O.interpolate_W_matmul(p.W_R, p.R, p.w_R, dense_kmesh(p.nk))
    X = random_block(p.N, 2, seed=2)
    plan = B.plan_from_problem(p, T(W), prec="bf16x3", max_nb=2)
    H, Bm = O.build_H(p, W), O.build_B(p, W)
    e = kernel_err(plan.apply(T(X)).cpu().numpy(), H @ X, diag_times(p, X))
    b = rel(plan.apply_coupling(T(X)).cpu().numpy(), Bm @ X)
    plan.close()
    print("[rounded two-centre] A %.1e B %.1e" % (e, b), flush=True)
    assert max(e, b) < KERNEL_TOL["bf16x3"]


def test_spectrum_gradient_and_density_start():
    from paper_2607_05853_amd import bse as B
    p = make_problem(dict(cfg_id=74, coarse=(2, 2, 2), dense=(3, 2, 2), n_ao=10, nv=2, nc=2, n_aux=18), 0, "G2")
    W = O.interpolate_W_matmul(p.W_R, p.R, p.w_R, dense_kmesh(p.nk))
    om = np.linspace(2.0, 6.0, 5)
    out = {}
    for prec in ("f64", "bf16x3"):
        plan = B.plan_from_problem(p, T(W), prec=prec, max_nb=2)
        plan.set_R(p.R, p.w_R)
        P = plan.velocity_start(T(p.vel), T(p.eps_ks, torch.float64), polarisations(2))
        h = plan.haydock(P, 20, om, 0.1, keep_basis=True)
        g = plan.haydock_vjp(h, om, 0.1, np.ones((2, 5)), want_Wq=True)
        D = plan.density_start(T(p.psi))
        out[prec] = [h["S"]] + [x.cpu().numpy() for x in (g["W_q"], g["W_R"], g["eps"], D)]
        plan.close()
    d = [rel(a, b) for a, b in zip(out["bf16x3"], out["f64"])]
    print("[rounded spectrum] %s" % ["%.1e" % x for x in d], flush=True)
    assert d[0] < 1e-5 and max(d[1:4]) < GRAD_TOL["bf16x3"]
    assert d[4] < 1e-12 or np.abs(out["f64"][4]).max() < 1e-12   # zero for orthonormal bands at Q = 0


@pytest.mark.parametrize("nc,na,dense", [(4, 24, (2, 2, 2)), (7, 136, (3, 3, 2)), (9, 128, (4, 2, 3)), (12, 40, (3, 3, 3))])
def test_paired_gradient(nc, na, dense):
    # n_v = 4: both Z products from one pass over M_c, at fewer than 64, 81 and 144 rows (c'c), a ragged last column
    # tile, no q, few q and all q but one with a partner -q
    from paper_2607_05853_amd import bse as B
    p = make_problem(dict(cfg_id=75, coarse=(2, 2, 2), dense=dense, n_ao=2 * nc, nv=4, nc=nc, n_aux=na), 1, "G2")
    W = O.interpolate_W_matmul(p.W_R, p.R, p.w_R, dense_kmesh(p.nk))
    X, Yb = random_block(p.N, 2, seed=2), random_block(p.N, 2, seed=4)
    plan = B.plan_from_problem(p, T(W), prec="bf16x3", max_nb=2)
    g = plan.apply_adjoint(T(Yb), T(X), want_WR=False, want_Wq=True)
    plan.close()
    qs = sorted({0, 1, p.Nk // 2, p.Nk - 1})
    ref = np.stack([O.grad_Wq_at(p, Yb, X, [q])[0] for q in qs])
    e = rel(g["W_q"].cpu().numpy()[qs], ref)
    print("[paired gradient nc %d na %d %s] %.1e" % (nc, na, dense, e), flush=True)
    assert e < GRAD_TOL["bf16x3"]
