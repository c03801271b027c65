"""BF16x3 plans store N_ao and N_aux rounded up; everything a caller sees goes by the sizes as given."""
import numpy as np
import pytest
import torch

import oracle as O
from synth import dense_kmesh, make_problem, polarisations, random_block

pytestmark = pytest.mark.gpu
ESHAPE = 2


def T(a, dt=torch.complex128):
    return torch.as_tensor(np.ascontiguousarray(a)).to(torch.device("cuda:0"), dt)


def crystal(**kw):
    return make_problem(dict(dict(cfg_id=76, coarse=(2, 2, 2), dense=(3, 2, 2), n_ao=10, nv=2, nc=3, n_aux=20), **kw),
                        0, "G2")


def plan_of(B, p, prec, nb=2, **kw):
    W = O.interpolate_W_matmul(p.W_R, p.R, p.w_R, dense_kmesh(p.nk))
    return B.plan_from_problem(p, T(W), prec=prec, max_nb=nb, **kw)


def start(plan, p):
    return plan.velocity_start(T(p.vel), T(p.eps_ks, torch.float64), polarisations(2))


def test_offset_average_over_precisions():
    # one ragged crystal, an FP64 and a BF16x3 plan: the average of their two spectra (FP64 sums of two terms)
    from paper_2607_05853_amd import bse as B
    p = crystal()
    om = np.linspace(2.0, 6.0, 11)
    plans = [plan_of(B, p, prec) for prec in ("f64", "bf16x3")]
    Ps = [start(q, p) for q in plans]
    S = [q.haydock(P, 12, om, 0.1)["S"] for q, P in zip(plans, Ps)]
    out = B.offset_spectrum(plans, Ps, [0.25, 0.75], 12, om, 0.1)["S"]
    for q in plans:
        q.close()
    assert np.abs(out - (0.25 * S[0] + 0.75 * S[1])).max() < 1e-12 * np.abs(out).max()


@pytest.mark.parametrize("other", [dict(n_aux=17), dict(n_ao=12)])
def test_offset_average_refuses_other_sizes(other):
    # 17 and 20 auxiliary functions are both stored as 32, 10 and 12 orbitals as 16: still different problems
    from paper_2607_05853_amd import bse as B
    ps = [crystal(), crystal(**other)]
    plans = [plan_of(B, p, "bf16x3") for p in ps]
    Ps = [start(q, p) for q, p in zip(plans, ps)]
    with pytest.raises(B.BSEError) as e:
        B.offset_spectrum(plans, Ps, [0.5, 0.5], 4, np.linspace(2.0, 6.0, 3), 0.1)
    for q in plans:
        q.close()
    assert e.value.status == ESHAPE


@pytest.mark.parametrize("conduction", ["mc", "u"])
@pytest.mark.parametrize("two_centre", [False, True])
def test_batch_buffers_stay_below_the_limit(monkeypatch, conduction, two_centre):
    # 17 auxiliary functions stored as 32: the q-batch buffers are those of the stored sizes, and they keep the limit
    from paper_2607_05853_amd import bse as B
    if two_centre and conduction == "u":
        pytest.skip("two-centre plans form M_cc'")
    p = make_problem(dict(cfg_id=76, coarse=(2, 2, 2), dense=(4, 4, 4), n_ao=10, nv=2, nc=3, n_aux=17), 0, "G2",
                     two_centre=two_centre)
    kw = dict(conduction=None if two_centre else conduction)
    monkeypatch.setenv("BSE_QBATCH", "1")
    one = plan_of(B, p, "bf16x3", **kw)
    monkeypatch.delenv("BSE_QBATCH")
    monkeypatch.setenv("BSE_WORKSPACE_GB", "%.9f" % (4 / 1024))
    plan = plan_of(B, p, "bf16x3", **kw)
    held = plan.bytes - one.bytes       # all but one q of the batch
    one.close(), plan.close()
    print("[batch buffers %s two-centre %s] %.2f MB" % (conduction, two_centre, held / 2 ** 20), flush=True)
    assert held < 4 * 2 ** 20


def test_plan_that_fits_only_in_the_given_sizes(monkeypatch):
    # N_ao 97 stored as 128: about 2.5 GB while the plan is made, 1.7 GB in the given sizes, with 2.25 GB free
    from paper_2607_05853_amd import bse as B
    p = make_problem(dict(cfg_id=76, coarse=(2, 2, 2), dense=(6, 6, 6), n_ao=97, nv=4, nc=6, n_aux=250), 0, "G2")
    t = lambda a, dt=torch.complex128: T(a, dt)
    Wq = B.interpolate_W(T(p.W_R), p.R, p.w_R, dense_kmesh(p.nk))
    args = (p.nk, p.n_ao, p.nv, p.nc, p.n_aux, t(p.eps_qp, torch.float64), t(p.psi), t(p.C), t(p.Vbar), Wq)
    X = T(random_block(p.N, 2, seed=1))
    Y = torch.empty_like(X)
    monkeypatch.setenv("BSE_WORKSPACE_GB", "0.1")
    plan = B.Plan(*args, prec="bf16x3", max_nb=2)
    ref, rounded = plan.apply(X).clone(), plan.bytes
    plan.close()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    left = int(2.25e9)
    fill = [torch.empty(torch.cuda.mem_get_info()[0] - left - (1 << 30), dtype=torch.uint8, device="cuda:0")]
    while torch.cuda.mem_get_info()[0] > left:
        fill.append(torch.empty(32 << 20, dtype=torch.uint8, device="cuda:0"))
    plan = B.Plan(*args, prec="bf16x3", max_nb=2)
    given = plan.bytes
    print("[given sizes] %.2f GB against %.2f rounded" % (given / 1e9, rounded / 1e9), flush=True)
    plan.apply(X, out=Y)
    torch.cuda.synchronize()
    plan.close()
    del fill
    torch.cuda.empty_cache()
    assert given < 0.9 * rounded
    assert (Y - ref).abs().max() < 1e-12 * ref.abs().max()
