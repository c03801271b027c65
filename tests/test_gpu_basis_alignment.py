"""The Lanczos basis into a caller's buffer that is aligned to its doubles, not to its complex numbers."""
import numpy as np
import pytest
import torch

import oracle as O
from synth import dense_kmesh, make_problem, random_block

pytestmark = pytest.mark.gpu


def T(a, dt=torch.complex128):
    return torch.as_tensor(np.ascontiguousarray(a)).to(torch.device("cuda:0"), dt)


def test_basis_at_eight_bytes():
    from paper_2607_05853_amd import bse as B
    p = make_problem(dict(cfg_id=80, coarse=(2, 2, 2), dense=(3, 3, 2), n_ao=8, nv=2, nc=3, n_aux=12), 0, "G2")
    W = O.interpolate_W_matmul(p.W_R, p.R, p.w_R, dense_kmesh(p.nk))
    nb, m, om = 2, 6, np.linspace(1.0, 5.0, 7)
    plan = B.plan_from_problem(p, T(W), prec="f64", max_nb=nb)
    P = T(random_block(p.N, nb, seed=3))
    h = plan.haydock(P, m, om, 0.1, keep_basis=True)
    flat = torch.full((2 * nb * m * p.N + 2,), float("nan"), dtype=torch.float64, device="cuda:0")
    assert flat.data_ptr() % 16 == 0
    S, a, b = np.zeros((nb, 7)), np.zeros((nb, m)), np.zeros((nb, m + 1))
    steps = np.zeros(nb, dtype=np.int32)
    s = B.lib().bse_haydock_spectrum(plan._ptr, P.data_ptr(), nb, m, om.ctypes.data, 7, 0.1, S.ctypes.data, a.ctypes.data,
                                     b.ctypes.data, steps.ctypes.data, flat.data_ptr() + 8,
                                     torch.cuda.current_stream().cuda_stream)
    plan.close()
    assert s == 0
    assert np.array_equal(S, h["S"]) and np.array_equal(a, h["a"]) and np.array_equal(b, h["b"])
    assert torch.equal(torch.view_as_complex(flat[1:-1].clone().reshape(nb, m, p.N, 2)), h["basis"])
    assert torch.isnan(flat[0]) and torch.isnan(flat[-1])
