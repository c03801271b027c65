"""The Lanczos recurrence at the sizes where its launches change (apply block read in place or gathered, shared sums over
the basis, partial norms summed by their own launch), against the same recurrence in numpy on the plan's own applies:
coefficients and basis to the rounding of FP64 sums of N terms (1e-12 of the operator's scale)."""
import numpy as np
import pytest
import torch

import oracle as O
from synth import dense_kmesh, make_problem, random_block

pytestmark = pytest.mark.gpu


def T(a, dt=torch.complex128):
    return torch.as_tensor(np.ascontiguousarray(a)).to(torch.device("cuda:0"), dt)


# dense, nv, nc, nb: N = 24; 8190 (in place at one vector, gathered at three); 8196; 8640; 36864
CASES = [((3, 2, 2), 1, 2, 3), ((13, 9, 7), 2, 5, 1), ((13, 9, 7), 2, 5, 3), ((13, 9, 7), 2, 6, 2), ((16, 16, 16), 3, 3, 2)]


@pytest.mark.parametrize("dense,nv,nc,nb", CASES)
def test_recurrence(dense, nv, nc, nb):
    from paper_2607_05853_amd import bse as B
    p = make_problem(dict(cfg_id=80, coarse=(2, 2, 2), dense=dense, n_ao=2 * nc, nv=nv, nc=nc, n_aux=4), 0, "G2")
    W = B.interpolate_W(T(p.W_R), p.R, p.w_R, dense_kmesh(p.nk))
    plan = B.plan_from_problem(p, W, prec="f64", max_nb=nb)
    P = random_block(p.N, nb, seed=3) * 7.0
    m = 8
    h = plan.haydock(T(P), m, np.linspace(1, 5, 3), 0.1, keep_basis=True)
    a, b = np.zeros((nb, m)), np.zeros((nb, m + 1))
    b[:, 0] = np.linalg.norm(P, axis=0)
    q = P / b[:, 0]
    basis = []
    for j in range(m):
        basis.append(q)
        w = plan.apply(T(q)).cpu().numpy()
        a[:, j] = np.einsum("ib,ib->b", q.conj(), w).real
        for _ in range(2):
            for i in range(nb):
                Q = np.stack([x[:, i] for x in basis], 1)
                w[:, i] -= Q @ (Q.conj().T @ w[:, i])
        b[:, j + 1] = np.linalg.norm(w, axis=0)
        q = w / b[:, j + 1]
    plan.close()
    scale = np.abs(a).max()
    e = [np.abs(h["a"] - a).max() / scale, np.abs(h["b"] - b).max() / max(scale, 7.0),
         np.abs(h["basis"].cpu().numpy() - np.stack(basis).transpose(2, 0, 1)).max()]
    print("[recurrence N %d nb %d] a %.1e b %.1e basis %.1e" % (p.N, nb, *e), flush=True)
    assert max(e) < 1e-12
    assert (h["steps"] == m).all() and not h["breakdown"]
