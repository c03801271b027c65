"""The separable Fourier sums over flat and uneven boxes of R: every size of the last two axes that has a kernel of its own,
few q1 (whose q2 are shared between rows of threads) and every tile width, against the oracle's direct sums.  FP64 bound
1e-12 of the largest element, as for the other separable sums."""
import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu


def T(a, dt=torch.complex128):
    return torch.as_tensor(np.ascontiguousarray(a)).to(torch.device("cuda:0"), dt)


def rel(a, b):
    return np.abs(a - b).max() / np.abs(b).max()


def grid(axes):
    return np.stack(np.meshgrid(*axes, indexing="ij"), -1).reshape(-1, 3)


def box(*r):
    return grid([np.arange(-(m // 2), m - m // 2) for m in r]).astype(np.int32)


# q, R, N_aux: R2 x R3 of 1 .. 7 each; then N_aux 182 (33124 elements: 32 a tile) to 350 (122500: 64 to 256 a tile) with
# one to four q1, an odd number of q2 (a part without a second one), nine q1 (one round of 16) and more than a round
CASES = [((3, 5, 4), (2, y, z), 6) for y in (1, 2, 3, 4, 5, 6, 7) for z in (1, 3, 4, 7)]
CASES += [((1, 9, 2), (1, 5, 2), 350), ((1, 3, 1), (1, 2, 1), 350), ((2, 7, 1), (2, 7, 1), 350), ((3, 4, 2), (3, 1, 2), 182),
          ((4, 5, 3), (3, 5, 1), 182), ((9, 2, 3), (5, 1, 3), 182), ((17, 3, 1), (7, 3, 1), 182), ((1, 24, 1), (1, 7, 1), 9),
          ((1, 1, 1), (1, 1, 1), 350), ((1, 2, 8), (1, 2, 7), 350), ((2, 1, 3), (2, 1, 3), 350), ((5, 1, 6), (3, 1, 5), 20)]


@pytest.mark.parametrize("n,r,na", CASES)
def test_boxes(n, r, na):
    from paper_2607_05853_amd import bse as B
    q, R = grid([np.arange(m) / m for m in n]), box(*r)
    rng = np.random.default_rng(sum(n) + 10 * sum(r))
    w = rng.random(len(R))
    W = rng.standard_normal((len(R), na, na)) + 1j * rng.standard_normal((len(R), na, na))
    e = [rel(B.interpolate_W(T(W), R, w, q).cpu().numpy(), O.interpolate_W_matmul(W, R, w, q))]
    g = rng.standard_normal((len(q), na, na)) + 1j * rng.standard_normal((len(q), na, na))
    back = B.interpolate_W_adjoint(T(g), R, w, q)
    ph = np.exp(-2j * np.pi * (R @ q.T))
    e.append(rel(back.cpu().numpy(), (w[:, None] * (ph @ g.reshape(len(q), -1))).reshape(len(R), na, na)))
    print("[boxes %s on %s, N_aux %d] %.1e %.1e" % (n, r, na, *e), flush=True)
    assert max(e) < 1e-12
    assert torch.equal(back, B.interpolate_W_adjoint(T(g), R, w, q))
