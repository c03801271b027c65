"""The separable Fourier sums (product grids of q, R in a small box) at the edges of their rule, and the lists
just outside it that take the phase table, against the oracle's direct sums.  FP64 bound 1e-12 of the largest
element: a sum of at most 4096 products of order one rounds to well below it."""
import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu


def T(a, dt=torch.complex128):
    return torch.as_tensor(np.ascontiguousarray(a)).to(torch.device("cuda:0"), dt)


def rel(a, b):
    return np.abs(a - b).max() / np.abs(b).max()


def box(*r):
    return np.stack(np.meshgrid(*[np.arange(-(m // 2), m - m // 2) for m in r], indexing="ij"), -1).reshape(-1, 3)


def grid(axes):
    return np.stack(np.meshgrid(*axes, indexing="ij"), -1).reshape(-1, 3)


def uniform(*n):
    return grid([np.arange(m) / m for m in n])


SPHERE = [r for r in box(7, 7, 7) if (r ** 2).sum() <= 9]  # 123 vectors, gaps in the box
rng0 = np.random.default_rng(3)
CASES = {
    "one q, one R": (uniform(1, 1, 1), [[0, 0, 0]], 3),
    "one element per matrix": (uniform(4, 3, 2), box(3, 3, 3), 1),
    "8 8 8 on 5 5 5": (uniform(8, 8, 8), box(5, 5, 5), 17),
    "sphere, odd grid": (uniform(9, 5, 7), SPHERE, 12),
    "more q1 than a round": (uniform(17, 2, 3), box(7, 1, 2), 20),
    "longest axis": (uniform(24, 1, 1), box(7, 3, 1), 9),
    "longest last axis": (uniform(1, 1, 24), box(1, 2, 7), 9),
    "uneven axes": (grid([rng0.random(5), rng0.random(4), rng0.random(6)]), box(4, 5, 6)[rng0.permutation(120)], 130),
    "most R": (uniform(5, 3, 4), box(7, 7, 7)[:256], 6),
    "axis too long": (uniform(25, 1, 1), box(3, 1, 1), 5),
    "too many R": (uniform(3, 3, 3), box(7, 7, 7), 5),
    "box too wide": (uniform(3, 3, 3), [[i, 0, 0] for i in range(8)], 5),
    "R listed twice": (uniform(4, 4, 4), [[0, 0, 0], [1, 0, 0], [1, 0, 0]], 5),
    "not a grid": (rng0.random((30, 3)), box(3, 3, 3), 5),
    "almost a grid": (np.vstack([uniform(4, 4, 4)[:-1], [[0.75, 0.75, 0.7]]]), box(3, 3, 3), 5),
}


@pytest.mark.parametrize("name", list(CASES))
def test_fourier_sums_match_direct_sums(name):
    from paper_2607_05853_amd import bse as B
    q, R, na = CASES[name]
    R = np.asarray(R, dtype=np.int32)
    rng = np.random.default_rng(len(q))
    w = rng.random(len(R))
    W = rng.standard_normal((len(R), na, na)) + 1j * rng.standard_normal((len(R), na, na))
    ref = O.interpolate_W(W, R, w, q)
    got = B.interpolate_W(T(W), R, w, q).cpu().numpy()
    got32 = B.interpolate_W(T(W), R, w, q, out_prec="f32").cpu().numpy()
    print("[fourier] %s: %.1e" % (name, rel(got, ref)), flush=True)
    assert rel(got, ref) < 1e-12
    assert rel(got32, ref) < 1e-6
    out = torch.full((len(q), na, na), float("nan"), dtype=torch.complex128, device="cuda:0")
    B.interpolate_W_noalloc(T(W), R, w, q, out)
    assert rel(out.cpu().numpy(), ref) < 1e-12
    g = rng.standard_normal((len(q), na, na)) + 1j * rng.standard_normal((len(q), na, na))
    back = B.interpolate_W_adjoint(T(g), R, w, q).cpu().numpy()
    assert rel(back, O.grad_WR_from_Wq(g, R, w, q)) < 1e-12
