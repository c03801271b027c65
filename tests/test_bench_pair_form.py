"""bench.py times the pair form its operation count stands for: plans created inside bench.pair_form() form pairs."""
import os
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402


def test_environment_is_given_back(monkeypatch):
    monkeypatch.delenv("BSE_LATTICE", raising=False)
    with bench.pair_form():
        assert os.environ["BSE_LATTICE"] == "0"
    assert "BSE_LATTICE" not in os.environ
    monkeypatch.setenv("BSE_LATTICE", "contract")
    with pytest.raises(RuntimeError):
        with bench.pair_form():
            assert os.environ["BSE_LATTICE"] == "0"
            raise RuntimeError
    assert os.environ["BSE_LATTICE"] == "contract"


@pytest.mark.gpu
def test_plans_inside_form_pairs():
    import torch
    import oracle as O
    from paper_2607_05853_amd import bse as B
    from synth import dense_kmesh, make_problem
    p = make_problem(dict(cfg_id=94, coarse=(2, 2, 2), dense=(4, 4, 4), n_ao=8, nv=2, nc=2, n_aux=16), 0, "G2")
    W = torch.as_tensor(np.ascontiguousarray(O.interpolate_W_matmul(p.W_R, p.R, p.w_R, dense_kmesh(p.nk)))).to("cuda:0")
    n = []
    for inside in (True, False):
        if inside:
            with bench.pair_form():
                plan = B.plan_from_problem(p, W, prec="f64", max_nb=2)
        else:
            plan = B.plan_from_problem(p, W, prec="f64", max_nb=2)
        n.append(plan.lattice())
        plan.close()
    assert n[0] == 0 < n[1]
