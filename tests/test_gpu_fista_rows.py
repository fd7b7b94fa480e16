"""FISTA where the objective has more rows than the acceptance test adds by itself
(2048): one iteration against the FP64 reference; decisions are compared where the
sufficient-decrease slack exceeds the objective's FP32 error, points and objective
at the tolerances of tests/test_gpu_fista.py."""
import numpy as np
import pytest

import workloads
from gpu_cases import var_scale
from oracle import fista as ofista

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("pull", ["off", "le3"])
def test_many_objective_rows(pull):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_15020_amd as ffs
    inst = workloads.random_hybrid(400, 5, n_or=17000, or_len=(3, 5), n_card=5, card_len=(8, 40))
    B, eta0 = 12, 0.2
    plan = ffs.Plan(ffs.Problem(inst), B, pull=pull)
    assert sum(-(-b["count"] // b["cpw"]) for b in plan.describe()["bins"]["f32"]) > 2048
    x = torch.from_numpy(workloads.points(inst.n_vars, B, 77)).to(DEV)
    st = plan.fista_state(x, eta0)
    S = var_scale(inst)[:, None]
    fscale = float(inst.m)
    f64 = lambda t: t.detach().cpu().numpy().astype(np.float64)   # noqa: E731
    compared = 0
    for it in range(3):
        xs, ys, es, ts = f64(x), f64(st["y"]), f64(st["eta"]), f64(st["t"])
        F = torch.full((B,), float("nan"), device=DEV)
        plan.fista(x, st, 1, max_ls=15, F=F)
        ox, oy, oe, ot, _, OFx, _, margin = ofista.iterate(inst, xs, ys, es, ts)
        c = margin > 1e-4 * fscale
        assert np.array_equal(f64(st["eta"])[c], oe[c])
        tol = 2e-5 * np.maximum(1.0, oe[c][None, :] * S)
        assert np.all(np.abs(f64(x)[:, c] - ox[:, c]) <= tol) and np.all(np.abs(f64(st["y"])[:, c] - oy[:, c]) <= 2 * tol)
        assert np.all(np.abs(f64(F)[c] - OFx[c]) <= 1e-5 * fscale)
        compared += int(c.sum())
    assert compared >= 2 * B
